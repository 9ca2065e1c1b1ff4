// Which buffer the pinned pool hands out and which it keeps; exit status 0 if
// all is as expected, else the line that failed.
#include "pinned_pool.h"

#include <cstdint>
#include <cstdio>

#define EXPECT(c)                                  \
    do {                                           \
        if (!(c)) {                                \
            std::printf("line %d: %s\n", __LINE__, #c); \
            return 1;                              \
        }                                          \
    } while (0)

using mcl::PinnedBuffer;
using mcl::PinnedPool;

static PinnedBuffer make(uintptr_t id, size_t bytes, int device = 0)
{
    PinnedBuffer b;
    b.host = (void*)id;
    b.bytes = bytes;
    b.device = device;
    return b;
}

int main()
{
    const size_t K = 1024, M = K * K;
    PinnedPool p;
    PinnedBuffer b;
    EXPECT(!p.take(1, 0, b));
    // the smallest that fits, whatever the order they came back in
    EXPECT(p.give(make(1, 4 * M)).host == nullptr);
    EXPECT(p.give(make(2, 64 * K)).host == nullptr);
    EXPECT(p.give(make(3, 256 * K)).host == nullptr);
    EXPECT(p.take(1000, 0, b) && b.host == (void*)2);
    EXPECT(p.take(65 * K, 0, b) && b.host == (void*)3);
    EXPECT(p.take(4 * M, 0, b) && b.host == (void*)1);
    EXPECT(!p.take(1, 0, b));
    // another device's buffer is not handed out
    EXPECT(p.give(make(4, 64 * K, 1)).host == nullptr);
    EXPECT(!p.take(1, 0, b));
    EXPECT(p.take(1, 1, b) && b.host == (void*)4 && b.device == 1);
    // too large to keep
    EXPECT(p.give(make(5, PinnedPool::kMost + 1)).host == (void*)5);
    // a pool full of small buffers makes room for large ones, smallest first,
    // and the ones it lets go come back to be freed
    for (int i = 0; i < PinnedPool::kKept; ++i) EXPECT(p.give(make(10 + i, (64 + i) * K)).host == nullptr);
    EXPECT(p.give(make(30, 4 * M)).host == (void*)10);
    EXPECT(p.give(make(31, 4 * M)).host == (void*)11);
    EXPECT(p.give(make(32, 66 * K)).host == (void*)32);         // no larger than the smallest kept
    EXPECT(p.take(4 * M, 0, b) && b.bytes == 4 * M);
    EXPECT(p.take(4 * M, 0, b) && b.bytes == 4 * M);
    EXPECT(!p.take(4 * M, 0, b));
    EXPECT(p.take(1, 0, b) && b.host == (void*)12);
    return 0;
}
