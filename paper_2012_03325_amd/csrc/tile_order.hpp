// Launch order: which work items the workgroups of each XCD take.  The dispatcher
// hands workgroup b to XCD b % 8, and each XCD has its own L2, so consecutive items
// should go to the same XCD; but items of an image cost unequally (sky, ground), so
// every XCD also has to get its share of the costly ones.
#pragma once

#include <hip/hip_runtime.h>

namespace epb {

constexpr int kNumXcd = 8;  // MI355X: 256 CUs in 8 accelerator complex dies

// XCD x's contiguous share of `total` items: with one workgroup per item a bijection
// for any total.  A batch of small views takes it in every stage: an XCD gets whole
// views, or runs of views, and with them the cheap and the costly parts.
struct XcdShare {
    int first, count;
};
__host__ __device__ inline XcdShare xcd_share(int x, int total) {
    int q = total / kNumXcd, r = total % kNumXcd;
    return XcdShare{x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q, q + (x < r ? 1 : 0)};
}

// The same as the item of workgroup b of nb.
__host__ __device__ inline int xcd_tile(int b, int nb) {
    int q = nb / kNumXcd, r = nb % kNumXcd;
    int x = b % kNumXcd, local = b / kNumXcd;
    return x < r ? x * (q + 1) + local : r * (q + 1) + (x - r) * q + local;
}

// The shading pass's order for one view, and for a batch with large views: chunks of
// kShadeChunk consecutive tiles go to the XCDs in turn, so that every XCD gets its share
// of the costly rows (a contiguous eighth of the image leaves the XCDs of the sky
// idle) while neighbouring tiles still share an L2; what does not fill a round of
// chunks is split as above.  An XCD's chunk moves on by one every second round and every
// eighth: at one place in every round, an image whose rows fill 512 tiles a whole number of
// times (4096 pixels wide, 8192, 16384) would give an XCD the same columns all the way down
// (4096x1024 with only sky in its right half: 74 us so, 52 with the shift, 53 with contiguous
// shares).  A larger shift changes images of two rounds, which have nothing to gain
// (512x512 in half storage 10.0 us, with one a round 10.4).
// Tile `it` of XCD x (0 <= it < xcd_share(x, total).count):
constexpr int kShadeChunk = 64;
__host__ __device__ inline int xcd_chunk_item(int x, int it, int total) {
    int rounds = total / (kNumXcd * kShadeChunk), round = it / kShadeChunk;
    if (round < rounds) {
        int chunk = (x + (round >> 1) + (round >> 3)) % kNumXcd;
        return (round * kNumXcd + chunk) * kShadeChunk + it % kShadeChunk;
    }
    int first = rounds * (kNumXcd * kShadeChunk);
    return first + xcd_share(x, total - first).first + (it - rounds * kShadeChunk);
}

// Whether a batch's shading takes that order (largest: tiles of its largest view).  Not with
// views of up to eight rounds: chunks are then too few to share a view out evenly, and a view
// of 256 or 512 tiles gives an XCD the same part of every view (without the shift above 256 views of
// 256x256 in half storage 397 us, float32 451; with it 320 and 376; by contiguous shares 316 and
// 371; 8 of 320x240 45.4 / 41.8).  With larger views a contiguous share is a part of one view, the
// sky or the ground (8 of 1920x1080 in float32 532 us, 507 in chunks; 13 of up to 1920x1080 431 /
// 422; 12 of 1280x720, 3600 tiles, equal).  Not with grids that loop over the tiles either, where
// contiguous shares are ahead at every size (16 views of up to 1920x1080, half storage, 8 / 16 / 32
// workgroups per CU: chunks 479 / 466 / 447 us, shares 437 / 388 / 378).
inline bool shade_in_chunks(long long largest, bool looping) {
    return !looping && largest > 8LL * kNumXcd * kShadeChunk;
}

}  // namespace epb
