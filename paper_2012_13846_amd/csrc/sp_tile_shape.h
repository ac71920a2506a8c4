// How gather_tile_kernel cuts a layer, and where it finds the weights: arithmetic that the host and the kernel share.
// No device code and no other header, so that a test on the CPU can check every address.
#pragma once

#include <cstddef>
#include <cstdint>

#ifdef __HIPCC__
#define SP_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define SP_HOST_DEVICE inline
#endif

namespace sp {

// KC contraction channels a slice, NCS * 16 destination channels a workgroup.
struct TileShape {
    int kc, ncs, nsl, ny;
};
constexpr int kBigNcs = 4;  // NCS of the BIG kernels; their KC is 32 or 64

// Slices of the contraction and channel tiles of gather_tile_kernel: the cut with the least padding, where a further
// slice (another accumulator update per link) or channel tile (the rows are gathered again) counts as 8 more padded
// channels (80 fp32 channels: 2 x 48 measured faster than 5 x 16).
inline TileShape tile_shape(int cc, int co, bool is_f32, bool big) {
    TileShape t{0, 0, 0, 0};
    if (big) {
        t.kc = cc <= 32 ? 32 : 64;
        t.nsl = (cc + t.kc - 1) / t.kc;
        t.ncs = kBigNcs;
        t.ny = (co + 16 * kBigNcs - 1) / (16 * kBigNcs);
        return t;
    }
    const int kcs[] = {64, 48, 32, 16}, ncss[] = {8, 4, 3, 2, 1};
    int best = 1 << 30;
    for (int kc : kcs) {
        if (!is_f32 && kc % 32) continue;
        const int n = (cc + kc - 1) / kc, cost = n * kc + 8 * (n - 1);
        if (cost < best) {
            best = cost;
            t.kc = kc;
            t.nsl = n;
        }
    }
    best = 1 << 30;
    for (int n : ncss) {
        const int ny = (co + 16 * n - 1) / (16 * n), cost = ny * 16 * n + 8 * (ny - 1);
        if (cost < best) {
            best = cost;
            t.ncs = n;
            t.ny = ny;
        }
    }
    return t;
}

// Where the weights are: byte offset of offset k, channel tile y, 16-channel group cs, slice, fragment s of a unit, and
// of lane n16 + 16 * g in it.
struct TileWeights {
    uint32_t bytes;     // the whole of them
    int channels;       // destination channels they have (copy: rounded up to whole channel tiles)
    uint32_t k, y, cs, slice, s, n16, g;
};

inline uint64_t tile_copy_bytes(const TileShape& t, int kvol, int elt) {
    return (uint64_t)kvol * t.ny * t.ncs * 16 * t.nsl * t.kc * elt;
}

// Fragment-major copy [k][channel tile][cs][slice][fragment][lane][16 bytes], zeros beyond the real channels.
inline TileWeights tile_weights_copied(const TileShape& t, int kvol, int elt) {
    TileWeights w{};
    const int groups = t.kc * elt / 64;
    w.bytes = (uint32_t)tile_copy_bytes(t, kvol, elt);
    w.channels = t.ny * t.ncs * 16;
    w.s = 1024;
    w.slice = (uint32_t)groups * w.s;
    w.cs = (uint32_t)t.nsl * w.slice;
    w.y = (uint32_t)t.ncs * w.cs;
    w.k = (uint32_t)t.ny * w.y;
    w.n16 = 16;
    w.g = 256;
    return w;
}

// The weights as the caller stores them, [kvol][co][cc]: cc has to be whole slices.
inline bool tile_in_place_ok(const TileShape& t, int cc) { return cc % t.kc == 0; }
inline TileWeights tile_weights_in_place(const TileShape& t, int kvol, int cc, int co, int elt) {
    TileWeights w{};
    w.bytes = (uint32_t)((uint64_t)kvol * cc * co * elt);
    w.channels = co;
    w.s = 64;
    w.slice = (uint32_t)(t.kc * elt);
    w.n16 = (uint32_t)(cc * elt);
    w.cs = 16 * w.n16;
    w.y = (uint32_t)t.ncs * w.cs;
    w.k = (uint32_t)co * w.n16;
    w.g = 16;
    return w;
}

// What channel tile y, group cs and the lane add to a fragment's address: *uniform in every lane, *lane in this one.
// Channels that the weights do not have (their products are dropped) read the last one there is: the uniform part of
// a buffer address is not checked against the buffer's end.
SP_HOST_DEVICE void tile_weight_at(const TileWeights& w, int ncs, int y, int cs, int n16, int g, uint32_t* uniform, uint32_t* lane) {
    int c0 = (y * ncs + cs) * 16;
    *uniform = (uint32_t)y * w.y + (uint32_t)cs * w.cs;
    if (c0 >= w.channels) {
        c0 = 0;
        *uniform = 0;
    }
    const int last = w.channels - 1 - c0;
    *lane = (uint32_t)(n16 < last ? n16 : last) * w.n16 + (uint32_t)g * w.g;
}

}  // namespace sp
