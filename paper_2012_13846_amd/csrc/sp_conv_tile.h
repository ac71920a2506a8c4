// Link-list gather-GEMM (Eq. 2 and its input gradient) for any channel counts: the kernel template and its
// launcher, instantiated per storage type in sp_conv_tile_f32.hip / sp_conv_tile_bf16.hip.
//
// A workgroup owns a tile of TR destination rows and 16 * NCS destination channels.  Its links, offset by offset,
// are cut into blocks of up to 16 links of one offset; a block times one KC-wide slice of the contraction is a
// unit, and SB units make a step.
//   - Producer wavefronts fetch.  They walk the units, gather the source rows' slices (16-byte pieces, a row's
//     pieces on adjacent lanes) kD steps ahead into registers and store them to one of two LDS buffers.
//   - Consumer wavefronts multiply.  Wavefront (cs, bs) owns channels cs*16 .. +15 of the slice and every NBS-th
//     unit: it reads the unit's rows as MFMA B fragments, takes the offset's weights (A operand, from a
//     fragment-major copy, one unit ahead in registers) and adds the transposed product (a lane holds 4 channels of
//     ONE link) to the link's destination row of its LDS accumulator, one unit later.
// One barrier per step.  Loads of one wavefront return in order, so a wavefront that fetches both rows (fabric
// latency) and weights (L2 latency) waits for the rows whenever it needs weights; split between wavefronts the two
// streams do not wait for each other.  The rows are gathered once for all 16 * NCS channels and a unit's weights
// are read once per TR rows, where a wavefront on its own (gather_wave_kernel) reads them for 64 rows.
// What bounds it: the matrix pipes (fp32) together with what does not overlap them; about 55 % of the time is MFMA.
// Measured, before (a workgroup-cooperative kernel without prefetch, or one thread per output) and now: fp32
// 128 -> 128 on 0.66 M links 815 -> 440 us (49 TFLOP/s of 157), 48 -> 48 on 0.61 M links 4200 -> 80 us, 80 -> 40
// 5900 -> 145 us, bf16 20 -> 24 405 -> 40 us.  128-row tiles against 64-row tiles: 440 against 550 us at 128 -> 128.
// A destination row belongs to one workgroup and occurs at most once per unit; with NBS > 1 every bs has its own
// accumulator and they are added in order at the end: no atomics, fixed order, reproducible.
#pragma once

#include <mutex>
#include <type_traits>

#include "sp_internal.h"
#include "sp_tile_shape.h"

namespace sp {

struct TileArgs {
    const int32_t* off;  // the side's lists (MapSide)
    const int32_t* src;
    const int32_t* dst;
    const void* f;   // source features [n_src][cc]
    const void* w;   // weights
    void* g;         // destination features [n_rows][co]
    int64_t n_rows;
    int kvol, co, flip;
    int big;                 // features or lists beyond 32-bit byte offsets: the BIG kernels
    int nsl;                 // slices of KC contraction channels
    int max_blk;             // room for block descriptors
    uint32_t row_bytes;      // one source row
    uint32_t f_bytes, list_bytes;  // buffer sizes: f, src and dst
    TileWeights wt;          // where w's elements are
};

template <typename T, int KC, int NCS, int TR>
struct TileCfg {
    static constexpr bool kIsF32 = std::is_same<T, float>::value;
    static constexpr int kGroup = kIsF32 ? 16 : 32;      // contraction channels of one 16-byte fragment
    static constexpr int kGroups = KC / kGroup;
    static constexpr int kNBS = NCS == 1 ? 4 : (NCS == 2 ? 2 : 1);
    static constexpr int kSB = 4 * (kNBS > 2 ? 2 : 1);   // units per step
    static constexpr int kUPW = kSB / kNBS;              // units of one consumer wavefront per step
    static constexpr int kRow = KC * (int)sizeof(T);     // bytes of one source row's slice
    static constexpr int kP = kRow / 16;                 // its 16-byte pieces
    static constexpr int kPitch = kRow + 32;             // staged row: b128 fragment reads at the full LDS rate
    static constexpr int kNP = kSB * 16 * kP >= 512 ? 2 : 1;  // producer wavefronts
    static constexpr int kPT = 64 * kNP;
    static constexpr int kL = kSB * 16 * kP / kPT;       // pieces per producer thread and step
    static constexpr int kD = 2;                         // steps whose rows are in flight
    static constexpr int kCW = NCS * kNBS;               // consumer wavefronts
    static constexpr int kThreads = 64 * (kCW + kNP);
    static constexpr int kCOT = 16 * NCS;
    static constexpr int kAccStride = kCOT + 4;          // floats
    static constexpr int kAccBytes = kNBS * (TR + 1) * kAccStride * 4;  // row TR takes the updates of links that do not exist
    static constexpr int kBuf = kSB * 16 * kPitch;
    static constexpr int kRowIdx = 2 * kSB * 16 * 4;     // destination rows (as accumulator offsets) of two steps
    static constexpr int kWoff = 4 * kSB * 4;            // weight offsets of four steps
    static constexpr int kFixed = kAccBytes + 2 * kBuf + kRowIdx + kWoff;
    static_assert(KC % kGroup == 0 && (kSB * 16 * kP) % kPT == 0 && kSB % kNBS == 0 && kUPW % 2 == 0, "whole loads, even units");
    static_assert(TR == 64 || TR == 128, "one or two sub-tiles");
};

// BIG: 64-bit addresses for features and lists (rows of whole 16-byte pieces).  A kernel of its own, and for one cut of
// the channels, because a choice inside the loop slows every launch: at the join the
// loads of both branches have to have come back (fp32 128 -> 128 under the profiler, 0.66 M links: 614 us).
template <typename T, int KC, int NCS, int TR, bool BIG>
__global__ __launch_bounds__((TileCfg<T, KC, NCS, TR>::kThreads)) void gather_tile_kernel(TileArgs a) {
    using Cfg = TileCfg<T, KC, NCS, TR>;
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    constexpr bool kIsF32 = Cfg::kIsF32;
    using Frag = typename std::conditional<kIsF32, f32x4, bf16x8>::type;
    constexpr int kSB = Cfg::kSB, kNBS = Cfg::kNBS, kGroups = Cfg::kGroups, kP = Cfg::kP, kNSub = TR / 64;
    constexpr uint32_t kOutside = 0xffffff00u;  // every buffer ends before it: loads from here return zeros

    extern __shared__ __align__(16) unsigned char smem[];
    float* acc = reinterpret_cast<float*>(smem);
    unsigned char* xbuf = smem + Cfg::kAccBytes;
    int* s_row = reinterpret_cast<int*>(xbuf + 2 * Cfg::kBuf);
    int* s_woff = s_row + 2 * kSB * 16;
    int4* s_blk = reinterpret_cast<int4*>(smem + Cfg::kFixed);
    __shared__ int s_nblk;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t tile = blockIdx.x;
    const int kvol = a.kvol;

    // ---- block descriptors {offset | links << 8, first link of sub-tile 0's part, of sub-tile 1's part, length of
    // sub-tile 0's part}: block i of offset k holds links 16 i .. of the sub-tiles' stretches put end to end
    if (wave == 0) {
        int base = 0;
        for (int kb = 0; kb < kvol; kb += 64) {
            const int k = kb + lane;
            int o0 = 0, l0 = 0, o1 = 0, l1 = 0;
            if (k < kvol) {
                const int32_t* p = a.off + ((tile * kNSub) * kvol + k) * kHalves;
                o0 = p[0];
                o1 = p[kvol * kHalves];  // the next sub-tile's begin: this one's end
                l0 = o1 - o0;
                if (kNSub == 2) l1 = p[2 * kvol * kHalves] - o1;
            }
            const int cnt = l0 + l1, nb = (cnt + 15) >> 4;
            int inc = nb;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int t = __shfl_up(inc, d, 64);
                if (lane >= d) inc += t;
            }
            const int ex = base + inc - nb;
            for (int i = 0; i < nb; ++i)
                s_blk[ex + i] = int4{k | (min(16, cnt - 16 * i) << 8), o0 + 16 * i, o1 + 16 * i - l0, l0 - 16 * i};
            base += __shfl(inc, 63, 64);
        }
        if (lane == 0) s_nblk = base;
    } else {
        for (int i = tid - 64; i < Cfg::kAccBytes / 16; i += Cfg::kThreads - 64)
            reinterpret_cast<f32x4*>(acc)[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    __syncthreads();
    const int nblk = __builtin_amdgcn_readfirstlane(s_nblk);
    const int nsteps = (nblk * a.nsl + kSB - 1) / kSB;

    constexpr int kRsrcFlags = 0x00020000;
    if (wave >= Cfg::kCW) {
        // ---------------------------------------------------------------- producers
        const __amdgpu_buffer_rsrc_t rF = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.f), 0, (int)a.f_bytes, kRsrcFlags);
        const __amdgpu_buffer_rsrc_t rSrc =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(a.src), 0, (int)a.list_bytes, kRsrcFlags);
        const __amdgpu_buffer_rsrc_t rRow =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(a.dst), 0, (int)a.list_bytes, kRsrcFlags);
        constexpr int kEN = kSB * 16 / 64;  // links of a step per lane (every producer wavefront looks at all of them)
        const int pt = tid - 64 * Cfg::kCW;
        struct Ent {
            int src[kEN];       // source row of link 64 e + lane of the step, in flight
            uint32_t add[kEN];  // byte offset of the slice inside the row, or kOutside: no such link
        };
        struct Rows {
            u32x4 x[Cfg::kL];
            int row[kEN];       // destination row (accumulator offset) of this lane's links
        };
        Ent ent[2] = {};
        Rows rows[Cfg::kD] = {};
        struct Link {
            uint32_t entry;
            uint32_t slice_off;
            bool live;
            int k_off;  // weight offset of the unit
        };
        auto link_of = [&](int step, int e) __attribute__((always_inline)) {
            const int lr = 64 * e + lane;
            const int unit = step * kSB + (lr >> 4);
            const int blk = a.nsl == 1 ? unit : unit / a.nsl, sl = a.nsl == 1 ? 0 : unit - blk * a.nsl;
            Link l;
            const int4 d = s_blk[min(blk, nblk - 1)];
            const int p = lr & 15;
            l.live = blk < nblk && p < (d.x >> 8);
            l.entry = (uint32_t)(p < d.w ? d.y + p : d.z + p);
            l.slice_off = (uint32_t)sl * Cfg::kRow;
            const int k = d.x & 255;
            l.k_off = (int)((uint32_t)(a.flip ? kvol - 1 - k : k) * a.wt.k + (uint32_t)sl * a.wt.slice);
            return l;
        };
        auto load_ent = [&](int step, Ent& en) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < kEN; ++e) {
                const Link l = link_of(step, e);
                if constexpr (BIG) en.src[e] = l.live ? a.src[l.entry] : 0;
                else en.src[e] = (int)__builtin_amdgcn_raw_buffer_load_b32(rSrc, l.live ? l.entry * 4u : kOutside, 0, 0);
                en.add[e] = l.live ? l.slice_off : kOutside;
            }
        };
        const bool vec = a.row_bytes % 16 == 0;
        auto issue = [&](int step, const Ent& en, Rows& r) __attribute__((always_inline)) {
            uint32_t off[kEN];
#pragma unroll
            for (int e = 0; e < kEN; ++e) {
                const Link l = link_of(step, e);
                if constexpr (BIG) r.row[e] = l.live ? a.dst[l.entry] : -1;
                else r.row[e] = (int)__builtin_amdgcn_raw_buffer_load_b32(rRow, l.live ? l.entry * 4u : kOutside, 0, 0);
                if (!l.live) r.row[e] = -1;
                off[e] = en.add[e] == kOutside ? kOutside : (uint32_t)en.src[e] * (BIG ? 1u : a.row_bytes);
            }
            const uint32_t left0 = a.row_bytes;
#pragma unroll
            for (int j = 0; j < Cfg::kL; ++j) {
                const int idx = j * Cfg::kPT + pt, lr = idx / kP, piece = idx % kP;
                // the link's row offset and slice, from the lane that looked the link up
                uint32_t o = 0, sl = 0;
#pragma unroll
                for (int e = 0; e < kEN; ++e) {
                    const uint32_t oo = (uint32_t)__shfl((int)off[e], lr & 63, 64), ss = (uint32_t)__shfl((int)en.add[e], lr & 63, 64);
                    if (kEN == 1 || (lr >> 6) == e) {
                        o = oo;
                        sl = ss;
                    }
                }
                const uint32_t at = sl + piece * 16;  // byte inside the row
                if constexpr (BIG) {  // o: the row's number
                    r.x[j] = u32x4{0u, 0u, 0u, 0u};
                    if (o != kOutside && at < left0)
                        r.x[j] = *reinterpret_cast<const u32x4*>(static_cast<const unsigned char*>(a.f) + (size_t)o * a.row_bytes + at);
                } else if (vec) {
                    r.x[j] = __builtin_amdgcn_raw_buffer_load_b128(rF, (o != kOutside && at < left0) ? o + at : kOutside, 0, 0);
                } else if (a.row_bytes % 4 == 0) {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        r.x[j][i] = __builtin_amdgcn_raw_buffer_load_b32(rF, (o != kOutside && at + 4 * i < left0) ? o + at + 4 * i : kOutside, 0, 0);
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint32_t b = at + 4 * i;
                        const uint32_t lo = __builtin_amdgcn_raw_buffer_load_b16(rF, (o != kOutside && b < left0) ? o + b : kOutside, 0, 0);
                        const uint32_t hi = __builtin_amdgcn_raw_buffer_load_b16(rF, (o != kOutside && b + 2 < left0) ? o + b + 2 : kOutside, 0, 0);
                        r.x[j][i] = (lo & 0xffffu) | (hi << 16);
                    }
                }
            }
        };
        auto store = [&](int step, const Rows& r) __attribute__((always_inline)) {
            unsigned char* b = xbuf + (step & 1) * Cfg::kBuf;
#pragma unroll
            for (int j = 0; j < Cfg::kL; ++j) {
                const int idx = j * Cfg::kPT + pt, lr = idx / kP, piece = idx % kP;
                *reinterpret_cast<u32x4*>(b + lr * Cfg::kPitch + piece * 16) = r.x[j];
            }
            if (pt < 64) {
#pragma unroll
                for (int e = 0; e < kEN; ++e)
                    s_row[(step & 1) * kSB * 16 + 64 * e + lane] = (r.row[e] < 0 ? TR : (r.row[e] & (TR - 1))) * Cfg::kAccStride;
            }
        };
        auto store_woff = [&](int step) __attribute__((always_inline)) {
            if (pt < 64) {
#pragma unroll
                for (int e = 0; e < kEN; ++e) {
                    const Link l = link_of(step, e);
                    if ((lane & 15) == 0) s_woff[(step & 3) * kSB + 4 * e + (lane >> 4)] = l.k_off;
                }
            }
        };
        if (nsteps > 0) {
            load_ent(0, ent[0]);
            load_ent(1, ent[1]);
            store_woff(0);
            store_woff(1);
            issue(0, ent[0], rows[0]);
            load_ent(2, ent[0]);
            issue(1, ent[1], rows[1]);
            load_ent(3, ent[1]);
            store(0, rows[0]);
            // iteration s: store step s + 1 (in rows[(s + 1) % 2]) while step s is multiplied, request step s + 2's
            // rows with the entries requested two iterations ago, and the entries of step s + 4
            issue(2, ent[0], rows[0]);
            load_ent(4, ent[0]);
            __syncthreads();
            for (int s = 0; s < nsteps; s += 2) {
                store(s + 1, rows[1]);
                store_woff(s + 2);
                issue(s + 3, ent[1], rows[1]);
                load_ent(s + 5, ent[1]);
                __syncthreads();
                if (s + 1 >= nsteps) break;
                store(s + 2, rows[0]);
                store_woff(s + 3);
                issue(s + 4, ent[0], rows[0]);
                load_ent(s + 6, ent[0]);
                __syncthreads();
            }
        }
    } else {
        // ---------------------------------------------------------------- consumers
        const __amdgpu_buffer_rsrc_t rW = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.w), 0, (int)a.wt.bytes, kRsrcFlags);
        const int n16 = lane & 15, g = lane >> 4;
        const int cs = wave % NCS, bs = wave / NCS;
        uint32_t w_base, w_lane;
        tile_weight_at(a.wt, NCS, (int)blockIdx.y, cs, n16, g, &w_base, &w_lane);
        float* my_acc = acc + bs * (TR + 1) * Cfg::kAccStride + cs * 16 + g * 4;
        auto load_w = [&](Frag (&w)[kGroups], int woff) __attribute__((always_inline)) {
            const uint32_t so = (uint32_t)__builtin_amdgcn_readfirstlane(woff) + w_base;
#pragma unroll
            for (int s = 0; s < kGroups; ++s)
                w[s] = __builtin_bit_cast(Frag, __builtin_amdgcn_raw_buffer_load_b128(rW, w_lane, (int)(so + s * a.wt.s), 0));
        };
        constexpr int kUPW = Cfg::kUPW;
        constexpr int kChains = kIsF32 ? 2 : 1;  // independent MFMA chains per unit
        if (nsteps > 0) {
            Frag w[2][kGroups], xf[2][kGroups];
            f32x4 d[kChains];
#pragma unroll
            for (int c = 0; c < kChains; ++c) d[c] = f32x4{0.f, 0.f, 0.f, 0.f};
            float* dst = my_acc + TR * Cfg::kAccStride;  // the previous unit's destination rows (none yet)
            __syncthreads();
            load_w(w[0], s_woff[bs]);
            for (int s = 0; s < nsteps; ++s) {
                const unsigned char* b = xbuf + (s & 1) * Cfg::kBuf + (bs * 16 + n16) * Cfg::kPitch + g * 16;
                int rows[kUPW], wo[kUPW];
#pragma unroll
                for (int u = 0; u < kUPW; ++u) {
                    rows[u] = s_row[(s & 1) * kSB * 16 + (u * kNBS + bs) * 16 + n16];
                    wo[u] = u + 1 < kUPW ? s_woff[(s & 3) * kSB + (u + 1) * kNBS + bs] : s_woff[((s + 1) & 3) * kSB + bs];
                }
#pragma unroll
                for (int t = 0; t < kGroups; ++t) xf[0][t] = *reinterpret_cast<const Frag*>(b + t * 64);
#pragma unroll
                for (int u = 0; u < kUPW; ++u) {
                    load_w(w[(u + 1) & 1], wo[u]);
                    const f32x4 av = *reinterpret_cast<const f32x4*>(dst);
                    if (u + 1 < kUPW) {
#pragma unroll
                        for (int t = 0; t < kGroups; ++t)
                            xf[(u + 1) & 1][t] = *reinterpret_cast<const Frag*>(b + (u + 1) * kNBS * 16 * Cfg::kPitch + t * 64);
                    }
                    f32x4 sum = d[0];
                    if constexpr (kChains == 2) sum += d[1];
#pragma unroll
                    for (int c = 0; c < kChains; ++c) d[c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int t = 0; t < kGroups; ++t) {
                        if constexpr (kIsF32) {
#pragma unroll
                            for (int i = 0; i < 4; ++i)
                                d[i & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[u & 1][t][i], xf[u & 1][t][i], d[i & 1], 0, 0, 0);
                        } else {
                            d[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[u & 1][t], xf[u & 1][t], d[0], 0, 0, 0);
                        }
                    }
                    *reinterpret_cast<f32x4*>(dst) = av + sum;
                    dst = my_acc + rows[u];
                }
                __syncthreads();
            }
            f32x4 sum = d[0];
            if constexpr (kChains == 2) sum += d[1];
            *reinterpret_cast<f32x4*>(dst) = *reinterpret_cast<const f32x4*>(dst) + sum;
        }
    }
    __syncthreads();

    // ---- one rounding, whole rows
    const int64_t row0 = tile * TR;
    const int co0 = blockIdx.y * Cfg::kCOT;
    constexpr int kQuads = Cfg::kCOT / 4;
    const bool whole = a.co % 4 == 0;
    for (int idx = tid; idx < TR * kQuads; idx += Cfg::kThreads) {
        const int r = idx / kQuads, c = co0 + (idx % kQuads) * 4;
        const int64_t row = row0 + r;
        if (row >= a.n_rows) break;
        if (c >= a.co) continue;
        f32x4 v = *reinterpret_cast<const f32x4*>(acc + r * Cfg::kAccStride + (idx % kQuads) * 4);
#pragma unroll
        for (int i = 1; i < kNBS; ++i)
            v += *reinterpret_cast<const f32x4*>(acc + (i * (TR + 1) + r) * Cfg::kAccStride + (idx % kQuads) * 4);
        auto bits = [](float f) -> uint32_t {  // bf16, nearest even; NaN stays NaN
            const uint32_t u = __float_as_uint(f);
            return (u & 0x7fffffffu) > 0x7f800000u ? ((u >> 16) | 0x40) : ((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
        };
        T* out = static_cast<T*>(a.g) + row * a.co + c;
        if (whole) {
            if constexpr (kIsF32) *reinterpret_cast<f32x4*>(out) = v;
            else *reinterpret_cast<uint2*>(out) = uint2{bits(v[0]) | (bits(v[1]) << 16), bits(v[2]) | (bits(v[3]) << 16)};
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (c + i < a.co) {
                    if constexpr (kIsF32) out[i] = v[i];
                    else out[i] = (T)bits(v[i]);
                }
        }
    }
}

// Weights as stored (element (k, co, cc) at w[k*per + co*s_co + cc*s_cc]) -> fragment-major copy
// [k][channel tile][cs][slice][fragment][lane][16 bytes], zeros beyond the real channels.  One thread per 16 bytes.
template <typename T>
__global__ __launch_bounds__(256) void tile_weights_kernel(const T* __restrict__ w, T* __restrict__ wf, int kvol, int co, int cc,
                                                           int s_co, int s_cc, int ny, int ncs, int nsl, int groups) {
    constexpr int kPer = 16 / (int)sizeof(T);
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t total = (int64_t)kvol * ny * ncs * nsl * groups * 64;
    if (idx >= total) return;
    int r = (int)idx;
    const int lane = r & 63; r >>= 6;
    const int s = r % groups; r /= groups;
    const int sl = r % nsl; r /= nsl;
    const int cs = r % ncs; r /= ncs;
    const int y = r % ny, k = r / ny;
    const int c = (y * ncs + cs) * 16 + (lane & 15);
    const int cc0 = (sl * groups + s) * kPer * 4 + (lane >> 4) * kPer;
    T v[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i)
        v[i] = (c < co && cc0 + i < cc) ? w[(size_t)k * co * cc + (size_t)c * s_co + (size_t)(cc0 + i) * s_cc] : (T)0;
    uint4 raw;
    __builtin_memcpy(&raw, v, 16);
    *reinterpret_cast<uint4*>(wf + idx * kPer) = raw;
}

template <typename T, int KC, int NCS, int TR, bool BIG = false>
int launch_tile(TileArgs a, hipStream_t s) {
    using Cfg = TileCfg<T, KC, NCS, TR>;
    auto kern = gather_tile_kernel<T, KC, NCS, TR, BIG>;
    a.max_blk = a.kvol * (TR / 16);
    const int lds = Cfg::kFixed + a.max_blk * 16;
    if (lds > 160 * 1024 - 64) return fail(SP_ERR_UNSUPPORTED, "internal: tile does not fit the LDS");
    {
        static std::mutex mu;
        static int attr_lds = 0;  // largest dynamic LDS size opted into so far
        std::lock_guard<std::mutex> lk(mu);
        if (lds > attr_lds) {
            SP_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds));
            attr_lds = lds;
        }
    }
    const int64_t tiles = (a.n_rows + TR - 1) / TR;
    const int ny = (a.co + Cfg::kCOT - 1) / Cfg::kCOT;
    hipLaunchKernelGGL(kern, dim3((unsigned)tiles, (unsigned)ny), dim3(Cfg::kThreads), lds, s, a);
    SP_HIP(hipGetLastError());
    return SP_OK;
}

}  // namespace sp
