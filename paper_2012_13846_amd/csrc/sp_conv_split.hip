// Link-list gather-GEMM (Eq. 2 and its input gradient) for fp32 layers on the bf16 matrix cores, without giving up fp32
// precision: every value, taken 2^24 times, is the exact sum of three bf16 numbers (8 + 8 + 8 significant bits; the exponent range
// is the same, so without the factor values below 2^-110 would lose bits, and with it a subnormal's last bit, 2^-149, becomes
// 2^-125, a normal bf16 number), and a product of two values is the six partial products that matter,
//   x w = x0 w0 + (x0 w1 + x1 w0) + (x1 w1 + x0 w2 + x2 w0)   (+ terms below 2^-24 of it),
// added smallest first in the matrix cores' fp32 accumulator.  Six bf16 MFMAs of 32 contraction channels take 96
// cycles where fp32 MFMAs take 256, and leave the vector pipe free meanwhile.
// Error against fp64 (one MI355X, normal inputs, 27 links of 64 channels, over the result's rms): 1.1e-7 rms, 8.7e-7
// largest; fp32 MFMAs 1.75e-7 and 1.0e-6 (32 channels 1.1e-7 / 9.8e-7 against 1.4e-7 / 9.3e-7, 128 1.2e-7 / 9.3e-7 against
// 2.3e-7 / 1.2e-6): a chain of 64 channels is rounded 12 times instead of 64.
// An infinity, a NaN or a value of 2^104 and more makes its link's products NaN, and sums of 2^80 (1e24) overflow.  A workgroup
// that finds a value that is not finite among its sums therefore computes its rows again with fp32 MFMAs (redo below), and what
// it writes is what those give.
#include <mutex>

#include "sp_internal.h"
#include "sp_split_shape.h"

namespace sp {
namespace {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct SplitArgs {
    const int32_t* off;  // the side's lists (MapSide)
    const int32_t* src;
    const int32_t* dst;
    const float* f;      // source features [n_src][cc]
    const void* w;       // split weights (split_weights_kernel)
    const float* w0;     // the weights as stored: element (k, co, cc) at w0[k*co*cc + co*s_co + cc*s_cc]
    float* g;            // destination features [n_rows][co]
    int64_t n_rows;
    int kvol, co, cc, flip;
    int s_co, s_cc;
    int nsl;             // slices of CC contraction channels
    int halves;          // 32-row halves of sub-tiles per workgroup (split_tile)
    uint32_t f_bytes, w_bytes, list_bytes;
};

// 2^24, of rows and of weights.  (Two more instructions for every eleven of a pair's split: a layer's three passes and its maps at
// 0.6 M rows, 64 -> 64, 1427 -> 1449 us.  Without it the error is 2.7e-6 of values around 1e-35 and 2.7e-4 around 1e-37.)
constexpr float kScale = 16777216.f;
constexpr float kUnscale = 1.f / kScale / kScale;

// The three bf16 pieces of two values, kScale times, nearest even: each remainder is exact in fp32.
__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}
__device__ __forceinline__ void split_two(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l) {
    a *= kScale;
    b *= kScale;
    h = bf16_pair(a, b);
    a -= __uint_as_float(h << 16);
    b -= __uint_as_float(h & 0xffff0000u);
    m = bf16_pair(a, b);
    a -= __uint_as_float(m << 16);
    b -= __uint_as_float(m & 0xffff0000u);
    l = bf16_pair(a, b);
}

// The six products: piece of the weights, piece of the rows, smallest first.
constexpr int kProducts = 6;
__device__ constexpr int kOrderW[kProducts] = {2, 1, 1, 0, 0, 0};
__device__ constexpr int kOrderX[kProducts] = {0, 1, 0, 2, 1, 0};

// CC contraction channels a slice, NW wavefronts of 16 destination channels each, steps of up to 16 G links.
template <int CC, int NW, int G>
struct SplitCfg {
    static constexpr int kK = CC / 32;                   // MFMA steps of the contraction
    static constexpr int kThreads = 64 * NW;
    static constexpr int kCOT = 16 * NW;
    static constexpr int kStride = kCOT + 4;             // floats per accumulator row
    static constexpr int kLinks = 16 * G;                // links of a step
    static constexpr int kPieces = CC / 4;               // 16-byte pieces of a row's slice
    static constexpr int kLoads = (kLinks * kPieces + kThreads - 1) / kThreads;  // per thread and step
    static constexpr int kPlane = CC * 2;                // one of the three pieces of a staged row
    static constexpr int kPitch = 3 * kPlane;            // staged row
    // Place of 16-byte piece p in a plane of staged row `link`: the fragment reads and the stores meet no bank twice (the LDS serves a
    // read of 16 bytes a lane in groups of lanes like 0-3, 12-15, 20-27).  A pad of 32 bytes instead left the stores conflicts and
    // took room: 32 -> 128 on 0.6 M links 107 us, one workgroup a CU, 86 so with two.
    static __device__ __forceinline__ int place(int link, int p) { return (CC == 64 ? p ^ (link >> 1 & 7) : p ^ (-(link >> 2) & 3)) * 16; }
    static constexpr int kBuf = kLinks * kPitch;
    static constexpr int kW = 3 * kK;                    // weight fragments of a step and wavefront
    static constexpr int kWBytes = kW * NW * 1024;       // split weights of one offset, slice and channel tile
    static_assert(split_lds(CC, NW, G, 2, 1) == 65 * kStride * 4 + 2 * kBuf + 2 * kLinks * 4 + (64 + kLinks - 1) / kLinks * 8, "the kernel's carving of smem");
};

// A workgroup owns `halves` x 32 destination rows and 16 NW channels and accumulates in LDS.  Its links of one offset (and one
// slice of the contraction) are cut into steps of up to 16 G.  In a step every wavefront
//   - asks for its 16 channels of the next step's weights, which then serve all links of that step;
//   - splits its share of the next step's rows, which it asked for a step ago, and stores the pieces to LDS;
//   - multiplies this step's blocks and adds a block's sums to the accumulator while the next one is multiplied.
// One barrier a step; every wavefront has the same number of blocks, so none waits long, and where registers and LDS allow it two or more
// workgroups share a CU (tiles of 128 channels: one; two of 32 -> 128).
// What bounds it (64 -> 64, 0.6 M rows, 5 M links: 425 us with pauses between launches, 496 between the other kernels of a training pass,
// where the clock is lower; 467 with rows asked for four steps ahead, padded rows in LDS and tiles of 128, 618 on fp32 MFMAs): the L1's data
// return is busy 98 % of the cycles (half of it the weights, 24 KB a step), its addresser 81 %, the LDS 57 %, the vector pipes 51 %, the
// matrix pipes 35 %; two or three wavefronts per SIMD issue in order and wait a third of their time, so what lets a third workgroup in
// pays.  Built and dropped: one wavefront per SIMD that owns 128 rows and 64 channels and meets no barrier
// (weights in 96 or 192 registers, everything dealt out between the MFMAs): 555 against 514 us, since a single wavefront issues one
// instruction in four cycles of whatever kind.  Requests in front of the blocks instead of between their MFMAs, and fragments read
// when they are due: 542.
template <int CC, int NW, int G>
__global__ __launch_bounds__(64 * NW) void gather_split_kernel(SplitArgs a) {
    using Cfg = SplitCfg<CC, NW, G>;
    constexpr int kK = Cfg::kK, kThreads = Cfg::kThreads, kPieces = Cfg::kPieces, kLoads = Cfg::kLoads, kLinks = Cfg::kLinks;
    constexpr int kR = 2;  // steps whose rows are in flight or being stored (even: the weights alternate between two sets)
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int s_steps;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n16 = lane & 15, g = lane >> 4;
    const int rows = a.halves * 32, kvol = a.kvol;
    const int64_t tile = blockIdx.x, row0 = tile * rows;
    float* acc = reinterpret_cast<float*>(smem);
    unsigned char* xbuf = smem + (rows + 1) * Cfg::kStride * 4;
    int* s_row = reinterpret_cast<int*>(xbuf + 2 * Cfg::kBuf);  // accumulator offsets of two steps' links
    int2* s_step = reinterpret_cast<int2*>(s_row + 2 * kLinks); // {first link, offset | (links - 1) << 7}
    const int co0 = blockIdx.y * Cfg::kCOT;

    auto clear = [&](int t0, int n) __attribute__((always_inline)) {
        for (int i = t0; i < (rows + 1) * Cfg::kStride / 4; i += n) reinterpret_cast<f32x4*>(acc)[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    if (wave == 0) {
        int ns = 0;
        const int64_t h0 = tile * a.halves, h_end = (a.n_rows + kTileRows - 1) / kTileRows * (kTileRows / 32);
        const int64_t h1 = h0 + a.halves < h_end ? h0 + a.halves : h_end;
        const int32_t* p0 = a.off + (h0 >> 1) * kvol * kHalves + (h0 & 1);
        const int32_t* p1 = a.off + (h1 >> 1) * kvol * kHalves + (h1 & 1);
        for (int kb = 0; kb < kvol; kb += 64) {
            const int k = kb + lane;
            int o0 = 0, cnt = 0;
            if (k < kvol) {
                o0 = p0[k * kHalves];
                cnt = p1[k * kHalves] - o0;
            }
            const int nb = (cnt + kLinks - 1) / kLinks;
            int inc = nb;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int t = __shfl_up(inc, d, 64);
                if (lane >= d) inc += t;
            }
            const int ex = ns + inc - nb;
            for (int i = 0; i < nb; ++i) s_step[ex + i] = int2{o0 + kLinks * i, k | ((min(kLinks, cnt - kLinks * i) - 1) << 7)};
            ns += __shfl(inc, 63, 64);
        }
        if (lane == 0) s_steps = ns;
    } else {
        clear(tid - 64, kThreads - 64);
    }
    __syncthreads();
    const int ns = __builtin_amdgcn_readfirstlane(s_steps);
    const int total = ns * a.nsl;  // steps of all slices, slice by slice

    constexpr int kRsrcFlags = 0x00020000;
    constexpr uint32_t kOutside = 0xffffff00u;  // every buffer ends before it: loads from here return zeros
    const __amdgpu_buffer_rsrc_t rF = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.f), 0, (int)a.f_bytes, kRsrcFlags);
    const __amdgpu_buffer_rsrc_t rW = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.w), 0, (int)a.w_bytes, kRsrcFlags);
    const __amdgpu_buffer_rsrc_t rSrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(a.src), 0, (int)a.list_bytes, kRsrcFlags);
    const __amdgpu_buffer_rsrc_t rRow =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(a.dst), 0, (int)a.list_bytes, kRsrcFlags);
    const uint32_t row_bytes = (uint32_t)a.cc * 4u;
    const uint32_t w_base = blockIdx.y * (uint32_t)(kvol * a.nsl) * Cfg::kWBytes + wave * (Cfg::kW * 1024);

    // Cursors walk the steps and stay on the last one.
    struct Cursor {
        int at, sl;
    };
    auto advance = [&](Cursor& c) __attribute__((always_inline)) {
        const bool wrap = c.at + 1 == ns, more = !wrap || c.sl + 1 < a.nsl;
        c.at = more ? (wrap ? 0 : c.at + 1) : c.at;
        c.sl = more && wrap ? c.sl + 1 : c.sl;
    };
    struct Ent {
        int src, row;  // lane l: source and destination row of the step's link l (past its end: of the last one)
        int last;      // its last link
        int sl;        // and slice, the same in every lane
    };
    Cursor ahead{0, 0}, here{0, 0};
    auto entries = [&](Ent& e, const int2& d) __attribute__((always_inline)) {
        e.last = __builtin_amdgcn_readfirstlane(d.y >> 7);
        e.sl = ahead.sl;
        const uint32_t o = (uint32_t)(d.x + min(lane, e.last)) * 4u;
        e.src = (int)__builtin_amdgcn_raw_buffer_load_b32(rSrc, o, 0, 0);
        e.row = (int)__builtin_amdgcn_raw_buffer_load_b32(rRow, o, 0, 0);
        advance(ahead);
    };
    auto look_up = [&](Ent& e) __attribute__((always_inline)) { entries(e, s_step[ahead.at]); };
    struct Rows {
        u32x4 x[kLoads];
        int row;  // lane l: accumulator offset of link l
    };
    // thread t fetches pieces t, t + kThreads, ... of the step's rows (kPieces adjacent threads per row)
    const int my_piece = tid % kPieces, my_link = tid / kPieces;
    constexpr int kLinkStep = kThreads / kPieces;
    static_assert(kThreads % kPieces == 0, "a thread's pieces lie in one column");
    struct Where {
        uint32_t row[kLoads];  // source row of each load
    };
    auto locate = [&](Where& wh, const Ent& e) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < kLoads; ++j) wh.row[j] = (uint32_t)__shfl(e.src, (my_link + j * kLinkStep) & 63, 64);
    };
    auto gather = [&](Rows& r, const Where& wh, const Ent& e, int j) __attribute__((always_inline)) {
        const uint32_t in_row = (uint32_t)e.sl * (CC * 4) + my_piece * 16;
        const bool there = in_row < row_bytes;  // the last slice may reach past the row's end
        r.x[j] = __builtin_amdgcn_raw_buffer_load_b128(rF, wh.row[j] * (there ? row_bytes : 0u) + (there ? in_row : kOutside), 0, 0);
    };
    auto target = [&](const Ent& e) __attribute__((always_inline)) { return (lane <= e.last ? e.row - (int)row0 : rows) * Cfg::kStride; };
    auto store = [&](const Rows& r, int par, int j) __attribute__((always_inline)) {
        const int link = my_link + j * kLinkStep;
        const f32x4 v = __builtin_bit_cast(f32x4, r.x[j]);
        uint32_t lo[3], hi[3];
        split_two(v[0], v[1], lo[0], lo[1], lo[2]);
        split_two(v[2], v[3], hi[0], hi[1], hi[2]);
        unsigned char* b = xbuf + par * Cfg::kBuf + Cfg::place(link, my_piece >> 1) + (my_piece & 1) * 8 + link * Cfg::kPitch;
        if (kLinks * kPieces % kThreads == 0 || link < kLinks)
#pragma unroll
            for (int q = 0; q < 3; ++q) *reinterpret_cast<u32x2*>(b + q * Cfg::kPlane) = u32x2{lo[q], hi[q]};
    };
    struct WSet {
        bf16x8 w[3][kK];
    };
    auto weights_at = [&](int key) __attribute__((always_inline)) {  // key: offset | (links - 1) << 7 | slice << 16
        const int k = key & 127;
        return (int)(w_base + (uint32_t)((a.flip ? kvol - 1 - k : k) * a.nsl + (key >> 16)) * Cfg::kWBytes);
    };
    auto load_weight = [&](WSet& s, int soff, int i) __attribute__((always_inline)) {  // fragment i, in the order of their first use
        const int p = 2 - i / kK, t = i % kK;
        s.w[p][t] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rW, lane * 16 + (p * kK + t) * 1024, soff, 0));
    };
    // Sums of a block, in two chains of dependent MFMAs: lane (link n16, channels wave*16 + 4 g .. + 3)
    struct Result {
        f32x4 d[2];
        float* dst;
    };
    struct Frags {
        bf16x8 x[3][kK];
        int row;
    };
    float* const my_acc = acc + wave * 16 + g * 4;
    const unsigned char* const my_frag[2] = {xbuf + n16 * Cfg::kPitch + Cfg::place(n16, g), xbuf + n16 * Cfg::kPitch + Cfg::place(n16, (4 + g) % (CC / 8))};
    auto read_frags = [&](Frags& f, int par, int block) __attribute__((always_inline)) {
        const int b = par * Cfg::kBuf + block * 16 * Cfg::kPitch;
#pragma unroll
        for (int q = 0; q < 3; ++q)
#pragma unroll
            for (int t = 0; t < kK; ++t) f.x[q][t] = *reinterpret_cast<const bf16x8*>(my_frag[t] + b + q * Cfg::kPlane);
        f.row = s_row[par * kLinks + block * 16 + n16];
    };
    // A block: its MFMAs, product by product, and between them the previous block's sums go to the accumulator and
    // extra(product) does its part.
    auto multiply = [&](Result& r, const Result& prev, const WSet& w, const Frags& f, auto&& extra) __attribute__((always_inline)) {
        r.d[0] = r.d[1] = f32x4{0.f, 0.f, 0.f, 0.f};
        f32x4 av;
#pragma unroll
        for (int o = 0; o < kProducts; ++o) {
            if (o == 0) av = *reinterpret_cast<const f32x4*>(prev.dst);
            extra(o);
            if (o == kProducts - 2) *reinterpret_cast<f32x4*>(prev.dst) = av + (prev.d[0] + prev.d[1]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < kK; ++t) {
                const int c = (kK == 1 ? o : t) & 1;
                r.d[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.w[kOrderW[o]][t], f.x[kOrderX[o]][t], r.d[c], 0, 0, 0);
            }
        }
        r.dst = my_acc + f.row;
        __builtin_amdgcn_sched_barrier(0);
    };

    if (total > 0) {
        Ent ents[4];
        Rows xs[kR];
        WSet ws[2];
        Result res;
        res.d[0] = res.d[1] = f32x4{0.f, 0.f, 0.f, 0.f};
        res.dst = my_acc + rows * Cfg::kStride;
        auto key_at = [&](const Cursor& c) __attribute__((always_inline)) { return s_step[c.at].y | c.sl << 16; };
        int key0 = __builtin_amdgcn_readfirstlane(key_at(here));
        advance(here);
        int key1 = __builtin_amdgcn_readfirstlane(key_at(here));
        advance(here);
        {
            Ent first[kR];
#pragma unroll
            for (int i = 0; i < kR; ++i) look_up(first[i]);
#pragma unroll
            for (int i = 0; i < 3; ++i) look_up(ents[i]);
            const int soff = weights_at(key0);
#pragma unroll
            for (int i = 0; i < Cfg::kW; ++i) load_weight(ws[0], soff, i);
#pragma unroll
            for (int i = 0; i < kR; ++i) {
                Where wh;
                locate(wh, first[i]);
#pragma unroll
                for (int j = 0; j < kLoads; ++j) gather(xs[i], wh, first[i], j);
                xs[i].row = target(first[i]);
            }
        }
#pragma unroll
        for (int j = 0; j < kLoads; ++j) store(xs[0], 0, j);
        if (tid < kLinks) s_row[tid] = xs[0].row;
        __syncthreads();
        // A step out of LDS buffer par.  x: the registers its rows came from, for those kR steps ahead; xn: the next step's rows.
        auto body = [&](int par, Rows& x, const Rows& xn, const WSet& w, WSet& wn, const Ent& e, Ent& e3) __attribute__((always_inline)) {
            const int last = key0 >> 7 & 511;
            Frags f[2];
            read_frags(f[0], par, 0);
            Where wh;
            locate(wh, e);
            const int key2 = key_at(here);
            const int2 d = s_step[ahead.at];
            const int soff = weights_at(key1);
            Result r0;
            __builtin_amdgcn_sched_barrier(0);
            multiply(r0, res, w, f[0], [&](int o) __attribute__((always_inline)) {
                if (o == 0 && G > 1) read_frags(f[1], par, 1);
#pragma unroll
                for (int i = 0; i < Cfg::kW; ++i)
                    if (i * kProducts / Cfg::kW == o) load_weight(wn, soff, i);
#pragma unroll
                for (int j = 0; j < kLoads; ++j) {
                    if (j * kProducts / kLoads == o) store(xn, par ^ 1, j);
                    if (j * kProducts / kLoads == o) gather(x, wh, e, j);
                }
                if (o == kProducts - 1) {
                    if (tid < kLinks) s_row[(par ^ 1) * kLinks + tid] = xn.row;
                    x.row = target(e);
                    entries(e3, d);
                }
            });
            res = r0;
#pragma unroll
            for (int b = 1; b < G; ++b) {
                if (last >= 16 * b) {
                    Result r;
                    multiply(r, res, w, f[b & 1], [&](int o) __attribute__((always_inline)) {
                        if (o == 0 && b + 1 < G) read_frags(f[(b + 1) & 1], par, b + 1);
                    });
                    res = r;
                }
            }
            advance(here);
            key0 = key1;
            key1 = __builtin_amdgcn_readfirstlane(key2);
            __syncthreads();
        };
        for (int left = total;; left -= 4) {
            body(0, xs[0], xs[1], ws[0], ws[1], ents[0], ents[3]);
            if (left <= 1) break;
            body(1, xs[1], xs[0], ws[1], ws[0], ents[1], ents[0]);
            if (left <= 2) break;
            body(0, xs[0], xs[1], ws[0], ws[1], ents[2], ents[1]);
            if (left <= 3) break;
            body(1, xs[1], xs[0], ws[1], ws[0], ents[3], ents[2]);
            if (left <= 4) break;
        }
        f32x4* p = reinterpret_cast<f32x4*>(res.dst);
        *p = *p + (res.d[0] + res.d[1]);
    }
    __syncthreads();

    // whole rows; is any sum not finite?
    auto write = [&](float unscale) __attribute__((always_inline)) {
        constexpr int kQuads = Cfg::kCOT / 4;
        const bool whole = a.co % 4 == 0;
        bool bad = false;
        for (int idx = tid; idx < rows * kQuads; idx += kThreads) {
            const int r = idx / kQuads, c = co0 + (idx % kQuads) * 4;
            const int64_t row = row0 + r;
            if (row >= a.n_rows) break;
            if (c >= a.co) continue;
            f32x4 v = *reinterpret_cast<const f32x4*>(acc + r * Cfg::kStride + (idx % kQuads) * 4);
            const float z = (v[0] - v[0]) + (v[1] - v[1]) + (v[2] - v[2]) + (v[3] - v[3]);  // 0, or NaN
            bad = bad || !(z == 0.f);
            v *= unscale;
            float* out = a.g + row * a.co + c;
            if (whole) {
                *reinterpret_cast<f32x4*>(out) = v;
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (c + i < a.co) out[i] = v[i];
            }
        }
        return bad;
    };
    if (!__syncthreads_or(write(kUnscale) ? 1 : 0)) return;

    // ---- redo: the same rows with fp32 MFMAs, one block at a time, each wavefront its own channels
    clear(tid, kThreads);
    __syncthreads();
    const int o = co0 + wave * 16 + n16;
    for (int i = 0; i < ns; ++i) {
        const int beg = __builtin_amdgcn_readfirstlane(s_step[i].x), key = __builtin_amdgcn_readfirstlane(s_step[i].y);
        const int k = key & 127, links = (key >> 7) + 1;
        const float* wk = a.w0 + (size_t)(a.flip ? kvol - 1 - k : k) * a.co * a.cc;
        for (int b = 0; b < links; b += 16) {
            const int e = beg + min(b + n16, links - 1);
            const float* x = a.f + (size_t)a.src[e] * a.cc;
            const int row = a.dst[e] - (int)row0;
            f32x4 d = {0.f, 0.f, 0.f, 0.f};
            for (int c = 0; c < a.cc; c += 4) {
                const bool in = c + g < a.cc;
                const float xv = in ? x[c + g] : 0.f;
                const float wv = in && o < a.co ? wk[(size_t)o * a.s_co + (size_t)(c + g) * a.s_cc] : 0.f;
                d = __builtin_amdgcn_mfma_f32_16x16x4f32(wv, xv, d, 0, 0, 0);
            }
            if (b + n16 < links) {
                f32x4* p = reinterpret_cast<f32x4*>(my_acc + row * Cfg::kStride);
                *p = *p + d;
            }
        }
    }
    __syncthreads();
    write(1.f);
}

// Weights as stored (element (k, co, cc) at w[k*co*cc + co*s_co + cc*s_cc]) -> their pieces, fragment-major:
// [channel tile][offset][slice][16-channel group][piece][MFMA step][lane][16 bytes], zeros beyond the real channels.
// One thread per 8 weights.
__global__ __launch_bounds__(256) void split_weights_kernel(const float* __restrict__ w, u32x4* __restrict__ ws, int kvol, int co, int cc,
                                                            int s_co, int s_cc, int ny, int nsl, int steps, int groups) {
    const int idx = blockIdx.x * 256 + threadIdx.x;
    if (idx >= ny * kvol * nsl * steps * groups * 64) return;
    int r = idx;
    const int lane = r & 63; r >>= 6;
    const int t = r % steps; r /= steps;
    const int cs = r % groups; r /= groups;
    const int sl = r % nsl; r /= nsl;
    const int k = r % kvol, y = r / kvol;
    const int c = (y * groups + cs) * 16 + (lane & 15);
    const int cc0 = (sl * steps + t) * 32 + (lane >> 4) * 8;
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = c < co && cc0 + j < cc ? w[(size_t)k * co * cc + (size_t)c * s_co + (size_t)(cc0 + j) * s_cc] : 0.f;
    u32x4 p[3];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t h, m, l;
        split_two(v[2 * i], v[2 * i + 1], h, m, l);
        p[0][i] = h;
        p[1][i] = m;
        p[2][i] = l;
    }
    const size_t base = (size_t)(((y * kvol + k) * nsl + sl) * groups + cs) * 3 * steps * 64;
#pragma unroll
    for (int q = 0; q < 3; ++q) ws[base + (size_t)(q * steps + t) * 64 + lane] = p[q];
}

template <int CC, int NW, int G>
int launch_split(const SplitArgs& a, int ny, hipStream_t s) {
    using Cfg = SplitCfg<CC, NW, G>;
    auto kern = gather_split_kernel<CC, NW, G>;
    const int lds = split_lds(CC, NW, G, a.halves, a.kvol);
    {
        static std::mutex mu;
        static int attr_lds = 0;  // largest dynamic LDS size opted into so far
        std::lock_guard<std::mutex> lk(mu);
        if (lds > attr_lds) {
            SP_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds));
            attr_lds = lds;
        }
    }
    const int64_t tiles = (a.n_rows + a.halves * 32 - 1) / (a.halves * 32);
    hipLaunchKernelGGL(kern, dim3((unsigned)tiles, (unsigned)ny), dim3(Cfg::kThreads), lds, s, a);
    SP_HIP(hipGetLastError());
    return SP_OK;
}

}  // namespace

int conv_gather_split(const MapSide& side, int kvol, int64_t links, const float* d_f, const float* d_w, bool w_transposed, float* d_g, int cc, int co,
                      void* d_ws, hipStream_t s) {
    const SplitShape t = split_shape(cc, co);
    SplitArgs a{};
    a.off = ptr<int32_t>(side.off);
    a.src = ptr<int32_t>(side.src);
    a.dst = ptr<int32_t>(side.dst);
    a.f = d_f;
    a.w = d_ws;
    a.w0 = d_w;
    a.g = d_g;
    a.n_rows = side.n_rows;
    a.kvol = kvol;
    a.co = co;
    a.cc = cc;
    a.flip = side.flip ? 1 : 0;
    a.s_co = w_transposed ? 1 : cc;
    a.s_cc = w_transposed ? co : 1;
    a.nsl = t.nsl;
    a.f_bytes = (uint32_t)((uint64_t)side.n_src * cc * 4);
    a.w_bytes = (uint32_t)split_copy_bytes(t, kvol);
    a.list_bytes = (uint32_t)((uint64_t)side.pitch * kvol * 4);
    const int threads = t.ny * kvol * t.nsl * (t.cc / 32) * (t.cot / 16) * 64;
    hipLaunchKernelGGL(split_weights_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, d_w, static_cast<u32x4*>(d_ws), kvol,
                       co, cc, a.s_co, a.s_cc, t.ny, t.nsl, t.cc / 32, t.cot / 16);
    const SplitTile tile = split_tile(t, side.n_rows, kvol, links);
    a.halves = tile.halves;
#define SP_SPLIT(CC, NW, G) \
    if (t.cc == CC && t.cot == 16 * NW && tile.g == G) return launch_split<CC, NW, G>(a, t.ny, s)
    SP_SPLIT(64, 8, 2);
    SP_SPLIT(64, 8, 3);
    SP_SPLIT(64, 4, 2);
    SP_SPLIT(64, 4, 3);
    SP_SPLIT(64, 3, 3);
    SP_SPLIT(64, 2, 2);
    SP_SPLIT(32, 8, 2);
    SP_SPLIT(32, 4, 2);
    SP_SPLIT(32, 3, 3);
    SP_SPLIT(32, 2, 2);
#undef SP_SPLIT
    return fail(SP_ERR_UNSUPPORTED, "internal: no split kernel for %d -> %d channels", cc, co);
}

}  // namespace sp
