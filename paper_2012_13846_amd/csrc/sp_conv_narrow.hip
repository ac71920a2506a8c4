// Step 3 of the generalized sparse convolution (Eq. 2) and its input gradient for layers with few channels on one side (the
// first layer of a network: 3 to 6 values a point): plain multiply-adds, a few threads per destination row, all weights in
// LDS, a row's neighbours requested together.  The matrix cores multiply four fifths of padding there.  A row's links are
// added in offset order, each one's dot product first, nine offsets before the total: fixed order, rounded once (one sum of all
// links was up to 10 % further from fp64 than the tile kernel is).  (Only links that exist are multiplied: an
// infinite weight does not reach rows it is not linked to.)
// What bounds it: one trip through the address unit per row and offset, live or not, and the multiply-adds of an offset
// that any of a wavefront's rows has (nearly all).  Times against the tile kernel's at narrow_us.
#include <algorithm>
#include <cmath>

#include "sp_internal.h"
#include "sp_tile_shape.h"

namespace sp {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t bf16_t;

__device__ __forceinline__ float load_f32(const float* p) { return *p; }
__device__ __forceinline__ float load_f32(const bf16_t* p) { return __uint_as_float((uint32_t)(*p) << 16); }
__device__ __forceinline__ void store_f32(float* p, float v) { *p = v; }
__device__ __forceinline__ void store_f32(bf16_t* p, float v) {  // nearest even; NaN stays NaN
    const uint32_t u = __float_as_uint(v);
    *p = (bf16_t)((u & 0x7fffffffu) > 0x7f800000u ? ((u >> 16) | 0x40) : ((u + 0x7fffu + ((u >> 16) & 1u)) >> 16));
}

struct NarrowArgs {
    const int32_t* nbr;  // [kvol][n_rows] source row or -1
    const void* f;       // source features [n_src][cc]
    const void* w;       // weights as stored: element (k, co, cc) at w[k*co*cc + co*s_co + cc*s_cc]
    void* g;             // destination features [n_rows][co]
    int64_t n_rows;
    int kvol, co, cc, flip;
    int s_co, s_cc;
};

constexpr int kThreads = 256;
constexpr int kAhead = 27;  // offsets whose neighbours are requested together

// The row numbers of the next kAhead offsets of one row.
__device__ __forceinline__ void load_neighbours(const NarrowArgs& a, int k0, int64_t row, bool in, int32_t (&src)[kAhead]) {
#pragma unroll
    for (int i = 0; i < kAhead; ++i) src[i] = in && k0 + i < a.kvol ? a.nbr[(int64_t)(k0 + i) * a.n_rows + row] : -1;
}

// CC source channels: a thread sums OC destination channels of one row, cop / OC threads per row.
// LDS: weights [offset][CC][cop], zeros beyond the real destination channels.
template <typename T, int CC, int OC>
__global__ __launch_bounds__(kThreads) void narrow_in_kernel(NarrowArgs a, int cop) {
    extern __shared__ __align__(16) float s_w[];
    const T* __restrict__ w = static_cast<const T*>(a.w);
    const T* __restrict__ f = static_cast<const T*>(a.f);
    const int tpr = cop / OC, rows = kThreads / tpr, o0 = (int)threadIdx.x % tpr * OC;
    int64_t row = (int64_t)blockIdx.x * rows + threadIdx.x / tpr;
    const bool mine = (int)threadIdx.x < rows * tpr;
    int32_t src[kAhead];
    load_neighbours(a, 0, row, mine && row < a.n_rows, src);
    {
        const int per = kThreads / cop, o = (int)threadIdx.x % cop;
        for (int k = (int)threadIdx.x / cop; k < a.kvol && (int)threadIdx.x < per * cop; k += per) {
            const T* p = w + (size_t)(a.flip ? a.kvol - 1 - k : k) * a.co * CC + (size_t)o * a.s_co;
#pragma unroll
            for (int c = 0; c < CC; ++c) s_w[(k * CC + c) * cop + o] = o < a.co ? load_f32(p + c * a.s_cc) : 0.f;
        }
    }
    __syncthreads();
    if (!mine) return;
    for (; row < a.n_rows; row += (int64_t)gridDim.x * rows) {
        float acc[OC];
#pragma unroll
        for (int j = 0; j < OC; ++j) acc[j] = 0.f;
        for (int k0 = 0; k0 < a.kvol; k0 += kAhead) {
            if (k0 > 0 || row >= (int64_t)gridDim.x * rows) load_neighbours(a, k0, row, true, src);
            constexpr int kN = 9;  // links whose rows are requested together
#pragma unroll
            for (int i0 = 0; i0 < kAhead; i0 += kN) {
                float x[kN][CC];
#pragma unroll
                for (int i = 0; i < kN; ++i) {
                    const T* p = f + (int64_t)(src[i0 + i] < 0 ? 0 : src[i0 + i]) * CC;
                    T v[CC];
                    __builtin_memcpy(v, p, sizeof(v));
#pragma unroll
                    for (int c = 0; c < CC; ++c) x[i][c] = load_f32(v + c);
                }
                float part[OC];
#pragma unroll
                for (int j = 0; j < OC; ++j) part[j] = 0.f;
#pragma unroll
                for (int i = 0; i < kN; ++i) {
                    if (src[i0 + i] < 0) continue;
                    const float* wk = s_w + (k0 + i0 + i) * CC * cop + o0;
                    constexpr int kHalf = CC > 4 ? (CC + 1) / 2 : CC;
                    float dot[2][OC];  // more than four products in two chains: fewer roundings of large sums
#pragma unroll
                    for (int j = 0; j < OC; ++j) dot[0][j] = dot[1][j] = 0.f;
#pragma unroll
                    for (int c = 0; c < CC; ++c)
#pragma unroll
                        for (int j = 0; j < OC; ++j) dot[c / kHalf][j] = fmaf(wk[c * cop + j], x[i][c], dot[c / kHalf][j]);
#pragma unroll
                    for (int j = 0; j < OC; ++j) part[j] += CC > 4 ? dot[0][j] + dot[1][j] : dot[0][j];
                }
#pragma unroll
                for (int j = 0; j < OC; ++j) acc[j] += part[j];
            }
        }
        T* out = static_cast<T*>(a.g) + row * a.co + o0;
#pragma unroll
        for (int j = 0; j < OC; ++j)
            if (o0 + j < a.co) store_f32(out + j, acc[j]);
    }
}

// OM destination channels: a thread sums the part of them that 8 source channels make, cc / 8 threads per row (a power of
// two), which add their parts at the end.  LDS: weights [offset][OM][cc].  (Three wavefronts a SIMD: 170 registers would be two,
// 64 -> 6 on 2.4 M links 220 us against 126.)
template <typename T, int OM>
__global__ __launch_bounds__(kThreads, 3) void narrow_out_kernel(NarrowArgs a) {
    extern __shared__ __align__(16) float s_w[];
    const T* __restrict__ w = static_cast<const T*>(a.w);
    const T* __restrict__ f = static_cast<const T*>(a.f);
    const int tpr = a.cc / 8, c0 = (int)threadIdx.x % tpr * 8;
    const int rows = kThreads / tpr;
    const int64_t first = (int64_t)blockIdx.x * rows;
    int32_t src[kAhead];
    load_neighbours(a, 0, first + threadIdx.x / tpr, first + threadIdx.x / tpr < a.n_rows, src);
    {
        const int per = max(kThreads / a.cc, 1);
        for (int c = (int)threadIdx.x % min(a.cc, kThreads); c < a.cc; c += kThreads)
            for (int k = (int)threadIdx.x / min(a.cc, kThreads); k < a.kvol; k += per) {
                const T* p = w + (size_t)(a.flip ? a.kvol - 1 - k : k) * OM * a.cc + (size_t)c * a.s_cc;
#pragma unroll
                for (int o = 0; o < OM; ++o) s_w[(k * OM + o) * a.cc + c] = load_f32(p + o * a.s_co);
            }
    }
    __syncthreads();
    for (int64_t base = first; base < a.n_rows; base += (int64_t)gridDim.x * rows) {
        const int64_t row = base + threadIdx.x / tpr;
        const bool in = row < a.n_rows;
        float acc[OM];
#pragma unroll
        for (int j = 0; j < OM; ++j) acc[j] = 0.f;
        for (int k0 = 0; k0 < a.kvol; k0 += kAhead) {
            if (k0 > 0 || base > first) load_neighbours(a, k0, row, in, src);
            constexpr int kV = sizeof(T) == 4 ? 2 : 1;
            constexpr int kN = 9;
#pragma unroll
            for (int i0 = 0; i0 < kAhead; i0 += kN) {
                u32x4 x[kN][kV];
#pragma unroll
                for (int i = 0; i < kN; ++i) {
                    const u32x4* p = reinterpret_cast<const u32x4*>(f + (int64_t)(src[i0 + i] < 0 ? 0 : src[i0 + i]) * a.cc + c0);
#pragma unroll
                    for (int v = 0; v < kV; ++v) x[i][v] = p[v];
                }
                float part[OM];
#pragma unroll
                for (int j = 0; j < OM; ++j) part[j] = 0.f;
#pragma unroll
                for (int i = 0; i < kN; ++i) {
                    if (src[i0 + i] < 0) continue;
                    float xv[8];
#pragma unroll
                    for (int c = 0; c < 8; ++c) {
                        if constexpr (sizeof(T) == 4) xv[c] = __uint_as_float(x[i][c / 4][c % 4]);
                        else xv[c] = __uint_as_float(c & 1 ? x[i][0][c / 2] & 0xffff0000u : x[i][0][c / 2] << 16);
                    }
                    const float* wk = s_w + (k0 + i0 + i) * OM * a.cc + c0;
#pragma unroll
                    for (int j = 0; j < OM; ++j) {
                        const f32x4 lo = *reinterpret_cast<const f32x4*>(wk + j * a.cc), hi = *reinterpret_cast<const f32x4*>(wk + j * a.cc + 4);
                        float dot[2] = {0.f, 0.f};
#pragma unroll
                        for (int c = 0; c < 4; ++c) dot[0] = fmaf(lo[c], xv[c], dot[0]);
#pragma unroll
                        for (int c = 0; c < 4; ++c) dot[1] = fmaf(hi[c], xv[4 + c], dot[1]);
                        part[j] += dot[0] + dot[1];
                    }
                }
#pragma unroll
                for (int j = 0; j < OM; ++j) acc[j] += part[j];
            }
        }
#pragma unroll
        for (int j = 0; j < OM; ++j)
            for (int d = tpr >> 1; d > 0; d >>= 1) acc[j] += __shfl_xor(acc[j], d, 64);
        if (in && c0 == 0) {
            T* out = static_cast<T*>(a.g) + row * OM;
#pragma unroll
            for (int j = 0; j < OM; ++j) store_f32(out + j, acc[j]);
        }
    }
}

constexpr int kMaxLds = 64 * 1024;  // what a kernel may ask for without opting in

template <class... Args>
int launch(void (*kern)(Args...), int64_t n_rows, int rows_per_wg, size_t lds, hipStream_t s, Args... args) {
    // every workgroup loads the weights: no more of them than the chip takes at once
    const int64_t resident = 256 * std::min<int64_t>(8, 160 * 1024 / (int64_t)(lds + 1));
    const int64_t wgs = std::min((n_rows + rows_per_wg - 1) / rows_per_wg, resident);
    hipLaunchKernelGGL(kern, dim3((unsigned)wgs), dim3(kThreads), lds, s, args...);
    SP_HIP(hipGetLastError());
    return SP_OK;
}

bool pow2(int v) { return (v & (v - 1)) == 0; }

}  // namespace

namespace {
bool narrow_in_ok(int cc, int co, int kvol) { return cc <= 7 && cc * co <= 128 && co <= 64 && (size_t)kvol * cc * ((co + 7) / 8 * 8) * 4 <= (size_t)kMaxLds; }
bool narrow_out_ok(int cc, int co, int kvol) {
    return co <= 8 && cc >= 8 && cc <= 256 && pow2(cc) && (size_t)kvol * co * cc * 4 <= (size_t)kMaxLds;
}
// Destination channels per thread: twice the threads where 8 would leave the chip half empty (3 -> 32 on 23 k rows 13.7 against
// 11.3 us, 96 k 31.7 against 36.6).
int narrow_in_channels(int64_t rows, int co) { return co > 4 && rows * ((co + 7) / 8) >= 131072 ? 8 : 4; }
}  // namespace

// Microseconds of a launch: this kernel's, and the tile kernel's on the same rows.  Fitted to 13000 pairs of times each (300 to
// 613 k rows with 1 to 34 links each, K = 1 to 5, strides 1 and 2, both directions); off by 13 % rms, the tile kernel's on few fp32
// destinations by 22 %.  This kernel pays for every offset of a row, 27 at a time, and for the products of an offset that any row of
// a wavefront has (live); the tile kernel for the blocks of 16 links that a tile of rows has of each offset.
// this kernel / the tile kernel in us, fp32 | bf16:
//   few destinations, K = 3   64 -> 3, 96 k rows, 0.61 M links 46 / 130 | 43 / 58    32 -> 3  26 / 61 | 25 / 36    16 -> 6  19 / 38 | 17 / 36
//                             64 -> 6, 29 k rows, 52 k links   17 / 39  | 17 / 17    32 -> 6  12 / 18 | 12 / 14    8 -> 8   18 / 14 | 18 / 14
//                             64 -> 8, 213 k rows, 2.4 M links 200 / 356 | 207 / 154 32 -> 8  91 / 164 | 94 / 87   16 -> 8  54 / 93 | 54 / 86
//                      K = 5   8 -> 3, 1.9 k rows, 8 k links    33 / 25  | 37 / 23    8 -> 8   71 / 24 | 76 / 23
//   few sources, K = 3        3 -> 16, 148 k rows, 0.37 M links 27 / 54 | 24 / 68     3 -> 32 41 / 51 | 38 / 68     4 -> 32 48 / 42 | 43 / 47
//                             7 -> 16                           40 / 54 | 41 / 74     2 -> 64 58 / 44 | 47 / 39     3 -> 40 48 / 40 | 47 / 52
//                             4 -> 32, 1.9 k rows, 4 k links    8 / 13  | 9 / 16      2 -> 64 7 / 17 | 7 / 17
//                      K = 5   4 -> 32, 56 k rows, 0.28 M links  66 / 42 | 65 / 43
namespace {
struct Layer {
    double rows, links, k, cc, co;
    bool f32;
};
double live(const Layer& l, double rows_of_a_wave) { return 1.0 - std::pow(1.0 - std::min(1.0, l.links / (l.rows * l.k)), rows_of_a_wave); }
double blocks_of_a_tile(const Layer& l, double tile_rows) {
    const double per = l.links * tile_rows / (l.rows * l.k);
    return l.k * (1.0 - std::exp(-per) + per / 16.0);
}
double narrow_us(const Layer& l, bool few_out) {
    const double walked = std::ceil(l.k / kAhead) * kAhead, weights = l.k * l.cc * l.co / 1000.0;
    if (few_out) {
        const double tpr = l.cc / 8.0, turns = l.rows * tpr / 65536.0;   // 65536: a wavefront per SIMD
        const double chain = l.f32 ? 0.080 * walked + 0.044 * l.k * l.co * live(l, 64.0 / tpr) : 0.091 * walked + 0.047 * l.k * l.co * live(l, 64.0 / tpr);
        const double resident = std::min(8.0, std::floor(160.0 * 1024.0 / (l.k * l.co * l.cc * 4.0 + 1.0)));  // workgroups a CU, by LDS
        const double full = chain * std::max(1.0, (l.f32 ? 0.45 : 0.48) * turns * std::max(1.0, 2.7 / resident));
        return l.f32 ? 4.3 + 0.26 * weights + full + 0.029 * turns * walked + 0.22e-6 * l.links * l.cc
                     : 3.8 + 0.29 * weights + full + 0.0056 * turns * walked + 0.19e-6 * l.links * l.cc;
    }
    const int oc = narrow_in_channels((int64_t)l.rows, (int)l.co);
    const double tpr = std::ceil(l.co / oc), turns = l.rows * tpr / 65536.0;
    const double chain = 0.050 * walked + 0.008 * l.k * l.cc * oc * live(l, 64.0 / tpr);
    const double full = chain * std::max(1.0, 0.53 * turns);
    return l.f32 ? 4.9 + 0.40 * weights + full + 0.014 * turns * walked + 1.5e-6 * l.rows * l.co
                 : 4.7 + 0.47 * weights + full + 0.011 * turns * walked + 0.51e-6 * l.rows * l.co;
}
double tile_us(const Layer& l, bool few_out) {
    const TileShape t = tile_shape((int)l.cc, (int)l.co, l.f32, false);
    if (few_out) {
        const double unit = (l.f32 ? 0.0054 : 0.0030) * t.kc * t.nsl * blocks_of_a_tile(l, 64.0), tiles = l.rows / 64.0;
        return l.f32 ? 8.7 + (1.3 + unit) * std::max(1.0, tiles / 240.0) : 7.3 + (2.4 + unit) * std::max(1.0, tiles / 350.0);
    }
    const double tr = t.ncs >= 3 && l.rows / 128.0 * t.ny >= 512.0 ? 128.0 : 64.0, tiles = l.rows / tr * t.ny;
    const int row_bytes = (int)l.cc * (l.f32 ? 4 : 2);   // rows that are no whole 16-byte pieces are loaded in smaller ones
    const double loads = 1.0 + (row_bytes % 16 ? (l.f32 ? 0.36 : 0.30) : 0.0) + (row_bytes % 4 ? 0.98 : 0.0);
    const double unit = ((l.f32 ? 0.11 : 0.10) + (l.f32 ? 0.011 : 0.010) * t.ncs * tr / 64.0) * loads * blocks_of_a_tile(l, tr);
    return l.f32 ? 6.9 + (2.7 + unit) * std::max(1.0, tiles / 450.0) : 7.0 + (3.4 + unit) * std::max(1.0, tiles / 490.0);
}
}  // namespace

bool narrow_ok(int cc, int co, int kvol) { return narrow_out_ok(cc, co, kvol) || narrow_in_ok(cc, co, kvol); }

// A tenth between the two estimates.  Of 10000 launches that the fit had not seen, 63 are slower than on the tile kernel by more than
// 10 % (935 if channels alone decide) and 157 left to it would be more than 20 % faster here.
bool narrow_pays(int cc, int co, int kvol, int64_t rows, int64_t links, sp_dtype dt) {
    const bool few_out = narrow_out_ok(cc, co, kvol);
    if (!few_out && !narrow_in_ok(cc, co, kvol)) return false;
    const Layer l{(double)rows, (double)links, (double)kvol, (double)cc, (double)co, dt == SP_F32};
    return 1.1 * narrow_us(l, few_out) < tile_us(l, few_out);
}

int conv_narrow(const MapSide& side, int kvol, const void* d_f, const void* d_w, bool w_transposed, void* d_g, int cc, int co, sp_dtype dt,
                hipStream_t s) {
    NarrowArgs a;
    a.nbr = ptr<int32_t>(side.nbr);
    a.f = d_f;
    a.w = d_w;
    a.g = d_g;
    a.n_rows = side.n_rows;
    a.kvol = kvol;
    a.co = co;
    a.cc = cc;
    a.flip = side.flip ? 1 : 0;
    a.s_co = w_transposed ? 1 : cc;
    a.s_cc = w_transposed ? co : 1;
    if (narrow_out_ok(cc, co, kvol)) {
        const int rows = kThreads / (cc / 8);
        const size_t lds = (size_t)kvol * co * cc * 4;
#define SP_OUT(OM) \
    case OM: return dt == SP_F32 ? launch(narrow_out_kernel<float, OM>, a.n_rows, rows, lds, s, a) : launch(narrow_out_kernel<bf16_t, OM>, a.n_rows, rows, lds, s, a)
        switch (co) {
            SP_OUT(1);
            SP_OUT(2);
            SP_OUT(3);
            SP_OUT(4);
            SP_OUT(5);
            SP_OUT(6);
            SP_OUT(7);
            SP_OUT(8);
        }
#undef SP_OUT
    }
    if (narrow_in_ok(cc, co, kvol)) {
        const int oc = narrow_in_channels(a.n_rows, co);
        const int cop = (co + oc - 1) / oc * oc, rows = kThreads / (cop / oc);
        const size_t lds = (size_t)kvol * cc * cop * 4;
#define SP_IN_OC(CC, OC) \
    return dt == SP_F32 ? launch(narrow_in_kernel<float, CC, OC>, a.n_rows, rows, lds, s, a, cop) : launch(narrow_in_kernel<bf16_t, CC, OC>, a.n_rows, rows, lds, s, a, cop)
#define SP_IN(CC)                     \
    case CC:                          \
        if (oc == 8) SP_IN_OC(CC, 8); \
        SP_IN_OC(CC, 4)
        switch (cc) {
            SP_IN(1);
            SP_IN(2);
            SP_IN(3);
            SP_IN(4);
            SP_IN(5);
            SP_IN(6);
            SP_IN(7);
        }
#undef SP_IN
#undef SP_IN_OC
    }
    return fail(SP_ERR_UNSUPPORTED, "internal: no narrow kernel for %d -> %d channels", cc, co);
}

}  // namespace sp
