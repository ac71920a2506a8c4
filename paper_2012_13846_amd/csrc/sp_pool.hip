// Pooling over a kernel map: Eq. 2 with the weighted sum replaced by a reduction over the same neighbour set
// (the pooling layers that sit between the SparseConv blocks, Sec. III figure caption).  Both directions are
// destination-row stationary walks of the neighbour table: no atomics, fixed order, reproducible bits.
//   forward:  y[o,c]  = max / sum / mean over k with i = nbr_out[k][o] >= 0 of x[i,c]
//   backward: dx[i,c] = sum over k with o = nbr_in[k][i] >= 0 of  dy[o,c] * (max: the link is the one that gave
//             the maximum | sum: 1 | mean: 1 / links of o)
// Memory bound: a row of c channels is gathered once per link.  Two round trips per kBatch offsets, whatever their number:
// a thread requests the entries of kBatch offsets, then the rows that exist, and only then reduces.  (One offset at a
// time is a chain of two dependent loads per offset, and a 64-bit division per thread beside it.)
// Backward, the rows of a wavefront have their links at different offsets (one of 8 at 2 x 2 x 2, stride 2): a thread's
// u-th link goes out with the other rows' u-th, kSlots at a time, not one offset and so one row after the other.
// 2 x 2 x 2, stride 2, 64 bf16 channels, 0.37 M input rows: forward 37.7 -> 24.6 us; backward 42.9 -> 33.3 us by the batches,
// -> 25.4 us by the slots (compulsory bytes at a large copy's rate: 13 and 16 us).
#include <mutex>

#include "sp_internal.h"

namespace sp {
namespace {

typedef uint16_t bf16_t;
constexpr int kThreads = 256;
constexpr uint8_t kNoArg = 255;
constexpr int kSlots = 4;  // links of a row that the backward pass has in flight
constexpr int kBatch = 8;  // offsets whose entries, then rows, a thread has in flight (the whole of a 2 x 2 x 2 kernel)

__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(bf16_t v) { return __uint_as_float((uint32_t)v << 16); }
__device__ __forceinline__ void from_f32(float f, float* o) { *o = f; }
__device__ __forceinline__ void from_f32(float f, bf16_t* o) {  // round to nearest even; NaN stays NaN
    uint32_t u = __float_as_uint(f);
    *o = (u & 0x7fffffffu) > 0x7f800000u ? (bf16_t)((u >> 16) | 0x40) : (bf16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

// V channels (16 bytes) of one row
template <typename T, int V>
struct Vec {
    T v[V];
};
template <typename T, int V>
__device__ __forceinline__ Vec<T, V> load_vec(const T* p) {
    Vec<T, V> r;
    if constexpr (V * sizeof(T) == 16) {
        const uint4 raw = *reinterpret_cast<const uint4*>(p);
        __builtin_memcpy(&r, &raw, 16);
    } else {
#pragma unroll
        for (int i = 0; i < V; ++i) r.v[i] = p[i];
    }
    return r;
}
template <typename T, int V>
__device__ __forceinline__ void store_vec(T* p, const Vec<T, V>& r) {
    if constexpr (V * sizeof(T) == 16) {
        uint4 raw;
        __builtin_memcpy(&raw, &r, 16);
        *reinterpret_cast<uint4*>(p) = raw;
    } else {
#pragma unroll
        for (int i = 0; i < V; ++i) p[i] = r.v[i];
    }
}

// Nothing is done with r before this point: what the compiler moves up to the load (unpacking) would wait for it there.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
template <typename T, int V>
__device__ __forceinline__ void arrive(Vec<T, V>& r) {
    if constexpr (V * sizeof(T) == 16) {
        u32x4 raw;
        __builtin_memcpy(&raw, &r, 16);
        asm volatile("" : "+v"(raw));
        __builtin_memcpy(&r, &raw, 16);
    }
}
// V offset numbers as one word, whatever their address; kept as a word for the same reason
template <int V>
struct ArgWord {
    typedef uint8_t type;
};
template <>
struct ArgWord<4> {
    typedef uint32_t type;
};
template <>
struct ArgWord<8> {
    typedef uint64_t type;
};
template <typename W>
__device__ __forceinline__ void arrive(W& w) {
    if constexpr (sizeof(W) >= 4) asm volatile("" : "+v"(w));
}

// This thread's (row, piece): the workgroup's first by one uniform division, the rest in 32 bits (pieces <= 65536).
__device__ __forceinline__ int64_t row_and_piece(int pieces, int* piece) {
    const int64_t t0 = (int64_t)blockIdx.x * kThreads, row0 = t0 / pieces;
    const uint32_t t = (uint32_t)(t0 - row0 * pieces) + threadIdx.x, q = t / (uint32_t)pieces;
    *piece = (int)(t - q * (uint32_t)pieces);
    return row0 + q;
}

// The table entries of offsets k0 .. k0 + kBatch - 1 for one row, -1 past the last offset.  All of them have arrived on
// return: a wait for the next entry between two row requests would be a wait for the rows too.
__device__ __forceinline__ void load_entries(const int32_t* __restrict__ nbr, int64_t n_rows, int64_t row, int kvol, int flip,
                                             int k0, int32_t (&e)[kBatch]) {
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
        const int k = k0 + j < kvol ? k0 + j : kvol - 1;
        e[j] = nbr[(int64_t)(flip ? kvol - 1 - k : k) * n_rows + row];
    }
#pragma unroll
    for (int j = 0; j < kBatch; ++j) e[j] = k0 + j < kvol ? e[j] : -1;
    asm volatile("" : "+v"(e[0]), "+v"(e[1]), "+v"(e[2]), "+v"(e[3]), "+v"(e[4]), "+v"(e[5]), "+v"(e[6]), "+v"(e[7]));
}
static_assert(kBatch == 8, "load_entries names its entries");

// links per destination row of a neighbour table
__global__ __launch_bounds__(kThreads) void link_count_kernel(const int32_t* __restrict__ nbr, int64_t n_rows, int kvol,
                                                              int32_t* __restrict__ cnt) {
    const int64_t r = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (r >= n_rows) return;
    int c = 0;
    for (int k = 0; k < kvol; ++k) c += nbr[(int64_t)k * n_rows + r] >= 0 ? 1 : 0;
    cnt[r] = c;
}

// Thread = (destination row, piece of V channels); c = pieces * V.  Offsets are visited in ascending TRUE
// offset number (a table derived by the stride-1 symmetry holds offset kvol-1-kk in block kk), so that among
// equal maxima the lowest offset number wins.
template <typename T, int V, int MODE>
__global__ __launch_bounds__(kThreads) void pool_fwd_kernel(const int32_t* __restrict__ nbr, int64_t n_rows, int kvol,
                                                            int flip, const T* __restrict__ x, int c, int pieces,
                                                            T* __restrict__ y, uint8_t* __restrict__ arg) {
    int piece;
    const int64_t row = row_and_piece(pieces, &piece);
    if (row >= n_rows) return;
    const int c0 = piece * V;
    float acc[V];
    Vec<uint8_t, V> best;
#pragma unroll
    for (int i = 0; i < V; ++i) {
        acc[i] = 0.f;
        best.v[i] = kNoArg;
    }
    int links = 0;
    for (int k0 = 0; k0 < kvol; k0 += kBatch) {
        int32_t src[kBatch];
        load_entries(nbr, n_rows, row, kvol, flip, k0, src);
        Vec<T, V> v[kBatch] = {};
#pragma unroll
        for (int j = 0; j < kBatch; ++j)
            if (src[j] >= 0) v[j] = load_vec<T, V>(x + (size_t)src[j] * c + c0);
#pragma unroll
        for (int j = 0; j < kBatch; ++j) arrive(v[j]);
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            if (src[j] < 0) continue;
            ++links;
#pragma unroll
            for (int i = 0; i < V; ++i) {
                const float f = to_f32(v[j].v[i]);
                if constexpr (MODE == SP_POOL_MAX) {
                    if (best.v[i] == kNoArg || f > acc[i]) {
                        acc[i] = f;
                        best.v[i] = (uint8_t)(k0 + j);
                    }
                } else {
                    acc[i] += f;
                }
            }
        }
    }
    Vec<T, V> out;
    const float scale = (MODE == SP_POOL_AVG && links > 0) ? 1.f / (float)links : 1.f;
#pragma unroll
    for (int i = 0; i < V; ++i) from_f32(MODE == SP_POOL_AVG ? acc[i] * scale : acc[i], &out.v[i]);
    store_vec<T, V>(y + (size_t)row * c + c0, out);
    if (MODE == SP_POOL_MAX && arg) {
#pragma unroll
        for (int i = 0; i < V; ++i) arg[(size_t)row * c + c0 + i] = best.v[i];
    }
}

// Thread = (input row, piece).  nbr is the input side's table: nbr[kk][i] = output row linked at (table block kk).
template <typename T, int V, int MODE>
__global__ __launch_bounds__(kThreads) void pool_bwd_kernel(const int32_t* __restrict__ nbr, int64_t n_rows, int kvol,
                                                            int flip, const T* __restrict__ dy, const uint8_t* __restrict__ arg,
                                                            const int32_t* __restrict__ link_cnt, int c, int pieces,
                                                            T* __restrict__ dx) {
    int piece;
    const int64_t row = row_and_piece(pieces, &piece);
    if (row >= n_rows) return;
    const int c0 = piece * V;
    float acc[V];
#pragma unroll
    for (int i = 0; i < V; ++i) acc[i] = 0.f;
    for (int k0 = 0; k0 < kvol; k0 += kBatch) {
        int32_t o[kBatch];
        load_entries(nbr, n_rows, row, kvol, flip, k0, o);
        uint32_t live = 0;
#pragma unroll
        for (int j = 0; j < kBatch; ++j) live |= o[j] >= 0 ? 1u << j : 0u;
        while (live) {
            Vec<T, V> g[kSlots] = {};
            typename ArgWord<V>::type a[kSlots] = {};
            int32_t links[kSlots] = {}, at[kSlots];
#pragma unroll
            for (int u = 0; u < kSlots; ++u) {  // the next link of this row, whatever its offset
                at[u] = live ? __ffs(live) - 1 : -1;
                live &= live - 1;
                int32_t src = o[0];
#pragma unroll
                for (int j = 1; j < kBatch; ++j) src = at[u] == j ? o[j] : src;
                if (at[u] < 0) continue;
                const size_t e = (size_t)src * c + c0;
                g[u] = load_vec<T, V>(dy + e);
                if constexpr (MODE == SP_POOL_MAX) __builtin_memcpy(&a[u], arg + e, V);
                if constexpr (MODE == SP_POOL_AVG) links[u] = link_cnt[src];  // the output has at least this link
            }
#pragma unroll
            for (int u = 0; u < kSlots; ++u) {
                arrive(g[u]);
                if constexpr (MODE == SP_POOL_MAX) arrive(a[u]);
            }
#pragma unroll
            for (int u = 0; u < kSlots; ++u) {
                if (at[u] < 0) continue;
                const float scale = MODE == SP_POOL_AVG ? 1.f / (float)links[u] : 1.f;
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    if constexpr (MODE == SP_POOL_MAX) {
                        if ((uint8_t)(a[u] >> (8 * i)) == (uint8_t)(k0 + at[u])) acc[i] += to_f32(g[u].v[i]);
                    } else if constexpr (MODE == SP_POOL_AVG) {
                        acc[i] += to_f32(g[u].v[i]) * scale;
                    } else {
                        acc[i] += to_f32(g[u].v[i]);
                    }
                }
            }
        }
    }
    Vec<T, V> out;
#pragma unroll
    for (int i = 0; i < V; ++i) from_f32(acc[i], &out.v[i]);
    store_vec<T, V>(dx + (size_t)row * c + c0, out);
}

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + kThreads - 1) / kThreads); }

template <typename T, int V>
int fwd_typed(const MapSide& side, int kvol, const void* x, void* y, uint8_t* arg, int c, int mode, hipStream_t s) {
    const int pieces = c / V;
    const int64_t n = side.n_rows * pieces;
    if (n == 0) return SP_OK;
    const dim3 g(blocks_for(n)), b(kThreads);
    const int32_t* nbr = ptr<int32_t>(side.nbr);
    const int flip = side.flip ? 1 : 0;
#define SP_GO(M)                                                                                                    \
    hipLaunchKernelGGL((pool_fwd_kernel<T, V, M>), g, b, 0, s, nbr, side.n_rows, kvol, flip, static_cast<const T*>(x), c, \
                       pieces, static_cast<T*>(y), arg)
    if (mode == SP_POOL_MAX) SP_GO(SP_POOL_MAX);
    else if (mode == SP_POOL_AVG) SP_GO(SP_POOL_AVG);
    else SP_GO(SP_POOL_SUM);
#undef SP_GO
    SP_HIP(hipGetLastError());
    return SP_OK;
}

template <typename T, int V>
int bwd_typed(const MapSide& side, int kvol, const void* dy, const uint8_t* arg, const int32_t* cnt, void* dx, int c,
              int mode, hipStream_t s) {
    const int pieces = c / V;
    const int64_t n = side.n_rows * pieces;
    if (n == 0) return SP_OK;
    const dim3 g(blocks_for(n)), b(kThreads);
    const int32_t* nbr = ptr<int32_t>(side.nbr);
    const int flip = side.flip ? 1 : 0;
#define SP_GO(M)                                                                                                     \
    hipLaunchKernelGGL((pool_bwd_kernel<T, V, M>), g, b, 0, s, nbr, side.n_rows, kvol, flip, static_cast<const T*>(dy), arg, \
                       cnt, c, pieces, static_cast<T*>(dx))
    if (mode == SP_POOL_MAX) SP_GO(SP_POOL_MAX);
    else if (mode == SP_POOL_AVG) SP_GO(SP_POOL_AVG);
    else SP_GO(SP_POOL_SUM);
#undef SP_GO
    SP_HIP(hipGetLastError());
    return SP_OK;
}

int check_pool_args(const sp_kmap_t* m, const void* a, int64_t rows_a, const void* b, int64_t rows_b, int c, int mode,
                    sp_dtype dt) {
    if (!m) return fail(SP_ERR_INVALID_ARG, "kmap handle is NULL");
    if (c < 1 || c > 65536) return fail(SP_ERR_INVALID_ARG, "bad channel count");
    if (dt != SP_F32 && dt != SP_BF16) return fail(SP_ERR_INVALID_ARG, "bad dtype");
    if (mode != SP_POOL_MAX && mode != SP_POOL_AVG && mode != SP_POOL_SUM) return fail(SP_ERR_INVALID_ARG, "bad pooling mode");
    if (m->kvol > 254) return fail(SP_ERR_UNSUPPORTED, "kernel volume above 254");
    if ((!a && rows_a > 0) || (!b && rows_b > 0)) return fail(SP_ERR_INVALID_ARG, "a feature pointer is NULL");
    return SP_OK;
}

// 16-byte vectors when the channel count and the pointers allow it, else one channel per thread
bool vector_ok(const void* a, const void* b, int c, sp_dtype dt) {
    const int v = dt == SP_F32 ? 4 : 8;
    return c % v == 0 && (((uintptr_t)a | (uintptr_t)b) & 15) == 0;
}

}  // namespace
}  // namespace sp

using namespace sp;

extern "C" {

int sp_pool_fwd(const sp_kmap_t* m, const void* d_x, void* d_y, uint8_t* d_arg, int32_t c, sp_pool_mode mode, sp_dtype dt,
                void* stream) {
    if (!m) return fail(SP_ERR_INVALID_ARG, "kmap handle is NULL");
    SP_TRY(kmap_resolve(m));
    SP_TRY(check_pool_args(m, d_x, m->n_in, d_y, m->n_out, c, mode, dt));
    hipStream_t s = (hipStream_t)stream;
    const MapSide& side = m->out_side;
    if (vector_ok(d_x, d_y, c, dt))
        return dt == SP_F32 ? fwd_typed<float, 4>(side, m->kvol, d_x, d_y, d_arg, c, mode, s)
                            : fwd_typed<bf16_t, 8>(side, m->kvol, d_x, d_y, d_arg, c, mode, s);
    return dt == SP_F32 ? fwd_typed<float, 1>(side, m->kvol, d_x, d_y, d_arg, c, mode, s)
                        : fwd_typed<bf16_t, 1>(side, m->kvol, d_x, d_y, d_arg, c, mode, s);
}

int sp_pool_bwd(const sp_kmap_t* m, const void* d_dy, const uint8_t* d_arg, void* d_dx, int32_t c, sp_pool_mode mode,
                sp_dtype dt, void* stream) {
    if (!m) return fail(SP_ERR_INVALID_ARG, "kmap handle is NULL");
    SP_TRY(kmap_resolve(m));
    SP_TRY(check_pool_args(m, d_dy, m->n_out, d_dx, m->n_in, c, mode, dt));
    if (mode == SP_POOL_MAX && !d_arg && m->n_out > 0) return fail(SP_ERR_INVALID_ARG, "max pooling backward needs d_arg");
    hipStream_t s = (hipStream_t)stream;
    const MapSide& side = m->in_side;
    const int32_t* cnt = nullptr;
    if (mode == SP_POOL_AVG && m->n_out > 0) {
        // links per output row: counted once per handle, on the first call that needs them
        std::lock_guard<std::mutex> lk(m->cache_mu);
        if (!m->out_link_cnt) {
            m->out_link_cnt = dev_alloc((size_t)m->n_out * 4, s);
            if (!m->out_link_cnt) return SP_ERR_ALLOC;
            hipLaunchKernelGGL(link_count_kernel, dim3(blocks_for(m->n_out)), dim3(kThreads), 0, s,
                               ptr<int32_t>(m->out_side.nbr), m->n_out, m->kvol, ptr<int32_t>(m->out_link_cnt));
            SP_HIP(hipGetLastError());
        }
        cnt = ptr<int32_t>(m->out_link_cnt);
    }
    if (vector_ok(d_dy, d_dx, c, dt))
        return dt == SP_F32 ? bwd_typed<float, 4>(side, m->kvol, d_dy, d_arg, cnt, d_dx, c, mode, s)
                            : bwd_typed<bf16_t, 8>(side, m->kvol, d_dy, d_arg, cnt, d_dx, c, mode, s);
    return dt == SP_F32 ? bwd_typed<float, 1>(side, m->kvol, d_dy, d_arg, cnt, d_dx, c, mode, s)
                        : bwd_typed<bf16_t, 1>(side, m->kvol, d_dy, d_arg, cnt, d_dx, c, mode, s);
}

}  // extern "C"
