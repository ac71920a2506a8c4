// Coordinate sets: duplicate merging in first-occurrence order through a grid or a hash table (sp_hash.h), strided
// (coarser) coordinate generation.  Sec. III-B: sparse tensor definition and step 1.
//
// No host round trip.  Up to kSmallRows one workgroup does everything in one launch, with the hash table in LDS.  Up to
// kGridRows (where every launch counts): reset the hash table, insert every row (slot.first = smallest row carrying
// the key), number, inverse.  Larger sets: the extent of the coordinates (a coarser set takes its parent's), prepare
// (every workgroup derives the grid's box, or that a hash table is needed, and clears that table), mark the occupied
// blocks (or insert into the hash table), number the blocks and clear their cells, put the smallest row of each cell
// into it, number, inverse.
// A set of half the resolution (floor step = twice the parent's lattice step) whose parent is a grid needs no atomics at all: a
// block of the parent's grid holds two coarse cells whole, so one thread sees all rows of a cell (mark_coarse_kernel) and
// knows the first of them; number and inverse read what it left.
// number: from 65537 to 2^21 rows in two passes over tiles of rows (firsts_kernel, rank_kernel), otherwise in one: every block of
// rows counts its first occurrences, gets the count of all earlier blocks by decoupled look-back, ranks its rows with ballots
// and writes coordinates + row numbers; the last block writes the row count N to device memory for later kernels and to a
// mail slot for the host.  inverse: the row number of every source row.  The host learns N when it first asks
// (coords_resolve).
#include <algorithm>

#include "sp_hash.h"
#include "sp_internal.h"
#include "sp_lookback.h"

namespace sp {
namespace {

constexpr int kThreads = 256;
constexpr int kRowsPerThread = 4;
constexpr int kNumberThreads = 1024;           // most threads of a numbering block; threads of the one that builds a small set
constexpr int64_t kSmallRows = 8192;           // up to here one workgroup (8 rows a thread, keys and slots in LDS)
constexpr int kSmallSlots = 16384;             // most slots of its table
// Up to here a hash table: four launches instead of seven.  Coordinates / + K = 3 map / + 2 x 2 x 2 stride 2 map in us, hash
// (eight slots a row) against grid: 46.7 k rows 25 / 46 / 67 against 37 / 52 / 86, 65 k 27 / 55 / 70 against 39 / 54 / 88,
// 82 k 32 / 65 / 78 against 43 / 60 / 92, 130 k 38 / 81 / 92 against 48 / 70 / 102.
constexpr int64_t kGridRows = 65536;
constexpr int kBoxBlocks = 256;                // blocks of the extent kernel = threads of a prepare block
constexpr int kBoxWords = 12;                  // min and max of b, x, y, z; out of range; off the lattice
constexpr int kScanThreads = 1024;
constexpr int kScanWords = 16 * kScanThreads;  // dir words numbered by one block
constexpr int64_t kFewScanWords = 2 << 20;     // up to here blocks of a quarter of that

__device__ __forceinline__ int32_t floor_to_multiple(int32_t v, int32_t s) {
    int32_t q = v / s;
    if ((v % s != 0) && (v < 0)) --q;  // s > 0: true floor, not truncation
    return q * s;
}

__device__ __forceinline__ int4 load_row(const int4* __restrict__ src, int64_t i, int32_t floor_step) {
    int4 c = src[i];
    if (floor_step > 1) {
        c.y = floor_to_multiple(c.y, floor_step);
        c.z = floor_to_multiple(c.z, floor_step);
        c.w = floor_to_multiple(c.w, floor_step);
    }
    return c;
}

// the source row count: a host value, or a count in device memory that the host has not seen yet
__device__ __forceinline__ int64_t row_count(int64_t n_host, const int32_t* __restrict__ d_n) {
    return d_n ? (int64_t)*d_n : n_host;
}

// The table while it is built.
struct Build {
    HashSlot* slots;
    uint32_t cap;
    int zshift;
    int32_t* dir;       // grid form; shares the memory of slots
    int32_t* cells;
    int64_t dir_words;  // room (whole blocks of the scan); 0: hash form for certain
    int32_t* meta;
    int ts;
};
__device__ __forceinline__ bool is_grid(const Build& t) { return t.dir_words > 0 && t.meta[kMetaGrid] != 0; }

__device__ __forceinline__ void clear_slot(HashSlot* slot) {
    uint4 v;
    v.x = 0xffffffffu;
    v.y = 0xffffffffu;
    v.z = (uint32_t)kNoRow;
    v.w = (uint32_t)-1;
    *reinterpret_cast<uint4*>(slot) = v;
}

// table slots <- empty; meta words and look-back words <- 0
__global__ __launch_bounds__(kThreads) void reset_kernel(HashSlot* __restrict__ tab, uint32_t cap,
                                                         int32_t* __restrict__ meta, unsigned long long* __restrict__ desc,
                                                         int64_t n_desc) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i < cap) clear_slot(&tab[i]);
    if (i < kMetaWords) meta[i] = 0;
    if (i < n_desc) desc[i] = 0ull;
}

// A small set in one launch: hash, merge, number, inverse, and the table written out as the searches read it.  Bound by
// latency: the four launches it replaces spent 25 us on 2048 rows, most of it in chains of dependent atomics on the
// fabric, which are LDS operations here.  Slot: -1, or the smallest source row of its key; once numbered, that row
// and its rank << 16.
__global__ __launch_bounds__(kNumberThreads) void small_build_kernel(const int4* __restrict__ src, int64_t n_host,
                                                                     const int32_t* __restrict__ d_n, int32_t floor_step, Build t,
                                                                     int4* __restrict__ coords, int32_t* __restrict__ inverse,
                                                                     uint32_t* __restrict__ mail, uint32_t mail_seq) {
    constexpr int kPer = (int)(kSmallRows / kNumberThreads);
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int s_row[kPer][kNumberThreads / 64];
    __shared__ int s_err;
    const int cap = (int)t.cap;
    int* slots = reinterpret_cast<int*>(smem);
    uint64_t* keys = reinterpret_cast<uint64_t*>(smem + (size_t)cap * 4);
    const int n = (int)row_count(n_host, d_n);
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    for (int i = tid; i < cap; i += kNumberThreads) slots[i] = -1;
    if (tid == 0) s_err = 0;
    int4 c[kPer];
    bool ok[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int i = j * kNumberThreads + tid;
        ok[j] = i < n;
        if (ok[j]) c[j] = load_row(src, i, floor_step);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        if (!ok[j]) continue;
        uint64_t key;
        ok[j] = pack_key(c[j].x, c[j].y, c[j].z, c[j].w, &key);
        if (ok[j]) keys[j * kNumberThreads + tid] = key;
        else s_err = 1;
    }
    __syncthreads();
    int at[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        at[j] = 0;
        if (!ok[j]) continue;
        const int i = j * kNumberThreads + tid;
        const uint64_t key = keys[i];
        uint32_t bucket, pos;
        hash_home(key, (uint32_t)cap, t.zshift, &bucket, &pos);
        int s = (int)(bucket * 4 + pos);
        for (int probe = 0; probe < cap; ++probe) {  // at most half of the slots are ever taken: an empty one is met
            int cur = slots[s];
            if (cur == -1) cur = atomicCAS(&slots[s], -1, i);
            if (cur == -1) break;
            if (keys[cur] == key) {
                if (cur > i) atomicMin(&slots[s], i);
                break;
            }
            s = (s + 1) & (cap - 1);
        }
        at[j] = s;
    }
    __syncthreads();
    bool f[kPer];
    int pos[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        f[j] = ok[j] && slots[at[j]] == j * kNumberThreads + tid;
        const unsigned long long m = __ballot(f[j]);
        pos[j] = __popcll(m & ((1ull << lane) - 1ull));
        if (lane == 0) s_row[j][w] = __popcll(m);
    }
    __syncthreads();
    int run = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        int mine = run;
        for (int ww = 0; ww < kNumberThreads / 64; ++ww) {
            if (ww < w) mine += s_row[j][ww];
            run += s_row[j][ww];
        }
        if (f[j]) {
            const int r = mine + pos[j];
            coords[r] = c[j];
            slots[at[j]] = (j * kNumberThreads + tid) | (r << 16);
        }
    }
    __syncthreads();
    if (tid == 0) {
        const int err = s_err;
        t.meta[kMetaN] = run;
        t.meta[kMetaErr] = err;
        t.meta[kMetaGrid] = 0;
        if (mail) {
            mail[0] = (uint32_t)run;
            mail[1] = (uint32_t)err;
            __threadfence_system();
            __hip_atomic_store(mail + kMailSeqWord, mail_seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int i = j * kNumberThreads + tid;
        if (i < n) inverse[i] = ok[j] ? slots[at[j]] >> 16 : -1;
    }
    for (int i = tid; i < cap; i += kNumberThreads) {
        const int v = slots[i];
        const uint64_t key = v >= 0 ? keys[v & 0xffff] : kEmptyKey;
        uint4 o;
        o.x = (uint32_t)key;
        o.y = (uint32_t)(key >> 32);
        o.z = (uint32_t)(v >= 0 ? v & 0xffff : kNoRow);
        o.w = (uint32_t)(v >= 0 ? v >> 16 : -1);
        *reinterpret_cast<uint4*>(&t.slots[i]) = o;
    }
}

// Extent of the source rows, per block: part[block][kBoxWords].
__global__ __launch_bounds__(kThreads) void box_kernel(const int4* __restrict__ src, int64_t n_host, const int32_t* __restrict__ d_n,
                                                       int ts, int32_t* __restrict__ part) {
    __shared__ int s_red[kThreads / 64][10];
    const int64_t n = row_count(n_host, d_n);
    int v[10];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        v[a] = 0x7fffffff;
        v[4 + a] = -0x7fffffff - 1;
    }
    v[8] = v[9] = 0;
    const int4 c0 = n > 0 ? src[0] : int4{0, 0, 0, 0};
    const int64_t stride = (int64_t)gridDim.x * kThreads;
    for (int64_t i0 = (int64_t)blockIdx.x * kThreads + threadIdx.x; i0 < n; i0 += 4 * stride) {
        int4 c[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) c[j] = src[min(i0 + j * stride, n - 1)];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int w[4] = {c[j].x, c[j].y, c[j].z, c[j].w};
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                v[a] = min(v[a], w[a]);
                v[4 + a] = max(v[4 + a], w[a]);
            }
            uint64_t key;
            if (!pack_key(w[0], w[1], w[2], w[3], &key)) v[8] = 1;
            else if (ts > 1 && ((w[1] - c0.y) % ts != 0 || (w[2] - c0.z) % ts != 0 || (w[3] - c0.w) % ts != 0)) v[9] = 1;
        }
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1)
#pragma unroll
        for (int a = 0; a < 10; ++a) {
            const int o = __shfl_xor(v[a], d, 64);
            v[a] = a < 4 ? min(v[a], o) : max(v[a], o);
        }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int a = 0; a < 10; ++a) s_red[w][a] = v[a];
    __syncthreads();
    if (threadIdx.x < 10) {
        const int a = threadIdx.x;
        int r = s_red[0][a];
        for (int j = 1; j < kThreads / 64; ++j) r = a < 4 ? min(r, s_red[j][a]) : max(r, s_red[j][a]);
        part[blockIdx.x * kBoxWords + a] = r;
    }
}

// Every block derives the box and the form of the table for itself and clears its share of it; block 0 writes meta.
// (512 blocks: 0.5 and 1 M rows 10.4 and 12.1 us with up to 2048, which all reduce the extents first, 5.6 and 8.8 so.)
// part: the extents box_kernel left, or null: the parent's box (parent_meta, lattice step parent_ts), floored to t.ts.
__global__ __launch_bounds__(kBoxBlocks) void prepare_kernel(Build t, int64_t n_host, const int32_t* __restrict__ d_n,
                                                             const int32_t* __restrict__ part,
                                                             const int32_t* __restrict__ parent_meta, int parent_ts,
                                                             unsigned long long* __restrict__ desc, int64_t n_desc) {
    __shared__ int s_red[kBoxBlocks / 64][10];
    __shared__ int s_box[10];
    const int tid = threadIdx.x;
    const int64_t n = row_count(n_host, d_n);
    if (part) {
        int v[10];
#pragma unroll
        for (int a = 0; a < 10; ++a) v[a] = part[tid * kBoxWords + a];
#pragma unroll
        for (int d = 32; d > 0; d >>= 1)
#pragma unroll
            for (int a = 0; a < 10; ++a) {
                const int o = __shfl_xor(v[a], d, 64);
                v[a] = a < 4 ? min(v[a], o) : max(v[a], o);
            }
        if ((tid & 63) == 0)
#pragma unroll
            for (int a = 0; a < 10; ++a) s_red[tid >> 6][a] = v[a];
        __syncthreads();
        if (tid < 10) {
            int r = s_red[0][tid];
            for (int j = 1; j < kBoxBlocks / 64; ++j) r = tid < 4 ? min(r, s_red[j][tid]) : max(r, s_red[j][tid]);
            s_box[tid] = r;
        }
    } else if (tid < 10) {
        const bool grid = parent_meta[kMetaGrid] != 0;
        int r = tid == 8 ? 0 : (grid ? 0 : 1);  // a parent that is no grid: word 9 sends this set to the hash form too
        if (grid && tid < 8) {
            const int a = tid & 3, low = parent_meta[kMetaLow + a];
            const int cells = parent_meta[kMetaExt + a] * (a == 0 ? 1 : (a == 3 ? 16 : 8));
            r = tid < 4 ? low : low + (cells - 1) * (a == 0 ? 1 : parent_ts);
            if (a > 0) r = floor_to_multiple(r, t.ts);
        }
        s_box[tid] = r;
    }
    __syncthreads();
    int64_t ext[4], words = 1;
    int low[4];
    bool ok = n > 0 && s_box[8] == 0 && s_box[9] == 0;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        ok = ok && s_box[a] >= (a == 0 ? 0 : -32768);
        // the lower half of a cell of twice the size: cells of a coarser set are whole in the grid's blocks
        low[a] = a > 0 && s_box[a] - floor_to_multiple(s_box[a], 2 * t.ts) >= t.ts ? s_box[a] - t.ts : s_box[a];
        const int64_t cells = ((int64_t)s_box[4 + a] - low[a]) / (a == 0 ? 1 : t.ts) + 1;
        ext[a] = a == 0 ? cells : (a == 3 ? (cells + 15) / 16 : (cells + 7) / 8);
        ok = ok && cells >= 1 && cells <= 65537;
    }
    if (ok) words = ext[0] * ext[1] * ext[2] * ext[3] * 64;
    ok = ok && words <= t.dir_words;
    const int64_t gid = (int64_t)blockIdx.x * kBoxBlocks + tid, stride = (int64_t)gridDim.x * kBoxBlocks;
    if (gid == 0) {
        t.meta[kMetaN] = 0;
        t.meta[kMetaErr] = s_box[8] != 0 ? 1 : 0;
        t.meta[kMetaGrid] = ok ? 1 : 0;
        t.meta[kMetaBlocks] = 0;
        for (int a = 0; a < 4; ++a) {
            t.meta[kMetaLow + a] = low[a];
            t.meta[kMetaExt + a] = ok ? (int)ext[a] : 0;
        }
    }
    for (int64_t i = gid; i < n_desc; i += stride) desc[i] = 0ull;
    if (ok) {
        const int64_t quads = (words + kScanWords - 1) / kScanWords * (kScanWords / 4);
        for (int64_t i = gid; i < quads; i += stride) reinterpret_cast<int4*>(t.dir)[i] = int4{-1, -1, -1, -1};
    } else {
        for (int64_t i = gid; i < (int64_t)t.cap; i += stride) clear_slot(&t.slots[i]);
    }
}

// Every source row inserts its key; slot.first becomes the smallest source row carrying that key.
__device__ __forceinline__ void insert_row(const Build& t, const int4& c, int64_t i, int always, int32_t* __restrict__ at) {
    uint64_t key;
    if (!pack_key(c.x, c.y, c.z, c.w, &key)) {
        atomicOr(t.meta + kMetaErr, 1);
        at[i] = -1;
        return;
    }
    bool fresh;
    const int64_t slot = hash_insert(t.slots, t.cap, t.zshift, key, &fresh);
    if (slot < 0) {
        atomicOr(t.meta + kMetaErr, 2);
        at[i] = -1;
        return;
    }
    // A duplicate that sees a smaller row already recorded has nothing to add (the value only ever decreases).
    // Looking first costs a round trip and saves an atomic: measured 5 us slower on 157 k rows, 50 us faster
    // on 4.1 M rows (where the atomics' throughput binds), so the host asks for it from 1 M rows (always = 0).
    if (always || fresh || __builtin_nontemporal_load(&t.slots[slot].first) > (int32_t)i) atomicMin(&t.slots[slot].first, (int32_t)i);
    at[i] = (int32_t)slot;
}

// Hash: insert.  Grid: the row's block is occupied (all rows of a block store the same word), at[i] = its cell.
__global__ __launch_bounds__(kThreads) void mark_kernel(const int4* __restrict__ src, int64_t n_host,
                                                        const int32_t* __restrict__ d_n, int32_t floor_step, Build t,
                                                        int32_t* __restrict__ at, int always) {
    const int64_t n = row_count(n_host, d_n);
    const int64_t tile = xcd_tile(blockIdx.x, (n + kThreads - 1) / kThreads), i = tile * kThreads + threadIdx.x;
    if (tile < 0 || i >= n) return;
    const int4 c = load_row(src, i, floor_step);
    if (!is_grid(t)) {
        insert_row(t, c, i, always, at);
        return;
    }
    const Grid g = load_grid(t.meta);
    int qx, qy, qz;
    lattice(c.y - g.x0, t.ts, &qx);
    lattice(c.z - g.y0, t.ts, &qy);
    lattice(c.w - g.z0, t.ts, &qz);
    const uint32_t blk = grid_block(g, c.x - g.b0, qx, qy, qz >> 2);
    t.dir[blk] = 0;
    at[i] = (int32_t)(blk * 16u + (uint32_t)(grid_run(qx, qy) * 4 + (qz & 3)));
}

// What a set of half the resolution takes from its parent's grid.
struct Halved {
    const int32_t* meta;   // the parent's; null: not such a set
    const int32_t* dir;
    const int32_t* cells;
    int ts;
    int32_t* rank_of;      // [2 * blocks of the parent]: row number of a pair's coarse cell
    int32_t* pair_of;      // [rows]: the pair a row came from; or null
};

// The parent's grid, block by block: a block of 2 x 2 x 4 cells is two coarse cells, "pair" 2 * block + half.  at[row of the
// parent] = its pair (its complement for a row that is not the first of its cell), and the coarse set's own block is occupied.
// One coalesced pass over the parent's dir and a line per occupied block, where marking, placing and numbering the rows one by
// one spent two scattered trips and an atomic each (0.5 M rows, 4 spheres: mark, place and number 43 us; this, firsts and rank 31).
// A coarse set that is a hash table: insert_row, as mark_kernel.
__global__ __launch_bounds__(kThreads) void mark_coarse_kernel(const int4* __restrict__ src, int64_t n_host, const int32_t* __restrict__ d_n,
                                                               int32_t floor_step, Build t, Halved hv, int32_t* __restrict__ at, int always) {
    const int64_t first = (int64_t)blockIdx.x * kThreads + threadIdx.x, stride = (int64_t)gridDim.x * kThreads;
    if (!is_grid(t)) {
        const int64_t n = row_count(n_host, d_n);
        for (int64_t i = first; i < n; i += stride) insert_row(t, load_row(src, i, floor_step), i, always, at);
        return;
    }
    const Grid pg = load_grid(hv.meta), g = load_grid(t.meta);  // a coarse set is a grid only if its parent is one
    // four blocks in a row along z; each XCD takes a stretch of them, i.e. a few clouds, whose rows' at words are its own
    const uint32_t quads = (uint32_t)pg.nb * pg.gx * pg.gy * pg.gz * 16u, per = (quads / 8 + 63) / 64 * 64 + 64;
    const uint32_t lo = (blockIdx.x & 7) * per, hi = min(lo + per, quads);
    for (uint32_t i = lo + (blockIdx.x >> 3) * kThreads + threadIdx.x; i < hi; i += gridDim.x / 8 * kThreads) {
        const int4 d4 = reinterpret_cast<const int4*>(hv.dir)[i];
        if ((d4.x & d4.y & d4.z & d4.w) < 0) continue;
        uint32_t group = i >> 4;
        const int bz0 = (int)(group % (uint32_t)pg.gz) * 4;
        group /= (uint32_t)pg.gz;
        const int by = (int)(group % (uint32_t)pg.gy) * 4 + (int)(i & 3u);
        group /= (uint32_t)pg.gy;
        const int bx = (int)(group % (uint32_t)pg.gx) * 4 + (int)(i >> 2 & 3u), qb = (int)(group / (uint32_t)pg.gx);
        const int qx = (floor_to_multiple(pg.x0 + 2 * bx * hv.ts, t.ts) - g.x0) / t.ts;
        const int qy = (floor_to_multiple(pg.y0 + 2 * by * hv.ts, t.ts) - g.y0) / t.ts;
        const int qz0 = (floor_to_multiple(pg.z0 + 4 * bz0 * hv.ts, t.ts) - g.z0) / t.ts;
        const int nums[4] = {d4.x, d4.y, d4.z, d4.w};
        int4 c[4][4];  // the cells of all four, requested together
#pragma unroll
        for (int z = 0; z < 4; ++z) {
            const int4* runs = reinterpret_cast<const int4*>(hv.cells) + (int64_t)nums[z] * 4;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                c[z][r] = int4{kNoRow, kNoRow, kNoRow, kNoRow};
                if (nums[z] >= 0) c[z][r] = runs[r];
            }
        }
#pragma unroll
        for (int z = 0; z < 4; ++z)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                int m[8];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    m[2 * r] = h ? c[z][r].z : c[z][r].x;
                    m[2 * r + 1] = h ? c[z][r].w : c[z][r].y;
                }
                int lowest = m[0];
#pragma unroll
                for (int j = 1; j < 8; ++j) lowest = min(lowest, m[j]);
                if (lowest == kNoRow) continue;
                const int pair = 2 * nums[z] + h;
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (m[j] != kNoRow) at[m[j]] = m[j] == lowest ? pair : ~pair;
                t.dir[grid_block(g, pg.b0 + qb - g.b0, qx, qy, (qz0 + 2 * z + h) >> 2)] = 0;
            }
    }
}

// Grid: occupied blocks are numbered, their cells cleared.  16 words a thread.  The numbers need no order (nothing
// that the build returns depends on them), so a workgroup takes as many as it needs from a counter: 12 ns per
// workgroup, where a look-back made the launch wait 8 us.  Scans stay inside the wavefronts but for one: 0.15, 0.5 and 1 M rows
// 7.7, 9.8 and 15.8 us with a scan of the whole workgroup for every four words, 6.2, 9.0 and 13.4 so; small sets in blocks of
// a quarter, which else fill 77 CUs.
__global__ __launch_bounds__(kScanThreads) void number_blocks_kernel(Build t) {
    __shared__ int s_base;
    __shared__ int s_wave[kScanThreads / 64];
    if (!is_grid(t)) return;
    const Grid g = load_grid(t.meta);
    const int64_t words = (int64_t)g.nb * g.gx * g.gy * g.gz * 64;
    const int nthreads = blockDim.x;
    if ((int64_t)blockIdx.x * 16 * nthreads >= words) return;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    // a wavefront takes 256 quads in a row, 64 at a time; its numbers follow quad by quad
    int4* q = reinterpret_cast<int4*>(t.dir + (int64_t)blockIdx.x * 16 * nthreads) + w * 256 + lane;
    int4 v[4];
    int pos[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = q[j * 64];
#pragma unroll
    for (int j = 0; j < 4; ++j) pos[j] = (v[j].x == 0) + (v[j].y == 0) + (v[j].z == 0) + (v[j].w == 0);
    int mine[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) mine[j] = pos[j];
#pragma unroll
    for (int d = 1; d < 64; d <<= 1)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int u = __shfl_up(pos[j], d, 64);
            if (lane >= d) pos[j] += u;
        }
    int total = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int all = __shfl(pos[j], 63, 64);
        pos[j] += total - mine[j];
        total += all;
    }
    if (lane == 0) s_wave[w] = total;
    __syncthreads();
    if (w == 0) {
        const int nw = nthreads / 64, own = lane < nw ? s_wave[lane] : 0;
        int inc = own;
#pragma unroll
        for (int d = 1; d < kScanThreads / 64; d <<= 1) {
            const int u = __shfl_up(inc, d, 64);
            if (lane >= d) inc += u;
        }
        if (lane < nw) s_wave[lane] = inc - own;
        if (lane == nw - 1) s_base = inc ? atomicAdd(t.meta + kMetaBlocks, inc) : 0;
    }
    __syncthreads();
    const int base = s_base + s_wave[w];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        int r = base + pos[j];
        if ((v[j].x & v[j].y & v[j].z & v[j].w) == -1) continue;  // none of the four is occupied
        if (v[j].x == 0) v[j].x = r++;
        if (v[j].y == 0) v[j].y = r++;
        if (v[j].z == 0) v[j].z = r++;
        if (v[j].w == 0) v[j].w = r++;
        q[j * 64] = v[j];
    }
    int4* cells = reinterpret_cast<int4*>(t.cells) + (int64_t)base * 4;  // each wavefront clears its own
    for (int i = lane; i < total * 4; i += 64) cells[i] = int4{kNoRow, kNoRow, kNoRow, kNoRow};
}

// Grid: at[i] becomes the row's place in cells (its complement for a row that is not the first of its cell), and the
// cell ends up with its smallest row.  A cell's value is one of its rows and only ever decreases, so a row that reads
// one smaller than itself, however old the copy it reads, can stay away: most duplicates spend no atomic.  (Plain
// stores followed by a pass of atomics for the rows that lost would be faster still, but two XCDs that store different
// values to one word are left with an L2 copy each, and later kernels have been seen to read both.)
__global__ __launch_bounds__(kThreads) void place_kernel(Build t, int64_t n_host, const int32_t* __restrict__ d_n,
                                                         int32_t* __restrict__ at) {
    if (!is_grid(t)) return;
    const int64_t n = row_count(n_host, d_n);
    // rows in ascending order over time, not dealt to the XCDs: a later row then mostly finds a smaller one in place
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    const uint32_t c = (uint32_t)at[i];
    const int32_t p = t.dir[c >> 4] * 16 + (int32_t)(c & 15u);
    const bool maybe = t.cells[p] > (int32_t)i;
    if (maybe) atomicMin(&t.cells[p], (int32_t)i);
    at[i] = maybe ? p : ~p;
}

// kGridRows < rows <= kTiledRows: which rows are the first of their cell (or key), a bit per row and a sum per tile of kTile
// rows.  Two launches, this and rank_kernel, since they may deal the rows to the XCDs in stretches, so that their scattered
// trips meet lines of one or two clouds' tables in that XCD's L2, and nobody looks back; number_kernel has to take its blocks
// in order.  us, number_kernel / these two: 0.16 M rows 13.0 / 12.3, 0.5 M 23.1 / 17.5, 1 M 24.6 / 20.3; a single cloud of
// 4.6 M 52 / 73 (its table is in no L2 by the second launch), so the largest sets stay with one launch.
constexpr int kTile = 1024;
constexpr int kTileWords = kTile / 64;
constexpr int64_t kTiledRows = 2 << 20;  // = 2048 tiles: each adds up the sums of those before it
__global__ __launch_bounds__(kThreads) void firsts_kernel(Build t, int64_t n_host, const int32_t* __restrict__ d_n, const int32_t* __restrict__ at,
                                                          int halved, unsigned long long* __restrict__ mask, int32_t* __restrict__ sums) {
    __shared__ int s_sum[kThreads / 64];
    const int64_t n = row_count(n_host, d_n);
    const int64_t tile = xcd_tile(blockIdx.x, (n + kTile - 1) / kTile);
    if (tile < 0) return;
    const bool grid = is_grid(t);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    constexpr int kPer = kTile / kThreads;
    const int64_t base = tile * kTile + threadIdx.x;
    int32_t s[kPer], first[kPer];
    int sum = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int64_t i = base + j * kThreads;
        s[j] = i < n ? at[i] : -1;
    }
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        first[j] = -1;
        if (s[j] >= 0) first[j] = !grid ? t.slots[s[j]].first : halved ? (int32_t)(base + j * kThreads) : t.cells[s[j]];
    }
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int64_t i = base + j * kThreads;
        const unsigned long long m = __ballot(s[j] >= 0 && first[j] == (int32_t)i);
        if (lane == 0 && i < n) mask[i >> 6] = m;
        sum += __popcll(m);
    }
    if (lane == 0) s_sum[w] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < kThreads / 64; ++i) sum += s_sum[i];
        sums[tile] = sum;
    }
}

// ... and their numbers: first rows of earlier tiles, of earlier 64-row stretches, of earlier lanes.  Writes the (floored)
// coordinates at that rank and the rank into the table; the last tile delivers the total.  (Grid: the rank replaces the row
// in the cell.)
__global__ __launch_bounds__(kThreads) void rank_kernel(const int4* __restrict__ src, int64_t n_host, const int32_t* __restrict__ d_n,
                                                        int32_t floor_step, Build t, const int32_t* __restrict__ at, Halved hv,
                                                        const unsigned long long* __restrict__ mask, const int32_t* __restrict__ sums,
                                                        int4* __restrict__ coords, uint32_t* __restrict__ mail, uint32_t mail_seq) {
    __shared__ int s_red[kThreads / 64];
    const int64_t n = row_count(n_host, d_n), tiles = (n + kTile - 1) / kTile;
    const int64_t tile = xcd_tile(blockIdx.x, tiles);
    if (tile < 0 && !(blockIdx.x == 0 && n == 0)) return;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    int run = 0;
    for (int64_t i0 = tid; i0 < tile; i0 += 4 * kThreads) {  // four loads at a time
        int v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = i0 + i * kThreads < tile ? sums[i0 + i * kThreads] : 0;
        run += (v[0] + v[1]) + (v[2] + v[3]);
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) run += __shfl_xor(run, d, 64);
    if (lane == 0) s_red[w] = run;
    __syncthreads();
    run = 0;
    for (int i = 0; i < kThreads / 64; ++i) run += s_red[i];
    const bool grid = is_grid(t), halved = grid && hv.meta;
    const Grid g = load_grid(t.meta);
    if (tile >= 0) {
        constexpr int kPer = kTile / kThreads;
        const int64_t base = tile * kTile;
        // lane l: the bits of the tile's 64-row stretch l (16 of them), and how many there are before them
        const unsigned long long mine = lane < kTileWords && base + 64 * lane < n ? mask[(base >> 6) + lane] : 0ull;
        const int cnt = __popcll(mine);
        int inc = cnt;
#pragma unroll
        for (int d = 1; d < kTileWords; d <<= 1) {
            const int u = __shfl_up(inc, d, 64);
            if (lane >= d) inc += u;
        }
        const int total = __shfl(inc, kTileWords - 1, 64);
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int word = j * (kThreads / 64) + w;
            const unsigned long long m = ((unsigned long long)(unsigned)__shfl((int)(mine >> 32), word, 64) << 32) | (unsigned)__shfl((int)mine, word, 64);
            const int before = __shfl(inc - cnt, word, 64);
            if (!(m >> lane & 1ull)) continue;
            const int64_t i = base + j * kThreads + tid;
            const int32_t r = run + before + __popcll(m & ((1ull << lane) - 1ull)), s = at[i];
            const int4 co = load_row(src, i, floor_step);
            coords[r] = co;
            if (halved) {
                int qx, qy, qz;
                lattice(co.y - g.x0, t.ts, &qx);
                lattice(co.z - g.y0, t.ts, &qy);
                lattice(co.w - g.z0, t.ts, &qz);
                t.cells[(int64_t)t.dir[grid_block(g, co.x - g.b0, qx, qy, qz >> 2)] * 16 + grid_run(qx, qy) * 4 + (qz & 3)] = r;
                hv.rank_of[s] = r;
                if (hv.pair_of) hv.pair_of[r] = s;
            } else if (grid) {
                t.cells[s] = r;
            } else {
                t.slots[s].row = r;
            }
        }
        run += total;
    }
    if (tile == tiles - 1 && tid == 0) {  // (no rows at all: tile -1 of 0)
        t.meta[kMetaN] = run;
        if (mail) {
            mail[0] = (uint32_t)run;
            mail[1] = (uint32_t)__hip_atomic_load(t.meta + kMetaErr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __threadfence_system();
            __hip_atomic_store(mail + kMailSeqWord, mail_seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

// Middle-sized sets (always a hash table) and the largest, in one launch.
// Block b numbers the first occurrences among its rows: rank = (first occurrences in earlier blocks, by look-back) +
// (those before it in this block, row order).  Writes the (floored) coordinates at that rank and the rank into the
// table.  The block holding the last rows delivers the total.
// (Grid: the rank replaces the row in the cell.  It is smaller than every later row of the cell, so none of those
// takes itself for the first.)
__global__ __launch_bounds__(kNumberThreads) void number_kernel(const int4* __restrict__ src, int64_t n_host,
                                                                const int32_t* __restrict__ d_n, int32_t floor_step, Build t,
                                                                const int32_t* __restrict__ at,
                                                                unsigned long long* __restrict__ desc,
                                                                int4* __restrict__ coords, uint32_t* __restrict__ mail,
                                                                uint32_t mail_seq) {
    __shared__ int s_own, s_before;  // first occurrences in this block, in all earlier ones
    __shared__ int s_row[kRowsPerThread * (kNumberThreads / 64)];  // first occurrences in earlier 64-row stretches of the block
    static_assert(kRowsPerThread * (kNumberThreads / 64) <= 64, "one wavefront scans them");
    const int nthreads = blockDim.x, nw = nthreads >> 6;
    const int rows = nthreads * kRowsPerThread;
    const int64_t n = row_count(n_host, d_n);
    const int64_t nb = (n + rows - 1) / rows;
    const int b = blockIdx.x;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int32_t* meta = t.meta;
    if (b >= nb) {
        if (b == 0 && threadIdx.x == 0) {  // no rows at all: block 0 reports N = 0
            meta[kMetaN] = 0;
            if (mail) {
                mail[0] = 0u;
                mail[1] = (uint32_t)meta[kMetaErr];
                __threadfence_system();
                __hip_atomic_store(mail + kMailSeqWord, mail_seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
            }
        }
        return;
    }
    const bool grid = is_grid(t);
    const int64_t base = (int64_t)b * rows;
    bool f[kRowsPerThread];
    int pos[kRowsPerThread];
    int32_t s[kRowsPerThread], first[kRowsPerThread];
#pragma unroll
    for (int j = 0; j < kRowsPerThread; ++j) {
        const int64_t i = base + j * nthreads + threadIdx.x;
        s[j] = i < n ? at[i] : -1;
    }
#pragma unroll
    for (int j = 0; j < kRowsPerThread; ++j) {
        first[j] = -1;
        if (s[j] >= 0) first[j] = grid ? t.cells[s[j]] : t.slots[s[j]].first;
    }
#pragma unroll
    for (int j = 0; j < kRowsPerThread; ++j) {
        f[j] = s[j] >= 0 && first[j] == (int32_t)(base + j * nthreads + threadIdx.x);
        const unsigned long long m = __ballot(f[j]);
        pos[j] = __popcll(m & ((1ull << lane) - 1ull));
        if (lane == 0) s_row[j * nw + w] = __popcll(m);
    }
    __syncthreads();
    if (threadIdx.x < 64) {
        const int v = lane < kRowsPerThread * nw ? s_row[lane] : 0;
        int inc = v;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int u = __shfl_up(inc, d, 64);
            if (lane >= d) inc += u;
        }
        if (lane < kRowsPerThread * nw) s_row[lane] = inc - v;
        const int own = __shfl(inc, 63, 64), earlier = lookback(desc, b, own, meta + kMetaErr);
        if (lane == 0) {
            s_own = own;
            s_before = earlier;
        }
    }
    __syncthreads();
    const int before = s_before;
#pragma unroll
    for (int j = 0; j < kRowsPerThread; ++j) {
        if (f[j]) {
            const int32_t r = before + s_row[j * nw + w] + pos[j];
            coords[r] = load_row(src, base + j * nthreads + threadIdx.x, floor_step);
            if (grid) t.cells[s[j]] = r;
            else t.slots[s[j]].row = r;
        }
    }
    if (b == nb - 1 && threadIdx.x == 0) {
        const int run = before + s_own;
        meta[kMetaN] = run;
        if (mail) {
            mail[0] = (uint32_t)run;
            mail[1] = (uint32_t)__hip_atomic_load(meta + kMetaErr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __threadfence_system();
            __hip_atomic_store(mail + kMailSeqWord, mail_seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

__global__ __launch_bounds__(kThreads) void inverse_kernel(Build t, const int32_t* __restrict__ at, Halved hv, int64_t n_host,
                                                           const int32_t* __restrict__ d_n, int32_t* __restrict__ inverse) {
    const int64_t n = row_count(n_host, d_n);
    const int64_t tile = xcd_tile(blockIdx.x, (n + kThreads - 1) / kThreads), i = tile * kThreads + threadIdx.x;
    if (tile < 0 || i >= n) return;
    const int32_t s = at[i];
    inverse[i] = is_grid(t) ? (hv.meta ? hv.rank_of : t.cells)[s < 0 ? ~s : s] : (s < 0 ? -1 : t.slots[s].row);
}

inline unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

TableView table_view(const sp_coords* c) {
    TableView v;
    v.slots = ptr<HashSlot>(c->tab.mem);
    v.cap = c->tab.cap;
    v.zshift = c->tab.zshift;
    v.meta = ptr<int32_t>(c->meta);
    v.dir = ptr<int32_t>(c->tab.mem);
    v.cells = v.dir + c->tab.dir_words;
    v.ts = c->ts;
    v.maybe_grid = c->tab.dir_words > 0 ? 1 : 0;
    return v;
}

int coords_build_impl(const int32_t* d_src, int64_t n_src, const int32_t* d_n_src, int32_t floor_step,
                      int32_t tensor_stride, const sp_coords* parent, bool want_pairs, hipStream_t s, sp_coords_t** out) {
    if (n_src >= (int64_t)1 << 30) return fail(SP_ERR_INVALID_ARG, "too many rows (%lld)", (long long)n_src);
    std::unique_ptr<sp_coords> c(new sp_coords);
    c->n_raw = n_src;
    c->ts = tensor_stride;
    c->on_lattice = floor_step % tensor_stride == 0;
    c->stream = s;
    const bool small = n_src <= kSmallRows;
    // A grid: 32 bytes of dir per source row (128 cells of the box; 4 MB at least), whole scan blocks, and 64 bytes per
    // block that can be occupied.  Cell numbers have to fit 32 bits, places in cells 31.
    int64_t dir_words = 0;
    if (n_src > kGridRows && n_src < ((int64_t)1 << 26) && (!parent || parent->tab.dir_words > 0))
        dir_words = std::min<int64_t>((std::max<int64_t>(8 * n_src, 1 << 20) + kScanWords - 1) / kScanWords * kScanWords, (int64_t)1 << 28);
    const bool may_grid = dir_words > 0;
    c->tab.dir_words = dir_words;
    // Slots, a power of two.  Builds and searches wait for the longest chain of collisions among a wavefront's rows, so
    // room is time: eight per row for sets that take the hash form; where a grid is reserved (96 bytes a row) at least four
    // up to 2^20 rows (at most 128 bytes), three beyond, which take no more (262 k rows in a box too wide for a grid,
    // coordinates + K = 3 map: two a row 232 us, three 169; 160 k, 330 k: three 131, 225, four 119, 202, six 119, 202);
    // the largest sets, and what is made from them, room for every row at half load.
    uint32_t cap = 1024;
    while ((int64_t)cap < (n_src <= kGridRows ? 8 : (may_grid ? (n_src <= ((int64_t)1 << 20) ? 4 : 3) : 2)) * n_src) cap <<= 1;
    if (small) cap = std::min<uint32_t>(cap, kSmallSlots);
    c->tab.cap = cap;
    for (int t = tensor_stride; t > 1; t >>= 1) ++c->tab.zshift;
    const size_t grid_bytes = may_grid ? (size_t)dir_words * 4 + (size_t)n_src * 64 : 0;
    const bool tiled = n_src > kGridRows && n_src <= kTiledRows;  // numbered by firsts_kernel and rank_kernel
    const int nthreads = n_src > kTiledRows ? kNumberThreads : kThreads;
    const int block_rows = nthreads * kRowsPerThread;
    const int64_t nb = tiled ? 0 : (n_src + block_rows - 1) / block_rows;
    const int64_t tiles = tiled ? (n_src + kTile - 1) / kTile : 0;
    c->tab.mem = dev_alloc(std::max((size_t)cap * sizeof(HashSlot), grid_bytes), s);
    c->coords = dev_alloc((size_t)(n_src ? n_src : 1) * 16, s);
    c->inverse = dev_alloc((size_t)(n_src ? n_src : 1) * 4, s);
    c->meta = dev_alloc(kMetaWords * 4, s);
    // scratch: a slot or cell per source row; the look-back words; tiles: a bit per row and their sums; where a grid is possible: the
    // extents; for a set of half the resolution the row number of each pair of the parent's blocks (no more blocks than rows)
    const bool halved = tiled && may_grid && parent && floor_step == 2 * parent->ts;
    const size_t at_bytes = ((size_t)(n_src ? n_src : 1) * 4 + 15) / 16 * 16, mask_bytes = tiled ? ((size_t)n_src + 63) / 64 * 8 : 0;
    const int64_t n_desc = nb ? nb : 1;
    Buf scratch = small ? Buf() : dev_alloc(at_bytes + (size_t)n_desc * 8 + mask_bytes + (size_t)tiles * 4 +
                                                (may_grid ? kBoxBlocks * kBoxWords * 4 : 0) + (halved ? (size_t)n_src * 8 : 0), s);
    if (halved && want_pairs) {
        c->pairs = dev_alloc((size_t)n_src * 4, s);
        if (!c->pairs) return SP_ERR_ALLOC;
    }
    if (!c->tab.mem || !c->coords || !c->inverse || !c->meta || (!small && !scratch)) return SP_ERR_ALLOC;
    int32_t* at = ptr<int32_t>(scratch);
    unsigned long long* desc = small ? nullptr : reinterpret_cast<unsigned long long*>(ptr<unsigned char>(scratch) + at_bytes);
    Build t;
    t.slots = ptr<HashSlot>(c->tab.mem);
    t.cap = cap;
    t.zshift = c->tab.zshift;
    t.dir = ptr<int32_t>(c->tab.mem);
    t.cells = t.dir + dir_words;
    t.dir_words = dir_words;
    t.meta = ptr<int32_t>(c->meta);
    t.ts = tensor_stride;
    Halved hv{};
    if (halved) {
        hv.meta = ptr<int32_t>(parent->meta);
        hv.dir = ptr<int32_t>(parent->tab.mem);
        hv.cells = hv.dir + parent->tab.dir_words;
        hv.ts = parent->ts;
        hv.pair_of = ptr<int32_t>(c->pairs);
    }
    unsigned long long* mask = small ? nullptr : desc + n_desc;
    int32_t* sums = small ? nullptr : reinterpret_cast<int32_t*>(reinterpret_cast<unsigned char*>(mask) + mask_bytes);
    int32_t* part = small ? nullptr : sums + tiles;
    if (halved) hv.rank_of = part + kBoxBlocks * kBoxWords;
    const bool mailed = mail_acquire(&c->mail);
    const int4* src = reinterpret_cast<const int4*>(d_src);
    const dim3 rows(xcd_grid(blocks_for(n_src, kThreads))), threads(kThreads);
    const int always = n_src < (1 << 20) ? 1 : 0;

    auto hand_over = [&]() -> int {  // the last launch is enqueued
        c->mail.armed = mailed;
        c->mail.stream = s;
        SP_HIP(hipGetLastError());
        if (!mailed) {  // no mail slot free: wait here, the old way
            int32_t h[2] = {0, 0};
            SP_TRY(read_back(h, t.meta, 8, s));
            c->n = h[0];
            c->status = (h[1] & 1) ? SP_ERR_RANGE : (h[1] & 2) ? SP_ERR_TABLE_FULL : (h[1] & kErrLookback) ? SP_ERR_HIP : SP_OK;
            c->resolved = true;
        }
        *out = c.release();
        return SP_OK;
    };
    if (small) {
        const int lds = (int)cap * 4 + (int)(n_src ? n_src : 1) * 8;
        {
            static std::mutex mu;
            static bool attr_set = false;  // one-time opt-in to > 64 KB of dynamic LDS
            std::lock_guard<std::mutex> lk(mu);
            if (!attr_set) {
                SP_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(small_build_kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)(kSmallSlots * 4 + kSmallRows * 8)));
                attr_set = true;
            }
        }
        hipLaunchKernelGGL(small_build_kernel, dim3(1), dim3(kNumberThreads), lds, s, src, n_src, d_n_src, floor_step, t,
                           ptr<int4>(c->coords), ptr<int32_t>(c->inverse), mailed ? c->mail.d : (uint32_t*)nullptr, c->mail.seq);
        return hand_over();
    }
    if (may_grid) {
        if (!parent) hipLaunchKernelGGL(box_kernel, dim3(kBoxBlocks), threads, 0, s, src, n_src, d_n_src, tensor_stride, part);
        hipLaunchKernelGGL(prepare_kernel, dim3((unsigned)std::min<int64_t>(512, dir_words / 4 / kBoxBlocks)), dim3(kBoxBlocks), 0, s,
                           t, n_src, d_n_src, parent ? (const int32_t*)nullptr : part, parent ? ptr<int32_t>(parent->meta) : nullptr, parent ? parent->ts : 1, desc,
                           n_desc);
        if (halved)
            hipLaunchKernelGGL(mark_coarse_kernel, dim3(2048), threads, 0, s, src, n_src, d_n_src, floor_step, t, hv, at, always);
        else
            hipLaunchKernelGGL(mark_kernel, rows, threads, 0, s, src, n_src, d_n_src, floor_step, t, at, always);
        const int scan = dir_words <= kFewScanWords ? kScanThreads / 4 : kScanThreads;
        hipLaunchKernelGGL(number_blocks_kernel, dim3((unsigned)(dir_words / (16 * scan))), dim3(scan), 0, s, t);
        if (!halved) hipLaunchKernelGGL(place_kernel, rows, threads, 0, s, t, n_src, d_n_src, at);
    } else {
        hipLaunchKernelGGL(reset_kernel, dim3(blocks_for(std::max<int64_t>(cap, n_desc), kThreads)), threads, 0, s, t.slots, cap,
                           t.meta, desc, n_desc);
        hipLaunchKernelGGL(mark_kernel, rows, threads, 0, s, src, n_src, d_n_src, floor_step, t, at, always);
    }
    uint32_t* mail = mailed ? c->mail.d : nullptr;
    if (tiled) {
        const dim3 tile_grid(xcd_grid(tiles));
        hipLaunchKernelGGL(firsts_kernel, tile_grid, threads, 0, s, t, n_src, d_n_src, at, halved ? 1 : 0, mask, sums);
        hipLaunchKernelGGL(rank_kernel, tile_grid, threads, 0, s, src, n_src, d_n_src, floor_step, t, at, hv, mask, sums,
                           ptr<int4>(c->coords), mail, c->mail.seq);
    } else {
        hipLaunchKernelGGL(number_kernel, dim3((unsigned)nb), dim3(nthreads), 0, s, src, n_src, d_n_src, floor_step, t, at, desc, ptr<int4>(c->coords),
                           mail, c->mail.seq);
    }
    hipLaunchKernelGGL(inverse_kernel, rows, threads, 0, s, t, at, hv, n_src, d_n_src, ptr<int32_t>(c->inverse));
    return hand_over();
}

static int status_message(int status) {
    if (status == SP_ERR_RANGE) return fail(SP_ERR_RANGE, "a coordinate is outside 0 <= b < 65536, -32768 <= x,y,z < 32768");
    if (status == SP_ERR_TABLE_FULL) return fail(SP_ERR_TABLE_FULL, "hash table overflow");
    if (status == SP_ERR_HIP) return fail(SP_ERR_HIP, "internal: a look-back wait gave up");
    return status;
}

int coords_resolve(const sp_coords_t* c) {
    std::lock_guard<std::mutex> lk(c->mu);
    if (!c->resolved) {
        SP_TRY(mail_wait(c->mail, c->stream));
        const uint32_t n = c->mail.h[0], e = c->mail.h[1];
        c->n = (int64_t)n;
        c->status = (e & 1) ? SP_ERR_RANGE : (e & 2) ? SP_ERR_TABLE_FULL : (e & kErrLookback) ? SP_ERR_HIP : SP_OK;
        c->resolved = true;
        mail_release(&c->mail);
    }
    return status_message(c->status);
}

}  // namespace sp

sp_coords::~sp_coords() {
    sp::mail_release(&mail);
    if (src_of) sp_coords_destroy(src_of);
}

extern "C" {

int sp_coords_build(const int32_t* d_raw, int64_t n_raw, int32_t tensor_stride, void* stream, sp_coords_t** out) {
    if (!out) return sp::fail(SP_ERR_INVALID_ARG, "out is NULL");
    *out = nullptr;
    if (n_raw < 0) return sp::fail(SP_ERR_INVALID_ARG, "n_raw < 0");
    if (n_raw > 0 && !d_raw) return sp::fail(SP_ERR_INVALID_ARG, "d_raw is NULL");
    if (tensor_stride < 1) return sp::fail(SP_ERR_INVALID_ARG, "tensor_stride < 1");
    if (((uintptr_t)d_raw & 15) != 0) return sp::fail(SP_ERR_INVALID_ARG, "d_raw must be 16-byte aligned");
    return sp::coords_build_impl(d_raw, n_raw, nullptr, 1, tensor_stride, nullptr, false, (hipStream_t)stream, out);
}

int sp_coords_size(const sp_coords_t* c, int64_t* n, int32_t* tensor_stride) {
    if (!c) return sp::fail(SP_ERR_INVALID_ARG, "coords handle is NULL");
    if (tensor_stride) *tensor_stride = c->ts;
    if (n) {
        SP_TRY(sp::coords_resolve(c));
        *n = c->n;
    }
    return SP_OK;
}

int sp_coords_data(const sp_coords_t* c, const int32_t** d_coords, const int32_t** d_inverse, int64_t* n_raw) {
    if (!c) return sp::fail(SP_ERR_INVALID_ARG, "coords handle is NULL");
    if (d_coords) *d_coords = sp::ptr<int32_t>(c->coords);
    if (d_inverse) *d_inverse = sp::ptr<int32_t>(c->inverse);
    if (n_raw) {
        *n_raw = c->n_raw;
        if (c->src_of) {  // derived from a set whose row count may have been unknown then: its rows are the source rows
            SP_TRY(sp::coords_resolve(c->src_of));
            *n_raw = c->src_of->n;
        }
    }
    return SP_OK;
}

int sp_coords_destroy(sp_coords_t* c) {
    if (!c) return SP_OK;
    if (c->ref.fetch_sub(1) == 1) delete c;
    return SP_OK;
}

}  // extern "C"
