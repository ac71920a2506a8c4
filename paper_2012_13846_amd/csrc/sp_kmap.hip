// Kernel maps (Sec. III-B step 2): for every kernel offset the (input row, output row) pairs it links, found by
// searching the input coordinate set's table, then compacted with wavefront ballots and prefix sums into per-offset
// lists that the gather-GEMM kernels and the weight gradient read.
//
// No host round trip.  (1) The searches: one thread per output row and column of offsets fills the neighbour table
// and counts the links per (64-row sub-tile, offset); a workgroup is a tile of 1024 rows, so it also leaves the
// tile's sum per offset.  (2) emit: every tile adds up the sums of the tiles before it (up to kSumTiles of them; beyond
// that a prefix launch does it once for all) and writes its stretch of every offset's list; the last tile delivers the
// counts to device memory and to a mail slot, which the host reads when it first asks (kmap_resolve).  Row counts
// that the host has not seen yet (the input set's N, the coarse set's N) are read from device memory by the kernels;
// grids and allocations use upper bounds.  (A single-pass count + look-back + emit kernel was measured slower: the
// look-back's device-coherent loads cost ~2 us a round trip and a tile near the end of a launch that starts all at
// once needs several of them per offset.)
// The lists of an input side of its own (strided maps, even kernels) and its class order are made by the first call
// that walks them.
#include <algorithm>

#include "sp_hash.h"
#include "sp_internal.h"

namespace sp {
namespace {

constexpr int kThreads = 256;

// A row count: the host's value, or (d != null) a count in device memory that the host has not seen yet.
struct Count {
    const int32_t* d;
    int64_t h;
};
__device__ __forceinline__ int64_t get(const Count& c) { return c.d ? (int64_t)*c.d : c.h; }

// table[0, kvol * n) <- -1 (n may live on the device), 16 bytes a thread
__global__ __launch_bounds__(kThreads) void reset_kernel(int32_t* __restrict__ table, Count cn, int kvol) {
    const int64_t total = get(cn) * kvol, i = ((int64_t)blockIdx.x * kThreads + threadIdx.x) * 4;
    if (i + 4 <= total) *reinterpret_cast<int4*>(table + i) = int4{-1, -1, -1, -1};
    else
        for (int64_t j = i; j < total; ++j) table[j] = -1;
}

// Links per (tile, sub-tile, offset, 32-row half) and per (tile, offset): what emit_kernel places its entries by.
struct Counts {
    int32_t* cnt;  // [tile][sub][kvol][half]
    int32_t* agg;  // [kvol][pitch]: a wavefront sums an offset's row of them
    int32_t* pre;  // null, or [kvol][pitch + 1]: those sums (prefix_kernel)
    int64_t pitch;
};

// Up to this many tiles a workgroup adds up the tiles before its own by itself (no launch: 0.5 M rows, K = 1, 13 us against
// 17), beyond it prefix_kernel does it once, or the work would grow with the square of the rows: K = 1 on 1 M rows 18 us
// either way, 4.1 M 55 against 46, 16.8 M 346 against 182 (K = 3: 2560 against 2020).
constexpr int64_t kSumTiles = 1024;

// pre[row][t] = agg[row][0] + .. + agg[row][t - 1], t = 0 .. tiles.  A workgroup per row.  (Not in place: a build that is
// repeated on another stream writes the same words to the same places, and readers of either find what they expect.)
__global__ __launch_bounds__(kTileRows) void prefix_kernel(const int32_t* __restrict__ agg, int32_t* __restrict__ pre, int64_t pitch,
                                                           Count n_rows) {
    __shared__ int s_wave[2][kTileRows / 64];
    const int64_t tiles = (get(n_rows) + kTileRows - 1) / kTileRows;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    agg += blockIdx.x * pitch;
    pre += blockIdx.x * (pitch + 1);
    int run = 0;
    for (int64_t t0 = 0, turn = 0; t0 < tiles; t0 += 4 * kTileRows, ++turn) {
        const int64_t t = t0 + 4 * tid;
        int v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = t + i < tiles ? agg[t + i] : 0;
        const int mine = (v[0] + v[1]) + (v[2] + v[3]);
        int inc = mine;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int u = __shfl_up(inc, d, 64);
            if (lane >= d) inc += u;
        }
        int* sums = s_wave[turn & 1];  // the next turn's writes meet this turn's reads only beyond its barrier
        if (lane == 63) sums[w] = inc;
        __syncthreads();
        int at = run + inc - mine;
        for (int ww = 0; ww < kTileRows / 64; ++ww) {
            if (ww < w) at += sums[ww];
            run += sums[ww];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (t + i < tiles) pre[t + i] = at;
            at += v[i];
        }
    }
    if (tid == 0) pre[tiles] = run;
}

// A workgroup's share of the counts: offsets k(0) .. k(NO-1) of its tile, v[j] = this row's entry of the j-th.
template <int NO, class Koff>
__device__ __forceinline__ void count_rows(const Counts& c, int kvol, int64_t tile, const int32_t (&v)[NO], int (&s_cnt)[kSubTiles][NO][kHalves],
                                           Koff k_of) {
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
#pragma unroll
    for (int j = 0; j < NO; ++j) {
        const unsigned long long live = __ballot(v[j] >= 0);
        if (lane == 0) {
            s_cnt[w][j][0] = __popc((unsigned)live);
            s_cnt[w][j][1] = __popc((unsigned)(live >> 32));
        }
    }
    __syncthreads();
    if (tid < kSubTiles * NO) {
        const int ww = tid / NO, j = tid % NO, k = k_of(j);
        if (k < kvol) {
            int2 two;
            two.x = s_cnt[ww][j][0];
            two.y = s_cnt[ww][j][1];
            *reinterpret_cast<int2*>(c.cnt + (((tile * kSubTiles + ww) * kvol + k) * kHalves)) = two;
        }
    }
    if (tid >= 512 && tid < 512 + NO) {
        const int j = tid - 512, k = k_of(j);
        if (k < kvol) {
            int sum = 0;
            for (int ww = 0; ww < kSubTiles; ++ww) sum += s_cnt[ww][j][0] + s_cnt[ww][j][1];
            c.agg[k * c.pitch + tile] = sum;
        }
    }
}

// The K searches of one column (ax, ay) of offsets for one row, in the hash table.  They advance in lockstep: every
// turn issues the next slot's load of all searches still running and only then looks at the answers, so their memory
// latencies overlap (run one after the other, each costs as many round trips as the longest probe sequence among
// the 64 lanes).
template <int K>
__device__ __forceinline__ void search_hash(const TableView& t, const int4& c, int dx, int dy, int step, int skip, int32_t* v) {
    constexpr int centre = (K & 1) ? (K - 1) / 2 : 0;
    uint64_t key[K];
    uint32_t slot[K];
    bool run[K];
    bool any = false;
#pragma unroll
    for (int az = 0; az < K; ++az) {
        v[az] = -1;
        run[az] = pack_key(c.x, c.y + dx * step, c.z + dy * step, c.w + (az - centre) * step, &key[az]) && az != skip;
        uint32_t bucket, pos;
        hash_home(key[az], t.cap, t.zshift, &bucket, &pos);
        slot[az] = bucket * 4 + pos;
        any = any || run[az];
    }
    for (uint32_t turn = 0; any && turn < t.cap; ++turn) {
        uint4 raw[K];
#pragma unroll
        for (int az = 0; az < K; ++az)
            if (run[az]) raw[az] = *reinterpret_cast<const uint4*>(&t.slots[slot[az]]);
        any = false;
#pragma unroll
        for (int az = 0; az < K; ++az) {
            if (!run[az]) continue;
            const unsigned long long cur = ((unsigned long long)raw[az].y << 32) | raw[az].x;
            if (cur == key[az]) {
                v[az] = (int32_t)raw[az].w;
                run[az] = false;
            } else if (cur == kEmptyKey) {
                run[az] = false;
            } else {
                slot[az] = (slot[az] + 1) & (t.cap - 1);
                any = true;
            }
        }
    }
}

// grid (tiles, K*K / NC): thread (o, columns) searches the K offsets along z of NC columns (ax, ay).  Writes
// nbr_out[k][o], scatters nbr_in[k][i] = o when nbr_in is given, and counts the links.
// identity: input and output rows are the same set, the centre offset links every row to itself.
// Bound by the rate of scattered loads (a wavefront's 64 lanes touch 64 lines).  In a grid a column is at most two
// blocks: two loads of dir and two of four cells each, all of the thread's columns requested together.  (0.37 M
// rows, K = 3: 84 us when the lower half of the offsets was searched in the hash table and mirrored, plus 29 us for
// resetting the table and counting its entries.)
template <int K, int NC>
__global__ __launch_bounds__(kTileRows) void search_kernel(const int4* __restrict__ c_out, Count cn_out, TableView t, int dilation,
                                                           int identity, int32_t* __restrict__ nbr_out,
                                                           int32_t* __restrict__ nbr_in, Count cn_in, Counts counts,
                                                           int32_t* __restrict__ done) {
    constexpr int kvol = K * K * K, centre = (K & 1) ? (K - 1) / 2 : 0;
    __shared__ int s_cnt[kSubTiles][NC * K][kHalves];
    const int64_t n_out = get(cn_out);
    const int64_t tile = xcd_tile(blockIdx.x, (n_out + kTileRows - 1) / kTileRows);
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *done = 0;
    if (tile < 0) return;
    const int64_t o = tile * kTileRows + threadIdx.x;
    const int col0 = blockIdx.y * NC;
    int32_t v[NC * K];
#pragma unroll
    for (int j = 0; j < NC * K; ++j) v[j] = -1;
    if (o < n_out) {
        const int4 c = c_out[o];
        if (t.maybe_grid && t.meta[kMetaGrid]) {
            const Grid g = load_grid(t.meta);
            const int qb = c.x - g.b0;
            int qx, qy, qz;
            const bool onx = lattice(c.y - g.x0, t.ts, &qx), ony = lattice(c.z - g.y0, t.ts, &qy), onz = lattice(c.w - g.z0, t.ts, &qz);
            const bool on = onx && ony && onz && (unsigned)qb < (unsigned)g.nb;
            const int zl = qz - centre * dilation, zh = qz + (K - 1 - centre) * dilation;
            const bool narrow = (zh >> 2) - (zl >> 2) <= 1;  // the column's cells lie in at most two blocks: uniform for dilation 1
            int lo[NC], hi[NC], run[NC];
#pragma unroll
            for (int m = 0; m < NC; ++m) {
                const int x = qx + ((col0 + m) / K - centre) * dilation, y = qy + ((col0 + m) % K - centre) * dilation;
                const bool in = on && (unsigned)x < (unsigned)(8 * g.gx) && (unsigned)y < (unsigned)(8 * g.gy);
                const int bl = zl >> 2, bh = zh >> 2, nbz = 4 * g.gz;
                run[m] = grid_run(x, y);
                lo[m] = hi[m] = -1;
                if (in && (unsigned)bl < (unsigned)nbz) lo[m] = t.dir[grid_block(g, qb, x, y, bl)];
                if (in && bh != bl && (unsigned)bh < (unsigned)nbz) hi[m] = t.dir[grid_block(g, qb, x, y, bh)];
                if (!narrow && in) {  // wide spacing: one search at a time
#pragma unroll
                    for (int az = 0; az < K; ++az) {
                        const int z = zl + az * dilation;
                        if ((unsigned)(z >> 2) < (unsigned)nbz) {
                            const int b = t.dir[grid_block(g, qb, x, y, z >> 2)];
                            if (b >= 0) v[m * K + az] = t.cells[(int64_t)b * 16 + run[m] * 4 + (z & 3)];
                        }
                    }
                }
            }
            if (narrow) {
                int4 a[NC], b[NC];
#pragma unroll
                for (int m = 0; m < NC; ++m) {
                    a[m] = b[m] = int4{kNoRow, kNoRow, kNoRow, kNoRow};
                    if (lo[m] >= 0) a[m] = reinterpret_cast<const int4*>(t.cells)[(int64_t)lo[m] * 4 + run[m]];
                    if (hi[m] >= 0) b[m] = reinterpret_cast<const int4*>(t.cells)[(int64_t)hi[m] * 4 + run[m]];
                }
#pragma unroll
                for (int m = 0; m < NC; ++m)
#pragma unroll
                    for (int az = 0; az < K; ++az) {
                        const int z = zl + az * dilation, e = z & 3;
                        const bool low = (z >> 2) == (zl >> 2);
                        const int p0 = low ? a[m].x : b[m].x, p1 = low ? a[m].y : b[m].y, p2 = low ? a[m].z : b[m].z, p3 = low ? a[m].w : b[m].w;
                        v[m * K + az] = e < 2 ? (e == 0 ? p0 : p1) : (e == 2 ? p2 : p3);
                    }
            }
#pragma unroll
            for (int j = 0; j < NC * K; ++j) v[j] = v[j] == kNoRow ? -1 : v[j];
        } else {
#pragma unroll
            for (int m = 0; m < NC; ++m) {
                const int ax = (col0 + m) / K, ay = (col0 + m) % K;
                const int skip = identity && ax == centre && ay == centre ? centre : -1;
                search_hash<K>(t, c, ax - centre, ay - centre, dilation * t.ts, skip, v + m * K);
                if (skip >= 0) v[m * K + centre] = (int32_t)o;
            }
        }
        const int64_t n_in = nbr_in ? get(cn_in) : 0;
#pragma unroll
        for (int j = 0; j < NC * K; ++j) {
            const int64_t k = col0 * K + j;
            nbr_out[k * n_out + o] = v[j];
            if (nbr_in && v[j] >= 0) nbr_in[k * n_in + v[j]] = (int32_t)o;
        }
    }
    count_rows<NC * K>(counts, kvol, tile, v, s_cnt, [&](int j) { return col0 * K + j; });
}

// Position class of an input row inside its coarse cell: ((x/ts) mod s, (y/ts) mod s, (z/ts) mod s) as one number.
__device__ __forceinline__ int cell_class(const int4& c, int ts, int stride) {
    auto r = [&](int v) { const int q = v / ts % stride; return q < 0 ? q + stride : q; };  // coordinates are multiples of ts
    return (r(c.y) * stride + r(c.z)) * stride + r(c.w);
}

// Even kernel as wide as the stride (offsets 0 .. K-1 = the positions inside a coarse cell): every input row
// has exactly one link, to its own coarse cell (parent[i], from the coarse coordinates' merge), at the offset
// that is its position in the cell.  No searches.
__global__ __launch_bounds__(kThreads) void child_map_kernel(const int4* __restrict__ c_in, Count cn_in, int ts, int stride,
                                                             const int32_t* __restrict__ parent, Count cn_out, int kvol,
                                                             int32_t* __restrict__ nbr_out, int32_t* __restrict__ nbr_in) {
    const int64_t n_in = get(cn_in), n_out = get(cn_out);
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n_in) return;
    const int k = cell_class(c_in[i], ts, stride);
    const int32_t o = parent[i];
    for (int j = 0; j < kvol; ++j) nbr_in[(int64_t)j * n_in + i] = j == k ? o : -1;
    if (nbr_out) nbr_out[(int64_t)k * n_out + o] = (int32_t)i;
}

// One search, in either form of table.
__device__ __forceinline__ int32_t find_row(const TableView& t, int b, int x, int y, int z) {
    if (!(t.maybe_grid && t.meta[kMetaGrid])) {
        uint64_t key;
        if (!pack_key(b, x, y, z, &key)) return -1;
        uint32_t bucket, pos;
        hash_home(key, t.cap, t.zshift, &bucket, &pos);
        uint32_t slot = bucket * 4 + pos;
        for (uint32_t probe = 0; probe < t.cap; ++probe, slot = (slot + 1) & (t.cap - 1)) {
            if (t.slots[slot].key == key) return t.slots[slot].row;
            if (t.slots[slot].key == kEmptyKey) break;
        }
        return -1;
    }
    const Grid g = load_grid(t.meta);
    int qx, qy, qz;
    const bool onx = lattice(x - g.x0, t.ts, &qx), ony = lattice(y - g.y0, t.ts, &qy), onz = lattice(z - g.z0, t.ts, &qz);
    if (!onx || !ony || !onz || (unsigned)(b - g.b0) >= (unsigned)g.nb || (unsigned)qx >= (unsigned)(8 * g.gx) ||
        (unsigned)qy >= (unsigned)(8 * g.gy) || (unsigned)(qz >> 2) >= (unsigned)(4 * g.gz))
        return -1;
    const int32_t num = t.dir[grid_block(g, b - g.b0, qx, qy, qz >> 2)];
    if (num < 0) return -1;
    const int32_t r = t.cells[(int64_t)num * 16 + grid_run(qx, qy) * 4 + (qz & 3)];
    return r == kNoRow ? -1 : r;
}

// Output side of a 2 x 2 x 2 stride-2 map whose input set may be a grid: a coarse row's eight children are one half of a block,
// 32 bytes apart from its pair number (c_out's pairs, valid if c_out is a grid itself), written and counted in one pass over the
// coarse rows: no table preset, no scattered stores, no counting of the table (0.5 M rows: with child_map_kernel 18 us, now 13).
// Only for rows that are multiples of the tensor stride for certain: a child is then at its cell's corner plus 0 or one stride per
// axis, which is what child_map_kernel goes by for the input side.
__global__ __launch_bounds__(kTileRows) void child_rows_kernel(const int4* __restrict__ c_out, Count cn_out, const int32_t* __restrict__ meta_out,
                                                               const int32_t* __restrict__ pairs, TableView t, int32_t* __restrict__ nbr_out,
                                                               Counts counts, int32_t* __restrict__ done) {
    __shared__ int s_cnt[kSubTiles][8][kHalves];
    const int64_t n_out = get(cn_out), tile = blockIdx.x, o = tile * kTileRows + threadIdx.x;
    if (tile == 0 && threadIdx.x == 0) *done = 0;
    if (tile * kTileRows >= n_out) return;
    int32_t v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = -1;
    if (o < n_out) {
        if (meta_out[kMetaGrid]) {
            const int32_t pair = pairs[o];
            const int2* runs = reinterpret_cast<const int2*>(t.cells) + (int64_t)(pair >> 1) * 8 + (pair & 1);
#pragma unroll
            for (int r = 0; r < 4; ++r) {  // run = 2 * ax + ay
                const int2 two = runs[2 * r];
                v[2 * r] = two.x == kNoRow ? -1 : two.x;
                v[2 * r + 1] = two.y == kNoRow ? -1 : two.y;
            }
        } else {
            const int4 c = c_out[o];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = find_row(t, c.x, c.y + (k >> 2) * t.ts, c.z + (k >> 1 & 1) * t.ts, c.w + (k & 1) * t.ts);
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) nbr_out[k * n_out + o] = v[k];
    }
    count_rows<8>(counts, 8, tile, v, s_cnt, [](int j) { return j; });
}

// Generative transposed convolution.  Candidate (j, k) = input row j displaced by offset k times the output
// lattice step; rows (j*kvol + k) of cand, i.e. input row by input row, offsets in offset order.
__global__ __launch_bounds__(kThreads) void gen_candidates_kernel(const int4* __restrict__ c_in, int64_t n_in, int K,
                                                                  int step, int4* __restrict__ cand) {
    const int kvol = K * K * K;
    const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (t >= n_in * kvol) return;
    const int64_t j = t / kvol;
    const int k = (int)(t % kvol);
    const int centre = (K & 1) ? (K - 1) / 2 : 0;
    int4 c = c_in[j];
    c.y += (k / (K * K) - centre) * step;
    c.z += (k / K % K - centre) * step;
    c.w += (k % K - centre) * step;
    cand[t] = c;
}

// where[j*kvol + k] = fine row of candidate (j, k).  As a stride-s convolution from the fine rows (inputs) to
// the coarse rows (outputs) every candidate is one link: nbr_out[k][j] = that fine row, nbr_in[k][fine] = j.
__global__ __launch_bounds__(kThreads) void gen_tables_kernel(const int32_t* __restrict__ where, int64_t n_coarse,
                                                              Count cn_fine, int kvol, int32_t* __restrict__ nbr_out,
                                                              int32_t* __restrict__ nbr_in) {
    const int64_t n_fine = get(cn_fine);
    const int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;   // = k * n_coarse + j: coalesced table writes
    if (t >= n_coarse * kvol) return;
    const int k = (int)(t / n_coarse);
    const int64_t j = t % n_coarse;
    const int32_t f = where[j * kvol + k];
    nbr_out[t] = f;
    nbr_in[(int64_t)k * n_fine + f] = (int32_t)j;
}

constexpr int kChunk = 9;  // offsets whose table entries a thread requests before it looks at any of them

// Counts of a table that no search has counted: grid (tiles, chunks of kChunk offsets).
__global__ __launch_bounds__(kTileRows) void count_kernel(const int32_t* __restrict__ nbr, Count n_rows, int kvol, Counts counts,
                                                          int32_t* __restrict__ done) {
    __shared__ int s_cnt[kSubTiles][kChunk][kHalves];
    const int64_t n = get(n_rows), t = blockIdx.x;
    if (done && t == 0 && blockIdx.y == 0 && threadIdx.x == 0) *done = 0;
    if (t * kTileRows >= n) return;
    const int64_t r = t * kTileRows + threadIdx.x;
    const int k0 = blockIdx.y * kChunk;
    int32_t v[kChunk];
#pragma unroll
    for (int j = 0; j < kChunk; ++j) v[j] = (r < n && k0 + j < kvol) ? nbr[(int64_t)(k0 + j) * n + r] : -1;
    count_rows<kChunk>(counts, kvol, t, v, s_cnt, [&](int j) { return k0 + j; });
}

struct EmitArgs {
    const int32_t* nbr;
    Count n_rows;
    int kvol;
    Counts counts;
    int32_t* off;       // [(sub-tile)][kvol][half], and one row of ends
    int32_t* src;       // [kvol][pitch]
    int32_t* dst;
    int64_t pitch;
    // results (the side the build walks only)
    int32_t* d_counts;  // null, or [kvol] and the word that counts the workgroups which have delivered
    uint32_t* mail;     // null or the mail slot: n_in, n_out, error bits, counts[0..kvol)
    uint32_t mail_seq;
    Count n_in, n_out;  // for the mail
};

// grid (tiles, chunks of kChunk offsets): entries of a tile for one chunk.
__global__ __launch_bounds__(kTileRows) void emit_kernel(EmitArgs a) {
    __shared__ int s_start[kSubTiles][kChunk];
    __shared__ int s_total[kChunk];
    const int kvol = a.kvol;
    const int64_t n = get(a.n_rows);
    const int64_t ntiles = (n + kTileRows - 1) / kTileRows;
    const int64_t t = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if (t >= ntiles && !(t == 0 && ntiles == 0)) return;
    const int k0 = blockIdx.y * kChunk;
    const int64_t r = t * kTileRows + tid;
    int32_t v[kChunk];
#pragma unroll
    for (int j = 0; j < kChunk; ++j) v[j] = (r < n && k0 + j < kvol) ? a.nbr[(int64_t)(k0 + j) * n + r] : -1;

    // wavefront j: offset k0 + j.  Links of the tiles before this one, then where each sub-tile's begin.
    if (w < kChunk && k0 + w < kvol) {
        const int k = k0 + w;
        int sum = 0;
        if (a.counts.pre) {
            sum = a.counts.pre[k * (a.counts.pitch + 1) + t];
        } else {
            const int32_t* agg = a.counts.agg + k * a.counts.pitch;
            for (int64_t t0 = lane; t0 < t; t0 += 256) {  // four loads at a time
                int v4[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) v4[i] = t0 + 64 * i < t ? agg[t0 + 64 * i] : 0;
                sum += (v4[0] + v4[1]) + (v4[2] + v4[3]);
            }
#pragma unroll
            for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d, 64);
        }
        int2 c = {0, 0};
        if (ntiles && lane < kSubTiles) c = *reinterpret_cast<const int2*>(a.counts.cnt + ((t * kSubTiles + lane) * kvol + k) * kHalves);
        int inc = c.x + c.y;
#pragma unroll
        for (int d = 1; d < kSubTiles; d <<= 1) {
            const int u = __shfl_up(inc, d, 64);
            if (lane >= d) inc += u;
        }
        const int start = (int)(k * a.pitch) + sum + inc - (c.x + c.y);
        if (ntiles && lane < kSubTiles) {
            s_start[lane][w] = start;
            *reinterpret_cast<int2*>(a.off + ((t * kSubTiles + lane) * kvol + k) * kHalves) = int2{start, start + c.x};
        }
        const int end = (int)(k * a.pitch) + sum + __shfl(inc, kSubTiles - 1, 64);
        if (t == (ntiles ? ntiles - 1 : 0) && lane == 0) {  // the last tile: the ends, the counts
            *reinterpret_cast<int2*>(a.off + ((ntiles * kSubTiles) * kvol + k) * kHalves) = int2{end, end};
            s_total[w] = ntiles ? end - (int)(k * a.pitch) : 0;
        }
    }
    __syncthreads();
    if (a.d_counts && t == (ntiles ? ntiles - 1 : 0) && tid == 0) {
        // the workgroups of the last tile each deliver their chunk; the one that finishes last also sends the mail off
        for (int j = 0; j < kChunk && k0 + j < kvol; ++j) {
            a.d_counts[k0 + j] = s_total[j];
            if (a.mail) a.mail[3 + k0 + j] = (uint32_t)s_total[j];
        }
        if (a.mail) {
            __threadfence_system();
            if (atomicAdd(a.d_counts + kvol, 1) == (int)gridDim.y - 1) {
                a.mail[0] = (uint32_t)get(a.n_in);
                a.mail[1] = (uint32_t)get(a.n_out);
                a.mail[2] = 0u;
                __threadfence_system();
                __hip_atomic_store(a.mail + kMailSeqWord, a.mail_seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
            }
        }
    }
    if (ntiles == 0) return;

    // every live (row, k) writes its entry at start + (number of live lanes below it)
#pragma unroll
    for (int j = 0; j < kChunk; ++j) {
        const unsigned long long live = __ballot(v[j] >= 0);
        if (v[j] >= 0) {
            const int e = s_start[w][j] + __popcll(live & ((1ull << lane) - 1ull));
            a.src[e] = v[j];
            a.dst[e] = (int32_t)r;
        }
    }
}

// Rows per position class and tile.
__global__ __launch_bounds__(kTileRows) void class_count_kernel(const int4* __restrict__ coords, int64_t n, int ts, int stride,
                                                                int nclass, int32_t* __restrict__ agg, int64_t pitch) {
    __shared__ int s_cls[32][kSubTiles];
    const int64_t t = blockIdx.x, r = t * kTileRows + threadIdx.x;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int cls = r < n ? cell_class(coords[r], ts, stride) : -1;
    for (int c = 0; c < nclass; ++c) {
        const unsigned long long m = __ballot(cls == c);
        if (lane == 0) s_cls[c][w] = __popcll(m);
    }
    __syncthreads();
    if ((int)threadIdx.x < nclass) {
        int sum = 0;
        for (int ww = 0; ww < kSubTiles; ++ww) sum += s_cls[threadIdx.x][ww];
        agg[threadIdx.x * pitch + t] = sum;
    }
}

// Rows of a strided map's input side in position-class order, and per 256 entries of that order the offsets
// that can link them.  perm[(rows of lower classes) + (rows of class c in earlier tiles) + rank in the tile] = row.
// mask[tile][k / 32] bit k % 32 = offset k can link a row of one of the position classes present in
// perm[tile*256 .. +255]: offset (ax, ay, az) links an input at class r to an output only if, per axis, the
// offset's displacement is congruent to r modulo the stride (output coordinates are multiples of the stride).
__global__ __launch_bounds__(kTileRows) void class_emit_kernel(const int4* __restrict__ coords, int64_t n, int ts, int stride,
                                                               int nclass, int K, const int32_t* __restrict__ agg,
                                                               const int32_t* __restrict__ pre, int64_t pitch,
                                                               int32_t* __restrict__ perm, uint32_t* __restrict__ mask) {
    __shared__ int s_cnt[32][kSubTiles];
    __shared__ int s_total[32], s_before[32], s_base[33];
    __shared__ uint32_t s_cm[32][4];  // offsets possible for each class
    const int64_t t = blockIdx.x, ntiles = (n + kTileRows - 1) / kTileRows;
    const int64_t r = t * kTileRows + threadIdx.x;
    const int cls = r < n ? cell_class(coords[r], ts, stride) : -1;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    int rank = 0;
    for (int c = 0; c < nclass; ++c) {
        const unsigned long long m = __ballot(cls == c);
        if (lane == 0) s_cnt[c][w] = __popcll(m);
        if (cls == c) rank = __popcll(m & ((1ull << lane) - 1ull));
    }
    for (int c = w; c < nclass; c += kSubTiles) {  // a wavefront per class: rows of the class before this tile, and in all
        int before = 0, all = 0;
        if (pre) {
            before = pre[c * (pitch + 1) + t];
            all = pre[c * (pitch + 1) + ntiles];
        } else {
            for (int64_t tt = lane; tt < ntiles; tt += 64) {
                const int v = agg[c * pitch + tt];
                all += v;
                before += tt < t ? v : 0;
            }
#pragma unroll
            for (int d = 32; d > 0; d >>= 1) {
                before += __shfl_xor(before, d, 64);
                all += __shfl_xor(all, d, 64);
            }
        }
        if (lane == 0) {
            s_before[c] = before;
            s_total[c] = all;
        }
    }
    const int centre = (K & 1) ? (K - 1) / 2 : 0;
    if (tid >= 64 && tid < 64 + nclass) {
        const int c = tid - 64;
        const int rr[3] = {c / (stride * stride), c / stride % stride, c % stride};
        uint32_t m[4] = {0u, 0u, 0u, 0u};
        for (int k = 0; k < K * K * K; ++k) {
            const int d[3] = {k / (K * K) - centre, k / K % K - centre, k % K - centre};
            bool ok = true;
            for (int ax = 0; ax < 3; ++ax) ok = ok && ((d[ax] % stride + stride) % stride == rr[ax]);
            if (ok) m[k >> 5] |= 1u << (k & 31);
        }
        for (int i = 0; i < 4; ++i) s_cm[c][i] = m[i];
    }
    __syncthreads();
    if (tid == 0) {
        int run = 0;
        for (int c = 0; c < nclass; ++c) {
            s_base[c] = run;
            run += s_total[c];
        }
        s_base[nclass] = run;
    }
    __syncthreads();
    if (cls >= 0) {
        for (int j = 0; j < w; ++j) rank += s_cnt[cls][j];
        perm[s_base[cls] + s_before[cls] + rank] = (int32_t)r;
    }
    if (tid < 16) {  // the masks of this tile's four 256-entry stretches of the class-sorted order
        const int64_t mt = t * 4 + (tid >> 2), lo = mt * 256, hi = lo + 256 < n ? lo + 256 : n;
        if (lo < n) {
            uint32_t m = 0u;
            for (int c = 0; c < nclass; ++c)
                if (s_base[c] < hi && s_base[c + 1] > lo) m |= s_cm[c][tid & 3];
            mask[mt * 4 + (tid & 3)] = m;
        }
    }
}

inline unsigned blocks256(int64_t n) { return (unsigned)((n + 255) / 256); }
inline int64_t tiles_of(int64_t n) { return (n + kTileRows - 1) / kTileRows; }
inline unsigned chunks_of(int kvol) { return (unsigned)((kvol + kChunk - 1) / kChunk); }

// Memory of a side's lists: `pitch` entries per offset.
int reserve_lists(MapSide& side, int64_t n_ub, int64_t pitch, int kvol, hipStream_t s) {
    const size_t entries = (size_t)(pitch ? pitch : 1) * kvol;
    side.pitch = pitch;
    side.off = dev_alloc((size_t)(tiles_of(n_ub) * kSubTiles + 1) * kvol * kHalves * 4, s);
    side.src = dev_alloc(entries * 4, s);
    side.dst = dev_alloc(entries * 4, s);
    return side.off && side.src && side.dst ? SP_OK : SP_ERR_ALLOC;
}

// Sums of `width` things per tile, with room for their prefixes where prefix_kernel makes them.
int64_t sum_words(int64_t nt, int width) { return nt * width + (nt > kSumTiles ? (nt + 1) * width : 0); }
int32_t* prefixes_in(int32_t* agg, int64_t nt, int width) { return nt > kSumTiles ? agg + nt * width : nullptr; }

size_t counts_bytes(int64_t n_ub, int kvol) {
    const int64_t nt = tiles_of(n_ub) ? tiles_of(n_ub) : 1;
    return (size_t)(nt * kvol * kSubTiles * kHalves + sum_words(nt, kvol)) * 4;
}
Counts counts_in(const Buf& b, int64_t n_ub, int kvol) {
    const int64_t nt = tiles_of(n_ub) ? tiles_of(n_ub) : 1;
    int32_t *p = ptr<int32_t>(b), *agg = p + nt * kvol * kSubTiles * kHalves;
    return Counts{p, agg, prefixes_in(agg, nt, kvol), nt};
}

void launch_emit(const EmitArgs& a, int64_t n_ub, hipStream_t s) {
    const int64_t nt = tiles_of(n_ub);
    if (a.counts.pre)
        hipLaunchKernelGGL(prefix_kernel, dim3((unsigned)a.kvol), dim3(kTileRows), 0, s, a.counts.agg, a.counts.pre, a.counts.pitch, a.n_rows);
    hipLaunchKernelGGL(emit_kernel, dim3((unsigned)(nt ? nt : 1), chunks_of(a.kvol)), dim3(kTileRows), 0, s, a);
}

EmitArgs emit_args(const MapSide& side, Count n_rows, int kvol, const Counts& counts) {
    EmitArgs a{};
    a.nbr = ptr<int32_t>(side.nbr);
    a.n_rows = n_rows;
    a.kvol = kvol;
    a.counts = counts;
    a.off = ptr<int32_t>(side.off);
    a.src = ptr<int32_t>(side.src);
    a.dst = ptr<int32_t>(side.dst);
    a.pitch = side.pitch;
    return a;
}

// Second half of a map build, shared by every way of filling the neighbour tables: on entry both tables and the
// output side's counts are complete (on the stream).  n_in_ub / n_out_ub: upper bounds of the row counts, cn_in /
// cn_out: where the kernels find the true ones.  Emits the output side's lists; an input side of its own gets the
// memory for lists and class order.
int finish_map(sp_kmap* m, bool symmetric, const Counts& counts, int64_t n_in_ub, int64_t n_out_ub, Count cn_in, Count cn_out,
               int nclass, hipStream_t s) {
    MapSide& so = m->out_side;
    MapSide& si = m->in_side;
    const int kvol = m->kvol;
    // All memory first: whoever has seen the counts then knows that the stream is past every wait for a block's last user.
    if (!symmetric) {
        SP_TRY(reserve_lists(si, n_in_ub, so.pitch, kvol, s));
        si.work = std::make_shared<SideWork>();
        SideWork& w = *si.work;
        w.counts = dev_alloc(counts_bytes(n_in_ub, kvol), s);
        if (!w.counts) return SP_ERR_ALLOC;
        if (nclass && n_in_ub > 0) {
            si.perm = dev_alloc((size_t)n_in_ub * 4, s);
            si.tile_mask = dev_alloc((size_t)((n_in_ub + 255) / 256) * 16, s);
            w.class_counts = dev_alloc((size_t)sum_words(tiles_of(n_in_ub), nclass) * 4, s);
            if (!si.perm || !si.tile_mask || !w.class_counts) return SP_ERR_ALLOC;
            w.coords = m->c_in->coords;
            w.ts = m->c_in->ts;
            w.stride = m->stride;
            w.K = m->K;
            w.nclass = nclass;
        }
    }
    const bool mailed = mail_acquire(&m->mail);
    EmitArgs a = emit_args(so, cn_out, kvol, counts);
    a.d_counts = ptr<int32_t>(m->d_counts);
    a.mail = mailed ? m->mail.d : nullptr;
    a.mail_seq = m->mail.seq;
    a.n_in = cn_in;
    a.n_out = cn_out;
    launch_emit(a, n_out_ub, s);
    m->mail.armed = mailed;
    m->mail.stream = s;
    m->pair_in = so.src;
    m->pair_out = so.dst;
    m->pair_stride = so.pitch;
    if (symmetric) {
        si = so;  // same lists; the link (i, o) at offset k is the link (o, i) at offset kvol-1-k
        si.flip = true;
    }
    SP_HIP(hipGetLastError());
    if (!mailed) {  // no mail slot free: wait here
        std::vector<uint32_t> h(kvol);
        SP_TRY(read_back(h.data(), ptr<int32_t>(m->d_counts), (size_t)kvol * 4, s));
        SP_TRY(coords_resolve(m->c_in));
        SP_TRY(coords_resolve(m->c_out));
        m->set_sizes(m->c_in->n, m->c_out->n, h.data());
        m->status = SP_OK;
        m->resolved = true;
    }
    return SP_OK;
}

// Calls of this thread that a capture under way elsewhere would forbid (making a stream, waiting for it).
struct RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

// build(stream) enqueues the work; what s runs from here on finds it done.
// (Events would not do: the runtime refuses an event, and draws who waits for it into the capture, while the stream it
// was recorded on is being captured, also if it was recorded before.)
// Under graph capture the work stays out of the graph, or every replay would repeat it: it runs on a stream of its own and
// the host waits for it.  All that it reads is complete: the host has had the map's counts.
template <class Build>
int once(Once& o, hipStream_t s, Build build) {
    if (o.ready) return SP_OK;
    if (o.mail.index >= 0 && mail_arrived(o.mail)) {
        mail_release(&o.mail);
        o.ready = true;
        return SP_OK;
    }
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &cap) != hipSuccess) (void)hipGetLastError();
    if (cap != hipStreamCaptureStatusNone) {
        RelaxedCapture relaxed;
        hipStream_t own = nullptr;
        SP_HIP(hipStreamCreateWithFlags(&own, hipStreamNonBlocking));
        const int rc = build(own);
        const hipError_t e = hipStreamSynchronize(own);
        (void)hipStreamDestroy(own);
        SP_TRY(rc);
        SP_HIP(e);
        mail_release(&o.mail);
        o.ready = true;
        return SP_OK;
    }
    if (o.mail.index >= 0 && o.on == s) return SP_OK;
    SP_TRY(build(s));
    mail_release(&o.mail);
    if (!mail_acquire(&o.mail)) {  // no mail slot free: wait here
        SP_HIP(hipStreamSynchronize(s));
        o.ready = true;
        return SP_OK;
    }
    mail_send(&o.mail, s);
    SP_HIP(hipGetLastError());
    o.on = s;
    return SP_OK;
}

}  // namespace

int need_lists(const MapSide& side, int kvol, hipStream_t s) {
    if (!side.work || side.n_rows == 0) return SP_OK;
    SideWork& w = *side.work;
    std::lock_guard<std::mutex> lk(w.mu);
    return once(w.lists, s, [&](hipStream_t on) -> int {
        const Count n{nullptr, side.n_rows};
        const Counts c = counts_in(w.counts, side.n_rows, kvol);
        const dim3 grid((unsigned)tiles_of(side.n_rows), chunks_of(kvol));
        hipLaunchKernelGGL(count_kernel, grid, dim3(kTileRows), 0, on, ptr<int32_t>(side.nbr), n, kvol, c, (int32_t*)nullptr);
        launch_emit(emit_args(side, n, kvol, c), side.n_rows, on);
        SP_HIP(hipGetLastError());
        return SP_OK;
    });
}

int need_classes(const MapSide& side, hipStream_t s) {
    if (!side.tile_mask || !side.work || side.n_rows == 0) return SP_OK;
    SideWork& w = *side.work;
    std::lock_guard<std::mutex> lk(w.mu);
    return once(w.classes, s, [&](hipStream_t on) -> int {
        const int64_t nt = tiles_of(side.n_rows);
        const dim3 grid((unsigned)nt);
        int32_t *agg = ptr<int32_t>(w.class_counts), *pre = prefixes_in(agg, nt, w.nclass);
        hipLaunchKernelGGL(class_count_kernel, grid, dim3(kTileRows), 0, on, ptr<int4>(w.coords), side.n_rows, w.ts, w.stride, w.nclass, agg,
                           nt);
        if (pre)
            hipLaunchKernelGGL(prefix_kernel, dim3((unsigned)w.nclass), dim3(kTileRows), 0, on, agg, pre, nt, Count{nullptr, side.n_rows});
        hipLaunchKernelGGL(class_emit_kernel, grid, dim3(kTileRows), 0, on, ptr<int4>(w.coords), side.n_rows, w.ts, w.stride, w.nclass,
                           w.K, agg, pre, nt, ptr<int32_t>(side.perm), ptr<uint32_t>(side.tile_mask));
        SP_HIP(hipGetLastError());
        return SP_OK;
    });
}

int kmap_resolve(const sp_kmap_t* m) {
    std::lock_guard<std::mutex> lk(m->mu);
    if (!m->resolved) {
        SP_TRY(mail_wait(m->mail, m->stream));
        const uint32_t* h = m->mail.h;
        m->set_sizes((int64_t)h[0], (int64_t)h[1], h + 3);
        m->status = SP_OK;
        m->resolved = true;
        mail_release(&m->mail);
    }
    // an error found while the coordinate sets were built (a coordinate out of range) makes the map invalid too
    if (m->c_in) SP_TRY(coords_resolve(m->c_in));
    if (m->c_out && m->c_out != m->c_in) SP_TRY(coords_resolve(m->c_out));
    return SP_OK;
}

}  // namespace sp

// host copies of the sizes, once they have arrived: counts per offset
void sp_kmap::set_sizes(int64_t ni, int64_t no, const uint32_t* count_words) const {
    n_in = ni;
    n_out = no;
    koff.resize(kvol + 1);
    counts.resize(kvol);
    koff[0] = 0;
    for (int k = 0; k < kvol; ++k) {
        counts[k] = count_words[k];
        koff[k + 1] = koff[k] + counts[k];
    }
    total = koff[kvol];
    out_side.n_rows = no;
    out_side.n_src = ni;
    in_side.n_rows = ni;
    in_side.n_src = no;
}

using namespace sp;

extern "C" {

int sp_kmap_build(const sp_coords_t* in, int32_t kernel_size, int32_t stride, int32_t dilation, void* stream,
                  sp_kmap_t** kmap, sp_coords_t** out_coords) {
    if (kmap) *kmap = nullptr;
    if (out_coords) *out_coords = nullptr;
    if (!in || !kmap) return fail(SP_ERR_INVALID_ARG, "coords handle or kmap out pointer is NULL");
    if (kernel_size < 1 || kernel_size > 5) return fail(SP_ERR_INVALID_ARG, "kernel_size %d not in 1..5", kernel_size);
    if (stride < 1 || dilation < 1) return fail(SP_ERR_INVALID_ARG, "stride and dilation must be >= 1");
    if (stride > 1 && dilation > 1) return fail(SP_ERR_UNSUPPORTED, "dilation > 1 together with stride > 1");
    if ((int64_t)in->ts * stride > 32768 || (int64_t)in->ts * dilation * kernel_size > 65536)
        return fail(SP_ERR_RANGE, "tensor stride * stride / dilation leaves the packable coordinate range");
    hipStream_t s = (hipStream_t)stream;
    const int kvol = kernel_size * kernel_size * kernel_size;
    // Sizes: the input set's row count may not have reached the host yet.  Then its source row count bounds it;
    // when that bound would make the tables and lists much larger than they can need to be (many duplicates in
    // a large input), waiting for the count is the cheaper choice.
    bool known;
    {
        std::lock_guard<std::mutex> lk(in->mu);
        known = in->resolved;
    }
    if (!known && in->n_raw * (int64_t)kvol * 18 > ((int64_t)1 << 30)) {
        SP_TRY(coords_resolve(in));
        known = true;
    }
    if (known) SP_TRY(coords_resolve(in));  // reports an error found while it was built
    const int64_t n_in_ub = known ? in->n : in->n_raw;
    if (n_in_ub * (int64_t)kvol >= ((int64_t)1 << 31) - 4096)
        return fail(SP_ERR_INVALID_ARG, "n * kernel volume exceeds 32-bit list offsets");
    const Count cn_in{known ? nullptr : ptr<int32_t>(in->meta) + kMetaN, known ? in->n : 0};

    std::unique_ptr<sp_kmap, int (*)(sp_kmap*)> m(new sp_kmap, sp_kmap_destroy);
    m->K = kernel_size;
    m->kvol = kvol;
    m->stride = stride;
    m->dilation = dilation;
    m->stream = s;
    // (Rows off the lattice, which a caller may have, are found by their place in the cell on both sides: child_map_kernel.)
    const bool child_rows = stride == 2 && kernel_size == 2 && in->on_lattice;
    sp_coords* cin = const_cast<sp_coords*>(in);
    cin->ref.fetch_add(1);
    m->c_in = cin;
    Count cn_out = cn_in;
    int64_t n_out_ub = n_in_ub;
    if (stride == 1) {
        cin->ref.fetch_add(1);
        m->c_out = cin;
    } else {
        sp_coords* co = nullptr;
        SP_TRY(coords_build_impl(ptr<int32_t>(in->coords), n_in_ub, cn_in.d, in->ts * stride, in->ts * stride, in, child_rows, s, &co));
        cin->ref.fetch_add(1);
        co->src_of = cin;  // its inverse array has one entry per row of `in`
        m->c_out = co;
        cn_out = co->resolved ? Count{nullptr, co->n} : Count{ptr<int32_t>(co->meta) + kMetaN, 0};
        if (co->resolved) n_out_ub = co->n;
    }
    const bool symmetric = (stride == 1) && (kernel_size & 1);
    const int nclass = (stride > 1 && stride * stride * stride <= 32) ? stride * stride * stride : 0;

    MapSide& so = m->out_side;
    MapSide& si = m->in_side;
    so.nbr = dev_alloc((size_t)(n_out_ub ? n_out_ub : 1) * kvol * 4, s);
    SP_TRY(reserve_lists(so, n_out_ub, std::min(n_out_ub, n_in_ub), kvol, s));
    m->d_counts = dev_alloc((size_t)(kvol + 1) * 4, s);
    Buf work = dev_alloc(counts_bytes(n_out_ub, kvol), s);
    if (!so.nbr || !m->d_counts || !work) return SP_ERR_ALLOC;
    if (!symmetric) {
        si.nbr = dev_alloc((size_t)(n_in_ub ? n_in_ub : 1) * kvol * 4, s);
        if (!si.nbr) return SP_ERR_ALLOC;
    }
    const Counts counts = counts_in(work, n_out_ub, kvol);
    int32_t* done = ptr<int32_t>(m->d_counts) + kvol;
    const unsigned nt = (unsigned)(tiles_of(n_out_ub) ? tiles_of(n_out_ub) : 1);
    if (child_rows && m->c_out->pairs) {
        hipLaunchKernelGGL(child_map_kernel, dim3(blocks256(n_in_ub)), dim3(kThreads), 0, s, ptr<int4>(in->coords), cn_in, in->ts, stride,
                           ptr<int32_t>(m->c_out->inverse), cn_out, kvol, (int32_t*)nullptr, ptr<int32_t>(si.nbr));
        hipLaunchKernelGGL(child_rows_kernel, dim3(nt), dim3(kTileRows), 0, s, ptr<int4>(m->c_out->coords), cn_out, ptr<int32_t>(m->c_out->meta),
                           ptr<int32_t>(m->c_out->pairs), table_view(in), ptr<int32_t>(so.nbr), counts, done);
        m->c_out->pairs.reset();  // (later users of the memory are ordered behind this launch on the stream)
    } else if (stride > 1 && kernel_size == stride && kernel_size % 2 == 0) {
        if (n_out_ub > 0) {
            hipLaunchKernelGGL(reset_kernel, dim3(blocks256((n_out_ub * (int64_t)kvol + 3) / 4)), dim3(kThreads), 0, s, ptr<int32_t>(so.nbr),
                               cn_out, kvol);
            hipLaunchKernelGGL(child_map_kernel, dim3(blocks256(n_in_ub)), dim3(kThreads), 0, s, ptr<int4>(in->coords), cn_in, in->ts,
                               stride, ptr<int32_t>(m->c_out->inverse), cn_out, kvol, ptr<int32_t>(so.nbr), ptr<int32_t>(si.nbr));
        }
        hipLaunchKernelGGL(count_kernel, dim3(nt, chunks_of(kvol)), dim3(kTileRows), 0, s, ptr<int32_t>(so.nbr), cn_out, kvol, counts, done);
    } else {
        if (!symmetric && n_in_ub > 0)
            hipLaunchKernelGGL(reset_kernel, dim3(blocks256((n_in_ub * (int64_t)kvol + 3) / 4)), dim3(kThreads), 0, s, ptr<int32_t>(si.nbr),
                               cn_in, kvol);
        const TableView tab = table_view(in);
        // Columns per thread: all K of one ax where the rows alone fill the chip, one where they do not (coordinates + map,
        // one against three: 71 k rows 57 against 60 us, 130 k 71 against 75, 174 k 74 against 76, 255 k 82 against 83).
        const bool few = n_out_ub < (1 << 18);
#define SP_SEARCH(KS, NC)                                                                                                   \
    hipLaunchKernelGGL((search_kernel<KS, NC>), dim3(xcd_grid(nt), KS * KS / NC), dim3(kTileRows), 0, s, ptr<int4>(m->c_out->coords), cn_out, tab, \
                       dilation, symmetric ? 1 : 0, ptr<int32_t>(so.nbr), symmetric ? (int32_t*)nullptr : ptr<int32_t>(si.nbr), cn_in, \
                       counts, done)
        switch (kernel_size) {
            case 1: SP_SEARCH(1, 1); break;
            case 2: SP_SEARCH(2, 1); break;
            case 3:
                if (few) SP_SEARCH(3, 1);
                else SP_SEARCH(3, 3);
                break;
            case 4: SP_SEARCH(4, 1); break;
            default: SP_SEARCH(5, 1); break;
        }
#undef SP_SEARCH
    }
    SP_HIP(hipGetLastError());
    SP_TRY(finish_map(m.get(), symmetric, counts, n_in_ub, n_out_ub, cn_in, cn_out, nclass, s));
    if (out_coords) {
        m->c_out->ref.fetch_add(1);
        *out_coords = m->c_out;
    }
    *kmap = m.release();
    return SP_OK;
}

int sp_kmap_build_generative(const sp_coords_t* in, int32_t kernel_size, int32_t stride, void* stream, sp_kmap_t** kmap,
                             sp_coords_t** out_coords) {
    if (kmap) *kmap = nullptr;
    if (out_coords) *out_coords = nullptr;
    if (!in || !kmap) return fail(SP_ERR_INVALID_ARG, "coords handle or kmap out pointer is NULL");
    if (kernel_size < 1 || kernel_size > 5) return fail(SP_ERR_INVALID_ARG, "kernel_size %d not in 1..5", kernel_size);
    if (stride < 1) return fail(SP_ERR_INVALID_ARG, "stride must be >= 1");
    if (in->ts % stride != 0)
        return fail(SP_ERR_INVALID_ARG, "the tensor stride (%d) must be a multiple of the layer stride (%d)", in->ts, stride);
    hipStream_t s = (hipStream_t)stream;
    const int kvol = kernel_size * kernel_size * kernel_size;
    SP_TRY(coords_resolve(in));  // the candidate count sizes everything
    const int64_t n_coarse = in->n, n_cand = n_coarse * kvol;
    if (n_cand >= ((int64_t)1 << 30)) return fail(SP_ERR_INVALID_ARG, "n * kernel volume exceeds 2^30 candidates");
    const int ts_out = in->ts / stride;

    // candidates -> fine coordinates (first-occurrence order) and the candidate -> fine row table
    Buf cand = dev_alloc((size_t)(n_cand ? n_cand : 1) * 16, s);
    if (!cand) return SP_ERR_ALLOC;
    if (n_cand > 0)
        hipLaunchKernelGGL(gen_candidates_kernel, dim3(blocks256(n_cand)), dim3(kThreads), 0, s, ptr<int4>(in->coords),
                           n_coarse, kernel_size, ts_out, ptr<int4>(cand));
    SP_HIP(hipGetLastError());
    sp_coords* fine = nullptr;
    SP_TRY(coords_build_impl(ptr<int32_t>(cand), n_cand, nullptr, 1, ts_out, nullptr, false, s, &fine));
    fine->on_lattice = in->on_lattice;

    // the stride-s convolution's map from the fine rows (inputs) to the coarse rows (outputs) ...
    std::unique_ptr<sp_kmap, int (*)(sp_kmap*)> m(new sp_kmap, sp_kmap_destroy);
    m->K = kernel_size;
    m->kvol = kvol;
    m->stride = stride;
    m->dilation = 1;
    m->stream = s;
    m->c_in = fine;  // takes over the reference
    sp_coords* coarse = const_cast<sp_coords*>(in);
    coarse->ref.fetch_add(1);
    m->c_out = coarse;
    SP_TRY(coords_resolve(fine));  // the created rows' count: the lists are sized from it, not from the candidates
    const int64_t n_fine = fine->n;
    const Count cn_fine{nullptr, n_fine}, cn_coarse{nullptr, n_coarse};
    if (n_fine * (int64_t)kvol >= ((int64_t)1 << 31) - 4096)
        return fail(SP_ERR_INVALID_ARG, "n * kernel volume exceeds 32-bit list offsets");
    const int nclass = (stride > 1 && stride * stride * stride <= 32) ? stride * stride * stride : 0;
    MapSide& so = m->out_side;
    MapSide& si = m->in_side;
    so.nbr = dev_alloc((size_t)(n_cand ? n_cand : 1) * 4, s);
    si.nbr = dev_alloc((size_t)(n_fine ? n_fine : 1) * kvol * 4, s);
    SP_TRY(reserve_lists(so, n_coarse, std::min(n_coarse, n_fine), kvol, s));
    m->d_counts = dev_alloc((size_t)(kvol + 1) * 4, s);
    Buf work = dev_alloc(counts_bytes(n_coarse, kvol), s);
    if (!so.nbr || !si.nbr || !m->d_counts || !work) return SP_ERR_ALLOC;
    const Counts counts = counts_in(work, n_coarse, kvol);
    if (n_fine > 0)
        hipLaunchKernelGGL(reset_kernel, dim3(blocks256((n_fine * (int64_t)kvol + 3) / 4)), dim3(kThreads), 0, s, ptr<int32_t>(si.nbr), cn_fine,
                           kvol);
    if (n_cand > 0)
        hipLaunchKernelGGL(gen_tables_kernel, dim3(blocks256(n_cand)), dim3(kThreads), 0, s, ptr<int32_t>(fine->inverse),
                           n_coarse, cn_fine, kvol, ptr<int32_t>(so.nbr), ptr<int32_t>(si.nbr));
    hipLaunchKernelGGL(count_kernel, dim3((unsigned)(tiles_of(n_coarse) ? tiles_of(n_coarse) : 1), chunks_of(kvol)), dim3(kTileRows), 0, s,
                       ptr<int32_t>(so.nbr), cn_coarse, kvol, counts, ptr<int32_t>(m->d_counts) + kvol);
    SP_HIP(hipGetLastError());
    SP_TRY(finish_map(m.get(), false, counts, n_fine, n_coarse, cn_fine, cn_coarse, nclass, s));
    // ... handed out with the roles swapped: inputs = the given (coarse) rows, outputs = the created rows
    sp_kmap_t* t = nullptr;
    SP_TRY(sp_kmap_transpose(m.get(), &t));
    if (out_coords) {
        fine->ref.fetch_add(1);
        *out_coords = fine;
    }
    *kmap = t;
    return SP_OK;
}

int sp_kmap_transpose(const sp_kmap_t* f, sp_kmap_t** transposed) {
    if (transposed) *transposed = nullptr;
    if (!f || !transposed) return fail(SP_ERR_INVALID_ARG, "kmap handle or out pointer is NULL");
    SP_TRY(kmap_resolve(f));
    sp_kmap* t = new sp_kmap;
    t->n_in = f->n_out;
    t->n_out = f->n_in;
    t->total = f->total;
    t->K = f->K;
    t->kvol = f->kvol;
    t->stride = f->stride;
    t->dilation = f->dilation;
    t->out_side = f->in_side;
    t->in_side = f->out_side;
    t->pair_in = f->pair_out;
    t->pair_out = f->pair_in;
    t->pair_stride = f->pair_stride;
    t->counts = f->counts;
    t->koff = f->koff;
    t->d_counts = f->d_counts;
    t->c_in = f->c_out;
    t->c_out = f->c_in;
    t->stream = f->stream;
    t->resolved = true;
    t->status = SP_OK;
    if (t->c_in) t->c_in->ref.fetch_add(1);
    if (t->c_out) t->c_out->ref.fetch_add(1);
    *transposed = t;
    return SP_OK;
}

int sp_kmap_info(const sp_kmap_t* m, int64_t* n_in, int64_t* n_out, int32_t* kvol, int64_t* total_pairs,
                 int64_t* h_counts) {
    if (!m) return fail(SP_ERR_INVALID_ARG, "kmap handle is NULL");
    if (kvol) *kvol = m->kvol;
    if (n_in || n_out || total_pairs || h_counts) SP_TRY(kmap_resolve(m));
    if (n_in) *n_in = m->n_in;
    if (n_out) *n_out = m->n_out;
    if (total_pairs) *total_pairs = m->total;
    if (h_counts)
        for (int k = 0; k < m->kvol; ++k) h_counts[k] = m->counts[k];
    return SP_OK;
}

int sp_kmap_pairs(const sp_kmap_t* m, const int32_t** d_pair_in, const int32_t** d_pair_out, int64_t* pair_stride) {
    if (!m) return fail(SP_ERR_INVALID_ARG, "kmap handle is NULL");
    if (d_pair_in) *d_pair_in = ptr<int32_t>(m->pair_in);
    if (d_pair_out) *d_pair_out = ptr<int32_t>(m->pair_out);
    if (pair_stride) *pair_stride = m->pair_stride;
    return SP_OK;
}

int sp_kmap_table(const sp_kmap_t* m, const int32_t** d_nbr_out, const int32_t** d_nbr_in, int32_t* out_reversed,
                  int32_t* in_reversed) {
    if (!m) return fail(SP_ERR_INVALID_ARG, "kmap handle is NULL");
    if (d_nbr_out) *d_nbr_out = ptr<int32_t>(m->out_side.nbr);
    if (d_nbr_in) *d_nbr_in = ptr<int32_t>(m->in_side.nbr);
    if (out_reversed) *out_reversed = m->out_side.flip ? 1 : 0;
    if (in_reversed) *in_reversed = m->in_side.flip ? 1 : 0;
    return SP_OK;
}

int sp_kmap_destroy(sp_kmap_t* m) {
    if (!m) return SP_OK;
    sp_coords_destroy(m->c_in);
    sp_coords_destroy(m->c_out);
    delete m;
    return SP_OK;
}

}  // extern "C"
