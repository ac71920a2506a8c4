// Step 3 of the generalized sparse convolution (Eq. 2) and its input gradient: dispatch over the gather-GEMM kernels,
// the wavefront-private link-list kernel and the plain one.
//
// All of them are destination stationary: a destination row (output row for the forward pass, input row for the
// data gradient) belongs to exactly one workgroup, its fp32 accumulator stays on the chip, links are added in a
// fixed order without atomics (results are reproducible run to run), and the result is written once, rounded once.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "sp_conv_tile.h"
#include "sp_internal.h"
#include "sp_split_shape.h"

namespace sp {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t bf16_t;  // storage

__device__ __forceinline__ float bf16_to_f32(bf16_t v) { return __uint_as_float((uint32_t)v << 16); }
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {  // round to nearest even; NaN stays NaN
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (bf16_t)((u >> 16) | 0x40);
    return (bf16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

struct GatherArgs {
    const int32_t* off;  // the side's lists (MapSide)
    const int32_t* src;
    const int32_t* dst;
    const void* f;   // source features [n_src][CC]
    const void* w;   // weights [kvol][co_total][CC] (contraction index fastest)
    void* g;         // destination features [n_rows][co_total]
    int64_t n_rows;
    int kvol;
    int co_total;
    int flip;        // weight matrix of list k is kvol-1-k
    int lds_per_wave;  // bytes of LDS of one wavefront in gather_wave_kernel
    int runs;          // sub-tiles are dealt to the XCDs in runs (xcd_run)
    int split_blocks;  // sub-tiles with at least this many 16-link blocks are shared by two wavefronts
    uint32_t f_bytes, w_bytes, list_bytes;  // sizes of f / w / src and dst for buffer addressing (< 4 GiB)
    int may_in_place;  // host-side only: ... instead of a copy into `scratch`, under capture, or if there is no memory for one
    int w_transposed;  // host-side only: the stored weights are [k][cc][co] (data gradient) instead of [k][co][cc]
    void* scratch;     // host-side only: if set, device memory for the weight copy instead of a pool allocation
    size_t scratch_bytes;
};

// ---------------------------------------------------------------------------------------------------------
// Narrow-channel variant: every wavefront owns 64 destination rows (one sub-tile) and all COT channels of a
// channel tile, and runs on its own: no workgroup barrier anywhere.
//
//  (Small launches: four wavefronts share a sub-tile, kWaveShare, and meet once, at the end.)
//  - The wavefront first cuts its links into blocks of up to 16 links of one offset and writes one packed
//    descriptor per block into LDS, so that block b+n is addressable without walking a cursor.
//  - Everything a block needs is requested well ahead of its use and kept in registers: link entries
//    (source row, destination row) 2*kDX = 6 blocks ahead, the gathered source rows kDX = 3 blocks ahead, the
//    weight matrix two blocks ahead (a matrix too large for two register copies: in halves, half a block ahead).
//  - Source rows are gathered with coalesced 16-byte loads (adjacent lanes = adjacent pieces of one row; a
//    fragment-shaped global load would cost one L1 tag lookup per lane) and pass through a small
//    wavefront-private LDS buffer to be re-read as MFMA fragments, one block ahead of the MFMAs using them.
//  - The offset's weight matrix is the MFMA A operand (rows = destination channels), read from a
//    fragment-major copy of the weights so that one wavefront load is 1 KB of consecutive bytes.  (In the
//    stored layout a lane's 16-byte piece is contiguous too, so the forward pass could skip the copy, but a
//    wavefront's load is then 16 stretches of 64 bytes: measured 81 us against 61 with the copy.)
//  - The gathered rows are the B operand (columns = links), so the product comes out transposed: a lane
//    holds 4 consecutive channels of ONE link and adds them with one 16-byte LDS read-modify-write to that
//    link's destination row in the wavefront's private fp32 accumulator.
// ---------------------------------------------------------------------------------------------------------
template <typename T, int CC, int COT>
struct WaveCfg {
    static constexpr bool kIsF32 = std::is_same<T, float>::value;
    static constexpr int kGroup = kIsF32 ? 16 : 32;       // contraction channels per 16-byte fragment group
    static constexpr int kGroups = CC / kGroup;
    static constexpr int kNCT = COT / 16;
    static constexpr int kStride = COT + 4;               // floats per accumulator row
    static constexpr int kAccBytes = 64 * kStride * 4;
    static constexpr int kRowBytes = CC * (int)sizeof(T); // one source row
    static constexpr int kPieces = kRowBytes / 16;        // 16-byte pieces per source row
    static constexpr int kXStride = kRowBytes + 32;       // staged row + pad (b128 fragment reads at the full LDS rate)
    static constexpr int kXBytes = 16 * kXStride - 32;  // the last row needs no pad
    static constexpr int kXLoads = (16 * kPieces + 63) / 64;  // coalesced load instructions per 16-link block
    // Up to 4 blocks per offset.  A descriptor says offset, links and which block of the offset it is, in 16 bits.  Where
    // the block's first link is, a table of the offsets' begins says (a second LDS trip), or, wide descriptors, a word per
    // block, read side by side with it.  The trip costs 64-byte rows 3-6 % (bf16 32 -> 64 on 0.6 M links 28.6 against 27.8 us);
    // the room costs wider rows, and every row beyond 27 offsets, a wavefront per CU (fp32 32 -> 64: 59 against 68 us; bf16
    // 32 -> 32, K = 5 on 0.37 M rows 140 against 172 us).  LDS is handed out in steps of 1280 bytes: wide descriptors of
    // 8 bytes took bf16 32 -> 32 at K = 3 from nine steps to ten, from 14 wavefronts a CU to 12 (0.22 M rows, one round of
    // wavefronts or two: 32 against 43 us), 4-byte descriptors fp32 32 -> 32 at K = 5 from 11 to 10 (0.37 M rows 303 against 334 us).
    static constexpr bool kMayWide = kRowBytes == 64;
    static bool wide(int kvol) { return kMayWide && kvol <= 27; }
    static int desc_bytes(int kvol) { return (kvol * (wide(kvol) ? 24 : 12) + 15) / 16 * 16; }
    static constexpr bool kMayRun = kRowBytes == 64 || !kIsF32;  // see xcd_run; the others gain nothing from it
    static int per_wave_bytes(int kvol) { return kAccBytes + kXBytes + desc_bytes(kvol); }
    // fragment-major weights: [kvol][co_total/COT][kNCT][kGroups][64 lanes][16 bytes]
    static constexpr size_t kWFragBytesPerOffsetTile = (size_t)kNCT * kGroups * 64 * 16;
};

__device__ __forceinline__ void wave_sync() {
    // LDS traffic of one wavefront is processed in order; this only stops the compiler from moving
    // the wavefront's own LDS accesses across the point.
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Workgroup -> sub-tile such that an XCD (workgroup id % 8) takes runs of kRun neighbours.  A sub-tile's stretch of an
// offset's list is half a cache line or less: neighbours on one XCD fetch the line once.  Large launches only (kRunRows):
// bf16 32 -> 32 on 0.37 M rows 56.2 -> 53.5 us, 0.62 M rows 103 -> 95, on 0.16 M rows equal; 64 -> 128 on 0.1 M rows,
// which fill the chip once and a half, 61.5 -> 66.
constexpr int kRun = 8;
constexpr int64_t kRunRows = 1 << 17;
__device__ __forceinline__ int64_t xcd_run(int64_t wg) { return wg / (8 * kRun) * (8 * kRun) + (wg & 7) * kRun + (wg >> 3) % kRun; }

// kShare wavefronts share a sub-tile, each a stretch of its blocks with an accumulator of its own; the accumulators are added at
// the end.  For launches whose length is one sub-tile's chain of blocks (share_fits).
// kStored: the weights are read as they are stored, [kvol][co_total][CC], instead of from the fragment-major copy.
template <typename T, int CC, int COT, bool kWideDesc, int kShare, bool kStored>
__global__ __launch_bounds__(64 * kShare) void gather_wave_kernel(GatherArgs a) {
    using Cfg = WaveCfg<T, CC, COT>;
    constexpr bool kIsF32 = Cfg::kIsF32;
    constexpr int kGroups = Cfg::kGroups, kNCT = Cfg::kNCT, kPieces = Cfg::kPieces, kXLoads = Cfg::kXLoads;
    using Frag = typename std::conditional<kIsF32, f32x4, bf16x8>::type;  // 16 bytes
    static_assert(CC % Cfg::kGroup == 0, "contraction channels must fill whole fragment groups");
    static_assert(kPieces % 4 == 0, "a source row must be a multiple of 64 bytes");
    // Blocks whose gathers are in flight, and blocks whose weights are.  A gather is two dependent trips to
    // memory behind the entry loads and mostly misses the L2; the weights are one trip that mostly hits.  Rows
    // cost few registers per block and weights many, so narrow rows are fetched deep and weights shallow.
    constexpr int kDX = 3;  // loads return in order: a deeper ring for the rows alone would still wait for the weights issued after it
    constexpr int kDW = 2;
    // A weight matrix of more than 32 fragment registers (e.g. fp32 64 x 64) does not fit a ring of two whole
    // matrices.  Then the two weight slots hold the two halves (channel tiles 0..kNCT/2-1 and the rest) of ONE
    // block's matrix: a half is re-requested for the next block as soon as this block's MFMAs on it are issued,
    // i.e. half a block ahead of its next use, which is enough for a matrix that lives in L2.
    constexpr bool kHalfW = kNCT * kGroups > 8;
    constexpr int kWT = kHalfW ? kNCT / 2 : kNCT;  // channel tiles per weight slot
    static_assert(!kHalfW || kNCT % 2 == 0, "halves");
    constexpr int kTurn = 6;  // bodies per loop turn: a multiple of kDX, kDW and the two result sets
    static_assert(kTurn % kDX == 0 && kTurn % kDW == 0 && kTurn % 2 == 0, "ring sizes must divide the turn");

    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = kShare == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // grid.x = 2 * sub-tiles: the first half of the grid takes half 0 (or the whole sub-tile), the second half
    // of the grid half 1.  (Workgroups are dealt to the 8 XCDs round-robin: pairing (u,0),(u,1) on adjacent
    // indices would leave every other XCD with nothing but wavefronts that leave at once.)
    const int64_t nwt = (a.n_rows + 63) / 64;
    const bool runs = Cfg::kMayRun && a.runs;
    const int half = !runs && blockIdx.x >= nwt ? 1 : 0;  // which 32-row half it takes if the sub-tile is split
    const int64_t wt = runs ? xcd_run(blockIdx.x) : (int64_t)blockIdx.x - (half ? nwt : 0);  // this wavefront's sub-tile
    if (Cfg::kMayRun && wt >= nwt) return;
    const int kvol = a.kvol;
    unsigned char* base = smem + wave * a.lds_per_wave;
    float* acc = reinterpret_cast<float*>(base);
    unsigned char* xbuf = base + Cfg::kAccBytes;
    int* s_beg = reinterpret_cast<int*>(xbuf + Cfg::kXBytes);  // where this wavefront's links begin, per offset; kWideDesc: per block
    uint16_t* s_blk = reinterpret_cast<uint16_t*>(s_beg + (kWideDesc ? 4 : 1) * kvol);  // the blocks' descriptors
    const int n16 = lane & 15, g = lane >> 4;

    for (int i = lane; i < Cfg::kAccBytes / 16; i += 64) reinterpret_cast<f32x4*>(acc)[i] = f32x4{0.f, 0.f, 0.f, 0.f};

    // ---- block descriptors: k | (links-1) << 7 | (block of the offset) << 11
    // Two wavefronts are launched per sub-tile.  When the launch is small (a.split_blocks set by the host)
    // and the sub-tile is long, each takes one 32-row half, which halves the longest dependent chain of the
    // launch; otherwise the first takes all 64 rows and the second leaves.
    const int32_t* __restrict__ offp = a.off + wt * kvol * kHalves;
    const int32_t* __restrict__ offn = offp + kvol * kHalves;  // the next sub-tile's begins: this one's ends
    int nblk_whole = 0;
    for (int kb = 0; kb < kvol; kb += 64) {
        const int k = kb + lane;
        int nb = k < kvol ? (offn[k * kHalves] - offp[k * kHalves] + 15) >> 4 : 0;
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) nb += __shfl_xor(nb, d, 64);
        nblk_whole += nb;
    }
    const bool split = nblk_whole >= a.split_blocks;
    if (!split && half == 1) return;
    const int row_base = split ? 32 * half : 0;
    const int row_count = split ? 32 : 64;
    int nblk = 0;
    for (int kb = 0; kb < kvol; kb += 64) {
        const int k = kb + lane;
        int o0 = 0, o1 = 0;
        if (k < kvol) {
            o0 = offp[k * kHalves + (split ? half : 0)];
            o1 = split && half == 0 ? offp[k * kHalves + 1] : offn[k * kHalves];
        }
        const int cnt = o1 - o0, nb = (cnt + 15) >> 4;
        int inc = nb;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int t = __shfl_up(inc, d, 64);
            if (lane >= d) inc += t;
        }
        const int ex = nblk + inc - nb;
        if (!kWideDesc && k < kvol) s_beg[k] = o0;
        for (int i = 0; i < nb; ++i) {
            s_blk[ex + i] = (uint16_t)(k | ((min(16, cnt - 16 * i) - 1) << 7) | (i << 11));
            if (kWideDesc) s_beg[ex + i] = o0 + 16 * i;
        }
        nblk += __shfl(inc, 63, 64);
    }
    wave_sync();
    // this wavefront's blocks: all, or its share of them
    const int b0 = kShare == 1 ? 0 : nblk * wave / kShare, b1 = kShare == 1 ? nblk : nblk * (wave + 1) / kShare;

    // Buffer addressing: a 32-bit byte offset per lane against a descriptor in scalar registers costs one
    // integer multiply-add per load instead of 64-bit pointer arithmetic, and reads past the end return 0.
    constexpr int kRsrcFlags = 0x00020000;
    const __amdgpu_buffer_rsrc_t rF = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.f), 0, (int)a.f_bytes, kRsrcFlags);
    const __amdgpu_buffer_rsrc_t rW = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.w), 0, (int)a.w_bytes, kRsrcFlags);
    const __amdgpu_buffer_rsrc_t rSrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(a.src), 0, (int)a.list_bytes, kRsrcFlags);
    const __amdgpu_buffer_rsrc_t rRow =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(a.dst), 0, (int)a.list_bytes, kRsrcFlags);
    const uint32_t w_tile_off = (uint32_t)(blockIdx.y * Cfg::kWFragBytesPerOffsetTile);  // (the same in both layouts)
    const int w_lane = kStored ? n16 * Cfg::kRowBytes + g * 16 : lane * 16;
    const uint32_t w_offset_stride = (uint32_t)((a.co_total / COT) * Cfg::kWFragBytesPerOffsetTile);

    auto load_weights = [&](int k, Frag (&wf)[kWT][kGroups], int ct0) __attribute__((always_inline)) {
        const int wk = a.flip ? kvol - 1 - k : k;
        // the offset index is the same in every lane, but it came through LDS: tell the compiler
        const int soff = __builtin_amdgcn_readfirstlane((int)(w_tile_off + (uint32_t)wk * w_offset_stride));
#pragma unroll
        for (int ct = 0; ct < kWT; ++ct)
#pragma unroll
            for (int s = 0; s < kGroups; ++s)
                wf[ct][s] = __builtin_bit_cast(
                    Frag, __builtin_amdgcn_raw_buffer_load_b128(rW, w_lane + (kStored ? (ct0 + ct) * 16 * Cfg::kRowBytes + s * 64 : ((ct0 + ct) * kGroups + s) * 1024), soff, 0));
    };

    // The main loop is straight-line code with the same loads in every turn (blocks past the end are
    // clamped to the last one and their results dropped): the compiler can then count outstanding loads
    // exactly and wait only for the oldest, instead of draining the whole prefetch queue at every branch.
    struct Slot {
        int dc;                   // descriptor of the block whose gathered rows are in x
        int drow;                 // destination row of that block's link n16
        int de;                   // descriptor of the block whose entries are in esrc / erow
        int esrc[kXLoads];        // source row of the link this lane gathers a piece of, per load
        int erow;                 // destination row of link n16
        u32x4 x[kXLoads];         // gathered pieces, coalesced layout: piece (t*64 + lane) of the block
    };
    struct WSlot {
        Frag w[kWT][kGroups];     // a block's weight matrix (kHalfW: one half of it)
    };
    const int last = b1 - 1;
    // (Starting each wavefront at a block of its own, so that the wavefronts of a compute unit do not ask for
    // the same weight lines at the same moment, was measured and is slower: in step, they share the lines in L1.)
    auto request = [&](Slot& sl, int de, int e0) __attribute__((always_inline)) {
        sl.de = de;
        const int cnt = ((de >> 7) & 15) + 1;
#pragma unroll
        for (int t = 0; t < kXLoads; ++t)
            sl.esrc[t] = (int)__builtin_amdgcn_raw_buffer_load_b32(rSrc, (e0 + min((t * 64 + lane) / kPieces, cnt - 1)) * 4, 0, 0);
        sl.erow = (int)__builtin_amdgcn_raw_buffer_load_b32(rRow, (e0 + min(n16, cnt - 1)) * 4, 0, 0);
    };
    auto look_up = [&](Slot& sl, int b) __attribute__((always_inline)) {
        const int de = s_blk[min(b, last)];
        request(sl, de, kWideDesc ? s_beg[min(b, last)] : s_beg[de & 127] + ((de >> 11) << 4));
    };
    // bf16 rows of 128 bytes and more: in the main loop, which asks for blocks in order, the descriptors run ahead in registers,
    // b's was read two calls ago (64 -> 128 on 2.4 M links 193 -> 188 us, 64 -> 32 on 0.22 M rows 53 -> 50; fp32, whose turns are
    // longer, loses 1 % by the registers).  The first blocks are looked up directly: their trips overlap.
    constexpr bool kAhead = !kWideDesc && !kIsF32;
    int de_0 = 0, de_1 = 0, beg_0 = 0;
    auto run_ahead = [&](int b) __attribute__((always_inline)) {
        if constexpr (kAhead) {
            de_0 = s_blk[min(b, last)];
            de_1 = s_blk[min(b + 1, last)];
            beg_0 = s_beg[de_0 & 127];
        }
    };
    auto load_entries = [&](Slot& sl, int b) __attribute__((always_inline)) {
        if constexpr (kAhead) {
            request(sl, de_0, beg_0 + ((de_0 >> 11) << 4));
            de_0 = de_1;
            beg_0 = s_beg[de_1 & 127];
            de_1 = s_blk[min(b + 2, last)];
        } else {
            look_up(sl, b);
        }
    };
    auto issue_gather = [&](Slot& sl) __attribute__((always_inline)) {
        sl.dc = sl.de;
        sl.drow = (sl.erow & 63) - row_base;
#pragma unroll
        for (int t = 0; t < kXLoads; ++t)
            sl.x[t] = __builtin_amdgcn_raw_buffer_load_b128(rF, sl.esrc[t] * Cfg::kRowBytes + ((t * 64 + lane) % kPieces) * 16, 0, 0);
    };
    auto issue_weights = [&](WSlot& ws, int b, int ct0 = 0) __attribute__((always_inline)) {
        load_weights(s_blk[min(b, last)] & 127, ws.w, ct0);
    };
    auto stage = [&](const Slot& sl) __attribute__((always_inline)) {  // gathered rows -> LDS, row-major, padded
#pragma unroll
        for (int t = 0; t < kXLoads; ++t) {
            const int idx = t * 64 + lane;
            *reinterpret_cast<u32x4*>(xbuf + (idx / kPieces) * Cfg::kXStride + (idx % kPieces) * 16) = sl.x[t];
        }
    };
    auto read_frags = [&](Frag (&xf)[kGroups]) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < kGroups; ++s)
            xf[s] = *reinterpret_cast<const Frag*>(xbuf + n16 * Cfg::kXStride + s * 64 + g * 16);
    };

    if (b1 > b0) {
        Slot xs[kDX] = {};
        WSlot ws[kDW] = {};
#pragma unroll
        for (int j = 0; j < kDX; ++j) look_up(xs[j], b0 + j);
#pragma unroll
        for (int j = 0; j < kDW; ++j) {
            if constexpr (kHalfW) issue_weights(ws[j], b0, j * kWT);  // both halves of the first block
            else issue_weights(ws[j], b0 + j);
        }
#pragma unroll
        for (int j = 0; j < kDX; ++j) issue_gather(xs[j]);
#pragma unroll
        for (int j = 0; j < kDX; ++j) look_up(xs[j], b0 + kDX + j);
        run_ahead(b0 + 2 * kDX);
        Frag xf_c[kGroups];
        stage(xs[0]);
        wave_sync();
        read_frags(xf_c);
        wave_sync();

        // One block: sl holds block b, sn holds block b + 1.  A wavefront issues in order, so the block's
        // MFMAs only overlap with its other work if that work does not depend on them and is interleaved
        // with them: the accumulator update of block b-1, the staging of block b+1 and the loads for
        // later blocks are therefore issued between the MFMAs of block b.
        // Two result sets alternate, so a block's products stay where the MFMAs left them until the next
        // block's turn adds them to the accumulator.
        struct Result {
            f32x4 d[kNCT];  // d[ct][i] = channel ct*16 + 4*g + i of link n16 of the block
            float* dst;     // accumulator row of that link (+ 4*g)
            bool valid;     // this lane's link exists
        };
        Result res[2] = {};
        res[0].dst = res[1].dst = acc + g * 4;
        // the accumulator rows are read at the start of a turn and written back at its end, so the LDS
        // latency is paid once, under the turn's MFMAs
        auto flush_read = [&](const Result& r, f32x4 (&av)[kNCT]) __attribute__((always_inline)) {
#pragma unroll
            for (int ct = 0; ct < kNCT; ++ct) av[ct] = *reinterpret_cast<const f32x4*>(r.dst + ct * 16);
        };
        // (Letting lanes without a link update spare LDS bytes instead, one row for all or 16 bytes per lane, makes
        // a turn one basic block in which the compiler deals the update and the loads out between the MFMAs;
        // both were measured at 73-76 us against 62 with this branch.)
        auto flush_write = [&](const Result& r, const f32x4 (&av)[kNCT]) __attribute__((always_inline)) {
            if (r.valid) {
#pragma unroll
                for (int ct = 0; ct < kNCT; ++ct) *reinterpret_cast<f32x4*>(r.dst + ct * 16) = av[ct] + r.d[ct];
            }
        };
        auto mfmas = [&](Result& cur, const WSlot& wl, int ct0, const Frag (&xf)[kGroups]) __attribute__((always_inline)) {
#pragma unroll
            for (int s = 0; s < kGroups; ++s)
#pragma unroll
                for (int c = 0; c < kWT; ++c) {
                    const int ct = ct0 + c;
                    if constexpr (kIsF32) {
                        cur.d[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(wl.w[c][s][0], xf[s][0], cur.d[ct], 0, 0, 0);
                        cur.d[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(wl.w[c][s][1], xf[s][1], cur.d[ct], 0, 0, 0);
                        cur.d[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(wl.w[c][s][2], xf[s][2], cur.d[ct], 0, 0, 0);
                        cur.d[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(wl.w[c][s][3], xf[s][3], cur.d[ct], 0, 0, 0);
                    } else {
                        cur.d[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wl.w[c][s], xf[s], cur.d[ct], 0, 0, 0);
                    }
                }
        };
        auto body = [&](int b, Slot& sl, const Slot& sn, WSlot& wl, WSlot& wl2, Result& cur, const Result& prev) __attribute__((always_inline)) {
            const int cnt = ((sl.dc >> 7) & 15) + 1;
            cur.valid = n16 < cnt;
            cur.dst = acc + sl.drow * Cfg::kStride + g * 4;
            stage(sn);  // the next block's rows (this block's fragments are already in registers)
            wave_sync();
            f32x4 av[kNCT];
            flush_read(prev, av);
            Frag xf_n[kGroups];
            read_frags(xf_n);

#pragma unroll
            for (int ct = 0; ct < kNCT; ++ct) cur.d[ct] = f32x4{0.f, 0.f, 0.f, 0.f};
            if constexpr (kHalfW) {
                mfmas(cur, wl, 0, xf_c);
                issue_weights(wl, b + 1, 0);        // first half of the next block's matrix
                mfmas(cur, wl2, kWT, xf_c);
                issue_gather(sl);
                load_entries(sl, b + 2 * kDX);
                issue_weights(wl2, b + 1, kWT);     // its second half
            } else {
                mfmas(cur, wl, 0, xf_c);
                issue_gather(sl);               // block b + kDX: its entries arrived kDX turns ago
                load_entries(sl, b + 2 * kDX);
                issue_weights(wl, b + kDW);
            }
            flush_write(prev, av);
#pragma unroll
            for (int s = 0; s < kGroups; ++s) xf_c[s] = xf_n[s];
            // scheduling hint: one MFMA, then a few of the other instructions, repeated
            if constexpr (kIsF32) {
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
                    __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);  // VALU
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // DS read
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
                    __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);  // VMEM read
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
                    __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);  // DS write
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
                    __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
                }
            }
        };
        int done = b0;  // blocks computed, the ones before b0 counted; the last one's result is still to be added
        for (int b = b0; b < b1; b += kTurn) {
            bool stop = false;
#pragma unroll
            for (int j = 0; j < kTurn; ++j) {
                if (!stop) {
                    body(b + j, xs[j % kDX], xs[(j + 1) % kDX], ws[kHalfW ? 0 : j % kDW], ws[1], res[j % 2], res[(j + 1) % 2]);
                    done = b + j + 1;
                    stop = b + j + 1 >= b1;
                }
            }
        }
        f32x4 av[kNCT];
        if ((done - b0 + 1) % 2 == 0) { flush_read(res[0], av); flush_write(res[0], av); }  // the set of block done-1
        else { flush_read(res[1], av); flush_write(res[1], av); }
    }
    if constexpr (kShare == 1) wave_sync();
    else __syncthreads();
    const int co0 = blockIdx.y * COT;
    constexpr int kQuads = COT / 4;
    for (int idx = threadIdx.x; idx < row_count * kQuads; idx += 64 * kShare) {
        const int r = idx / kQuads, c4 = (idx % kQuads) * 4;
        const int64_t row = wt * 64 + row_base + r;
        if (row >= a.n_rows) break;
        f32x4 v = *reinterpret_cast<const f32x4*>(smem + (r * Cfg::kStride + c4) * 4);
#pragma unroll
        for (int w = 1; w < kShare; ++w) v += *reinterpret_cast<const f32x4*>(smem + w * a.lds_per_wave + (r * Cfg::kStride + c4) * 4);
        if constexpr (kIsF32) {
            *reinterpret_cast<f32x4*>(static_cast<float*>(a.g) + row * a.co_total + co0 + c4) = v;
        } else {
            ushort4 o;
            o.x = f32_to_bf16(v[0]);
            o.y = f32_to_bf16(v[1]);
            o.z = f32_to_bf16(v[2]);
            o.w = f32_to_bf16(v[3]);
            *reinterpret_cast<ushort4*>(static_cast<bf16_t*>(a.g) + row * a.co_total + co0 + c4) = o;
        }
    }
}

// Weights as stored (element (k, co, cc) at w[k*per + co*s_co + cc*s_cc]) -> fragment-major copy for
// gather_wave_kernel: [k][co tile][ct][s][lane = n16 + 16*g][16 bytes] holding channels
// co = tile*COT + ct*16 + n16, cc = s*kGroup + g*(kGroup/4) + 0..kGroup/4-1.
template <typename T, int CC, int COT>
__global__ __launch_bounds__(256) void weight_frag_kernel(const T* __restrict__ w, T* __restrict__ wf, int kvol,
                                                          int co_total, int s_co, int s_cc) {
    using Cfg = WaveCfg<T, CC, COT>;
    constexpr int kPer = Cfg::kGroup / 4;  // elements per 16-byte fragment
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t total = (int64_t)kvol * co_total * CC;
    if (idx >= total) return;
    int64_t r = idx;
    const int i = (int)(r % kPer); r /= kPer;
    const int lane = (int)(r % 64); r /= 64;
    const int s = (int)(r % Cfg::kGroups); r /= Cfg::kGroups;
    const int ct = (int)(r % Cfg::kNCT); r /= Cfg::kNCT;
    const int tile = (int)(r % (co_total / COT)); r /= (co_total / COT);
    const int k = (int)r;
    const int co = tile * COT + ct * 16 + (lane & 15);
    const int cc = s * Cfg::kGroup + (lane >> 4) * kPer + i;
    wf[idx] = w[(size_t)k * co_total * CC + (size_t)co * s_co + (size_t)cc * s_cc];
}

template <typename T, int CC, int COT, bool kWideDesc, int kShare, bool kStored>
int run_wave(const GatherArgs& a, dim3 grid, hipStream_t s) {
    auto kern = gather_wave_kernel<T, CC, COT, kWideDesc, kShare, kStored>;
    const int lds = a.lds_per_wave * kShare;
    {
        static std::mutex mu;
        static int attr_lds = 0;  // largest dynamic LDS size opted into so far
        std::lock_guard<std::mutex> lk(mu);
        if (lds > attr_lds) {
            SP_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds));
            attr_lds = lds;
        }
    }
    hipLaunchKernelGGL(kern, grid, dim3(64 * kShare), lds, s, a);
    SP_HIP(hipGetLastError());
    return SP_OK;
}

// LDS is handed out in steps of 1280 bytes: workgroups of a launch that the GPU's 256 CUs hold at once
inline int64_t resident_wgs(int64_t lds) { return 256 * (160 * 1024 / ((lds + 1279) / 1280 * 1280)); }

// Four wavefronts per sub-tile where all sub-tiles then still fit the GPU at once: such a launch is as long as one sub-tile's
// chain of 27 and more blocks, each behind the one before it.  Forward in us, one wavefront / four (host included, 10 us at
// least), K = 3 on 1.5 k rows with 4.6 k links | 16 k, 67 k | 32 k, 0.22 M:
//   fp32 16 -> 16   15.1 / 9.9  | 15.0 / 9.8  | 17.5 / 10.5     bf16 32 -> 32   15.9 / 10.4 | 16.3 / 9.8  | 18.5 / 11.0
//   fp32 32 -> 32   18 / 11.8   | 21.9 / 11.8 | 27.7 / 16.4     bf16 64 -> 64   20.4 / 11.7 | 20.8 / 12.3 | 30 / 18.1
// Where they do not fit the blocks of all sub-tiles matter and not the longest chain: bf16 32 -> 32 on 64 k rows, 0.83 M links 23.3
// / 26.5, fp32 64 -> 32 63 / 75.  Eight wavefronts gain nothing over four.
constexpr int kWaveShare = 4;
inline int64_t wave_lds(int cc, int cot, int elt, int kvol) {
    return 64 * (cot + 4) * 4 + 16 * (cc * elt + 32) - 32 + (kvol * (cc * elt == 64 && kvol <= 27 ? 24 : 12) + 15) / 16 * 16;
}
inline bool share_fits(int64_t waves, int64_t lds_per_wave) { return waves <= resident_wgs(kWaveShare * lds_per_wave); }

template <typename T, int CC, int COT, bool kWideDesc>
int launch_wave(GatherArgs a, hipStream_t s) {
    using Cfg = WaveCfg<T, CC, COT>;
    if constexpr (!kWideDesc && Cfg::kMayWide)
        if (Cfg::wide(a.kvol)) return launch_wave<T, CC, COT, true>(a, s);
    a.lds_per_wave = Cfg::per_wave_bytes(a.kvol);
    a.w_bytes = (uint32_t)((size_t)a.kvol * a.co_total * CC * sizeof(T));
    const int64_t nwt = (a.n_rows + 63) / 64, waves = nwt * (a.co_total / COT);
    const bool share = share_fits(waves, a.lds_per_wave);
    // A shared sub-tile's wavefronts read few matrices each: small ones are read as they are stored, 16 stretches of 64 bytes a load
    // instead of 1 KB, which saves the copy's launch (fp32 16 -> 16 on 1.5 k rows 9.9 -> 8.4 us, 32 -> 32 11.8 -> 9.7; 32 -> 32 on
    // 32 k rows 16.4 -> 17.9, bf16 64 -> 64 on 1.5 k 11.7 -> 14.4).
    constexpr int kMatrix = CC * COT * (int)sizeof(T);
    bool stored = !a.w_transposed && ((share && (kMatrix <= 2048 || (kMatrix <= 4096 && waves <= 256))) || (a.scratch && a.may_in_place));
    const int64_t n = (int64_t)a.kvol * a.co_total * CC;
    if (a.scratch && !a.may_in_place && (size_t)n * sizeof(T) > a.scratch_bytes)  // the same layers at every size of the map
        return fail(SP_ERR_UNSUPPORTED, "weights of %lld bytes exceed the %zu bytes of static scratch",
                    (long long)(n * sizeof(T)), a.scratch_bytes);
    Buf wf;
    if (!stored && !a.scratch && !a.w_transposed && a.may_in_place) {  // a graph must not hold on to a block of the pool
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(s, &cap) != hipSuccess) (void)hipGetLastError();
        stored = cap != hipStreamCaptureStatusNone;
    }
    if (!stored && !a.scratch) {
        wf = dev_alloc((size_t)n * sizeof(T), s);
        stored = !wf && !a.w_transposed && a.may_in_place;
        if (!wf && !stored) return SP_ERR_ALLOC;
    }
    if (!stored) {  // fragment-major copy of the weights (also undoes the data gradient's transposition)
        T* d_wf = a.scratch ? static_cast<T*>(a.scratch) : ptr<T>(wf);
        const int s_co = a.w_transposed ? 1 : CC, s_cc = a.w_transposed ? a.co_total : 1;
        hipLaunchKernelGGL((weight_frag_kernel<T, CC, COT>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                           static_cast<const T*>(a.w), d_wf, a.kvol, a.co_total, s_co, s_cc);
        a.w = d_wf;
    }
    // A launch whose sub-tiles fit the GPU's LDS at once runs as long as its longest wavefront: then long
    // sub-tiles (48 blocks and more at 27 offsets, against a typical 27-35; measured best of 32..64) are shared by two
    // wavefronts.  More offsets have more blocks, all of them: sharing every sub-tile pays only if the halves fit at once too
    // (K = 5, bf16 32 -> 32 on 0.15 M rows: 108-119 us with every sub-tile shared, 63 with none).  Larger launches run in
    // several rounds, where splitting would only add padding.
    const int64_t resident = resident_wgs(a.lds_per_wave);
    a.split_blocks = 2 * waves <= resident ? 48 : (waves * 5 / 4 <= resident ? std::max(48, 48 * a.kvol / 27) : 0x7fffffff);
    a.runs = Cfg::kMayRun && a.split_blocks == 0x7fffffff && a.n_rows >= kRunRows ? 1 : 0;
    // two wavefronts per sub-tile only where sub-tiles may be split (the second one leaves at once otherwise)
    const int64_t wgs = a.runs ? (nwt + 8 * kRun - 1) / (8 * kRun) * (8 * kRun) : (a.split_blocks == 0x7fffffff ? 1 : 2) * nwt;
    const dim3 grid((unsigned)wgs, (unsigned)(a.co_total / COT));
    // (the copy goes back to the pool; later users are ordered behind this launch on the stream)
    if constexpr (kMatrix <= 4096 || (!Cfg::kIsF32 && CC >= 64))
        if (share && stored) return run_wave<T, CC, COT, kWideDesc, kWaveShare, true>(a, grid, s);
    if constexpr (!Cfg::kIsF32 && CC >= 64)
        if (stored) return run_wave<T, CC, COT, kWideDesc, 1, true>(a, grid, s);
    return share ? run_wave<T, CC, COT, kWideDesc, kWaveShare, false>(a, grid, s) : run_wave<T, CC, COT, kWideDesc, 1, false>(a, grid, s);
}

// Plain kernel for what the other kernels' 32-bit buffer offsets cannot address: one thread per (row, channel),
// walking the neighbour table.  Weights as stored, W[kvol][cout][cin]; (w_cc, w_co) are the element strides
// of the contraction / destination channel inside one offset's matrix.
template <typename T>
__global__ __launch_bounds__(256) void gather_plain_kernel(const int32_t* __restrict__ nbr, int64_t n_rows, int kvol,
                                                           int flip, const T* __restrict__ F, const T* __restrict__ W,
                                                           T* __restrict__ G, int cc, int co, int w_cc, int w_co) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= n_rows * co) return;
    const int64_t row = idx / co;
    const int c = (int)(idx % co);
    float acc = 0.f;
    for (int kk = 0; kk < kvol; ++kk) {
        const int32_t src = nbr[(int64_t)kk * n_rows + row];
        if (src < 0) continue;
        const int wk = flip ? kvol - 1 - kk : kk;
        const T* wp = W + (size_t)wk * cc * co + (size_t)c * w_co;
        const T* fp = F + (size_t)src * cc;
        // one link's dot product first, then added: a single chain over all kvol * cc terms (6000 for a 5x5x5
        // kernel on 48 channels) measured 8e-6 against the fp64 definition, this 1e-6
        float dot = 0.f;
        for (int j = 0; j < cc; ++j) {
            if constexpr (std::is_same<T, float>::value)
                dot = fmaf(wp[(size_t)j * w_cc], fp[j], dot);
            else
                dot = fmaf(bf16_to_f32(wp[(size_t)j * w_cc]), bf16_to_f32(fp[j]), dot);
        }
        acc += dot;
    }
    if constexpr (std::is_same<T, float>::value)
        G[idx] = acc;
    else
        G[idx] = f32_to_bf16(acc);
}

// W[kvol][cout][cin] -> Wt[kvol][cin][cout]
template <typename T>
__global__ __launch_bounds__(256) void transpose_w_kernel(const T* __restrict__ w, T* __restrict__ wt, int kvol,
                                                          int cout, int cin) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t per = (int64_t)cout * cin;
    if (idx >= per * kvol) return;
    const int k = (int)(idx / per);
    const int rem = (int)(idx % per);
    const int ci = rem / cout, co = rem % cout;  // destination order
    wt[idx] = w[(size_t)k * per + (size_t)co * cin + ci];
}

// Narrow layers take the wavefront-private kernel, with the widest channel tile whose weight matrix fits in
// 32 fragment registers (CC/group * COT/16 fragments of 4 registers each).  Returns that tile, or 0 when the tile
// kernel takes the layer.
int wave_tile(int cc, int co, bool is_f32) {
    const int groups = cc / (is_f32 ? 16 : 32);
    if (groups * 4 <= 16 && co % 64 == 0) return 64;  // more than 8 fragments per lane: the matrix is held in two halves
    if (groups * 2 <= 8 && co % 32 == 0) return 32;
    if (groups <= 2 && (co == 16 || co == 48)) return 16;
    return 0;
}

template <typename T, int CC>
int dispatch_co(const GatherArgs& a, hipStream_t s) {
    constexpr int kGroups = CC / (std::is_same<T, float>::value ? 16 : 32);
    const int cot = wave_tile(CC, a.co_total, std::is_same<T, float>::value);
    if constexpr (kGroups * 4 <= 16)
        if (cot == 64) return launch_wave<T, CC, 64, false>(a, s);
    if constexpr (kGroups * 2 <= 8)
        if (cot == 32) return launch_wave<T, CC, 32, false>(a, s);
    if constexpr (kGroups <= 2)
        if (cot == 16) return launch_wave<T, CC, 16, false>(a, s);
    return fail(SP_ERR_UNSUPPORTED, "internal: no wavefront kernel for %d -> %d channels", CC, a.co_total);
}

template <typename T>
int dispatch_cc(int cc, const GatherArgs& a, hipStream_t s) {
    switch (cc) {
        case 16:
            if constexpr (std::is_same<T, float>::value) return dispatch_co<T, 16>(a, s);
            break;
        case 32: return dispatch_co<T, 32>(a, s);
        case 64: return dispatch_co<T, 64>(a, s);
        case 128: return dispatch_co<T, 128>(a, s);
        default: break;
    }
    return SP_ERR_UNSUPPORTED;
}

bool wave_shape_ok(int cc, int co, sp_dtype dt) {
    if (co % 16 != 0) return false;
    if (dt == SP_F32) return cc == 16 || cc == 32 || cc == 64;
    return cc == 32 || cc == 64 || cc == 128;
}

constexpr uint64_t kLim32 = 0xffffff00ull;
// The allocation-free entry point's scratch: copies of weights as they are, and pieces of fp32 weights, which take half as
// much again (what it refuses goes by the first).
constexpr size_t kStaticScratchBytes = (size_t)4 << 20;
constexpr size_t kSplitScratchBytes = kStaticScratchBytes / 2 * 3;
bool tile_big(const MapSide& side, int kvol, int cc, sp_dtype dt) {
    return (uint64_t)side.n_src * cc * (dt == SP_F32 ? 4 : 2) >= kLim32 || (uint64_t)side.pitch * kvol * 4 >= kLim32;
}

// The allocation-free entry point has room for this much of a weight copy.  Weights larger than that are read from where
// they are stored if they are whole fragments (a fragment load is then 16 stretches of 64 bytes instead of 1 KB in a
// row); other widths are left to the plain kernel.
bool tile_fits_scratch(const MapSide& side, int cc, int co, int kvol, sp_dtype dt, size_t scratch_bytes) {
    const TileShape t = tile_shape(cc, co, dt == SP_F32, tile_big(side, kvol, cc, dt));
    return tile_in_place_ok(t, cc) || tile_copy_bytes(t, kvol, dt == SP_F32 ? 4 : 2) <= scratch_bytes;
}

int conv_gather_tile(const MapSide& side, int kvol, const void* d_f, const void* d_w, bool w_transposed,
                     void* d_g, int cc, int co, sp_dtype dt, hipStream_t s, void* scratch, size_t scratch_bytes) {
    const bool f32 = dt == SP_F32;
    const int elt = f32 ? 4 : 2;
    const bool big = tile_big(side, kvol, cc, dt);
    const TileShape t = tile_shape(cc, co, f32, big);
    TileArgs a{};
    a.off = ptr<int32_t>(side.off);
    a.src = ptr<int32_t>(side.src);
    a.dst = ptr<int32_t>(side.dst);
    a.f = d_f;
    a.g = d_g;
    a.n_rows = side.n_rows;
    a.kvol = kvol;
    a.co = co;
    a.flip = side.flip ? 1 : 0;
    a.nsl = t.nsl;
    a.big = big ? 1 : 0;
    a.row_bytes = (uint32_t)(cc * elt);
    a.f_bytes = (uint32_t)((uint64_t)side.n_src * cc * elt);
    a.list_bytes = (uint32_t)((uint64_t)side.pitch * kvol * 4);
    const size_t copy = tile_copy_bytes(t, kvol, elt);
    const int groups = t.kc / (f32 ? 16 : 32);
    Buf wf;
    void* d_wf = scratch;
    if (!scratch) {
        wf = dev_alloc(copy, s);
        if (!wf && (w_transposed || !tile_in_place_ok(t, cc))) return SP_ERR_ALLOC;  // the caller has another way
        d_wf = wf ? wf->p : nullptr;
    } else if (copy > scratch_bytes) {
        d_wf = nullptr;
    }
    if (d_wf) {
        a.w = d_wf;
        a.wt = tile_weights_copied(t, kvol, elt);
        const int s_co = w_transposed ? 1 : cc, s_cc = w_transposed ? co : 1;
        const dim3 grid((unsigned)((copy / 16 + 255) / 256));
        if (f32)
            hipLaunchKernelGGL(tile_weights_kernel<float>, grid, dim3(256), 0, s, static_cast<const float*>(d_w),
                               static_cast<float*>(d_wf), kvol, co, cc, s_co, s_cc, t.ny, t.ncs, t.nsl, groups);
        else
            hipLaunchKernelGGL(tile_weights_kernel<bf16_t>, grid, dim3(256), 0, s, static_cast<const bf16_t*>(d_w),
                               static_cast<bf16_t*>(d_wf), kvol, co, cc, s_co, s_cc, t.ny, t.ncs, t.nsl, groups);
    } else {
        a.w = d_w;
        a.wt = tile_weights_in_place(t, kvol, cc, co, elt);
    }
    // 128-row tiles fill the 16-link blocks better, 64-row tiles give twice the workgroups and leave more LDS to
    // the tiles with several accumulators (ncs < 3)
    const int tr = t.ncs >= 3 && (side.n_rows + 127) / 128 * t.ny >= 512 ? 128 : 64;
    return f32 ? conv_tile_f32(a, t.kc, t.ncs, tr, s) : conv_tile_bf16(a, t.kc, t.ncs, tr, s);
}

}  // namespace

namespace {
// fp32: the split kernel against the one that has the layer otherwise (wave: the wavefront-private one).  Forward in us, before /
// split, on 1.5 k rows with 9 k links | 23 k, 0.14 M | 96 k, 0.61 M | 160 k, 0.66 M | 213 k, 2.4 M | 613 k, 5.0 M (one kernel's launches
// back to back, which takes the clock down: with pauses 64 -> 64 on the last takes 618 / 425):
// (wavefront-private: one wavefront a sub-tile; where four share one, 64 -> 64 takes 20 us on 1.5 k and 22 on 16 k rows, 32 -> 64
// 14 and 15, 32 k rows 24, the split kernel 25, 29, 20, 24 and 30: share_fits is the line.)
//   wavefront-private  64 -> 64    56 / 26 | 66 / 38  | 124 / 81  | 180 / 104 | 345 / 250  | 681 / 503
//                      32 -> 64    35 / 21 | 37 / 29  | 58 / 50   | 93 / 70   | 165 / 133  | 328 / 264
//                      64 -> 128   56 / 31 | 96 / 47  | 200 / 143 | 280 / 195 | 602 / 451  | 1180 / 853
//                      64 -> 32    36 / 28 | 39 / 39  | 64 / 73   | 100 / 97  | 194 / 227  | 373 / 418
//                      32 -> 32    25 / 22 | 26 / 30  | 40 / 52   | 62 / 65   | 108 / 114  | 202 / 210
//   tile               128 -> 128  66 / 50 | 130 / 78 | 362 / 264 | 446 / 322 | 1124 / 763 | 2484 / 1617
//                      160 -> 64   67 / 74 | 94 / 106 | 265 / 211 | 358 / 278 | 839 / 596  | 1755 / 1220
//                      96 -> 96    38 / 55 | 68 / 78  | 240 / 212 | 308 / 303 | 783 / 580  | 1743 / 1216
//                      24 -> 40    19 / 23 | 23 / 27  | 55 / 49   | 73 / 64   | 158 / 113  | 298 / 225
//                      48 -> 48    24 / 28 | 30 / 36  | 77 / 73   | 100 / 109 | 224 / 199  | 465 / 407
// The line between few and many rows (links of an offset in 128 rows: per):  50 k rows, per 49: 48 -> 48 76 / 65, 128 -> 64 213 / 129,
// 24 -> 40 47 / 48; 55 k, per 63: 48 -> 48 84 / 77, 128 -> 32 195 / 100, 24 -> 40 51 / 53; 48 -> 48, 96 k rows, per 30: 77 / 73, per 19:
// 105 / 109.  Padded ones of two channel tiles with more links (48 -> 80, 50 k to 62 k rows, split over tile kernel: per 25 0.93, per 28 0.96,
// per 31 0.98 to 1.04, per 46 to 69 0.97 to 1.12); tiles of 128 channels gain on both sides of it with few links too (48 -> 128, 50 k,
// per 10: 91 / 61; 60 k, per 12: 91 / 60, 36 -> 100 the same).
// Channel tiles of 32 leave its wavefronts too little to do per row: not in place of the wavefront-private kernel, and of the tile
// kernel only on large sets.  What the tile kernel pads a third less (48 channels, which are 64 here) only where many links share a
// read of the weights.  A read serves the links of one offset in a tile, padded to steps of 32 or 48: where a tile of 128 rows has few
// of an offset (per), the tile kernel's blocks of 16 are less work.  us, before / split, per and rows in front:
//   K = 3, stride 2, input side  per 10, 68 k rows   24 -> 40 26 / 34    64 -> 40 49 / 60    96 -> 96 106 / 125  72 -> 56 74 / 71    128 -> 64 92 / 88
//   K = 5                        per 11, 68 k        24 -> 40 106 / 109  64 -> 40 158 / 216  96 -> 96 413 / 519  72 -> 56 280 / 379  128 -> 64 439 / 355
//   K = 3                        per 37, 99 k                            64 -> 40 119 / 86   96 -> 96 294 / 221
//   128 -> 128                   K = 5, per 1.4, 16 k 71 / 94   K = 3, per 5.3, 16 k 39 / 45   K = 4, per 6.7, 20 k 188 / 104
//   padded                       36 -> 100, K = 3, per 14, 12 k 26 / 29, per 33, 8 k 32 / 36, per 84, 12 k 55 / 47, per 18, 20 k 48 / 35
//                                40 -> 24, K = 3, per 53, 146 k 139 / 158
// Of the wavefront-private kernel's layers it leaves K = 1 (64 -> 128 on 374 k rows 106 / 132, 32 -> 128 69 / 94), and 32 -> 128 channels on
// many rows with few links (K = 2, stride 2, input side, one link a row: 374 k rows 97 / 117, 30 k rows 21 / 17).
bool split_pays(const MapSide& side, int kvol, int64_t links, int cc, int co, bool wave) {
    if (cc % 4 != 0 || cc <= 16 || co <= 16 || kvol > 125) return false;
    const SplitShape t = split_shape(cc, co);
    if (split_copy_bytes(t, kvol) >= kLim32) return false;
    if (wave) {
        if (t.cot <= 32 || kvol == 1 || (kvol <= 8 && cc <= 32 && t.cot == 128 && side.n_rows >= 32768 && links < 5 * side.n_rows)) return false;
        return !share_fits((side.n_rows + 63) / 64 * (co / wave_tile(cc, co, true)), wave_lds(cc, wave_tile(cc, co, true), 4, kvol));
    }
    if (side.n_rows < 1024) return false;
    const TileShape o = tile_shape(cc, co, true, false);
    // More slices are more roundings: 80 -> 24 in three of 32 is 1.18e-7 of the rms off, 1.10e-7 in the tile kernel's two of 48.
    if (t.cot == 32 && t.nsl > o.nsl) return false;
    const double per = (double)links * 128.0 / ((double)side.n_rows * kvol);
    const bool padded = 10 * (int64_t)t.cc * t.nsl * t.cot * t.ny > 13 * (int64_t)o.kc * o.nsl * 16 * o.ncs * o.ny;
    const bool many_rows = side.n_rows >= (t.cc == 32 || t.cot == 128 ? 65536 : 49152);
    const double enough = !many_rows ? 40.0 : t.ny > 1 && side.n_rows < 65536 ? 31.0 : 26.0;
    if (padded && (t.cot == 32 || ((per < enough || kvol == 1) && (side.n_rows <= 16384 || many_rows)))) return false;
    if (!many_rows) return t.cot == 128 && per >= 6.0;
    return per >= (t.cot == 48 ? 20.0 : t.cot == 64 && t.cc == 32 ? 14.0 : 6.0);
}

bool dense_pays(const MapSide& side, int kvol, int64_t links, int cc) {
    return side.tile_mask || (double)links >= dense_min_fill(cc) * (double)side.n_rows * kvol;
}

// Small launches of layers that have a row-stationary kernel: its length is one tile's chain of kvol steps, whatever the number of
// rows, and few CUs have one; the wavefront-private kernel's follows the blocks.  Line: sub-tiles times channel tiles, times
// the blocks of 16 links an offset has in one on average (estimated).  Forward in us, row-stationary / wavefront-private, K = 3 on
// 1 k rows with 11 k links | 16 k, 67 k | 16 k, 0.39 M | 32 k, 0.22 M | 48 k, 0.48 M (- : the link-list kernel before, too):
//   64 -> 64    29 / 12 | - | 29 / 20 | 30 / 18 | 32 / 27       128 -> 64   44 / 14 | 45 / 16 | 50 / 34 | 47 / 35 | 48 / 45
//   64 -> 128   37 / 12 | - | 38 / 33 | 40 / 32 | 42 / 47       128 -> 128  60 / 15 | 61 / 29 | 65 / 47 | 64 / 43 | 64 / 77
//   64 -> 256   49 / 13 | - | 52 / 48 | 53 / 44 | 55 / 78       128 -> 256  76 / 17 | 80 / 38 | 82 / 107 | 82 / 85 | 85 / 154
// Few offsets are few steps, and channel counts that are no multiples of 128 have the cheaper ones (row-stationary / wavefront-private
// in us): K = 1, 64 -> 64 on 13 k rows 8.4 / 9.4, 128 -> 128 on 3 k 13 / 10, on 8 k 13 / 17; K = 2 64 -> 64 on 12 k rows 14.1 / 12.2, on 42 k
// 14.1 / 19, 64 -> 192 on 14 k 14.3 / 22, 128 -> 128 on 34 k 26.6 / 26.6; K = 3 128 -> 64 on 50 k rows 49 / 57, 64 -> 192 on 12 k 30 / 36.
// Not on a side with position classes, whose row-stationary steps are few.  bf16 sums are fp32 and rounded once in both.
bool small_wave(const MapSide& side, int kvol, int64_t links, int cc, int co, sp_dtype dt) {
    if (side.tile_mask || tile_big(side, kvol, cc, dt) || !wave_shape_ok(cc, co, dt)) return false;
    const int cot = wave_tile(cc, co, dt == SP_F32);
    if (!cot) return false;
    const int64_t nwt = (side.n_rows + 63) / 64;
    const double per = (double)links * 64 / ((double)side.n_rows * kvol), blocks = std::max(1.0, per / 16 + 0.5);
    // (64 -> 64 at K = 3 is level between 1400 and 2100: 32 / 33 on 49 k rows, 32 / 33 on 59 k.)
    const double line = co % 128 == 0 ? (kvol == 1 ? 800.0 : kvol <= 8 ? 1900.0 : 2100.0)
                                      : (kvol == 1 ? 0.0 : kvol <= 8 ? 600.0 : cc * co == 4096 ? 2100.0 : kvol > 27 && cc == 128 ? 1900.0 : 1400.0);
    return (double)(nwt * (co / cot)) * blocks <= line;
}

// Which gather kernel a layer takes: 0 row-stationary (sp_conv_dense.hip), 1 wavefront-private link lists,
// 2 link lists with producer wavefronts (sp_conv_tile.h), 3 plain, 4 few channels on one side (sp_conv_narrow.hip),
// 5 fp32 link lists on the bf16 matrix cores (sp_conv_split.hip).  The wavefront-private kernel keeps the whole
// weight matrix of a narrow layer in registers; everything else, wide or not a multiple of its tiles, takes the tile kernel.
// Forward in us, wavefront-private / tile kernel, on 1.5 k rows with 9 k links | 96 k, 0.61 M | 160 k, 0.66 M | 374 k, 2.4 M |
// 613 k, 5.0 M:
//   fp32 16 -> 16   16 / 14 | 23 / 38   | 27 / 51   | 55 / 115  | 88 / 206       bf16 32 -> 32   17 / 15 | 23 / 31 | 28 / 44  | 54 / 93   | 95 / 167
//   fp32 32 -> 32   24 / 16 | 36 / 45   | 49 / 63   | 90 / 139  | 175 / 260      bf16 32 -> 64   21 / 16 | 28 / 38 | 48 / 51  | 78 / 103  | 142 / 192
//   fp32 32 -> 64   34 / 19 | 56 / 62   | 89 / 84   | 153 / 195 | 310 / 376      bf16 64 -> 64   22 / 16 | 37 / 49 | 57 / 63  | 101 / 143 | (row-stationary)
//   fp32 64 -> 32   35 / 22 | 57 / 87   | 92 / 123  | 160 / 292 | 324 / 554      bf16 64 -> 128  23 / 19 | 62 / 84 | 84 / 107 | 189 / 287 | (row-stationary)
//   fp32 64 -> 64   54 / 27 | 114 / 100 | 166 / 134 | 305 / 341 | 604 / 664
// So one rule for both types (the smallest launches, which one sub-tile's chain bounds, are four wavefronts a sub-tile since: 10
// to 12 us, fp32 64 -> 64 20).  It gives away fp32 64 -> 64 between about 0.1 and 0.2 M rows where the split kernel has not taken
// it, since the tile kernel's 128 rows fill the blocks of few links better.
int select_gather(const MapSide& side, int kvol, int64_t total_links, int cc, int co, sp_dtype dt, bool may_split = true) {
    const size_t elt = dt == SP_F32 ? 4 : 2;
    // (features and lists beyond 32-bit offsets, which the tile kernel takes slowly or not at all, are nothing special to kind 4)
    if (narrow_pays(cc, co, kvol, side.n_rows, total_links, dt) || (narrow_ok(cc, co, kvol) && tile_big(side, kvol, cc, dt))) return 4;
    // Row-stationary kernel: it multiplies all kvol offsets of every row, the link-list kernels only the links
    // that exist but pay per link for bookkeeping, weight re-reads and the accumulator update.  Measured, it is
    // the faster one from about 1 link in 20 row-offsets upwards on 128- and 256-channel inputs, from 1 in 4
    // on 64-channel inputs.
    // (A side with position classes skips the offsets its tiles cannot have: its cost follows the links.)
    const uint64_t lim = 0x7fffffffull;
    if (dense_shape_ok(cc, co, dt) && dense_pays(side, kvol, total_links, cc) && !small_wave(side, kvol, total_links, cc, co, dt) &&
        (uint64_t)side.n_src * cc * elt < lim && (uint64_t)side.n_rows * kvol * 4 < lim && (uint64_t)kvol * cc * co * elt < lim)
        return 0;
    // the link-list kernels address their buffers with 32-bit offsets; the tile kernel takes larger features and lists
    // too if a row is whole 16-byte pieces
    const bool big = tile_big(side, kvol, cc, dt);
    const bool wave = !big && wave_shape_ok(cc, co, dt) && wave_tile(cc, co, dt == SP_F32);
    if (may_split && dt == SP_F32 && !big && split_pays(side, kvol, total_links, cc, co, wave)) return 5;
    if (wave) return 1;
    if ((big && cc * elt % 16) || tile_copy_bytes(tile_shape(cc, co, dt == SP_F32, big), kvol, (int)elt) >= kLim32) return 3;
    return 2;
}
}  // namespace

// side: which rows are destinations.  w_transposed = false: W[k][co][cc] as stored (forward);
// true: the stored W is [k][cc][co] (data gradient), transposed into pool memory first for the MFMA path.
int conv_gather(const MapSide& side, int kvol, int64_t total_links, const void* d_f, const void* d_w, bool w_transposed,
                void* d_g, int cc, int co, sp_dtype dt, hipStream_t s, void* scratch, size_t scratch_bytes) {
    if (side.n_rows == 0) return SP_OK;
    if (scratch && w_transposed) return fail(SP_ERR_UNSUPPORTED, "no allocation-free path for transposed weights");
    const size_t elt = dt == SP_F32 ? 4 : 2;
    int kind = select_gather(side, kvol, total_links, cc, co, dt);
    if (kind == 5) {
        const size_t bytes = split_copy_bytes(split_shape(cc, co), kvol);
        Buf ws;
        void* d_ws = scratch;
        if (!scratch) {
            ws = dev_alloc(bytes, s);
            d_ws = ws ? ws->p : nullptr;
        } else if (bytes > kSplitScratchBytes) {
            d_ws = nullptr;
        }
        if (d_ws) {
            SP_TRY(need_lists(side, kvol, s));
            return conv_gather_split(side, kvol, total_links, static_cast<const float*>(d_f), static_cast<const float*>(d_w), w_transposed,
                                     static_cast<float*>(d_g), cc, co, d_ws, s);
        }
        kind = select_gather(side, kvol, total_links, cc, co, dt, false);  // no room for the weights' pieces
    }
    if (scratch && kind == 2 && !tile_fits_scratch(side, cc, co, kvol, dt, scratch_bytes)) kind = 3;
    if (kind == 4) return conv_narrow(side, kvol, d_f, d_w, w_transposed, d_g, cc, co, dt, s);
    if (kind == 1 || kind == 2) SP_TRY(need_lists(side, kvol, s));
    if (kind == 0) {
        SP_TRY(need_classes(side, s));
        Buf wt;
        const void* w = d_w;
        if (w_transposed) {  // stored matrix is [cout = cc][cin = co]; the kernel wants [co][cc]
            const int64_t n = (int64_t)kvol * cc * co;
            wt = dev_alloc((size_t)n * elt, s);
            if (!wt) return SP_ERR_ALLOC;
            hipLaunchKernelGGL(transpose_w_kernel<bf16_t>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                               static_cast<const bf16_t*>(d_w), ptr<bf16_t>(wt), kvol, cc, co);
            w = wt->p;
        }
        return conv_gather_dense(side, kvol, d_f, w, d_g, cc, co, s);
    }
    if (kind == 2) {
        const int rc = conv_gather_tile(side, kvol, d_f, d_w, w_transposed, d_g, cc, co, dt, s, scratch, scratch_bytes);
        if (rc != SP_ERR_ALLOC) return rc;  // no memory for the weight copy: the plain kernel needs none
    }
    if (kind == 1) {
        GatherArgs a;
        a.off = ptr<int32_t>(side.off);
        a.src = ptr<int32_t>(side.src);
        a.dst = ptr<int32_t>(side.dst);
        a.f = d_f;
        a.w = d_w;
        a.w_transposed = w_transposed ? 1 : 0;
        a.scratch = scratch;
        // Layers that the row-stationary kernel has on larger maps: it copies no weights, so the allocation-free entry point never
        // touches its static array for them, and calls on two streams at once do not meet there.  (bf16 64 -> 64 on 1.5 k rows
        // 14.4 us, 11.7 with a copy, 29 row-stationary.)
        a.may_in_place = dense_shape_ok(cc, co, dt) && dense_pays(side, kvol, total_links, cc) ? 1 : 0;
        a.scratch_bytes = scratch_bytes;
        const uint64_t fb = (uint64_t)side.n_src * cc * elt;
        a.f_bytes = (uint32_t)fb;
        a.list_bytes = (uint32_t)((uint64_t)side.pitch * kvol * 4);
        a.g = d_g;
        a.n_rows = side.n_rows;
        a.kvol = kvol;
        a.co_total = co;
        a.flip = side.flip ? 1 : 0;
        return dt == SP_F32 ? dispatch_cc<float>(cc, a, s) : dispatch_cc<bf16_t>(cc, a, s);
    }
    const int64_t n = side.n_rows * co;
    const int w_cc = w_transposed ? co : 1, w_co = w_transposed ? 1 : cc;
    if (dt == SP_F32)
        hipLaunchKernelGGL(gather_plain_kernel<float>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                           ptr<int32_t>(side.nbr), side.n_rows, kvol, side.flip ? 1 : 0, static_cast<const float*>(d_f),
                           static_cast<const float*>(d_w), static_cast<float*>(d_g), cc, co, w_cc, w_co);
    else
        hipLaunchKernelGGL(gather_plain_kernel<bf16_t>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                           ptr<int32_t>(side.nbr), side.n_rows, kvol, side.flip ? 1 : 0,
                           static_cast<const bf16_t*>(d_f), static_cast<const bf16_t*>(d_w),
                           static_cast<bf16_t*>(d_g), cc, co, w_cc, w_co);
    SP_HIP(hipGetLastError());
    return SP_OK;
}

}  // namespace sp

using namespace sp;

// Scratch of the allocation-free entry point: the fragment-major weight copy that sp_conv_fwd takes from the
// pool.  One copy of the array exists on every GPU the library is loaded on, at its own address; host code
// must not use the array's name as a pointer, only the address hipGetSymbolAddress reports for the current
// device.
static __device__ __align__(256) unsigned char scratch[kSplitScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device (looked up once per device).
int static_scratch(void** out) {
    int dev = 0;
    SP_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(SP_ERR_UNSUPPORTED, "device %d: more devices than expected", dev);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        SP_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return fail(SP_ERR_HIP, "hipGetSymbolAddress returned a null address");
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return SP_OK;
}

// a: source features (rows_a), b: weights, c: destination (rows_c); a zero-sized buffer may be NULL
// a_is_in: a holds the map's input rows and c its output rows (forward), else the other way round
int check_conv_args(const sp_kmap_t* m, const void* a, bool a_is_in, const void* b, const void* c, int cin, int cout,
                    sp_dtype dt) {
    if (!m) return fail(SP_ERR_INVALID_ARG, "kmap handle is NULL");
    SP_TRY(kmap_resolve(m));  // the sizes of a map whose build has not reported yet
    const int64_t rows_a = a_is_in ? m->n_in : m->n_out, rows_c = a_is_in ? m->n_out : m->n_in;
    if (cin < 1 || cout < 1 || cin > 4096 || cout > 4096) return fail(SP_ERR_INVALID_ARG, "bad channel count");
    if (dt != SP_F32 && dt != SP_BF16) return fail(SP_ERR_INVALID_ARG, "bad dtype");
    if (!b || (!a && rows_a > 0) || (!c && rows_c > 0))
        return fail(SP_ERR_INVALID_ARG, "a feature/weight pointer is NULL");
    if ((((uintptr_t)a | (uintptr_t)b | (uintptr_t)c) & 15) != 0)
        return fail(SP_ERR_INVALID_ARG, "feature/weight pointers must be 16-byte aligned");
    return SP_OK;
}
}  // namespace

extern "C" {

int sp_conv_fwd(const sp_kmap_t* m, const void* d_x, const void* d_w, void* d_y, int32_t cin, int32_t cout,
                sp_dtype dt, void* stream) {
    SP_TRY(check_conv_args(m, d_x, true, d_w, d_y, cin, cout, dt));
    return conv_gather(m->out_side, m->kvol, m->total, d_x, d_w, false, d_y, cin, cout, dt, (hipStream_t)stream);
}

int sp_conv_bwd_data(const sp_kmap_t* m, const void* d_dy, const void* d_w, void* d_dx, int32_t cin, int32_t cout,
                     sp_dtype dt, void* stream) {
    SP_TRY(check_conv_args(m, d_dy, false, d_w, d_dx, cin, cout, dt));
    return conv_gather(m->in_side, m->kvol, m->total, d_dy, d_w, true, d_dx, cout, cin, dt, (hipStream_t)stream);
}

const char* sp_conv_kernel_name(const sp_kmap_t* m, int32_t cin, int32_t cout, sp_dtype dt, int32_t direction) {
    static const char* const names[] = {"gather_dense_kernel", "gather_wave_kernel", "gather_tile_kernel",
                                        "gather_plain_kernel", "gather_narrow_kernel", "gather_split_kernel"};
    if (!m || cin < 1 || cout < 1 || (dt != SP_F32 && dt != SP_BF16) || kmap_resolve(m) != SP_OK) return "";
    return direction == 0 ? names[select_gather(m->out_side, m->kvol, m->total, cin, cout, dt)]
                          : names[select_gather(m->in_side, m->kvol, m->total, cout, cin, dt)];
}

int sp_conv_fwd_noalloc(const sp_kmap_t* m, const void* d_x, const void* d_w, void* d_y, int32_t cin, int32_t cout,
                        sp_dtype dt, void* stream) {
    SP_TRY(check_conv_args(m, d_x, true, d_w, d_y, cin, cout, dt));
    void* scratch = nullptr;
    SP_TRY(static_scratch(&scratch));
    return conv_gather(m->out_side, m->kvol, m->total, d_x, d_w, false, d_y, cin, cout, dt, (hipStream_t)stream,
                       scratch, kStaticScratchBytes);
}

}  // extern "C"
