// Single-pass device-wide prefix sum over the workgroups of ONE launch ("decoupled look-back"): a workgroup
// publishes the sum of its own items, adds up what its predecessors published and publishes its inclusive prefix,
// so that later workgroups stop looking back there.  Replaces "count kernel, scan kernels, emit kernel" by one
// kernel that counts, ranks and emits.
//
// Storage: desc[t], one 64-bit word per tile t, holding a 2-bit state and the value:
//   0 nothing yet | 1 the tile's own sum | 2 the inclusive prefix (sums of tiles 0..t).     (must start at 0)
// State and value travel in one word, written and read with relaxed device-scope atomics: no fences (a release
// fence writes the whole L2 back on this chip: measured 0.5 us per workgroup, serialised).
//
// Tile = workgroup index.  Workgroups are handed to each XCD in index order, so the lowest-numbered unfinished
// workgroup is always resident (its XCD started it before any later one) and waits for nobody that has not
// finished: the waits below always end.  (A ticket from an atomic counter would not need that argument, but
// one atomic per workgroup on ONE address costs ~0.5 us each across the XCDs.)  The waits are bounded all the
// same: a wait that exceeds kSpinLimit polls sets an error bit and gives up, so the grid drains whatever happens.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace sp {

constexpr unsigned kSpinLimit = 1u << 22;  // polls of ~1 us: seconds, far beyond any real wait
constexpr int kErrLookback = 4;            // error bit: a look-back wait gave up

constexpr unsigned long long kDescOwn = 1ull << 62, kDescPrefix = 2ull << 62, kDescValue = (1ull << 62) - 1ull;

__device__ __forceinline__ unsigned long long load_desc(const unsigned long long* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_desc(unsigned long long* p, unsigned long long v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Called by all 64 lanes of ONE wavefront of the workgroup.  own: this tile's sum.  Publishes the tile's inclusive prefix
// and returns the sum of all earlier tiles.  err: device error word.
__device__ __forceinline__ int lookback(unsigned long long* desc, int tile, int own, int32_t* err) {
    const int lane = threadIdx.x & 63;
    if (tile > 0 && lane == 0) store_desc(desc + tile, kDescOwn | (unsigned long long)(unsigned)own);
    int before = 0;
    unsigned spins = 0;
    for (int end = tile; end > 0;) {  // the window still to look at is tiles [end - 64, end), lane l's is end - 1 - l
        const int t = end - 1 - lane;
        const unsigned long long v = t >= 0 ? load_desc(desc + t) : kDescPrefix;  // before tile 0: an inclusive prefix of 0
        const int state = (int)(v >> 62);
        const unsigned long long have_pre = __ballot(state == 2);
        const unsigned long long missing = __ballot(state == 0);
        const int first_pre = have_pre ? __ffsll((long long)have_pre) - 1 : 64;
        const unsigned long long needed = first_pre >= 63 ? ~0ull : ((2ull << first_pre) - 1ull);
        if (missing & needed) {  // a tile nearer than the nearest prefix has nothing yet: ask again
            if (++spins > kSpinLimit) {
                if (lane == 0) atomicOr(err, kErrLookback);
                break;  // gave up: results are garbage, the error bit says so
            }
            __builtin_amdgcn_s_sleep(1);
            continue;
        }
        int sum = lane <= first_pre ? (int)(v & kDescValue) : 0;
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d, 64);
        before += sum;
        end = first_pre < 64 ? 0 : end - 64;  // no prefix in the window: go on further back
    }
    if (lane == 0) store_desc(desc + tile, kDescPrefix | (unsigned long long)(unsigned)(before + own));
    return before;
}

}  // namespace sp
