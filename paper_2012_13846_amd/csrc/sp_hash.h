// Coordinate tables: which row has a given (b, x, y, z), the GPU hashmap of Sec. III-B.  Two forms, one chosen on the
// device by the build (sp_coords.hip) from the extent of the coordinates.
//
// Grid (bounded clouds, at most 128 cells of the bounding box per source row): the box is cut into blocks of 2 x 2 x 4
// cells (x, y, z); dir[block] is the number of an occupied block or -1, cells[16 * number + cell] the row or kNoRow.
// dir is laid out in groups of 4 x 4 x 4 blocks, so that the words a surface touches are few lines (four clouds of a
// 230^3 box: 2.3 MB instead of 5-10, an L2 holds 4).
// Two dependent loads per search, both from arrays a fraction of a hash table's size, and four z-neighbours share
// 16 bytes.  Building it takes one atomic per distinct row, non-returning, where a hash table takes two and a chain of
// dependent ones on every collision: 25 G random atomics a second is the most this chip does, whatever their scope
// and wherever the line is (0.5 M rows: 21 us, plain stores 2), and that is what bounds the insertion.
//
// Hash (everything else): open addressing on the 64-bit packed coordinate.  One slot is 16 bytes {key, first, row}, so a
// search resolves key and row with a single 16-byte access.
//
// The hash table is made of buckets of 4 slots (64 bytes).  Four coordinates that are neighbours along z (same b,
// x, y, same z / (4 * lattice step)) hash to the same bucket and have the slot given by their position in
// that group of four as home slot; collisions are resolved by plain linear probing over all slots, so the
// table fills evenly even when the coordinates use one position only (a plane of constant z).  The kernel-map search
// asks for a voxel's neighbours along z in one thread, so its 2-3 searches usually fall into one 64-byte line
// instead of 2-3 random ones.
// zshift = floor(log2(lattice step)): which two bits of z number the four group members.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "sp_internal.h"

namespace sp {

constexpr uint64_t kEmptyKey = ~0ull;
constexpr int32_t kNoRow = 0x7fffffff;

struct __align__(16) HashSlot {
    unsigned long long key;  // packed (b,x,y,z) or kEmptyKey
    int32_t first;           // smallest source row that carried this key (atomicMin while inserting)
    int32_t row;             // row number of the key among the distinct coordinates
};

// b in [0, 65536), x,y,z in [-32768, 32768).  Returns false when the row cannot be packed.
__device__ __forceinline__ bool pack_key(int32_t b, int32_t x, int32_t y, int32_t z, uint64_t* key) {
    const uint32_t ux = (uint32_t)(x + 32768), uy = (uint32_t)(y + 32768), uz = (uint32_t)(z + 32768);
    const bool ok = ((uint32_t)b < 65536u) & (ux < 65536u) & (uy < 65536u) & (uz < 65536u);
    *key = ((uint64_t)(uint32_t)b << 48) | ((uint64_t)ux << 32) | ((uint64_t)uy << 16) | (uint64_t)uz;
    return ok;
}

__device__ __forceinline__ uint32_t hash_key(uint64_t k) {
    // 64-bit finaliser (xor-shift-multiply), folded to 32 bits
    k ^= k >> 33;
    k *= 0xff51afd7ed558ccdull;
    k ^= k >> 33;
    k *= 0xc4ceb9fe1a85ec53ull;
    k ^= k >> 33;
    return (uint32_t)k;
}

// home bucket and slot position of a key (cap slots = cap / 4 buckets, cap a power of two >= 4)
__device__ __forceinline__ void hash_home(uint64_t key, uint32_t cap, int zshift, uint32_t* bucket, uint32_t* pos) {
    *pos = (uint32_t)(key >> zshift) & 3u;
    *bucket = hash_key(key & ~(3ull << zshift)) & (cap / 4 - 1);
}

// Insert-or-find.  Returns the slot of `key`, or -1 if the table is full (never at load factor <= 0.5).
// *fresh: this call put the key in (otherwise it was there, or arrived from another thread meanwhile).
__device__ __forceinline__ int64_t hash_insert(HashSlot* __restrict__ tab, uint32_t cap, int zshift, uint64_t key,
                                               bool* fresh) {
    uint32_t bucket, pos;
    hash_home(key, cap, zshift, &bucket, &pos);
    uint32_t slot = bucket * 4 + pos;
    *fresh = false;
    for (uint32_t probe = 0; probe < cap; ++probe) {
        unsigned long long cur = tab[slot].key;
        if (cur == key) return slot;
        if (cur == kEmptyKey) {
            unsigned long long prev = atomicCAS(&tab[slot].key, (unsigned long long)kEmptyKey, (unsigned long long)key);
            *fresh = prev == kEmptyKey;
            if (prev == kEmptyKey || prev == key) return slot;
        }
        slot = (slot + 1) & (cap - 1);
    }
    return -1;
}

// ---- grid ----------------------------------------------------------------------------------------------------
struct TableView {
    const HashSlot* slots;  // hash form
    uint32_t cap;
    int zshift;
    const int32_t* meta;    // which form, and the grid's box
    const int32_t* dir;     // grid form
    const int32_t* cells;
    int ts;                 // lattice step
    int maybe_grid;         // 0: the hash form for certain
};

// The box of a grid, from the set's meta words.
struct Grid {
    int b0, x0, y0, z0;
    int nb, gx, gy, gz;     // clouds, groups of 4 x 4 x 4 blocks along x, y, z
};
__device__ __forceinline__ Grid load_grid(const int32_t* __restrict__ meta) {
    return Grid{meta[kMetaLow], meta[kMetaLow + 1], meta[kMetaLow + 2], meta[kMetaLow + 3],
                meta[kMetaExt], meta[kMetaExt + 1], meta[kMetaExt + 2], meta[kMetaExt + 3]};
}
// Lattice position of d = coordinate - lowest (d may be negative): true if d is on the lattice.
__device__ __forceinline__ bool lattice(int d, int ts, int* q) {
    if (ts == 1) {
        *q = d;
        return true;
    }
    int t = d / ts;
    if (t * ts > d) --t;
    *q = t;
    return t * ts == d;
}
// dir word of the block that holds lattice position (qx, qy, 4 bz ..)
__device__ __forceinline__ uint32_t grid_block(const Grid& g, int qb, int qx, int qy, int bz) {
    const uint32_t group = ((uint32_t)(qb * g.gx + (qx >> 3)) * (uint32_t)g.gy + (uint32_t)(qy >> 3)) * (uint32_t)g.gz + (uint32_t)(bz >> 2);
    return group * 64u + (uint32_t)(((qx >> 1) & 3) * 16 + ((qy >> 1) & 3) * 4 + (bz & 3));
}
__device__ __forceinline__ int grid_run(int qx, int qy) { return (qx & 1) * 2 + (qy & 1); }  // which 4-cell run of the block

// Workgroup -> tile such that each XCD (workgroup id % 8) walks a contiguous eighth of the rows: clouds lie one behind
// the other, so an XCD's L2 sees a few clouds' tables instead of all.  -1: nothing left.  Launch a multiple of 8.
__device__ __forceinline__ int64_t xcd_tile(int64_t wg, int64_t tiles) {
    const int64_t per = (tiles + 7) / 8, j = wg / 8, t = (wg & 7) * per + j;
    return j < per && t < tiles ? t : -1;
}
inline unsigned xcd_grid(int64_t tiles) { return (unsigned)((tiles + 7) / 8 * 8); }

}  // namespace sp
