// Kernel-map construction (paper Sec. 2.1: output coordinates, Alg. 3; map search, Alg. 1).
//
// Keys: (b,x,y,z) -> order-preserving 64 bits, one integer per coordinate (Sec. 2.1.2).  Every build leaves, per output,
// the row of neighbour indices and its offset bitmask, and per 64 outputs and offset a presence bitmap with its count.
// By kind of map, on one stream:
//   3x3x3, stride 1   up to 5120 points: small_map, one launch.  Beyond: fill (clears the block entries), block_insert (pack,
//            insert by blocks of 4x4x4 cells), block_search (a thread per point: Alg. 1's 27 offsets from at most 8 blocks).  Row
//            numbers are packed, by block_base and block_place, only where memory for one per cell is lacking.
//   2x2x2, stride 2   down_pack, _clear, _mark, _count, _expand, _scatter, rows: the box, the number of outputs and what
//            is sized by them stay on the device, nothing waits in between; its transposed map: up_rows
//   other strided and transposed maps   pack; candidate keys (p - delta)/s (Alg. 3, stages 1-4), made distinct and sorted
//            either in a bitmap over their box, whose ranks then are the map (rank_scatter, rows), or by radix sort and
//            unique, with a search through a hash table of points (insert, probe).  The host waits for the box, where
//            that is measured, and for the number of outputs.
//   1x1x1    pack_insert, probe: the hash table of points (64-bit CAS)
//   stride 1 in a coordinate grid (`grid` of Sec. 4.4: collision-free, one memory access per insertion and per lookup), when
//            the caller states the bounds of its coordinates: pack_insert, probe_symmetric (one thread per point and
//            offset below the centre, the mirrored entry written alongside, Sec. 4.2.1), grid_erase; rows goes with the scan
// and for all of them
//   scan     per-offset exclusive scan of the block counts -> where each pair sits in the offset-major lists, and the
//            per-offset totals; the order of the tiles.  Put off for 3x3x3 stride-1 maps that nobody has asked for sizes.
// The kernels tell the host what it needs (verdict on the input, number of outputs, sizes) in pinned words, which it
// watches when something first asks.
// Alg. 3's boundary check is applied where the candidates are formed.
//   compact  pair lists M[W_n] (in, out), ordered by output index inside an offset: derived from
//            the above when first asked for (ts_kmap_pairs, the explicit dataflow's gather)
//
// ts_kmap_sort_rows (optional, for maps that serve several layers) orders the output rows by
// offset bitmask: distinct bitmasks are counted in a small hash table, ranked, and every row
// goes to (first position of its bitmask) + (arrival rank).
#include "ts_internal.h"

#include <chrono>
#include <cstdlib>
#include <cstring>
#include <new>
#include <type_traits>

#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_select.hpp>

using namespace ts;


namespace {

constexpr int kThreads = 256;

// Status words of a build.  They live in pinned host memory: the kernels report there directly (plain
// system-scope stores, on bad input or once per offset), and the host watches the words instead of waiting
// for a copy and a stream synchronisation, which cost a small build more than its kernels.
enum {
    ST_RANGE = 0,       // a coordinate was outside the packable range
    ST_DUP = 1,         // two input rows held the same coordinate
    ST_DCOUNT = 2,      // distinct offset bitmasks seen (ts_kmap_sort_rows)
    ST_OVERFLOW = 3,    // the bitmask table could not hold them all
    ST_SEARCHED = 4,    // set once every kernel that raises ST_RANGE or ST_DUP has finished
    ST_COUNT = 5,       // coarse points of a strided build (-1: not there yet, kBoxTooLarge: build the map by sorting)
    ST_TILES = 6,       // set once the tile order is complete
    ST_BOXED = 7,       // set once the box of the points, which a strided build chooses its route by, is at ST_BOX
    ST_TOTALS = 8,      // [32] per-offset map sizes (-1: not there yet)
    ST_BOX = 40,        // [7] lo, hi, batches of the box of a 2x2x2 stride-2 map's outputs, there with ST_COUNT; or, with
                        // ST_BOXED, the maxima of -x, -y, -z, x, y, z, batch over the valid points (INT32_MIN: none)
    ST_WORDS = 48
};

// A word the host reads.  Every writer of a flag stores the same value.
__device__ __forceinline__ void tell_host(int *status, int which, int value) {
    __hip_atomic_store(&status[which], value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
// A word that says that what the workgroup has written is complete: whoever has read it may use that, on any stream.
// (All of the workgroup's threads call it.  Kernels that ran before on the stream are complete anyway.)
__device__ __forceinline__ void tell_host_done(int *status, int which, int value) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // a barrier alone does not wait for the stores of the other waves
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(&status[which], value, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ void raise_flag(int *status, int which) { tell_host(status, which, 1); }

__device__ __forceinline__ bool coord_ok(int4 c) {
    return c.x >= 0 && c.x <= TS_BATCH_MAX && c.y >= TS_COORD_MIN && c.y <= TS_COORD_MAX &&
           c.z >= TS_COORD_MIN && c.z <= TS_COORD_MAX && c.w >= TS_COORD_MIN && c.w <= TS_COORD_MAX;
}

// ---- coordinate hash table ------------------------------------------------------------------------
// Open addressing over two arrays: 64-bit keys (what lookups read) and 32-bit values (read on a
// hit only).  Random lookups cost about twice as much once the array they walk no longer fits a
// 4 MiB L2 slice, so the probed array is kept as small as the key allows.  8 keys form a 64-byte
// bucket addressed by the hash of the point's 2x2x2 block, the home slot inside the bucket by the
// three parity bits: the cells around a point share a few buckets.
struct Table {
    uint64_t *keys;
    int32_t *vals;
    uint32_t mask;   // capacity - 1 (capacity: power of two >= 4 * entries, >= 1024)
    int shift;       // 64 - log2(capacity / slots per bucket)
};

// The cells of a small box of space (2^kBx x 2^kBy x 2^kBz cells) share a bucket of consecutive slots,
// addressed by the hash of the box; the home slot inside the bucket is the cell's position in the box.
// 2 x 2 x 2 is the measured optimum on the LiDAR-like scenes from 153 k to 15 M points: boxes of 4 x 4 x 4
// (64 slots), 1 x 1 x 8 and 1 x 2 x 4 put the slots of points inserted by neighbouring lanes into the same
// cache lines, whose atomics are then served one after the other (insertion 1.4 to 1.9 times slower), and do
// not make the search faster; smaller boxes (2 x 2 x 1, 1 x 2 x 2, 1 x 1 x 2, none) make it slower (20.4, 21.0,
// 26.8 and 32.5 us against 17.3 on 153 k points: a point's 13 lookups then touch more cache lines).
constexpr int kBx = 1, kBy = 1, kBz = 1;
constexpr uint64_t kSubBits = ((1ull << kBz) - 1) | (((1ull << kBy) - 1) << kFieldBits) | (((1ull << kBx) - 1) << (2 * kFieldBits));
constexpr int kBucketLog2 = kBx + kBy + kBz;

__device__ __forceinline__ uint32_t home_sub(uint64_t key) {
    return ((uint32_t)key & ((1u << kBz) - 1)) | (((uint32_t)(key >> kFieldBits) & ((1u << kBy) - 1)) << kBz) |
           (((uint32_t)(key >> (2 * kFieldBits)) & ((1u << kBx) - 1)) << (kBz + kBy));
}
// (Placing the buckets of neighbouring boxes next to each other - hashing only a region of 4, 8 or 16 boxes
// per axis and using a box's position in its region as the low part of the bucket number - was measured as
// well, for the sake of the large scenes whose table no longer fits the caches: occupied boxes then crowd
// into few stretches of the table, probe chains grow, and both insertion and search take 1.3 to 6 times as
// long at every size from 20 k to 15 M points.  Scattering the boxes is worth more than keeping them together.)
__device__ __forceinline__ uint32_t home_slot(uint64_t key, int shift) {
    const uint64_t cell = key & ~kSubBits;
    return ((uint32_t)((cell * 0x9E3779B97F4A7C15ull) >> shift) << kBucketLog2) + home_sub(key);   // multiplicative (Fibonacci) hashing
}
// Slot after `slot` in a probe sequence: 9 further (next bucket, next position; odd, so the sequence
// visits every slot of the power-of-two table).  A miss ends at the first empty slot it meets, which
// for a point's absent neighbour is usually the home slot itself.  (The slot right after, in the same
// cache line, is the home of the cell's neighbour in z: a key put there displaces that neighbour in turn,
// and the line's atomics queue up; measured, insertion took 15.1 instead of 11.1 us on 153 k points and the
// search 19.5 instead of 17.3.)
// What decides the length of the chains is how many occupied boxes there are per bucket, not points per slot:
// a LiDAR-like scene fills a 2x2x2 box with 1.5 to 2 points, so at a load of 0.29 points per slot there were
// about 1.5 boxes per bucket.  Hence the table's size of four slots per point or more: against two it took
// the search of 153 k points from 18.8 to 17.3 us, their insertion from 13.2 to 11.1, and the build of 15 M
// points from 6.1 to 4.9 ms; eight slots per point gained nothing more at 153 k and cost clearing time.
__device__ __forceinline__ uint32_t next_slot(uint32_t slot, uint32_t mask) { return (slot + 9u) & mask; }

// Loads by 32-bit byte offset from the array base (capacity is at most 2^28 slots), which keeps
// one register per lookup for the address instead of two.
__device__ __forceinline__ uint64_t slot_key(const Table &t, uint32_t slot) {
    return *reinterpret_cast<const uint64_t *>(reinterpret_cast<const char *>(t.keys) + (slot << 3));
}
__device__ __forceinline__ int32_t slot_val(const Table &t, uint32_t slot) {
    return *reinterpret_cast<const int32_t *>(reinterpret_cast<const char *>(t.vals) + (slot << 2));
}

__device__ __forceinline__ void table_insert(const Table &t, uint64_t key, int32_t value, int *status) {
    uint32_t slot = home_slot(key, t.shift);
    for (;;) {
        unsigned long long prev = atomicCAS(reinterpret_cast<unsigned long long *>(&t.keys[slot]),
                                            (unsigned long long)kEmptyKey, (unsigned long long)key);
        if (prev == kEmptyKey) {
            t.vals[slot] = value;
            return;
        }
        if (prev == key) {
            raise_flag(status, ST_DUP);
            return;
        }
        slot = next_slot(slot, t.mask);   // the table is at most a quarter full, so an empty slot exists
    }
}

// ---- coordinate grid ------------------------------------------------------------------------------------
// The collision-free table of Sec. 4.4 (`grid`): one int32 cell per coordinate of a box, holding the
// row of the point there or -1.  An insertion is one store, a lookup one load, whatever the
// occupancy; the price is the box's volume in memory.  The cells live in a buffer the library keeps
// between builds with every cell at -1: a build writes its points in, searches, and takes them out
// again, so it touches 2 N cells and never clears the volume.
struct Grid {
    int32_t *vals;      // [batches][ext x][ext y][ext z]
    int32_t lo[3];      // coordinate of cell 0 on each axis
    uint32_t ext[3];    // cells per axis
    uint32_t batches;
};

// Cell of a packed coordinate, or -1 outside the box.
__device__ __forceinline__ int64_t grid_cell(const Grid &g, uint64_t key) {
    int32_t c[4];
    unpack_key(key, c);
    const uint32_t x = (uint32_t)(c[1] - g.lo[0]), y = (uint32_t)(c[2] - g.lo[1]), z = (uint32_t)(c[3] - g.lo[2]);
    if ((uint32_t)c[0] >= g.batches || x >= g.ext[0] || y >= g.ext[1] || z >= g.ext[2]) return -1;
    return (((int64_t)c[0] * g.ext[0] + x) * g.ext[1] + y) * g.ext[2] + z;
}

__device__ __forceinline__ void table_insert(const Grid &g, uint64_t key, int32_t value, int *status) {
    const int64_t cell = grid_cell(g, key);
    if (cell < 0) {
        raise_flag(status, ST_RANGE);
        return;
    }
    if (atomicCAS(&g.vals[cell], -1, value) != -1) raise_flag(status, ST_DUP);
}

__device__ __forceinline__ int32_t table_find(const Grid &g, uint64_t want) {
    const int64_t cell = grid_cell(g, want);
    return cell < 0 ? -1 : g.vals[cell];
}

// ---- block table -----------------------------------------------------------------------------------------
// What 3x3x3 stride-1 builds search: one entry per occupied block of 4x4x4 cells - its key and a 64-bit
// occupancy mask, 16 bytes that one load fetches - and beside it 64 row numbers, valid where the mask says so.
// A point's 27 neighbours lie in at most 8 blocks (3.4 on average), so a whole neighbourhood costs that many
// lookups instead of 26, an absent neighbour costs a bit test, and a LiDAR-like scene of 153 k points has 28 k
// entries: they stay in the caches where a table of points does not.  Nothing but the entries is cleared.
struct BlockTable {
    uint64_t *ent;     // [capacity][2]: block key (kEmptyKey = free), occupancy mask
    int32_t *rows;     // [capacity][64], valid where the mask says so; or, packed, [points]: those of an entry's set bits
                       // one after the other
    int32_t *base;     // packed rows: [capacity], where an entry's begin (else NULL)
    uint32_t mask;     // capacity - 1 (capacity: power of two, at least 1.5 per point, >= 1024)
    int shift;         // 64 - log2(capacity / 8)
};
constexpr uint64_t kCellBits = 3ull | (3ull << kFieldBits) | (3ull << (2 * kFieldBits));

// The eight blocks of a 2x2x2 group have their home slots side by side (128 bytes of entries): most lookups of a
// point's neighbourhood then fall into one or two cache lines.  A collision moves on by 9 slots, as in the table
// of points above.
constexpr uint64_t kBlockInGroup = 4ull | (4ull << kFieldBits) | (4ull << (2 * kFieldBits));
__device__ __forceinline__ uint32_t block_home(uint64_t bkey, int shift) {
    const uint32_t in_group = ((uint32_t)(bkey >> 2) & 1u) | (((uint32_t)(bkey >> (kFieldBits + 2)) & 1u) << 1) | (((uint32_t)(bkey >> (2 * kFieldBits + 2)) & 1u) << 2);
    return ((uint32_t)(((bkey & ~kBlockInGroup) * 0x9E3779B97F4A7C15ull) >> shift) << 3) + in_group;
}
__device__ __forceinline__ uint32_t cell_of(uint64_t key) {
    return ((uint32_t)key & 3u) | (((uint32_t)(key >> kFieldBits) & 3u) << 2) | (((uint32_t)(key >> (2 * kFieldBits)) & 3u) << 4);
}

// Stride-1 front end: pack and insert.  Points that follow each other in the same block (scan and raster orders:
// 2.7 to 3.7 of them) go in together: the first lane of such a run claims the block's entry and sets the run's
// occupancy bits with one atomic each, because atomics are what bounds this kernel (about 20 G/s over the chip: one
// claim and one mask update per point took 17.5 us for 153 k points and 46 us for 470 k; by runs 10.4 and 17).
// A bit that was set before, or twice in a run, is how equal points are found.
// Packed rows have no place before all bits are set: the points' slots are kept instead (slots).
template <bool PACKED>
__global__ void __launch_bounds__(kThreads) k_block_insert(const int4 *__restrict__ coords, int64_t n, uint64_t *__restrict__ keys,
                                                           BlockTable t, uint32_t *__restrict__ slots, int *status) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const int lane = threadIdx.x & 63;
    uint64_t key = kEmptyKey;
    if (i < n) {
        const int4 c = coords[i];
        if (coord_ok(c)) key = pack_key(c.x, c.y, c.z, c.w);
        else raise_flag(status, ST_RANGE);
        keys[i] = key;
    }
    const bool ok = key != kEmptyKey;
    const uint64_t bkey = ok ? key & ~kCellBits : kEmptyKey;
    const uint32_t cell = cell_of(key);
    // runs of equal block keys: the run's first lane, and the lane behind its last
    const uint64_t before = (uint64_t)__shfl_up((unsigned long long)bkey, 1, 64);
    const uint64_t heads = __ballot(lane == 0 || before != bkey);
    const uint64_t upto = ~0ull >> (63 - lane);
    const int first = 63 - __clzll((long long)(heads & upto));
    const uint64_t after = heads & ~upto;
    const int end = after ? __builtin_ctzll(after) : 64;
    uint64_t bits = ok ? 1ull << cell : 0ull;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint64_t other = (uint64_t)__shfl_down((unsigned long long)bits, d, 64);
        if (lane + d < end) bits |= other;
    }
    uint32_t slot = 0;
    if (ok && lane == first) {
        slot = block_home(bkey, t.shift);
        for (;;) {   // the table holds at most one block per point and has half as many slots again: a free one exists
            uint64_t found = t.ent[2 * (uint64_t)slot];   // a key never changes once set; a stale "free" is decided by the swap
            if (found == kEmptyKey)
                found = atomicCAS(reinterpret_cast<unsigned long long *>(&t.ent[2 * (uint64_t)slot]), (unsigned long long)kEmptyKey,
                                  (unsigned long long)bkey);
            if (found == kEmptyKey || found == bkey) break;
            slot = next_slot(slot, t.mask);
        }
        const uint64_t taken = atomicOr(reinterpret_cast<unsigned long long *>(&t.ent[2 * (uint64_t)slot + 1]), (unsigned long long)bits);
        if ((taken & bits) != 0 || __popcll(bits) != end - lane) raise_flag(status, ST_DUP);
    }
    slot = (uint32_t)__shfl((int)slot, first, 64);
    if (!ok) return;
    if constexpr (PACKED) slots[i] = slot;
    else t.rows[(uint64_t)slot * 64 + cell] = (int32_t)i;
}

// Packed rows: where those of every entry begin.  A thread takes the eight slots of a group of blocks, so that their
// rows stand together; workgroups take stretches off a counter.
constexpr int kBlockBasePer = 8;
__global__ void __launch_bounds__(kThreads) k_block_base(BlockTable t, int32_t *counter) {
    __shared__ int wave_sum[kThreads / 64], s_first;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t first = ((uint64_t)blockIdx.x * kThreads + tid) * kBlockBasePer;
    int count[kBlockBasePer], sum = 0;
#pragma unroll
    for (int v = 0; v < kBlockBasePer; ++v) count[v] = first <= t.mask ? __popcll((long long)t.ent[2 * (first + v) + 1]) : 0;
#pragma unroll
    for (int v = 0; v < kBlockBasePer; ++v) sum += count[v];
    int incl = sum;
    for (int d = 1; d < 64; d <<= 1) {
        const int up = __shfl_up(incl, d, 64);
        if (lane >= d) incl += up;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    if (tid == 0) {
        int all = 0;
        for (int w = 0; w < kThreads / 64; ++w) all += wave_sum[w];
        s_first = atomicAdd(counter, all);
    }
    __syncthreads();
    int at = s_first + incl - sum;
    for (int w = 0; w < wave; ++w) at += wave_sum[w];
    if (first > t.mask) return;
#pragma unroll
    for (int v = 0; v < kBlockBasePer; v += 4) {
        int4 b;
        b.x = at;
        b.y = b.x + count[v];
        b.z = b.y + count[v + 1];
        b.w = b.z + count[v + 2];
        at = b.w + count[v + 3];
        *reinterpret_cast<int4 *>(t.base + first + v) = b;
    }
}

__device__ __forceinline__ uint32_t bits_below(uint64_t mask, uint32_t cell) { return (uint32_t)__popcll(mask & ((1ull << cell) - 1ull)); }

// Packed rows: every point's number to its place.  (Of two equal points one stays; there are as many places as cells.)
__global__ void __launch_bounds__(kThreads) k_block_place(const uint64_t *__restrict__ keys, const uint32_t *__restrict__ slots, int64_t n, BlockTable t) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    const uint64_t key = keys[i];
    if (key == kEmptyKey) return;
    const uint64_t slot = slots[i];
    t.rows[(uint32_t)t.base[slot] + bits_below(t.ent[2 * slot + 1], cell_of(key))] = (int32_t)i;
}

// Takes the points out again: the cells of `keys` go back to -1.
__global__ void k_grid_erase(const uint64_t *keys, int64_t n, Grid g) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint64_t key = keys[i];
    if (key == kEmptyKey) return;
    const int64_t cell = grid_cell(g, key);
    if (cell >= 0) g.vals[cell] = -1;
}

// Bounds the caller states for its coordinates (grid search); on == 0: none stated.
struct Box {
    int on;
    int32_t lo[3], hi[3];   // inclusive
    int32_t batches;
};
// Alg. 3's boundary: a candidate u is kept when 0 <= u < hi on every axis (hi = s * b); on == 0: no boundary.
struct Bound {
    int on;
    int32_t hi[3];
};


__host__ __device__ constexpr int offset_component(int K, int n, int axis) {
    const int r = (K - 1) / 2;
    return axis == 0 ? n / (K * K) - r : (axis == 1 ? (n / K) % K - r : n % K - r);
}

__device__ __forceinline__ bool in_box(int4 c, const Box &b) {
    return !b.on || (c.x < b.batches && c.y >= b.lo[0] && c.y <= b.hi[0] && c.z >= b.lo[1] && c.z <= b.hi[1] &&
                     c.w >= b.lo[2] && c.w <= b.hi[2]);
}

__host__ __device__ __forceinline__ int floor_div(int a, int s) { return a >= 0 ? a / s : -((-a + s - 1) / s); }

// ---- one launch for every buffer that must start at a known value -----------------------------------
struct FillSeg {
    uint4 *p;
    uint64_t n_vec;        // 16-byte vectors
    uint32_t value, high;  // the 32-bit words of the first and of the second half of every vector
};
struct FillArgs {
    FillSeg seg[8];
    int n = 0;
    void add(void *p, size_t bytes, uint32_t value) { add_pairs(p, bytes, value, value); }
    void add_pairs(void *p, size_t bytes, uint32_t value, uint32_t high) {
        if (bytes == 0) return;
        seg[n].p = static_cast<uint4 *>(p);
        seg[n].n_vec = (bytes + 15) / 16;
        seg[n].value = value;
        seg[n].high = high;
        ++n;
    }
};

__global__ void k_fill(FillArgs a) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (int s = 0; s < a.n; ++s) {
        const uint32_t v = a.seg[s].value, h = a.seg[s].high;
        const uint4 vv = make_uint4(v, v, h, h);
        for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < a.seg[s].n_vec; i += stride)
            a.seg[s].p[i] = vv;
    }
}

constexpr int kBoxTooLarge = -2;

// keys[i] = pack(coords[i]); out-of-range rows get the empty key and raise ST_RANGE.
__global__ void __launch_bounds__(kThreads) k_pack(const int4 *coords, int64_t n, uint64_t *keys, int *status, Box box) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int4 c = coords[i];
    const bool ok = coord_ok(c) && in_box(c, box);
    if (!ok) raise_flag(status, ST_RANGE);
    keys[i] = ok ? pack_key(c.x, c.y, c.z, c.w) : kEmptyKey;
}

// Insert (keys[i] -> i).
template <class TableT>
__global__ void k_insert(const uint64_t *keys, int64_t n, TableT t, int *status) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint64_t key = keys[i];
    if (key == kEmptyKey) return;
    table_insert(t, key, (int32_t)i, status);
}

// Stride-1 front end in one pass: pack and insert (key -> i).  With `rows` (the neighbour table of a 3x3x3
// map, 8 16-byte vectors per point) the workgroup also sets its points' rows to "no neighbour": the symmetric
// search writes hits only, and these stores ride along with a kernel that waits for its atomics anyway
// instead of tripling what the clearing launch before it has to write.
template <class TableT>
__global__ void k_pack_insert(const int4 *coords, int64_t n, uint64_t *keys, TableT t, int *status, Box box, int4 *rows) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        const int4 c = coords[i];
        if (!coord_ok(c) || !in_box(c, box)) {
            raise_flag(status, ST_RANGE);
            keys[i] = kEmptyKey;
        } else {
            const uint64_t key = pack_key(c.x, c.y, c.z, c.w);
            keys[i] = key;
            table_insert(t, key, (int32_t)i, status);
        }
    }
    // (after the insertion: stores issued before it would have to complete before the atomic's answer is seen)
    if (rows) {
        const int64_t first = (int64_t)blockIdx.x * blockDim.x * 8, end = n * 8;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int64_t at = first + (int64_t)k * blockDim.x + threadIdx.x;
            if (at < end) rows[at] = make_int4(-1, -1, -1, -1);
        }
    }
}

// Alg. 3 stages 1-4 in registers: candidate u = p - delta, modular check, boundary check, key of u/s.
// Along an axis the admissible offsets are those congruent to p modulo s, at most A = ceil(K/s) of
// the K; a thread takes one of the A^3 combinations of one input (blockIdx.y), so nothing is formed
// for the offsets the modular check would throw out.  Returns the empty key when the combination
// does not exist for this point or falls outside the boundary.
__device__ __forceinline__ uint64_t candidate_key(uint64_t key, int slot, int K, int s, int A, const Bound &bound) {
    if (key == kEmptyKey) return kEmptyKey;
    int32_t c[4];
    unpack_key(key, c);
    const int r = (K - 1) / 2;
    const int t[3] = {slot / (A * A), (slot / A) % A, slot % A};
    int32_t q[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int p = c[1 + a];
        const int first = -r + (((p + r) % s) + s) % s;   // smallest offset >= -r congruent to p
        const int d = first + t[a] * s;
        if (d > K - 1 - r) return kEmptyKey;
        const int u = p - d;                               // a multiple of s
        if (bound.on && (u < 0 || u >= bound.hi[a])) return kEmptyKey;
        q[a] = u / s;
    }
    return pack_key(c[0], q[0], q[1], q[2]);
}

__global__ void k_candidates(const uint64_t *keys, int64_t n, int K, int s, int A, Bound bound, uint64_t *cand) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    cand[i * (int64_t)gridDim.y + blockIdx.y] = candidate_key(keys[i], blockIdx.y, K, s, A, bound);
}

// The same candidates, marked in a bitmap over the box the outputs can lie in (one bit per cell, cells
// in (batch, x, y, z) order): Alg. 3's Unique() without a sort, for callers that state their bounds.
__global__ void k_candidates_mark(const uint64_t *keys, int64_t n, int K, int s, int A, Bound bound, Grid cbox,
                                  uint32_t *bits, int *status) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t cand = i < n ? candidate_key(keys[i], blockIdx.y, K, s, A, bound) : kEmptyKey;
    const int64_t cell = cand == kEmptyKey ? -1 : grid_cell(cbox, cand);
    // neighbours in row order are often neighbours in space: a lane whose predecessor marks the same cell stays silent
    const int64_t before = __shfl_up(cell, 1, 64);
    if (cand == kEmptyKey) return;
    if (cell < 0) {
        raise_flag(status, ST_RANGE);
        return;
    }
    if ((threadIdx.x & 63) != 0 && before == cell) return;
    atomicOr(&bits[cell >> 5], 1u << (cell & 31));
}

// The number of distinct candidates for the host.  The empty key, if any candidate was rejected, is the last of them:
// it is not counted.
__global__ void k_tell_count(const uint64_t *uniq, const int64_t *count, int *status) {
    const int64_t n = *count;
    tell_host(status, ST_COUNT, (int)(n - (n > 0 && uniq[n - 1] == kEmptyKey)));
}

__global__ void k_unpack(const uint64_t *keys, int64_t n, int4 *coords) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int32_t c[4];
    unpack_key(keys[i], c);
    coords[i] = make_int4(c[0], c[1], c[2], c[3]);
}

// ---- distinct offset bitmasks ------------------------------------------------------------------------
// A small open-addressing table bitmask -> number of rows.  Rows take an arrival rank from the
// counter; the distinct masks are ranked afterwards, so rows with equal masks end up adjacent.
// Which of those rows comes first depends on arrival order, which no result depends on: the
// compute kernels add a row's terms in offset order whatever tile the row sits in.
struct MaskHash {
    uint32_t *key;      // [cap]  0xFFFFFFFF = empty
    int32_t *cnt;       // [cap]  rows holding the mask
    int32_t *start;     // [cap]  first sorted position of the mask (filled by the rank step)
    int32_t *dlist;     // [dmax] slots in use, in arrival order
    uint32_t cap_mask;  // cap - 1
    int shift;          // 32 - log2(cap)
    int dmax;           // most distinct masks the fast path ranks
};
constexpr int kMaskHashCap = 1 << 16;
constexpr int kMaskHashMaxDistinct = 1 << 14;
constexpr int kMaskHashMaxSteps = 128;

__device__ __forceinline__ int mask_hash_insert(const MaskHash &mh, uint32_t mask, int *status) {
    // bitmasks are structured keys: mix all bits before taking the top ones
    uint32_t h = mask;
    h ^= h >> 16;
    h *= 0x85EBCA6Bu;
    h ^= h >> 13;
    h *= 0xC2B2AE35u;
    h ^= h >> 16;
    uint32_t sl = h >> mh.shift;
    for (int step = 0; step < kMaskHashMaxSteps; ++step) {
        // An ordinary (cached) load first: most masks are in the table already, and a key never
        // changes once set.  A stale "empty" only means the compare-and-swap below decides.
        uint32_t prev = mh.key[sl];
        if (prev == 0xFFFFFFFFu) prev = __hip_atomic_load(&mh.key[sl], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (prev == 0xFFFFFFFFu) prev = atomicCAS(&mh.key[sl], 0xFFFFFFFFu, mask);
        if (prev == 0xFFFFFFFFu) {
            const int id = atomicAdd(&status[ST_DCOUNT], 1);
            if (id < mh.dmax)
                mh.dlist[id] = (int32_t)sl;
            else
                atomicOr(&status[ST_OVERFLOW], 1);
            return (int)sl;
        }
        if (prev == mask) return (int)sl;
        sl = (sl + 1) & mh.cap_mask;
    }
    atomicOr(&status[ST_OVERFLOW], 1);   // too crowded: the build falls back to a radix sort of the masks
    return -1;
}

// Order in which distinct masks are laid out.  For K = 3 the bits of rarely present offsets
// (corners, then edges, then faces, then the centre) are made the most significant, so that
// neighbouring masks in the order differ in few offsets where rows of several masks share a tile.
struct BitPos27 {
    uint8_t p[27];
};
constexpr BitPos27 make_bitpos27() {
    BitPos27 b{};
    int next = 0;
    for (int cls = 0; cls <= 3; ++cls)
        for (int n = 0; n < 27; ++n) {
            const int nz = (n / 9 != 1) + ((n / 3) % 3 != 1) + (n % 3 != 1);
            if (nz == cls) b.p[n] = (uint8_t)next++;
        }
    return b;
}
__host__ __device__ __forceinline__ uint32_t mask_sort_key(uint32_t mask, int K3) {
    if (K3 != 27) return mask;
    constexpr BitPos27 bp = make_bitpos27();
    uint32_t key = 0;
#pragma unroll
    for (int n = 0; n < 27; ++n) key |= ((mask >> n) & 1u) << bp.p[n];
    return key;
}

// What every search kernel does once a thread knows the offset bitmask of its output row:
// presence bitmaps of the wave's 64 outputs, one per offset, their counts, and the wave's OR.
template <int K3>
__device__ __forceinline__ void finish_rows(uint32_t mask, uint64_t *__restrict__ colbits, int32_t *__restrict__ colcnt,
                                            uint32_t *__restrict__ wavemask, int64_t n_blocks, int64_t block64) {
    const int lane = threadIdx.x & 63;
    uint64_t mine = 0;
#pragma unroll
    for (int n = 0; n < K3; ++n) {
        const uint64_t b = __ballot((mask >> n) & 1u);
        if (lane == n) mine = b;
    }
    if (lane < K3 && block64 < n_blocks) {
        colbits[(int64_t)lane * n_blocks + block64] = mine;
        colcnt[(int64_t)lane * n_blocks + block64] = __popcll(mine);
    }
    // offsets present anywhere in the wave's 64 rows (what a tile of the fused kernel has to visit)
    const uint64_t any = __ballot(lane < K3 && mine != 0);
    if (lane == 0 && block64 < n_blocks) wavemask[block64] = (uint32_t)any;
}
template <int K3>
__device__ __forceinline__ void finish_rows(uint32_t mask, uint64_t *__restrict__ colbits, int32_t *__restrict__ colcnt,
                                            uint32_t *__restrict__ wavemask, int64_t n_blocks) {
    finish_rows<K3>(mask, colbits, colcnt, wavemask, n_blocks, (int64_t)blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6));   // wave-uniform
}

// Map search for stride 1, K = 3 (Alg. 1) through the block table: a thread per point.  All block lookups of
// a thread are in flight together, then all row numbers of its neighbours; rows leave the workgroup through
// LDS as whole cache lines, with the centre entry and the offset bitmask, and the presence bitmaps of 64
// outputs come out of the same pass.  What it replaces - a lane per (point, offset below the centre) probing a
// table of points, mirrored 4-byte stores, and a second pass over the rows - took 17.4 + 9 us for 153 k points.
// At: what holds the position of a row number in the table; 32 bits reach 2^26 entries (44.7 M points).
template <bool PACKED, typename At>
__global__ void __launch_bounds__(kThreads) k_block_search(const uint64_t *__restrict__ keys, int64_t n, BlockTable t,
                                                           int32_t *__restrict__ nbr, uint64_t *__restrict__ colbits,
                                                           int32_t *__restrict__ colcnt, uint32_t *__restrict__ wavemask,
                                                           int64_t n_blocks, uint32_t *__restrict__ rowmask, int *status) {
    if (blockIdx.x == 0 && threadIdx.x == 0) tell_host(status, ST_SEARCHED, 1);   // the insertion kernel came before
    constexpr int K3 = 27, STRIDE = 32, WORDS = 28, PITCH = 29;   // an odd pitch: a thread's writes of its row are conflict-free
    __shared__ union {
        struct {
            uint64_t mask[8][kThreads];
            uint32_t slot[8][kThreads];
        } found;                                                  // per octant and thread: the block's mask and slot (packed rows: their base)
        int32_t rows[kThreads * PITCH];
    } lds;
    const int tid = threadIdx.x;
    const int64_t k = (int64_t)blockIdx.x * kThreads + tid;
    const uint64_t key = k < n ? keys[k] : kEmptyKey;
    const bool ok = key != kEmptyKey;
    const uint64_t bkey = key & ~kCellBits;
    const uint32_t c[3] = {(uint32_t)(key >> (2 * kFieldBits)) & 3u, (uint32_t)(key >> kFieldBits) & 3u, (uint32_t)key & 3u};
    // octant o = (ox, oy, oz): the point's own block, or along an axis the block on the side of the nearer face
    // (a cell inside the block along that axis needs no second block there)
    int64_t step[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) step[a] = (int64_t)(c[a] == 0 ? -4 : 4) << ((2 - a) * kFieldBits);
    const uint32_t edge = (c[0] == 0 || c[0] == 3 ? 4u : 0u) | (c[1] == 0 || c[1] == 3 ? 2u : 0u) | (c[2] == 0 || c[2] == 3 ? 1u : 0u);
    uint32_t slot[8];
    ulonglong2 got[8];
    uint32_t pending = 0;
#pragma unroll
    for (int o = 0; o < 8; ++o) {
        if (ok && (o & ~edge) == 0) {
            pending |= 1u << o;
            slot[o] = block_home(bkey + (o & 4 ? step[0] : 0) + (o & 2 ? step[1] : 0) + (o & 1 ? step[2] : 0), t.shift);
            got[o] = reinterpret_cast<const ulonglong2 *>(t.ent)[slot[o]];
        }
    }
    uint32_t present = 0;
    for (;;) {
#pragma unroll
        for (int o = 0; o < 8; ++o) {
            if ((pending >> o) & 1u) {
                const uint64_t want = bkey + (o & 4 ? step[0] : 0) + (o & 2 ? step[1] : 0) + (o & 1 ? step[2] : 0);
                if (got[o].x == want) present |= 1u << o;
                if (got[o].x == want || got[o].x == kEmptyKey) pending &= ~(1u << o);
            }
        }
        if (__ballot(pending != 0) == 0) break;
#pragma unroll
        for (int o = 0; o < 8; ++o) {
            if ((pending >> o) & 1u) {
                slot[o] = next_slot(slot[o], t.mask);
                got[o] = reinterpret_cast<const ulonglong2 *>(t.ent)[slot[o]];
            }
        }
    }
    if constexpr (PACKED) {
#pragma unroll
        for (int o = 0; o < 8; ++o)
            if ((present >> o) & 1u) slot[o] = (uint32_t)t.base[slot[o]];
    }
#pragma unroll
    for (int o = 0; o < 8; ++o) {
        lds.found.mask[o][tid] = (present >> o) & 1u ? (uint64_t)got[o].y : 0ull;
        lds.found.slot[o][tid] = slot[o];
    }
    // Where each neighbour's row number stands, and which neighbours there are.  (A thread reads back only what
    // it wrote itself, by an octant that depends on the lane; all reads first, then all loads they lead to.)
    uint32_t mask = 0;
    At at[K3];
#pragma unroll
    for (int q = 0; q < K3; ++q) {
        const int d[3] = {q / 9 - 1, (q / 3) % 3 - 1, q % 3 - 1};
        uint32_t o = 0, cell = 0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const bool out = (d[a] < 0 && c[a] == 0) || (d[a] > 0 && c[a] == 3);
            o |= out ? 4u >> a : 0u;
            cell |= ((c[a] + (uint32_t)d[a]) & 3u) << (2 * (2 - a));
        }
        const uint64_t m = lds.found.mask[o][tid];
        if constexpr (PACKED) at[q] = lds.found.slot[o][tid] + bits_below(m, cell);
        else at[q] = (At)lds.found.slot[o][tid] * 64 + cell;
        mask |= (uint32_t)(m >> cell & 1ull) << q;
    }
    mask = ok ? mask | 1u << (K3 / 2) : 0u;   // (of two equal points one is not in the table: it still has itself)
    int32_t j[K3];
#pragma unroll
    for (int q = 0; q < K3; ++q) {
        j[q] = -1;
        if (q != K3 / 2 && ((mask >> q) & 1u)) j[q] = t.rows[at[q]];
    }
    if (ok) j[K3 / 2] = (int32_t)k;
    if (k < n) rowmask[k] = mask;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < K3; ++q) lds.rows[tid * PITCH + q] = j[q];
    lds.rows[tid * PITCH + K3] = (int32_t)mask;
    __syncthreads();
    const int64_t first = (int64_t)blockIdx.x * kThreads;
#pragma unroll
    for (int v = 0; v < WORDS / 4; ++v) {
        const int at = v * kThreads + tid, row = at / (WORDS / 4), ch = at % (WORDS / 4);
        if (first + row < n) {
            const int32_t *src = &lds.rows[row * PITCH + ch * 4];
            *reinterpret_cast<int4 *>(nbr + (first + row) * STRIDE + ch * 4) = make_int4(src[0], src[1], src[2], src[3]);
        }
    }
    finish_rows<K3>(mask, colbits, colcnt, wavemask, n_blocks);
}

// The whole 3x3x3 stride-1 build of a small point set in one launch.  On a few thousand points the three launches above are
// chains of dependent loads through memory (2.3 + 5 + 8.5 us), so every workgroup makes the table of all points for itself,
// in LDS, and searches the rows that are its own: nothing is cleared in memory, and nothing waits for another workgroup.
// What bounds it are the walks through that table, so it is as large as LDS allows: a map of 1 k points took 9.2 us with half
// of the slots in use and 7.0 with a quarter, one of 2 k 10.0 and 8.2.  32 bits a slot: a tag of the hash, which spares most
// reads of a key, and the point's number, its key standing beside the table.  64 rows a workgroup: a thread has two lookups.
// Maps by the launches above and by this one, scan, surfaces, scattered points (us, back to back): 1 k points 19 13 15 and
// 7.0 7.6 7.1, 4 k 19 13 16 and 10.8 10.3 10.4, 5 k 18 13 15.5 and 12.3 12.2 12.0, 6 k 18 13 15 and 13.9 14.5 14.6, 8 k, where
// slots run short, 19 13 15 and 20 20 18.5.  So up to 5 k.
constexpr int kSmallPoints = 5120, kSmallSlots = 16384, kSmallThreads = 1024, kSmallRows = 64;
constexpr int kSmallPer = kSmallPoints / kSmallThreads;
__global__ void __launch_bounds__(kSmallThreads) k_small_map(const int4 *__restrict__ coords, int n, int cap, uint64_t *__restrict__ keys,
                                                             int32_t *__restrict__ nbr, uint64_t *__restrict__ colbits,
                                                             int32_t *__restrict__ colcnt, uint32_t *__restrict__ wavemask,
                                                             int64_t n_blocks, uint32_t *__restrict__ rowmask, uint4 *__restrict__ sched, int *status) {
    constexpr int K3 = 27, STRIDE = 32, WORDS = 28, PITCH = 29, PER_ROW = kSmallThreads / kSmallRows;
    constexpr uint32_t FREE = ~0u, TAG = 0x7FFFE000u, POINT = 0x1FFFu;   // (a tag without the top bit: no slot in use equals a free one)
    static_assert(kSmallPoints <= (int)POINT + 1 && 2 * kSmallPoints <= kSmallSlots && kSmallPoints % kSmallThreads == 0, "a slot holds a point's number");
    __shared__ uint64_t key_of[kSmallPoints];
    __shared__ uint32_t slots[kSmallSlots];
    __shared__ int32_t rows[kSmallRows * PITCH];
    const int tid = threadIdx.x, first = blockIdx.x * kSmallRows;
    for (int v = blockIdx.x * kSmallThreads + tid; v < kMaxSchedSlices * kSchedWords / 4; v += gridDim.x * kSmallThreads)
        sched[v] = make_uint4(0, 0, 0, 0);
    int4 c[kSmallPer];
#pragma unroll
    for (int q = 0; q < kSmallPer; ++q)
        if (q * kSmallThreads + tid < n) c[q] = coords[q * kSmallThreads + tid];
    for (int v = tid; v < cap; v += kSmallThreads) slots[v] = FREE;
    bool bad = false;
#pragma unroll
    for (int q = 0; q < kSmallPer; ++q) {
        const int i = q * kSmallThreads + tid;
        if (i >= n) continue;
        const bool ok = coord_ok(c[q]);
        bad |= !ok;
        key_of[i] = ok ? pack_key(c[q].x, c[q].y, c[q].z, c[q].w) : kEmptyKey;
    }
    __syncthreads();
    // cap is a power of two and at least three times n, the step is odd: every walk meets a free slot
    const uint32_t wrap = (uint32_t)cap - 1;
    auto walk = [&](uint64_t key, uint32_t &slot, uint32_t &step, uint32_t &tag) {
        // (one product leaves the points of a plane on a lattice, many of them in a few slots: 18 us for 2 k points of surfaces)
        uint64_t h = key * 0x9E3779B97F4A7C15ull;
        h = (h ^ h >> 32) * 0xD6E8FEB86659FD93ull;
        slot = (uint32_t)(h >> 50) & wrap;   // (the top bits hang on all of the key's)
        step = (uint32_t)(h >> 36) | 1u;
        tag = (uint32_t)(h >> 19) & TAG;
    };
    bool twice = false;
#pragma unroll
    for (int q = 0; q < kSmallPer; ++q) {
        const int i = q * kSmallThreads + tid;
        if (i >= n) continue;
        const uint64_t key = key_of[i];
        if (key == kEmptyKey) continue;
        uint32_t slot, step, tag;
        for (walk(key, slot, step, tag);; slot = (slot + step) & wrap) {
            const uint32_t found = atomicCAS(&slots[slot], FREE, tag | (uint32_t)i);
            if (found == FREE) break;
            if ((found & TAG) == tag && key_of[found & POINT] == key) {
                twice = true;
                break;
            }
        }
    }
    if (blockIdx.x == 0) {
        if (bad) raise_flag(status, ST_RANGE);
        if (twice) raise_flag(status, ST_DUP);
        tell_host_done(status, ST_SEARCHED, 1);
    }
    __syncthreads();
    {
        const int r = tid / PER_ROW, part = tid % PER_ROW;
        const uint64_t key = first + r < n ? key_of[first + r] : kEmptyKey;
#pragma unroll
        for (int q = part; q < K3; q += PER_ROW) {
            int32_t j = -1;
            if (q == K3 / 2) {
                if (key != kEmptyKey) j = first + r;   // (of two equal points one is not in the table: it still has itself)
            } else if (key != kEmptyKey) {
                const uint64_t want = key + key_delta(q / 9 - 1, q / 3 % 3 - 1, q % 3 - 1);
                uint32_t slot, step, tag;
                for (walk(want, slot, step, tag);; slot = (slot + step) & wrap) {
                    const uint32_t found = slots[slot];
                    if (found == FREE) break;
                    if ((found & TAG) == tag && key_of[found & POINT] == want) {
                        j = (int32_t)(found & POINT);
                        break;
                    }
                }
            }
            rows[r * PITCH + q] = j;
        }
    }
    __syncthreads();
    if (tid < kSmallRows) {   // one wave: the bitmask of every row
        uint32_t mask = 0;
#pragma unroll
        for (int q = 0; q < K3; ++q) mask |= rows[tid * PITCH + q] >= 0 ? 1u << q : 0u;
        rows[tid * PITCH + K3] = (int32_t)mask;
        if (first + tid < n) {
            rowmask[first + tid] = mask;
            keys[first + tid] = key_of[first + tid];
        }
        finish_rows<K3>(mask, colbits, colcnt, wavemask, n_blocks, (int64_t)blockIdx.x);
    }
    __syncthreads();
    if (tid < kSmallRows * (WORDS / 4)) {
        const int row = tid / (WORDS / 4), ch = tid % (WORDS / 4);
        if (first + row < n) {
            const int32_t *src = &rows[row * PITCH + ch * 4];
            *reinterpret_cast<int4 *>(nbr + (int64_t)(first + row) * STRIDE + ch * 4) = make_int4(src[0], src[1], src[2], src[3]);
        }
    }
}

// Row order for the output-stationary kernel: a tile of 128 rows walks every offset that any of its rows meets
// (natural order of a LiDAR scan of 153 k points: 18.8 of 27, and 1.85 times the matrix work there is), so rows that meet
// the same offsets should share tiles.  Sorting all rows by bitmask does that best (9.6, 1.15) but costs more than a map;
// inside a window of 4096 rows one counting sort by 12 bits of the bitmask does most of it (11.5, 1.38; windows of 1024
// rows 13.8, 1.51): the three z levels met first, then the nine (x, y) columns, which beats the bitmask as a number.  A workgroup per
// window; the tiles of all windows are dealt out longest first, window by window, so that the longest start first.
// 8.5 us for 153 k rows, most of it latency (additions in LDS that return, three scans); it was 15 us with an addition for
// every row.  Rows of equal keys nearly keep their order, so that rows next to each other read rows next to each other: map and
// first layer of 600 k points of surfaces, 64 -> 64, take 153 us, and 178 with a wave's lanes on rows far apart.  Where a run
// of rows ends up among others of its key depends on arrival; no result depends on that.
constexpr int kWindowRows = 4096, kWindowThreads = 1024, kWindowPer = kWindowRows / kWindowThreads, kWindowBins = 4096;
constexpr int kWindowTiles = kWindowRows / kTileRows;
__device__ __forceinline__ uint32_t window_key(uint32_t m) {
    uint32_t z = m | m >> 9 | m >> 18;
    z |= z >> 3 | z >> 6;
    uint32_t c = (m | m >> 1 | m >> 2) & 0x01249249u;   // bit 3 c: column c is met; then the nine bits are moved together
    c = (c | c >> 2) & 0x030C30C3u;
    c = (c | c >> 4) & 0x0300F00Fu;
    c = (c | c >> 8) & 0xFF0000FFu;
    c = (c | c >> 16) & 0x1FFu;
    return (z & 7u) << 9 | c;
}
__global__ void __launch_bounds__(kWindowThreads) k_window_sort(const uint32_t *__restrict__ rowmask, int64_t n, int32_t *__restrict__ perm) {
    __shared__ __attribute__((aligned(16))) int bins[kWindowBins];
    __shared__ uint32_t smask[kWindowRows];
    __shared__ uint16_t srow[kWindowRows];
    __shared__ int wave_sum[kWindowThreads / 64], length[kWindowTiles], place[kWindowTiles];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t base = (int64_t)blockIdx.x * kWindowRows;
    const int rows = (int)min((int64_t)kWindowRows, n - base), tiles = (rows + kTileRows - 1) / kTileRows;
    const int mine = wave * (64 * kWindowPer) + lane;   // and the rows 64, 128, ... further
    uint32_t m[kWindowPer], key[kWindowPer];
#pragma unroll
    for (int i = 0; i < kWindowPer; ++i) m[i] = mine + i * 64 < rows ? rowmask[base + mine + i * 64] : 0u;
    constexpr int B = kWindowBins / kWindowThreads;
    static_assert(B == 4, "a thread's bins are a vector");
    reinterpret_cast<int4 *>(bins)[tid] = make_int4(0, 0, 0, 0);
    __syncthreads();
    // Neighbouring rows often have one key, and additions to one word of LDS are served one after the other: a run of lanes
    // with one key adds once.  Rows of a run stay side by side, whose neighbours lie side by side, too.
    int rank[kWindowPer];
#pragma unroll
    for (int i = 0; i < kWindowPer; ++i) {
        key[i] = mine + i * 64 < rows ? window_key(m[i]) : ~0u;
        const uint32_t before = (uint32_t)__shfl_up((int)key[i], 1, 64);
        const uint64_t heads = __ballot(lane == 0 || before != key[i]), upto = ~0ull >> (63 - lane), after = heads & ~upto;
        const int first = 63 - __clzll((long long)(heads & upto)), end = after ? __builtin_ctzll(after) : 64;
        int at = 0;
        if (lane == first && key[i] != ~0u) at = atomicAdd(&bins[key[i]], end - lane);
        rank[i] = __shfl(at, first, 64) + lane - first;
    }
    __syncthreads();
    // bins -> where each begins
    const int4 own = reinterpret_cast<const int4 *>(bins)[tid];
    const int v[B] = {own.x, own.y, own.z, own.w};
    const int sum = own.x + own.y + own.z + own.w;
    int incl = sum;
    for (int d = 1; d < 64; d <<= 1) {
        const int up = __shfl_up(incl, d, 64);
        if (lane >= d) incl += up;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    int at = incl - sum;
    for (int w = 0; w < wave; ++w) at += wave_sum[w];
    reinterpret_cast<int4 *>(bins)[tid] = make_int4(at, at + v[0], at + v[0] + v[1], at + v[0] + v[1] + v[2]);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kWindowPer; ++i) {
        if (mine + i * 64 < rows) {
            const int pos = bins[key[i]] + rank[i];
            smask[pos] = m[i];
            srow[pos] = (uint16_t)(mine + i * 64);
        }
    }
    __syncthreads();
    constexpr int TPW = kWindowTiles / (kWindowThreads / 64);   // tiles per wave, side by side
    uint32_t any[TPW];
#pragma unroll
    for (int q = 0; q < TPW; ++q) {
        const int p = (wave * TPW + q) * kTileRows + lane;
        any[q] = (p < rows ? smask[p] : 0u) | (p + 64 < rows ? smask[p + 64] : 0u);
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1)
#pragma unroll
        for (int q = 0; q < TPW; ++q) any[q] |= (uint32_t)__shfl_xor((int)any[q], d, 64);
    if (lane == 0) {
#pragma unroll
        for (int q = 0; q < TPW; ++q) length[wave * TPW + q] = __builtin_popcount(any[q]);
    }
    __syncthreads();
    if (tid < tiles) {
        int s = 0;
        const int own = length[tid];
#pragma unroll
        for (int o = 0; o < kWindowTiles; ++o) s += o < tiles && (length[o] > own || (length[o] == own && o < tid));
        // the s-th longest tiles of all windows come before the (s + 1)-th; the last window has fewer of them
        const int windows = (int)gridDim.x;
        const int64_t last = (n - (int64_t)(windows - 1) * kWindowRows + kTileRows - 1) / kTileRows;
        place[tid] = (int)(s < last ? s * (int64_t)windows + blockIdx.x : last * windows + (s - last) * (windows - 1) + blockIdx.x);
    }
    __syncthreads();
    for (int p = tid; p < tiles * kTileRows; p += kWindowThreads)
        perm[(int64_t)place[p / kTileRows] * kTileRows + p % kTileRows] = p < rows ? (int32_t)(base + srow[p]) : -1;
}

// ts_kmap_sort_rows, step 1: register every row's bitmask in the mask table; slot_rank[k] = (table
// slot, arrival rank among the rows of that mask).  Lanes of a wave holding the same mask share
// one counter update: first the wave's classes of equal masks (registers only), then every class
// leader talks to the table at once.
__global__ void __launch_bounds__(kThreads) k_register(const int32_t *__restrict__ nbr, int64_t n_out, int stride, int K3,
                                                       int *__restrict__ status, MaskHash mh, int2 *__restrict__ slot_rank) {
    const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const int lane = threadIdx.x & 63;
    const bool ok = k < n_out;
    const uint32_t mask = ok ? (uint32_t)nbr[k * stride + K3] : 0u;
    int my_leader = lane;
    uint64_t my_class = 0;
    uint64_t todo = __ballot(ok);
    while (todo) {
        const int leader = __ffsll((unsigned long long)todo) - 1;
        const uint32_t lm = (uint32_t)__shfl((int)mask, leader, 64);
        const uint64_t same = __ballot(ok && mask == lm);
        if ((same >> lane) & 1ull) {
            my_leader = leader;
            my_class = same;
        }
        todo &= ~same;
    }
    int sl = -1, first = 0;
    if (ok && lane == my_leader) {
        sl = mask_hash_insert(mh, mask, status);
        if (sl >= 0) first = atomicAdd(&mh.cnt[sl], __popcll(my_class));
    }
    const int my_slot = __shfl(sl, my_leader, 64);
    const int my_rank = __shfl(first, my_leader, 64) + __popcll(my_class & ((1ull << lane) - 1ull));
    if (ok) slot_rank[k] = make_int2(my_slot, my_rank);
}

// ---- map search (Alg. 1) -------------------------------------------------------------------------------
enum { MODE_SUB = 0, MODE_FWD = 1, MODE_TR = 2 };

// One thread per output point k.
//   MODE_SUB  stride 1, odd K: neighbour key = key_k + key_delta(delta_n); the centre is k itself
//   MODE_FWD  stride s: input at s*q_k + delta_n
//   MODE_TR   transposed: coarse point (p_k - delta_n)/s when s divides the difference
// Writes nbr[k][0..K3) (input row or -1) and nbr[k][K3] = bitmask of the offsets present; per wave
// (64 consecutive outputs) and offset the presence bitmap and its popcount.  (No global counters
// here: atomics from every wave on one cache line are served one after the other.)
template <int MODE, int K, class TableT>
__global__ void __launch_bounds__(kThreads, 3) k_probe(const uint64_t *__restrict__ out_keys, int64_t n_out, TableT t, int s,
                                                    int32_t *__restrict__ nbr, uint64_t *__restrict__ colbits,
                                                    int32_t *__restrict__ colcnt, uint32_t *__restrict__ wavemask,
                                                    int64_t n_blocks) {
    constexpr int K3 = K * K * K, STRIDE = nbr_stride(K3), CENTRE = (K3 - 1) / 2;
    const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const uint64_t key = k < n_out ? out_keys[k] : kEmptyKey;
    const bool ok = key != kEmptyKey;
    int32_t c[4] = {0, 0, 0, 0};
    if (MODE != MODE_SUB && ok) unpack_key(key, c);

    // Key searched for offset n.  Stride 1 and forward maps: a base key plus the constant
    // key_delta(delta_n), so a loaded key is tested as (loaded - base == constant) and nothing per
    // offset stays in registers but the slot; transposed maps keep the searched keys.
    uint64_t base = key;
    if (MODE == MODE_FWD) base = pack_key(c[0], s * c[1], s * c[2], s * c[3]);
    auto delta_of = [](int n) -> int64_t {
        constexpr int r = (K - 1) / 2;
        return key_delta(n / (K * K) - r, (n / K) % K - r, n % K - r);
    };
    uint64_t want_tr[MODE == MODE_TR ? K3 : 1];
    auto is_wanted = [&](int n, uint64_t loaded) -> bool {
        if (MODE == MODE_TR) return loaded == want_tr[MODE == MODE_TR ? n : 0];
        return (int64_t)(loaded - base) == delta_of(n);
    };
    // All lookups advance together.  The first load of each (its key only) is issued before any
    // is examined; then rounds: lookups whose slot held another key move on together, so a wave
    // pays one memory access time per round, not per collision.  A finished lookup leaves the
    // slot it hit (or none); the values are fetched in one last batch.
    // searched key of offset n, and whether there is anything to search for
    auto wanted = [&](int n, bool *probe) -> uint64_t {
        *probe = ok && !(MODE == MODE_SUB && n == CENTRE);
        uint64_t want = base + (uint64_t)delta_of(n);
        if (MODE == MODE_TR) {
            constexpr int r = (K - 1) / 2;
            const int ux = c[1] - (n / (K * K) - r), uy = c[2] - ((n / K) % K - r), uz = c[3] - (n % K - r);
            *probe = ok && ux % s == 0 && uy % s == 0 && uz % s == 0;
            want = pack_key(c[0], ux / s, uy / s, uz / s);
        }
        return want;
    };
    int32_t j[K3];
    if constexpr (std::is_same<TableT, Grid>::value) {
        // a grid lookup is one load and the K3 loads of a thread do not depend on each other
#pragma unroll
        for (int n = 0; n < K3; ++n) {
            bool probe;
            const uint64_t want = wanted(n, &probe);
            j[n] = (MODE == MODE_SUB && n == CENTRE && ok) ? (int32_t)k : -1;
            if (probe) j[n] = table_find(t, want);
        }
    } else {
    constexpr uint32_t kNone = 0xFFFFFFFFu;
    uint32_t slot[K3];
    uint64_t got[K3];
    uint32_t pending = 0;   // bit n: lookup n has not ended yet
#pragma unroll
    for (int n = 0; n < K3; ++n) {
        bool probe;
        const uint64_t want = wanted(n, &probe);
        if (MODE == MODE_TR) want_tr[MODE == MODE_TR ? n : 0] = want;
        slot[n] = kNone;
        if (probe) {
            pending |= 1u << n;
            slot[n] = home_slot(want, t.shift);
            got[n] = slot_key(t, slot[n]);
        }
    }
    for (;;) {
#pragma unroll
        for (int n = 0; n < K3; ++n) {
            if ((pending >> n) & 1u) {
                if (is_wanted(n, got[n])) {
                    pending &= ~(1u << n);
                } else if (got[n] == kEmptyKey) {
                    pending &= ~(1u << n);
                    slot[n] = kNone;
                }
            }
        }
        if (__ballot(pending != 0) == 0) break;
#pragma unroll
        for (int n = 0; n < K3; ++n) {
            if ((pending >> n) & 1u) {
                slot[n] = next_slot(slot[n], t.mask);
                got[n] = slot_key(t, slot[n]);
            }
        }
    }
#pragma unroll
    for (int n = 0; n < K3; ++n) {
        j[n] = (MODE == MODE_SUB && n == CENTRE && ok) ? (int32_t)k : -1;
        if (slot[n] != kNone) j[n] = slot_val(t, slot[n]);
    }
    }
    uint32_t mask = 0;
#pragma unroll
    for (int n = 0; n < K3; ++n)
        if (j[n] >= 0) mask |= 1u << n;

    // the row of the out-major table
    if (k < n_out) {
        constexpr int CHUNKS = (K3 + 1 + 3) / 4;
        int4 *dst = reinterpret_cast<int4 *>(nbr + k * STRIDE);
#pragma unroll
        for (int ch = 0; ch < CHUNKS; ++ch) {
            int32_t v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int idx = ch * 4 + q;
                v[q] = idx < K3 ? j[idx < K3 ? idx : 0] : (idx == K3 ? (int32_t)mask : 0);
            }
            dst[ch] = make_int4(v[0], v[1], v[2], v[3]);
        }
    }

    finish_rows<K3>(mask, colbits, colcnt, wavemask, n_blocks);
}

// Map search for stride 1, K = 3 through the coordinate grid, one lane per (point i, offset n) with n below the
// centre.  A hit (j at p_i + delta_n) gives two entries: (j, i, n) in row i and, by symmetry (Sec. 4.2.1),
// (i, j, K^3-1-n) in row j; rows start out all -1.  The 13 offsets of a point sit in neighbouring lanes
// (16 lanes per point), so a point's own entries land in one cache line of the table.
__global__ void k_probe_symmetric(const uint64_t *__restrict__ keys, int64_t n_pts, Grid t, int K,
                                  int32_t *__restrict__ nbr, int stride, int *status) {
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g == 0) tell_host(status, ST_SEARCHED, 1);   // the insertion kernel came before
    const int64_t i = g >> 4;
    const int n = (int)(g & 15), K3 = K * K * K;
    if (i >= n_pts || n >= K3 / 2) return;
    const uint64_t key = keys[i];
    if (key == kEmptyKey) return;
    const uint64_t want = (uint64_t)((int64_t)key + key_delta(offset_component(K, n, 0), offset_component(K, n, 1), offset_component(K, n, 2)));
    const int32_t j = table_find(t, want);
    if (j >= 0) {
        nbr[i * stride + n] = j;
        nbr[(int64_t)j * stride + (K3 - 1 - n)] = (int32_t)i;
    }
}

// Row pass over a neighbour table whose hits have been written into rows that started out as -1
// (the symmetric probe of a grid; the transposition of a forward map): a thread per output row reads its
// row, sets the centre entry where the map has one (stride 1: output k is input k) and the row's
// offset bitmask, and does what every search kernel does once the bitmask is known.
// `count`, if given, holds the number of rows on the device; n_out is then a bound on it.
template <int K3, bool HAS_CENTRE>
__global__ void __launch_bounds__(kThreads) k_rows(int32_t *__restrict__ nbr, const uint64_t *__restrict__ keys, int64_t n_out,
                                                   const int32_t *__restrict__ count, uint64_t *__restrict__ colbits,
                                                   int32_t *__restrict__ colcnt, uint32_t *__restrict__ wavemask, int64_t n_blocks) {
    constexpr int STRIDE = nbr_stride(K3), CHUNKS = (K3 + 3) / 4, CENTRE = (K3 - 1) / 2;
    if (count) {
        n_out = *count;
        n_blocks = (n_out + 63) / 64;
        if ((int64_t)blockIdx.x * kThreads >= n_out) return;
    }
    const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const bool ok = k < n_out && keys[k] != kEmptyKey;
    uint32_t mask = 0;
    if (ok) {
        int32_t j[CHUNKS * 4];
#pragma unroll
        for (int ch = 0; ch < CHUNKS; ++ch) {
            const int4 v = reinterpret_cast<const int4 *>(nbr + k * STRIDE)[ch];
            j[ch * 4 + 0] = v.x;
            j[ch * 4 + 1] = v.y;
            j[ch * 4 + 2] = v.z;
            j[ch * 4 + 3] = v.w;
        }
#pragma unroll
        for (int n = 0; n < K3; ++n)
            if ((HAS_CENTRE && n == CENTRE) || j[n] >= 0) mask |= 1u << n;
        if (HAS_CENTRE) nbr[k * STRIDE + CENTRE] = (int32_t)k;
        nbr[k * STRIDE + K3] = (int32_t)mask;
    } else if (k < n_out) {
        nbr[k * STRIDE + K3] = 0;   // a row of an invalid coordinate (the build reports the error) has no neighbours
    }
    finish_rows<K3>(mask, colbits, colcnt, wavemask, n_blocks);
}

// Transposition of a forward map: entry (input j, output k, offset n) of the forward table becomes
// entry (input k, output j, offset n).  A thread per forward output row.
template <int K3>
__global__ void __launch_bounds__(kThreads) k_transpose(const int32_t *__restrict__ fwd, int64_t n_fwd_out,
                                                        int32_t *__restrict__ tnbr) {
    constexpr int STRIDE = nbr_stride(K3), CHUNKS = (K3 + 3) / 4;
    const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (k >= n_fwd_out) return;
    int32_t j[CHUNKS * 4];
#pragma unroll
    for (int ch = 0; ch < CHUNKS; ++ch) {
        const int4 v = reinterpret_cast<const int4 *>(fwd + k * STRIDE)[ch];
        j[ch * 4 + 0] = v.x;
        j[ch * 4 + 1] = v.y;
        j[ch * 4 + 2] = v.z;
        j[ch * 4 + 3] = v.w;
    }
#pragma unroll
    for (int n = 0; n < K3; ++n)
        if (j[n] >= 0) tnbr[(int64_t)j[n] * STRIDE + n] = (int32_t)k;
}

template <int THREADS = kThreads>
__device__ __forceinline__ int block_exclusive_scan(int v, int *total) {
    __shared__ int wave_sums[THREADS / 64];
    int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int incl = v;
    for (int d = 1; d < 64; d <<= 1) {
        int up = __shfl_up(incl, d, 64);
        if (lane >= d) incl += up;
    }
    if (lane == 63) wave_sums[wave] = incl;
    __syncthreads();
    int base = 0, all = 0;
    for (int w = 0; w < THREADS / 64; ++w) {
        int sw = wave_sums[w];
        if (w < wave) base += sw;
        all += sw;
    }
    __syncthreads();
    *total = all;
    return base + incl - v;
}

// ---- marked cells -> sorted distinct keys ------------------------------------------------------------------
// Bits set per block of 256 words.
__global__ void __launch_bounds__(kThreads) k_bits_count(const uint64_t *__restrict__ words, int64_t n_words,
                                                         int32_t *__restrict__ block_total) {
    const int64_t w = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    int total;
    block_exclusive_scan(w < n_words ? __popcll(words[w]) : 0, &total);
    if (threadIdx.x == 0) block_total[blockIdx.x] = total;
}

// One block: block_total[] -> its exclusive prefix in place, and the grand total for the host.
__global__ void __launch_bounds__(kThreads) k_bits_scan(int32_t *__restrict__ block_total, int64_t n, int *status) {
    int64_t run = 0;
    for (int64_t base = 0; base < n; base += kThreads) {
        const int64_t i = base + threadIdx.x;
        const int v = i < n ? block_total[i] : 0;
        int total;
        const int before = block_exclusive_scan(v, &total);
        if (i < n) block_total[i] = (int32_t)(run + before);
        run += total;
    }
    if (threadIdx.x == 0) tell_host(status, ST_COUNT, (int)run);
}

// Every set bit becomes the key of its cell, at the rank of the bit: cells are numbered in
// (batch, x, y, z) order, which is the order of the keys.  word_base[w] receives the rank of word w's
// first set bit (the number of set bits before the word): the rank of any marked cell is then one load
// of it, one of the word, and a popcount.  self_scan: block_total[] still holds the per-block counts and
// every block sums the ones before it itself (a few thousand L2-resident words), which saves the scan
// launch in between; the last block then also tells the host the grand total.
__global__ void __launch_bounds__(kThreads) k_bits_expand(const uint64_t *__restrict__ words, int64_t n_words,
                                                          const int32_t *__restrict__ block_base, Grid cbox,
                                                          uint64_t *__restrict__ out_keys, int32_t *__restrict__ word_base,
                                                          int self_scan, int *status) {
    const int64_t w = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    uint64_t bits = w < n_words ? words[w] : 0;
    int64_t before = 0;
    if (self_scan) {
        int part = 0;
        for (int i = threadIdx.x; i < (int)blockIdx.x; i += kThreads) part += block_base[i];
        int sum;
        block_exclusive_scan(part, &sum);
        before = sum;
    } else {
        before = block_base[blockIdx.x];
    }
    int total;
    int64_t at = before + block_exclusive_scan(__popcll(bits), &total);
    if (self_scan && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) tell_host(status, ST_COUNT, (int)(before + total));
    if (w < n_words) word_base[w] = (int32_t)at;
    if (bits == 0) return;
    // coordinates of the word's first cell once (a box holds at most 2^30 cells: 32-bit arithmetic),
    // then every set bit is that cell moved along z, carrying into y, x and the batch index
    uint32_t cell = (uint32_t)w * 64u;
    uint32_t z0 = cell % cbox.ext[2];
    cell /= cbox.ext[2];
    uint32_t y0 = cell % cbox.ext[1];
    cell /= cbox.ext[1];
    uint32_t x0 = cell % cbox.ext[0], b0 = cell / cbox.ext[0];
    // (the bits come in ascending order, so the cell only ever moves forward: a word costs 64 / ext z
    // carries in all, not that many per set bit, which on the flat boxes of coarse levels was the whole kernel)
    uint32_t z = z0, y = y0, x = x0, b = b0;
    int prev = 0;
    while (bits) {
        const int bit = __builtin_ctzll(bits);
        bits &= bits - 1;
        z += (uint32_t)(bit - prev);
        prev = bit;
        while (z >= cbox.ext[2]) {
            z -= cbox.ext[2];
            if (++y == cbox.ext[1]) {
                y = 0;
                if (++x == cbox.ext[0]) {
                    x = 0;
                    ++b;
                }
            }
        }
        out_keys[at++] = pack_key((int32_t)b, (int32_t)x + cbox.lo[0], (int32_t)y + cbox.lo[1], (int32_t)z + cbox.lo[2]);
    }
}

// Strided maps without a search.  Every admissible candidate (p_j - delta_n) / s of an input p_j that
// Alg. 3 keeps IS an output point, so the pair (j, k, n) of Alg. 1 follows from the candidate alone: k is
// the rank of the candidate's cell among the marked cells (outputs are numbered in cell order).  A lane per
// (input, admissible offset combination), as in k_candidates_mark.
//   forward     nbr[k][n] = j, written with a compare-and-swap against -1: two inputs with one coordinate
//               meet in one entry, which is how duplicates are found
//   transposed  nbr[j][n] = k (rows belong to the given fine points; the roles are swapped)
// Rows start out as -1; the row pass (k_rows) adds bitmasks and presence bitmaps afterwards.
template <bool TRANSPOSED>
__global__ void __launch_bounds__(kThreads) k_rank_scatter(const uint64_t *__restrict__ keys, int64_t n, int K, int s, int A,
                                                           Bound bound, Grid cbox, const uint64_t *__restrict__ words,
                                                           const int32_t *__restrict__ word_base, int32_t *__restrict__ nbr,
                                                           int stride, int *status) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint64_t key = keys[i];
    const uint64_t cand = candidate_key(key, blockIdx.y, K, s, A, bound);
    if (cand == kEmptyKey) return;
    const int64_t cell = grid_cell(cbox, cand);
    if (cell < 0) return;                       // k_candidates_mark has raised the flag
    const int32_t k = word_base[cell >> 6] + __popcll(words[cell >> 6] & ((1ull << (cell & 63)) - 1ull));
    // the offset: delta = p - s * q per axis
    int32_t p[4], q[4];
    unpack_key(key, p);
    unpack_key(cand, q);
    const int r = (K - 1) / 2;
    const int nidx = ((p[1] - s * q[1] + r) * K + (p[2] - s * q[2] + r)) * K + (p[3] - s * q[3] + r);
    if (TRANSPOSED) {
        nbr[i * stride + nidx] = k;
    } else {
        if (atomicCAS(&nbr[(int64_t)k * stride + nidx], -1, (int32_t)i) != -1) raise_flag(status, ST_DUP);
    }
}

// ---- 2x2x2 stride-2 maps ------------------------------------------------------------------------------------
// Every input has exactly one output, the cell (x >> 1, y >> 1, z >> 1), and meets it through the offset made of
// its three parity bits.  The whole build is enqueued at once: what its kernels do not know beforehand - the
// box of the points, the number of outputs - they leave for one another in this header, and the host reads
// the number of outputs from a pinned word when it needs it.  (With the host in between, once for the box and
// once for the count, 153 k points took about 110 us, half of that in two waits and the gaps behind them.)
// Since every input owns one entry, equal points show as fewer entries than inputs: no atomics in the scatter.
struct DownHead {
    int32_t lo[3];       // coarse cell 0 of the bitmap
    uint32_t ext[3];     // cells per axis
    int32_t n_words;     // 64-cell words of the bitmap; 0: no valid point, or the box is too large
    int32_t too_large;
    int32_t count;       // output points
};
constexpr int kDownPack = 512;      // workgroups that pack: as many partial boxes
constexpr int kDownSweep = 1024;    // workgroups that sweep the bitmap
constexpr int kDownWaves = kDownSweep * (kThreads / 64);   // each wave sweeps a stretch of whole 64-word steps: no
                                                           // barriers, which would wait for the step's stores

__device__ __forceinline__ int down_stretch(const DownHead &h) {   // words per wave (a bitmap has at most 2^24)
    return (h.n_words + kDownWaves * 64 - 1) / (kDownWaves * 64) * 64;
}
__device__ __forceinline__ uint32_t down_cell(const DownHead &h, uint64_t key) {   // at most 2^30 cells
    int32_t c[4];
    unpack_key(key, c);
    return (((uint32_t)c[0] * h.ext[0] + (uint32_t)((c[1] >> 1) - h.lo[0])) * h.ext[1] + (uint32_t)((c[2] >> 1) - h.lo[1])) * h.ext[2] +
           (uint32_t)((c[3] >> 1) - h.lo[2]);
}
__device__ __forceinline__ int down_offset(uint64_t key) {
    return ((int)(key >> (2 * kFieldBits)) & 1) * 4 + ((int)(key >> kFieldBits) & 1) * 2 + ((int)key & 1);
}

// Keys, and the box of the valid points in one part per workgroup: 8 words, the maxima of -x, -y, -z, x, y, z, batch.
__global__ void __launch_bounds__(kThreads) k_down_pack(const int4 *__restrict__ coords, int64_t n, uint64_t *__restrict__ keys,
                                                        int *status, Box box, int4 *__restrict__ parts) {
    __shared__ int32_t sh[kThreads / 64][8];
    int32_t v[7];
#pragma unroll
    for (int q = 0; q < 7; ++q) v[q] = INT32_MIN;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads) {
        const int4 c = coords[i];
        uint64_t key = kEmptyKey;
        if (!coord_ok(c) || !in_box(c, box)) {
            raise_flag(status, ST_RANGE);
        } else {
            key = pack_key(c.x, c.y, c.z, c.w);
            const int32_t w[7] = {-c.y, -c.z, -c.w, c.y, c.z, c.w, c.x};
#pragma unroll
            for (int q = 0; q < 7; ++q) v[q] = max(v[q], w[q]);
        }
        keys[i] = key;
    }
#pragma unroll
    for (int q = 0; q < 7; ++q)
        for (int d = 32; d >= 1; d >>= 1) v[q] = max(v[q], __shfl_xor(v[q], d, 64));
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int q = 0; q < 7; ++q) sh[threadIdx.x >> 6][q] = v[q];
    }
    __syncthreads();
    if (threadIdx.x < 7) {
        int32_t m = sh[0][threadIdx.x];
        for (int w = 1; w < kThreads / 64; ++w) m = max(m, sh[w][threadIdx.x]);
        reinterpret_cast<int32_t *>(parts)[blockIdx.x * 8 + threadIdx.x] = m;
    }
}

// The partial boxes folded, by every thread's workgroup for itself (16 KB from L2).
__device__ __forceinline__ void fold_parts(const int4 *__restrict__ parts, int n_parts, int32_t (&v)[7]) {
    __shared__ int32_t sh[kThreads / 64][8];
#pragma unroll
    for (int q = 0; q < 7; ++q) v[q] = INT32_MIN;
    for (int i = threadIdx.x; i < n_parts; i += kThreads) {
        const int4 a = parts[2 * i], b = parts[2 * i + 1];
        const int32_t w[7] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z};
#pragma unroll
        for (int q = 0; q < 7; ++q) v[q] = max(v[q], w[q]);
    }
#pragma unroll
    for (int q = 0; q < 7; ++q)
        for (int d = 32; d >= 1; d >>= 1) v[q] = max(v[q], __shfl_xor(v[q], d, 64));
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int q = 0; q < 7; ++q) sh[threadIdx.x >> 6][q] = v[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 7; ++q) v[q] = max(max(sh[0][q], sh[1][q]), max(sh[2][q], sh[3][q]));
}

// One workgroup: the box of the points, for the host.
__global__ void __launch_bounds__(kThreads) k_tell_box(const int4 *__restrict__ parts, int n_parts, int *status) {
    int32_t v[7];
    fold_parts(parts, n_parts, v);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int q = 0; q < 7; ++q) tell_host(status, ST_BOX + q, v[q]);
    }
    tell_host_done(status, ST_BOXED, 1);
}

// Folds the partial boxes, clears the bitmap over the box and the map's tile counters; the first workgroup leaves the
// header, and the box for the host.
__global__ void __launch_bounds__(kThreads) k_down_clear(const int4 *__restrict__ parts, int n_parts, Box box, uint64_t max_words,
                                                         uint4 *__restrict__ words, uint4 *__restrict__ sched, DownHead *head, int *status) {
    int32_t v[7];
    fold_parts(parts, n_parts, v);
    const bool none = v[6] == INT32_MIN;   // no valid point
    DownHead h;
    int32_t hi[3];
    uint64_t cells = none ? 0 : (uint64_t)(box.on ? box.batches : v[6] + 1);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        h.lo[a] = none ? 0 : (box.on ? box.lo[a] : -v[a]) >> 1;
        hi[a] = none ? 0 : (box.on ? box.hi[a] : v[3 + a]) >> 1;
        h.ext[a] = (uint32_t)(hi[a] - h.lo[a] + 1);
        cells *= h.ext[a];
    }
    const uint64_t n_words = (cells + 63) / 64;
    h.too_large = n_words > max_words;
    h.n_words = h.too_large ? 0 : (int32_t)n_words;
    h.count = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *head = h;
        for (int a = 0; a < 3; ++a) {
            tell_host(status, ST_BOX + a, h.lo[a]);
            tell_host(status, ST_BOX + 3 + a, hi[a]);
        }
        tell_host(status, ST_BOX + 6, none ? 0 : box.on ? box.batches : v[6] + 1);
    }
    const uint4 zero = make_uint4(0, 0, 0, 0);
    const int64_t first = (int64_t)blockIdx.x * kThreads + threadIdx.x, step = (int64_t)gridDim.x * kThreads;
    for (int64_t i = first; i < ((int64_t)h.n_words + 1) / 2; i += step) words[i] = zero;
    for (int64_t i = first; i < kMaxSchedSlices * kSchedWords / 4; i += step) sched[i] = zero;
}

__global__ void __launch_bounds__(kThreads) k_down_mark(const uint64_t *__restrict__ keys, int64_t n, const DownHead *__restrict__ head,
                                                        uint32_t *__restrict__ bits) {
    const DownHead h = *head;
    if (h.n_words == 0) return;
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const uint64_t key = i < n ? keys[i] : kEmptyKey;
    const uint32_t cell = key == kEmptyKey ? ~0u : down_cell(h, key);
    // a lane whose predecessor marks the same cell stays silent
    const uint32_t before = __shfl_up(cell, 1, 64);
    if (cell == ~0u || ((threadIdx.x & 63) != 0 && before == cell)) return;
    atomicOr(&bits[cell >> 5], 1u << (cell & 31));
}

__global__ void __launch_bounds__(kThreads) k_down_count(const uint64_t *__restrict__ words, const DownHead *__restrict__ head,
                                                         int32_t *__restrict__ totals) {
    const DownHead h = *head;
    const int wave = (int)blockIdx.x * (kThreads / 64) + (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int len = down_stretch(h), first = wave * len, end = min(first + len, h.n_words);
    int mine = 0;
    for (int w = first + lane; w < end; w += 64) mine += __popcll(words[w]);
    for (int d = 32; d >= 1; d >>= 1) mine += __shfl_xor(mine, d, 64);
    if (lane == 0) totals[wave] = mine;
}

// Every set bit becomes the key of its cell at the rank of the bit (see k_bits_expand), and the neighbour rows of
// the outputs found start out as "no neighbour": only as many rows are cleared as there are.  The positions of a
// step's bits go through LDS, so that a lane makes one output at a time (a lane making all outputs of its word
// kept its wave for up to 64 of them where points are dense: 14 us for 153 k points).
__global__ void __launch_bounds__(kThreads) k_down_expand(const uint64_t *__restrict__ words, const int4 *__restrict__ totals,
                                                          DownHead *__restrict__ head, uint64_t *__restrict__ out_keys,
                                                          int32_t *__restrict__ word_base, int4 *__restrict__ nbr, int *status) {
    __shared__ int sums[kThreads / 64];
    __shared__ uint16_t places[kThreads / 64][64 * 64];
    uint16_t *place = places[threadIdx.x >> 6];
    const DownHead h = *head;
    const int wave = (int)blockIdx.x * (kThreads / 64) + (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int len = down_stretch(h), first = wave * len, end = min(first + len, h.n_words);
    const bool last = blockIdx.x == kDownSweep - 1;
    if ((int)blockIdx.x * (kThreads / 64) * len >= h.n_words && !last) return;
    // outputs before this wave's stretch: the workgroup adds up the waves of all workgroups before it
    const int4 own = totals[blockIdx.x];
    int part = 0;
    for (int i = threadIdx.x; i < (int)blockIdx.x; i += kThreads) {
        const int4 t = totals[i];
        part += t.x + t.y + t.z + t.w;
    }
    for (int d = 32; d >= 1; d >>= 1) part += __shfl_xor(part, d, 64);
    if (lane == 0) sums[threadIdx.x >> 6] = part;
    __syncthreads();
    int before = sums[0] + sums[1] + sums[2] + sums[3];
    const int q = threadIdx.x >> 6;
    before += (q > 0 ? own.x : 0) + (q > 1 ? own.y : 0) + (q > 2 ? own.z : 0);
    for (int base = first; base < end; base += 64) {
        const int w = base + lane;
        uint64_t bits = w < end ? words[w] : 0;
        const int mine = __popcll(bits);
        int incl = mine;
        for (int d = 1; d < 64; d <<= 1) {
            const int up = __shfl_up(incl, d, 64);
            if (lane >= d) incl += up;
        }
        const int total = __shfl(incl, 63, 64);
        if (w < end) word_base[w] = before + incl - mine;
        for (int at = incl - mine; bits; bits &= bits - 1) place[at++] = (uint16_t)(lane * 64 + __builtin_ctzll(bits));
        __builtin_amdgcn_wave_barrier();
        for (int i = lane; i < total; i += 64) {
            uint32_t cell = (uint32_t)base * 64u + place[i];
            const int32_t z = (int32_t)(cell % h.ext[2]) + h.lo[2];
            cell /= h.ext[2];
            const int32_t y = (int32_t)(cell % h.ext[1]) + h.lo[1];
            cell /= h.ext[1];
            out_keys[before + i] = pack_key((int32_t)(cell / h.ext[0]), (int32_t)(cell % h.ext[0]) + h.lo[0], y, z);
        }
        for (int i = lane; i < total * (nbr_stride(8) / 4); i += 64)
            nbr[(int64_t)before * (nbr_stride(8) / 4) + i] = make_int4(-1, -1, -1, -1);
        __builtin_amdgcn_wave_barrier();
        before += total;
    }
    if (last && threadIdx.x == kThreads - 64) {   // the last stretch, empty or not
        head->count = before;
        tell_host(status, ST_COUNT, h.too_large ? kBoxTooLarge : before);
    }
}

// nbr[output][offset] = input, and the input's output, which is all that a transposed map needs.
__global__ void __launch_bounds__(kThreads) k_down_scatter(const uint64_t *__restrict__ keys, int64_t n, const DownHead *__restrict__ head,
                                                           const uint64_t *__restrict__ words, const int32_t *__restrict__ word_base,
                                                           int32_t *__restrict__ nbr, int32_t *__restrict__ parent) {
    const DownHead h = *head;
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n || h.n_words == 0) return;
    const uint64_t key = keys[i];
    int32_t k = -1;
    if (key != kEmptyKey) {
        const uint32_t cell = down_cell(h, key);
        k = word_base[cell >> 6] + __popcll(words[cell >> 6] & ((1ull << (cell & 63)) - 1ull));
        nbr[(int64_t)k * nbr_stride(8) + down_offset(key)] = (int32_t)i;
    }
    parent[i] = k;
}

// A row order for the output-stationary kernel on 2x2x2 maps that go up, where a row has one entry: a tile of 128
// neighbouring rows meets all eight offsets, each for an eighth of its rows; inside a window of 2048 rows those of one offset
// stand together, and a tile meets 1.4; a layer's stages fall by that much (128 -> 64 channels on 153 k rows of a scan 29.9 ->
// 23.1 us, on 100 k scattered ones 33.4 -> 23.3; 128 -> 96 on 64 k 21.8 -> 17.0).  Ranks come from ballots: the order is the
// same every time.  A workgroup takes a window, each thread kUpPer rows of it, own[r] being the offset of row
// base + r * kUpThreads + threadIdx.x: 0 to 7, 8 for a row without an entry, -1 past the last row.
constexpr int kUpThreads = 1024, kUpPer = 2, kUpRows = kUpThreads * kUpPer;
__device__ __forceinline__ void group_by_offset(const int (&own)[kUpPer], int64_t base, int64_t n, int32_t *__restrict__ perm) {
    constexpr int WAVES = kUpThreads / 64, CHUNKS = WAVES * kUpPer, CLASSES = 9;   // offsets, and none
    __shared__ int32_t before[CLASSES][CHUNKS], total[CLASSES];   // rows of a class in the chunks of 64 rows before
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int rank[kUpPer];   // how many of the row's chunk stand before it in its class
#pragma unroll
    for (int r = 0; r < kUpPer; ++r) {
        rank[r] = 0;
#pragma unroll
        for (int c = 0; c < CLASSES; ++c) {
            const uint64_t of_c = __ballot(own[r] == c);
            if (own[r] == c) rank[r] = __popcll(of_c & ((1ull << lane) - 1ull));
            if (lane == c) before[c][r * WAVES + wave] = __popcll(of_c);
        }
    }
    __syncthreads();
    if (wave < CLASSES) {
        const int rows = lane < CHUNKS ? before[wave][lane] : 0;
        int incl = rows;
        for (int d = 1; d < CHUNKS; d <<= 1) {
            const int up = __shfl_up(incl, d, 64);
            if (lane >= d) incl += up;
        }
        if (lane < CHUNKS) before[wave][lane] = incl - rows;
        if (lane == CHUNKS - 1) total[wave] = incl;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kUpPer; ++r) {
        const int64_t i = base + r * kUpThreads + threadIdx.x;
        if (own[r] >= 0) {
            int at = before[own[r]][r * WAVES + wave] + rank[r];
            for (int c = 0; c < own[r]; ++c) at += total[c];
            perm[base + at] = (int32_t)i;
        } else if (i < (n + kTileRows - 1) / kTileRows * kTileRows) {
            perm[i] = -1;
        }
    }
}

// That order for a map that was not transposed from one that goes down and has served a layer, or is about to serve one that
// gains by it (ts::order_windows).
__global__ void __launch_bounds__(kUpThreads) k_up_order(const int32_t *__restrict__ nbr, int64_t n, int32_t *__restrict__ perm) {
    const int64_t base = (int64_t)blockIdx.x * kUpRows;
    int own[kUpPer];
#pragma unroll
    for (int r = 0; r < kUpPer; ++r) {
        const int64_t i = base + r * kUpThreads + threadIdx.x;
        own[r] = -1;
        if (i < n) {
            const int4 *row = reinterpret_cast<const int4 *>(nbr + i * nbr_stride(8));
            const int4 a = row[0], b = row[1];
            own[r] = a.x >= 0 ? 0 : a.y >= 0 ? 1 : a.z >= 0 ? 2 : a.w >= 0 ? 3 : b.x >= 0 ? 4 : b.y >= 0 ? 5 : b.z >= 0 ? 6 : b.w >= 0 ? 7 : 8;
        }
    }
    group_by_offset(own, base, n, perm);
}

// The transposed map of such a map, in one pass over the fine points: a row has the one entry (offset of the
// point, its coarse cell).  Keys of both point sets are copied and the tile counters cleared on the way.
// (By scattering the forward rows into cleared rows and reading those again it took five launches.)
// perm, if not NULL: the rows' order, which costs the pass 1 to 2 us.
__global__ void __launch_bounds__(kUpThreads) k_up_rows(const uint64_t *__restrict__ fine, const int32_t *__restrict__ parent, int64_t n,
                                                        const uint64_t *__restrict__ coarse, int64_t n_coarse,
                                                        uint64_t *__restrict__ fine_copy, uint64_t *__restrict__ coarse_copy,
                                                        int32_t *__restrict__ nbr, uint64_t *__restrict__ colbits,
                                                        int32_t *__restrict__ colcnt, uint32_t *__restrict__ wavemask,
                                                        int64_t n_blocks, uint4 *__restrict__ sched, int32_t *__restrict__ perm) {
    constexpr int STRIDE = nbr_stride(8);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t base = (int64_t)blockIdx.x * kUpRows;
    for (int64_t v = (int64_t)blockIdx.x * kUpThreads + threadIdx.x; v < kMaxSchedSlices * kSchedWords / 4; v += (int64_t)gridDim.x * kUpThreads)
        sched[v] = make_uint4(0, 0, 0, 0);
    // A lane knows a row, four lanes write one: a wave's stores cover whole lines (a lane writing its own row touched 64 lines a
    // store: 10.2 us for 153 k rows, and 8.5).
    int own[kUpPer];
    uint64_t key[kUpPer];
    int32_t k[kUpPer];
#pragma unroll
    for (int r = 0; r < kUpPer; ++r) {
        const int64_t i = base + r * kUpThreads + threadIdx.x;
        key[r] = i < n ? fine[i] : 0;
        k[r] = i < n ? parent[i] : -1;
    }
#pragma unroll
    for (int r = 0; r < kUpPer; ++r) {
        const int64_t i = base + r * kUpThreads + threadIdx.x;
        if (i < n_coarse) coarse_copy[i] = coarse[i];   // (never more coarse points than fine ones)
        if (i < n) fine_copy[i] = key[r];
        const int q = down_offset(key[r]);
        const uint32_t mask = k[r] >= 0 ? 1u << q : 0u;
#pragma unroll
        for (int p = 0; p < STRIDE / 4; ++p) {
            const int unit = lane % (STRIDE / 4), from = p * (64 * 4 / STRIDE) + lane / (STRIDE / 4);
            const int32_t kk = __shfl(k[r], from, 64);
            const int at = __shfl(q, from, 64) - unit * 4, none = -1;
            const int64_t row = base + r * kUpThreads + wave * 64 + from;
            if (row < n) {
                const int4 v = unit < 2 ? make_int4(at == 0 ? kk : none, at == 1 ? kk : none, at == 2 ? kk : none, at == 3 ? kk : none)
                                        : make_int4(unit == 2 && kk >= 0 ? 1 << (at + 8) : unit == 2 ? 0 : none, none, none, none);
                reinterpret_cast<int4 *>(nbr)[row * (STRIDE / 4) + unit] = v;
            }
        }
        finish_rows<8>(mask, colbits, colcnt, wavemask, n_blocks, base / 64 + r * (kUpThreads / 64) + wave);
        own[r] = i >= n ? -1 : mask ? __builtin_ctz(mask) : 8;
    }
    if (perm) group_by_offset(own, base, n, perm);
}

// Block n: exclusive scan in place of the counts col[n][*] -> col[n][b] = pairs of offset n in the 64-row
// blocks before b (relative to the start of the offset's list), and the offset's total (the host
// turns the totals into offs[], the start of each offset's list, and hands them to later kernels
// by value).  The host takes the totals and ST_TILES for the end of the build, and may hand the map to another stream
// then: they are told after everything else, by workgroup.
constexpr int kScanThreads = 1024, kScanItems = 4;
__global__ void __launch_bounds__(kScanThreads) k_scan(int32_t *__restrict__ col, int64_t n_blocks, int *status, int K3,
                                                       const uint32_t *__restrict__ wavemask, int64_t n_tiles,
                                                       int32_t *__restrict__ tile_order, const int32_t *__restrict__ count) {
    if (count) {   // the number of rows is on the device only
        n_blocks = ((int64_t)*count + 63) / 64;
        n_tiles = ((int64_t)*count + kTileRows - 1) / kTileRows;
    }
    if ((int)blockIdx.x == K3) {
        // The extra block: tiles of 128 outputs (two waves of the search) in descending order of
        // the number of offsets they meet, a counting sort.  The fused kernel takes tiles in this
        // order, so that the long ones do not start when everything else is done.
        __shared__ int hist[32], base[32];
        if (threadIdx.x < 32) hist[threadIdx.x] = 0;
        __syncthreads();
        auto offsets_of = [&](int64_t t) {
            const uint32_t a = wavemask[2 * t], b = 2 * t + 1 < n_blocks ? wavemask[2 * t + 1] : 0u;
            return __builtin_popcount(a | b);
        };
        for (int64_t t = threadIdx.x; t < n_tiles; t += kScanThreads) atomicAdd(&hist[offsets_of(t)], 1);
        __syncthreads();
        if (threadIdx.x == 0) {
            int at = 0;
            for (int c = 31; c >= 0; --c) {
                base[c] = at;
                at += hist[c];
            }
        }
        __syncthreads();
        for (int64_t t = threadIdx.x; t < n_tiles; t += kScanThreads) tile_order[atomicAdd(&base[offsets_of(t)], 1)] = (int32_t)t;
        tell_host_done(status, ST_TILES, 1);
        return;
    }
    const int n = blockIdx.x;
    int32_t *c = col + (int64_t)n * n_blocks;
    int run = 0;
    for (int64_t base = 0; base < n_blocks; base += kScanThreads * kScanItems) {
        const int64_t i0 = base + (int64_t)threadIdx.x * kScanItems;
        int v[kScanItems], sum = 0;
#pragma unroll
        for (int e = 0; e < kScanItems; ++e) {
            v[e] = i0 + e < n_blocks ? c[i0 + e] : 0;
            sum += v[e];
        }
        int total;
        int at = run + block_exclusive_scan<kScanThreads>(sum, &total);
#pragma unroll
        for (int e = 0; e < kScanItems; ++e) {
            if (i0 + e < n_blocks) c[i0 + e] = at;
            at += v[e];
        }
        run += total;
    }
    tell_host_done(status, ST_TOTALS + n, run);
}

// ts_kmap_sort_rows, step 2: the distinct bitmasks as a dense list of (sort key, rows), followed
// by sentinel entries that sort last and hold no rows.
constexpr int kRankSlices = 32, kRankPer = 4, kRankUnroll = 16;
constexpr int kDensePad = kRankSlices * kRankUnroll;
__global__ void k_dense(const int *__restrict__ status, MaskHash mh, int K3, int2 *__restrict__ dense) {
    int D = status[ST_DCOUNT];
    D = D < mh.dmax ? D : mh.dmax;
    const int d = blockIdx.x * blockDim.x + threadIdx.x;
    if (d < D) {
        const int sl = mh.dlist[d];
        dense[d] = make_int2((int)mask_sort_key(mh.key[sl], K3), mh.cnt[sl]);
    } else if (d < mh.dmax + kDensePad) {
        dense[d] = make_int2(-1, 0);
    }
}

// ts_kmap_sort_rows, step 3: start of mask d = rows whose mask sorts lower.  Block (d-block, slice)
// adds up, for 1024 masks (4 per thread), the rows of the lower masks found in one slice of the
// list; k_rank_sum adds the slices.  The list is read with wave-uniform addresses (scalar loads),
// so the inner loop is compare / select / add only.
__global__ void __launch_bounds__(kThreads) k_rank_partial(const int2 *__restrict__ dense, const int *__restrict__ status,
                                                           int dmax, int32_t *__restrict__ partial) {
    const int rb = blockIdx.x, dblk = rb / kRankSlices, slice = rb % kRankSlices;
    int D = status[ST_DCOUNT];
    D = D < dmax ? D : dmax;
    if (dblk * kThreads * kRankPer >= D) return;
    // slices are whole groups of kRankUnroll entries; what lies behind the list are sentinels
    const int per = ((D + kRankSlices - 1) / kRankSlices + kRankUnroll - 1) / kRankUnroll * kRankUnroll;
    const int lo = slice * per, hi = lo + per;
    uint32_t my_key[kRankPer];
    int sum[kRankPer];
#pragma unroll
    for (int e = 0; e < kRankPer; ++e) {
        const int d = (dblk * kRankPer + e) * kThreads + threadIdx.x;
        my_key[e] = d < D ? (uint32_t)dense[d].x : 0u;
        sum[e] = 0;
    }
    for (int q = lo; q < hi; q += kRankUnroll) {
        int2 kc[kRankUnroll];   // same addresses in every lane; all loaded before the first use
#pragma unroll
        for (int u = 0; u < kRankUnroll; ++u) kc[u] = dense[q + u];
#pragma unroll
        for (int u = 0; u < kRankUnroll; ++u)
#pragma unroll
            for (int e = 0; e < kRankPer; ++e) sum[e] += (uint32_t)kc[u].x < my_key[e] ? kc[u].y : 0;
    }
#pragma unroll
    for (int e = 0; e < kRankPer; ++e) {
        const int d = (dblk * kRankPer + e) * kThreads + threadIdx.x;
        if (d < D) partial[(int64_t)slice * dmax + d] = sum[e];
    }
}

__global__ void k_rank_sum(const int32_t *__restrict__ partial, const int *__restrict__ status, MaskHash mh) {
    int D = status[ST_DCOUNT];
    D = D < mh.dmax ? D : mh.dmax;
    const int d = blockIdx.x * blockDim.x + threadIdx.x;
    if (d >= D) return;
    int sum = 0;
#pragma unroll
    for (int sl = 0; sl < kRankSlices; ++sl) sum += partial[(int64_t)sl * mh.dmax + d];
    mh.start[mh.dlist[d]] = sum;
}

// ts_kmap_sort_rows, step 4: perm[start of the row's mask + arrival rank] = row.
__global__ void k_place(const int2 *__restrict__ slot_rank, int64_t n_out, MaskHash mh, int32_t *__restrict__ perm) {
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n_out) return;
    const int2 sr = slot_rank[k];
    if (sr.x < 0) return;
    const int64_t pos = (int64_t)mh.start[sr.x] + sr.y;
    if (pos >= 0 && pos < n_out) perm[pos] = (int32_t)k;   // (out of range only when the table overflowed)
}

// Pair lists: thread per output row; the pair (k, n) goes to offs[n] + colbase[n][k/64] + (outputs of the
// same 64-block with offset n before k), which keeps ascending output order inside an offset.  A caller's own lists, where they
// were asked for, are written along with the map's: for the 4.6 M pairs of 471 k points 32.5 us, where the map's lists take
// 23.2 and two copies 14.5.  (Pairs put in order in LDS first, 256 rows at a time, so that those of an offset leave as whole
// lines: 37 us.)
template <int K3>
__global__ void __launch_bounds__(kThreads) k_compact(const int32_t *__restrict__ nbr, int64_t n_out,
                                                      const int32_t *__restrict__ colbase, int64_t n_blocks,
                                                      Offs offs, int32_t *__restrict__ in_idx, int32_t *__restrict__ out_idx,
                                                      int32_t *__restrict__ in_copy, int32_t *__restrict__ out_copy) {
    constexpr int STRIDE = nbr_stride(K3), CHUNKS = (K3 + 3) / 4;
    const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const int lane = threadIdx.x & 63;
    const int64_t block64 = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    int base_mine = 0;
    if (lane < K3 && block64 < n_blocks) base_mine = offs.v[lane] + colbase[(int64_t)lane * n_blocks + block64];
    int32_t j[CHUNKS * 4];
#pragma unroll
    for (int ch = 0; ch < CHUNKS; ++ch) {
        int4 v = make_int4(-1, -1, -1, -1);
        if (k < n_out) v = reinterpret_cast<const int4 *>(nbr + k * STRIDE)[ch];
        j[ch * 4 + 0] = v.x;
        j[ch * 4 + 1] = v.y;
        j[ch * 4 + 2] = v.z;
        j[ch * 4 + 3] = v.w;
    }
#pragma unroll
    for (int n = 0; n < K3; ++n) {
        const bool has = j[n] >= 0;
        const uint64_t bal = __ballot(has);
        const int base = __shfl(base_mine, n, 64);
        if (has) {
            const int p = base + __popcll(bal & ((1ull << lane) - 1ull));
            in_idx[p] = j[n];
            out_idx[p] = (int32_t)k;
            if (in_copy) in_copy[p] = j[n];
            if (out_copy) out_copy[p] = (int32_t)k;
        }
    }
}

// Fallback ordering input: the sort key of each row's bitmask and the identity row list.
__global__ void k_extract_masks(const int32_t *__restrict__ nbr, int64_t n_out, int stride, int K3,
                                uint32_t *__restrict__ keys, int32_t *__restrict__ rows) {
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n_out) return;
    keys[k] = mask_sort_key((uint32_t)nbr[k * stride + K3], K3);
    rows[k] = (int32_t)k;
}

inline unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

// Owns the temporaries of one build; everything goes back to the pool on scope exit.
struct Temps {
    void *p[48];
    int n = 0;
    template <class T>
    int get(T **out, size_t count) {
        int rc = alloc_n(out, count);
        if (rc == TS_OK) p[n++] = *out;
        return rc;
    }
    ~Temps() {
        for (int i = 0; i < n; ++i) dev_free(p[i]);
    }
};

int launch_fill(const FillArgs &f) {
    if (f.n == 0) return TS_OK;
    uint64_t most = 0;
    for (int i = 0; i < f.n; ++i) most = f.seg[i].n_vec > most ? f.seg[i].n_vec : most;
    unsigned blocks = blocks_for((int64_t)most, kThreads);
    if (blocks > 4096) blocks = 4096;
    TS_LAUNCH("k_fill", k_fill, dim3(blocks), dim3(kThreads), f);
    return TS_OK;
}

// Allocates the table; its clearing is added to `fill`.
int make_table(Temps &tmp, int64_t entries, Table *t, FillArgs *fill) {
    uint64_t cap = 1024;
    while (cap < (uint64_t)(4 * entries)) cap <<= 1;
    if (cap > (1ull << 28)) return fail(TS_ERR_UNSUPPORTED, "too many points for the hash table");
    TS_TRY(tmp.get(&t->keys, cap));
    TS_TRY(tmp.get(&t->vals, cap));
    t->mask = (uint32_t)(cap - 1);
    t->shift = 64 - __builtin_ctzll(cap >> kBucketLog2);
    fill->add(t->keys, cap * sizeof(uint64_t), 0xFFFFFFFFu);
    return TS_OK;
}

// Allocates the block table; the clearing of its entries (free key, empty mask) is added to `fill`.
// A row number per cell of every slot takes 384 to 768 bytes per point, nearly all of it never touched, and is gone when
// the build is.  Where that much cannot be had the rows are packed, which takes 10 to 16: two launches more, over the
// entries and over the points (LiDAR scenes: 153 k points 26 us and 35, 1.5 M 178 and 245, 15 M 1.87 ms and 2.33).
// counter: what k_block_base counts with then.
int make_block_table(Temps &tmp, int64_t points, BlockTable *t, int32_t **counter, FillArgs *fill) {
    uint64_t cap = 1024;
    while (2 * cap < (uint64_t)(3 * points)) cap <<= 1;
    TS_TRY(tmp.get(&t->ent, 2 * cap));
    t->base = nullptr;
    int rc = tmp.get(&t->rows, 64 * cap);
    if (rc == TS_ERR_OOM) {
        TS_TRY(tmp.get(&t->rows, (size_t)points));
        TS_TRY(tmp.get(&t->base, cap));
        TS_TRY(tmp.get(counter, 4));
        fill->add(*counter, 16, 0u);
    } else if (rc != TS_OK) {
        return rc;
    }
    t->mask = (uint32_t)(cap - 1);
    t->shift = 64 - __builtin_ctzll(cap >> 3);
    fill->add_pairs(t->ent, cap * 16, 0xFFFFFFFFu, 0u);
    return TS_OK;
}

// How a build was asked to run.
struct BuildOpts {
    bool wait = true;
    bool measure = false;   // strided builds: measure the bounding box on the device and use the grid if it is small enough
    bool grid = false;      // hold the searched set in the coordinate grid instead of the hash table
    Box box = {};           // bounds stated for the caller's coordinates (grid search)
    Bound bound = {};       // Alg. 3's boundary, already multiplied by the stride
};

// The searched point set of a build: in the hash table or in the grid.
struct Searched {
    bool grid = false;
    Table t = {};
    Grid g = {};
};

// The grid's cells: kept between builds, every cell -1 whenever no build is using them.
constexpr uint64_t kMaxGridCells = 1ull << 30;    // 4 GiB of cells: what a caller may ask for
constexpr uint64_t kAutoGridCells = 1ull << 28;   // output cells (bits of the bitmap: 32 MiB) up to which a strided build
                                                  // that measures its own box marks its candidates instead of sorting them
int32_t *g_grid = nullptr;
uint64_t g_grid_cells = 0;
bool g_grid_dirty = false;   // a build put points in and did not get as far as taking them out

// A grid over batches x [lo, hi] (inclusive).  Grows the buffer when the box needs more cells than it
// has; clears it only when new or left dirty by a build that failed half way.
int acquire_grid(const int32_t lo[3], const int32_t hi[3], int batches, Grid *g) {
    uint64_t cells = (uint64_t)batches;
    for (int a = 0; a < 3; ++a) {
        const int64_t ext = (int64_t)hi[a] - lo[a] + 1;
        if (ext <= 0 || batches <= 0) return fail(TS_ERR_INVALID_ARG, "empty grid bounds");
        g->lo[a] = lo[a];
        g->ext[a] = (uint32_t)ext;
        cells *= (uint64_t)ext;
        if (cells > kMaxGridCells)
            return fail(TS_ERR_UNSUPPORTED, "the grid bounds span more than %llu cells", (unsigned long long)kMaxGridCells);
    }
    g->batches = (uint32_t)batches;
    if (cells > g_grid_cells) {
        if (g_grid) {
            TS_HIP(hipStreamSynchronize(stream()));
            (void)hipFree(g_grid);
            g_grid = nullptr;
            g_grid_cells = 0;
        }
        const uint64_t want = (cells + 3) & ~3ull;
        if (hipMalloc(&g_grid, want * sizeof(int32_t)) != hipSuccess) {
            (void)hipGetLastError();
            g_grid = nullptr;
            return fail(TS_ERR_OOM, "no memory for a grid of %llu cells", (unsigned long long)cells);
        }
        g_grid_cells = want;
        g_grid_dirty = true;
    }
    if (g_grid_dirty) {
        FillArgs f;
        f.add(g_grid, g_grid_cells * sizeof(int32_t), 0xFFFFFFFFu);
        TS_TRY(launch_fill(f));
    }
    g_grid_dirty = true;   // until this build has taken its points out again
    g->vals = g_grid;
    return TS_OK;
}

// Table or grid for `entries` points inside batches x [lo, hi].
int make_searched(Temps &tmp, const BuildOpts &o, int64_t entries, const int32_t lo[3], const int32_t hi[3], Searched *sd,
                  FillArgs *fill) {
    sd->grid = o.grid;
    if (o.grid) return acquire_grid(lo, hi, o.box.batches, &sd->g);
    return make_table(tmp, entries, &sd->t, fill);
}

int make_mask_hash(Temps &tmp, MaskHash *mh, FillArgs *fill) {
    int32_t *cnt_start;
    TS_TRY(tmp.get(&mh->key, (size_t)kMaskHashCap));
    TS_TRY(tmp.get(&cnt_start, (size_t)2 * kMaskHashCap));
    TS_TRY(tmp.get(&mh->dlist, (size_t)kMaskHashMaxDistinct));
    mh->cnt = cnt_start;
    mh->start = cnt_start + kMaskHashCap;
    mh->cap_mask = kMaskHashCap - 1;
    mh->shift = 32 - __builtin_ctz(kMaskHashCap);
    mh->dmax = kMaskHashMaxDistinct;
    fill->add(mh->key, (size_t)kMaskHashCap * sizeof(uint32_t), 0xFFFFFFFFu);
    // counts and first positions: a mask that entered the table after the list of distinct masks
    // was full is never ranked, and its rows must not be placed through a stale position
    fill->add(cnt_start, (size_t)2 * kMaskHashCap * sizeof(int32_t), 0u);
    return TS_OK;
}

// The status words of a build, in pinned host memory (see ST_*).  A map that nobody has asked anything yet
// keeps its slot; a slot whose map was freed first is handed out again once its build has reported.
struct StatusSlot {
    int32_t *host = nullptr;
    int32_t *dev = nullptr;     // the same words as kernels address them
    bool busy = false;          // a build reports, or will report, here
    bool totals = false;        // ... the map sizes as well
    int K3 = 0;
    const ts_kmap *owner = nullptr;   // NULL while busy: the map was freed before anyone asked
    bool recorded = false;      // a graph reports here, at every replay: the slot stays its own
    hipStream_t stream = nullptr;     // where that was recorded
};
constexpr int kSlotChunk = 64, kSlotChunks = 1024;   // slots come 64 to an allocation, 65536 at most
StatusSlot *g_slots[kSlotChunks] = {nullptr};

inline StatusSlot &slot_at(int i) { return g_slots[i / kSlotChunk][i % kSlotChunk]; }

// Whether what the slot's build reports has arrived: the box of its points or the number of coarse ones (strided
// builds), the verdict on its input, or the sizes too.
enum Awaited { kBox, kCount, kVerdict, kSizes };
inline bool slot_landed(const StatusSlot &s, Awaited what) {
    const volatile int32_t *h = s.host;
    if (what == kBox) return h[ST_BOXED] != 0;
    if (what == kCount) return h[ST_COUNT] != -1;
    if (what == kVerdict) return h[ST_SEARCHED] != 0 || (s.totals && slot_landed(s, kSizes));   // sizes come after everything else
    for (int n = 0; n < s.K3; ++n)
        if (h[ST_TOTALS + n] < 0) return false;
    return h[ST_TILES] != 0;
}

inline void slot_reset(StatusSlot &s, int K3) {
    std::memset(s.host, 0, ST_WORDS * sizeof(int32_t));
    for (int n = 0; n < kMaxK3; ++n) s.host[ST_TOTALS + n] = -1;
    s.host[ST_COUNT] = -1;
    s.K3 = K3;
    s.totals = false;
}

// Call when work that reports to the slot is enqueued.
inline void slot_recorded(StatusSlot &s) {
    if (s.recorded || !stream_capturing(stream())) return;
    s.recorded = true;
    s.stream = stream();
}

// A free slot, its words reset; -1 with the error set.
int slot_acquire(int K3) {
    for (int ch = 0; ch < kSlotChunks; ++ch) {
        if (!g_slots[ch]) {
            int32_t *mem = nullptr;
            void *dview = nullptr;
            if (hipHostMalloc(&mem, kSlotChunk * ST_WORDS * sizeof(int32_t), hipHostMallocDefault) != hipSuccess ||
                hipHostGetDevicePointer(&dview, mem, 0) != hipSuccess) {
                (void)hipGetLastError();
                if (mem) (void)hipHostFree(mem);
                fail(TS_ERR_OOM, "no pinned memory for a build's status words");
                return -1;
            }
            StatusSlot *sl = new (std::nothrow) StatusSlot[kSlotChunk];
            if (!sl) {
                (void)hipHostFree(mem);
                fail(TS_ERR_OOM, "host allocation failed");
                return -1;
            }
            for (int i = 0; i < kSlotChunk; ++i) {
                sl[i].host = mem + i * ST_WORDS;
                sl[i].dev = static_cast<int32_t *>(dview) + i * ST_WORDS;
            }
            g_slots[ch] = sl;
        }
        for (int i = 0; i < kSlotChunk; ++i) {
            StatusSlot &s = g_slots[ch][i];
            if (s.recorded || (s.busy && (s.owner || !slot_landed(s, s.totals ? kSizes : kVerdict)))) continue;
            slot_reset(s, K3);
            s.busy = true;
            s.owner = nullptr;
            slot_recorded(s);
            return ch * kSlotChunk + i;
        }
    }
    fail(TS_ERR_OOM, "more than %d maps await their build's verdict", kSlotChunk * kSlotChunks);
    return -1;
}

inline void slot_release(int i) {
    slot_at(i).busy = false;
    slot_at(i).owner = nullptr;
}

// Watches the slot's words.  The stream is asked now and then whether it has finished or failed, so that a
// build that cannot report any more (an error of the device) ends the wait.  A stream that is being captured must
// not be asked: what was enqueued before reports all the same, what is being recorded does not.
constexpr int kCaptureWaitSeconds = 20;
int slot_wait(int i, Awaited what) {
    const StatusSlot &s = slot_at(i);
    std::chrono::steady_clock::time_point begin{};
    for (;;) {
        for (int spin = 0; spin < 20000; ++spin) {
            if (slot_landed(s, what)) return TS_OK;
            __builtin_ia32_pause();
        }
        if (s.recorded && stream_capturing(s.stream))
            return fail(TS_ERR_UNSUPPORTED, "the build of this map is being recorded into a graph and reports nothing before that runs");
        if (stream_capturing(stream())) {
            const auto now = std::chrono::steady_clock::now();
            if (begin == std::chrono::steady_clock::time_point{}) begin = now;
            if (now - begin > std::chrono::seconds(kCaptureWaitSeconds)) return fail(TS_ERR_HIP, "a map build has not reported for %d s", kCaptureWaitSeconds);
            continue;
        }
        const hipError_t e = hipStreamQuery(stream());
        if (e == hipErrorNotReady) {
            (void)hipGetLastError();
            continue;
        }
        if (slot_landed(s, what)) return TS_OK;
        if (e != hipSuccess) return fail(TS_ERR_HIP, "waiting for a map build: %s", hipGetErrorString(e));
        TS_HIP(hipDeviceSynchronize());   // another stream than the one the build ran on is current
        if (slot_landed(s, what)) return TS_OK;
        return fail(TS_ERR_HIP, "a map build finished without reporting");
    }
}

// Status words on the host -> the map's error, or that and its sizes.
int take_verdict(ts_kmap *m, const int32_t *h) {
    if (h[ST_RANGE]) m->error = TS_ERR_COORD_RANGE;
    else if (h[ST_DUP]) m->error = TS_ERR_DUPLICATE_COORD;
    return m->error;
}

int take_status(ts_kmap *m, const int32_t *h) {
    take_verdict(m, h);
    m->offs[0] = 0;
    for (int n = 0; n < m->K3; ++n) m->offs[n + 1] = m->offs[n] + h[ST_TOTALS + n];
    for (int n = 0; n < m->K3; ++n) m->sizes[n] = m->offs[n + 1] - m->offs[n];
    m->M = m->offs[m->K3];
    if (m->one_pair_per_input && m->error == TS_OK && m->M < m->n_in) m->error = TS_ERR_DUPLICATE_COORD;
    return m->error;
}

int report(const ts_kmap *m) {
    if (m->error == TS_ERR_COORD_RANGE)
        return fail(TS_ERR_COORD_RANGE, "coordinate outside batch [0,%d] / xyz [%d,%d], or outside the grid bounds given", TS_BATCH_MAX, TS_COORD_MIN, TS_COORD_MAX);
    if (m->error == TS_ERR_DUPLICATE_COORD) return fail(TS_ERR_DUPLICATE_COORD, "input coordinates are not distinct");
    return m->error;
}

// The map of a 1x1x1 convolution at stride 1 over n distinct points, written out directly: output k
// takes input k through the only offset (Eq. 1 with delta = 0).  One pass fills the neighbour rows
// (entry, then the bitmask word), the rank structure (every row present: bitmap words of ones, base 64 b)
// and the tile order, and clears the tile counters (2.3 us by a launch of their own).
__global__ void __launch_bounds__(kThreads) k_identity_map(int32_t *__restrict__ nbr, int stride, uint64_t *__restrict__ colbits,
                                                           int32_t *__restrict__ colbase, int32_t *__restrict__ tile_order,
                                                           int64_t n, int64_t n_blocks, int64_t n_tiles, uint4 *__restrict__ sched) {
    const int64_t g = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    for (int64_t v = g; v < kMaxSchedSlices * kSchedWords / 4; v += (int64_t)gridDim.x * kThreads) sched[v] = make_uint4(0, 0, 0, 0);
    if (g < n) {
        int4 row = make_int4((int32_t)g, 1, -1, -1);
        *reinterpret_cast<int4 *>(nbr + g * stride) = row;
    }
    if (g < n_blocks) {
        const int64_t left = n - g * 64;
        colbits[g] = left >= 64 ? ~0ull : ((1ull << left) - 1ull);
        colbase[g] = (int32_t)(g * 64);
    }
    if (g < n_tiles) tile_order[g] = (int32_t)g;
}

void destroy(ts_kmap *m) {
    if (!m) return;
    if (m->pending_slot >= 0) slot_at(m->pending_slot).owner = nullptr;   // handed out again once the build has reported
    if (m->d_out_keys != m->d_in_keys) dev_free(m->d_out_keys);
    dev_free(m->d_in_keys);
    dev_free(m->d_nbr);
    dev_free(m->d_in_idx);
    dev_free(m->d_out_idx);
    dev_free(m->d_colbits);
    dev_free(m->d_colbase);
    dev_free(m->d_perm);
    dev_free(m->d_sched);
    dev_free(m->d_tile_order);
    dev_free(m->d_wavemask);
    dev_free(m->d_parent);
    dev_free(m->d_rowmask);
    dev_free(m->d_window_perm);
    delete m;
}

int sort_keys(Temps &tmp, uint64_t *in, uint64_t *out, size_t n) {
    size_t bytes = 0;
    TS_HIP(rocprim::radix_sort_keys(nullptr, bytes, in, out, n, 0, 64, stream()));
    void *ws;
    TS_TRY(tmp.get((char **)&ws, bytes));
    ProfScope ps("sort_keys");
    TS_HIP(rocprim::radix_sort_keys(ws, bytes, in, out, n, 0, 64, stream()));
    return TS_OK;
}

template <int MODE, int K>
void launch_probe(const ts_kmap *m, const Searched &sd) {
    if (sd.grid)
        TS_LAUNCH("k_probe_grid", (k_probe<MODE, K, Grid>), dim3(blocks_for(m->n_out, kThreads)), dim3(kThreads), m->d_out_keys,
                  m->n_out, sd.g, m->s, m->d_nbr, m->d_colbits, m->d_colbase, m->d_wavemask, m->n_blocks);
    else
        TS_LAUNCH("k_probe", (k_probe<MODE, K, Table>), dim3(blocks_for(m->n_out, kThreads)), dim3(kThreads), m->d_out_keys,
                  m->n_out, sd.t, m->s, m->d_nbr, m->d_colbits, m->d_colbase, m->d_wavemask, m->n_blocks);
}

void launch_rows(const ts_kmap *m) {
    const dim3 grid(blocks_for(m->n_out, kThreads)), block(kThreads);
#define TS_ROWS(K3, CENTRE) TS_LAUNCH("k_rows", (k_rows<K3, CENTRE>), grid, block, m->d_nbr, m->d_out_keys, m->n_out, nullptr, m->d_colbits, m->d_colbase, m->d_wavemask, m->n_blocks)
    if (m->K3 == 27 && m->centre >= 0) TS_ROWS(27, true);
    else if (m->K3 == 27) TS_ROWS(27, false);
    else if (m->K3 == 8) TS_ROWS(8, false);
    else TS_ROWS(1, false);
#undef TS_ROWS
}

// Counts of the 64-row blocks -> ranks, sizes (into the status words at `status`) and tile order.
void launch_scan(const ts_kmap *m, int32_t *status) {
    TS_LAUNCH("k_scan", k_scan, dim3(m->K3 + 1), dim3(kScanThreads), m->d_colbase, m->n_blocks, status, m->K3, m->d_wavemask,
              m->n_tiles, m->d_tile_order, nullptr);
}

// Map search through the hash table or the coordinate grid.  `table` holds the searched point set (the map's
// inputs), m->d_out_keys the outputs.  Leaves the neighbour rows and the presence bitmaps and counts; those of the
// grid's symmetric search come from the row pass, which is left to the caller or to ts::prepare (rows_put_off).
int search(ts_kmap *m, const Searched &table, int *status) {
    const int K = m->K, mode = m->s == 1 ? MODE_SUB : (m->transposed ? MODE_TR : MODE_FWD);
    const bool symmetric = mode == MODE_SUB && K == 3;   // only the grid: tables of points search k_block_search's way
    if (mode == MODE_SUB && K == 1) launch_probe<MODE_SUB, 1>(m, table);
    else if (symmetric)
        TS_LAUNCH("k_probe_symmetric_grid", k_probe_symmetric, dim3(blocks_for(m->n_out * 16, kThreads)), dim3(kThreads), m->d_out_keys,
                  m->n_out, table.g, K, m->d_nbr, m->stride, status);
    else if (mode == MODE_FWD && K == 1) launch_probe<MODE_FWD, 1>(m, table);
    else if (mode == MODE_TR && K == 1) launch_probe<MODE_TR, 1>(m, table);
    else if (mode == MODE_FWD && K == 2) launch_probe<MODE_FWD, 2>(m, table);
    else if (mode == MODE_FWD && K == 3) launch_probe<MODE_FWD, 3>(m, table);
    else if (mode == MODE_TR && K == 2) launch_probe<MODE_TR, 2>(m, table);
    else if (mode == MODE_TR && K == 3) launch_probe<MODE_TR, 3>(m, table);
    else return fail(TS_ERR_UNSUPPORTED, "no map search for kernel_size %d, stride %d", K, m->s);
    if (table.grid) {   // the grid gets its points taken out as soon as the search has been enqueued
        TS_LAUNCH("k_grid_erase", k_grid_erase, dim3(blocks_for(m->n_in, kThreads)), dim3(kThreads), m->d_in_keys, m->n_in, table.g);
        g_grid_dirty = false;
    }
    m->rows_put_off = symmetric;
    return TS_OK;
}

// End of a build whose rows and presence bitmaps have been enqueued: the scan, and a wait for the sizes or
// none.  scan_later: the scan is put off until something needs it (ts_kmap_prepare, ts::resolve); the kernels
// of such a build report ST_SEARCHED.
int finish(ts_kmap *m, int slot, bool wait, bool scan_later = false) {
    StatusSlot &sl = slot_at(slot);
    if (!scan_later || wait) {
        if (m->rows_put_off) launch_rows(m);
        m->rows_put_off = false;
        launch_scan(m, sl.dev);
        sl.totals = true;
        m->scan_enqueued = true;
    }
    m->scan_done = false;
    m->stream = stream();
    sl.owner = m;
    m->pending_slot = slot;
    TS_HIP(hipGetLastError());
    // temporaries go back to the pool when the caller's Temps dies; later work on the same
    // stream is ordered after the kernels above, so reuse is safe without a wait
    return wait ? resolve(m) : TS_OK;
}

// Whether the table of bitmasks was too small, for the host.
__global__ void k_tell_overflow(const int *d_status, int *status) { tell_host(status, ST_COUNT, d_status[ST_OVERFLOW] != 0); }

// Orders the output rows by offset bitmask (see the head of this file).  The order is complete on return.
int sort_rows(ts_kmap *m) {
    hipStream_t st = stream();
    Temps tmp;
    const int K3 = m->K3;
    const int64_t n_out = m->n_out;
    int *d_status;
    int2 *slot_rank, *dense;
    int32_t *partial, *perm;
    MaskHash mh;
    FillArgs fill;
    const int64_t n_tiles = (n_out + kTileRows - 1) / kTileRows;
    TS_TRY(tmp.get(&d_status, ST_WORDS));
    TS_TRY(tmp.get(&slot_rank, (size_t)n_out));
    TS_TRY(alloc_n(&perm, (size_t)n_tiles * kTileRows));
    fill.add(d_status, ST_WORDS * sizeof(int), 0u);
    fill.add(perm, (size_t)n_tiles * kTileRows * sizeof(int32_t), 0xFFFFFFFFu);
    int rc = make_mask_hash(tmp, &mh, &fill);
    if (rc == TS_OK) rc = tmp.get(&dense, (size_t)mh.dmax + kDensePad);
    if (rc == TS_OK) rc = tmp.get(&partial, (size_t)kRankSlices * mh.dmax);
    const int slot = rc == TS_OK ? slot_acquire(0) : -1;   // (see build_strided: 127 -> 114 us with the build of 153 k points, 83 -> 60 of 8 k)
    if (rc == TS_OK && slot < 0) rc = last_fail_code();
    if (rc != TS_OK) {
        dev_free(perm);
        return rc;
    }
    auto body = [&]() -> int {
        TS_TRY(launch_fill(fill));
        const dim3 grid(blocks_for(n_out, kThreads)), block(kThreads);
        TS_LAUNCH("k_register", k_register, grid, block, m->d_nbr, n_out, m->stride, K3, d_status, mh, slot_rank);
        TS_LAUNCH("k_dense", k_dense, dim3(blocks_for(mh.dmax + kDensePad, kThreads)), block, d_status, mh, K3, dense);
        {
            const unsigned rank_blocks = (unsigned)(mh.dmax / (kThreads * kRankPer)) * kRankSlices;
            ProfScope ps("k_rank");
            hipLaunchKernelGGL(k_rank_partial, dim3(rank_blocks), block, 0, st, dense, d_status, mh.dmax, partial);
            hipLaunchKernelGGL(k_rank_sum, dim3(mh.dmax / kThreads), block, 0, st, partial, d_status, mh);
        }
        TS_LAUNCH("k_place", k_place, grid, block, slot_rank, n_out, mh, perm);
        TS_LAUNCH("k_tell_overflow", k_tell_overflow, dim3(1), dim3(1), d_status, slot_at(slot).dev);
        TS_TRY(slot_wait(slot, kCount));
        if (slot_at(slot).host[ST_COUNT]) {
            // more distinct bitmasks than the table ranks: order the rows with a radix sort instead
            uint32_t *keys, *keys_sorted;
            int32_t *rows;
            TS_TRY(tmp.get(&keys, (size_t)n_out));
            TS_TRY(tmp.get(&keys_sorted, (size_t)n_out));
            TS_TRY(tmp.get(&rows, (size_t)n_out));
            TS_LAUNCH("k_extract_masks", k_extract_masks, grid, block, m->d_nbr, n_out, m->stride, K3, keys, rows);
            size_t bytes = 0;
            TS_HIP(rocprim::radix_sort_pairs(nullptr, bytes, keys, keys_sorted, rows, perm, (size_t)n_out, 0, K3, st));
            void *ws;
            TS_TRY(tmp.get((char **)&ws, bytes));
            ProfScope ps("sort_masks");
            TS_HIP(rocprim::radix_sort_pairs(ws, bytes, keys, keys_sorted, rows, perm, (size_t)n_out, 0, K3, st));
            TS_HIP(hipStreamSynchronize(st));
        }
        TS_HIP(hipGetLastError());
        return TS_OK;
    };
    rc = body();
    if (rc != TS_OK) (void)hipStreamSynchronize(st);
    slot_release(slot);
    if (rc != TS_OK) {
        dev_free(perm);
        return rc;
    }
    m->d_perm = perm;
    return TS_OK;
}

// Allocations of the map that depend on n_out only.
int alloc_outputs(ts_kmap *m, FillArgs *fill) {
    const int K3 = m->K3;
    m->stride = nbr_stride(K3);
    m->n_blocks = (m->n_out + 63) / 64;
    m->n_tiles = (m->n_out + kTileRows - 1) / kTileRows;
    TS_TRY(alloc_n(&m->d_nbr, (size_t)m->n_out * m->stride));
    TS_TRY(alloc_n(&m->d_colbits, (size_t)K3 * m->n_blocks));
    TS_TRY(alloc_n(&m->d_colbase, (size_t)K3 * m->n_blocks));
    TS_TRY(alloc_n(&m->d_tile_order, (size_t)m->n_tiles));
    TS_TRY(alloc_n(&m->d_wavemask, (size_t)m->n_blocks));
    TS_TRY(alloc_n(&m->d_sched, (size_t)kMaxSchedSlices * kSchedWords));
    if (fill) fill->add(m->d_sched, (size_t)kMaxSchedSlices * kSchedWords * sizeof(int32_t), 0u);   // (else the caller's kernel clears them)
    return TS_OK;
}

// The device-driven build of a 2x2x2 stride-2 map (see DownHead): arrays for the most outputs there can be, all
// launches, no wait.  The bitmap of a box that has to be measured first holds as many cells as one may have.
int build_down(Temps &tmp, const int32_t *coords, int64_t N, ts_kmap *m, const BuildOpts &opt, int slot) {
    StatusSlot &sl = slot_at(slot);
    uint64_t max_cells = kAutoGridCells;
    if (opt.grid) {
        max_cells = (uint64_t)opt.box.batches;
        for (int a = 0; a < 3; ++a) {
            max_cells *= (uint64_t)((opt.box.hi[a] >> 1) - (opt.box.lo[a] >> 1) + 1);
            if (max_cells > kMaxGridCells)
                return fail(TS_ERR_UNSUPPORTED, "the grid bounds span more than %llu cells", (unsigned long long)kMaxGridCells);
        }
    }
    const uint64_t max_words = (max_cells + 63) / 64;
    uint64_t *words;
    int32_t *word_base, *totals;
    int4 *parts;
    DownHead *head;
    TS_TRY(tmp.get(&words, max_words + 1));   // (cleared two at a time)
    TS_TRY(tmp.get(&word_base, max_words));
    TS_TRY(tmp.get(&totals, kDownWaves));
    TS_TRY(tmp.get(&parts, 2 * kDownPack));
    TS_TRY(tmp.get(&head, 1));
    m->n_in = N;
    m->n_out = N;   // what the arrays are made for
    TS_TRY(alloc_outputs(m, nullptr));
    TS_TRY(alloc_n(&m->d_out_keys, (size_t)N));
    TS_TRY(alloc_n(&m->d_parent, (size_t)N));
    const unsigned n_parts = blocks_for(N, kThreads) < kDownPack ? blocks_for(N, kThreads) : kDownPack;
    const dim3 per_point(blocks_for(N, kThreads)), sweep(kDownSweep), block(kThreads);
    TS_LAUNCH("k_down_pack", k_down_pack, dim3(n_parts), block, reinterpret_cast<const int4 *>(coords), N, m->d_in_keys, sl.dev, opt.box, parts);
    TS_LAUNCH("k_down_clear", k_down_clear, sweep, block, parts, (int)n_parts, opt.box, max_words, reinterpret_cast<uint4 *>(words),
              reinterpret_cast<uint4 *>(m->d_sched), head, sl.dev);
    TS_LAUNCH("k_down_mark", k_down_mark, per_point, block, m->d_in_keys, N, head, reinterpret_cast<uint32_t *>(words));
    TS_LAUNCH("k_down_count", k_down_count, sweep, block, words, head, totals);
    TS_LAUNCH("k_down_expand", k_down_expand, sweep, block, words, reinterpret_cast<const int4 *>(totals), head, m->d_out_keys, word_base, reinterpret_cast<int4 *>(m->d_nbr), sl.dev);
    TS_LAUNCH("k_down_scatter", k_down_scatter, per_point, block, m->d_in_keys, N, head, words, word_base, m->d_nbr, m->d_parent);
    TS_LAUNCH("k_rows", (k_rows<8, false>), per_point, block, m->d_nbr, m->d_out_keys, N, &head->count, m->d_colbits, m->d_colbase, m->d_wavemask, (int64_t)0);
    TS_LAUNCH("k_scan", k_scan, dim3(m->K3 + 1), dim3(kScanThreads), m->d_colbase, (int64_t)0, sl.dev, m->K3, m->d_wavemask, (int64_t)0,
              m->d_tile_order, &head->count);
    m->n_out = -1;
    m->count_pending = true;
    m->one_pair_per_input = true;
    m->scan_enqueued = true;
    m->scan_done = false;
    sl.totals = true;
    m->stream = stream();
    sl.owner = m;
    m->pending_slot = slot;
    TS_HIP(hipGetLastError());
    return TS_OK;
}

// A strided build that the host takes part in: it waits for the box of the points where that is measured, and for
// the number of coarse points.  coords == NULL: `given` holds the keys already.  *reports is set once all that
// writes to the slot has been enqueued and the map owns it.
int build_strided(Temps &tmp, const int32_t *coords, uint64_t *given, int64_t N, ts_kmap *m, const BuildOpts &asked, int slot,
                  bool *reports) {
    BuildOpts opt = asked;   // a build that measures its bounding box may turn the grid on
    const bool wait = opt.wait;
    const int K = m->K, s = m->s, transposed = m->transposed;
    hipStream_t st = stream();
    int32_t *d_status = slot_at(slot).dev;
    FillArgs fill;
    Searched table;
    const dim3 per_point(blocks_for(N, kThreads)), block(kThreads);
    // coarse set: the distinct admissible candidates in ascending order (Alg. 3)
    const int A = (K + s - 1) / s, slots = A * A * A;
    const size_t n_cand = (size_t)N * slots;
    uint64_t *uniq;
    TS_TRY(tmp.get(&uniq, n_cand));
    const bool measure = coords && opt.measure && !opt.grid;
    int4 *parts = nullptr;
    if (measure) TS_TRY(tmp.get(&parts, 2 * kDownPack));
    Grid cbox = {};
    uint64_t *words = nullptr;
    int32_t *word_base = nullptr, *block_total = nullptr;
    int64_t n_words = 0, n_wblocks = 0;
    auto bitmap_over_box = [&]() -> int {
        // the coarse points lie in the box of the fine ones, moved by less than K and divided by s
        uint64_t cells = (uint64_t)opt.box.batches;
        for (int a = 0; a < 3; ++a) {
            cbox.lo[a] = floor_div(opt.box.lo[a] - K, s);
            cbox.ext[a] = (uint32_t)(floor_div(opt.box.hi[a] + K, s) - cbox.lo[a] + 1);
            cells *= cbox.ext[a];
            if (cells > kMaxGridCells)
                return fail(TS_ERR_UNSUPPORTED, "the grid bounds span more than %llu cells", (unsigned long long)kMaxGridCells);
        }
        cbox.batches = (uint32_t)opt.box.batches;
        n_words = (int64_t)((cells + 63) / 64);
        n_wblocks = (n_words + kThreads - 1) / kThreads;
        TS_TRY(tmp.get(&words, (size_t)n_words));
        TS_TRY(tmp.get(&word_base, (size_t)n_words));
        TS_TRY(tmp.get(&block_total, (size_t)n_wblocks));
        fill.add(words, (size_t)n_words * sizeof(uint64_t), 0u);
        return TS_OK;
    };
    // What the host needs on the way it reads off the status words too.  Copies and stream synchronisations instead cost
    // 30 us here (153 k points, 3x3x3 stride 2: 131 us and 101, with a boundary 144 and 115): behind a build that was waited
    // for by its words, of which the runtime knows nothing, they take longer still than by themselves (128 and 141).
    const int4 *c4 = reinterpret_cast<const int4 *>(coords);
    if (measure) {
        // one more host round trip buys a build without a sort and a search without collisions
        const unsigned n_parts = blocks_for(N, kThreads) < kDownPack ? blocks_for(N, kThreads) : kDownPack;
        TS_LAUNCH("k_down_pack", k_down_pack, dim3(n_parts), block, c4, N, given, d_status, opt.box, parts);
        TS_LAUNCH("k_tell_box", k_tell_box, dim3(1), block, parts, (int)n_parts, d_status);
        TS_TRY(slot_wait(slot, kBox));
        const volatile int32_t *top = slot_at(slot).host + ST_BOX;
        if (top[6] != INT32_MIN) {   // at least one valid point
            // the bitmap has one bit per cell of the box the outputs can lie in
            Box bx = {};
            uint64_t cells = (uint64_t)top[6] + 1;
            for (int a = 0; a < 3; ++a) {
                bx.lo[a] = -top[a];
                bx.hi[a] = top[3 + a];
                cells *= (uint64_t)((int64_t)floor_div(bx.hi[a] + K, s) - floor_div(bx.lo[a] - K, s) + 1);
                if (cells > kAutoGridCells) cells = kAutoGridCells + 1;
            }
            bx.batches = top[6] + 1;
            if (cells <= kAutoGridCells) {
                opt.grid = true;
                opt.box = bx;   // on stays 0: nothing to check, the box is the points' own
            }
        }
    } else if (coords) {
        TS_LAUNCH("k_pack", k_pack, per_point, block, c4, N, given, d_status, opt.box);
    }
    // the coarse points lie in the box of the fine ones, moved by less than K and divided by s
    int32_t clo[3] = {0, 0, 0}, chi[3] = {0, 0, 0};
    for (int a = 0; a < 3; ++a) {
        clo[a] = floor_div(opt.box.lo[a] - K, s);
        chi[a] = floor_div(opt.box.hi[a] + K, s);
    }
    const bool ranked = opt.grid;   // outputs found through the bitmap: the map follows without a search
    if (opt.grid) {
        // bounds are stated or measured: mark the candidates' cells in a bitmap and read the set bits
        // off in order, which sorts and removes duplicates at once
        TS_TRY(bitmap_over_box());
        TS_TRY(launch_fill(fill));
        fill = FillArgs();
        TS_LAUNCH("k_candidates_mark", k_candidates_mark, dim3(blocks_for(N, kThreads), slots), block, given, N, K, s, A, opt.bound,
                  cbox, reinterpret_cast<uint32_t *>(words), d_status);
        TS_LAUNCH("k_bits_count", k_bits_count, dim3((unsigned)n_wblocks), block, words, n_words, block_total);
        // up to a few thousand blocks every block sums the totals before it by itself; beyond, a scan launch
        const int self_scan = n_wblocks <= 8192;
        if (!self_scan) TS_LAUNCH("k_bits_scan", k_bits_scan, dim3(1), block, block_total, n_wblocks, d_status);
        TS_LAUNCH("k_bits_expand", k_bits_expand, dim3((unsigned)n_wblocks), block, words, n_words, block_total, cbox, uniq,
                  word_base, self_scan, d_status);
    } else {
        // candidates -> sort -> unique (the empty key, if present, sorts last)
        uint64_t *cand, *sorted;
        int64_t *d_count;
        TS_TRY(tmp.get(&d_count, 1));
        TS_TRY(tmp.get(&cand, n_cand));
        TS_TRY(tmp.get(&sorted, n_cand));
        TS_LAUNCH("k_candidates", k_candidates, dim3(blocks_for(N, kThreads), slots), block, given, N, K, s, A, opt.bound, cand);
        TS_TRY(sort_keys(tmp, cand, sorted, n_cand));
        size_t bytes = 0;
        TS_HIP(rocprim::unique(nullptr, bytes, sorted, uniq, d_count, n_cand, rocprim::equal_to<uint64_t>(), st));
        void *ws;
        TS_TRY(tmp.get((char **)&ws, bytes));
        {
            ProfScope ps("unique_keys");
            TS_HIP(rocprim::unique(ws, bytes, sorted, uniq, d_count, n_cand, rocprim::equal_to<uint64_t>(), st));
        }
        TS_LAUNCH("k_tell_count", k_tell_count, dim3(1), dim3(1), uniq, d_count, d_status);
    }
    TS_TRY(slot_wait(slot, kCount));
    const int64_t n_coarse = slot_at(slot).host[ST_COUNT];
    if (n_coarse == 0) {
        // No candidate passed the modular check (or every coordinate was out of range): a map
        // without pairs.  The inputs are still checked for duplicates and range.
        Table t0;
        TS_TRY(make_table(tmp, N, &t0, &fill));
        if (!transposed) {
            m->n_in = N;
            m->n_out = 0;
        } else {
            m->n_in = 0;
            m->n_out = N;
            m->d_in_keys = nullptr;
            m->d_out_keys = given;
            TS_TRY(alloc_outputs(m, &fill));
            fill.add(m->d_nbr, (size_t)N * m->stride * sizeof(int32_t), 0xFFFFFFFFu);
        }
        TS_TRY(launch_fill(fill));
        TS_LAUNCH("k_insert", k_insert<Table>, per_point, block, given, N, t0, d_status);
        if (transposed) {
            launch_rows(m);
            *reports = true;
            return finish(m, slot, true);
        }
        TS_HIP(hipStreamSynchronize(st));
        return take_verdict(m, slot_at(slot).host) == TS_OK ? TS_OK : report(m);
    }
    uint64_t *coarse;
    TS_TRY(alloc_n(&coarse, (size_t)n_coarse));
    TS_HIP(hipMemcpyAsync(coarse, uniq, (size_t)n_coarse * sizeof(uint64_t), hipMemcpyDeviceToDevice, st));
    if (ranked) {
        // No search: an input's admissible candidates are outputs, and an output's row number is the rank
        // of its cell among the marked ones (k_rank_scatter).  Neither hash table nor coordinate grid.
        const dim3 per_cand(blocks_for(N, kThreads), slots);
        if (!transposed) {
            m->n_in = N;
            m->n_out = n_coarse;
            m->d_out_keys = coarse;
        } else {
            m->n_in = n_coarse;
            m->n_out = N;
            m->d_in_keys = coarse;
            m->d_out_keys = given;
        }
        TS_TRY(alloc_outputs(m, &fill));
        fill.add(m->d_nbr, (size_t)m->n_out * m->stride * sizeof(int32_t), 0xFFFFFFFFu);
        if (!transposed && !opt.bound.on) {
            TS_TRY(launch_fill(fill));
            TS_LAUNCH("k_rank_scatter", k_rank_scatter<false>, per_cand, block, given, N, K, s, A, opt.bound, cbox, words, word_base,
                      m->d_nbr, m->stride, d_status);
        } else if (!transposed) {
            // with a boundary an input may lose all its candidates and then meets nobody in the table: equal
            // points are found through a hash table here as well
            Table fine_table;
            TS_TRY(make_table(tmp, N, &fine_table, &fill));
            TS_TRY(launch_fill(fill));
            TS_LAUNCH("k_insert", k_insert<Table>, per_point, block, given, N, fine_table, d_status);
            TS_LAUNCH("k_rank_scatter", k_rank_scatter<false>, per_cand, block, given, N, K, s, A, opt.bound, cbox, words, word_base,
                      m->d_nbr, m->stride, d_status);
        } else {
            // rows belong to the given points here, so equal points do not meet in an entry: they are found
            // by inserting the points into a hash table, which nothing else uses
            Table fine_table;
            TS_TRY(make_table(tmp, N, &fine_table, &fill));
            TS_TRY(launch_fill(fill));
            TS_LAUNCH("k_insert", k_insert<Table>, per_point, block, given, N, fine_table, d_status);
            TS_LAUNCH("k_rank_scatter", k_rank_scatter<true>, per_cand, block, given, N, K, s, A, opt.bound, cbox, words, word_base,
                      m->d_nbr, m->stride, d_status);
        }
        // where the next level's points can lie, for a caller that builds a pyramid
        if (!transposed) {
            m->out_box_batches = (int32_t)cbox.batches;
            for (int a = 0; a < 3; ++a) {
                m->out_box_lo[a] = cbox.lo[a];
                m->out_box_hi[a] = cbox.lo[a] + (int32_t)cbox.ext[a] - 1;
            }
        }
        launch_rows(m);
        *reports = true;
        return finish(m, slot, wait);
    }
    if (!transposed) {
        m->n_in = N;
        m->n_out = n_coarse;
        m->d_out_keys = coarse;
        TS_TRY(alloc_outputs(m, &fill));
        TS_TRY(make_searched(tmp, opt, N, opt.box.lo, opt.box.hi, &table, &fill));
        TS_TRY(launch_fill(fill));
        if (table.grid) TS_LAUNCH("k_insert_grid", k_insert<Grid>, per_point, block, given, N, table.g, d_status);
        else TS_LAUNCH("k_insert", k_insert<Table>, per_point, block, given, N, table.t, d_status);
    } else {
        m->n_in = n_coarse;
        m->n_out = N;
        m->d_in_keys = coarse;
        m->d_out_keys = given;
        TS_TRY(alloc_outputs(m, &fill));
        // duplicates among the fine points are found by inserting them as well
        Table fine_table;
        TS_TRY(make_table(tmp, N, &fine_table, &fill));
        TS_TRY(make_searched(tmp, opt, n_coarse, clo, chi, &table, &fill));
        TS_TRY(launch_fill(fill));
        TS_LAUNCH("k_insert", k_insert<Table>, per_point, block, given, N, fine_table, d_status);
        const dim3 per_coarse(blocks_for(n_coarse, kThreads));
        if (table.grid) TS_LAUNCH("k_insert_grid", k_insert<Grid>, per_coarse, block, coarse, n_coarse, table.g, d_status);
        else TS_LAUNCH("k_insert", k_insert<Table>, per_coarse, block, coarse, n_coarse, table.t, d_status);
    }
    TS_TRY(search(m, table, d_status));
    *reports = true;
    return finish(m, slot, wait);
}

int build(const int32_t *coords, int64_t N, int K, int s, int transposed, ts_kmap *m, const BuildOpts &asked) {
    const BuildOpts &opt = asked;
    const bool wait = opt.wait;
    Temps tmp;
    const int K3 = K * K * K;
    m->K = K;
    m->s = s;
    m->transposed = transposed;
    m->K3 = K3;
    m->stride = nbr_stride(K3);
    m->centre = (s == 1) ? (K3 - 1) / 2 : -1;
    if (N == 0) return TS_OK;

    uint64_t *given;   // keys of the caller's coordinates
    TS_TRY(alloc_n(&given, (size_t)N));
    m->d_in_keys = given;   // provisional owner, so that an early error frees it

    // where the build reports; a build that ends early gives the slot back once nothing can write to it any more
    struct SlotGuard {
        int slot;
        bool committed = false;
        ~SlotGuard() {
            if (slot >= 0 && !committed) {
                (void)hipStreamSynchronize(stream());
                slot_release(slot);
            }
        }
    } guard{slot_acquire(K3)};
    if (guard.slot < 0) return last_fail_code();
    const int slot = guard.slot;
    int32_t *d_status = slot_at(slot).dev;
    FillArgs fill;

    Searched table;
    const dim3 per_point(blocks_for(N, kThreads)), block(kThreads);
    if (s == 1) {
        m->n_in = m->n_out = N;
        m->d_out_keys = given;
        TS_TRY(alloc_outputs(m, &fill));
        const int4 *c4 = reinterpret_cast<const int4 *>(coords);
        if (K == 3 && !opt.grid) {
            TS_TRY(alloc_n(&m->d_rowmask, ((size_t)N + 3) & ~size_t(3)));   // what the map keeps comes before what the build can do without
            if (N <= kSmallPoints) {   // no table in memory, and nothing to clear
                int cap = 64;
                while (cap < 4 * N && cap < kSmallSlots) cap <<= 1;
                TS_LAUNCH("k_small_map", k_small_map, dim3(blocks_for(N, kSmallRows)), dim3(kSmallThreads), c4, (int)N, cap, given, m->d_nbr,
                          m->d_colbits, m->d_colbase, m->d_wavemask, m->n_blocks, m->d_rowmask, reinterpret_cast<uint4 *>(m->d_sched), d_status);
                guard.committed = true;
                return finish(m, slot, wait, true);
            }
            BlockTable bt;
            int32_t *counter = nullptr;
            TS_TRY(make_block_table(tmp, N, &bt, &counter, &fill));
            TS_TRY(launch_fill(fill));
#define TS_BLOCK_SEARCH(...) TS_LAUNCH("k_block_search", (k_block_search<__VA_ARGS__>), per_point, block, given, N, bt, m->d_nbr, m->d_colbits, m->d_colbase, m->d_wavemask, m->n_blocks, m->d_rowmask, d_status)
            if (bt.base) {   // (the points' slots stand where the search puts the bitmasks)
                TS_LAUNCH("k_block_insert", k_block_insert<true>, per_point, block, c4, N, given, bt, m->d_rowmask, d_status);
                TS_LAUNCH("k_block_base", k_block_base, dim3(blocks_for((int64_t)bt.mask + 1, kThreads * kBlockBasePer)), block, bt, counter);
                TS_LAUNCH("k_block_place", k_block_place, per_point, block, given, m->d_rowmask, N, bt);
                TS_BLOCK_SEARCH(true, uint32_t);
            } else {
                TS_LAUNCH("k_block_insert", k_block_insert<false>, per_point, block, c4, N, given, bt, nullptr, d_status);
                if (bt.mask >> 26 == 0) TS_BLOCK_SEARCH(false, uint32_t);
                else TS_BLOCK_SEARCH(false, uint64_t);
            }
#undef TS_BLOCK_SEARCH
            guard.committed = true;
            return finish(m, slot, wait, true);
        }
        TS_TRY(make_searched(tmp, opt, N, opt.box.lo, opt.box.hi, &table, &fill));
        TS_TRY(launch_fill(fill));
        int4 *rows = K == 3 ? reinterpret_cast<int4 *>(m->d_nbr) : nullptr;   // the symmetric probe of the grid writes hits only
        if (table.grid)
            TS_LAUNCH("k_pack_insert_grid", k_pack_insert<Grid>, per_point, block, c4, N, given, table.g, d_status, opt.box, rows);
        else
            TS_LAUNCH("k_pack_insert", k_pack_insert<Table>, per_point, block, c4, N, given, table.t, d_status, opt.box, rows);
        TS_TRY(search(m, table, d_status));
        guard.committed = true;
        return finish(m, slot, wait, m->rows_put_off);   // (9 us for 153 k points that a layer does not need)
    }
    if (K == 2 && s == 2 && !transposed && !opt.bound.on && (opt.grid || opt.measure)) {
        TS_TRY(build_down(tmp, coords, N, m, opt, slot));
        guard.committed = true;
        return wait ? resolve(m) : TS_OK;
    }
    return build_strided(tmp, coords, given, N, m, opt, slot, &guard.committed);
}

}  // namespace

namespace {

// The transposed map of a forward strided map, derived from its neighbour table: no search, and no
// host round trip either, because the sizes are those of the forward map.
int transpose(const ts_kmap *f, ts_kmap *m) {
    hipStream_t st = stream();
    Temps tmp;
    const int K3 = f->K3;
    m->K = f->K;
    m->s = f->s;
    m->transposed = 1;
    m->K3 = K3;
    m->centre = -1;
    m->n_in = f->n_out;
    m->n_out = f->n_in;
    m->M = f->M;
    for (int n = 0; n < K3; ++n) m->sizes[n] = f->sizes[n];
    for (int n = 0; n <= K3; ++n) m->offs[n] = f->offs[n];
    if (m->n_out == 0) return TS_OK;
    TS_TRY(alloc_n(&m->d_in_keys, (size_t)m->n_in));
    TS_TRY(alloc_n(&m->d_out_keys, (size_t)m->n_out));
    if (f->d_parent) {
        int32_t *sizes;   // written by the scan, known already
        TS_TRY(tmp.get(&sizes, ST_WORDS));
        TS_TRY(alloc_outputs(m, nullptr));
        if (alloc_n(&m->d_window_perm, (size_t)m->n_tiles * kTileRows) != TS_OK) m->d_window_perm = nullptr;   // the natural order then
        m->window_settled = true;   // whoever may read the map's rows may read their order
        TS_LAUNCH("k_up_rows", k_up_rows, dim3(blocks_for(m->n_out, kUpRows)), dim3(kUpThreads), f->d_in_keys, f->d_parent, m->n_out,
                  f->d_out_keys, m->n_in, m->d_out_keys, m->d_in_keys, m->d_nbr, m->d_colbits, m->d_colbase, m->d_wavemask, m->n_blocks,
                  reinterpret_cast<uint4 *>(m->d_sched), m->d_window_perm);
        launch_scan(m, sizes);
        TS_HIP(hipGetLastError());
        return TS_OK;
    }
    if (m->n_in > 0) TS_HIP(hipMemcpyAsync(m->d_in_keys, f->d_out_keys, (size_t)m->n_in * sizeof(uint64_t), hipMemcpyDeviceToDevice, st));
    TS_HIP(hipMemcpyAsync(m->d_out_keys, f->d_in_keys, (size_t)m->n_out * sizeof(uint64_t), hipMemcpyDeviceToDevice, st));
    FillArgs fill;
    int32_t *sizes;   // written by the scan, known already
    TS_TRY(tmp.get(&sizes, ST_WORDS));
    TS_TRY(alloc_outputs(m, &fill));
    fill.add(m->d_nbr, (size_t)m->n_out * m->stride * sizeof(int32_t), 0xFFFFFFFFu);
    TS_TRY(launch_fill(fill));
    if (f->n_out > 0) {
        const dim3 gf(blocks_for(f->n_out, kThreads)), block(kThreads);
        if (K3 == 27) TS_LAUNCH("k_transpose", k_transpose<27>, gf, block, f->d_nbr, f->n_out, m->d_nbr);
        else if (K3 == 8) TS_LAUNCH("k_transpose", k_transpose<8>, gf, block, f->d_nbr, f->n_out, m->d_nbr);
        else TS_LAUNCH("k_transpose", k_transpose<1>, gf, block, f->d_nbr, f->n_out, m->d_nbr);
    }
    launch_rows(m);
    launch_scan(m, sizes);
    TS_HIP(hipGetLastError());
    return TS_OK;
}

}  // namespace

namespace ts {

// The number of outputs of a map whose build left it to be read here (build_down).  A box too large for the bitmap
// ends in a build by sorting, from the keys.  That runs on the stream that is current now, while the caller orders his
// work by the stream he built the map on: it is waited for (the host takes part in it twice anyway).
int resolve_count(const ts_kmap *kmap, bool may_build) {
    ts_kmap *m = const_cast<ts_kmap *>(kmap);
    if (!m->count_pending) return m->n_out >= 0 ? TS_OK : fail(m->error, "the build of this map failed after its outputs had been asked for");
    const int slot = m->pending_slot;
    TS_TRY(slot_wait(slot, kCount));
    int32_t *h = slot_at(slot).host;
    if (h[ST_COUNT] >= 0) {
        m->n_out = h[ST_COUNT];
        m->n_blocks = (m->n_out + 63) / 64;
        m->n_tiles = (m->n_out + kTileRows - 1) / kTileRows;
        m->out_box_batches = h[ST_BOX + 6];
        for (int a = 0; a < 3; ++a) {
            m->out_box_lo[a] = h[ST_BOX + a];
            m->out_box_hi[a] = h[ST_BOX + 3 + a];
        }
        m->count_pending = false;
        return TS_OK;
    }
    if (!may_build)
        return fail(TS_ERR_UNSUPPORTED, "the box of this map's points is too large for a bitmap: building it needs memory, which this call must not take; ask ts_kmap_num_out first");
    if (stream_capturing(stream()))
        return fail(TS_ERR_UNSUPPORTED, "the box of this map's points is too large for a bitmap: its number of outputs must have been asked for before the stream is captured");
    TS_TRY(slot_wait(slot, kSizes));   // nothing more is written there
    TS_HIP(hipStreamSynchronize(stream()));
    for (int n = 0; n < kMaxK3; ++n) h[ST_TOTALS + n] = -1;
    h[ST_TILES] = 0;
    h[ST_COUNT] = -1;
    slot_at(slot).totals = false;
    m->count_pending = m->one_pair_per_input = m->scan_enqueued = false;
    for (void *p : {(void *)m->d_nbr, (void *)m->d_colbits, (void *)m->d_colbase, (void *)m->d_tile_order, (void *)m->d_wavemask,
                    (void *)m->d_sched, (void *)m->d_parent, (void *)m->d_out_keys})
        dev_free(p);
    m->d_nbr = m->d_colbase = m->d_tile_order = m->d_sched = m->d_parent = nullptr;
    m->d_colbits = m->d_out_keys = nullptr;
    m->d_wavemask = nullptr;
    Temps tmp;
    BuildOpts opt;
    opt.wait = false;
    bool reports = false;
    int rc = build_strided(tmp, nullptr, m->d_in_keys, m->n_in, m, opt, slot, &reports);
    if (rc == TS_OK && reports) rc = slot_wait(slot, kSizes);
    if (rc != TS_OK || !reports) {
        (void)hipStreamSynchronize(stream());
        slot_release(slot);
        m->pending_slot = -1;
    }
    if (rc != TS_OK) {
        m->n_out = -1;
        m->error = rc;
    }
    return rc;
}

// The host waits for a stream that is not the current one (which may be being captured).
static int wait_for(hipStream_t other) {
    if (stream_capturing(other))
        return fail(TS_ERR_UNSUPPORTED, "a map's build must have finished before its stream is captured and the map is used on another one");
    const bool capturing = stream_capturing(stream());
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    if (capturing) TS_HIP(hipThreadExchangeStreamCaptureMode(&mode));
    hipError_t e = hipStreamSynchronize(other);
    if (e != hipSuccess) {   // e.g. a stream that no longer exists
        (void)hipGetLastError();
        e = hipDeviceSynchronize();
    }
    if (capturing) TS_HIP(hipThreadExchangeStreamCaptureMode(&mode));
    return e == hipSuccess ? TS_OK : fail(TS_ERR_HIP, "waiting for a map build: %s", hipGetErrorString(e));
}

int settle(const ts_kmap *kmap) {
    if (!kmap->verdict_only || kmap->stream == stream()) return TS_OK;
    TS_TRY(wait_for(kmap->stream));
    const_cast<ts_kmap *>(kmap)->verdict_only = false;
    return TS_OK;
}

int resolve(const ts_kmap *kmap, bool need_sizes) {
    ts_kmap *m = const_cast<ts_kmap *>(kmap);
    TS_TRY(resolve_count(m));
    if (m->pending_slot >= 0) {
        const int slot = m->pending_slot;
        if (need_sizes && !m->scan_enqueued) {
            if (stream_capturing(stream()))
                return fail(TS_ERR_UNSUPPORTED, "the sizes of a map must have been asked for, or ts_kmap_prepare called, before the stream is captured");
            if (m->stream != stream()) TS_TRY(wait_for(m->stream));   // the scan reads what the search leaves
            TS_TRY(prepare(m));
        }
        const bool totals = m->scan_enqueued;
        TS_TRY(slot_wait(slot, totals ? kSizes : kVerdict));
        if (totals) {
            take_status(m, slot_at(slot).host);
            m->scan_done = true;
        } else {
            take_verdict(m, slot_at(slot).host);
        }
        m->verdict_only = !totals;
        if (totals || m->error != TS_OK) {   // else the slot stays for the sizes
            slot_release(slot);
            m->pending_slot = -1;
        }
    }
    return m->error == TS_OK ? TS_OK : report(m);
}

void release_grid() {
    if (g_grid) (void)hipFree(g_grid);
    g_grid = nullptr;
    g_grid_cells = 0;
    g_grid_dirty = false;
}

// The scan that an asynchronous 3x3x3 stride-1 build put off, enqueued without a wait: its sizes land in the
// words that the build's verdict goes to.
int prepare(const ts_kmap *kmap) {
    ts_kmap *m = const_cast<ts_kmap *>(kmap);
    if (m->scan_done || m->scan_enqueued || m->pending_slot < 0) return TS_OK;   // nothing put off
    TS_TRY(settle(m));
    StatusSlot &sl = slot_at(m->pending_slot);
    if (m->rows_put_off) launch_rows(m);
    m->rows_put_off = false;
    slot_recorded(sl);
    launch_scan(m, sl.dev);
    sl.totals = true;
    m->scan_enqueued = true;
    m->stream = stream();
    TS_HIP(hipGetLastError());
    return TS_OK;
}

void order_windows(const ts_kmap *kmap) {
    ts_kmap *m = const_cast<ts_kmap *>(kmap);
    const bool up = goes_up_by_two(m);
    if (!(m->d_rowmask || up) || m->d_window_perm || m->d_perm || m->n_out == 0 || stream_capturing(stream())) return;
    if (alloc_n(&m->d_window_perm, (size_t)m->n_tiles * kTileRows) != TS_OK) return;
    if (up) TS_LAUNCH("k_up_order", k_up_order, dim3(blocks_for(m->n_out, kUpRows)), dim3(kUpThreads), m->d_nbr, m->n_out, m->d_window_perm);
    else TS_LAUNCH("k_window_sort", k_window_sort, dim3(blocks_for(m->n_out, kWindowRows)), dim3(kWindowThreads), m->d_rowmask, m->n_out, m->d_window_perm);
    m->window_stream = stream();
}

// Asked of the stream itself: an event recorded behind the ordering made the first layer 7 us longer.
const int32_t *row_order(const ts_kmap *kmap) {
    if (kmap->d_perm) return kmap->d_perm;
    if (!kmap->d_window_perm || kmap->window_settled || kmap->window_stream == stream()) return kmap->d_window_perm;
    if (stream_capturing(kmap->window_stream)) return nullptr;   // asking would end the capture
    const bool capturing = stream_capturing(stream());
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;   // the question is about a stream outside the capture
    if (capturing && hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) return nullptr;
    const hipError_t e = hipStreamQuery(kmap->window_stream);
    if (e != hipSuccess) (void)hipGetLastError();
    if (capturing) (void)hipThreadExchangeStreamCaptureMode(&mode);
    if (e != hipSuccess) return nullptr;
    const_cast<ts_kmap *>(kmap)->window_settled = true;
    return kmap->d_window_perm;
}

Offs offs_of(const ts_kmap *kmap) {
    Offs o;
    for (int n = 0; n <= kMaxK3; ++n) o.v[n] = n <= kmap->K3 ? (int32_t)kmap->offs[n] : (int32_t)kmap->offs[kmap->K3];
    return o;
}

// The offset-major pair lists are derived from the out-major table when something first asks for
// them (ts_kmap_pairs, the gather of the explicit dataflow); the fused kernel never does.
static int make_pairs(const ts_kmap *kmap, int32_t *in_copy, int32_t *out_copy, bool *copied) {
    ts_kmap *m = const_cast<ts_kmap *>(kmap);
    *copied = false;
    TS_TRY(resolve(m));
    if (m->d_in_idx || m->M == 0) return TS_OK;
    int32_t *in_idx, *out_idx;
    TS_TRY(alloc_n(&in_idx, (size_t)m->M));
    if (alloc_n(&out_idx, (size_t)m->M) != TS_OK) {
        dev_free(in_idx);
        return TS_ERR_OOM;
    }
    const dim3 grid(blocks_for(m->n_out, kThreads)), block(kThreads);
    if (m->K3 == 27) TS_LAUNCH("k_compact", k_compact<27>, grid, block, m->d_nbr, m->n_out, m->d_colbase, m->n_blocks, offs_of(m), in_idx, out_idx, in_copy, out_copy);
    else if (m->K3 == 8) TS_LAUNCH("k_compact", k_compact<8>, grid, block, m->d_nbr, m->n_out, m->d_colbase, m->n_blocks, offs_of(m), in_idx, out_idx, in_copy, out_copy);
    else TS_LAUNCH("k_compact", k_compact<1>, grid, block, m->d_nbr, m->n_out, m->d_colbase, m->n_blocks, offs_of(m), in_idx, out_idx, in_copy, out_copy);
    m->d_in_idx = in_idx;
    m->d_out_idx = out_idx;
    *copied = true;
    TS_HIP(hipGetLastError());
    return TS_OK;
}

int ensure_pairs(const ts_kmap *kmap) {
    bool copied;
    return make_pairs(kmap, nullptr, nullptr, &copied);
}

}  // namespace ts

extern "C" {

static int build_checked(const int32_t *coords, int64_t N, int kernel_size, int stride, int transposed, ts_kmap **out_kmap,
                         const BuildOpts &opt) {
    if (!out_kmap) return fail(TS_ERR_INVALID_ARG, "out_kmap is NULL");
    *out_kmap = nullptr;
    if (N < 0) return fail(TS_ERR_INVALID_ARG, "N is negative");
    if (N > 0 && !coords) return fail(TS_ERR_INVALID_ARG, "coords is NULL");
    if (N > 0 && (reinterpret_cast<uintptr_t>(coords) & 15)) return fail(TS_ERR_INVALID_ARG, "coords must be 16-byte aligned");
    if (kernel_size < 1 || kernel_size > 3) return fail(TS_ERR_INVALID_ARG, "kernel_size must be 1, 2 or 3");
    if (stride < 1 || stride > 2) return fail(TS_ERR_INVALID_ARG, "stride must be 1 or 2");
    if (stride == 1 && kernel_size % 2 == 0) return fail(TS_ERR_INVALID_ARG, "stride 1 needs an odd kernel_size");
    if (transposed != 0 && transposed != 1) return fail(TS_ERR_INVALID_ARG, "transposed must be 0 or 1");
    if (transposed && stride == 1) return fail(TS_ERR_INVALID_ARG, "a transposed map needs stride > 1");
    if (N > (int64_t)((1u << 31) - 1) / (ts::kMaxK3 + 5)) return fail(TS_ERR_UNSUPPORTED, "N too large for 32-bit pair indices");
    ts_kmap *m = new (std::nothrow) ts_kmap();
    if (!m) return fail(TS_ERR_OOM, "host allocation failed");
    int rc = build(coords, N, kernel_size, stride, transposed, m, opt);
    if (rc != TS_OK) {
        (void)hipStreamSynchronize(ts::stream());
        destroy(m);
        return rc;
    }
    *out_kmap = m;
    return TS_OK;
}

int ts_build_kmap(const int32_t *coords, int64_t N, int kernel_size, int stride, int transposed,
                  ts_kmap **out_kmap) {
    BuildOpts opt;
    opt.measure = true;
    return build_checked(coords, N, kernel_size, stride, transposed, out_kmap, opt);
}

int ts_build_kmap_async(const int32_t *coords, int64_t N, int kernel_size, int stride, int transposed,
                        ts_kmap **out_kmap) {
    BuildOpts opt;
    opt.wait = false;
    opt.measure = true;
    return build_checked(coords, N, kernel_size, stride, transposed, out_kmap, opt);
}

int ts_identity_kmap(int64_t n, ts_kmap **out_kmap) {
    if (!out_kmap) return fail(TS_ERR_INVALID_ARG, "out_kmap is NULL");
    *out_kmap = nullptr;
    if (n < 0 || n > INT32_MAX) return fail(TS_ERR_INVALID_ARG, "n must be in [0, 2^31)");
    ts_kmap *m = new (std::nothrow) ts_kmap();
    if (!m) return fail(TS_ERR_OOM, "host allocation failed");
    m->K = 1;
    m->s = 1;
    m->K3 = 1;
    m->centre = 0;
    m->stride = ts::nbr_stride(1);
    m->n_in = m->n_out = m->M = n;
    m->sizes[0] = n;
    m->offs[1] = n;
    auto body = [&]() -> int {
        if (n == 0) return TS_OK;
        TS_TRY(alloc_outputs(m, nullptr));
        TS_LAUNCH("k_identity_map", k_identity_map, dim3(blocks_for(n, kThreads)), dim3(kThreads), m->d_nbr, m->stride,
                  m->d_colbits, m->d_colbase, m->d_tile_order, n, m->n_blocks, m->n_tiles, reinterpret_cast<uint4 *>(m->d_sched));
        TS_HIP(hipGetLastError());
        return TS_OK;
    };
    const int rc = body();
    if (rc != TS_OK) {
        (void)hipStreamSynchronize(ts::stream());
        destroy(m);
        return rc;
    }
    *out_kmap = m;
    return TS_OK;
}

int ts_build_kmap_ex(const int32_t *coords, int64_t N, int kernel_size, int stride, int transposed,
                     const ts_kmap_options *options, ts_kmap **out_kmap) {
    BuildOpts opt;
    opt.measure = true;
    if (out_kmap) *out_kmap = nullptr;
    if (options) {
        opt.wait = options->wait != 0;
        opt.measure = options->search == TS_SEARCH_AUTO;
        if (options->search != TS_SEARCH_HASH && options->search != TS_SEARCH_GRID && options->search != TS_SEARCH_AUTO)
            return fail(TS_ERR_INVALID_ARG, "search must be TS_SEARCH_AUTO, TS_SEARCH_HASH or TS_SEARCH_GRID");
        // TS_SEARCH_AUTO with a box stated (grid_batches > 0): a strided build takes the box instead of measuring
        // one (one host round trip less); a stride-1 build stays on the hash table and ignores it
        const bool hinted = options->search == TS_SEARCH_AUTO && options->grid_batches > 0 && stride > 1;
        if (options->search == TS_SEARCH_GRID || hinted) {
            opt.grid = true;
            opt.box.on = 1;
            opt.box.batches = options->grid_batches;
            if (options->grid_batches < 1 || options->grid_batches > TS_BATCH_MAX + 1)
                return fail(TS_ERR_INVALID_ARG, "grid_batches must be in [1, %d]", TS_BATCH_MAX + 1);
            for (int a = 0; a < 3; ++a) {
                opt.box.lo[a] = options->grid_lo[a];
                opt.box.hi[a] = options->grid_hi[a];
                if (options->grid_lo[a] > options->grid_hi[a] || options->grid_lo[a] < TS_COORD_MIN || options->grid_hi[a] > TS_COORD_MAX)
                    return fail(TS_ERR_INVALID_ARG, "grid bounds must satisfy %d <= lo <= hi <= %d", TS_COORD_MIN, TS_COORD_MAX);
            }
        }
        if (options->has_boundary && stride > 1) {
            opt.bound.on = 1;
            for (int a = 0; a < 3; ++a) {
                if (options->boundary[a] < 1 || (int64_t)options->boundary[a] * stride > (int64_t)TS_COORD_MAX + 1)
                    return fail(TS_ERR_INVALID_ARG, "boundary must be positive and stride * boundary at most %d", TS_COORD_MAX + 1);
                opt.bound.hi[a] = options->boundary[a] * stride;
            }
        }
    }
    return build_checked(coords, N, kernel_size, stride, transposed, out_kmap, opt);
}

int ts_kmap_status(const ts_kmap *kmap) {
    if (!kmap) return fail(TS_ERR_INVALID_ARG, "kmap is NULL");
    return ts::resolve(kmap, false);   // the verdict only: what a build put off stays put off
}

int ts_kmap_prepare(const ts_kmap *kmap) {
    if (!kmap) return fail(TS_ERR_INVALID_ARG, "kmap is NULL");
    return ts::prepare(kmap);
}

void ts_free(ts_kmap *kmap) { destroy(kmap); }

int ts_kmap_transpose(const ts_kmap *forward, ts_kmap **out_kmap) {
    if (!out_kmap) return fail(TS_ERR_INVALID_ARG, "out_kmap is NULL");
    *out_kmap = nullptr;
    if (!forward) return fail(TS_ERR_INVALID_ARG, "forward is NULL");
    if (forward->s == 1 || forward->transposed) return fail(TS_ERR_INVALID_ARG, "a forward map with stride > 1 is needed");
    TS_TRY(ts::resolve(forward));
    ts_kmap *m = new (std::nothrow) ts_kmap();
    if (!m) return fail(TS_ERR_OOM, "host allocation failed");
    int rc = transpose(forward, m);
    if (rc != TS_OK) {
        (void)hipStreamSynchronize(ts::stream());
        destroy(m);
        return rc;
    }
    *out_kmap = m;
    return TS_OK;
}

int ts_kmap_sort_rows(ts_kmap *kmap) {
    if (!kmap) return fail(TS_ERR_INVALID_ARG, "kmap is NULL");
    TS_TRY(ts::resolve(kmap));
    if (kmap->d_perm || kmap->n_out == 0) return TS_OK;
    return sort_rows(kmap);
}

int64_t ts_kmap_num_in(const ts_kmap *kmap) { return kmap ? kmap->n_in : -1; }
int64_t ts_kmap_num_out(const ts_kmap *kmap) {
    if (!kmap) return fail(TS_ERR_INVALID_ARG, "kmap is NULL");
    const int rc = ts::resolve_count(kmap);
    return rc == TS_OK ? kmap->n_out : rc;
}
int64_t ts_kmap_num_pairs(const ts_kmap *kmap) { return kmap && ts::resolve(kmap) == TS_OK ? kmap->M : -1; }
int ts_kmap_kernel_volume(const ts_kmap *kmap) { return kmap ? kmap->K3 : -1; }

int ts_kmap_out_coords(const ts_kmap *kmap, int32_t *dst) {
    if (!kmap) return fail(TS_ERR_INVALID_ARG, "kmap is NULL");
    TS_TRY(ts::resolve_count(kmap));
    if (kmap->n_out == 0) return TS_OK;
    if (!kmap->d_out_keys) return fail(TS_ERR_UNSUPPORTED, "a map made by ts_identity_kmap holds no coordinates");
    if (!dst || (reinterpret_cast<uintptr_t>(dst) & 15)) return fail(TS_ERR_INVALID_ARG, "dst is NULL or not 16-byte aligned");
    TS_LAUNCH("k_unpack", k_unpack, dim3(blocks_for(kmap->n_out, kThreads)), dim3(kThreads), kmap->d_out_keys, kmap->n_out, reinterpret_cast<int4 *>(dst));
    TS_HIP(hipGetLastError());
    return TS_OK;
}

int ts_kmap_out_box(const ts_kmap *kmap, int32_t *lo, int32_t *hi, int32_t *batches) {
    if (!kmap || !lo || !hi || !batches) return fail(TS_ERR_INVALID_ARG, "NULL argument");
    TS_TRY(ts::resolve_count(kmap));
    if (kmap->out_box_batches <= 0) return fail(TS_ERR_UNSUPPORTED, "this map's build did not bound its output coordinates");
    for (int a = 0; a < 3; ++a) {
        lo[a] = kmap->out_box_lo[a];
        hi[a] = kmap->out_box_hi[a];
    }
    *batches = kmap->out_box_batches;
    return TS_OK;
}

int ts_kmap_in_coords(const ts_kmap *kmap, int32_t *dst) {
    if (!kmap) return fail(TS_ERR_INVALID_ARG, "kmap is NULL");
    if (kmap->n_in == 0) return TS_OK;
    if (!kmap->d_in_keys) return fail(TS_ERR_UNSUPPORTED, "a map made by ts_identity_kmap holds no coordinates");
    if (!dst || (reinterpret_cast<uintptr_t>(dst) & 15)) return fail(TS_ERR_INVALID_ARG, "dst is NULL or not 16-byte aligned");
    TS_LAUNCH("k_unpack", k_unpack, dim3(blocks_for(kmap->n_in, kThreads)), dim3(kThreads), kmap->d_in_keys, kmap->n_in, reinterpret_cast<int4 *>(dst));
    TS_HIP(hipGetLastError());
    return TS_OK;
}

int ts_kmap_sizes(const ts_kmap *kmap, int64_t *dst) {
    if (!kmap || !dst) return fail(TS_ERR_INVALID_ARG, "NULL argument");
    TS_TRY(ts::resolve(kmap));
    for (int n = 0; n < kmap->K3; ++n) dst[n] = kmap->sizes[n];
    return TS_OK;
}

int ts_kmap_pairs(const ts_kmap *kmap, int32_t *in_idx, int32_t *out_idx) {
    if (!kmap) return fail(TS_ERR_INVALID_ARG, "kmap is NULL");
    TS_TRY(ts::resolve(kmap));
    if (kmap->M == 0) return TS_OK;
    bool copied;   // the caller's lists were written along with the map's own
    TS_TRY(ts::make_pairs(kmap, in_idx, out_idx, &copied));
    if (copied) return TS_OK;
    size_t bytes = (size_t)kmap->M * sizeof(int32_t);
    if (in_idx) TS_HIP(hipMemcpyAsync(in_idx, kmap->d_in_idx, bytes, hipMemcpyDeviceToDevice, ts::stream()));
    if (out_idx) TS_HIP(hipMemcpyAsync(out_idx, kmap->d_out_idx, bytes, hipMemcpyDeviceToDevice, ts::stream()));
    return TS_OK;
}

}  // extern "C"
