// Index-grid build on the GPU (Sec. 3.3) and the grid queries (Listing 1).
//
// The paper orders the voxels with two radix sorts (tile key a, then key b) and derives the
// nodes from runs of equal key prefixes.  Here the tree does the ordering itself: every level
// keeps a child bitmask, set bit by bit (the paper's "register ... into its parent" steps
// 11.1-11.4), and a popcount prefix scan over the masks numbers the children in exactly the
// order the sorts would give (bit order of a mask = Listing 2's offset order; node order =
// parent order).  Only the few root tiles are ranked by comparison.  One streaming pass over
// ijk collects the distinct leaves and their voxel masks in a hash table; the levels above are
// built from those leaves (tens of thousands) instead of from the voxels (millions).
#include <cmath>

#include "common.h"
#include "tree_device.h"

#include <string.h>

#include <algorithm>
#include <new>
#include <vector>

namespace fx {

// ---------------------------------------------------------------------------------- helpers
struct GridPtrs {
    GridHeader* hdr;
    int64_t* vox_base;
    uint64_t* root_key;
    int32_t* root_batch;
    uint64_t* upper_mask;
    uint32_t* upper_prefix;
    uint64_t* lower_mask;
    uint32_t* lower_prefix;
    fx_leaf* leaf;
    int32_t cap_upper, cap_lower, cap_leaf, B;
};

// Row ranges of the grids of a batch, as the build's kernels take them: up to eight grids travel in the kernel
// arguments (no upload, no dependent load per row), more in a device array of (begin, end) pairs.
constexpr int kInlineRanges = 8;
struct BatchRanges {
    const int64_t* d;
    int64_t begin[kInlineRanges], end[kInlineRanges];
};

// grid that owns row r (ranges sorted, non-overlapping), or -1
__device__ __forceinline__ int find_batch(const BatchRanges& J, int B, int64_t r) {
    if (B <= kInlineRanges) {
        int b = -1;
#pragma unroll
        for (int q = 0; q < kInlineRanges; ++q)
            if (q < B && r >= J.begin[q] && r < J.end[q]) b = q;
        return b;
    }
    const int64_t* __restrict__ joff = J.d;
    int lo = 0, hi = B;  // last b with start_b <= r
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (joff[2 * mid] <= r) lo = mid + 1; else hi = mid;
    }
    int b = lo - 1;
    if (b < 0 || r >= joff[2 * b + 1]) return -1;
    return b;
}

// What the build's rows are: voxel coordinates, or points that are turned into the cells they lie in as they are read
// (by the one row pass; a pass of its own that writes the cells cost 85 us for 10 M points).
struct RowSource {
    const int32_t* ijk;
    const float* xyz;          // kPoints only
    float o[3], s[3], inv_s[3];
};

// Cell of a coordinate.  Subtraction and division are the correctly rounded single-precision ones (no reciprocal, no
// contraction), so that the cell of a point near a face is the same on every implementation.  The division itself is only made
// where it decides: the quotient times the rounded reciprocal is within 2^-22 of it (three roundings of 2^-24 and the
// quotient's own), and unless a face lies within 2^-21 of its size both have the same floor.
__device__ __forceinline__ int cell_of(float x, float o, float s, float inv_s, int& bad) {
    const float d = __fsub_rn(x, o), near = __fmul_rn(d, inv_s), reach = __fmul_rn(fabsf(near), 4.76837158203125e-7f);
    float t = floorf(near);
    const float above = __fsub_rn(near, t);
    if (!(above > reach && __fsub_rn(1.0f, above) > reach)) t = floorf(__fdiv_rn(d, s));     // NaN and infinities too
    const bool ok = t >= -1073741824.0f && t < 1073741824.0f;
    bad += ok ? 0 : 1;
    return ok ? (int32_t)t : 0;
}

template <bool kPoints>
__device__ __forceinline__ int3 row_from_words(const RowSource& R, uint32_t w0, uint32_t w1, uint32_t w2, int& bad) {
    if (!kPoints) return make_int3((int)w0, (int)w1, (int)w2);
    return make_int3(cell_of(__uint_as_float(w0), R.o[0], R.s[0], R.inv_s[0], bad), cell_of(__uint_as_float(w1), R.o[1], R.s[1], R.inv_s[1], bad),
                     cell_of(__uint_as_float(w2), R.o[2], R.s[2], R.inv_s[2], bad));
}

template <bool kPoints>
__device__ __forceinline__ int3 load_row(const RowSource& R, int64_t r, int& bad) {
    const uint32_t* p = (kPoints ? reinterpret_cast<const uint32_t*>(R.xyz) : reinterpret_cast<const uint32_t*>(R.ijk)) + 3 * r;
    return row_from_words<kPoints>(R, p[0], p[1], p[2], bad);
}

// Four consecutive rows starting at r in three 16-byte loads (the tail row by row); returns how many exist.
typedef __attribute__((ext_vector_type(4), aligned(4))) uint32_t u32x4_u;
template <bool kPoints>
__device__ __forceinline__ int load_four_rows(const RowSource& R, int64_t n_rows, int64_t r, int3 (&v)[4], int& bad) {
    const uint32_t* p = (kPoints ? reinterpret_cast<const uint32_t*>(R.xyz) : reinterpret_cast<const uint32_t*>(R.ijk)) + 3 * r;
    if (r + 4 <= n_rows) {
        const u32x4_u a = *reinterpret_cast<const u32x4_u*>(p), b = *reinterpret_cast<const u32x4_u*>(p + 4),
                      c = *reinterpret_cast<const u32x4_u*>(p + 8);
        v[0] = row_from_words<kPoints>(R, a.x, a.y, a.z, bad);
        v[1] = row_from_words<kPoints>(R, a.w, b.x, b.y, bad);
        v[2] = row_from_words<kPoints>(R, b.z, b.w, c.x, bad);
        v[3] = row_from_words<kPoints>(R, c.y, c.z, c.w, bad);
        return 4;
    }
    const int n = r < n_rows ? (int)(n_rows - r) : 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = q < n ? load_row<kPoints>(R, r + q, bad) : make_int3(0, 0, 0);
    return n;
}

__device__ __forceinline__ uint32_t mix32(uint32_t h, uint32_t v) {
    h ^= v;
    h *= 0x9E3779B1u;
    h ^= h >> 15;
    return h;
}

// ---------------------------------------------------------------------------------- block scan
constexpr int kScanThreads = 1024;
constexpr int kWordsPerThread = 4;
constexpr int kWordChunk = kScanThreads * kWordsPerThread;  // mask words per block
constexpr int kLeavesPerThread = 1;
constexpr int kLeafChunk = kScanThreads * kLeavesPerThread;

// exclusive scan of one value per thread over a 1024-thread block; returns the block total
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* total) {
    __shared__ uint32_t wave_sums[kScanThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t incl = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        uint32_t o = __shfl_up(incl, d);
        if (lane >= d) incl += o;
    }
    if (lane == 63) wave_sums[wave] = incl;
    __syncthreads();
    if (wave == 0) {
        uint32_t s = lane < kScanThreads / 64 ? wave_sums[lane] : 0;
#pragma unroll
        for (int d = 1; d < kScanThreads / 64; d <<= 1) {
            uint32_t o = __shfl_up(s, d);
            if (lane >= d) s += o;
        }
        if (lane < kScanThreads / 64) wave_sums[lane] = s;  // inclusive over waves
    }
    __syncthreads();
    const uint32_t wave_base = wave ? wave_sums[wave - 1] : 0;
    *total = wave_sums[kScanThreads / 64 - 1];
    __syncthreads();
    return wave_base + incl - v;
}

// ---------------------------------------------------------------------------------- voxels -> leaves
// The input rows are reduced to the set of distinct (grid, leaf) pairs, each with the 512-bit
// mask of its voxels (step 11.4; duplicates collapse in the bit).  Everything above the leaves
// -- root tiles, upper and lower nodes, the order of the leaves -- is derived afterwards from
// these few leaves instead of from the rows.  Two ways to get there:
//   * partitioned (large inputs): the rows are first scattered into buckets by a hash of their
//     leaf, so that all voxels of a leaf meet in one workgroup, which then builds the masks
//     of its bucket in LDS -- no global atomic per voxel (device-scope atomics run at memory,
//     about 13 G/s on this part, and would cost more than the rest of the build together);
//   * direct (small inputs, or when a bucket holds more leaves than its LDS table): one global
//     open-addressing table, one compare-and-swap per new leaf and one atomic OR per voxel.
struct LeafList {
    int4* key;           // [cap] (leaf i, leaf j, leaf k, grid): leaf coordinates = voxel coordinates >> 3
    int32_t* mask_idx;   // [cap] where the leaf's mask sits in `mask` (units of 8 words)
    int32_t* node;       // [cap] the leaf's upper node, from the launch that numbers the lower ones on its lower node (-1: none)
    uint64_t* mask;
    int32_t cap;
};

// Positions for the items of one workgroup in the list: rank inside the wave, the wave's place inside the
// workgroup, the workgroup's place -- one counter update per workgroup.  Called by all threads; -1 for threads without.
__device__ __forceinline__ int append_positions(bool claimed, int32_t* counter) {
    __shared__ int in_block, base;
    if (threadIdx.x == 0) in_block = 0;
    __syncthreads();
    const uint64_t cl = __ballot(claimed);
    const int lane = threadIdx.x & 63;
    int wave_base = 0;
    if (lane == 0 && cl) wave_base = atomicAdd(&in_block, __popcll(cl));
    wave_base = __shfl(wave_base, 0);
    __syncthreads();
    if (threadIdx.x == 0) base = in_block ? atomicAdd(counter, in_block) : 0;
    __syncthreads();
    return claimed ? base + wave_base + __popcll(cl & ((1ull << lane) - 1)) : -1;
}

__device__ __forceinline__ uint32_t leaf_hash(int b, int li, int lj, int lk) {
    return mix32(mix32(mix32(mix32(0x811C9DC5u, (uint32_t)b), (uint32_t)li), (uint32_t)lj), (uint32_t)lk);
}

// Points of a batch without grids: no pass reads them, but coordinates that no cell holds are refused there too.
__global__ void k_count_bad_points(const RowSource rows, int64_t n_rows, GridHeader* hdr) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int bad = 0;
    if (r < n_rows) load_row<true>(rows, r, bad);
    if (bad) atomicAdd(&hdr->n_bad, bad);
}

// ---- direct path
constexpr int kDirectThreads = 256;
template <bool kPoints>
__global__ void __launch_bounds__(kDirectThreads)
k_voxels_to_leaves(const RowSource rows, int64_t n_rows, const BatchRanges joff, int B,
                   int32_t* __restrict__ slots, uint32_t slot_mask, LeafList L, GridHeader* hdr) {
    const int64_t r = (int64_t)blockIdx.x * kDirectThreads + threadIdx.x;
    int li = 0, lj = 0, lk = 0, b = -1;
    uint32_t h = 0;
    bool claimed = false;
    if (r < n_rows) {
        int bad = 0, ignored = 0;
        const int3 v = load_row<kPoints>(rows, r, bad);
        if (bad) atomicAdd(&hdr->n_bad, bad);
        b = find_batch(joff, B, r);
        if (b >= 0) {
            li = v.x >> 3; lj = v.y >> 3; lk = v.z >> 3;
            h = leaf_hash(b, li, lj, lk) & slot_mask;
            bool found = false;
            for (uint32_t probe = 0; probe <= slot_mask; ++probe) {
                // slots hold a representative input row + 1 (0 = empty); device-coherent read: a slot
                // claimed from another XCD must be seen
                int32_t s = __hip_atomic_load(&slots[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (s == 0) {
                    const int32_t old = atomicCAS(&slots[h], 0, (int32_t)r + 1);
                    if (old == 0) { found = claimed = true; break; }
                    s = old;
                }
                const int64_t q = s - 1;
                const int3 o = load_row<kPoints>(rows, q, ignored);
                if ((o.x >> 3) == li && (o.y >> 3) == lj && (o.z >> 3) == lk && find_batch(joff, B, q) == b) {
                    found = true;
                    break;
                }
                h = (h + 1) & slot_mask;
            }
            if (!found) atomicOr(&hdr->overflow, 4 | 32);   // table full: the leaf count is incomplete
            else atomicOr((unsigned long long*)&L.mask[(size_t)h * 8 + (v.x & 7)], 1ull << (((v.y & 7) << 3) | (v.z & 7)));
        }
    }
    const int pos = append_positions(claimed, &hdr->n_leaf_raw);
    if (pos >= 0) {
        if (pos < L.cap) { L.key[pos] = make_int4(li, lj, lk, b); L.mask_idx[pos] = (int32_t)h; }
        else atomicOr(&hdr->overflow, 4);
    }
}

// ---- coarse grid straight from the fine grid's leaves (Sec. 3.6.2: the grid of floor(ijk / 2))
// A fine leaf covers a 4x4x4 block of one coarse leaf: its 512-bit mask folds to 64 bits (a coarse voxel is active
// when any of its 8 children is), 16 bits in each of four words of the coarse leaf's mask.  One thread per fine
// leaf claims the coarse leaf in the table of the direct path (slots hold a representative fine leaf + 1) and ORs
// its four words in -- tens of thousands of items instead of a row per fine voxel through the whole voxel pass.
struct CoarsePiece { int li, lj, lk, first_word; uint64_t word[4]; };
__device__ __forceinline__ CoarsePiece coarse_piece(const fx_leaf* __restrict__ lf) {
    CoarsePiece c;
    const int oi = lf->origin[0], oj = lf->origin[1], ok = lf->origin[2];
    c.li = oi >> 4; c.lj = oj >> 4; c.lk = ok >> 4;                // coarse leaf coordinate: (origin >> 1) >> 3
    c.first_word = (oi >> 1) & 7;                                  // 0 or 4 along each axis: the block inside the coarse leaf
    const int bj = (oj >> 1) & 7, bk = (ok >> 1) & 7;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        uint64_t m = lf->mask[2 * a] | lf->mask[2 * a + 1];         // pairs along i
        m = (m | (m >> 1)) & 0x5555555555555555ull;                 // pairs along k, kept at the even bits
        m = (m | (m >> 1)) & 0x3333333333333333ull;                 // ... gathered into the low nibble of every byte
        m = (m | (m >> 2)) & 0x0F0F0F0F0F0F0F0Full;
        m = (m | (m >> 8)) & 0x00FF00FF00FF00FFull;                 // pairs along j: bytes 0, 2, 4, 6
        uint64_t r = 0;
#pragma unroll
        for (int cj = 0; cj < 4; ++cj) r |= ((m >> (16 * cj)) & 0xFull) << ((bj + cj) * 8 + bk);
        c.word[a] = r;
    }
    return c;
}

constexpr int kCoarseThreads = 512;
__global__ void __launch_bounds__(kCoarseThreads)
k_coarse_leaves(TreeView fine, int32_t* __restrict__ slots, uint32_t slot_mask, LeafList L, GridHeader* hdr) {
    const int f = (int)((int64_t)blockIdx.x * blockDim.x + threadIdx.x);
    const bool has = f < fine.n_leaf;
    int li = 0, lj = 0, lk = 0, b = 0;
    uint32_t h = 0;
    bool claimed = false;
    if (has) {
        const fx_leaf* lf = fine.leaf + f;
        const CoarsePiece c = coarse_piece(lf);
        b = lf->batch;
        li = c.li; lj = c.lj; lk = c.lk;
        h = leaf_hash(b, li, lj, lk) & slot_mask;
        bool found = false;
        for (uint32_t probe = 0; probe <= slot_mask; ++probe) {
            int32_t sl = __hip_atomic_load(&slots[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (sl == 0) {
                const int32_t old = atomicCAS(&slots[h], 0, f + 1);
                if (old == 0) { found = claimed = true; break; }
                sl = old;
            }
            const fx_leaf* o = fine.leaf + (sl - 1);
            if ((o->origin[0] >> 4) == li && (o->origin[1] >> 4) == lj && (o->origin[2] >> 4) == lk && o->batch == b) {
                found = true;
                break;
            }
            h = (h + 1) & slot_mask;
        }
        if (!found) atomicOr(&hdr->overflow, 4 | 32);
        else {
#pragma unroll
            for (int a = 0; a < 4; ++a)
                if (c.word[a]) atomicOr((unsigned long long*)&L.mask[(size_t)h * 8 + c.first_word + a], (unsigned long long)c.word[a]);
        }
    }
    // (with an update of the list's counter per wave, 590 of them for 38 k fine leaves, this launch took 14 us)
    const int pos = append_positions(claimed, &hdr->n_leaf_raw);
    if (pos >= 0) {
        if (pos < L.cap) { L.key[pos] = make_int4(li, lj, lk, b); L.mask_idx[pos] = (int32_t)h; }
        else atomicOr(&hdr->overflow, 4);
    }
}

// ---- padded grid straight from the grid's leaves (Sec. 3.6.2 grid construction by padding; Sec. 3.3's dilation)
// Dilation by r <= 8 moves a leaf's voxels into at most the 27 leaves around it, and a leaf of the padded grid
// takes voxels from at most the 27 source leaves around it.  Two passes, neither with an atomic per voxel or per
// mask word (atomics run at memory; an OR per word of every (leaf, neighbour) pair cost 220 us on a 38 k-leaf grid):
//   k_pad_claim   thread = (source leaf, one of its 27 neighbour positions): the neighbour receives a voxel iff the
//                 leaf has one within r of the shared face, edge or corner -- a mask test; such neighbours are
//                 claimed in the direct path's leaf table (a slot's representative is (source leaf, position) + 1);
//   k_pad_masks   wave = listed leaf of the padded grid: gathers the masks of the 27 source leaves around it into a
//                 24^3 box, dilates axis by axis towards the centre 8^3 and stores the leaf's mask with plain stores.
__device__ __forceinline__ uint32_t reach_bits(int p, int r) {
    // positions 0..7 along one axis whose voxels reach the neighbour at p - 1 (p = 1: the leaf itself) under dilation by r
    return p == 1 ? 0xFFu : (r == 0 ? 0u : (p == 0 ? (0xFFu >> (8 - r)) : ((0xFFu << (8 - r)) & 0xFFu)));
}

constexpr int kPadClaimThreads = 1024;
__global__ void __launch_bounds__(kPadClaimThreads)
k_pad_claim(TreeView src, int r, int32_t* __restrict__ slots, uint32_t slot_mask, LeafList L, GridHeader* hdr,
            int32_t* __restrict__ bad) {
    // Most leaves of the padded grid are leaves of the source grid.  Those are listed by their own thread (position
    // 13, the leaf itself) without the table: their masks sit behind the table's, at slot_mask + 1 + leaf.  A
    // neighbour position first looks its leaf up in the source tree (plain cached loads) and goes to the table only
    // when the leaf is new -- table probes are loads and compare-and-swaps that must see other workgroups' writes,
    // they run at memory, and one per (leaf, position) pair was 800 k of them on a 38 k-leaf grid (40 us).
    // List positions come from one counter; an update per wave would be 19 k updates of one address (150 us, they
    // run one after the other), so a workgroup counts its leaves in LDS and takes its run with one update.
    __shared__ int block_claims, block_base;
    const int lane = threadIdx.x & 63;
    if (threadIdx.x == 0) block_claims = 0;
    __syncthreads();
    const int64_t t = (int64_t)blockIdx.x * kPadClaimThreads + threadIdx.x;
    const int64_t f = t >> 5;
    const int piece = (int)(t & 31);
    int4 my_key = make_int4(0, 0, 0, 0);
    int32_t my_slot = -1;
    if (f < src.n_leaf && piece < 27) {
        const fx_leaf* lf = src.leaf + f;
        const int pa = piece / 9, pb = (piece / 3) % 3, pc = piece % 3;
        const uint32_t ia = reach_bits(pa, r), jb = reach_bits(pb, r), kc = reach_bits(pc, r);
        uint64_t region = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) if ((jb >> j) & 1) region |= (uint64_t)kc << (8 * j);
        uint64_t any = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) if ((ia >> i) & 1) any |= lf->mask[i] & region;
        const int b = lf->batch;
        const int64_t pi = (int64_t)lf->origin[0] + 8 * (pa - 1), pj = (int64_t)lf->origin[1] + 8 * (pb - 1),
                      pk = (int64_t)lf->origin[2] + 8 * (pc - 1);
        const int64_t lo = INT32_MIN, hi = (int64_t)INT32_MAX - 7;
        if (piece == 13) {
            my_slot = (int32_t)(slot_mask + 1 + (uint32_t)f);
            my_key = make_int4((int)(pi >> 3), (int)(pj >> 3), (int)(pk >> 3), b);
        } else if (any) {
            if (pi < lo || pi > hi || pj < lo || pj > hi || pk < lo || pk > hi) {
                atomicAdd(bad, 1);
            } else if (find_leaf<true>(src, b, (int)pi, (int)pj, (int)pk) < 0) {
                const int li = (int)(pi >> 3), lj = (int)(pj >> 3), lk = (int)(pk >> 3);
                uint32_t h = leaf_hash(b, li, lj, lk) & slot_mask;
                bool found = false;
                for (uint32_t probe = 0; probe <= slot_mask; ++probe) {
                    int32_t sl = __hip_atomic_load(&slots[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (sl == 0) {
                        const int32_t old = atomicCAS(&slots[h], 0, (int32_t)(f * 27 + piece + 1));
                        if (old == 0) {
                            found = true;
                            my_slot = (int32_t)h;
                            my_key = make_int4(li, lj, lk, b);
                            break;
                        }
                        sl = old;
                    }
                    const int rf = (sl - 1) / 27, rp = (sl - 1) - 27 * rf;
                    const fx_leaf* ro = src.leaf + rf;
                    if ((ro->origin[0] >> 3) + (rp / 9 - 1) == li && (ro->origin[1] >> 3) + ((rp / 3) % 3 - 1) == lj &&
                        (ro->origin[2] >> 3) + (rp % 3 - 1) == lk && ro->batch == b) {
                        found = true;
                        break;
                    }
                    h = (h + 1) & slot_mask;
                }
                if (!found) atomicOr(&hdr->overflow, 4 | 32);     // table full: the leaf count is incomplete
            }
        }
    }
    // positions: rank of the leaf inside the wave, the wave's run inside the workgroup, the workgroup's run
    const uint64_t cl = __ballot(my_slot >= 0);
    int wave_base = 0;
    if (lane == 0 && cl) wave_base = atomicAdd(&block_claims, __popcll(cl));
    wave_base = __shfl(wave_base, 0);
    __syncthreads();
    if (threadIdx.x == 0) block_base = block_claims ? atomicAdd(&hdr->n_leaf_raw, block_claims) : 0;
    __syncthreads();
    if (my_slot >= 0) {
        const int pos = block_base + wave_base + __popcll(cl & ((1ull << lane) - 1));
        if (pos < L.cap) { L.key[pos] = my_key; L.mask_idx[pos] = my_slot; }
        else atomicOr(&hdr->overflow, 4);
    }
}

constexpr int kPadWaves = 4;
__global__ void __launch_bounds__(64 * kPadWaves)
k_pad_masks(TreeView src, int r, LeafList L, const GridHeader* hdr) {
    __shared__ uint32_t box[kPadWaves][24][24];           // [i][j], bit = k: the 27 source leaves, then dilated along k
    __shared__ uint32_t along_j[kPadWaves][24][8];        // [i][centre j], 8 bits of k
    __shared__ unsigned long long centre[kPadWaves][8];   // the leaf's mask, byte (i, j) written by lane (i, j)
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int pos = blockIdx.x * kPadWaves + wave;
    const int n_listed = min(hdr->n_leaf_raw, L.cap);
    if (pos >= n_listed) return;
    auto wave_sync = [] { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); __builtin_amdgcn_wave_barrier(); };
    const int4 key = L.key[pos];
    // the source leaves around the leaf: lane < 27 looks one up
    int around = -1;
    if (lane < 27) {
        const int64_t ni = (int64_t)key.x + (lane / 9 - 1), nj = (int64_t)key.y + ((lane / 3) % 3 - 1), nk = (int64_t)key.z + (lane % 3 - 1);
        const int64_t lo = -(1ll << 28), hi = (1ll << 28) - 1;      // leaf coordinates of int32 voxels
        if (ni >= lo && ni <= hi && nj >= lo && nj <= hi && nk >= lo && nk <= hi)
            around = find_leaf<true>(src, key.w, (int)(ni * 8), (int)(nj * 8), (int)(nk * 8));
    }
    // box rows: task = (pa, pb, i) takes word i of the three leaves (pa, pb, 0..2) and writes rows j = 0..7 of plane
    // 8 pa + i; only the planes and rows within r of the centre are read later
    const int first = 8 - r, last = 15 + r, width = 8 + 2 * r;
    for (int e = lane; e < 128; e += 64) {
        const int pa = e / 24, pb = (e / 8) % 3, i = e & 7;      // e < 72 are tasks
        const int plane = 8 * pa + i;
        const bool wanted = e < 72 && plane >= first && plane <= last && 8 * pb + 7 >= first && 8 * pb <= last;
        uint64_t w[3];
#pragma unroll
        for (int pc = 0; pc < 3; ++pc) {
            const int from = e < 72 ? (pa * 3 + pb) * 3 + pc : 0;
            const int f = __shfl(around, from);
            w[pc] = (wanted && f >= 0) ? src.leaf[f].mask[i] : 0ull;
        }
        if (wanted) {
#pragma unroll
            for (int j = 0; j < 8; ++j)
                box[wave][plane][8 * pb + j] = (uint32_t)((w[0] >> (8 * j)) & 0xFF) | ((uint32_t)((w[1] >> (8 * j)) & 0xFF) << 8) |
                                               ((uint32_t)((w[2] >> (8 * j)) & 0xFF) << 16);
        }
    }
    wave_sync();
    // along k: the centre byte of every row that the later steps read (|i - centre| and |j - centre| within r)
    for (int e = lane; e < width * width; e += 64) {
        const int a = e / width, ii = first + a, jj = first + (e - a * width);
        const uint32_t row = box[wave][ii][jj];
        uint32_t acc = 0;
        for (int sft = 8 - r; sft <= 8 + r; ++sft) acc |= row >> sft;
        box[wave][ii][jj] = acc & 0xFFu;
    }
    wave_sync();
    // along j
    for (int e = lane; e < width * 8; e += 64) {
        const int ii = first + (e >> 3), j = e & 7;
        uint32_t acc = 0;
        for (int d = -r; d <= r; ++d) acc |= box[wave][ii][j + 8 + d];
        along_j[wave][ii][j] = acc;
    }
    wave_sync();
    // along i: lane = (i, j) of the leaf
    {
        const int i = lane >> 3, j = lane & 7;
        uint32_t acc = 0;
        for (int d = -r; d <= r; ++d) acc |= along_j[wave][i + 8 + d][j];
        reinterpret_cast<unsigned char*>(centre[wave])[lane] = (unsigned char)acc;
    }
    wave_sync();
    if (lane < 8) L.mask[(size_t)L.mask_idx[pos] * 8 + lane] = centre[wave][lane];
}

// ---- subdivided grid straight from the grid's leaves (Sec. 3.6.2 grid construction by subdivision)
// A leaf of the fine grid is one octant (4^3 voxels) of a coarse leaf with every voxel doubled along each axis;
// it has exactly one source, so there is no table and no claim: thread = (coarse leaf, octant) expands the octant's
// 64 bits into the fine leaf's 512 (mask slot 8 * leaf + octant) and lists the leaf if the octant is not empty.
constexpr int kSubdivideThreads = 1024;
__global__ void __launch_bounds__(kSubdivideThreads)
k_subdivide_leaves(TreeView coarse, LeafList L, GridHeader* hdr, int32_t* __restrict__ bad) {
    __shared__ int block_count, block_base;
    const int lane = threadIdx.x & 63;
    if (threadIdx.x == 0) block_count = 0;
    __syncthreads();
    const int64_t t = (int64_t)blockIdx.x * kSubdivideThreads + threadIdx.x;
    const int64_t f = t >> 3;
    const int q = (int)(t & 7), bi = q >> 2, bj = (q >> 1) & 1, bk = q & 1;
    bool listed = false;
    int4 key = make_int4(0, 0, 0, 0);
    if (f < coarse.n_leaf) {
        const fx_leaf* lf = coarse.leaf + f;
        uint64_t fine[4];
        uint64_t any = 0;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const uint64_t w = lf->mask[4 * bi + a];
            uint64_t rows = 0;
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                uint32_t x = (uint32_t)(w >> (8 * (4 * bj + jj) + 4 * bk)) & 0xFu;     // k = 4 bk .. 4 bk + 3 of row j
                x = (x | (x << 2)) & 0x33u;
                x = (x | (x << 1)) & 0x55u;
                x |= x << 1;                                                           // every bit twice
                rows |= (uint64_t)(x | (x << 8)) << (16 * jj);                         // the row twice
            }
            fine[a] = rows;
            any |= rows;
        }
        if (any) {
            const int o0 = lf->origin[0], o1 = lf->origin[1], o2 = lf->origin[2];
            const int lo = -(1 << 30), hi = (1 << 30) - 8;                             // doubled coordinates stay int32
            if (o0 < lo || o0 > hi || o1 < lo || o1 > hi || o2 < lo || o2 > hi) {
                atomicAdd(bad, 1);
            } else {
                listed = true;
                key = make_int4(2 * (o0 >> 3) + bi, 2 * (o1 >> 3) + bj, 2 * (o2 >> 3) + bk, lf->batch);
                uint64_t* m = L.mask + (size_t)t * 8;
#pragma unroll
                for (int a = 0; a < 4; ++a) { m[2 * a] = fine[a]; m[2 * a + 1] = fine[a]; }      // the plane twice
            }
        }
    }
    const uint64_t li = __ballot(listed);
    int wave_base = 0;
    if (lane == 0 && li) wave_base = atomicAdd(&block_count, __popcll(li));
    wave_base = __shfl(wave_base, 0);
    __syncthreads();
    if (threadIdx.x == 0) block_base = block_count ? atomicAdd(&hdr->n_leaf_raw, block_count) : 0;
    __syncthreads();
    if (listed) {
        const int pos = block_base + wave_base + __popcll(li & ((1ull << lane) - 1));
        if (pos < L.cap) { L.key[pos] = key; L.mask_idx[pos] = (int32_t)t; }
        else atomicOr(&hdr->overflow, 4);
    }
}

// ---- partitioned path
constexpr int kPartThreads = 1024;
constexpr int kMaxBuckets = 2048;
constexpr int kRowsPerBucket = 3072;                             // upper bound of the mean while the bucket count is below its cap
constexpr int kBucketSlots = 1024;                               // LDS leaf table of one bucket

// A row on its way through the buckets is one 8-byte record when every coordinate of the input lies in [-2^19, 2^19)
// and there are at most 16 grids (grid, i, j, k in 4 + 3 x 20 bits): half the bytes of four 32-bit words in the
// row pass's writes and the leaf pass's reads.  Otherwise it is two words, (i, j) and (k, grid).
__device__ __forceinline__ bool row_is_wide(const int3& v) {
    constexpr uint32_t half = 1u << 19;
    return (((uint32_t)v.x + half) | ((uint32_t)v.y + half) | ((uint32_t)v.z + half)) >= 2 * half;
}
__device__ __forceinline__ uint64_t pack_row(const int3& v, int b) {
    constexpr uint32_t half = 1u << 19;
    return ((uint64_t)(uint32_t)b << 60) | ((uint64_t)((uint32_t)v.x + half) << 40) | ((uint64_t)((uint32_t)v.y + half) << 20) |
           (uint64_t)((uint32_t)v.z + half);
}
__device__ __forceinline__ int4 unpack_row(uint64_t r) {
    constexpr int half = 1 << 19;
    constexpr uint32_t m = (1u << 20) - 1;
    return make_int4((int)((uint32_t)(r >> 40) & m) - half, (int)((uint32_t)(r >> 20) & m) - half, (int)((uint32_t)r & m) - half, (int)(r >> 60));
}
__device__ __forceinline__ uint64_t two_words(int a, int b) { return (uint64_t)(uint32_t)a | ((uint64_t)(uint32_t)b << 32); }

// What the first kernel of a build clears besides its own work: the head of the grid buffer (header, bases,
// root table, child masks) and the head of the scratch buffer (scan tickets and block sums, root-tile table).
// Nothing reads or updates either before the next launch.
struct ClearRanges {
    uint4* p[2];
    uint32_t n16[2];   // 16-byte units
};

// One pass over the rows: a workgroup takes a piece of 4096 to 16384 of them, orders their records by bucket in LDS and writes
// them behind one another, whole lines at a time; starts[piece][bucket] says where a bucket's run begins, [n_buckets] how many
// rows the piece has in grids.  The leaf pass picks its bucket's runs out of all pieces.  (A counting pass, a scan over
// (piece, bucket) and a scatter that gave every bucket one contiguous range of records read the rows twice: 10 M points
// 52 + 14 + 81 us, now 75; 1 M rows 7 + 6 + 10, now 10.  The leaf pass takes 2 to 3 us more for its runs.)  info[piece]: 1 if some row does not fit a packed record (all records of the piece are
// then two words), and twice the number of points whose cell is not representable.
template <bool kPoints, int QUADS>
__global__ void __launch_bounds__(kPartThreads)
k_bucket_sort(const RowSource rows, int64_t n_rows, const BatchRanges joff, int B, uint32_t bucket_mask,
              uint64_t* __restrict__ records, int64_t second_word, uint16_t* __restrict__ starts, int32_t* __restrict__ info, ClearRanges clr) {
    extern __shared__ __align__(16) unsigned char part_lds[];
    constexpr int kRows = 4 * QUADS * kPartThreads;
    static_assert(kRows <= 1 << 16, "runs begin at 16-bit places");
    const uint32_t n_buckets = bucket_mask + 1;
    uint64_t* rec = reinterpret_cast<uint64_t*>(part_lds);                  // [kRows]
    uint32_t* cnt = reinterpret_cast<uint32_t*>(rec + kRows);               // [n_buckets] rows of this piece, then the first LDS slot
    const int tid = threadIdx.x;
    int3 v[4 * QUADS];
    int b[4 * QUADS];
    int bad = 0;
    bool is_wide = B > 16;
    // nearly all pieces lie in one grid, which is then looked up once
    const int64_t r0 = (int64_t)blockIdx.x * kRows, r_last = min(r0 + kRows, n_rows) - 1;
    const int b_first = find_batch(joff, B, r0), b_all = b_first == find_batch(joff, B, r_last) ? b_first : -1;
#pragma unroll
    for (int c = 0; c < QUADS; ++c) {
        const int64_t r = r0 + (int64_t)c * (4 * kPartThreads) + 4 * tid;
        int3 w[4];
        const int n = load_four_rows<kPoints>(rows, n_rows, r, w, bad);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            v[4 * c + q] = w[q];
            b[4 * c + q] = q < n ? b_all : -1;
        }
    }
    if (b_all < 0) {
#pragma unroll
        for (int q = 0; q < 4 * QUADS; ++q) {
            const int64_t r = r0 + (int64_t)(q >> 2) * (4 * kPartThreads) + 4 * tid + (q & 3);
            b[q] = r < n_rows ? find_batch(joff, B, r) : -1;
        }
    }
#pragma unroll
    for (int q = 0; q < 4 * QUADS; ++q) is_wide |= b[q] >= 0 && row_is_wide(v[q]);
#pragma unroll
    for (int c = 0; c < 2; ++c)
        for (uint32_t e = blockIdx.x * kPartThreads + tid; e < clr.n16[c]; e += gridDim.x * kPartThreads)
            clr.p[c][e] = make_uint4(0u, 0u, 0u, 0u);
    __shared__ int n_bad;
    if (tid == 0) n_bad = 0;
    for (uint32_t e = tid; e < n_buckets; e += kPartThreads) cnt[e] = 0;
    is_wide = __syncthreads_or(is_wide);
    if (kPoints && bad) atomicAdd(&n_bad, bad);
    uint32_t bucket[4 * QUADS], rank[4 * QUADS];
#pragma unroll
    for (int q = 0; q < 4 * QUADS; ++q) {
        bucket[q] = leaf_hash(b[q], v[q].x >> 3, v[q].y >> 3, v[q].z >> 3) & bucket_mask;
        rank[q] = b[q] >= 0 ? atomicAdd(&cnt[bucket[q]], 1u) : 0u;
    }
    __syncthreads();
    // first LDS slot of every bucket = exclusive scan of the counts, in place
    uint32_t n_local;
    {
        uint32_t t[2], sum = 0;
#pragma unroll
        for (int q = 0; q < 2; ++q) { const uint32_t e = tid * 2 + q; t[q] = e < n_buckets ? cnt[e] : 0u; sum += t[q]; }
        uint32_t run = block_exclusive_scan(sum, &n_local);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const uint32_t e = tid * 2 + q;
            if (e < n_buckets) cnt[e] = run;
            run += t[q];
        }
    }
    if (tid == 0) info[blockIdx.x] = (is_wide ? 1 : 0) | 2 * n_bad;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4 * QUADS; ++q)
        if (b[q] >= 0) rec[cnt[bucket[q]] + rank[q]] = is_wide ? two_words(v[q].x, v[q].y) : pack_row(v[q], b[q]);
    uint16_t* my_starts = starts + (size_t)blockIdx.x * (n_buckets + 1);
    for (uint32_t e = tid; e <= n_buckets; e += kPartThreads) my_starts[e] = (uint16_t)(e < n_buckets ? cnt[e] : n_local);
    __syncthreads();
    uint64_t* out = records + (int64_t)blockIdx.x * kRows;
    for (uint32_t s = tid; s < n_local; s += kPartThreads) out[s] = rec[s];
    if (!is_wide) return;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4 * QUADS; ++q)
        if (b[q] >= 0) rec[cnt[bucket[q]] + rank[q]] = two_words(v[q].z, b[q]);
    __syncthreads();
    for (uint32_t s = tid; s < n_local; s += kPartThreads) out[second_word + s] = rec[s];
}

// One workgroup per bucket: the bucket's distinct leaves and their masks, built in LDS.  The table's slots hold the
// leaf itself when the rows are packed records (17 bits per leaf coordinate, so a probe is one LDS read), a
// representative row + 1 otherwise.  A bucket with more leaves than slots (very sparse points) is walked in rounds, each
// of which takes the leaves of one class by two further bits of their hash; a class that is still too large is cut once
// more by two.  A row that finds no slot within kBucketProbes steps (one longer each time) says so: rows that walked a
// full table to its end read 1024 slots one after the other, in every round that came to nothing.
// The bucket's rows are the runs that the pieces of the row pass have of it, eight rows each on average at 10 M rows: their
// starts, 1024 pieces at a time, and a scan of their lengths go to LDS, and every thread takes up to four consecutive
// rows at a time, whose run it finds by bisection -- input in the order of its voxels has all rows of a piece in few runs.  Workgroup b
// runs on XCD b % 8: neighbouring buckets, whose runs and starts share lines, meet in one L2.
// kTwoWords: more than 16 grids, whose records have two words in every piece.  Both are then requested together; with the piece
// asked first and the second word behind it they were three loads one after the other, for every row and for every row that it is
// compared with (9 M rows of 40 grids in nearly as many leaves: this launch 2118 -> 1742 us, the build 6.32 -> 5.51 ms).
constexpr int kBucketThreads = 1024, kBucketProbes = 64, kBucketBatch = 4;
template <bool kTwoWords>
__global__ void __launch_bounds__(kBucketThreads, 8)
k_bucket_leaves(const uint64_t* __restrict__ records, int64_t second_word, const uint16_t* __restrict__ starts, const int32_t* __restrict__ info,
                int n_pieces, int piece_rows_log2, LeafList L, GridHeader* hdr) {
    __shared__ unsigned long long slot[kBucketSlots];     // 0 = empty
    __shared__ __align__(16) unsigned long long mask[kBucketSlots * 8];
    __shared__ uint32_t run_first[kBucketThreads];        // rows of the bucket in the pieces before (of these 1024)
    __shared__ uint16_t run_start[kBucketThreads];        // where the run begins in its piece
    __shared__ int32_t list_base;
    static_assert(kBucketSlots == kBucketThreads, "one table slot per thread in the listing step");
    const int tid = threadIdx.x;
    const uint32_t n_buckets = gridDim.x, bucket = (blockIdx.x & 7) * (n_buckets >> 3) + (blockIdx.x >> 3);
    uint32_t n_run_rows = 0, from = 0, to = 0;
    auto request_runs = [&](int p0) {                     // the runs of pieces p0 .. p0 + 1023
        const uint16_t* s = starts + (size_t)min(p0 + tid, n_pieces - 1) * (n_buckets + 1) + bucket;
        from = s[0];
        to = s[1];
    };
    auto place_runs = [&](int p0) {
        const uint32_t first = block_exclusive_scan(p0 + tid < n_pieces ? to - from : 0u, &n_run_rows);
        run_first[tid] = first;
        run_start[tid] = (uint16_t)from;
        __syncthreads();
    };
    auto clear = [&]() {
        slot[tid] = 0ull;
        for (int e = tid; e < kBucketSlots * 4; e += kBucketThreads) reinterpret_cast<ulonglong2*>(mask)[e] = make_ulonglong2(0ull, 0ull);
    };
    request_runs(0);
    int all_info = 0;
    for (int e = tid; e < n_pieces; e += kBucketThreads) {
        const int i = info[e];
        all_info |= i;
        if (blockIdx.x == 0 && i > 1) atomicAdd(&hdr->n_bad, i >> 1);
    }
    clear();                                              // while those are under way
    const bool is_wide = __syncthreads_or(all_info & 1) || kTwoWords;
    if (n_pieces <= kBucketThreads) place_runs(0);
    // a row by its place among the records; with wide rows a piece says whether its records are two words (kTwoWords: all do)
    auto second_of = [&](uint32_t r) { return kTwoWords ? records[second_word + r] : 0ull; };
    auto unpack_at = [&](uint32_t r, uint64_t a, uint64_t c) {
        if (!kTwoWords) {
            if (!is_wide || !(info[r >> piece_rows_log2] & 1)) return unpack_row(a);
            c = records[second_word + r];
        }
        return make_int4((int)(uint32_t)a, (int)(uint32_t)(a >> 32), (int)(uint32_t)c, (int)(uint32_t)(c >> 32));
    };
    auto row_at = [&](uint32_t r) { return unpack_at(r, records[r], second_of(r)); };
    uint32_t class_mask = 0, class_value = 0;             // this round's leaves: hash bits 24.. under the mask
    for (bool first_round = true;; first_round = false) {
        if (!first_round) { clear(); __syncthreads(); }
        bool full = false;
        auto take_row = [&](uint32_t r, uint64_t record, uint64_t second) {      // false: no slot found
            const int4 v = unpack_at(r, record, second);
            const int li = v.x >> 3, lj = v.y >> 3, lk = v.z >> 3;
            const uint32_t hash = leaf_hash(v.w, li, lj, lk);
            if (((hash >> 24) & class_mask) != class_value) return true;
            uint32_t h = (hash >> 12) & (kBucketSlots - 1);   // other bits than the bucket's
            // the leaf as a nonzero word: biased coordinates of 17 bits, grid, a set top bit
            const unsigned long long self = is_wide ? (unsigned long long)r + 1ull
                : (1ull << 63) | ((unsigned long long)(uint32_t)v.w << 51) | ((unsigned long long)(uint32_t)(li + (1 << 16)) << 34) |
                  ((unsigned long long)(uint32_t)(lj + (1 << 16)) << 17) | (unsigned long long)(uint32_t)(lk + (1 << 16));
            bool found = false;
            for (int probe = 0; probe < kBucketProbes; ++probe) {
                unsigned long long s = __hip_atomic_load(&slot[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                if (s == 0ull) {
                    s = atomicCAS(&slot[h], 0ull, self);
                    if (s == 0ull) { found = true; break; }
                }
                if (!is_wide) {
                    if (s == self) { found = true; break; }
                } else {
                    const int4 o = row_at((uint32_t)(s - 1ull));
                    if ((o.x >> 3) == li && (o.y >> 3) == lj && (o.z >> 3) == lk && o.w == v.w) { found = true; break; }
                }
                h = (h + probe + 1) & (kBucketSlots - 1);
            }
            if (!found) return false;
            // rows of one voxel mostly find it there: updates of one word run one after the other
            const unsigned long long bit = 1ull << (((v.y & 7) << 3) | (v.z & 7));
            unsigned long long* const word = &mask[h * 8 + (v.x & 7)];
            if (!(__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) & bit)) atomicOr(word, bit);
            return true;
        };
        for (int p0 = 0; p0 < n_pieces; p0 += kBucketThreads) {
            if (n_pieces > kBucketThreads) { __syncthreads(); request_runs(p0); place_runs(p0); }
            const uint32_t per = min((n_run_rows + kBucketThreads - 1) / kBucketThreads, (uint32_t)kBucketBatch);
            uint32_t r = tid * per;
            if (r >= n_run_rows) continue;
            int run = 0;                                  // the last run that begins at or before row r
#pragma unroll
            for (int step = kBucketThreads / 2; step > 0; step >>= 1)
                if (run_first[run + step] <= r) run += step;
            for (; r < n_run_rows && !full; r += kBucketThreads * per) {
                const uint32_t n = min(per, n_run_rows - r);
                uint32_t at[kBucketBatch];
                uint64_t rec[kBucketBatch], rec2[kBucketBatch];
#pragma unroll
                for (int u = 0; u < kBucketBatch; ++u) {  // past the n-th the last row again
                    const uint32_t ru = r + min((uint32_t)u, n - 1);
                    if (run + 1 < kBucketThreads && run_first[run + 1] <= ru) ++run;
                    if (run + 1 < kBucketThreads && run_first[run + 1] <= ru) {       // over the empty runs between
#pragma unroll 1
                        for (int step = kBucketThreads / 2; step > 0; step >>= 1)
                            if (run + step < kBucketThreads && run_first[run + step] <= ru) run += step;
                    }
                    at[u] = ((uint32_t)(p0 + run) << piece_rows_log2) + run_start[run] + (ru - run_first[run]);
                    rec[u] = records[at[u]];
                    rec2[u] = second_of(at[u]);
                }
#pragma unroll
                for (int u = 0; u < kBucketBatch; ++u)
                    if (u < (int)n && !full) full = !take_row(at[u], rec[u], rec2[u]);
            }
        }
        if (__syncthreads_or(full)) {
            // nothing of this class has been listed: take its first quarter instead.  A sixteenth of a bucket that still
            // fills the table is left to the path without buckets.
            if (class_mask == 15) { if (tid == 0) atomicOr(&hdr->overflow, 64); return; }
            class_mask = class_mask * 4 + 3;
            continue;
        }
        // append the leaves to the list (thread = table slot)
        const unsigned long long s = slot[tid];
        uint32_t total;
        const uint32_t before = block_exclusive_scan(s != 0ull ? 1u : 0u, &total);
        if (tid == 0) list_base = total ? atomicAdd(&hdr->n_leaf_raw, (int)total) : 0;
        __syncthreads();
        const int pos = list_base + (int)before;
        if (s != 0ull && pos < L.cap) {
            if (is_wide) {
                const int4 v = row_at((uint32_t)(s - 1ull));
                L.key[pos] = make_int4(v.x >> 3, v.y >> 3, v.z >> 3, v.w);
            } else {
                constexpr uint32_t m = (1u << 17) - 1;
                constexpr int half = 1 << 16;
                L.key[pos] = make_int4((int)((uint32_t)(s >> 34) & m) - half, (int)((uint32_t)(s >> 17) & m) - half,
                                       (int)((uint32_t)s & m) - half, (int)((uint32_t)(s >> 51) & 15u));
            }
            L.mask_idx[pos] = pos;
#pragma unroll
            for (int w = 0; w < 8; w += 2)
                *reinterpret_cast<ulonglong2*>(&L.mask[(size_t)pos * 8 + w]) = *reinterpret_cast<const ulonglong2*>(&mask[tid * 8 + w]);
        } else if (s != 0ull) {
            atomicOr(&hdr->overflow, 4);
        }
        // the next class: the next quarter of the same one, then the next one (class_value & 3), cut the same way
        if (class_mask == 0) return;
        if (class_mask == 3) {
            if (++class_value == 4) return;
        } else {
            class_value += 4;
            if (class_value == 19) return;            // the last quarter of class 3
            if (class_value > 15) class_value = (class_value & 3) + 1;
        }
        __syncthreads();
    }
}

// key of distinct leaf `idx`, or false past the end
__device__ __forceinline__ bool leaf_at(const LeafList& L, const GridHeader* hdr, int64_t idx, int4* key) {
    if (idx >= L.cap) return false;
    *key = L.key[idx];            // fetched together with the count, not after it (entries past the count are unused)
    return idx < hdr->n_leaf_raw;
}

// ---------------------------------------------------------------------------------- root tiles
// Distinct (grid, tile) pairs of the leaves go into a small open-addressing table whose slots
// hold a representative leaf (+1; 0 = empty).  Called by all threads of a workgroup together (`has`:
// this thread holds leaf `idx` with key `key`).
constexpr int kFindTilesThreads = 1024;
constexpr int kKnownTiles = 64;
__device__ __forceinline__ void find_tile_item(const LeafList& L, GridHeader* hdr, int idx, bool has, const int4& key,
                                               int32_t* __restrict__ tile_slots, int32_t* __restrict__ rep_leaves) {
    const int4 tile = make_int4(key.x >> 9, key.y >> 9, key.z >> 9, key.w);   // leaf coordinate >> 9 = voxel >> 12
    auto same = [](const int4& a, const int4& b) { return a.x == b.x && a.y == b.y && a.z == b.z && a.w == b.w; };
    // One thread per distinct tile of the WORKGROUP goes to the table: accesses to one address from all over the
    // device queue up at memory (a coherent read of one slot from each of 600 waves took longer than the rest of
    // this launch), and nearly all leaves share a few tiles.  Every wave names the tiles of its leaves one after the other (the
    // first lane still waiting, and all lanes with its tile are done), and the first wave that puts a tile into the table in
    // LDS speaks for it; a wave that finds no place there speaks for itself.  (Rounds of the whole workgroup, two barriers
    // for each distinct tile: 376 k leaves in eight tiles 19.7 -> 14.3 us, four indoor scenes 13.6 -> 10.2.)
    __shared__ unsigned long long known[kKnownTiles];
    const int tid = (int)threadIdx.x, lane = tid & 63;
    for (int e = tid; e < kKnownTiles; e += (int)blockDim.x) known[e] = 0ull;
    __syncthreads();
    bool waiting = has, speaker = false;
    for (uint64_t left = __ballot(waiting); left; left = __ballot(waiting)) {
        const int first = __ffsll((long long)left) - 1;
        const int4 t = make_int4(__builtin_amdgcn_readlane(tile.x, first), __builtin_amdgcn_readlane(tile.y, first),
                                 __builtin_amdgcn_readlane(tile.z, first), __builtin_amdgcn_readlane(tile.w, first));
        if (same(tile, t)) waiting = false;
        if (lane == first) {
            // a grid number of 15 bits and tile coordinates of 16 (voxels within 2^27); others speak for themselves
            const bool fits = (((uint32_t)t.x + 0x8000u) | ((uint32_t)t.y + 0x8000u) | ((uint32_t)t.z + 0x8000u)) < 0x10000u && (uint32_t)t.w < 0x8000u;
            const unsigned long long word = 1ull << 63 | (unsigned long long)(uint32_t)t.w << 48 | (unsigned long long)(t.x & 0xFFFF) << 32 |
                                            (unsigned long long)(t.y & 0xFFFF) << 16 | (unsigned long long)(t.z & 0xFFFF);
            speaker = true;
            uint32_t h = mix32(mix32(mix32(0x811C9DC5u, (uint32_t)t.x ^ (uint32_t)t.w << 16), (uint32_t)t.y), (uint32_t)t.z) & (kKnownTiles - 1);
            for (int probe = 0; probe < 4 && fits; ++probe) {
                const unsigned long long old = atomicCAS(&known[h], 0ull, word);
                if (old == 0ull) break;
                if (old == word) { speaker = false; break; }
                h = (h + 1) & (kKnownTiles - 1);
            }
        }
    }
    if (!speaker) return;
    uint32_t h = mix32(mix32(mix32(mix32(0x811C9DC5u, (uint32_t)tile.w), (uint32_t)tile.x), (uint32_t)tile.y), (uint32_t)tile.z);
    h &= (kTileHashSlots - 1);
    for (int probe = 0; probe < kTileHashSlots; ++probe) {
        // device-coherent read: once a tile is in, nobody else reaches the compare-and-swap
        int32_t s = __hip_atomic_load(&tile_slots[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (s == 0) {
            if (hdr->n_tiles_raw > kMaxTiles) break;  // over the limit: reported by the ranking step
            const int32_t old = atomicCAS(&tile_slots[h], 0, idx + 1);
            if (old == 0) {
                const int pos = atomicAdd(&hdr->n_tiles_raw, 1);
                if (pos < kMaxTiles) rep_leaves[pos] = idx;
                break;
            }
            s = old;
        }
        const int4 o = L.key[s - 1];
        if (o.w == tile.w && (o.x >> 9) == tile.x && (o.y >> 9) == tile.y && (o.z >> 9) == tile.z) break;
        h = (h + 1) & (kTileHashSlots - 1);
    }
}

__global__ void __launch_bounds__(kFindTilesThreads)
k_find_tiles(LeafList L, int32_t* __restrict__ tile_slots, int32_t* __restrict__ rep_leaves, GridHeader* hdr) {
    if (hdr->overflow) return;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int4 key = make_int4(0, 0, 0, 0);
    const bool has = leaf_at(L, hdr, idx, &key);
    find_tile_item(L, hdr, (int)idx, has, key, tile_slots, rep_leaves);
}

// Rank every tile among all tiles by (grid, signed tile i, j, k): its rank is its upper-node id
// (the run index M of Sec. 3.3 step 5).  O(T^2) comparisons; T is tiny for real scenes.
// `t` = global thread number of the launch.
__device__ __forceinline__ void rank_tile_item(const LeafList& L, const int32_t* __restrict__ rep_leaves, const GridPtrs& g,
                                               int t, int t_stride) {
    const int raw = g.hdr->n_tiles_raw;
    const int T = raw < kMaxTiles ? raw : kMaxTiles;
    if (t == 0) {
        int ov = 0;
        if (raw > kMaxTiles) ov |= 8;
        if (T > g.cap_upper) ov |= 1;
        g.hdr->n_upper = T;
        if (ov) atomicOr(&g.hdr->overflow, ov);
    }
    if (T > g.cap_upper) return;
    for (; t < T; t += t_stride) {
        const int4 me = L.key[rep_leaves[t]];
        const uint64_t key = tile_key(me.x << 3, me.y << 3, me.z << 3);
        int rank = 0;
        for (int o = 0; o < T; ++o) {
            const int4 ot = L.key[rep_leaves[o]];
            const uint64_t ko = tile_key(ot.x << 3, ot.y << 3, ot.z << 3);
            rank += (ot.w < me.w) || (ot.w == me.w && ko < key);
        }
        g.root_key[rank] = key;
        g.root_batch[rank] = me.w;
    }
}

__global__ void k_rank_tiles(LeafList L, const int32_t* __restrict__ rep_leaves, GridPtrs g) {
    if (g.hdr->overflow) return;
    rank_tile_item(L, rep_leaves, g, blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x);
}

// ---------------------------------------------------------------------------------- leaves -> tree
// The launches below are sized for the leaf capacity, which the leaves of a dense grid fill to a fifth: the number of
// workgroups is capped and they stride, because workgroups that only find out that there is nothing for them still
// cost some 0.3 us a thousand.
constexpr int kInsertMaxBlocks = 1024;

// One thread per distinct leaf: its bit in the lower node's child mask (step 11.3)
__global__ void k_insert_lower(LeafList L, GridPtrs g) {
    if (g.hdr->overflow) return;
    for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;; idx += (int64_t)gridDim.x * blockDim.x) {
        int4 key;
        if (!leaf_at(L, g.hdr, idx, &key)) return;
        const int u = L.node[idx];
        int l = -1;
        if (u >= 0)
            l = child_of(g.upper_mask + (size_t)u * kUpperWords, g.upper_prefix + (size_t)u * kUpperWords, upper_off(key.x << 3, key.y << 3, key.z << 3));
        if (l >= g.cap_lower) l = -1;
        L.node[idx] = l;
        if (l < 0) continue;
        const int off = lower_off(key.x << 3, key.y << 3, key.z << 3);
        atomicOr((unsigned long long*)(g.lower_mask + (size_t)l * kLowerWords + (off >> 6)), 1ull << (off & 63));
    }
}

// The leaf's final id is known: its mask moves into the leaf record, with the seven 9-bit inclusive word prefixes of
// Listing 1, origin and grid; its voxel count goes to a compact array for the scan that follows.  Eight threads per
// leaf, one per mask word, so that a leaf is read and written as 64 consecutive bytes (one thread per leaf: 64 lines
// touched by every one of 12 store instructions of a wave; 376 k leaves 51 us here and 23 in the scan that re-read them).
// The lower node comes from the launch before (LeafList::node): with the descent from the root made again, 376 k leaves took
// 40 us, now 26, 38 k 8.2, now 6.5.
__global__ void k_place_leaves(LeafList L, GridPtrs g, uint32_t* __restrict__ leaf_count) {
    if (g.hdr->overflow) return;
    const int w = threadIdx.x & 7;
    for (int64_t idx = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 3;; idx += ((int64_t)gridDim.x * blockDim.x) >> 3) {
        int4 key;
        if (!leaf_at(L, g.hdr, idx, &key)) return;           // the same for the eight threads of a leaf
        const uint64_t m = L.mask[(size_t)L.mask_idx[idx] * 8 + w];
        const int l = L.node[idx];
        int f = -1;
        if (l >= 0)
            f = child_of(g.lower_mask + (size_t)l * kLowerWords, g.lower_prefix + (size_t)l * kLowerWords,
                         lower_off(key.x << 3, key.y << 3, key.z << 3));
        uint32_t incl = (uint32_t)__popcll(m);
#pragma unroll
        for (int d = 1; d < 8; d <<= 1) {
            const uint32_t o = __shfl_up(incl, d, 8);
            if (w >= d) incl += o;
        }
        uint64_t pre = w < 7 ? (uint64_t)incl << (9 * w) : 0ull;
#pragma unroll
        for (int d = 1; d < 8; d <<= 1) pre |= (uint64_t)__shfl_xor((unsigned long long)pre, d, 8);
        if (f < 0 || f >= g.cap_leaf) continue;
        fx_leaf* lf = &g.leaf[f];
        lf->mask[w] = m;
        if (w < 4) reinterpret_cast<int32_t*>(lf->origin)[w] = w == 0 ? key.x << 3 : w == 1 ? key.y << 3 : w == 2 ? key.z << 3 : key.w;
        if (w == 4) lf->prefix = pre;
        if (w == 7) leaf_count[f] = incl;
    }
}

// LEVEL 0 for all leaves: thousands of leaves share every lower node, and atomics on one address queue up at
// memory one after the other.  A workgroup therefore collects the bits of its 1024 leaves in LDS copies of the
// first upper nodes' masks and sends each touched word to memory once, and only if memory does not show its bits
// already (a stale read only costs a redundant atomic); leaves of further upper nodes look before they update memory
// directly.  A scene around the origin of its coordinates has eight upper nodes, a batch eight per grid: with copies of
// four nodes and no look, 376 k leaves of a point cloud around the origin took 390 us here, now 19.  There are as many
// copies as nodes are possible (n_copies, 4 KB each), up to what a compute unit's LDS holds beside the tile table; with
// copies of twelve at most, 190 k leaves of two clouds around the origin took 113 us, now 13.
// Where the capacity is a guess and few nodes exist, the copies that stay unused cost nothing that shows (LDS for one
// workgroup a compute unit in the place of two): at most twelve -> all, in us, 980 k LiDAR voxels 6.1 -> 6.3, four and eight
// indoor scenes 7.6 -> 7.5, 25 -> 24, 1 M random voxels in four and eight grids 11.2 -> 11.5, 13.3 -> 14.9 (the whole build 804 -> 804),
// four LiDAR scans around the origin 18 -> 11.
constexpr int kInsertUpperThreads = 1024;
constexpr int kAggUpper = 38;
// With at most kRankInBlock root tiles possible (the capacity of the upper level says so) the launch that ranks the
// tiles is dropped: every workgroup ranks them itself into LDS (a handful of comparisons) and looks its leaves up
// there; the first workgroup also writes the root table and the count for the launches that follow.
constexpr int kRankInBlock = 72;
__global__ void __launch_bounds__(kInsertUpperThreads) k_insert_upper(LeafList L, GridPtrs g,
                                                                       const int32_t* __restrict__ rep_leaves, int rank_here, int n_copies) {
    extern __shared__ __align__(16) unsigned long long bits[];
    __shared__ uint64_t tile_keys[kRankInBlock], ranked_key[kRankInBlock];
    __shared__ int32_t tile_batch[kRankInBlock], ranked_batch[kRankInBlock];
    if (g.hdr->overflow) return;
    const uint64_t* root_key = g.root_key;
    const int32_t* root_batch = g.root_batch;
    int n_upper;
    if (rank_here) {
        const int raw = g.hdr->n_tiles_raw;
        const int T = raw < kMaxTiles ? raw : kMaxTiles;
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            int ov = 0;
            if (raw > kMaxTiles) ov |= 8;
            if (T > g.cap_upper) ov |= 1;
            g.hdr->n_upper = T;
            if (ov) atomicOr(&g.hdr->overflow, ov);
        }
        if (T > g.cap_upper) return;              // cap_upper <= kRankInBlock on this path
        if ((int)threadIdx.x < T) {
            const int4 me = L.key[rep_leaves[threadIdx.x]];
            tile_keys[threadIdx.x] = tile_key(me.x << 3, me.y << 3, me.z << 3);
            tile_batch[threadIdx.x] = me.w;
        }
        __syncthreads();
        if ((int)threadIdx.x < T) {
            const uint64_t key = tile_keys[threadIdx.x];
            const int32_t b = tile_batch[threadIdx.x];
            int rank = 0;
            for (int o = 0; o < T; ++o) rank += (tile_batch[o] < b) || (tile_batch[o] == b && tile_keys[o] < key);
            ranked_key[rank] = key;
            ranked_batch[rank] = b;
            if (blockIdx.x == 0) { g.root_key[rank] = key; g.root_batch[rank] = b; }
        }
        n_upper = T;
        root_key = ranked_key;
        root_batch = ranked_batch;
    } else {
        n_upper = g.hdr->n_upper;
    }
    const int n_agg_words = (n_upper < n_copies ? n_upper : n_copies) * kUpperWords;
    for (int e = threadIdx.x; e < n_agg_words; e += kInsertUpperThreads) bits[e] = 0ull;
    __syncthreads();
    const int64_t idx = (int64_t)blockIdx.x * kInsertUpperThreads + threadIdx.x;
    int4 key;
    if (leaf_at(L, g.hdr, idx, &key)) {
        const int i = key.x << 3, j = key.y << 3, k = key.z << 3;
        const int u = find_upper_short(root_key, root_batch, n_upper, key.w, tile_key(i, j, k));
        L.node[idx] = u;
        if (u >= 0) {
            const int off = upper_off(i, j, k);
            const int word = u * kUpperWords + (off >> 6);
            const unsigned long long bit = 1ull << (off & 63);
            if (word < n_agg_words) atomicOr(&bits[word], bit);
            else if (!(g.upper_mask[word] & bit)) atomicOr((unsigned long long*)g.upper_mask + word, bit);
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < n_agg_words; e += kInsertUpperThreads) {
        const unsigned long long v = bits[e];
        if (v && (v & ~g.upper_mask[e])) atomicOr((unsigned long long*)g.upper_mask + e, v);
    }
}

// ---------------------------------------------------------------------------------- popcount scans
// which level's masks a scan runs over
struct LevelScan {
    const uint64_t* words;
    uint32_t* prefix;
    const int32_t* n_nodes;   // device count of nodes at this level
    int words_per_node;
    int32_t* n_children;      // device count to write (next level)
    int32_t child_cap;
    int32_t overflow_bit;
};

// Single-pass scans over several workgroups.  Each scan has a ticket counter and one word per workgroup (both
// start at zero).  A workgroup takes the next chunk in the order in which workgroups start running, publishes its
// chunk's total as total + 1 in its word with one device-scope store -- the word carries the value, so no fence is
// needed -- and then adds up the words of the chunks before it, waiting for those not yet written.  It only ever
// waits for workgroups that started before it and that publish before they wait themselves, so every wait ends;
// the wait is bounded all the same and an expired one is reported through the overflow word (bit 7).
struct ScanSync {
    uint32_t* ticket;
    uint32_t* sums;
};
constexpr int kScanSpinLimit = 1 << 20;

// the workgroup's chunk, or -1 when an earlier step of the build has failed (one thread decides for all) or when the
// launch, sized for the capacity, has more workgroups than there are chunks: those leave without a ticket, whose
// updates run one after the other at memory (20 ns each: 1222 of them were most of the leaf scan of 376 k leaves)
__device__ __forceinline__ int ordered_chunk(uint32_t* ticket, const GridHeader* hdr, int64_t n_chunks) {
    __shared__ int chunk;
    if (blockIdx.x >= (n_chunks > 0 ? n_chunks : 1)) return -1;
    if (threadIdx.x == 0) chunk = hdr->overflow ? -1 : (int)atomicAdd(ticket, 1u);
    __syncthreads();
    return chunk;
}

// publishes `total` as the sum of chunk `mine`; returns the sum of the chunks before it (to every thread)
__device__ __forceinline__ uint64_t publish_and_sum_before(const ScanSync& y, int mine, uint32_t total, GridHeader* hdr) {
    __shared__ unsigned long long acc;
    if (threadIdx.x == 0) {
        acc = 0ull;
        __hip_atomic_store(&y.sums[mine], total + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    unsigned long long sb = 0;
    for (int i = threadIdx.x; i < mine; i += blockDim.x) {
        uint32_t v = 0;
        for (int spin = 0; spin < kScanSpinLimit; ++spin) {
            v = __hip_atomic_load(&y.sums[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (v) break;
            __builtin_amdgcn_s_sleep(2);
        }
        if (!v) { atomicOr(&hdr->overflow, 128); v = 1u; }
        sb += v - 1u;
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) sb += (unsigned long long)__shfl_xor((long long)sb, d);
    if ((threadIdx.x & 63) == 0 && sb) atomicAdd(&acc, sb);
    __syncthreads();
    const uint64_t before = acc;
    __syncthreads();
    return before;
}

// exclusive popcount prefix per mask word over all nodes of a level; the last chunk writes the number of children
__global__ void __launch_bounds__(kScanThreads) k_scan_words(LevelScan s, GridHeader* hdr, ScanSync y) {
    const int64_t n_words = (int64_t)(*s.n_nodes) * s.words_per_node;
    const int chunk = ordered_chunk(y.ticket, hdr, (n_words + kWordChunk - 1) / kWordChunk);
    if (chunk < 0) return;
    const int64_t base = (int64_t)chunk * kWordChunk;
    if (base >= n_words && chunk != 0) return;
    const int64_t w0 = base + (int64_t)threadIdx.x * kWordsPerThread;
    uint32_t pc[kWordsPerThread];
    uint32_t sum = 0;
#pragma unroll
    for (int q = 0; q < kWordsPerThread; ++q) {
        pc[q] = (w0 + q < n_words) ? (uint32_t)__popcll(s.words[w0 + q]) : 0u;
        sum += pc[q];
    }
    uint32_t total;
    uint32_t run = block_exclusive_scan(sum, &total);
    const uint64_t before = publish_and_sum_before(y, chunk, total, hdr);
    run += (uint32_t)before;
#pragma unroll
    for (int q = 0; q < kWordsPerThread; ++q) {
        if (w0 + q < n_words) s.prefix[w0 + q] = run;
        run += pc[q];
    }
    if (threadIdx.x == 0 && base + kWordChunk >= n_words) {
        const uint64_t all = before + total;
        *s.n_children = (int32_t)(all < (uint64_t)INT32_MAX ? all : (uint64_t)INT32_MAX);
        if ((int64_t)all > s.child_cap) atomicOr(&hdr->overflow, s.overflow_bit);
    }
}

// First voxel index of every grid of the batch (leaves are ordered by grid): the thread that owns
// the first leaf of a grid writes the entries of that grid and of the empty grids before it; the
// owner of the last leaf writes the entries after it.  (The buffer starts zeroed: no leaves, all 0.)
__device__ __forceinline__ void note_vox_base(const fx_leaf* __restrict__ leaf, int64_t l, int64_t n_leaf, int64_t offset,
                                              int64_t n_voxels, int64_t* __restrict__ vox_base, int B) {
    if (B == 1) {      // a single grid: its bases are 0 (the buffer's initial value) and the voxel count, no record is read
        if (l == n_leaf - 1) vox_base[1] = n_voxels;
        return;
    }
    const int bcur = leaf[l].batch;
    const int bprev = l ? leaf[l - 1].batch : -1;
    for (int b = bprev + 1; b <= bcur; ++b) vox_base[b] = offset;
    if (l == n_leaf - 1)
        for (int b = bcur + 1; b <= B; ++b) vox_base[b] = n_voxels;
}

// Leaf level: mOffset = exclusive scan of the leaves' active-voxel counts.
__global__ void __launch_bounds__(kScanThreads) k_scan_leaves(fx_leaf* __restrict__ leaf, const uint32_t* __restrict__ leaf_count,
                                                               GridHeader* hdr, ScanSync y,
                                                               int64_t* __restrict__ vox_base, int B) {
    const int64_t n_leaf = hdr->n_leaf;
    const int chunk = ordered_chunk(y.ticket, hdr, (n_leaf + kLeafChunk - 1) / kLeafChunk);
    if (chunk < 0) return;
    const int64_t base = (int64_t)chunk * kLeafChunk;
    if (base >= n_leaf && chunk != 0) return;
    const int64_t l0 = base + (int64_t)threadIdx.x * kLeavesPerThread;
    uint32_t cnt[kLeavesPerThread];
    uint32_t sum = 0;
#pragma unroll
    for (int q = 0; q < kLeavesPerThread; ++q) {
        cnt[q] = l0 + q < n_leaf ? leaf_count[l0 + q] : 0u;
        sum += cnt[q];
    }
    {   // voxels that sit in locally dense leaves, summed over the grid
        uint32_t dense = 0;
#pragma unroll
        for (int q = 0; q < kLeavesPerThread; ++q) dense += cnt[q] >= (uint32_t)kDenseLeafVoxels ? cnt[q] : 0u;
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) dense += (uint32_t)__shfl_xor((int)dense, d);
        if ((threadIdx.x & 63) == 0 && dense) atomicAdd((unsigned long long*)&hdr->n_voxels_dense, (unsigned long long)dense);
    }
    uint32_t total;
    const uint32_t local = block_exclusive_scan(sum, &total);
    const uint64_t before = publish_and_sum_before(y, chunk, total, hdr);
    const bool last = base + kLeafChunk >= n_leaf;
    const int64_t all = (int64_t)(before + total);      // the grid's voxel count, in the last chunk
    int64_t run = (int64_t)before + local;
#pragma unroll
    for (int q = 0; q < kLeavesPerThread; ++q) {
        if (l0 + q < n_leaf) {
            leaf[l0 + q].offset = run;
            // only the last chunk holds the last leaf, the one reader of the grand total
            note_vox_base(leaf, l0 + q, n_leaf, run, all, vox_base, B);
        }
        run += cnt[q];
    }
    if (threadIdx.x == 0 && last) {
        hdr->n_voxels = all;
        if (all > (int64_t)INT32_MAX) atomicOr(&hdr->overflow, 16);
    }
}

// The build's one read-back (Sec. 3.3 step 10): counts and per-grid voxel bases, written by the
// device straight into pinned host memory -- one tiny launch instead of two copy-engine transfers.
// The last word written is a ticket the host polls for, which returns sooner than a stream wait.
__global__ void k_publish(const GridHeader* __restrict__ hdr, const int64_t* __restrict__ vox_base, int B,
                          unsigned char* __restrict__ host, int32_t* __restrict__ host_ticket, int32_t ticket) {
    const int t = threadIdx.x;
    constexpr int kHdrWords = (int)(sizeof(GridHeader) / sizeof(int32_t));
    if (t < kHdrWords) reinterpret_cast<int32_t*>(host)[t] = reinterpret_cast<const int32_t*>(hdr)[t];
    for (int b = t; b <= B; b += blockDim.x) reinterpret_cast<int64_t*>(host + sizeof(GridHeader))[b] = vox_base[b];
    __threadfence_system();
    __syncthreads();
    if (t == 0) __hip_atomic_store(host_ticket, ticket, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ---------------------------------------------------------------------------------- small grids, one launch
// The passes above are a chain of a dozen launches of 3-6 us each, most of it latency, whatever the size: 10 k rows took
// 57 us, in this one launch 23.  Up to kSmallRows rows (or fine leaves, for a coarse grid) one workgroup does the whole build in LDS.  Its
// leaves are collected in an LDS table of (leaf, 512-bit mask); then they are simply sorted -- the fields of a leaf's
// coordinate in tree order (grid; root tile; upper offset; lower offset) are one integer -- and node numbers fall out as
// scans of the places where a prefix of that integer changes.  Counts and ranges go straight to the host.  What it does
// not hold -- more than kSmallSlots leaves, coordinates beyond 2^18, more than 16 grids, more root tiles than the
// capacity -- sets overflow bit 8 and the build starts over with the passes.  A leaf that finds no slot within kSmallProbes
// steps is the first sign of that, and every thread then stops: rows that walked a full table to its end, or the long
// runs of linear probing near it, took milliseconds (16 k rows alone in their leaves 5 ms, 1728 leaves 240 us where the
// passes take 110).  Steps grow by one each time: 1300 leaves need up to 16 of them, 1800 up to 64.  A row stops at 16,
// because beyond 1300 leaves the passes are as fast, and an attempt given up then costs 10 us; a fine leaf, of which a
// thread has a few only, at 64.  A coarse grid has no more leaves than the fine one; the leaves of surfaces join three or
// more to one (LiDAR scenes 2.8 to 3.5, indoor scenes, sheets and spheres 3.7 to 5.8), leaves of one or two voxels may not.
constexpr int kSmallThreads = 1024, kSmallSlots = 2048, kSmallRows = 16384;
constexpr int kSmallProbes = 16, kSmallProbesCoarse = 64;
constexpr int kSmallLeaves = 1700, kSmallFineLeaves = 6144, kFilledVoxels = 4;      // mean voxels of a leaf from which on neighbours are likely
constexpr size_t kSmallLds = sizeof(uint64_t) * 9 * kSmallSlots;
enum SmallSource { kSmallIjk = 0, kSmallPoints = 1, kSmallCoarse = 2 };

template <int SOURCE>
__global__ void __launch_bounds__(kSmallThreads)
k_small_grid(const RowSource rows, int n_rows, const BatchRanges joff, int B, TreeView fine, GridPtrs g, unsigned char* __restrict__ host,
             int32_t* __restrict__ host_ticket, int32_t ticket) {
    extern __shared__ __align__(16) unsigned char small_lds[];
    unsigned long long* slot = reinterpret_cast<unsigned long long*>(small_lds);     // [kSmallSlots] leaf (0: empty), later the sorted keys
    unsigned long long* mask = slot + kSmallSlots;                                   // [kSmallSlots][8]
    __shared__ int overflow, n_bad;
    __shared__ unsigned long long dense;
    const int tid = threadIdx.x;
    for (int e = tid; e < kSmallSlots * 9 / 2; e += kSmallThreads) reinterpret_cast<ulonglong2*>(small_lds)[e] = make_ulonglong2(0ull, 0ull);
    if (tid == 0) { overflow = 0; n_bad = 0; dense = 0ull; }
    __syncthreads();

    // ---- leaves: leaf coordinates biased by 2^15 (16 bits each), grid, a set top bit
    constexpr int half = 1 << 15;
    auto gave_up = [&]() { return __hip_atomic_load(&overflow, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != 0; };
    auto give_up = [&]() { __hip_atomic_store(&overflow, 256, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };
    auto claim = [&](int li, int lj, int lk, int b) -> int {
        if (((uint32_t)(li + half) | (uint32_t)(lj + half) | (uint32_t)(lk + half)) >= 2u * half) { give_up(); return -1; }
        const unsigned long long self = (1ull << 63) | ((unsigned long long)(uint32_t)b << 48) | ((unsigned long long)(uint32_t)(li + half) << 32) |
                                        ((unsigned long long)(uint32_t)(lj + half) << 16) | (unsigned long long)(uint32_t)(lk + half);
        uint32_t h = leaf_hash(b, li, lj, lk) & (kSmallSlots - 1);
        for (int probe = 0; probe < (SOURCE == kSmallCoarse ? kSmallProbesCoarse : kSmallProbes); ++probe) {
            unsigned long long s = __hip_atomic_load(&slot[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (s == 0ull) s = atomicCAS(&slot[h], 0ull, self);
            if (s == 0ull || s == self) return (int)h;
            if ((probe & 7) == 7 && gave_up()) return -1;
            h = (h + probe + 1) & (kSmallSlots - 1);
        }
        give_up();
        return -1;
    };
    if (SOURCE == kSmallCoarse) {
        for (int f = tid; f < n_rows && !gave_up(); f += kSmallThreads) {
            const fx_leaf* lf = fine.leaf + f;
            const CoarsePiece c = coarse_piece(lf);
            const int h = claim(c.li, c.lj, c.lk, lf->batch);
            if (h < 0) continue;
#pragma unroll
            for (int a = 0; a < 4; ++a)
                if (c.word[a]) atomicOr(&mask[h * 8 + c.first_word + a], (unsigned long long)c.word[a]);
        }
    } else {
        int bad = 0;
        constexpr int kGroups = kSmallRows / (4 * kSmallThreads);
        int3 v[kGroups][4];
        int n[kGroups];
#pragma unroll
        for (int c = 0; c < kGroups; ++c)        // all of the thread's rows are requested at once
            n[c] = load_four_rows<SOURCE == kSmallPoints>(rows, n_rows, 4 * (c * kSmallThreads + tid), v[c], bad);
#pragma unroll
        for (int c = 0; c < kGroups; ++c) {
            if (gave_up()) break;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int b = q < n[c] ? find_batch(joff, B, 4 * (c * kSmallThreads + tid) + q) : -1;
                if (b < 0) continue;
                const int3 x = v[c][q];
                const int h = claim(x.x >> 3, x.y >> 3, x.z >> 3, b);
                if (h >= 0) atomicOr(&mask[h * 8 + (x.x & 7)], 1ull << (((x.y & 7) << 3) | (x.z & 7)));
            }
        }
        if (SOURCE == kSmallPoints && bad) atomicAdd(&n_bad, bad);
    }
    __syncthreads();
    if (overflow) {                            // the same for all threads: nothing sets it between here and the next barrier
        if (tid == 0) {
            GridHeader hdr{};
            hdr.overflow = overflow;
            *g.hdr = hdr;
            *reinterpret_cast<GridHeader*>(host) = hdr;
            __threadfence_system();
            __hip_atomic_store(host_ticket, ticket, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        return;
    }

    // ---- keys: [grid 4][tile 3 x 7][upper offset 3 x 5][lower offset 3 x 4][slot 11], compacted, padded to a power of two
    unsigned long long key[2];
    uint32_t have = 0;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const unsigned long long s = slot[2 * tid + q];
        key[q] = ~0ull;
        if (s == 0ull) continue;
        ++have;
        const uint32_t a[3] = {(uint32_t)(s >> 32) & 0xFFFFu, (uint32_t)(s >> 16) & 0xFFFFu, (uint32_t)s & 0xFFFFu};
        unsigned long long k = (s >> 48) & 15ull;
#pragma unroll
        for (int d = 0; d < 3; ++d) k = (k << 7) | (a[d] >> 9);
#pragma unroll
        for (int d = 0; d < 3; ++d) k = (k << 5) | ((a[d] >> 4) & 31u);
#pragma unroll
        for (int d = 0; d < 3; ++d) k = (k << 4) | (a[d] & 15u);
        key[q] = (k << 11) | (uint32_t)(2 * tid + q);
    }
    uint32_t n_leaf_u;
    uint32_t at = block_exclusive_scan(have, &n_leaf_u);
    const int n_leaf = (int)n_leaf_u;
    int padded = 64;
    while (padded < n_leaf) padded <<= 1;
    for (int e = tid; e < padded; e += kSmallThreads) slot[e] = ~0ull;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q)
        if (key[q] != ~0ull) slot[at++] = key[q];
    __syncthreads();
    for (int size = 2; size <= padded; size <<= 1)
        for (int step = size >> 1; step > 0; step >>= 1) {
            if (tid < padded / 2) {
                const int i = 2 * tid - (tid & (step - 1)), j = i + step;
                const unsigned long long x = slot[i], y = slot[j];
                if ((x > y) == ((i & size) == 0)) { slot[i] = y; slot[j] = x; }
            }
            // a wave's 64 compare-exchanges of a step below 64 stay within the wave's own 128 elements
            if (step > 64 || (step == 1 && size >= 128)) __syncthreads();
            else { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup"); __builtin_amdgcn_wave_barrier(); }
        }
    __syncthreads();

    // ---- node numbers: thread = two consecutive leaves
    unsigned long long prev = tid ? slot[2 * tid - 1] : ~0ull;
    uint32_t heads = 0, cnt[2] = {0, 0};
    uint64_t pre[2] = {0, 0};
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int p = 2 * tid + q;
        key[q] = p < padded ? slot[p] : ~0ull;
        if (p >= n_leaf) continue;
        const unsigned long long before = q ? key[0] : prev;
        const bool first = p == 0;
        heads += (first || (key[q] >> 23) != (before >> 23)) ? 1u : 0u;                 // a new lower node
        heads += (first || (key[q] >> 38) != (before >> 38)) ? (1u << 16) : 0u;         // a new upper node
        const unsigned long long* m = mask + (size_t)(key[q] & (kSmallSlots - 1)) * 8;
        uint32_t acc = 0;
#pragma unroll
        for (int w = 0; w < 8; ++w) {
            acc += (uint32_t)__popcll(m[w]);
            if (w < 7) pre[q] |= (uint64_t)acc << (9 * w);
        }
        cnt[q] = acc;
    }
    {
        uint32_t d = (cnt[0] >= (uint32_t)kDenseLeafVoxels ? cnt[0] : 0u) + (cnt[1] >= (uint32_t)kDenseLeafVoxels ? cnt[1] : 0u);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) d += (uint32_t)__shfl_xor((int)d, o);
        if ((tid & 63) == 0 && d) atomicAdd(&dense, (unsigned long long)d);
    }
    uint32_t all_heads, n_vox;
    uint32_t nodes = block_exclusive_scan(heads, &all_heads);
    uint32_t offset = block_exclusive_scan(cnt[0] + cnt[1], &n_vox);
    const int n_lower = (int)(all_heads & 0xFFFFu), n_upper = (int)(all_heads >> 16);
    if (tid == 0 && (n_upper > g.cap_upper || n_lower > g.cap_lower || n_leaf > g.cap_leaf)) overflow = 256;
    __syncthreads();
    const bool fits = overflow == 0;
    if (fits) {
        for (int e = tid; e < n_upper * kUpperWords; e += kSmallThreads) g.upper_mask[e] = 0ull;
        for (int e = tid; e < n_lower * kLowerWords; e += kSmallThreads) g.lower_mask[e] = 0ull;
        for (int b = tid; b <= B; b += kSmallThreads) g.vox_base[b] = 0;
        __builtin_amdgcn_s_waitcnt(0);         // the zeros have arrived before other waves update them
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int p = 2 * tid + q;
            if (p >= n_leaf) continue;
            const unsigned long long k = key[q], before = q ? key[0] : prev;
            const bool first = p == 0;
            const bool new_lower = first || (k >> 23) != (before >> 23), new_upper = first || (k >> 38) != (before >> 38);
            nodes += (new_lower ? 1u : 0u) + (new_upper ? (1u << 16) : 0u);
            const int l = (int)(nodes & 0xFFFFu) - 1, u = (int)(nodes >> 16) - 1;
            const int loff = (int)(k >> 11) & 4095, uoff = (int)(k >> 23) & 32767;
            const int b = (int)(k >> 59);
            int o[3];
#pragma unroll
            for (int d = 0; d < 3; ++d) {      // field d of every level, most significant first
                const int tile = (int)(k >> (38 + 7 * (2 - d))) & 127, uo = (uoff >> (5 * (2 - d))) & 31, lo = (loff >> (4 * (2 - d))) & 15;
                o[d] = ((((tile << 9) | (uo << 4) | lo) - half) * 8);
            }
            if (new_upper) { g.root_key[u] = tile_key(o[0], o[1], o[2]); g.root_batch[u] = b; }
            if (new_lower) {
                atomicOr((unsigned long long*)(g.upper_mask + (size_t)u * kUpperWords + (uoff >> 6)), 1ull << (uoff & 63));
                if (first || (k >> 29) != (before >> 29)) g.upper_prefix[(size_t)u * kUpperWords + (uoff >> 6)] = (uint32_t)l;
            }
            atomicOr((unsigned long long*)(g.lower_mask + (size_t)l * kLowerWords + (loff >> 6)), 1ull << (loff & 63));
            if (first || (k >> 17) != (before >> 17)) g.lower_prefix[(size_t)l * kLowerWords + (loff >> 6)] = (uint32_t)p;
            fx_leaf* lf = g.leaf + p;
            const unsigned long long* m = mask + (size_t)(k & (kSmallSlots - 1)) * 8;
#pragma unroll
            for (int w = 0; w < 8; ++w) lf->mask[w] = m[w];
            lf->prefix = pre[q];
            lf->offset = offset;
            lf->origin[0] = o[0]; lf->origin[1] = o[1]; lf->origin[2] = o[2];
            lf->batch = b;
            // first voxel of this grid and of the empty ones before it; after the last leaf, of those behind
            for (int e = first ? 0 : (int)(before >> 59) + 1; e <= b; ++e) g.vox_base[e] = offset;
            if (p == n_leaf - 1)
                for (int e = b + 1; e <= B; ++e) g.vox_base[e] = n_vox;
            offset += cnt[q];
        }
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (tid == 0) {
        GridHeader hdr;
        hdr.n_tiles_raw = n_upper; hdr.n_upper = n_upper; hdr.n_lower = n_lower; hdr.n_leaf = n_leaf;
        hdr.overflow = overflow; hdr.n_leaf_raw = n_leaf; hdr.n_bad = n_bad; hdr.pad = 0;
        hdr.n_voxels = n_vox; hdr.n_voxels_dense = (int64_t)dense;
        *g.hdr = hdr;
        *reinterpret_cast<GridHeader*>(host) = hdr;
    }
    if (tid >= 64) return;                     // the first wave tells the host: B <= 16
    if (fits && tid <= B) reinterpret_cast<int64_t*>(host + sizeof(GridHeader))[tid] = g.vox_base[tid];
    __threadfence_system();
    __builtin_amdgcn_wave_barrier();
    if (tid == 0) __hip_atomic_store(host_ticket, ticket, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// ---------------------------------------------------------------------------------- queries
// A wave takes eight consecutive leaves, lane = (leaf, word of its mask): eight lanes' popcounts give every word its
// place among the leaf's voxels, and the leaves' voxels are consecutive by construction (offset), so the wave's voxels
// are one contiguous run of outputs.  Every lane lists the set bits of its own word in LDS (leaf number and position);
// then lane = voxel, one 12-byte store each, whole lines per wave.  A wave per leaf with a ballot-style listing (lane =
// bit) took six times the instructions on leaves of ~25 voxels: 9 M voxels in 376 k leaves took 155 us, now 34 (144 MB written).
constexpr int kIjkLeaves = 8, kIjkWaves = 4;
typedef __attribute__((ext_vector_type(3), aligned(4))) int32_t i32x3_u;
__global__ void __launch_bounds__(64 * kIjkWaves) k_grid_ijk(TreeView t, int32_t* __restrict__ ijk_out, int32_t* __restrict__ jidx_out,
                                                             int shift) {
    __shared__ uint16_t active[kIjkWaves][kIjkLeaves * 512];
    __shared__ int4 head[kIjkWaves][kIjkLeaves];              // origin and grid of each leaf
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t f0 = ((int64_t)blockIdx.x * kIjkWaves + wave) * kIjkLeaves;
    if (f0 >= t.n_leaf) return;
    const int l = lane >> 3, w = lane & 7;
    const bool has = f0 + l < t.n_leaf;
    const fx_leaf* lf = t.leaf + (has ? f0 + l : f0);
    uint64_t m = has ? lf->mask[w] : 0ull;
    if (w == 0) head[wave][l] = make_int4(lf->origin[0], lf->origin[1], lf->origin[2], lf->batch);
    const int64_t first = t.leaf[f0].offset;                  // uniform
    // place of the lane's first voxel in the run: words in lane order are voxels in index order
    const int cnt = __popcll(m);
    int incl = cnt;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int o = __shfl_up(incl, d);
        if (lane >= d) incl += o;
    }
    const int n = __shfl(incl, 63);
    int at = incl - cnt;
    while (m) {
        active[wave][at++] = (uint16_t)(lane * 64 + __ffsll((long long)m) - 1);    // leaf << 9 | word << 6 | bit
        m &= m - 1;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (int v = lane; v < n; v += 64) {
        const int pos = active[wave][v];
        const int4 o = head[wave][pos >> 9];
        i32x3_u c;
        c.x = (o.x + ((pos >> 6) & 7)) >> shift;
        c.y = (o.y + ((pos >> 3) & 7)) >> shift;
        c.z = (o.z + (pos & 7)) >> shift;
        *reinterpret_cast<i32x3_u*>(ijk_out + 3 * (first + v)) = c;
        if (jidx_out) jidx_out[first + v] = o.w;
    }
}

__global__ void k_ijk_to_index(TreeView t, const int32_t* __restrict__ ijk, const int32_t* __restrict__ jidx,
                               int64_t n, int32_t* __restrict__ out) {
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n) return;
    const int b = jidx ? jidx[r] : 0;
    int v = -1;
    if (b >= 0 && b < t.B) v = get_value(t, b, ijk[3 * r], ijk[3 * r + 1], ijk[3 * r + 2]);
    out[r] = v;
}

// ---------------------------------------------------------------------------------- host side
static size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

static void layout(fx_grid* g) {
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, 256); return o; };
    const size_t o_hdr = take(sizeof(GridHeader));
    const size_t o_vox = take(sizeof(int64_t) * ((size_t)g->B + 1));
    const size_t o_rk = take(sizeof(uint64_t) * g->cap_upper);
    const size_t o_rb = take(sizeof(int32_t) * g->cap_upper);
    const size_t o_um = take(sizeof(uint64_t) * kUpperWords * (size_t)g->cap_upper);
    const size_t o_up = take(sizeof(uint32_t) * kUpperWords * (size_t)g->cap_upper);
    const size_t o_lm = take(sizeof(uint64_t) * kLowerWords * (size_t)g->cap_lower);
    const size_t o_lp = take(sizeof(uint32_t) * kLowerWords * (size_t)g->cap_lower);
    const size_t o_lf = take(sizeof(fx_leaf) * (size_t)g->cap_leaf);
    g->buf_bytes = off;
    char* p = (char*)g->buf;
    if (!p) return;
    g->d_hdr = (GridHeader*)(p + o_hdr);
    g->d_vox_base = (int64_t*)(p + o_vox);
    g->d_root_key = (uint64_t*)(p + o_rk);
    g->d_root_batch = (int32_t*)(p + o_rb);
    g->d_upper_mask = (uint64_t*)(p + o_um);
    g->d_upper_prefix = (uint32_t*)(p + o_up);
    g->d_lower_mask = (uint64_t*)(p + o_lm);
    g->d_lower_prefix = (uint32_t*)(p + o_lp);
    g->d_leaf = (fx_leaf*)(p + o_lf);
}

static GridPtrs ptrs_of(const fx_grid* g) {
    GridPtrs q;
    q.hdr = g->d_hdr; q.vox_base = g->d_vox_base; q.root_key = g->d_root_key; q.root_batch = g->d_root_batch;
    q.upper_mask = g->d_upper_mask; q.upper_prefix = g->d_upper_prefix;
    q.lower_mask = g->d_lower_mask; q.lower_prefix = g->d_lower_prefix; q.leaf = g->d_leaf;
    q.cap_upper = g->cap_upper; q.cap_lower = g->cap_lower; q.cap_leaf = g->cap_leaf; q.B = g->B;
    return q;
}

static fx_status scan_level(const fx_grid* g, LevelScan s, int cap_nodes, ScanSync y, hipStream_t st) {
    const int64_t cap_words = (int64_t)cap_nodes * s.words_per_node;
    const int n_blocks = (int)std::max<int64_t>(1, (cap_words + kWordChunk - 1) / kWordChunk);
    k_scan_words<<<n_blocks, kScanThreads, 0, st>>>(s, g->d_hdr, y);
    FX_HIP_TRY(hipGetLastError());
    return FX_OK;
}

// The counts and ranges that the device writes into pinned host memory, and the ticket it writes last.
struct ReadBack {
    unsigned char* host = nullptr;
    int32_t* host_ticket = nullptr;
    int32_t ticket = 0;
    fx_status prepare(int B) {
        void* stage = nullptr;
        const size_t ticket_off = align_up(sizeof(GridHeader) + sizeof(int64_t) * ((size_t)B + 1), 64);
        FX_TRY(host_staging(&stage, ticket_off + 64));
        static thread_local int32_t next_ticket = 0;
        ticket = ++next_ticket == 0 ? ++next_ticket : next_ticket;   // never 0
        host = (unsigned char*)stage;
        host_ticket = reinterpret_cast<int32_t*>(host + ticket_off);
        *(volatile int32_t*)host_ticket = 0;
        return FX_OK;
    }
    hipError_t wait(hipStream_t st) const {
        // poll the ticket for a while (a few hundred microseconds at most for the sizes where latency
        // matters), then fall back to waiting for the stream, which also reports any device error
        volatile int32_t* t = host_ticket;
        bool seen = false;
        for (int spin = 0; spin < 200000 && !seen; ++spin) {
            seen = (*t == ticket);
            if (!seen) __builtin_ia32_pause();
        }
        const hipError_t e = seen ? hipSuccess : hipStreamSynchronize(st);
        std::atomic_thread_fence(std::memory_order_acquire);
        return e;
    }
    void take(fx_grid* g) const {
        memcpy(&g->hdr, host, sizeof(GridHeader));
        memcpy(g->h_vox_base, host + sizeof(GridHeader), sizeof(int64_t) * ((size_t)g->B + 1));
    }
};

// One attempt with the given node capacities.  On FX_OK, (*out)->hdr.overflow tells whether a
// capacity was too small (the counts found so far are valid up to the overflowing level).
constexpr int64_t kPartitionMinRows = 65536;   // below this the direct path's few kernels win

// Where the leaves of a grid come from when not from rows of voxel coordinates: the leaves of another grid
// (n_rows of build_attempt is then that grid's leaf count, and the direct path is taken).
struct LeafSource {
    enum Kind { kRows, kCoarsen, kPad, kSubdivide } kind = kRows;
    const fx_grid* grid = nullptr;
    int r = 0;                    // kPad: the padding
    int32_t* d_bad = nullptr;     // kPad, kSubdivide: counter of leaves beyond the int32 coordinate range
    int link_K = 0;               // kCoarsen: the grid becomes the output of a (link_K, 2) kernel map from `grid` (0: no)
};

static fx_status build_attempt(const RowSource& rows, int64_t n_rows, const BatchRanges& d_joff, int32_t B,
                               int cap_upper, int cap_lower, int cap_leaf, bool direct, hipStream_t st, fx_grid** out,
                               const LeafSource& from = LeafSource()) {
    fx_grid* g = new (std::nothrow) fx_grid();
    if (!g) { set_error("host allocation failed"); return FX_ENOMEM; }
    g->B = B; g->stream = st;
    g->cap_upper = std::max(cap_upper, 1); g->cap_lower = std::max(cap_lower, 1); g->cap_leaf = std::max(cap_leaf, 1);
    layout(g);
    fx_status rc = dev_alloc(&g->buf, g->buf_bytes, st);
    if (rc != FX_OK) { delete g; return rc; }
    layout(g);
    g->h_vox_base = (int64_t*)calloc((size_t)B + 1, sizeof(int64_t));

    // Leaf list capacity and the way to it.  Scratch layout:
    //   cleared by both paths:    [scan tickets and block words | tile table]
    //   cleared by the direct one [leaf table slots | leaf masks]
    //   not cleared:              [leaf keys | mask indices | tile representatives |
    //                              partitioned path: leaf masks, records, runs of the buckets, pieces]
    const bool partition = !direct && n_rows >= kPartitionMinRows;
    const int64_t max_items = std::max<int64_t>((int64_t)g->cap_lower * kLowerWords / kWordChunk,
                                                std::max<int64_t>((int64_t)g->cap_upper * kUpperWords / kWordChunk,
                                                                  (int64_t)g->cap_leaf / kLeafChunk)) + 2;
    size_t n_slots = 0;                       // direct path: table slots, masks indexed by slot
    const bool no_table = from.kind == LeafSource::kSubdivide;       // every leaf has one source: masks by (leaf, octant)
    if (!partition) { n_slots = 1024; while (n_slots < 2 * (size_t)g->cap_leaf) n_slots <<= 1; }
    if (no_table) n_slots = 0;
    // (a padded grid keeps the masks of the source grid's own leaves behind the table's)
    const size_t n_masks = partition ? (size_t)g->cap_leaf
                         : no_table ? 8 * (size_t)n_rows : n_slots + (from.kind == LeafSource::kPad ? (size_t)n_rows : 0);
    if (n_masks > 0x7FFFFFFFull) { fx_grid_destroy(g); set_error("grid build: too many leaves"); return FX_ERANGE; }
    // Buckets of 1500 to 3000 rows from 800 k rows on: fewer, fuller buckets give the row pass longer runs per bucket and the
    // leaf pass fewer workgroups that each clear a 64 KB table (1 M rows: 98 us with ~1000 rows per bucket, 90 with
    // ~2000, 91 with ~4000, 107 with ~8000, which leaves half the compute units without a bucket; four grids of
    // 1.07 M rows: 140 / 123 / 117 / 111 us for ~500 / 1000 / 2000 / 4000).
    // At least one bucket per compute unit: with 128 of 1770 rows half the chip had none, and the buckets of sparse points
    // overflowed their tables (226 k points in 190 k leaves: 60 -> 21 us for the leaf pass).
    int n_buckets = 256;
    while (n_buckets < kMaxBuckets && (int64_t)n_buckets * kRowsPerBucket < n_rows) n_buckets <<= 1;
    // Rows of a piece: 4096, or 8192 and 16384 once that still makes two pieces per compute unit: fewer pieces are fewer, longer
    // runs in the leaf pass (10 M points, pieces of 8192 / 16384: 77 / 80 us for the row pass, 110 / 85 for the leaf pass).
    const int quads = n_rows >= (int64_t)2 * 16384 * compute_units() ? 4 : n_rows >= (int64_t)2 * 8192 * compute_units() ? 2 : 1;
    const int part_chunk = kPartThreads * 4 * quads;
    const int n_part_wg = (int)((n_rows + part_chunk - 1) / part_chunk);
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, 256); return o; };
    const size_t o_sync = take(sizeof(uint32_t) * 3 * (64 + (size_t)max_items));   // three scans: a ticket, then the words
    const size_t o_tslot = take(sizeof(int32_t) * kTileHashSlots);
    const size_t clear_bytes_head = off;
    const size_t o_slots = take(sizeof(int32_t) * n_slots);
    const size_t clear_bytes_slots = off;
    const size_t o_mask = take(sizeof(uint64_t) * 8 * n_masks);
    // the padded grid's masks are stored whole, the other direct builds OR theirs together
    const bool whole_masks = from.kind == LeafSource::kPad || from.kind == LeafSource::kSubdivide;
    const size_t clear_bytes = partition ? clear_bytes_head : (whole_masks ? clear_bytes_slots : off);
    const size_t o_key = take(sizeof(int4) * (size_t)g->cap_leaf);
    const size_t o_midx = take(sizeof(int32_t) * (size_t)g->cap_leaf);
    const size_t o_node = take(sizeof(int32_t) * (size_t)g->cap_leaf);
    const size_t o_lcnt = take(sizeof(uint32_t) * (size_t)g->cap_leaf);
    const size_t o_rep = take(sizeof(int32_t) * kMaxTiles);
    const int64_t n_records = (int64_t)n_part_wg * part_chunk;
    const size_t o_rec = take(partition ? sizeof(int4) * (size_t)n_records : 0);
    const size_t o_starts = take(partition ? sizeof(uint16_t) * (size_t)(n_buckets + 1) * n_part_wg : 0);
    const size_t o_info = take(partition ? sizeof(int32_t) * (size_t)n_part_wg : 0);
    void* scratch = nullptr;
    rc = dev_alloc(&scratch, off, st);
    if (rc != FX_OK) { fx_grid_destroy(g); return rc; }
    char* sp = (char*)scratch;
    LeafList L;
    L.mask = (uint64_t*)(sp + o_mask);
    L.key = (int4*)(sp + o_key);
    L.mask_idx = (int32_t*)(sp + o_midx);
    L.node = (int32_t*)(sp + o_node);
    L.cap = g->cap_leaf;
    int32_t* d_tile_slots = (int32_t*)(sp + o_tslot);
    int32_t* d_slots = (int32_t*)(sp + o_slots);
    int32_t* d_rep = (int32_t*)(sp + o_rep);
    uint32_t* d_leaf_count = (uint32_t*)(sp + o_lcnt);
    auto scan_sync = [&](int which) {
        uint32_t* base = (uint32_t*)(sp + o_sync) + (size_t)which * (64 + (size_t)max_items);
        return ScanSync{base, base + 64};
    };
    uint64_t* d_records = (uint64_t*)(sp + o_rec);         // two words per row (the second: wide rows only)
    uint16_t* d_starts = (uint16_t*)(sp + o_starts);
    int32_t* d_info = (int32_t*)(sp + o_info);

    auto fail = [&](fx_status s) { dev_free(scratch, st); fx_grid_destroy(g); return s; };
#define FX_TRY_OR_FAIL(expr) do { hipError_t _e = (expr); if (_e != hipSuccess) { \
        set_error("%s failed: %s", #expr, hipGetErrorString(_e)); return fail(FX_EDEVICE); } } while (0)

    // header, bases, root table and the child masks start at zero; the leaf records (most of the buffer) do not
    // need to: every field of every leaf that exists is written by the build.  The partitioned path clears in its
    // first kernel, the direct path (small inputs) with two fills.
    const size_t grid_clear_bytes = (size_t)((char*)g->d_leaf - (char*)g->buf);
    const bool kernel_clears = partition && n_rows > 0 && B > 0;
    if (!kernel_clears) {
        ProfScope ps(kProfMemset, st);
        FX_TRY_OR_FAIL(hipMemsetAsync(g->buf, 0, grid_clear_bytes, st));
        FX_TRY_OR_FAIL(hipMemsetAsync(scratch, 0, clear_bytes, st));
    }
    const GridPtrs q = ptrs_of(g);
    if (n_rows > 0 && B > 0) {
        const unsigned nb_leaf = (unsigned)std::min<int64_t>(((int64_t)g->cap_leaf + 255) / 256, kInsertMaxBlocks);
        const unsigned nb_place = (unsigned)std::min<int64_t>(((int64_t)g->cap_leaf + 31) / 32, 4 * kInsertMaxBlocks);
        const unsigned nb_leaf_1024 = (unsigned)(((int64_t)g->cap_leaf + 1023) / 1024);
        if (partition) {
            const uint32_t bucket_mask = (uint32_t)n_buckets - 1;
            const size_t lds = sizeof(uint64_t) * part_chunk + sizeof(uint32_t) * n_buckets;
            ClearRanges clr;
            clr.p[0] = (uint4*)g->buf; clr.n16[0] = (uint32_t)(grid_clear_bytes / 16);
            clr.p[1] = (uint4*)scratch; clr.n16[1] = (uint32_t)(clear_bytes / 16);
#define FX_SORT(POINTS, QUADS)                                                                                          \
    if ((rows.xyz != nullptr) == POINTS && quads == QUADS) {                                                           \
        if (lds > 64 * 1024) FX_TRY_OR_FAIL(hipFuncSetAttribute((const void*)k_bucket_sort<POINTS, QUADS>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)); \
        k_bucket_sort<POINTS, QUADS><<<n_part_wg, kPartThreads, lds, st>>>(rows, n_rows, d_joff, B, bucket_mask, d_records, n_records, d_starts, d_info, clr); \
    }
            { ProfScope ps(kProfBucketSort, st);
              FX_SORT(true, 1) FX_SORT(true, 2) FX_SORT(true, 4) FX_SORT(false, 1) FX_SORT(false, 2) FX_SORT(false, 4) }
#undef FX_SORT
            { ProfScope ps(kProfBucketLeaves, st);
              const int piece_rows_log2 = quads == 4 ? 14 : quads == 2 ? 13 : 12;
              if (B > 16) k_bucket_leaves<true><<<n_buckets, kBucketThreads, 0, st>>>(d_records, n_records, d_starts, d_info, n_part_wg, piece_rows_log2, L, g->d_hdr);
              else k_bucket_leaves<false><<<n_buckets, kBucketThreads, 0, st>>>(d_records, n_records, d_starts, d_info, n_part_wg, piece_rows_log2, L, g->d_hdr); }
        } else {
            const unsigned nb_rows = (unsigned)((n_rows + kDirectThreads - 1) / kDirectThreads);
            // few fine leaves: more workgroups (15.8 k of them 10.1 us, 12.4 with 512 threads); many: fewer updates of the counter
            const unsigned coarse_threads = n_rows <= 16384 ? kCoarseThreads / 2 : kCoarseThreads;
            ProfScope ps(kProfVoxelsToLeaves, st);
            if (from.kind == LeafSource::kCoarsen)
                k_coarse_leaves<<<(unsigned)((n_rows + coarse_threads - 1) / coarse_threads), coarse_threads, 0, st>>>(from.grid->view(), d_slots, (uint32_t)(n_slots - 1), L, g->d_hdr);
            else if (from.kind == LeafSource::kPad) {
                k_pad_claim<<<(unsigned)((n_rows * 32 + kPadClaimThreads - 1) / kPadClaimThreads), kPadClaimThreads, 0, st>>>(
                    from.grid->view(), from.r, d_slots, (uint32_t)(n_slots - 1), L, g->d_hdr, from.d_bad);
                k_pad_masks<<<(unsigned)((g->cap_leaf + kPadWaves - 1) / kPadWaves), 64 * kPadWaves, 0, st>>>(from.grid->view(), from.r,
                                                                                                           L, g->d_hdr);
            } else if (from.kind == LeafSource::kSubdivide)
                k_subdivide_leaves<<<(unsigned)((n_rows * 8 + kSubdivideThreads - 1) / kSubdivideThreads), kSubdivideThreads, 0, st>>>(
                    from.grid->view(), L, g->d_hdr, from.d_bad);
            else if (rows.xyz)
                k_voxels_to_leaves<true><<<nb_rows, kDirectThreads, 0, st>>>(rows, n_rows, d_joff, B, d_slots, (uint32_t)(n_slots - 1), L, g->d_hdr);
            else
                k_voxels_to_leaves<false><<<nb_rows, kDirectThreads, 0, st>>>(rows, n_rows, d_joff, B, d_slots, (uint32_t)(n_slots - 1), L, g->d_hdr);
        }
        { ProfScope ps(kProfFindTiles, st); k_find_tiles<<<nb_leaf_1024, kFindTilesThreads, 0, st>>>(L, d_tile_slots, d_rep, g->d_hdr); }
        const bool rank_in_block = g->cap_upper <= kRankInBlock;
        if (!rank_in_block) { ProfScope ps(kProfRankTiles, st); k_rank_tiles<<<kMaxTiles / 256, 256, 0, st>>>(L, d_rep, q); }
        { ProfScope ps(kProfInsertUpper, st);
          const int n_copies = std::min(g->cap_upper, kAggUpper);
          const size_t lds = sizeof(uint64_t) * kUpperWords * (size_t)n_copies;
          if (lds > 64 * 1024) FX_TRY_OR_FAIL(hipFuncSetAttribute((const void*)k_insert_upper, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
          k_insert_upper<<<nb_leaf_1024, kInsertUpperThreads, lds, st>>>(
              L, q, d_rep, rank_in_block ? 1 : 0, n_copies); }
        LevelScan su{g->d_upper_mask, g->d_upper_prefix, &g->d_hdr->n_upper, kUpperWords, &g->d_hdr->n_lower,
                     g->cap_lower, 2};
        { ProfScope ps(kProfScanUpper, st); if (scan_level(g, su, g->cap_upper, scan_sync(0), st) != FX_OK) return fail(FX_EDEVICE); }
        { ProfScope ps(kProfInsertLower, st); k_insert_lower<<<nb_leaf, 256, 0, st>>>(L, q); }
        LevelScan sl{g->d_lower_mask, g->d_lower_prefix, &g->d_hdr->n_lower, kLowerWords, &g->d_hdr->n_leaf,
                     g->cap_leaf, 4};
        { ProfScope ps(kProfScanLower, st); if (scan_level(g, sl, g->cap_lower, scan_sync(1), st) != FX_OK) return fail(FX_EDEVICE); }
        { ProfScope ps(kProfInsertLeaf, st); k_place_leaves<<<nb_place, 256, 0, st>>>(L, q, d_leaf_count); }
        const int lb = std::max(1, (g->cap_leaf + kLeafChunk - 1) / kLeafChunk);
        { ProfScope ps(kProfScanLeaf, st);
          k_scan_leaves<<<lb, kScanThreads, 0, st>>>(g->d_leaf, d_leaf_count, g->d_hdr, scan_sync(2), g->d_vox_base, B); }
        FX_TRY_OR_FAIL(hipGetLastError());
    }
    if (n_rows > 0 && B == 0 && rows.xyz) {
        k_count_bad_points<<<(unsigned)((n_rows + 255) / 256), 256, 0, st>>>(rows, n_rows, g->d_hdr);
        FX_TRY_OR_FAIL(hipGetLastError());
    }
    // one read-back: counts + per-grid ranges (Sec. 3.3 step 10)
    ReadBack rb;
    rc = rb.prepare(B);
    if (rc != FX_OK) return fail(rc);
    k_publish<<<1, 256, 0, st>>>(g->d_hdr, g->d_vox_base, B, rb.host, rb.host_ticket, rb.ticket);
    FX_TRY_OR_FAIL(hipGetLastError());
    // runs on the device while the host waits for the ticket and returns to its caller
    if (from.kind == LeafSource::kCoarsen && from.link_K) enqueue_leaf_links(g, st, from.grid, from.link_K, 2);
    else enqueue_leaf_links(g, st, nullptr, 3, 1);
    FX_TRY_OR_FAIL(rb.wait(st));
    rb.take(g);
    if (g->d_leaf_links && g->hdr.n_leaf > g->links_max) {
        dev_free(g->d_leaf_links, st);
        g->d_leaf_links = nullptr; g->d_tile_first_leaf = nullptr;
    }
    dev_free(scratch, st);
#undef FX_TRY_OR_FAIL
    *out = g;
    return FX_OK;
}

// The whole build in one launch (k_small_grid).  *out stays null when the grid is not one it holds: the caller goes on with
// the passes.
static fx_status build_small(const RowSource& rows, int64_t n_rows, const BatchRanges& joff, int32_t B, hipStream_t st, const LeafSource& from,
                             fx_grid** out) {
    *out = nullptr;
    if (from.kind == LeafSource::kCoarsen && n_rows > kSmallLeaves &&
        (n_rows > kSmallFineLeaves || from.grid->hdr.n_voxels < kFilledVoxels * n_rows)) return FX_OK;
    if (n_rows < 1 || n_rows > kSmallRows || B < 1 || B > 16 || (B > kInlineRanges && from.kind == LeafSource::kRows) ||
        option(kOptGridDirect) == 1) return FX_OK;
    fx_grid* g = new (std::nothrow) fx_grid();
    if (!g) { set_error("host allocation failed"); return FX_ENOMEM; }
    g->B = B; g->stream = st;
    g->cap_leaf = g->cap_lower = (int)std::min<int64_t>(n_rows, kSmallSlots);
    g->cap_upper = (int)std::min<int64_t>(n_rows, kRankInBlock);
    layout(g);
    fx_status rc = dev_alloc(&g->buf, g->buf_bytes, st);
    if (rc != FX_OK) { delete g; return rc; }
    layout(g);
    g->h_vox_base = (int64_t*)calloc((size_t)B + 1, sizeof(int64_t));
    ReadBack rb;
    rc = rb.prepare(B);
    if (rc != FX_OK) { fx_grid_destroy(g); return rc; }
    hipError_t e = hipSuccess;
#define FX_SMALL(SOURCE, TREE)                                                                                                      \
    do {                                                                                                                            \
        e = hipFuncSetAttribute((const void*)k_small_grid<SOURCE>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kSmallLds);     \
        if (e == hipSuccess)                                                                                                        \
            k_small_grid<SOURCE><<<1, kSmallThreads, kSmallLds, st>>>(rows, (int)n_rows, joff, B, TREE, ptrs_of(g), rb.host,        \
                                                                      rb.host_ticket, rb.ticket);                                   \
    } while (0)
    {
        ProfScope ps(kProfSmallGrid, st);
        if (from.kind == LeafSource::kCoarsen) FX_SMALL(kSmallCoarse, from.grid->view());
        else if (rows.xyz) FX_SMALL(kSmallPoints, TreeView{});
        else FX_SMALL(kSmallIjk, TreeView{});
    }
#undef FX_SMALL
    if (e == hipSuccess) e = hipGetLastError();
    if (e == hipSuccess) {
        if (from.kind == LeafSource::kCoarsen && from.link_K) enqueue_leaf_links(g, st, from.grid, from.link_K, 2);
        else enqueue_leaf_links(g, st, nullptr, 3, 1);
        e = rb.wait(st);
    }
    if (e != hipSuccess) { fx_grid_destroy(g); set_error("grid build: %s", hipGetErrorString(e)); return FX_EDEVICE; }
    rb.take(g);
    if (g->hdr.overflow) { fx_grid_destroy(g); return FX_OK; }
    *out = g;
    return FX_OK;
}

static fx_status build_with_ranges(const RowSource& rows, int64_t n_rows, const BatchRanges& d_joff, int32_t B,
                                    hipStream_t st, fx_grid** out) {
    // First attempt with capacities that fit typical occupancy -- for up to some 70 k rows with any: a leaf per row --
    // and up to eight root tiles per grid (a scene around the origin); an attempt that overflows has
    // (almost always) counted the nodes of the overflowing level exactly and is repeated with those.
    const int64_t some = std::max<int64_t>(n_rows, 1);
    int cap_upper = (int)std::min<int64_t>(some, B <= 8 ? 8 * (int64_t)B + 8 : (int64_t)B + 64);
    int cap_lower = (int)std::min<int64_t>(some, 64 * (int64_t)std::max(B, 1) + 512 + n_rows / 256);
    int cap_leaf = (int)std::min<int64_t>(some, 65536 + n_rows / 8);
    bool direct = option(kOptGridDirect) == 1;
    FX_TRY(build_small(rows, n_rows, d_joff, B, st, LeafSource(), out));
    if (*out) return FX_OK;
    for (int attempt = 0; attempt < 9; ++attempt) {
        fx_grid* g = nullptr;
        FX_TRY(build_attempt(rows, n_rows, d_joff, B, cap_upper, cap_lower, cap_leaf, direct, st, &g));
        const int ov = g->hdr.overflow;
        if (!ov) { *out = g; return FX_OK; }
        if (ov & 8) {
            fx_grid_destroy(g);
            set_error("more than %d root tiles (4096^3 regions) in the batch", kMaxTiles);
            return FX_ERANGE;
        }
        if (ov & 16) {
            fx_grid_destroy(g);
            set_error("more than 2^31-1 active voxels");
            return FX_ERANGE;
        }
        if (ov & 128) {
            fx_grid_destroy(g);
            set_error("grid build: a workgroup of a scan waited for its predecessors beyond the limit");
            return FX_EDEVICE;
        }
        if (ov & 64) direct = true;   // a bucket held more leaves than its workgroup walks in rounds
        if (ov & 1) cap_upper = g->hdr.n_upper;
        if (ov & 2) { cap_upper = g->hdr.n_upper; cap_lower = g->hdr.n_lower; }
        if (ov & 4) {
            // The voxel pass counts every distinct leaf it can put in its table (twice the
            // capacity); only when the table itself filled up is the count a lower bound, and
            // the capacity grows geometrically instead (at most one leaf per input row exists).
            if (ov & 32) cap_leaf = (int)std::min<int64_t>(std::max<int64_t>(n_rows, 1), 4 * (int64_t)cap_leaf);
            else cap_leaf = g->hdr.n_leaf_raw;
        }
        fx_grid_destroy(g);
    }
    set_error("grid build did not converge");
    return FX_EDEVICE;
}

// The build from rows already on the device; h_pairs = (begin, end) rows of every grid of the batch, on the host.
// Up to eight grids need no upload at all; more go through pinned staging into a device array that lives until the build
// has synchronised the stream.
static fx_status build_index_grid_device(const RowSource& rows, int64_t n_rows, const int64_t* h_pairs, int32_t B,
                                  hipStream_t st, fx_grid** out) {
    BatchRanges J{};
    int64_t* d_pairs = nullptr;
    if (B <= kInlineRanges) {
        for (int b = 0; b < B; ++b) { J.begin[b] = h_pairs[2 * b]; J.end[b] = h_pairs[2 * b + 1]; }
    } else {
        const size_t jb = sizeof(int64_t) * 2 * (size_t)B;
        FX_TRY(dev_alloc((void**)&d_pairs, jb, st));
        void* stage = nullptr;
        fx_status rc = host_staging(&stage, jb, 1);
        if (rc != FX_OK) { dev_free(d_pairs, st); return rc; }
        memcpy(stage, h_pairs, jb);
        const hipError_t e = hipMemcpyAsync(d_pairs, stage, jb, hipMemcpyHostToDevice, st);
        if (e != hipSuccess) { dev_free(d_pairs, st); set_error("joffsets upload failed: %s", hipGetErrorString(e)); return FX_EDEVICE; }
        J.d = d_pairs;
    }
    const fx_status rc = build_with_ranges(rows, n_rows, J, B, st, out);
    if (d_pairs) dev_free(d_pairs, st);
    return rc;
}

}  // namespace fx

// ====================================================================================== C ABI
using namespace fx;

static fx_status build_index_grid_checked(const RowSource& rows, int64_t n_rows, const int64_t* h_joffsets, int32_t B, void* stream,
                                          fx_grid** out) {
    if (!out || B < 0 || n_rows < 0 || (B > 0 && !h_joffsets) || (n_rows > 0 && !rows.ijk && !rows.xyz)) {
        set_error("fx_build_index_grid: null pointer or negative size");
        return FX_EINVAL;
    }
    if (n_rows > (int64_t)INT32_MAX) { set_error("more than 2^31-1 input rows"); return FX_ERANGE; }
    int64_t prev_end = 0;
    for (int32_t b = 0; b < B; ++b) {
        const int64_t s = h_joffsets[2 * b], e = h_joffsets[2 * b + 1];
        if (s < prev_end || e < s || e > n_rows) {
            set_error("joffsets[%d] = (%lld, %lld) is out of range, overlapping or out of order", b, (long long)s,
                      (long long)e);
            return FX_EINVAL;
        }
        prev_end = e;
    }
    return build_index_grid_device(rows, n_rows, h_joffsets, B, (hipStream_t)stream, out);
}

extern "C" fx_status fx_build_index_grid(const int32_t* d_ijk, int64_t n_rows, const int64_t* h_joffsets,
                                         int32_t B, void* stream, fx_grid** out) {
    RowSource rows{};
    rows.ijk = d_ijk;
    return build_index_grid_checked(rows, n_rows, h_joffsets, B, stream, out);
}

extern "C" fx_status fx_grid_info(const fx_grid* g, int64_t* n_voxels, int32_t* B, int64_t* h_voxel_joffsets,
                                  int64_t* h_counts3) {
    if (!g) { set_error("fx_grid_info: null grid"); return FX_EINVAL; }
    if (n_voxels) *n_voxels = g->hdr.n_voxels;
    if (B) *B = g->B;
    if (h_voxel_joffsets)
        for (int b = 0; b < g->B; ++b) {
            h_voxel_joffsets[2 * b] = g->h_vox_base[b];
            h_voxel_joffsets[2 * b + 1] = g->h_vox_base[b + 1];
        }
    if (h_counts3) { h_counts3[0] = g->hdr.n_leaf; h_counts3[1] = g->hdr.n_lower; h_counts3[2] = g->hdr.n_upper; }
    return FX_OK;
}

extern "C" fx_status fx_grid_ijk(const fx_grid* g, int32_t* d_ijk_out, int32_t* d_jidx_out, void* stream) {
    if (!g || (!d_ijk_out && g->hdr.n_voxels > 0)) { set_error("fx_grid_ijk: null pointer"); return FX_EINVAL; }
    if (g->hdr.n_leaf == 0) return FX_OK;
    constexpr int kLeavesPerWg = kIjkLeaves * kIjkWaves;
    k_grid_ijk<<<(unsigned)((g->hdr.n_leaf + kLeavesPerWg - 1) / kLeavesPerWg), 64 * kIjkWaves, 0, (hipStream_t)stream>>>(
        g->view(), d_ijk_out, d_jidx_out, 0);
    FX_HIP_TRY(hipGetLastError());
    return FX_OK;
}

extern "C" fx_status fx_grid_ijk_to_index(const fx_grid* g, const int32_t* d_ijk, const int32_t* d_jidx, int64_t n,
                                          int32_t* d_index_out, void* stream) {
    if (!g || n < 0 || (n > 0 && (!d_ijk || !d_index_out))) {
        set_error("fx_grid_ijk_to_index: null pointer or negative size");
        return FX_EINVAL;
    }
    if (n == 0) return FX_OK;
    k_ijk_to_index<<<(unsigned)((n + 255) / 256), 256, 0, (hipStream_t)stream>>>(g->view(), d_ijk, d_jidx, n,
                                                                                  d_index_out);
    FX_HIP_TRY(hipGetLastError());
    return FX_OK;
}

extern "C" fx_status fx_grid_leaf_table(const fx_grid* g, fx_leaf* h_out, size_t bytes, void* stream) {
    if (!g) { set_error("fx_grid_leaf_table: null grid"); return FX_EINVAL; }
    const size_t need = sizeof(fx_leaf) * (size_t)g->hdr.n_leaf;
    if (bytes < need || (need && !h_out)) { set_error("fx_grid_leaf_table: buffer too small"); return FX_EINVAL; }
    if (!need) return FX_OK;
    FX_HIP_TRY(hipMemcpyAsync(h_out, g->d_leaf, need, hipMemcpyDeviceToHost, (hipStream_t)stream));
    FX_HIP_TRY(hipStreamSynchronize((hipStream_t)stream));
    return FX_OK;
}

extern "C" fx_status fx_build_index_grid_from_points(const float* d_xyz, int64_t n_rows, const int64_t* h_joffsets,
                                                     int32_t B, const float* h_origin, const float* h_voxel_size,
                                                     void* stream, fx_grid** out) {
    if (!out || !h_origin || !h_voxel_size || n_rows < 0 || (n_rows > 0 && !d_xyz)) {
        set_error("fx_build_index_grid_from_points: null pointer or negative size");
        return FX_EINVAL;
    }
    for (int a = 0; a < 3; ++a)
        if (!(h_voxel_size[a] > 0.f) || !std::isfinite(h_voxel_size[a]) || !std::isfinite(h_origin[a])) {
            set_error("fx_build_index_grid_from_points: voxel sizes must be positive and finite, the origin finite");
            return FX_EINVAL;
        }
    if (n_rows > (int64_t)INT32_MAX) { set_error("more than 2^31-1 input rows"); return FX_ERANGE; }
    RowSource rows{};
    rows.xyz = d_xyz;
    for (int a = 0; a < 3; ++a) { rows.o[a] = h_origin[a]; rows.s[a] = h_voxel_size[a]; rows.inv_s[a] = 1.0f / h_voxel_size[a]; }
    fx_grid* g = nullptr;
    FX_TRY(build_index_grid_checked(rows, n_rows, h_joffsets, B, stream, &g));
    if (g->hdr.n_bad > 0) {
        set_error("%d point coordinates are not finite or fall outside [-2^30, 2^30) voxels", g->hdr.n_bad);
        fx_grid_destroy(g);
        return FX_ERANGE;
    }
    *out = g;
    return FX_OK;
}

fx_status fx::grid_coarsen2_for_map(const fx_grid* g, int K, hipStream_t st, fx_grid** out) {
    // The coarse grid has at most as many nodes per level as the fine one, so one attempt with the fine grid's
    // counts as capacities always fits; its leaves come from the fine leaves, not from a row per voxel.
    fx_grid* o = nullptr;
    const BatchRanges none{};
    LeafSource from;
    from.kind = LeafSource::kCoarsen; from.grid = g; from.link_K = K;
    FX_TRY(build_small(RowSource{}, g->hdr.n_leaf, none, g->B, st, from, &o));
    if (o) { *out = o; return FX_OK; }
    FX_TRY(build_attempt(RowSource{}, g->hdr.n_leaf, none, g->B, g->hdr.n_upper, g->hdr.n_lower, g->hdr.n_leaf, true, st, &o, from));
    if (o->hdr.overflow) {
        const int ov = o->hdr.overflow;
        fx_grid_destroy(o);
        set_error("fx_grid_coarsen2: the coarse grid did not fit the fine grid's node counts (flags %d)", ov);
        return FX_EDEVICE;
    }
    *out = o;
    return FX_OK;
}

extern "C" fx_status fx_grid_coarsen2(const fx_grid* g, void* stream, fx_grid** out) {
    if (!g || !out) { set_error("fx_grid_coarsen2: null pointer"); return FX_EINVAL; }
    return grid_coarsen2_for_map(g, 0, (hipStream_t)stream, out);
}

extern "C" fx_status fx_grid_subdivide2(const fx_grid* g, void* stream, fx_grid** out) {
    if (!g || !out) { set_error("fx_grid_subdivide2: null pointer"); return FX_EINVAL; }
    hipStream_t st = (hipStream_t)stream;
    const int64_t n = g->hdr.n_voxels;
    if (8 * n > 0x7FFFFFFFll) { set_error("fx_grid_subdivide2: more than 2^31-1 voxels"); return FX_ERANGE; }
    // The fine grid's leaves are the non-empty octants of the coarse leaves (k_subdivide_leaves); a fine node of
    // any level covers an octant of the coarse node of that level, so eight times the coarse counts always fit.
    const int64_t cap_leaf = 8 * (int64_t)g->hdr.n_leaf, cap_lower = 8 * (int64_t)g->hdr.n_lower, cap_upper = 8 * (int64_t)g->hdr.n_upper;
    if (cap_leaf > 0x7FFFFFFFll / 8) { set_error("fx_grid_subdivide2: too many leaves"); return FX_ERANGE; }
    int32_t* d_bad = nullptr;     // octants whose doubled coordinates would leave the int32 range
    FX_TRY(dev_alloc((void**)&d_bad, 16, st));
    if (hipMemsetAsync(d_bad, 0, sizeof(int32_t), st) != hipSuccess) { dev_free(d_bad, st); set_error("fx_grid_subdivide2: fill failed"); return FX_EDEVICE; }
    LeafSource from;
    from.kind = LeafSource::kSubdivide; from.grid = g; from.d_bad = d_bad;
    const BatchRanges none{};
    fx_grid* o = nullptr;
    fx_status rc = build_attempt(RowSource{}, g->hdr.n_leaf, none, g->B, (int)cap_upper, (int)cap_lower, (int)cap_leaf, true, st, &o, from);
    int32_t bad = 0;
    if (rc == FX_OK && hipMemcpy(&bad, d_bad, sizeof(int32_t), hipMemcpyDeviceToHost) != hipSuccess) {
        rc = FX_EDEVICE; set_error("fx_grid_subdivide2: read-back failed");
    }
    dev_free(d_bad, st);
    if (rc == FX_OK && bad > 0) {
        set_error("fx_grid_subdivide2: %d leaves hold coordinates beyond +-2^30, whose doubles leave the int32 coordinate limits", bad);
        rc = FX_ERANGE;
    }
    if (rc == FX_OK && o->hdr.overflow) {
        set_error("fx_grid_subdivide2: the fine grid did not fit eight times the coarse grid's node counts (flags %d)", o->hdr.overflow);
        rc = (o->hdr.overflow & 16) ? FX_ERANGE : FX_EDEVICE;
    }
    if (rc != FX_OK) { if (o) fx_grid_destroy(o); return rc; }
    *out = o;
    return FX_OK;
}

extern "C" fx_status fx_grid_pad(const fx_grid* g, int32_t r, void* stream, fx_grid** out) {
    if (!g || !out) { set_error("fx_grid_pad: null pointer"); return FX_EINVAL; }
    if (r < 0) { set_error("fx_grid_pad: negative padding %d", r); return FX_EINVAL; }
    if (r > 8) { set_error("fx_grid_pad: padding %d is above the supported 8 voxels", r); return FX_EUNSUPPORTED; }
    hipStream_t st = (hipStream_t)stream;
    if ((int64_t)g->hdr.n_leaf * 27 > 0x7FFFFFFFll) { set_error("fx_grid_pad: too many leaves"); return FX_ERANGE; }
    int32_t* d_bad = nullptr;     // pieces that would leave the int32 coordinate range
    FX_TRY(dev_alloc((void**)&d_bad, 16, st));
    // The padded grid's leaves come from the source grid's leaves (k_pad_claim, k_pad_masks); every leaf reaches at most the 27
    // leaves around it.  First attempt with room for twice the nodes, then with the counts the attempt found.
    const int64_t nl = g->hdr.n_leaf, nlo = g->hdr.n_lower, nu = g->hdr.n_upper;
    int64_t cap_leaf = std::min<int64_t>(27 * nl, 2 * nl + 4096), cap_lower = std::min<int64_t>(27 * nlo, 2 * nlo + 64),
            cap_upper = std::min<int64_t>(27 * nu, 8 * nu + 8);
    fx_grid* o = nullptr;
    fx_status rc = FX_OK;
    const BatchRanges none{};
    LeafSource from;
    from.kind = LeafSource::kPad; from.grid = g; from.r = r; from.d_bad = d_bad;
    for (int attempt = 0; attempt < 6; ++attempt) {
        if (hipMemsetAsync(d_bad, 0, sizeof(int32_t), st) != hipSuccess) { rc = FX_EDEVICE; set_error("fx_grid_pad: fill failed"); break; }
        rc = build_attempt(RowSource{}, nl, none, g->B, (int)cap_upper, (int)cap_lower, (int)cap_leaf, true, st, &o, from);
        if (rc != FX_OK) break;
        const int ov = o->hdr.overflow;
        if (!ov) break;
        if (ov & (8 | 16 | 128) || attempt == 5) {
            fx_grid_destroy(o); o = nullptr;
            if (ov & 8) set_error("more than %d root tiles (4096^3 regions) in the batch", kMaxTiles);
            else if (ov & 16) set_error("fx_grid_pad: the padded grid has more than 2^31-1 active voxels");
            else set_error("fx_grid_pad: the build failed (flags %d)", ov);
            rc = ov & (8 | 16) ? FX_ERANGE : FX_EDEVICE;
            break;
        }
        if (ov & 1) cap_upper = o->hdr.n_upper;
        if (ov & 2) { cap_upper = o->hdr.n_upper; cap_lower = o->hdr.n_lower; }
        if (ov & 4) cap_leaf = (ov & 32) ? std::min<int64_t>(27 * nl, 4 * cap_leaf) : std::max<int64_t>(o->hdr.n_leaf_raw, cap_leaf + 1);
        fx_grid_destroy(o); o = nullptr;
    }
    int32_t bad = 0;
    if (rc == FX_OK) {
        const hipError_t e = hipMemcpy(&bad, d_bad, sizeof(int32_t), hipMemcpyDeviceToHost);
        if (e != hipSuccess) { rc = FX_EDEVICE; set_error("read-back failed: %s", hipGetErrorString(e)); }
    }
    dev_free(d_bad, st);
    if (rc == FX_OK && bad > 0) {
        set_error("fx_grid_pad: %d leaf blocks of the padded grid lie beyond the int32 coordinate limits (a voxel lies within %d of them)", bad, r);
        rc = FX_ERANGE;
    }
    if (rc != FX_OK) { if (o) fx_grid_destroy(o); return rc; }
    *out = o;
    return FX_OK;
}

extern "C" void fx_grid_retain(fx_grid* g) {
    if (g) g->refs.fetch_add(1);
}

extern "C" void fx_grid_destroy(fx_grid* g) {
    if (!g) return;
    if (g->refs.fetch_sub(1) != 1) return;
    if (g->buf) dev_free(g->buf, g->stream);
    if (g->d_leaf_links) dev_free(g->d_leaf_links, g->stream);
    free(g->h_vox_base);
    delete g;
}
