// Weight gradient on the matrix units where a tile's rows are not staged: strided maps, which share none, and listed tiles
// of submanifold maps.  Kernel and launch.
#include "conv_common.h"

namespace fx {

// On a stride-2 map the 512 outputs of a tile read rows that they share with few others (none at K = 2: one pair per
// input row), so nothing is gained by staging a tile's rows for all offsets, and the tile kernel (k_wgrad_mfma) spent
// its time turning such rows by a product with the identity, with a barrier on either side of every tile.  Here a WAVE
// owns one offset and a block of 64 input x 64 output channels of gw[kappa] (four accumulator tiles, 64 registers) and
// walks the column blocks of its range that have the offset, alone: its rows and its outputs' gout rows go through
// 8 KB of LDS of its own and are read back transposed (tr_read4: eight voxels along k for both operands), so no wave
// waits for another until the end.
//
// What bounds it is memory: an x row is read once per offset it has and 64-channel block of gout, a gout row once per
// offset.  Sixteen waves per compute unit (two per offset, each on half of the range's blocks; their sums meet in LDS)
// keep 8 KB each in flight, and a wave runs the chain header -> ids -> row list -> rows ahead of its multiplies: ids of
// block j + 3, row numbers of j + 2 and rows of j + 1 are requested before block j is multiplied.  Every lane issues
// every load (a lane without a voxel repeats the row of one that has, whose line is being fetched anyway), so the waits
// are counted exactly.  Rows of voxels without the offset are zeroed on their way into LDS in both operands: sums run
// over existing pairs only, whatever the values are.  Eight waves with two blocks in flight each are 3 us faster on
// maps of a few thousand outputs and as fast at K = 2, but 17 % slower at K = 3.
//
// LISTED: the same over a list of tiles of a submanifold map, those whose rows the tile kernel cannot stage (tile_list;
// such a tile may have a window).  Against a workgroup per column block of such a tile
// in the tile kernel's other form, the whole call, bf16: 221 k LiDAR voxels with five such tiles 64 -> 64 79 -> 69 us,
// 256 -> 256 536 -> 498; 195 k voxels of sheets with four 256 -> 256 581 -> 546; 980 k LiDAR voxels with three 181 -> 178.
//
// A workgroup takes eight consecutive offsets of a range; the jobs of one range (channel blocks and, at K = 3, four
// octets of offsets) are placed on one XCD (workgroup b runs on XCD b % 8) so that they share its L2.
// bf16, reduction included, k_wgrad_mfma -> here, in us: 980 k LiDAR voxels, (2,2) map 64 -> 64 89 -> 50, 64 -> 128 150 -> 85,
// 128 -> 256 728 -> 276; (3,2) map 64 -> 64 165 -> 104, 64 -> 128 329 -> 197, 24 -> 8 95 -> 102, which is the chain of a block
// whatever the channels are; 95 k LiDAR voxels (24 k outputs), (2,2) map 64 -> 64 21.5 -> 22, 24 -> 8 18 -> 16; 31 k (7.8 k outputs)
// 64 -> 64 18 -> 18, 64 -> 128 19 -> 22, (3,2) map 36 -> 24; 4.7 k outputs of sheets, (2,2) map 64 -> 128 25 -> 19.
// Small maps are a launch, the chain and the end: with the sums of both halves stored by one of them, a division of 64-bit
// block numbers and a few spilled registers a map of 62 outputs took 12.8 us here instead of 8.8.
constexpr int kPairsOffsets = 8;                               // offsets of a workgroup
constexpr int kPairsWaves = 2 * kPairsOffsets;               // two halves of a range
constexpr int kPairsBlk = 64;                                  // channels of a block, both sides
constexpr int kPairsRowBytes = kPairsBlk * 2;
constexpr int kPairsLdsBytes = kGroup * kPairsRowBytes;        // one side's rows of a column block
constexpr int kPairsLdsTotal = kPairsWaves * 2 * kPairsLdsBytes;
static_assert(kPairsLdsTotal <= 160 * 1024 && 4 * kPairsLdsBytes == kPairsBlk * kPairsBlk * 4, "LDS budget; a wave's rows hold half of its sums");

template <typename T, bool LISTED>
__global__ void __launch_bounds__(64 * kPairsWaves)
k_wgrad_pairs(const TileHeader* __restrict__ tile_hdr, const uint16_t* __restrict__ tile_perm,
              const int32_t* __restrict__ tile_rows, int row_stride, const uint16_t* __restrict__ tile_blocks,
              int block_stride, int64_t per_half, int extra, int n_ranges, const uint16_t* __restrict__ feat,
              const uint16_t* __restrict__ gout, int C_in, int C_out, int K3, float* __restrict__ part,
              const int32_t* __restrict__ tile_list) {
    typedef typename Elem<T>::vec8 vec8;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int lane = threadIdx.x & 63, wave = uni((int)(threadIdx.x >> 6));
    const int n_kg = (K3 + kPairsOffsets - 1) / kPairsOffsets;
    const int n_cib = (C_in + kPairsBlk - 1) / kPairsBlk, n_cob = (C_out + kPairsBlk - 1) / kPairsBlk;
    const int n_jobs = n_kg * n_cib * n_cob;
    int job = blockIdx.x % n_jobs, range = blockIdx.x / n_jobs;
    if (n_ranges % 8 == 0) {
        job = (blockIdx.x >> 3) % n_jobs;
        range = (int)(blockIdx.x / (8 * n_jobs)) * 8 + (blockIdx.x & 7);
    }
    const int oct = wave % kPairsOffsets, half = wave / kPairsOffsets;
    const int kappa = uni(job % n_kg * kPairsOffsets + oct);
    const int ci0 = job / n_kg % n_cib * kPairsBlk, co0 = job / n_kg / n_cib * kPairsBlk;
    // the wave's share of the column blocks: per_half, and one more for the first `extra` halves
    const int nth = 2 * range + half;
    const int64_t g_lo = nth * per_half + min(nth, extra);
    const int64_t g_hi = kappa < K3 ? g_lo + per_half + (nth < extra) : g_lo;
    unsigned char* lx = lds_raw + (oct * 2 + half) * 2 * kPairsLdsBytes;

    // ---- the column blocks of the range that have the offset, in order
    typedef const __attribute__((address_space(4))) TileHeader ConstHeader;
    struct Block { int tile, g; uint32_t id_block; int win_lo, win_n; bool valid; };
    typedef const __attribute__((address_space(4))) int32_t ConstInt;
    auto tile_of = [&](int i) __attribute__((always_inline)) { return LISTED ? (int)((ConstInt*)tile_list)[i] : i; };
    int it_tile = (int)(g_lo / kGroupsPerTile) - 1;
    const int last_tile = (int)((g_hi + kGroupsPerTile - 1) / kGroupsPerTile) - 1;
    uint32_t present = 0;                                      // column blocks of it_tile still to take
    auto next = [&]() __attribute__((always_inline)) -> Block {
        while (present == 0 && it_tile < last_tile) {
            ++it_tile;
            // scalar loads: they do not queue behind the rows in flight
            ConstHeader* H = (ConstHeader*)(tile_hdr + tile_of(it_tile));
#pragma unroll
            for (int g = 0; g < kGroupsPerTile; ++g) present |= ((H->group_mask[g] >> kappa) & 1u) << g;
            const int64_t first = (int64_t)it_tile * kGroupsPerTile;
            if (first < g_lo) present &= ~0u << (int)(g_lo - first);
            if (first + kGroupsPerTile > g_hi) present &= (1u << (int)(g_hi - first)) - 1u;
        }
        Block b = {0, 0, 0u, 0, 0, present != 0};
        if (b.valid) {
            b.tile = tile_of(it_tile);
            b.g = __ffs(present) - 1;
            present &= present - 1;
            ConstHeader* H = (ConstHeader*)(tile_hdr + b.tile);
            if (LISTED) { b.win_lo = H->win_lo; b.win_n = H->win_n; }
            const int w = tile_wave_of(b.g);
            b.id_block = H->wave_block0[w] + __popc(H->wave_mask[w] & ((1u << kappa) - 1u));
        }
        return b;
    };

    // ---- the stages of a column block
    // the lane number made anew where it is needed: the registers of four waves per SIMD are all taken, and one spilled to
    // memory is loaded in order with the rows in flight
    auto lane_now = [&]() __attribute__((always_inline)) -> uint32_t {
        uint32_t l;
        asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
        return l;
    };
    uint32_t id, loc;                   // local row id and output (inside the tile) of voxel n of the block whose ids are in flight
    Block blk;
    int32_t row, window_row, locr;      // row number (LISTED: that of the window where it is not -1) and output of the block before it
    uint32_t has;                       // and its voxels that have the offset
    int32_t out0;                       // first output row of its tile
    u32x4 X[4], Y[4];                   // rows of the block before that one
    uint32_t hasd;
    auto load_ids = [&]() __attribute__((always_inline)) {
        blk = next();
        const size_t b = (size_t)blk.tile * block_stride + blk.id_block;
        const uint32_t n = lane_now() & 31;
        id = (tile_blocks + b * kIdBlockElems + tile_slot_of(blk.g))[n * kGroupsPerWave];
        loc = (tile_perm + (int64_t)blk.tile * kTileT + blk.g * kGroup)[n];
    };
    auto load_row = [&]() __attribute__((always_inline)) {
        const bool mine = blk.valid && id != kNoRow;
        has = (uint32_t)__ballot(mine);                        // lanes 32 .. 63 repeat lanes 0 .. 31
        const bool in_window = LISTED && id < (uint32_t)blk.win_n;
        row = tile_rows[(int64_t)blk.tile * row_stride + (mine && !in_window ? id - (uint32_t)blk.win_n : 0u)];
        if (LISTED) window_row = mine && in_window ? blk.win_lo + (int32_t)id : -1;
        locr = (int32_t)loc;
        out0 = blk.tile * kTileT;
    };
    const int p8 = lane >> 3, piece = lane & 7;
    const bool x_in = ci0 + piece * 8 < C_in, y_in = co0 + piece * 8 < C_out;
    const unsigned char* x_at = reinterpret_cast<const unsigned char*>(feat + ci0 + (x_in ? piece * 8 : 0));
    const unsigned char* y_at = reinterpret_cast<const unsigned char*>(gout + co0 + (y_in ? piece * 8 : 0));
    const uint32_t x_pitch = 2u * (uint32_t)C_in, y_pitch = 2u * (uint32_t)C_out;
    // the row numbers of the lane's four pieces (voxels 8 * i + p8), and the rows themselves
    uint32_t rr[4], ll[4];
    auto spread_rows = [&]() __attribute__((always_inline)) {
        const uint32_t m = has;
        hasd = m;
        const int some = m ? __ffs(m) - 1 : 0;                 // a voxel that has the offset
        const int lane = (int)lane_now();
        if (LISTED && window_row >= 0) row = window_row;
        const int32_t r0 = m ? __builtin_amdgcn_readlane(row, some) : 0, l0 = m ? __builtin_amdgcn_readlane(locr, some) : 0;
        const bool mine = (m >> (lane & 31)) & 1u;
        const int32_t r = mine ? row : r0, l = (mine ? locr : l0) + out0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            rr[i] = (uint32_t)__builtin_amdgcn_ds_bpermute((lane >> 3) * 4 + 32 * i, r);
            ll[i] = (uint32_t)__builtin_amdgcn_ds_bpermute((lane >> 3) * 4 + 32 * i, l);
        }
    };
    auto load_rows = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            X[i] = *reinterpret_cast<const u32x4*>(x_at + (uint64_t)rr[i] * x_pitch);
            Y[i] = *reinterpret_cast<const u32x4*>(y_at + (uint64_t)ll[i] * y_pitch);
            __builtin_amdgcn_sched_barrier(0);                 // one pair of addresses at a time
        }
    };
    // voxel v's row: 16-byte piece p at position p ^ 4 * ((v >> 1) & 1), which spreads a transposing read over all banks
    unsigned char* st = lx + p8 * kPairsRowBytes + ((piece ^ (((p8 >> 1) & 1) << 2)) << 4);
    auto to_lds = [&]() __attribute__((always_inline)) {
        const uint32_t mine = hasd >> (lane_now() >> 3);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool on = (mine >> (8 * i)) & 1u;
            *reinterpret_cast<u32x4*>(st + i * 8 * kPairsRowBytes) = on && x_in ? X[i] : u32x4{0, 0, 0, 0};
            *reinterpret_cast<u32x4*>(st + i * 8 * kPairsRowBytes + kPairsLdsBytes) = on && y_in ? Y[i] : u32x4{0, 0, 0, 0};
        }
    };

    f32x16 acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][c][v] = 0.f;
    // what this lane's address contributes to a transposing read: voxel jv of four, channels 16 * g1 + 4 * q .. + 3
    const int h = lane >> 5, q = lane & 3, jv = (lane >> 2) & 3, g1 = (lane >> 4) & 1;
    // fragment [channels 32 * t + lane % 32][voxels 16 * ks + 8 * h .. + 7] of one side
    const unsigned char* tr0 = lx + (8 * h + jv) * kPairsRowBytes + (((2 * g1 + (q >> 1)) ^ (((jv >> 1) & 1) << 2)) << 4) + ((q & 1) << 3);
    const unsigned char* tr1 = lx + (8 * h + jv) * kPairsRowBytes + (((4 + 2 * g1 + (q >> 1)) ^ (((jv >> 1) & 1) << 2)) << 4) + ((q & 1) << 3);
    auto frag = [&](int side, int t, int ks) __attribute__((always_inline)) -> vec8 {
        const unsigned char* src = (t ? tr1 : tr0) + side * kPairsLdsBytes + ks * 16 * kPairsRowBytes;
        const u32x2 lo = tr_read4(src), hi = tr_read4(src + 4 * kPairsRowBytes);
        return vec8_from_words<T>(u32x4{lo[0], lo[1], hi[0], hi[1]});
    };
    auto multiply = [&]() {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            __builtin_amdgcn_sched_barrier(0);       // one step's fragments at a time: 128 registers
            const vec8 a0 = frag(0, 0, ks), a1 = frag(0, 1, ks), c0 = frag(1, 0, ks), c1 = frag(1, 1, ks);
            acc[0][0] = Elem<T>::mfma(a0, c0, acc[0][0]);
            acc[0][1] = Elem<T>::mfma(a0, c1, acc[0][1]);
            acc[1][0] = Elem<T>::mfma(a1, c0, acc[1][0]);
            acc[1][1] = Elem<T>::mfma(a1, c1, acc[1][1]);
        }
    };

    load_ids();
    load_row(); load_ids();
    spread_rows(); load_row(); load_ids(); load_rows();
    // What one lane writes to LDS others read, and no barrier stands between: a wave's LDS accesses are processed in order, and
    // the compiler is told to keep that order.
    auto wave_lds_sync = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
        __builtin_amdgcn_wave_barrier();
    };
    // block j goes to LDS; rows of j + 1, row numbers of j + 2 and ids of j + 3 are requested; block j is multiplied
    while (hasd) {                       // every block of the list has the offset for some voxel
        to_lds();
        wave_lds_sync();
        spread_rows();
        load_row();
        load_ids();
        load_rows();
        multiply();
        wave_lds_sync();                 // read before the next block takes its place
    }

    // ---- the two waves of an offset meet: each keeps the sums of 32 input channels and hands the others over
    const int ln = (int)lane_now();
    f32x4* mine = reinterpret_cast<f32x4*>(lx) + ln;
    const f32x4* theirs = reinterpret_cast<const f32x4*>(lds_raw + (oct * 2 + 1 - half) * 2 * kPairsLdsBytes) + ln;
    auto quad = [&](int a, int c, int b) { return f32x4{acc[a][c][4 * b], acc[a][c][4 * b + 1], acc[a][c][4 * b + 2], acc[a][c][4 * b + 3]}; };
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int b = 0; b < 4; ++b) mine[(c * 4 + b) * 64] = half ? quad(0, c, b) : quad(1, c, b);
    __syncthreads();
    if (kappa >= K3) return;
    // lane (co = n, h), register v -> ci = 8 * (v / 4) + 4 * h + v % 4: a half-wave stores 128 bytes of one row at a time
    const int ci = ci0 + 32 * half + 4 * (ln >> 5), co = co0 + (ln & 31);
    float* dst = part + (((int64_t)range * K3 + kappa) * C_in + ci) * (int64_t)C_out + co;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const f32x4 sum = (half ? quad(1, c, b) : quad(0, c, b)) + theirs[(c * 4 + b) * 64];
            if (ci + 8 * b < C_in && co + 32 * c < C_out)       // C_in is a multiple of 8
#pragma unroll
                for (int e = 0; e < 4; ++e) dst[(8 * b + e) * (int64_t)C_out + 32 * c] = sum[e];
        }
}

static int pairs_jobs(const fx_kmap* km, int C_in, int C_out) {
    return (km->K3 + kPairsOffsets - 1) / kPairsOffsets * ((C_in + kPairsBlk - 1) / kPairsBlk) * ((C_out + kPairsBlk - 1) / kPairsBlk);
}

int wgrad_pairs_ranges(const fx_kmap* km, int C_in, int C_out, int n_listed) {
    // one workgroup per compute unit; no range shorter than four column blocks (with two or three more partial sums than
    // that saves, 7.8 k outputs 64 -> 128 26 and 23 us for 22; with eight 21, but 1.2 k outputs 64 -> 64 19 for 15), or than eight
    // where there would be more than 16 MB of partial sums, which are written and read once; or, of a list, whose blocks are
    // few and whose latency is what counts, than two and at most sixteen ranges.  Four -> eight, us: (2,2) map 64 -> 128 and
    // 128 -> 128 of 8.1 k outputs (17 and 34 MB) 22 -> 20, 27 -> 24, 128 -> 256 of 3 k (25 MB) 25 -> 23, 64 -> 64 of 20 k (20 MB)
    // 23 -> 21, 64 -> 128 of 20 k (34 MB) 26 -> 25 and 24 -> 25; (3,2) map 64 -> 64 of 8.1 k (28 MB) 25 -> 22; but 128 -> 128 of
    // 3 k (13 MB) 20.3 -> 21.2, 64 -> 64 of 15 k (16 MB) 21.2 -> 22.2.
    const int most = compute_units() / pairs_jobs(km, C_in, C_out);
    if (n_listed) return std::max(1, std::min(most, std::min(16, n_listed * (kGroupsPerTile / 2))));
    auto ranges_of = [&](int blocks) {
        const int n = (int)std::max<int64_t>(1, std::min<int64_t>((km->n_out + blocks * kGroup - 1) / (blocks * kGroup), most));
        return n > 8 ? std::min((n + 3) / 8, std::max(most / 8, 1)) * 8 : n;        // see the block-to-XCD mapping in the kernel
    };
    const int n = ranges_of(4);
    return (int64_t)n * km->K3 * C_in * C_out * 4 > 16 * 1000 * 1000 ? ranges_of(8) : n;
}

hipError_t launch_wgrad_pairs(const fx_kmap* km, const void* d_feat, const void* d_gout, fx_dtype dt, int C_in, int C_out, float* part,
                              int n_ranges, int n_listed, hipStream_t st) {
    const unsigned grid = (unsigned)(pairs_jobs(km, C_in, C_out) * n_ranges);
    const int64_t n_groups = (n_listed ? n_listed : km->n_tiles) * (int64_t)kGroupsPerTile, n_halves = 2 * (int64_t)n_ranges;
    hipError_t e = hipSuccess;
#define FX_PAIRS(T, LISTED)                                                                                            \
    do {                                                                                                               \
        e = hipFuncSetAttribute((const void*)k_wgrad_pairs<T, LISTED>, hipFuncAttributeMaxDynamicSharedMemorySize, kPairsLdsTotal); \
        if (e == hipSuccess)                                                                                           \
            k_wgrad_pairs<T, LISTED><<<grid, 64 * kPairsWaves, kPairsLdsTotal, st>>>(                                  \
                km->d_tile_hdr, km->d_tile_perm, km->d_tile_rows, km->row_stride, km->d_tile_blocks, km->block_stride, \
                n_groups / n_halves, (int)(n_groups % n_halves), n_ranges, (const uint16_t*)d_feat, (const uint16_t*)d_gout, C_in, C_out, \
                km->K3, part, km->d_unstaged_list);                                                                    \
    } while (0)
    if (dt == FX_BF16) { if (n_listed) FX_PAIRS(__bf16, true); else FX_PAIRS(__bf16, false); }
    else { if (n_listed) FX_PAIRS(_Float16, true); else FX_PAIRS(_Float16, false); }
#undef FX_PAIRS
    return e == hipSuccess ? hipGetLastError() : e;
}

}  // namespace fx
