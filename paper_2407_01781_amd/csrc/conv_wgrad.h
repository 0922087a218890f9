// Weight gradient on the matrix units over the tiled map: kernel and launch, a template over the 16-bit type.  It is
// instantiated in conv_wgrad_bf16.hip and conv_wgrad_f16.hip: nine kernels a type, unrolled over offsets and column
// blocks, are most of the library's compile time, so the two types compile side by side.
#pragma once
#include "conv_common.h"

namespace fx {

// bit pattern of 1.0 in the storage type
template <typename T> __device__ __forceinline__ uint16_t one_bits();
template <> __device__ __forceinline__ uint16_t one_bits<__bf16>() { return 0x3F80; }
template <> __device__ __forceinline__ uint16_t one_bits<_Float16>() { return 0x3C00; }

// eight fp32 values that are exactly representable in T -> one operand fragment
template <typename T>
__device__ __forceinline__ typename Elem<T>::vec8 pack8(const f32x16& t, int first) {
    u32x4 w;
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = Elem<T>::pack2(t[first + 2 * e], t[first + 2 * e + 1]);
    return vec8_from_words<T>(w);
}

// A workgroup owns a block of 32 input channels x 64 output channels of every gw[kappa] (the last block of a channel
// count that is not a multiple holds fewer: 16-byte pieces beyond the rows are not staged, and what the operands then
// hold in those channels only reaches elements of gw that do not exist) and a contiguous range of tiles; its 8 waves split the offsets (wave w: kappa = w, w+8, w+16, w+24), so a wave
// keeps up to 4 offsets x 2 accumulator tiles (32 ci x 32 co) in registers over the whole range, and two
// waves per SIMD hide each other's LDS and matrix latencies (16 waves with two offsets each have 128 registers
// per wave, which the loop does not fit without spilling: 261 us against 208 on a 1 M-voxel LiDAR grid; 4 waves 279).  Per tile the workgroup stages,
// single-buffered and all with loads that go straight from global memory to LDS: the tile's input rows
// (32 channels, the forward kernel's LDS row layout, so the map's precomputed LDS offsets apply), its id
// blocks, and the gout rows of its 512 output slots (64 channels = 128 bytes per slot; 16-byte piece p of
// slot s sits at position p ^ 4*((s >> 1) & 1), which spreads a fragment read over all banks).
//
// Transposing read (tr_read4): in every group of 16 lanes, lane 4q+e receives, as element j, element e of
// the 8 bytes that lane 4j+q addresses.  With lane 4j+q pointing at channels 4q..4q+3 of voxel j's row,
// lane c of the group ends up with channel c of voxels 0..3: rows in, operand columns out.
//
// For one (column block g, offset kappa) a wave:
//   1. takes, per k-step ks and half t, the id of voxel 16ks + 8h + 4t + j of the block (h = lane / 32,
//      j = (lane / 4) % 4) -- the row its address contributes -- and reads the A fragment
//      [channel lane % 32][voxels 16ks + 8h .. + 7] of the gathered rows with two transposing reads;
//   2. reads the B fragments [voxel][co] of the gout slots 32g + 16ks + 8h .. + 7 the same way
//      (channels 32cb + lane % 32) and accumulates
//      gw[kappa][ci][co] += sum_voxel feat[voxel][ci] * gout[voxel][co].
// A voxel of the block without that tap reads the zero row and adds nothing; a slot past the end
// of the last tile has a zero gout row.  A tile of 817 to 1022 rows (more than a half of the forward kernel's buffer, so that the
// map holds row numbers for it) is staged like the others and its ids become LDS offsets once they are staged.  Tiles whose rows do
// not fit keep the older form of step 1: the lane reads the row of voxel lane % 32 (from LDS or from global memory), and a product with
// the identity on the matrix unit leaves the block in the accumulator layout, which is the operand layout
// with voxels along k; rounding back to the storage type is exact.
// Partial sums go to part[range][kappa][ci][co] (fp32); k_wgrad_reduce adds the ranges in
// ascending order, so the result does not depend on scheduling.
constexpr int kGoutRowBytes = kWgCo * 2;    // one slot of the staged gout tile
constexpr int kGoutSlabs = kTileT * kGoutRowBytes / 1024;     // 1 KB slabs: 8 slots each

struct WgradLds {
    unsigned char rows[(kWgRowCap + 1) * kRowBytes];       // rows kWgRowCap and, for ids made by the map, kRowCap are all zeros
    unsigned char blocks[kBlockBufBytes];
    unsigned char gt[kTileT * kGoutRowBytes];
};
static_assert(sizeof(WgradLds) <= 160 * 1024, "LDS budget of one compute unit");
static_assert(kGroupsPerWave == 4 && kTileWaves == 4, "id blocks of four column blocks, 8 bytes per voxel");

// Which tiles a launch takes.  Tiles whose rows are all staged in LDS (wgrad_stages; all of most submanifold maps') need
// neither the identity fragments nor the fallback loads of the older form: without that code the
// kernel fits 128 registers, runs sixteen waves with two offsets each -- four waves per SIMD to cover each other's
// LDS latencies -- and took 150 us where the eight-wave kernel with both forms took 204 (1 M-voxel LiDAR grid,
// 64 -> 64); 30 us of those 204 were one workgroup's single tile of the other kind, which costs as much as four
// staged ones.  When the map has at most kMaxListedTiles such tiles (counted once per map), kWgStaged (16 waves)
// takes the staged tiles of the ranges, and k_wgrad_pairs the listed ones, a wave per offset.  The same for a 3x3x3 map onto a grid of
// twice the input's voxels and more (kWgAll / this, us: 1.72 M voxels of a padded grid 64 -> 64 352 / 246, 4.7 k 37.8 / 25.0).  Other
// maps (onto another grid, a row per pair; strided maps go to k_wgrad_pairs) take one launch of
// kWgAll (8 waves, both forms, every tile of the range).  Either way a partial sum is made of the same terms in a
// fixed order.  With 816 rows staged, tiles above went to the pairs or, from 0.20 mean leaf occupancy on, the map to kWgAll; with
// 1022, bf16 64 -> 64, us: 24 k voxels of a sphere shell 38.8 -> 27.3, 116 k of LiDAR 48 -> 39, 195 k of sheets 61 -> 52, 88 k / 531 k of
// bodies, surfaces and scan lines 86 -> 74 / 235 -> 214; random voxels of a cube, 239 k at 0.18 of its volume 89.8 -> 65.6, 399 k at 0.30
// 191 -> 105.5; 40 -> 40 on 505 k at 0.38 303 -> 134.
enum WgradMode { kWgAll = 0, kWgStaged = 1 };

//
// SHAPE: kWgFull when both channel counts are whole blocks (no masks: with them the sixteen-wave kernel spills 16
// registers instead of 4), kWgPartial otherwise, kWgNarrow for up to 32 output channels (one accumulator tile per
// offset instead of two, of which the second would multiply nothing).
enum WgradShape { kWgFull = 0, kWgPartial = 1, kWgNarrow = 2 };

template <typename T, int W, int MODE, int SHAPE>
__global__ void __launch_bounds__(64 * W, 1)
k_wgrad_mfma(const TileHeader* __restrict__ tile_hdr, const uint16_t* __restrict__ tile_perm,
             const int32_t* __restrict__ tile_rows, int row_stride, const uint16_t* __restrict__ tile_blocks,
             int block_stride, int64_t n_tiles, int n_ranges, const uint16_t* __restrict__ feat,
             const uint16_t* __restrict__ gout, int C_in, int C_out, int K3, float* __restrict__ part) {
    constexpr int kWgWaves = W;
    constexpr int kGoutSlabsPerWave = kGoutSlabs / kWgWaves;
    constexpr int kWgOffsetsPerWave = (kMaxK3Tiled + kWgWaves - 1) / kWgWaves;
    constexpr bool kMasked = SHAPE != kWgFull;
    constexpr int kHalves = SHAPE == kWgNarrow ? 1 : 2;      // 32-channel halves of the block's output channels
    static_assert(kGoutSlabs % kWgWaves == 0, "gout slabs per wave");
    typedef typename Elem<T>::vec8 vec8;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    WgradLds& L = *reinterpret_cast<WgradLds*>(lds_raw);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = lane & 31, h = lane >> 5;
    const int n_cib = (C_in + kWgCi - 1) / kWgCi, n_cblk = n_cib * ((C_out + kWgCo - 1) / kWgCo);
    // Workgroup b runs on XCD b % 8.  The channel blocks of one tile range read the same gout tiles and
    // id blocks: with the number of ranges a multiple of 8 they get block indices 8 apart, so they share
    // an XCD and its L2 and run side by side.
    int blk = blockIdx.x % n_cblk, range = blockIdx.x / n_cblk;
    if (n_ranges % 8 == 0) {
        blk = (blockIdx.x >> 3) % n_cblk;
        range = (int)(blockIdx.x / (8 * n_cblk)) * 8 + (blockIdx.x & 7);
    }
    const int cib = blk % n_cib, cob = blk / n_cib;
    // channels from the block's first to the row's end
    const int ci_n = kMasked ? C_in - cib * kWgCi : kWgCi, co_n = kMasked ? C_out - cob * kWgCo : kWgCo;
    const int64_t t0 = n_tiles * range / n_ranges, t1 = n_tiles * (range + 1) / n_ranges;

    if (tid < kRowBytes / 16) reinterpret_cast<u32x4*>(L.rows + kWgRowCap * kRowBytes)[tid] = u32x4{0, 0, 0, 0};

    // identity fragments: element e of lane (n, h) in k-step ks is row k = 8h + e, column n of [I16 at columns 16ks..]
    vec8 ident[2];
    {
        u32x4 wds[2];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int e2 = 0; e2 < 4; ++e2) {
                const uint32_t lo = (n == 16 * ks + 8 * h + 2 * e2) ? one_bits<T>() : 0u;
                const uint32_t hi = (n == 16 * ks + 8 * h + 2 * e2 + 1) ? one_bits<T>() : 0u;
                wds[ks][e2] = lo | (hi << 16);
            }
        ident[0] = vec8_from_words<T>(wds[0]);
        ident[1] = vec8_from_words<T>(wds[1]);
    }

    f32x16 acc[kWgOffsetsPerWave][kHalves];
#pragma unroll
    for (int j = 0; j < kWgOffsetsPerWave; ++j)
#pragma unroll
        for (int cb = 0; cb < kHalves; ++cb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][cb][v] = 0.f;

    // what this lane's address contributes to a transposing read: voxel jv of four, channels 16*g1 + 4*q .. + 3
    const int q = lane & 3, jv = (lane >> 2) & 3, g1 = (lane >> 4) & 1;
    const uint32_t a_piece = (uint32_t)(2 * g1 + (q >> 1)) << 4, half8 = (uint32_t)(q & 1) << 3;
    constexpr int kWgSlabs = ((kWgRowCap + 15) / 16 + kWgWaves - 1) / kWgWaves;   // 1 KB row slabs per wave
    int32_t nx_gr[kWgSlabs];
    int nx_local[kGoutSlabsPerWave];      // output row (inside the tile) of the slot this lane stages in each of its slabs
    auto resolve = [&](int64_t t) {
        const TileHeader* Ht = tile_hdr + t;
        const int fl = uni(Ht->flags), wl = uni(Ht->win_lo), wn = uni(Ht->win_n), nl = uni(Ht->n_list);
        const int ns = (fl & kTileDirect) ? 0 : min(wn + nl, kWgRowCap);
        const int32_t* rows_t = tile_rows + t * (int64_t)row_stride;
#pragma unroll
        for (int j = 0; j < kWgSlabs; ++j) {
            const int r = 16 * (wave + kWgWaves * j) + (lane >> 2);
            nx_gr[j] = -1;
            if (r < ns) nx_gr[j] = r < wn ? wl + r : rows_t[r - wn];
        }
#pragma unroll
        for (int j = 0; j < kGoutSlabsPerWave; ++j) nx_local[j] = tile_perm[t * kTileT + 8 * (wave + kWgWaves * j) + (lane >> 3)];
    };
    // the tiles that this workgroup takes, in order: those of its range (kWgStaged: the staged ones among them)
    auto next_mine = [&](int64_t c) {
        if (MODE == kWgStaged)
            while (c < t1 && !wgrad_stages(uni(tile_hdr[c].flags), uni(tile_hdr[c].win_n), uni(tile_hdr[c].n_list))) ++c;
        return c;
    };
    int64_t cur = next_mine(t0);
    if (cur < t1) resolve(cur);
    while (cur < t1) {
        const int64_t cur_next = next_mine(cur + 1);
        const int64_t tile = cur;
        const TileHeader* H = tile_hdr + tile;
        const int flags = uni(H->flags), win_lo = uni(H->win_lo), win_n = uni(H->win_n), n_list = uni(H->n_list);
        const int n_blocks = uni(H->n_blocks), n_valid = uni(H->n_out);
        const int n_staged = (flags & kTileDirect) ? 0 : min(win_n + n_list, kWgRowCap);
        const bool general = MODE == kWgStaged ? false : !wgrad_stages(flags, win_n, n_list);
        const bool row_ids = !general && !(flags & kTileLdsOffsets);
        const int32_t* my_rows = tile_rows + tile * (int64_t)row_stride;
        uint32_t wmask[kTileWaves], gmask[kGroupsPerTile];
        int block0[kTileWaves];
#pragma unroll
        for (int fw = 0; fw < kTileWaves; ++fw) {
            wmask[fw] = (uint32_t)uni((int)H->wave_mask[fw]);
            block0[fw] = uni((int)H->wave_block0[fw]);
        }
#pragma unroll
        for (int g = 0; g < kGroupsPerTile; ++g) gmask[g] = (uint32_t)uni((int)H->group_mask[g]);

        // ---- stage: input rows (32 channels of this block), id blocks, gout rows.  The global
        // row of every slab piece and the output rows of the lane's slots were resolved while the
        // previous tile was staged, so all of this tile's loads leave at once.
        {
            const int piece = (lane & 3) ^ ((lane >> 4) & 3);
            int32_t gr[kWgSlabs];
#pragma unroll
            for (int j = 0; j < kWgSlabs; ++j) gr[j] = nx_gr[j];
            int local[kGoutSlabsPerWave];
#pragma unroll
            for (int j = 0; j < kGoutSlabsPerWave; ++j) local[j] = nx_local[j];
#pragma unroll
            for (int j = 0; j < kWgSlabs; ++j) {
                if (gr[j] >= 0 && piece * 8 < ci_n) {
                    const uint16_t* src = feat + (int64_t)gr[j] * C_in + cib * kWgCi + piece * 8;
                    __builtin_amdgcn_global_load_lds(src, (lds_ptr_t)(L.rows + (wave + kWgWaves * j) * 1024), 16, 0, 0);
                }
            }
#pragma unroll
            for (int j = 0; j < kGoutSlabsPerWave; ++j) {
                const int slab = wave + kWgWaves * j, slot = 8 * slab + (lane >> 3);
                const int gpiece = (lane & 7) ^ (((slot >> 1) & 1) << 2);        // the piece stored at position lane & 7
                if (local[j] < n_valid) {
                    const uint16_t* src = gout + (tile * kTileT + local[j]) * (int64_t)C_out + cob * kWgCo + gpiece * 8;
                    if (gpiece * 8 < co_n) __builtin_amdgcn_global_load_lds(src, (lds_ptr_t)(L.gt + slab * 1024), 16, 0, 0);
                } else {
                    *reinterpret_cast<u32x4*>(L.gt + slab * 1024 + lane * 16) = u32x4{0, 0, 0, 0};
                }
            }
            const unsigned char* bsrc =
                reinterpret_cast<const unsigned char*>(tile_blocks + (size_t)tile * block_stride * kIdBlockElems);
            const int bytes = n_blocks * kIdBlockElems * 2;
            for (int s = wave; s * 1024 < bytes; s += kWgWaves) {
                const int off = s * 1024 + lane * 16;
                if (off < bytes) __builtin_amdgcn_global_load_lds(bsrc + off, (lds_ptr_t)(L.blocks + s * 1024), 16, 0, 0);
            }
            // the zero row that the map's LDS offsets name; a tile of row numbers may have put a row there
            if ((flags & kTileLdsOffsets) && tid < kRowBytes / 16) reinterpret_cast<u32x4*>(L.rows + kRowCap * kRowBytes)[tid] = u32x4{0, 0, 0, 0};
            if (cur_next < t1) resolve(cur_next);
        }
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        // Row numbers -> LDS offsets, two to a word.  kWgStaged on whole blocks: an id block per wave at a time, a scalar loop, 1 to 5 %
        // less of launches of which no tile takes it (1x1x1 map of 940 k voxels, 128 -> 128, 359 -> 341 us).  Elsewhere that form cost
        // registers: kWgAll, where tiles listed pair by pair are most of the work, 3 to 5 % slower (map from a padded grid of 1.03 M,
        // 128 -> 128, 484 / 499), partial blocks 2 to 7 % (96 -> 96 on 200 k scattered voxels 83 / 89).
        if (row_ids) {
            static_assert(kIdBlockElems == 2 * 64, "a word of an id block per lane");
            uint32_t* words = reinterpret_cast<uint32_t*>(L.blocks);
            auto convert = [&](int i) {
                const uint32_t v = words[i];
                words[i] = lds_row_code(min(v & 0xFFFFu, (uint32_t)kWgRowCap)) | lds_row_code(min(v >> 16, (uint32_t)kWgRowCap)) << 16;
            };
            if (MODE == kWgStaged && SHAPE == kWgFull) {
                for (int b = uni(wave); b < n_blocks; b += W) convert(b * 64 + lane);
            } else {
                for (int i = tid; i < n_blocks * 64; i += 64 * W) convert(i);
            }
            __syncthreads();
        }

        // ---- multiply
#pragma unroll
        for (int j = 0; j < kWgOffsetsPerWave; ++j) {
            const int kappa = wave + kWgWaves * j;
            if (kappa >= K3) continue;
#pragma unroll
            for (int fw = 0; fw < kTileWaves; ++fw) {
                const uint32_t wm = wmask[fw];
                if (!((wm >> kappa) & 1u)) continue;
                const int b = block0[fw] + __popc(wm & ((1u << kappa) - 1u));
                const unsigned char* blk = L.blocks + (size_t)b * kGroup * 8;
                u32x2 ids = u32x2{0, 0}, idv[2][2];
                vec8 ga[2][2];
                if (general) {
                    ids = *reinterpret_cast<const u32x2*>(blk + n * 8);
                } else {
#pragma unroll
                    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                        for (int t = 0; t < 2; ++t) idv[ks][t] = *reinterpret_cast<const u32x2*>(blk + (16 * ks + 8 * h + 4 * t + jv) * 8);
                }
#pragma unroll
                for (int gi = 0; gi < kGroupsPerWave; ++gi) {
                    // general tiles: the rows of voxel lane % 32 in two groups are requested before the first of their
                    // products, so that the two latencies overlap (all four at once do not fit the registers)
                    if (general && (gi & 1) == 0) {
#pragma unroll
                        for (int gj = gi; gj < gi + 2; ++gj) {
                            if (!((gmask[tile_group_of(fw, gj)] >> kappa) & 1u)) continue;
                            const uint32_t id = (ids[gj >> 1] >> (16 * (gj & 1))) & 0xFFFFu;
                            const bool staged = id < (uint32_t)n_staged;
                            const int row = staged ? (int)id : kWgRowCap;
                            // pieces h and h + 2 of the row; a piece beyond the row's end is zero (the identity product
                            // below sums over all 32 channels)
                            const bool has0 = h * 8 < ci_n, has1 = h * 8 + 16 < ci_n;
                            ga[gj & 1][0] = *reinterpret_cast<const vec8*>(L.rows + lds_row_offset(has0 ? row : kWgRowCap, h));
                            ga[gj & 1][1] = *reinterpret_cast<const vec8*>(L.rows + lds_row_offset(has1 ? row : kWgRowCap, h + 2));
                            if (!staged && id != kNoRow) {
                                const int64_t gr = id < (uint32_t)win_n ? (int64_t)win_lo + id : (int64_t)my_rows[id - win_n];
                                const uint16_t* src = feat + gr * C_in + cib * kWgCi + h * 8;
                                if (has0) ga[gj & 1][0] = *reinterpret_cast<const vec8*>(src);
                                if (has1) ga[gj & 1][1] = *reinterpret_cast<const vec8*>(src + 16);
                            }
                        }
                    }
                    const int g = tile_group_of(fw, gi);
                    if (!((gmask[g] >> kappa) & 1u)) continue;
                    vec8 fT[2];
                    if (!general) {
#pragma unroll
                        for (int ks = 0; ks < 2; ++ks) {
                            u32x2 w[2];
#pragma unroll
                            for (int t = 0; t < 2; ++t) {
                                const uint32_t id = (idv[ks][t][gi >> 1] >> (16 * (gi & 1))) & 0xFFFFu;
                                w[t] = tr_read4(L.rows + ((id ^ a_piece) + half8));
                            }
                            fT[ks] = vec8_from_words<T>(u32x4{w[0][0], w[0][1], w[1][0], w[1][1]});
                        }
                    } else {
                        f32x16 t;
#pragma unroll
                        for (int v = 0; v < 16; ++v) t[v] = 0.f;
                        t = Elem<T>::mfma(ga[gi & 1][0], ident[0], t);
                        t = Elem<T>::mfma(ga[gi & 1][1], ident[1], t);
                        fT[0] = pack8<T>(t, 0);
                        fT[1] = pack8<T>(t, 8);
                    }
#pragma unroll
                    for (int cb = 0; cb < kHalves; ++cb) {
                        if (kMasked && cb == 1 && co_n <= 32) continue;
#pragma unroll
                        for (int ks = 0; ks < 2; ++ks) {
                            // slots 32g + 16ks + 8h + jv (+ 4), channels 32cb + 16g1 + 4q .. + 3: piece 4cb + 2g1 + q/2
                            // (after the identity product the A fragment holds voxels 4h .. 4h + 3 and 8 + 4h .. 8 + 4h + 3 instead)
                            const int slot = g * kGroup + 16 * ks + (general ? 4 : 8) * h + jv;
                            const uint32_t pos = (uint32_t)((4 * cb + 2 * g1 + (q >> 1)) ^ (((slot >> 1) & 1) << 2)) << 4;
                            const unsigned char* src = L.gt + slot * kGoutRowBytes + pos + half8;
                            const u32x2 lo = tr_read4(src);
                            const u32x2 hi = tr_read4(src + (general ? 8 : 4) * kGoutRowBytes);
                            acc[j][cb] = Elem<T>::mfma(fT[ks], vec8_from_words<T>(u32x4{lo[0], lo[1], hi[0], hi[1]}), acc[j][cb]);
                        }
                    }
                }
            }
        }
        __syncthreads();
        cur = cur_next;
    }

    // ---- partial sums of this range: lane (co = n, h), register 4b + r  ->  ci = 8b + 4h + r
#pragma unroll
    for (int j = 0; j < kWgOffsetsPerWave; ++j) {
        const int kappa = wave + kWgWaves * j;
        if (kappa >= K3) continue;
        float* dst = part + (((int64_t)range * K3 + kappa) * C_in + cib * kWgCi) * C_out + cob * kWgCo + n;
#pragma unroll
        for (int cb = 0; cb < kHalves; ++cb)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int ci = 8 * (v >> 2) + 4 * h + (v & 3);
                if (ci < ci_n && cb * 32 + n < co_n) dst[(int64_t)ci * C_out + cb * 32] = acc[j][cb][v];
            }
    }
    if (!kMasked) return;

    // A sum runs over the pairs that exist; the product gives a missing pair a row of zeros, which adds nothing unless
    // the voxel's gout is infinite or NaN (and the identity product mixes such a value of feat into its whole row).  Either
    // leaves sums that are not finite: the wave makes the sums of such an offset again, pair by pair.
    uint32_t again = 0;
#pragma unroll
    for (int j = 0; j < kWgOffsetsPerWave; ++j) {
        bool odd = false;
#pragma unroll
        for (int cb = 0; cb < kHalves; ++cb) {
            float all = 0.f;                          // of the channels that exist (whole pieces of eight)
#pragma unroll
            for (int p = 0; p < 4; ++p)
                if (8 * p < ci_n) all += (acc[j][cb][4 * p] + acc[j][cb][4 * p + 1]) + (acc[j][cb][4 * p + 2] + acc[j][cb][4 * p + 3]);
            odd |= cb * 32 + n < co_n && !isfinite(all);
        }
        if (__ballot(odd)) again |= 1u << j;
    }
#pragma unroll 1
    for (; again; again &= again - 1) {
        const int kappa = wave + kWgWaves * (__ffs(again) - 1);
        if (kappa >= K3) continue;
        float sum[kHalves][16];
#pragma unroll
        for (int cb = 0; cb < kHalves; ++cb)
#pragma unroll
            for (int v = 0; v < 16; ++v) sum[cb][v] = 0.f;
#pragma unroll 1
        for (int64_t c = next_mine(t0); c < t1; c = next_mine(c + 1)) {
            const int64_t tile = c;
            const TileHeader* H = tile_hdr + tile;
            const int flags = uni(H->flags), win_lo = uni(H->win_lo), win_n = uni(H->win_n), n_valid = uni(H->n_out);
#pragma unroll 1
            for (int g = 0; g < kGroupsPerTile; ++g) {
                if (!(((uint32_t)uni((int)H->group_mask[g]) >> kappa) & 1u)) continue;
                // lane n: the row of voxel n of the column block at this offset, and its output
                const int fw = tile_wave_of(g);
                const uint32_t wm = (uint32_t)uni((int)H->wave_mask[fw]);
                const size_t b = (size_t)tile * block_stride + (uint32_t)uni((int)H->wave_block0[fw]) + __popc(wm & ((1u << kappa) - 1u));
                const uint32_t id = tile_blocks[b * kIdBlockElems + n * kGroupsPerWave + tile_slot_of(g)];
                const int local = tile_perm[tile * kTileT + g * kGroup + n];
                const int row = local < n_valid ? tile_row_of(id, flags, win_lo, win_n, tile_rows + tile * (int64_t)row_stride) : -1;
#pragma unroll 1
                for (uint32_t m = (uint32_t)__ballot(row >= 0); m; m &= m - 1) {
                    const int voxel = __ffs(m) - 1;
                    const uint16_t* x = feat + (int64_t)__shfl(row, voxel) * C_in + cib * kWgCi;
                    const uint16_t* y = gout + (tile * kTileT + __shfl(local, voxel)) * (int64_t)C_out + cob * kWgCo + n;
                    float yv[kHalves];
#pragma unroll
                    for (int cb = 0; cb < kHalves; ++cb) yv[cb] = cb * 32 + n < co_n ? Elem<T>::to_float(y[cb * 32]) : 0.f;
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int ci = 8 * (v >> 2) + 4 * h + (v & 3);
                        const float xv = ci < ci_n ? Elem<T>::to_float(x[ci]) : 0.f;
#pragma unroll
                        for (int cb = 0; cb < kHalves; ++cb) sum[cb][v] = fmaf(xv, yv[cb], sum[cb][v]);
                    }
                }
            }
        }
        float* dst = part + (((int64_t)range * K3 + kappa) * C_in + cib * kWgCi) * C_out + cob * kWgCo + n;
#pragma unroll
        for (int cb = 0; cb < kHalves; ++cb)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int ci = 8 * (v >> 2) + 4 * h + (v & 3);
                if (ci < ci_n && cb * 32 + n < co_n) dst[(int64_t)ci * C_out + cb * 32] = sum[cb][v];
            }
    }
}

// The partial sums part[n_ranges][K3][C_in][C_out] of the map's tiles; staged_only: the sixteen-wave launch, which leaves
// out tiles that are not staged (see WgradMode).
template <typename T>
hipError_t launch_wgrad_tiles(const fx_kmap* km, const void* d_feat, const void* d_gout, int C_in, int C_out, float* part, int n_ranges,
                              bool staged_only, hipStream_t st) {
    const int n_cblk = ((C_in + kWgCi - 1) / kWgCi) * ((C_out + kWgCo - 1) / kWgCo);
    const size_t lds = sizeof(WgradLds);
    hipError_t e = hipSuccess;
#define FX_WGRAD_ONE(W, MODE, SHAPE)                                                                                   \
    do {                                                                                                               \
        e = hipFuncSetAttribute((const void*)k_wgrad_mfma<T, W, MODE, SHAPE>,                                          \
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);                                 \
        if (e == hipSuccess) {                                                                                         \
            k_wgrad_mfma<T, W, MODE, SHAPE><<<(unsigned)(n_cblk * n_ranges), 64 * W, lds, st>>>(                       \
                km->d_tile_hdr, km->d_tile_perm, km->d_tile_rows, km->row_stride, km->d_tile_blocks, km->block_stride, \
                km->n_tiles, n_ranges, (const uint16_t*)d_feat, (const uint16_t*)d_gout, C_in, C_out, km->K3, part);   \
            e = hipGetLastError();                                                                                     \
        }                                                                                                              \
    } while (0)
#define FX_WGRAD_SHAPE(SHAPE)                                                                                          \
    do {                                                                                                               \
        if (staged_only) FX_WGRAD_ONE(16, kWgStaged, SHAPE);                                                           \
        else FX_WGRAD_ONE(8, kWgAll, SHAPE);                                                                           \
    } while (0)
    if (C_in % kWgCi == 0 && C_out % kWgCo == 0) FX_WGRAD_SHAPE(kWgFull);
    else if (C_out <= 32) FX_WGRAD_SHAPE(kWgNarrow);
    else FX_WGRAD_SHAPE(kWgPartial);
#undef FX_WGRAD_SHAPE
#undef FX_WGRAD_ONE
    return e;
}

}  // namespace fx
