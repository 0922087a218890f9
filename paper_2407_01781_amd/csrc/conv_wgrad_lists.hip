// Weight gradient of wide layers (both channel counts multiples of 256) of a 16-bit type: a matrix product per offset over
// the list of its pairs.  Listing, product and reduction kernels, and their launch.
#include "conv_common.h"

namespace fx {

namespace {

constexpr int kListBlk = 256;                      // channels of a block, both sides
constexpr int kListUnit = 32;                      // pairs of a stage: of one tile and offset
constexpr int kListSide = kListBlk / 64, kListWaves = kListSide * kListSide;
constexpr int kListRow = kListBlk * 2, kListSlabRows = 1024 / kListRow;       // bytes of a staged row; rows of a wave's 1 KB slab
constexpr int kListSideBytes = kListUnit * kListRow, kListStageBytes = 2 * kListSideBytes;
constexpr int kListRing = 4;                       // stages in LDS
constexpr int kListEntryBytes = kListWaves * 256;  // list entries of a stage, a word per lane
constexpr int kListTable = 3072;                   // units of a piece in the LDS table at a time
constexpr int kListLds = kListRing * (kListStageBytes + kListEntryBytes) + kListTable * 4 + 256;
constexpr uint32_t kNoPair = 0xFFFFFFFFu;
constexpr int kListRowBits = 32 - 9;               // of an entry: input row, output inside the tile
constexpr int kListMaxTiles = 4096;                // 226 MB of lists (what the bound costs beyond: sheets, 256 -> 256, 1.99 M voxels 2.80 ms, 2.10 M 5.13)
static_assert(kTileT == 512 && kListLds <= 160 * 1024, "entry format; LDS budget");
static_assert(kListSlabRows * kListWaves == kListUnit, "a slab of either side per wave");

// In the tile kernel (k_wgrad_mfma) a block of 32 voxels that has an offset is multiplied whole, and on thin surfaces, where
// the voxels of a block have few of their offsets in common, more than half of the products are with rows of zeros (0.45 of
// them count on sheets); its LDS, which holds a tile's rows for all offsets, leaves a wave 32 x 64 channels, three reads of a
// fragment for two multiplies.  Here the pairs of an offset are listed without gaps first (k_pair_lists; 0.93 count), and a
// workgroup multiplies them like any matrix product, 256 x 256 channels at a time: four fragments for four multiplies, every row
// fetched once per pair.  195 k voxels of sheets, 256 -> 256, bf16, whole call: 527 -> 280 us (listing 20, product 245,
// reduction 14).  What bounds the product is its gathers: 1.7 GB of rows from beyond L2 at 7 TB/s (the same rows from
// L2 alone, by masked row numbers, and the loop before its reads ran ahead: 277).  The multiplies take 103 us.  Forward, input
// and weight gradient one after the other gain less than this call alone, 1396 -> 1271 us: the chip's clock follows its power,
// and the two convolutions beside the denser kernel ran 9 % slower.

// Loads straight from global memory to LDS (16 or 4 bytes a lane, to lds + 16 or 4 * lane), written out: behind the builtin the
// compiler lets no LDS read pass before all such loads have arrived, and the next three stages' would be waited for with this
// one's.  They are counted by hand; m0, which holds the LDS address, is the only register that they write.
__device__ __forceinline__ uint32_t lds_address(const void* p) { return (uint32_t)(uintptr_t)(lds_ptr_t)p; }
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"      // that m0 is not preserved is what the list says
__device__ __forceinline__ void to_lds16(const void* src, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(lds) : "m0", "memory");
}
__device__ __forceinline__ void to_lds4(const void* src, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" ::"v"(src), "s"(lds) : "m0", "memory");
}
#pragma clang diagnostic pop

__device__ __forceinline__ int units_of(int pairs) { return (pairs + kListUnit - 1) / kListUnit; }

// Runs that the units are cut into: no more than there are units, so that every run from the first to the last of an offset has units
// of it and writes the partial sum that the reduction reads.  (The map of one grid has a unit per 32 outputs at its centre offset alone;
// a map between two grids that hardly touch has any number, down to none.)
__device__ __forceinline__ int runs_with_units(int n_units, int n_runs) { return max(1, min(n_units, n_runs)); }

}  // namespace

// The pairs of every (tile, offset), packed: list[tile][kappa][0 .. n-1] = input row << 9 | output inside the tile, in the
// tile's order, then kNoPair up to a multiple of 32; counts[kappa][tile] = n.  Thread = output slot of the tile.
template <int K3MAX>
__global__ void __launch_bounds__(kTileT)
k_pair_lists(const TileHeader* __restrict__ tile_hdr, const uint16_t* __restrict__ tile_perm, const int32_t* __restrict__ tile_rows,
             int row_stride, const uint16_t* __restrict__ tile_blocks, int block_stride, int K3, int n_tiles, int tiles_pad,
             uint16_t* __restrict__ counts, uint32_t* __restrict__ list, uint32_t* __restrict__ zeros) {
    constexpr int kWaves = kTileT / 64;
    __shared__ int cnt[K3MAX][kWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, tile = blockIdx.x;
    if (tile == n_tiles) {                         // one workgroup more: the padding of the counts and the row of zeros
        for (int e = tid; e < K3 * (tiles_pad - n_tiles); e += kTileT) counts[(size_t)(e / (tiles_pad - n_tiles)) * tiles_pad + n_tiles + e % (tiles_pad - n_tiles)] = 0;
        if (tid < kListRow / 4) zeros[tid] = 0;
        return;
    }
    const TileHeader* H = tile_hdr + tile;
    const int flags = uni(H->flags), win_lo = uni(H->win_lo), win_n = uni(H->win_n), n_valid = uni(H->n_out);
    const int g = tid / kGroup, n = tid % kGroup, cw = tile_wave_of(g);
    const uint32_t wm = H->wave_mask[cw];
    const uint16_t* ids = tile_blocks + ((size_t)tile * block_stride + H->wave_block0[cw]) * kIdBlockElems + n * kGroupsPerWave + tile_slot_of(g);
    const int32_t* rows = tile_rows + (int64_t)tile * row_stride;
    const int local = tile_perm[(int64_t)tile * kTileT + tid];
    const uint32_t mine = local < n_valid ? wm : 0u;
    // every lane issues every load (one that has none repeats its first), so that all of them are in flight together
    int32_t row[K3MAX];
#pragma unroll
    for (int k = 0; k < K3MAX; ++k) row[k] = ids[(size_t)__popc(wm & ((1u << k) - 1u) & ((mine >> k) & 1u ? ~0u : 0u)) * kIdBlockElems];
#pragma unroll
    for (int k = 0; k < K3MAX; ++k) {
        uint32_t id = (uint32_t)row[k];
        if (flags & kTileLdsOffsets) id = id / kRowBytes == (uint32_t)kRowCap ? kNoRow : id / kRowBytes;
        row[k] = (mine >> k) & 1u ? (int32_t)id : (int32_t)kNoRow;
    }
    int32_t far[K3MAX];
#pragma unroll
    for (int k = 0; k < K3MAX; ++k) {
        const uint32_t id = (uint32_t)row[k];
        far[k] = rows[id != kNoRow && id >= (uint32_t)win_n ? id - (uint32_t)win_n : 0u];
    }
#pragma unroll
    for (int k = 0; k < K3MAX; ++k) {
        const uint32_t id = (uint32_t)row[k];
        row[k] = id == kNoRow ? -1 : id < (uint32_t)win_n ? win_lo + (int32_t)id : far[k];
    }
#pragma unroll
    for (int k = 0; k < K3MAX; ++k) {
        const uint64_t b = __ballot(row[k] >= 0);
        if (lane == 0) cnt[k][wave] = __popcll(b);
    }
    __syncthreads();
    uint32_t* mylist = list + (size_t)tile * K3 * kTileT;
    const uint64_t below = (1ull << lane) - 1;
#pragma unroll
    for (int k = 0; k < K3MAX; ++k) {
        if (k >= K3) continue;
        int at = 0, total = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) { const int c = cnt[k][w]; at += w < wave ? c : 0; total += c; }
        const uint64_t b = __ballot(row[k] >= 0);
        if (row[k] >= 0) mylist[k * kTileT + at + __popcll(b & below)] = (uint32_t)row[k] << 9 | (uint32_t)local;
        if (tid < units_of(total) * kListUnit - total) mylist[k * kTileT + total + tid] = kNoPair;
        if (tid == 0) counts[(size_t)k * tiles_pad + tile] = (uint16_t)total;
    }
}

// gw[kappa] = sum over the pairs of kappa of feat[in]^T gout[out], the pairs as the contracted dimension.  A workgroup owns 256 x 256
// channels, a wave 64 x 64 of them, and a run of units (32 pairs of one tile and offset), one of `n_runs` equal ones
// of all units in order of offset and tile (fewer if there are fewer units: the last workgroups then have none); where a run passes from one offset to the next it ends one partial sum and starts another.
template <typename T>
__global__ void __launch_bounds__(64 * kListWaves)
k_wgrad_lists(const uint16_t* __restrict__ counts, int n_tiles, int tiles_pad, const uint32_t* __restrict__ list, int K3, int n_runs,
              const unsigned char* __restrict__ feat, const unsigned char* __restrict__ gout, const unsigned char* __restrict__ zeros,
              int C_in, int C_out, float* __restrict__ part, int32_t* __restrict__ unit_base) {
    typedef typename Elem<T>::vec8 vec8;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    int32_t* table = reinterpret_cast<int32_t*>(lds_raw + kListRing * (kListStageBytes + kListEntryBytes));      // tile << 6 | unit of the tile
    int32_t* small = table + kListTable;                            // wave sums, totals per offset
    const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
    const int n_ib = C_in / kListBlk, n_jobs = n_ib * (C_out / kListBlk);
    int job = blockIdx.x % n_jobs, run = blockIdx.x / n_jobs;
    if (n_runs % 8 == 0) {
        job = (blockIdx.x >> 3) % n_jobs;
        run = (int)(blockIdx.x / (8 * n_jobs)) * 8 + (blockIdx.x & 7);
    }
    const int ib = job % n_ib, ob = job / n_ib;

    // ---- units per offset, and where they start
    for (int k = wave; k < K3; k += kListWaves) {
        int sum = 0;
        for (int t = lane * 8; t < tiles_pad; t += 64 * 8) {
            const u32x4 c = *reinterpret_cast<const u32x4*>(counts + (size_t)k * tiles_pad + t);
#pragma unroll
            for (int e = 0; e < 4; ++e) sum += units_of(c[e] & 0xFFFF) + units_of(c[e] >> 16);
        }
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) sum += __shfl_xor(sum, d);
        if (lane == 0) small[kListWaves + k] = sum;
    }
    __syncthreads();
    int upto = lane < K3 ? small[kListWaves + lane] : 0;            // lane kappa: units of offsets 0 .. kappa
#pragma unroll
    for (int d = 1; d < 32; d <<= 1) {
        const int o = __shfl_up(upto, d);
        if (lane >= d) upto += o;
    }
    const int n_units = __builtin_amdgcn_readlane(upto, K3 - 1);
    if (blockIdx.x == 0 && tid < K3) unit_base[1 + tid] = upto;
    if (blockIdx.x == 0 && tid == 0) unit_base[0] = 0;
    const int runs = runs_with_units(n_units, n_runs);
    const int u0 = (int)((int64_t)n_units * min(run, runs) / runs), u1 = (int)((int64_t)n_units * min(run + 1, runs) / runs);

    // ---- this wave's part of a stage: slab `wave` of either side
    const int wi = wave % kListSide, wo = wave / kListSide;
    const int lrow = wave * kListSlabRows + lane / (64 / kListSlabRows), lpos = lane % (64 / kListSlabRows);
    const uint32_t lpiece = (uint32_t)(lpos ^ ((lrow & 3) << 2)) * 16;      // 16-byte piece p of row r sits at p ^ 4 (r & 3): see the reads
    const unsigned char* fx0 = feat + (size_t)ib * kListRow + lpiece;
    const unsigned char* gx0 = gout + (size_t)ob * kListRow + lpiece;
    const unsigned char* z0 = zeros + lpiece;
    const uint32_t pin = (uint32_t)C_in * 2, pout = (uint32_t)C_out * 2;

    // ---- what this lane's address contributes to a transposing read: row jv of four, channels 16 g1 + 4 q .. + 3
    const int h = lane >> 5, q = lane & 3, jv = (lane >> 2) & 3, g1 = (lane >> 4) & 1;
    uint32_t tx[2], tg[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const uint32_t r = (uint32_t)(8 * h + jv) * kListRow + ((q & 1) << 3);
        tx[t] = r + (uint32_t)(((wi * 8 + 4 * t + 2 * g1 + (q >> 1)) ^ (jv << 2)) << 4);
        tg[t] = r + (uint32_t)(((wo * 8 + 4 * t + 2 * g1 + (q >> 1)) ^ (jv << 2)) << 4);
    }
    f32x16 acc[2][2];

    int base_k = 0;
    for (int k = 0; k < K3; ++k) {
        const int end_k = __builtin_amdgcn_readlane(upto, k);
        const int a = max(u0, base_k) - base_k, b = min(u1, end_k) - base_k;      // the run's units of this offset
        base_k = end_k;
        if (a >= b) continue;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int o = 0; o < 2; ++o)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][o][v] = 0.f;
        const uint32_t* klist = list + (size_t)k * kTileT;
        for (int a0 = a; a0 < b; a0 += kListTable) {
            const int n = min(b - a0, kListTable);
            // ---- the table of units a0 .. a0 + n - 1 of the offset: a thread per tile
            __syncthreads();
            int seen = 0;
            for (int t0 = 0; t0 < n_tiles && seen < a0 + n; t0 += 64 * kListWaves) {
                const int t = t0 + tid;
                const int nu = t < n_tiles ? units_of(counts[(size_t)k * tiles_pad + t]) : 0;
                int incl = nu;
#pragma unroll
                for (int d = 1; d < 64; d <<= 1) {
                    const int o = __shfl_up(incl, d);
                    if (lane >= d) incl += o;
                }
                if (lane == 63) small[wave] = incl;
                __syncthreads();
                int at = seen + incl - nu;
#pragma unroll
                for (int w = 0; w < kListWaves; ++w) { const int s = small[w]; at += w < wave ? s : 0; seen += s; }
                for (int u = max(0, a0 - at); u < nu && at + u < a0 + n; ++u) table[at + u - a0] = t << 6 | u;
                __syncthreads();
            }
            const uint32_t ring = uni((int)lds_address(lds_raw)), entry_ring = ring + kListRing * kListStageBytes + wave * 256;
            auto unit_of = [&](int t) __attribute__((always_inline)) { return uni(table[min(t, n - 1)]); };
            // the list entries of the wave's rows in stage t, a lane the one whose row it loads
            auto entries = [&](int t) __attribute__((always_inline)) {
                const int w = unit_of(t);
                to_lds4(klist + (size_t)(w >> 6) * K3 * kTileT + (w & 63) * kListUnit + lrow, entry_ring + (uint32_t)(t % kListRing) * kListEntryBytes);
            };
            auto rows = [&](int t) __attribute__((always_inline)) {
                const uint32_t v = *reinterpret_cast<const uint32_t*>(lds_raw + kListRing * kListStageBytes + (t % kListRing) * kListEntryBytes + tid * 4);
                const bool on = t < n && v != kNoPair;
                const unsigned char* x = fx0 + (uint64_t)(v >> 9) * pin;
                const unsigned char* y = gx0 + (uint64_t)((uint32_t)(unit_of(t) >> 6) * kTileT + (v & 511u)) * pout;
                x = on ? x : z0;
                y = on ? y : z0;
                const uint32_t dst = ring + (uint32_t)(t % kListRing) * kListStageBytes + wave * 1024;
                to_lds16(x, dst);
                to_lds16(y, dst + kListSideBytes);
            };
            struct Frags { vec8 x[2], y[2]; };
            auto read = [&](Frags& f, int t, int ks) __attribute__((always_inline)) {
                const unsigned char* st = lds_raw + (t % kListRing) * kListStageBytes + ks * 16 * kListRow;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const unsigned char *px = st + tx[i], *py = st + kListSideBytes + tg[i];
                    const u32x2 xl = tr_read4(px), xh = tr_read4(px + 4 * kListRow), yl = tr_read4(py), yh = tr_read4(py + 4 * kListRow);
                    f.x[i] = vec8_from_words<T>(u32x4{xl[0], xl[1], xh[0], xh[1]});
                    f.y[i] = vec8_from_words<T>(u32x4{yl[0], yl[1], yh[0], yh[1]});
                }
            };
            auto multiply = [&](const Frags& f) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int o = 0; o < 2; ++o) acc[i][o] = Elem<T>::mfma(f.x[i], f.y[o], acc[i][o]);
            };
            // Rows of stage t + 1 have arrived for all waves (of this wave's loads the newest seven may be under way: entries, then rows and entries
            // of the two stages after it, and the entries of stage t + 4 have arrived too), and everybody has read stage t,
            // whose place those of stage t + 4 take.
            auto hand_over = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt vmcnt(7) lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
#pragma unroll
            for (int t = 0; t < kListRing; ++t) entries(t);
            __builtin_amdgcn_s_waitcnt(0);
#pragma unroll
            for (int t = 0; t < kListRing; ++t) { rows(t); entries(t + kListRing); }
            asm volatile("s_waitcnt vmcnt(9) lgkmcnt(0)\n\ts_barrier" ::: "memory");           // stage 0
            Frags f0, f1;
            read(f0, 0, 0);
            for (int t = 0; t < n; ++t) {
                read(f1, t, 1);
                multiply(f0);
                hand_over();
                read(f0, t + 1, 0);
                multiply(f1);
                rows(t + kListRing);
                entries(t + 2 * kListRing);
            }
            __builtin_amdgcn_s_waitcnt(0);
        }
        // ---- the piece's sums: lane (co = n, h), register v -> ci = 8 (v / 4) + 4 h + v % 4
        float* dst = part + ((size_t)job * (n_runs + K3) + run + k) * (kListBlk * kListBlk) + (size_t)(wi * 64 + 4 * h) * kListBlk + wo * 64 + (lane & 31);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int o = 0; o < 2; ++o)
#pragma unroll
                for (int v = 0; v < 16; ++v) dst[(size_t)(32 * i + 8 * (v >> 2) + (v & 3)) * kListBlk + 32 * o] = acc[i][o][v];
    }
}

// gw from the partial sums: those of an offset are adjacent, one per run that has units of it, and are added in that order.
template <int OUT_DT>
__global__ void __launch_bounds__(256) k_wgrad_lists_reduce(const float* __restrict__ part, const int32_t* __restrict__ unit_base, int K3, int n_runs, int C_in, int C_out,
                                     void* __restrict__ gw) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int per_k = C_in * C_out / 4;
    const int k = (int)(blockIdx.x * (int64_t)blockDim.x / per_k);            // a workgroup stays within one offset
    const int e = (int)(q - (int64_t)k * per_k) * 4, ci = e / C_out, co = e % C_out;
    const int job = co / kListBlk * (C_in / kListBlk) + ci / kListBlk;
    const int64_t n = unit_base[K3], f = unit_base[k], l = (int64_t)unit_base[k + 1] - 1;
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    if (f <= l) {
        // run r holds units n r / runs (rounded down) and on: that of unit u is the last r with n r / runs <= u
        const int runs = runs_with_units((int)n, n_runs);
        const int r0 = (int)(((f + 1) * runs - 1) / n), r1 = (int)(((l + 1) * runs - 1) / n);
        const float* p = part + ((size_t)job * (n_runs + K3) + r0 + k) * (kListBlk * kListBlk) + (ci % kListBlk) * kListBlk + co % kListBlk;
        const int cnt = r1 - r0 + 1;
        for (int r = 0; r < cnt; r += 8) {
            f32x4 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const f32x4*>(p + (size_t)min(r + u, cnt - 1) * (kListBlk * kListBlk));
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (r + u < cnt) s += v[u];
        }
    }
    if (OUT_DT == FX_F32) *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(gw) + 4 * q) = s;
    else {
        typedef typename std::conditional<OUT_DT == FX_F16, _Float16, __bf16>::type T;
        *reinterpret_cast<u32x2*>(reinterpret_cast<uint16_t*>(gw) + 4 * q) = u32x2{Elem<T>::pack2(s[0], s[1]), Elem<T>::pack2(s[2], s[3])};
    }
}

// Whether the lists serve a stride-1 map and pay.  Their listing launch and the partial sums (74 MB at 256 -> 256) cost 20 to 60 us
// whatever the map; the tile kernel stages every row once per block of 32 x 64 channels.  The line is in outputs x blocks of 256 x 256.
// bf16, tile kernel / lists, whole call, us, 256 -> 256:
//   24 k from 8 voxels a leaf on: sheets 13 k voxels 66 / 68, 25 k 100 / 76, 57 k 166 / 114, 195 k 534 / 281; spheres 9.9 k 49 / 65,
//     26 k 102 / 85, 41 k 115 / 105; indoor 10.5 k 46 / 64, 21 k 67 / 76, 88 k 178 / 159; random voxels, 24 a leaf, 23.7 k 74 / 75, 27 k
//     82 / 64, 14 a leaf, 24.6 k 61 / 62, 29 k 69 / 64, 10 a leaf, 24.6 k 58 / 62, 26.5 k 62 / 62, 29 k 68 / 62; LiDAR 85 k 194 / 157, 269 k 587 / 396; 256 -> 512 on 9.9 k 70 / 78, 41 k 208 / 155; 512 -> 512 on 140 k 1224 / 710
//   32 k where a leaf has few voxels, and a voxel few pairs: random voxels, 1 to 7 a leaf, 24 k 50..54 / 60..62, 28 k 55..61 / 61..62,
//     33 k 62..68 / 62..64, 56 k 88..99 / 65..70; 512 -> 512 on 6.3 k 54..58 / 59..61, 8.4 k 65..70 / 60..62; but with full leaves among
//     them, whose tiles the tile kernel has side by side in one range, 24 k again: 7 voxels a leaf, 24 k with 2 % in full leaves 60 / 62, 4 %
//     64 / 63, 8 % 73 / 64, 17 % in one body 89 / 68
//   40 k for the one pair a voxel of a 1x1x1 map: 24 k 32 / 49, 30 k 43 / 50, 38 k 52 / 51, 50 k 66 / 53, 393 k 552 / 129; 512 -> 512 on
//     8.1 k 45 / 41
//   24 k between two grids, whose tiles list a row per pair: 32 k outputs, 3x3x3, input all of them 275 / 85, half 117 / 68, hardly any
//     43 / 40; 1x1x1, half 124 / 47, hardly any 25 / 22; 1.03 M of a padded grid 2587 / 365
// Blocks of 128 x 128 channels, which fetch every row twice as often for its products, were measured too: 128 -> 128 on 195 k
// voxels of sheets 158 / 153, LiDAR 269 k 155 / 218, 980 k 538 / 635.
bool wgrad_lists_pays(const fx_kmap* km, fx_dtype dt, int C_in, int C_out) {
    if (dt == FX_F32 || C_in % kListBlk != 0 || C_out % kListBlk != 0 || km->n_in >= (1 << kListRowBits) - 1 || km->n_tiles <= 0 ||
        km->n_tiles > kListMaxTiles)
        return false;
    const int64_t work = km->n_out * (C_in / kListBlk) * (C_out / kListBlk);
    if (km->gin != km->gout) return work >= 24000;
    if (km->K == 1) return work >= 40000;
    return work >= (km->n_in >= (int64_t)8 * km->gin->hdr.n_leaf || 32 * km->gin->hdr.n_voxels_dense >= km->n_in ? 24000 : 32000);
}

fx_status wgrad_lists(const fx_kmap* km, const void* d_feat, const void* d_gout, fx_dtype dt, int C_in, int C_out, void* d_gw, fx_dtype out_dt,
                      hipStream_t st) {
    const int n_jobs = (C_in / kListBlk) * (C_out / kListBlk), K3 = km->K3, n_tiles = (int)km->n_tiles, tiles_pad = (n_tiles + 7) / 8 * 8;
    int n_runs = std::max(1, compute_units() / n_jobs);
    if (n_runs > 8) n_runs -= n_runs % 8;              // see the block-to-XCD mapping in the kernel
    // scratch: partial sums | lists | counts | a row of zeros | the first unit of every offset
    const size_t part_b = sizeof(float) * (size_t)n_jobs * (n_runs + K3) * kListBlk * kListBlk;
    const size_t list_b = sizeof(uint32_t) * (size_t)n_tiles * K3 * kTileT, counts_b = ((size_t)K3 * tiles_pad * 2 + 15) / 16 * 16;
    unsigned char* scratch = nullptr;
    FX_TRY(dev_alloc((void**)&scratch, part_b + list_b + counts_b + kListRow + (kMaxK3Tiled + 1) * sizeof(int32_t), st));
    float* part = (float*)scratch;
    uint32_t* list = (uint32_t*)(scratch + part_b);
    uint16_t* counts = (uint16_t*)(scratch + part_b + list_b);
    uint32_t* zeros = (uint32_t*)(scratch + part_b + list_b + counts_b);
    int32_t* unit_base = (int32_t*)(scratch + part_b + list_b + counts_b + kListRow);
    hipError_t e = hipSuccess;
    {
        ProfScope ps(kProfWgrad, st);
        k_pair_lists<kMaxK3Tiled><<<n_tiles + 1, kTileT, 0, st>>>(km->d_tile_hdr, km->d_tile_perm, km->d_tile_rows, km->row_stride, km->d_tile_blocks,
                                                                  km->block_stride, K3, n_tiles, tiles_pad, counts, list, zeros);
        e = hipGetLastError();
#define FX_LISTS(T)                                                                                                                     \
    do {                                                                                                                                 \
        if (e == hipSuccess) e = hipFuncSetAttribute((const void*)k_wgrad_lists<T>, hipFuncAttributeMaxDynamicSharedMemorySize, kListLds); \
        if (e == hipSuccess) {                                                                                                           \
            k_wgrad_lists<T><<<n_jobs * n_runs, 64 * kListWaves, kListLds, st>>>(counts, n_tiles, tiles_pad, list, K3, n_runs,           \
                (const unsigned char*)d_feat, (const unsigned char*)d_gout, (const unsigned char*)zeros, C_in, C_out, part, unit_base);  \
            e = hipGetLastError();                                                                                                       \
        }                                                                                                                                \
    } while (0)
        if (dt == FX_BF16) FX_LISTS(__bf16);
        else FX_LISTS(_Float16);
#undef FX_LISTS
    }
    if (e == hipSuccess) {
        ProfScope ps(kProfWgradReduce, st);
        const unsigned nb = (unsigned)((size_t)K3 * C_in * C_out / 4 / 256);
        if (out_dt == FX_F32) k_wgrad_lists_reduce<FX_F32><<<nb, 256, 0, st>>>(part, unit_base, K3, n_runs, C_in, C_out, d_gw);
        else if (out_dt == FX_F16) k_wgrad_lists_reduce<FX_F16><<<nb, 256, 0, st>>>(part, unit_base, K3, n_runs, C_in, C_out, d_gw);
        else k_wgrad_lists_reduce<FX_BF16><<<nb, 256, 0, st>>>(part, unit_base, K3, n_runs, C_in, C_out, d_gw);
        e = hipGetLastError();
    }
    dev_free(scratch, st);
    if (e != hipSuccess) { set_error("weight-gradient launch failed: %s", hipGetErrorString(e)); return FX_EDEVICE; }
    return FX_OK;
}

}  // namespace fx
