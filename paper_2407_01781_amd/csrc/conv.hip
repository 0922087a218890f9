// Sparse convolution forward (Sec. 3.5 scenario 3, re-designed for CDNA4).
//
// MFMA path.  A workgroup owns one tile of 512 consecutive output voxels.  The tile's distinct
// input rows are staged once in LDS (the paper's per-offset gathers become LDS reads), the
// per-offset products run on v_mfma_f32_32x32x16_{bf16,f16}, and -- unlike the paper's shared-
// memory scatter buffer -- every output voxel keeps its accumulators in registers for all
// offsets: a column block of 32 outputs is fixed for the whole tile, and an offset contributes
// a block only if one of the 32 has a neighbour there (missing neighbours read a zero row).
// Nothing is scattered; the write-back is one sequential range per tile.
//
// Operand roles in the tile kernel: A = gathered features (32 voxels x 16 input channels per
// instruction), B = packed weights (16 input channels x 32 output channels), D = 32 voxels x 32
// channels with the channels across lanes; the two weight tiles of a 64-channel slice interleave
// the channels (column n of tile t = channel 2n + t), so lane n holds two adjacent channels of
// every voxel and the 32 lanes of a half-wave store one whole output row at a time.  The gather
// kernels for strided maps keep the same roles with their A fragments read straight from global memory.
#include "conv_common.h"
#include "dev_timing.h"

#include <mutex>

namespace fx {

// Whether the tile kernel starts with the items of long tiles, whose rows fill both halves of the row buffer or are gathered from
// global memory (k_conv_mfma): there are more items than workgroups, and the lower half of the last XCD's workgroups has static items (those of the workgroups
// that start with long tiles are claimed like the others).  However many items a workgroup takes, a long one claimed last ends
// the launch alone; where none is claimed late, starting with them costs a percent.  bf16, in the order of the list -> long
// tiles first, us: 269 k LiDAR voxels 256 -> 256 (8.2 items a workgroup) 516 -> 446; 988 k with a solid block among the last
// tiles 64 -> 64 (7.5) 152 -> 126, 128 -> 128 (15) 422 -> 384, 96 -> 192 (23) 480 -> 449; the block among the first 125 -> 127,
// 378 -> 386, 442 -> 448; no block 123.5 -> 124.5, 374 -> 376, 437 -> 437; 1.18 M voxels of indoor scenes 148 -> 147.
__host__ __device__ inline bool long_tiles_first(int64_t n_work, int wgs) {
    const int64_t per_xcd = (n_work + 7) / 8;
    return per_xcd > (wgs >> 3) && 7 * per_xcd + (wgs >> 3) / 2 < n_work;
}

// ---------------------------------------------------------------------------------- weight packing
// Wp[kappa][cin chunk][cout slice][ntile 0..1][kstep 0..1][lane 0..63][8]: the 16-byte B-operand
// fragment of each lane for one (offset, 32 input channels, 64 output channels): lane (n, kq) holds
// the eight input channels 16 * kstep + 8 * kq .. + 7 of column n.  Column n of n-tile t is output
// channel 2n + t of the slice, so that lane n of an accumulator row (32x32 accumulator layout: lane
// half h, register v -> voxel row 8*(v/4) + 4*h + v%4) holds two adjacent channels, one per n-tile,
// and the 32 lanes of a half-wave store one whole output row.  With one n-tile (n_nt = 1) a slice is 32
// channels and column n is channel n of it.
template <typename E>   // uint16_t or uint32_t: the bits of one element
__global__ void k_pack_weights(const E* __restrict__ w, E* __restrict__ wp, int K3, int C_in, int C_out, int n_clear,
                               int32_t* __restrict__ counters, int mode, int n_nt, const uint8_t* __restrict__ tile_long, int64_t n_tiles, PairArgs again) {
    if (blockIdx.x == 0 && (int)threadIdx.x < n_clear) counters[threadIdx.x] = 0;   // the convolution's work-list counters
    if (again.hdr && blockIdx.x == 0 && threadIdx.x == 0) *reinterpret_cast<PairArgs*>(counters + kPairArgsAt) = again;
    if (tile_long && blockIdx.x == gridDim.x - 1) {
        // a workgroup of its own lists the long tiles, in no particular order (their number, then the first kMaxLongTiles of
        // them): the tile kernel starts with those
        __shared__ int32_t found;
        if (threadIdx.x == 0) found = 0;
        __syncthreads();
        const uint32_t* words = reinterpret_cast<const uint32_t*>(tile_long);                // four tiles each; the last one's rest is zero
        const int64_t n_words = (n_tiles + 3) / 4;
        for (int64_t w0 = threadIdx.x; w0 < n_words; w0 += 4 * blockDim.x) {       // four words in flight
            uint32_t is_long[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) is_long[u] = words[min(w0 + u * (int)blockDim.x, n_words - 1)];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t w = w0 + u * (int)blockDim.x;
                uint32_t m = w < n_words ? is_long[u] : 0u;                        // a byte is 0 or 1
                if (!m) continue;
                int at = atomicAdd(&found, __popc(m));
                for (; m && at < kMaxLongTiles; m &= m - 1) counters[9 + at++] = (int32_t)(4 * w) + (__ffs(m) - 1) / 8;
            }
        }
        __syncthreads();
        if (threadIdx.x == 0) { counters[8] = found; counters[9 + kMaxLongTiles] = 0; }
        return;
    }
    constexpr int EPL = 16 / (int)sizeof(E);     // elements per lane fragment
    constexpr int kChunk = 4 * EPL;              // input channels per 64-byte row chunk
    typedef __attribute__((ext_vector_type(EPL))) E Frag;
    const uint32_t cols = 32 * n_nt;                                     // channels of a slice
    const uint32_t nchunk = (C_in + kChunk - 1) / kChunk, nslice = (C_out + cols - 1) / cols;
    const uint32_t total = (uint32_t)K3 * nchunk * nslice * n_nt * 128;  // fragments
    const uint32_t stride = (gridDim.x - (tile_long ? 1 : 0)) * blockDim.x;
    for (uint32_t f = blockIdx.x * blockDim.x + threadIdx.x; f < total; f += stride) {
        const uint32_t lane = f & 63, ks = (f >> 6) & 1;
        uint32_t r = f >> 7;
        const uint32_t nt = n_nt == 2 ? r & 1 : 0;
        if (n_nt == 2) r >>= 1;
        const uint32_t sl = r % nslice; r /= nslice;
        const uint32_t c = r % nchunk, kappa = r / nchunk;
        const int m = lane & 31, kq = lane >> 5;
        const int cin = c * kChunk + ks * 2 * EPL + kq * EPL, cout = sl * cols + n_nt * m + nt;
        Frag v;
        const int64_t kw = (mode & kWeightsFlipped) ? K3 - 1 - kappa : kappa;
        const int64_t at = (mode & kWeightsTransposed) ? (kw * C_out + cout) * C_in + cin : (kw * C_in + cin) * C_out + cout;
        const int64_t step = (mode & kWeightsTransposed) ? 1 : C_out;
        const bool in = cout < C_out && cin < C_in;             // C_in is a multiple of EPL
        if ((mode & kWeightsTransposed) && in && (reinterpret_cast<uintptr_t>(w) & 15) == 0) {
            v = *reinterpret_cast<const Frag*>(w + at);        // a fragment is contiguous
        } else {
#pragma unroll
            for (int el = 0; el < EPL; ++el) v[el] = in ? w[at + el * step] : (E)0;
        }
        reinterpret_cast<Frag*>(wp)[f] = v;
    }
}

size_t packed_weight_bytes(int K3, int C_in, int C_out, int elem_bytes) {
    const int chunk = kRowBytes / elem_bytes;
    return (size_t)elem_bytes * K3 * ((C_in + chunk - 1) / chunk * chunk) * ((C_out + kCoutSlice - 1) / kCoutSlice) * kCoutSlice;
}

void launch_pack_weights(const void* d_w, void* wp, int K3, int C_in, int C_out, int elem_bytes, int32_t* counters,
                         int mode, hipStream_t st, const uint8_t* tile_long, int64_t n_tiles, int n_nt, const PairArgs& again, int n_clear) {
    const int64_t total = (int64_t)(packed_weight_bytes(K3, C_in, C_out, elem_bytes) / 16);
    // small weights in workgroups of one wave, so that every compute unit has one
    const unsigned bs = tile_long || total > 65536 ? 256u : 64u;
    const unsigned nb = (unsigned)std::max<int64_t>(1, std::min<int64_t>((total + bs - 1) / bs, 4096)) + (tile_long ? 1 : 0);
    ProfScope ps(kProfPackWeights, st);
    if (elem_bytes == 2)
        k_pack_weights<uint16_t><<<nb, bs, 0, st>>>((const uint16_t*)d_w, (uint16_t*)wp, K3, C_in, C_out, n_clear, counters, mode, n_nt, tile_long, n_tiles, again);
    else
        k_pack_weights<uint32_t><<<nb, bs, 0, st>>>((const uint32_t*)d_w, (uint32_t*)wp, K3, C_in, C_out, n_clear, counters, mode, n_nt, tile_long, n_tiles, again);
}

// Write-back of one column block computed with the features as the A operand: register v of
// accumulator tile t in lane (n, h) is output channel 2n + t of the slice for the block's slot
// 8*(v/4) + 4*h + v%4.  perm_g points at the block's 32 entries of the tile permutation in LDS
// (slot -> local output number).  Each store instruction covers two whole output rows.
typedef __attribute__((address_space(1))) unsigned char global_byte;

template <typename T, bool OUT_F32, bool FULL, int NT>
__device__ __forceinline__ void store_block_rows_impl(const f32x16 (&acc)[NT], const uint16_t* perm_g, global_byte* tile_out,
                                                      uint32_t row_bytes, uint32_t lane_off, int n_valid, bool lane_ok, int h) {
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const u32x2 lp = *reinterpret_cast<const u32x2*>(perm_g + 8 * b + 4 * h);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t local = (lp[r >> 1] >> (16 * (r & 1))) & 0xFFFFu;
            if (!FULL && ((int)local >= n_valid || !lane_ok)) continue;
            global_byte* dst = tile_out + (uint32_t)(__umul24(local, row_bytes) + lane_off);   // 32-bit offset from a wave-uniform base
            const int v = 4 * b + r;
            if (NT == 1) {
                if (OUT_F32) *reinterpret_cast<__attribute__((address_space(1))) float*>(dst) = acc[0][v];
                else *reinterpret_cast<__attribute__((address_space(1))) uint16_t*>(dst) = (uint16_t)Elem<T>::pack2(acc[0][v], 0.f);
            } else if (OUT_F32) {
                typedef __attribute__((ext_vector_type(2))) float f32x2;
                *reinterpret_cast<__attribute__((address_space(1))) f32x2*>(dst) = f32x2{acc[0][v], acc[NT - 1][v]};
            } else {
                *reinterpret_cast<__attribute__((address_space(1))) uint32_t*>(dst) = Elem<T>::pack2(acc[0][v], acc[NT - 1][v]);
            }
        }
    }
}

// tile_out: first byte of the tile's first output row at the slice's first channel (wave-uniform);
// cols: channels of the slice that exist (64, or fewer in the last slice of a padded channel count).
// The same with the weights held in LDS as fp32 in forward order W'[kappa][ci][co] (read through `mode` once per
// workgroup): at low depth the weight reads are most of the kernel's loads, and all lanes of a wave that work
// on the same four produced channels read the same 16 bytes, which LDS serves as a broadcast.  Few, fat
// workgroups walk the outputs so that the copy of the weights is paid a few thousand times, not per 256 outputs.
// QV: groups of four produced channels per thread.  1 is what runs: with 4 (one thread per voxel and 16 channels)
// the 64 lanes of a wave walk 64 different map rows and input rows, and the kernel took twice as long.
template <int DT, bool OUT_F32, int QV>
__global__ void __launch_bounds__(256)
k_conv_scalar4_ldsw(const int32_t* __restrict__ nbmap, int64_t n_out, int K3, const void* __restrict__ feat,
                    const void* __restrict__ w, int C_in, int C_out, void* __restrict__ out, int mode) {
    extern __shared__ __align__(16) unsigned char lds_w_raw[];
    float* wl = reinterpret_cast<float*>(lds_w_raw);
    const int n_w = K3 * C_in * C_out;
    for (int e = threadIdx.x; e < n_w; e += blockDim.x) {
        const int co = e % C_out, ci = (e / C_out) % C_in, kappa = e / (C_out * C_in);
        const int64_t kw = (mode & kWeightsFlipped) ? K3 - 1 - kappa : kappa;
        const int64_t src = (mode & kWeightsTransposed) ? (kw * C_out + co) * C_in + ci : (kw * C_in + ci) * C_out + co;
        wl[e] = load_as_float<DT>(w, src);
    }
    __syncthreads();
    const int q_out = C_out / (4 * QV);
    const int64_t total = n_out * q_out;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t o = e / q_out;
        const int co = (int)(e - o * q_out) * 4 * QV;
        f32x4 acc[QV];
#pragma unroll
        for (int g = 0; g < QV; ++g) acc[g] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int kappa = 0; kappa < K3; ++kappa) {
            const int32_t in = nbmap[o * K3 + kappa];
            if (in < 0) continue;
            const int64_t fb = (int64_t)in * C_in;
            const float* wk = wl + kappa * C_in * C_out + co;
            for (int ci = 0; ci < C_in; ci += 4) {
                const f32x4 x = load4_as_float<DT>(feat, fb + ci);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
#pragma unroll
                    for (int g = 0; g < QV; ++g) {
                        const f32x4 wr = *reinterpret_cast<const f32x4*>(wk + (ci + j) * C_out + 4 * g);
#pragma unroll
                        for (int v = 0; v < 4; ++v) acc[g][v] = fmaf(x[j], wr[v], acc[g][v]);
                    }
                }
            }
        }
#pragma unroll
        for (int g = 0; g < QV; ++g) {
            const int64_t at = o * C_out + co + 4 * g;
            if (OUT_F32) {
                *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(out) + at) = acc[g];
            } else if (DT == FX_F16) {
                *reinterpret_cast<u32x2*>(reinterpret_cast<uint16_t*>(out) + at) =
                    u32x2{Elem<_Float16>::pack2(acc[g][0], acc[g][1]), Elem<_Float16>::pack2(acc[g][2], acc[g][3])};
            } else {
                *reinterpret_cast<u32x2*>(reinterpret_cast<uint16_t*>(out) + at) =
                    u32x2{Elem<__bf16>::pack2(acc[g][0], acc[g][1]), Elem<__bf16>::pack2(acc[g][2], acc[g][3])};
            }
        }
    }
}

template <typename T, bool OUT_F32, int NT>
__device__ __forceinline__ void store_block_rows(const f32x16 (&acc)[NT], const uint16_t* perm_g, unsigned char* tile_out,
                                                 int C_out, int cols, int n_valid, int n, int h, bool all_rows) {
    const uint32_t esize = OUT_F32 ? 4u : 2u;
    const uint32_t row_bytes = (uint32_t)C_out * esize, lane_off = (uint32_t)NT * (uint32_t)n * esize;
    // keep the base in scalar registers: the stores then take it as their scalar address operand
    const uint64_t bits = reinterpret_cast<uint64_t>(tile_out);
    const uint32_t lo = (uint32_t)uni((int)(uint32_t)bits), hi = (uint32_t)uni((int)(uint32_t)(bits >> 32));
    global_byte* base = (global_byte*)(((uint64_t)hi << 32) | lo);
    if (all_rows && n_valid == kTileT && cols == 32 * NT)      // otherwise: rows beyond the tile's end or left to another kernel (0xFFFF)
        store_block_rows_impl<T, OUT_F32, true, NT>(acc, perm_g, base, row_bytes, lane_off, n_valid, true, h);
    else
        store_block_rows_impl<T, OUT_F32, false, NT>(acc, perm_g, base, row_bytes, lane_off, n_valid, NT * n < cols, h);
}


// offset (in 16-byte fragments, wave-uniform) of the first weight fragment for (slice, chunk, offset)
// (the packed weights of one call stay far below 2^31 fragments)
template <int NT = 2>
__device__ __forceinline__ int w_frag(int nslice, int w_kappa_stride, int slice, int c, int kappa) {
    return ((c * nslice + slice) * 2 * NT) * 64 + kappa * w_kappa_stride;
}

// The products give a missing neighbour a row of zeros, which adds nothing unless a weight is infinite or NaN, and the gather
// kernels multiply what stands for a row's missing end by weights of zero, which adds nothing unless a feature is.  Shapes
// that a scalar kernel served before the matrix units did (C_in not a multiple of 32) keep its sums over existing pairs: a
// column block whose sums are not all finite is summed again here, offset by offset, and only rows that have the offset take
// its product.  One wave alone: the ids of the offset after next, the row numbers of the next one and the operands of the
// next step are in flight while one is multiplied.  A batch that is NaN throughout (an overflow step under loss scaling), 268 k
// LiDAR voxels, bf16, forward, in us, on finite values / here / in the scalar kernel: 3x3x3 48 -> 48 74 / 448 / 922, 24 -> 40 56 /
// 366 / 419; (2,2) map 48 -> 48 21 / 50 / 127; (3,2) map 48 -> 48 43 / 86 / 308.  (A lane per channel walking voxels, offsets and
// channels one after the other took 25 700, 12 200, 2 130 and 4 670.)
template <typename T, bool OUT_F32, int NT, int MT>      // MT n-tiles, from mt0 on, of the NT of a slice of 32 NT channels
__device__ __forceinline__ void sum_pairs_again(const PairArgs& P, const uint16_t* __restrict__ feat, const void* __restrict__ wp, int C_in, int C_out,
                                                int64_t tile, int g, int slice, int mt0, void* __restrict__ out) {
    typedef typename Elem<T>::vec8 vec8;
    const int lane = threadIdx.x & 63, n = lane & 31, h = lane >> 5;
    const int nchunk = (C_in + kCinChunk - 1) / kCinChunk, nslice = (C_out + 32 * NT - 1) / (32 * NT);
    const int w_kappa_stride = nchunk * nslice * 2 * NT * 64;
    const TileHeader* H = P.hdr + tile;
    const uint32_t wm = H->wave_mask[tile_wave_of(g)];
    const uint16_t* ids = P.blocks + ((size_t)tile * P.block_stride + H->wave_block0[tile_wave_of(g)]) * kIdBlockElems + n * kGroupsPerWave + tile_slot_of(g);
    const int flags = H->flags, win_lo = H->win_lo, win_n = H->win_n;
    const int32_t* rows = P.rows + tile * (int64_t)P.row_stride;
    uint32_t rest = (uint32_t)uni((int)H->group_mask[g]);
    auto pop = [&]() { const int k = __ffs(rest) - 1; rest &= rest - 1; return k; };     // -1: no offset left
    auto load_id = [&](int k) -> uint32_t { return k < 0 ? kNoRow : (uint32_t)ids[(size_t)__popc(wm & ((1u << k) - 1u)) * kIdBlockElems]; };
    auto row_behind = [&](uint32_t id) -> int32_t { return tile_row_of(id, flags, win_lo, win_n, rows); };
    auto fetch = [&](int k, int32_t row, int c, vec8 (&b)[2], vec8 (&w)[2 * MT]) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
            for (int e = 0; e < 8; ++e) b[ks][e] = 0;
            const int at = c * kCinChunk + ks * 16 + h * 8;                      // a row that ends inside its last chunk: zeros beyond
            if (row >= 0 && at < C_in) b[ks] = *reinterpret_cast<const vec8*>(feat + (int64_t)row * C_in + at);
        }
        const vec8* ws = reinterpret_cast<const vec8*>(wp) + lane + (w_frag<NT>(nslice, w_kappa_stride, slice, c, max(k, 0)) + mt0 * 128);
#pragma unroll
        for (int f = 0; f < 2 * MT; ++f) w[f] = ws[f * 64];
    };
    f32x16 acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[mt][v] = 0.f;
    int k0 = pop(), k1 = pop(), k2 = pop();
    const uint32_t id0 = load_id(k0), id1 = load_id(k1);
    uint32_t id2 = load_id(k2);
    int32_t r0 = k0 < 0 ? -1 : row_behind(id0), r1 = k1 < 0 ? -1 : row_behind(id1);
    vec8 b[2], w[2 * MT], bn[2], wn[2 * MT];
    fetch(k0, r0, 0, b, w);
#pragma unroll 1
    while (k0 >= 0) {
        const int k3 = pop();
        const uint32_t id3 = load_id(k3);
        const int32_t r2 = k2 < 0 ? -1 : row_behind(id2);
        const uint32_t has = (uint32_t)__ballot(r0 >= 0) >> (4 * h);            // lanes 32 .. 63 repeat lanes 0 .. 31
        f32x16 sum[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int v = 0; v < 16; ++v) sum[mt][v] = 0.f;
#pragma unroll 1
        for (int c = 0; c < nchunk; ++c) {
            const bool last = c == nchunk - 1;
            fetch(last ? k1 : k0, last ? r1 : r0, last ? 0 : c + 1, bn, wn);
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) sum[mt] = Elem<T>::mma(b[ks], w[mt * 2 + ks], sum[mt]);
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) b[ks] = bn[ks];
#pragma unroll
            for (int f = 0; f < 2 * MT; ++f) w[f] = wn[f];
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int v = 0; v < 16; ++v)                                         // accumulator row 8 * (v / 4) + 4 * h + v % 4
                acc[mt][v] = (has >> (8 * (v >> 2) + (v & 3))) & 1u ? acc[mt][v] + sum[mt][v] : acc[mt][v];
        k0 = k1; k1 = k2; k2 = k3;
        r0 = r1; r1 = r2; id2 = id3;
    }
    const int col = slice * (32 * NT) + NT * n + mt0;
    if (col >= C_out) return;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int local = P.perm[tile * kTileT + g * kGroup + 8 * (v >> 2) + 4 * h + (v & 3)];
        if (local >= H->n_out) continue;                                        // past the tile's end, or another kernel's
        const int64_t at = (tile * kTileT + local) * C_out + col;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            if (OUT_F32) reinterpret_cast<float*>(out)[at + mt] = acc[mt][v];
            else reinterpret_cast<uint16_t*>(out)[at + mt] = Elem<T>::from_float(acc[mt][v]);
        }
    }
}

// a real call for the tile kernel, so that its registers are allocated apart from the main loop's; one n-tile, because a call
// that takes more registers makes the compiler spill more around it (48 -> 48 4 % slower on finite values)
template <typename T, bool OUT_F32, int NT>
__device__ __noinline__ void sum_pairs_again_call(const PairArgs* args, const uint16_t* feat, const void* wp, int C_in, int C_out, int64_t tile,
                                                  int g, int slice, int mt, void* out) {
    sum_pairs_again<T, OUT_F32, NT, 1>(*args, feat, wp, C_in, C_out, tile, g, slice, mt, out);
}

// ---------------------------------------------------------------------------------- MFMA kernel
constexpr int kMetaSlots = 3;

// A work item (tile x slice of 32 NT output channels) as the workgroup sees it: its number in the work
// list (-1: the list is exhausted) and a copy of the tile header.
struct MetaSlot {
    int64_t work;
    int64_t pad;
    TileHeader hdr;
};

// Rows and id blocks are double-buffered: while the consumer waves multiply out of one half, the
// producer waves fill the other half straight from global memory.  The work items themselves are
// announced two steps ahead in a ring of three slots.
struct ConvLds {
    unsigned char rows[2][kRowBufBytes];     // 64-byte rows; 16-byte piece p stored at p ^ ((row >> 2) & 3)
    unsigned char blocks[2][kBlockBufBytes]; // id blocks [block][voxel n][group slot], u16
    uint16_t perm[3][kTileT];                // a ring of three: the write-back of item i reads its entry while item i+1 multiplies
    MetaSlot meta[kMetaSlots];
};
static_assert(sizeof(ConvLds) <= 160 * 1024, "LDS budget of one compute unit");


// What a wave needs to know about one work item; all fields are wave-uniform.
struct Item {
    int64_t tile;
    int slice;
    int win_lo, win_n, n_list, n_blocks, n_valid, n_staged;
    bool general, all_rows;
    bool both_halves;      // rows that fill more than one half of the row buffer, and no more than both
};

__device__ __forceinline__ int64_t slot_work(const MetaSlot& M) {
    const int lo = uni((int)(uint32_t)(M.work & 0xFFFFFFFFll)), hi = uni((int)(M.work >> 32));
    return ((int64_t)hi << 32) | (uint32_t)lo;
}

__device__ __forceinline__ Item item_of(const MetaSlot& M, int64_t work, int nslice) {
    Item I;
    I.tile = work / nslice;
    I.slice = (int)(work - I.tile * nslice);
    I.win_lo = uni(M.hdr.win_lo); I.win_n = uni(M.hdr.win_n); I.n_list = uni(M.hdr.n_list);
    I.n_blocks = uni(M.hdr.n_blocks); I.n_valid = uni(M.hdr.n_out);
    const int flags = uni(M.hdr.flags);
    const int n_rows = (flags & kTileDirect) ? 0 : I.win_n + I.n_list;
    I.both_halves = n_rows > kRowCap && n_rows <= 2 * kRowCap;
    I.n_staged = I.both_halves ? n_rows : min(n_rows, kRowCap);
    I.general = !(flags & kTileLdsOffsets);
    I.all_rows = !(flags & kTilePartial);
    return I;
}

// Phases of an item.  One whose rows need both halves of the row buffer takes turns: the producers fill both, the consumers
// multiply, chunk after chunk, and in a last phase the producers start the next item.  The sums are the same, in the same order,
// as when the rows past the first half were read from global memory by the lanes that need them, one dependent load ahead of
// every multiply; bf16 64 -> 64 on 24 k voxels of a sphere shell with one such tile 39.5 -> 30.3 us (21 where no tile has as many
// rows), 116 k LiDAR voxels 47.6 -> 38.7, 88 k / 531 k of bodies, surfaces and scan lines 114.3 -> 102.5 / 198 -> 190.  Filling the first half
// in the item before measured the same; 16 channels a phase, pipelined like the others, 36.4 / 43.7 / 107 / 190: twice the
// phases, each with the loads of ids and weights in front.
__device__ __forceinline__ int item_phases(const Item& I, int nchunk) { return I.both_halves ? 2 * nchunk + 1 : nchunk; }

// word e of a lane's id entry (a scalar when a wave has two groups, a vector otherwise)
__device__ __forceinline__ uint32_t id_word(uint32_t v, int) { return v; }
template <typename V>
__device__ __forceinline__ uint32_t id_word(const V& v, int e) { return v[e]; }

// Loop over the stencil offsets a wave needs for one 32-channel chunk.  Software pipeline per
// offset step i: the weights of step i+2, the B fragments of step i+1 and the ids of step i+2
// are fetched while the MFMAs of step i are issued (2 m-tiles x 2 k-steps per present column
// block).  The weights come from L2, whose latency exceeds one step, hence two steps of lead and
// three register sets; the sets are rotated by unrolling, never copied, and steps run in triples
// (the surplus steps multiply nothing) so that the rotation is the same at every exit.  Weight
// fragments are addressed as wbase0 (the packed array) + a wave-uniform offset + the lane's 16 bytes.
// The pipeline runs across calls: the last two steps fetch the fragments at offsets w_after0 and
// w_after1 -- the first two offsets of whatever this wave multiplies next -- into wa and wb, and
// wa_at / wb_at record what the two sets hold, so that a call normally starts with both in
// flight (and fetches them itself if a call in between was skipped).
enum class RowsAt {
    OneHalf,               // all rows staged in one half of the row buffer: ids are LDS offsets
    BothHalves,            // all rows staged, in both halves: ids are row numbers
    Anywhere,              // rows that are not staged are read from global memory
};
template <typename T, RowsAt ROWS, int NT, bool PARTIAL>
__device__ __forceinline__ void offsets_loop(const unsigned char* lds_rows, const unsigned char* lds_blocks,
                                             f32x16 (&acc)[kGroupsPerWave][NT],
                                             const uint32_t (&gmask)[kGroupsPerWave], uint32_t wave_mask,
                                             int wave_block0, const typename Elem<T>::vec8* __restrict__ wbase0,
                                             uint32_t lane_off, int w_base, int w_kappa_stride, typename Elem<T>::vec8 (&wa)[2 * NT],
                                             typename Elem<T>::vec8 (&wb)[2 * NT], int& wa_at, int& wb_at, int w_after0,
                                             int w_after1, int n, int h, int n_staged, int win_lo, int win_n,
                                             const int32_t* __restrict__ my_rows, const unsigned char* __restrict__ feat,
                                             int64_t pitch, int c) {
    typedef typename Elem<T>::vec8 vec8;
    constexpr int NG = kGroupsPerWave;
    const int n_off = __popc(wave_mask);
    const int n_steps = (n_off + 2) / 3 * 3;
    typedef __attribute__((ext_vector_type(NG / 2))) uint32_t IdVec;    // a lane's ids of one block: NG x u16
    const IdVec* idp = reinterpret_cast<const IdVec*>(lds_blocks) + (size_t)wave_block0 * kGroup + n;
    uint32_t rest = wave_mask;            // offsets not yet fetched; 31 (which no group has) once exhausted
    auto pop_kappa = [&]() {               // branch-free: 31 once the mask is exhausted
        const int k = __builtin_ctz(rest | 0x80000000u);
        rest &= rest - 1;
        return k;
    };
    // wave-uniform offset of the weights that step t multiplies (t may lie past this call's end);
    // written with masks so that it stays a handful of scalar instructions without branches
    auto w_offset = [&](int t, int k) {
        const int in = -(int)(t < n_off), last = -(int)(t == n_steps + 1);
        const int past = (w_after1 & last) | (w_after0 & ~last);
        return ((w_base + k * w_kappa_stride) & in) | (past & ~in);
    };
    auto fetch_w = [&](vec8 (&w)[2 * NT], int off) {   // [mtile*2 + kstep]; uniform base + 32-bit lane offset
        const unsigned char* ws = reinterpret_cast<const unsigned char*>(wbase0 + off);
#pragma unroll
        for (int f = 0; f < 2 * NT; ++f) w[f] = *reinterpret_cast<const vec8*>(ws + lane_off + f * 1024);
    };
    const uint32_t hsel = (uint32_t)h << 4;
    // B fragments (16 channels x 32 voxels, two k-steps) of column block gi for offset kappa
    auto fetch_b = [&](vec8 (&bf)[2], const IdVec& ids, int gi, int kappa) {
        // In the LDS-only variant the reads are issued for every group: an absent group's ids all
        // point at the zero row (one broadcast address).  With the reads unconditional every path
        // issues the same number of LDS instructions and the compiler waits for exactly the
        // fragments it needs; behind uniform branches it assumed the worst and drained the freshly
        // issued prefetch before every multiply.
        if (ROWS == RowsAt::Anywhere && !((gmask[gi] >> kappa) & 1u)) return;
        const uint32_t id = (id_word(ids, gi >> 1) >> (16 * (gi & 1))) & 0xFFFFu;
        if (ROWS == RowsAt::BothHalves) {                    // row kRowCap is the zero row; the second half's rows follow it
            const bool staged = id < (uint32_t)n_staged;
            const uint32_t a0 = (staged ? lds_row_code(id) + (id >= (uint32_t)kRowCap ? kRowBytes : 0) : lds_row_code(kRowCap)) ^ hsel;
            bf[0] = *reinterpret_cast<const vec8*>(lds_rows + a0);
            bf[1] = *reinterpret_cast<const vec8*>(lds_rows + (a0 ^ 32u));
        } else if (ROWS == RowsAt::Anywhere) {
            const bool staged = id < (uint32_t)n_staged;
            const int row = staged ? (int)id : kRowCap;
            bf[0] = *reinterpret_cast<const vec8*>(lds_rows + lds_row_offset(row, h));
            bf[1] = *reinterpret_cast<const vec8*>(lds_rows + lds_row_offset(row, h + 2));
            const bool from_global = !staged && id != kNoRow;
            if (__any(from_global)) {
                if (from_global) {
                    const int64_t gr = id < (uint32_t)win_n ? (int64_t)win_lo + id : (int64_t)my_rows[id - win_n];
                    const int at = c * kRowBytes + h * 16;       // a row that ends inside its last chunk: zeros beyond
                    const unsigned char* src = feat + gr * pitch + at;
                    if (!PARTIAL || at < pitch) bf[0] = *reinterpret_cast<const vec8*>(src);
                    if (!PARTIAL || at + 32 < pitch) bf[1] = *reinterpret_cast<const vec8*>(src + 32);
                }
            }
        } else {   // id = lds_row_code(row): 16-byte piece p of the row sits at id ^ (p << 4); pieces h and h + 2
            const uint32_t a0 = id ^ hsel;
            bf[0] = *reinterpret_cast<const vec8*>(lds_rows + a0);
            bf[1] = *reinterpret_cast<const vec8*>(lds_rows + (a0 ^ 32u));
        }
    };
    vec8 wc[2 * NT];
    vec8 bf[NG][2];   // one set: a group's fragments for the next offset are fetched right after its multiplies
    int q0 = pop_kappa(), q1 = pop_kappa(), q2 = pop_kappa(), it = 0;   // offsets of steps it, it+1, it+2
    if (wa_at != w_offset(0, q0)) fetch_w(wa, w_offset(0, q0));          // only after a call was skipped
    if (wb_at != w_offset(1, q1)) fetch_w(wb, w_offset(1, q1));
    wa_at = w_after0;
    wb_at = w_after1;
    // Both sets were requested at least two steps ago (or, rarely, just now).  Waiting for them here
    // costs nothing in the common case and tells the compiler so: without it the loop's wait counts
    // are computed for the rare case and every step also waits for the weights of the next one.
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0), other counters untouched
    IdVec idn = idp[min(1, n_off - 1) * kGroup];   // ids of step 1
    {
        const IdVec id0 = idp[0];
#pragma unroll
        for (int gi = 0; gi < NG; ++gi) fetch_b(bf[gi], id0, gi, q0);
    }
    // one step: fetch the weights of step it+2 and the ids of step it+2, then, group by group,
    // multiply the current offset and fetch the group's fragments for the next one
    auto step = [&](const vec8 (&wcur)[2 * NT], vec8 (&wload)[2 * NT]) {
        fetch_w(wload, w_offset(it + 2, q2));
        const IdVec ids_next = idn;
        idn = idp[min(it + 2, n_off - 1) * kGroup];
#pragma unroll
        for (int gi = 0; gi < NG; ++gi) {
            if ((gmask[gi] >> q0) & 1u) {
#pragma unroll
                for (int ks = 0; ks < 2; ++ks)      // k-step outermost: consecutive MFMAs never share an accumulator
#pragma unroll
                    for (int mt = 0; mt < NT; ++mt) acc[gi][mt] = Elem<T>::mma(bf[gi][ks], wcur[mt * 2 + ks], acc[gi][mt]);
            }
            fetch_b(bf[gi], ids_next, gi, q1);
        }
        ++it;
        q0 = q1; q1 = q2; q2 = pop_kappa();
    };
    while (it < n_off) {
        step(wa, wc);
        step(wb, wa);
        step(wc, wb);
    }
}

// Producer side: one wave copies 1 KB slabs (16 rows of 64 bytes, or 4 id blocks) from global
// memory straight into LDS; lane l of a slab load writes the 16 bytes at slab + 16*l.
// The global row of every slab a lane serves is kept in registers: the rows of a tile
// are the same for all its chunks, so only the first chunk pays the dependent load of the halo list.
constexpr int kSlabsPerProducer = ((kRowCap + 15) / 16 + kProducerWaves - 1) / kProducerWaves;

__device__ __forceinline__ void resolve_rows(int32_t (&gr)[kSlabsPerProducer], const Item& I, int first_row, int pwave, int lane,
                                             const int32_t* __restrict__ tile_rows, int row_stride) {
    const int32_t* my_rows = tile_rows + I.tile * (int64_t)row_stride;
#pragma unroll
    for (int j = 0; j < kSlabsPerProducer; ++j) {
        const int at = 16 * (pwave + kProducerWaves * j) + (lane >> 2), r = first_row + at;
        gr[j] = -1;
        if (at < kRowCap && r < I.n_staged) gr[j] = r < I.win_n ? I.win_lo + r : my_rows[r - I.win_n];
    }
}

template <bool PARTIAL>
__device__ __forceinline__ void produce_rows_resolved(unsigned char* lds_rows, const int32_t (&gr)[kSlabsPerProducer],
                                                      int pwave, int lane, const unsigned char* __restrict__ feat,
                                                      int64_t pitch, int c) {
    const int piece = (lane & 3) ^ ((lane >> 4) & 3);       // stored position lane&3 holds piece (lane&3) ^ ((row >> 2) & 3)
    const bool in = !PARTIAL || c * kRowBytes + piece * 16 < pitch;      // a row that ends inside its last chunk: zeros beyond
#pragma unroll
    for (int j = 0; j < kSlabsPerProducer; ++j) {
        if (gr[j] >= 0 && in) {
            const unsigned char* src = feat + (int64_t)gr[j] * pitch + c * kRowBytes + piece * 16;
            __builtin_amdgcn_global_load_lds(src, (lds_ptr_t)(lds_rows + (pwave + kProducerWaves * j) * 1024), 16, 0, 0);
        }
    }
    if (!in) {
#pragma unroll
        for (int j = 0; j < kSlabsPerProducer; ++j)
            if (gr[j] >= 0) *reinterpret_cast<u32x4*>(lds_rows + (pwave + kProducerWaves * j) * 1024 + lane * 16) = u32x4{0, 0, 0, 0};
    }
}

__device__ __forceinline__ void produce_meta(unsigned char* lds_blocks, uint16_t* lds_perm, const Item& I, int pwave, int lane,
                                             const uint16_t* __restrict__ tile_perm,
                                             const uint16_t* __restrict__ tile_blocks, int block_stride) {
    const unsigned char* src = reinterpret_cast<const unsigned char*>(tile_blocks + (size_t)I.tile * block_stride * kIdBlockElems);
    const int bytes = I.n_blocks * kIdBlockElems * 2;
    for (int s = pwave; s * 1024 < bytes; s += kProducerWaves) {
        const int off = s * 1024 + lane * 16;
        if (off < bytes) __builtin_amdgcn_global_load_lds(src + off, (lds_ptr_t)(lds_blocks + s * 1024), 16, 0, 0);
    }
    if (pwave == 0)
        __builtin_amdgcn_global_load_lds(reinterpret_cast<const unsigned char*>(tile_perm + I.tile * kTileT) + lane * 16,
                                         (lds_ptr_t)lds_perm, 16, 0, 0);
}

// Next unclaimed work item, taken by a whole wave: first from the list of the workgroup's own XCD, then from the others'.
// The first wg_per_xcd items of every list are taken statically by that XCD's workgroups.  Updates of the counters, which
// share a line, run one after the other at memory, 15-45 ns each: once its own list is empty a workgroup looks at all
// counters with one load and claims only from a list that still has items, and it stops asking when none has (open_lists
// holds what is left to ask: the own list, others).  With a claim tried on each of the eight lists the 2048 updates of the
// last items were most of a call of few items: 32 -> 32, 220 k voxels, 432 items, 71 -> 44 us.
__device__ __forceinline__ int64_t take_work(int32_t* __restrict__ counters, int xcd, int per_xcd, int wg_per_xcd,
                                             int64_t n_work, int lane, int n_orphans, int& open_lists) {
    // lane v < 8: the v-th list in order of preference; lane 8: the static items of workgroups 0 .. n_orphans - 1, which
    // start with something else
    const int x = (xcd + lane) & 7, counter = lane < 8 ? x : 9 + kMaxLongTiles;
    const int64_t begin = (int64_t)x * per_xcd + wg_per_xcd;
    const int64_t left = lane < 8 ? min(n_work, (int64_t)(x + 1) * per_xcd) - begin : n_orphans;
    while (open_lists) {
        uint32_t mask = 1u;
        if (!(open_lists & 1)) {
            bool some = false;
            if (lane < 9 && left > 0) some = (int64_t)__hip_atomic_load(&counters[counter], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < left;
            mask = (uint32_t)__ballot(some);
            if (!mask) open_lists = 0;
        }
        for (; mask; mask &= mask - 1) {
            const int v = __ffs(mask) - 1;
            int got = 0;
            bool hit = false;
            if (lane == v && left > 0) {
                got = atomicAdd(&counters[counter], 1);
                hit = got < left;
            }
            if (__ballot(hit)) {
                const int64_t nth = __builtin_amdgcn_readlane(got, v);
                return v < 8 ? (int64_t)((xcd + v) & 7) * per_xcd + wg_per_xcd + nth : (nth & 7) * per_xcd + (nth >> 3);
            }
        }
        open_lists &= ~1;
    }
    return -1;
}

// One wave announces work item `work` (or the end of the list) in a slot of the ring; returns the flags of its tile.
__device__ __forceinline__ int announce(MetaSlot& M, int64_t work, int nslice, const TileHeader* __restrict__ tile_hdr,
                                        int lane) {
    int32_t v = 0;
    if (work >= 0) {
        const int32_t* src = reinterpret_cast<const int32_t*>(tile_hdr + work / nslice);
        if (lane < (int)(sizeof(TileHeader) / 4)) {
            v = src[lane];
            reinterpret_cast<int32_t*>(&M.hdr)[lane] = v;
        }
    }
    if (lane == 0) M.work = work;
    return __builtin_amdgcn_readlane(v, offsetof(TileHeader, flags) / 4);
}

// workgroups of the tile kernel: one per compute unit, a multiple of 8 (one share per XCD), no more than the work needs
static int mfma_grid(int64_t n_work) {
    return (int)std::min<int64_t>(std::max(8, (compute_units() / 8) * 8), 8 * ((n_work + 7) / 8));
}

__device__ __forceinline__ int first_offset(uint32_t mask) { return mask ? __ffs(mask) - 1 : 0; }

// Consumer side of one work item: multiply all chunks (one barrier after each, matching the
// producers' barriers), then write the tile's outputs back (register v of lane (n, h) holds channels
// slice * 32 NT + NT n .. + NT - 1 of output slot 32 g + 8 (v / 4) + 4 h + v % 4).  `phase` counts chunks since kernel start and
// selects the LDS half; `mb` selects the half that holds this tile's id blocks.
// The weight pipeline (wa, wb and their tags) runs across chunks and, in the LDS-only variant,
// across items: the last steps of an item already fetch the first weights of the next one (MN
// is its slot), ahead of the write-back stores -- loads and stores retire in order, and weights
// requested after the stores would have to wait for them.
template <typename T, bool OUT_F32, RowsAt ROWS, int NT, bool PARTIAL>
__device__ __forceinline__ void consume_item(ConvLds& L, const MetaSlot& M, const MetaSlot& MN, const Item& I, int phase,
                                             int mb, int pb, int nchunk, int nslice, int wave, int lane,
                                             const int32_t* __restrict__ tile_rows, int row_stride,
                                             const unsigned char* __restrict__ feat, const unsigned char* __restrict__ wp,
                                             int64_t pitch, int C_out, void* __restrict__ out, typename Elem<T>::vec8 (&wa)[2 * NT],
                                             typename Elem<T>::vec8 (&wb)[2 * NT], int& wa_at, int& wb_at,
                                             const PairArgs* again, unsigned long long (&tm)[4]) {
    typedef typename Elem<T>::vec8 vec8;
    constexpr int NG = kGroupsPerWave;
    const int n = lane & 31, h = lane >> 5;
    uint32_t gmask[NG];
#pragma unroll
    for (int gi = 0; gi < NG; ++gi) gmask[gi] = (uint32_t)uni((int)M.hdr.group_mask[tile_group_of(wave, gi)]);
    const uint32_t wave_mask = (uint32_t)uni((int)M.hdr.wave_mask[wave]);
    const int wave_block0 = uni((int)M.hdr.wave_block0[wave]);
    const int32_t* my_rows = tile_rows + I.tile * (int64_t)row_stride;
    const int w_kappa_stride = nchunk * nslice * 2 * NT * 64;

    f32x16 acc[NG][NT];
#pragma unroll
    for (int gi = 0; gi < NG; ++gi)
#pragma unroll
        for (int mt = 0; mt < NT; ++mt)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[gi][mt][v] = 0.f;

    for (int c = 0; c < nchunk; ++c) {
        if (ROWS == RowsAt::BothHalves) __syncthreads();     // the producers fill both halves
        // where this wave's weights come from after this chunk
        int w_after0, w_after1;
        {
            int nsl = I.slice, nc = c + 1;
            uint32_t nmask = wave_mask;
            if (nc == nchunk) {      // the next item (if it is not one for this variant, the fetches go unused)
                const int64_t nwork = slot_work(MN);
                nc = 0;
                nsl = nwork >= 0 ? (int)(nwork % nslice) : I.slice;
                nmask = nwork >= 0 ? (uint32_t)uni((int)MN.hdr.wave_mask[wave]) : 0u;
            }
            w_after0 = w_frag<NT>(nslice, w_kappa_stride, nsl, nc, first_offset(nmask));
            const uint32_t more = nmask & (nmask - 1);
            w_after1 = more ? w_frag<NT>(nslice, w_kappa_stride, nsl, nc, first_offset(more)) : w_after0;
        }
        if (wave_mask) {
            FX_CYCLES_BEGIN();
            offsets_loop<T, ROWS, NT, PARTIAL>(L.rows[ROWS == RowsAt::BothHalves ? 0 : (phase + c) & 1], L.blocks[mb], acc, gmask, wave_mask, wave_block0,
                                     reinterpret_cast<const vec8*>(wp), (uint32_t)lane * 16u,
                                     w_frag<NT>(nslice, w_kappa_stride, I.slice, c, 0), w_kappa_stride, wa, wb, wa_at, wb_at,
                                     w_after0, w_after1, n, h, I.n_staged, I.win_lo, I.win_n, my_rows, feat, pitch, c);
            FX_CYCLES_ADD(tm[0]);
        }
        { FX_CYCLES_BEGIN(); __syncthreads(); FX_CYCLES_ADD(tm[1]); }
    }
    FX_CYCLES_BEGIN();
    uint32_t odd = 0;                                 // column blocks with a sum that is not finite
    if (PARTIAL) {
#pragma unroll
        for (int gi = 0; gi < NG; ++gi) {
            float all = 0.f;
#pragma unroll
            for (int mt = 0; mt < NT; ++mt)
#pragma unroll
                for (int v = 0; v < 16; ++v) all += acc[gi][mt][v];
            if (__ballot(!isfinite(all))) odd |= 1u << gi;
        }
    }
    unsigned char* tile_out = reinterpret_cast<unsigned char*>(out) +
                              ((I.tile * kTileT) * C_out + (int64_t)I.slice * (32 * NT)) * (OUT_F32 ? 4 : 2);
#pragma unroll
    for (int gi = 0; gi < NG; ++gi)
        store_block_rows<T, OUT_F32, NT>(acc[gi], L.perm[pb] + tile_group_of(wave, gi) * kGroup, tile_out, C_out,
                                     min(32 * NT, C_out - I.slice * (32 * NT)), I.n_valid, n, h, I.all_rows);
    if constexpr (PARTIAL) {
        if (odd) {
            __builtin_amdgcn_s_waitcnt(0);            // the rows are stored over
            for (; odd; odd &= odd - 1)
                for (int mt = 0; mt < NT; ++mt)
                    sum_pairs_again_call<T, OUT_F32, NT>(again, reinterpret_cast<const uint16_t*>(feat), wp, (int)(pitch / 2), C_out, I.tile,
                                                         tile_group_of(wave, __ffs(odd) - 1), I.slice, mt, out);
            wa_at = wb_at = -1;                       // nothing is handed over a call
#pragma unroll
            for (int f = 0; f < 2 * NT; ++f) { wa[f] = vec8{}; wb[f] = vec8{}; }
        }
    }
    FX_CYCLES_ADD(tm[2]);
}

// Items with more rows than one half holds take this path: a real call, so that its registers are allocated apart from the
// main loop's.
template <typename T, bool OUT_F32, int NT, bool PARTIAL>
__device__ __noinline__ int consume_long_item(int slot, int phase, int mb, int pb, int nchunk, int nslice, int wave, int lane,
                                                  const int32_t* __restrict__ tile_rows, int row_stride,
                                                  const unsigned char* __restrict__ feat, const unsigned char* __restrict__ wp,
                                                  int64_t pitch, int C_out, void* __restrict__ out, const PairArgs* again) {
    typedef typename Elem<T>::vec8 vec8;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    ConvLds& L = *reinterpret_cast<ConvLds*>(lds_raw);
    const MetaSlot& M = L.meta[slot];
    const Item I = item_of(M, slot_work(M), nslice);
    vec8 wa[2 * NT], wb[2 * NT];
    int wa_at = -1, wb_at = -1;
    unsigned long long tm[4] = {0, 0, 0, 0};
    if (I.both_halves) {
        consume_item<T, OUT_F32, RowsAt::BothHalves, NT, PARTIAL>(L, M, L.meta[(slot + 1) % kMetaSlots], I, phase, mb, pb, nchunk, nslice, wave, lane,
                                   tile_rows, row_stride, feat, wp, pitch, C_out, out, wa, wb, wa_at, wb_at, again, tm);
        __syncthreads();                                     // the producers fill a half for the next item
    } else {
        consume_item<T, OUT_F32, RowsAt::Anywhere, NT, PARTIAL>(L, M, L.meta[(slot + 1) % kMetaSlots], I, phase, mb, pb, nchunk, nslice, wave, lane,
                                   tile_rows, row_stride, feat, wp, pitch, C_out, out, wa, wb, wa_at, wb_at, again, tm);
    }
    return item_phases(I, nchunk);
}

// Persistent workgroups, one per compute unit.  Work items (tile of 512 consecutive outputs x
// slice of 32 NT output channels) are cut into eight contiguous lists, one per XCD, so that
// neighbouring tiles, which share halo rows, meet in the same L2; a workgroup starts with a fixed
// item of its XCD's list and then claims items through per-list counters (its own list first),
// which evens out tiles of different cost.  Time advances in phases of one 32-channel chunk.
// Waves 0-3 are consumers: wave w owns 4 of the tile's 16 column blocks (128 outputs, 4 x 2
// accumulator tiles of 32x32, 4 x 1 for NT = 1) and multiplies out of one half of LDS.  Waves 4-7 are producers:
// meanwhile they copy the rows of the next phase (and, at a tile change, its id blocks) from
// global memory straight into the other half, and the first of them announces the item that
// starts two phases later (claim + tile header) in a ring of three slots.  One barrier per phase
// hands everything over; both roles walk the same ring and execute the same barriers.
// Producers and consumers are separate waves because a wave's loads complete in order: the
// consumer's short weight fetches must not queue behind the long HBM reads.
// PARTIAL: rows that end inside their last 64-byte chunk (C_in not a multiple of 32; 16-bit types): zeros beyond, and sums that
// are not finite are made again pair by pair.  (In the one kernel the tests cost 3 % at 64 -> 64 on 980 k voxels.)
template <typename T, bool OUT_F32, int NT, bool PARTIAL>
__global__ void __launch_bounds__(kConvThreads, 1)
k_conv_mfma(const TileHeader* __restrict__ tile_hdr, const uint16_t* __restrict__ tile_perm,
            const int32_t* __restrict__ tile_rows, int row_stride, const uint16_t* __restrict__ tile_blocks,
            int block_stride, int64_t n_work, int per_xcd, int32_t* __restrict__ counters,
            const unsigned char* __restrict__ feat, const unsigned char* __restrict__ wp, int C_in, int C_out,
            void* __restrict__ out) {
    typedef typename Elem<T>::vec8 vec8;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    ConvLds& L = *reinterpret_cast<ConvLds*>(lds_raw);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t pitch = (int64_t)C_in * Elem<T>::kBytes;                      // bytes per feature row
    const int nchunk = (int)((pitch + kRowBytes - 1) / kRowBytes), nslice = (C_out + 32 * NT - 1) / (32 * NT);

    // workgroup b runs on XCD b % 8 (round-robin dispatch)
    const int xcd = blockIdx.x & 7, in_xcd = blockIdx.x >> 3, wg_per_xcd = gridDim.x >> 3;
    const int64_t first = (int64_t)xcd * per_xcd + in_xcd;
    if (in_xcd >= per_xcd || first >= n_work) return;

    if (tid < 2 * (kRowBytes / 16))   // the zero row of both halves
        reinterpret_cast<u32x4*>(L.rows[tid >> 2] + kRowCap * kRowBytes)[tid & 3] = u32x4{0, 0, 0, 0};

    if (wave >= kTileWaves) {
        // ---------------- producers
        const int pwave = wave - kTileWaves;
        int open_lists = 3;
        int64_t start = first;
        int n_orphans = 0;
        bool skip_long = false;
        int flags = 0;
        if (pwave == 0) {
            const int n_long = long_tiles_first(n_work, gridDim.x) ? uni(counters[8]) : 0;              // in flight beside the first header
            flags = announce(L.meta[0], first, nslice, tile_hdr, lane);
            // Items of long tiles (rows in both halves of the row buffer, or gathered from global memory: two to four times another item) would end the launch
            // alone if they were claimed last.  When all of them are listed the first workgroups start with one each, claims
            // pass them over, and the static items of those workgroups are claimed like the others (at most the lower half
            // of every XCD's workgroups, all of which have a static item: see long_tiles_first).  bf16 on 195 k voxels of sheets (four long tiles of 381), 128 -> 128
            // 165 -> 149 us, 256 -> 256 515 -> 457; 221 k LiDAR voxels (five of 432) 64 -> 64 61 -> 50, 256 -> 256 407 -> 372.
            if (n_long > 0 && n_long <= kMaxLongTiles && n_long * nslice <= (int)gridDim.x / 2) {
                skip_long = true;
                n_orphans = n_long * nslice;
                if ((int)blockIdx.x < n_orphans) {
                    start = (int64_t)counters[9 + blockIdx.x % n_long] * nslice + blockIdx.x / n_long;
                    flags = announce(L.meta[0], start, nslice, tile_hdr, lane);
                }
            }
        }
        auto announce_claimed = [&](MetaSlot& M, int64_t w) {
            while (!(announce(M, w, nslice, tile_hdr, lane) & kTileLdsOffsets) && w >= 0 && skip_long)
                w = take_work(counters, xcd, per_xcd, wg_per_xcd, n_work, lane, n_orphans, open_lists);
        };
        auto announce_next = [&](MetaSlot& M) {
            announce_claimed(M, take_work(counters, xcd, per_xcd, wg_per_xcd, n_work, lane, n_orphans, open_lists));
        };
        if (pwave == 0) {   // items that start in phases 0 and 1
            if (skip_long && start == first && (int)blockIdx.x >= n_orphans && !(flags & kTileLdsOffsets)) announce_next(L.meta[0]);
            if (nchunk == 1) announce_next(L.meta[1]);
        }
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        int32_t gr[kSlabsPerProducer];
        if (slot_work(L.meta[0]) >= 0) {       // a workgroup whose static item is another's start may find nothing left
            const Item cur = item_of(L.meta[0], slot_work(L.meta[0]), nslice);
            produce_meta(L.blocks[0], L.perm[0], cur, pwave, lane, tile_perm, tile_blocks, block_stride);
            if (!cur.both_halves) {
                resolve_rows(gr, cur, 0, pwave, lane, tile_rows, row_stride);
                produce_rows_resolved<PARTIAL>(L.rows[0], gr, pwave, lane, feat, pitch, 0);
            }
        }
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        int phase = 0;
        for (int item_no = 0;; ++item_no) {
            const MetaSlot& M = L.meta[item_no % kMetaSlots];
            const MetaSlot& MN = L.meta[(item_no + 1) % kMetaSlots];
            const int64_t work = slot_work(M);
            if (work < 0) break;
            const Item cur = item_of(M, work, nslice);
            MetaSlot& claim_slot = L.meta[(item_no + (nchunk == 1 ? 2 : 1)) % kMetaSlots];       // of the item that is claimed during this one
            // Items in both halves in a loop of their own.  The claim goes with the last chunk: with the first, 257 items of these on 256
            // workgroups took 77 us for 67, whoever claimed first was not who would be done first.
            if (cur.both_halves) {
                int32_t gr2[kSlabsPerProducer];
                resolve_rows(gr, cur, 0, pwave, lane, tile_rows, row_stride);
                resolve_rows(gr2, cur, kRowCap, pwave, lane, tile_rows, row_stride);
                for (int c = 0; c < nchunk; ++c) {
                    produce_rows_resolved<PARTIAL>(L.rows[0], gr, pwave, lane, feat, pitch, c);
                    produce_rows_resolved<PARTIAL>(L.rows[1], gr2, pwave, lane, feat, pitch, c);
                    if (c == nchunk - 1 && pwave == 0) announce_next(claim_slot);
                    __builtin_amdgcn_s_waitcnt(0);
                    __syncthreads();
                    __syncthreads();                         // the consumers have multiplied
                }
                phase += 2 * nchunk;
                const int64_t nwork = slot_work(MN);
                if (nwork >= 0) {
                    const Item nxt = item_of(MN, nwork, nslice);
                    if (!nxt.both_halves) {
                        resolve_rows(gr, nxt, 0, pwave, lane, tile_rows, row_stride);
                        produce_rows_resolved<PARTIAL>(L.rows[(phase + 1) & 1], gr, pwave, lane, feat, pitch, 0);
                    }
                    produce_meta(L.blocks[(item_no + 1) & 1], L.perm[(item_no + 1) % 3], nxt, pwave, lane, tile_perm, tile_blocks, block_stride);
                }
                __builtin_amdgcn_s_waitcnt(0);
                __syncthreads();
                ++phase;
                continue;
            }
            for (int c = 0; c < nchunk; ++c, ++phase) {
                const int rb = (phase + 1) & 1;
                const bool last = c == nchunk - 1;
                if (!last) produce_rows_resolved<PARTIAL>(L.rows[rb], gr, pwave, lane, feat, pitch, c + 1);
                // At one chunk an item two chains of dependent loads side by side: the next item's row numbers and the claim of
                // the item that starts two phases from now, then the rows and that item's header.  (One after the other they were longer than a
                // phase's multiplies at one chunk an item: f16 32 -> 32 on 221 k voxels 36.0 -> 34.7 us, on 980 k 72 -> 71.)
                const int64_t nwork = last ? slot_work(MN) : -1;
                const Item nxt = nwork >= 0 ? item_of(MN, nwork, nslice) : cur;
                const bool next_rows = nwork >= 0 && !nxt.both_halves;      // else they are staged by the next item
                if (next_rows) resolve_rows(gr, nxt, 0, pwave, lane, tile_rows, row_stride);
                const bool claims = pwave == 0 && c == max(nchunk - 2, 0);             // ahead of the phase that looks at it
                const int64_t claimed = claims ? take_work(counters, xcd, per_xcd, wg_per_xcd, n_work, lane, n_orphans, open_lists) : -1;
                if (nwork >= 0) {
                    if (next_rows) produce_rows_resolved<PARTIAL>(L.rows[rb], gr, pwave, lane, feat, pitch, 0);
                    produce_meta(L.blocks[(item_no + 1) & 1], L.perm[(item_no + 1) % 3], nxt, pwave, lane, tile_perm, tile_blocks, block_stride);
                }
                if (claims) announce_claimed(claim_slot, claimed);
                __builtin_amdgcn_s_waitcnt(0);
                __syncthreads();
            }
        }
    } else {
        // ---------------- consumers
        // Where the multiply's loop lies within the 32 bytes that are fetched at a time is worth 3 % of a launch (98 k voxels 128 -> 128,
        // by steps of 8 bytes: 67.5, 67.4, 69.2, 68.8), and any line above it moved it.  The code from here to the loop is the same but for PARTIAL.
        asm volatile(".p2align 5\n\t.rept %0\n\ts_nop 0\n\t.endr" ::"n"(PARTIAL ? 2 : 6));
        const PairArgs* again = reinterpret_cast<const PairArgs*>(counters + kPairArgsAt);
        unsigned long long tm[4] = {0, 0, 0, 0};
        const unsigned long long t_start = FX_CYCLES_NOW();
        __syncthreads();
        vec8 wa[2 * NT], wb[2 * NT];
        int wa_at, wb_at;
        {   // weights of the first two offsets of the first item
            const int w_kappa_stride = nchunk * nslice * 2 * NT * 64;
            const uint32_t m0 = (uint32_t)uni((int)L.meta[0].hdr.wave_mask[wave]);
            const uint32_t m1 = m0 & (m0 - 1);
            const int slice0 = (int)(max(slot_work(L.meta[0]), (int64_t)0) % nslice);
            wa_at = w_frag<NT>(nslice, w_kappa_stride, slice0, 0, first_offset(m0));
            wb_at = m1 ? w_frag<NT>(nslice, w_kappa_stride, slice0, 0, first_offset(m1)) : wa_at;
            const vec8* w0 = reinterpret_cast<const vec8*>(wp) + lane;
#pragma unroll
            for (int f = 0; f < 2 * NT; ++f) { wa[f] = (w0 + wa_at)[f * 64]; wb[f] = (w0 + wb_at)[f * 64]; }
        }
        __syncthreads();
        int phase = 0, n_items = 0;
        for (int item_no = 0;; ++item_no) {
            const int slot = item_no % kMetaSlots;
            const MetaSlot& M = L.meta[slot];
            const int64_t work = slot_work(M);
            if (work < 0) break;
            const Item cur = item_of(M, work, nslice);
            if (cur.general) {
                phase += uni(consume_long_item<T, OUT_F32, NT, PARTIAL>(slot, phase, item_no & 1, item_no % 3, nchunk, nslice, wave, lane, tile_rows,
                                                           row_stride, feat, wp, pitch, C_out, out, again));
                // What the call saved is read back before the next item, with a wait of its own; among the other items' the wait for it
                // was one for their weights and stores too.
                __builtin_amdgcn_s_waitcnt(0);
                wa_at = wb_at = -1;       // nothing is handed over a call
#pragma unroll
                for (int f = 0; f < 2 * NT; ++f) { wa[f] = vec8{}; wb[f] = vec8{}; }
            } else {
                consume_item<T, OUT_F32, RowsAt::OneHalf, NT, PARTIAL>(L, M, L.meta[(item_no + 1) % kMetaSlots], cur, phase, item_no & 1, item_no % 3, nchunk, nslice,
                                                wave, lane, tile_rows, row_stride, feat, wp, pitch, C_out, out, wa, wb, wa_at,
                                                wb_at, again, tm);
                phase += nchunk;
            }
            ++n_items;
        }
        // development builds: per-workgroup cycles of the first consumer wave (multiply, barrier waits, write-back, items)
        if (tid == 0) {
            FX_STAMP_VALUE(blockIdx.x, 0, tm[0]); FX_STAMP_VALUE(blockIdx.x, 1, tm[1]); FX_STAMP_VALUE(blockIdx.x, 2, tm[2]);
            FX_STAMP_VALUE(blockIdx.x, 3, FX_CYCLES_NOW() - t_start); FX_STAMP_VALUE(blockIdx.x, 4, (unsigned long long)n_items);
        }
        (void)t_start;
    }
}

// ---------------------------------------------------------------------------------- gather kernel
// For maps whose input rows are used (almost) once -- strided maps, where staging rows in LDS buys no
// reuse.  One wave owns one column block (32 outputs) x one 64-channel output slice for all
// offsets: it first resolves the block's (offset, voxel) -> input row table into LDS with independent
// loads, then walks the offsets, reading each lane's 16-byte A fragments straight from the feature
// rows (one step ahead) and the packed weights (the B operand, interleaved channels) from L2; a
// half-wave stores one output row's 64-channel slice in one piece.  No barriers, ~100 registers, so
// several waves per SIMD hide the gather latency.
constexpr int kGatherWaves = 4;

template <typename T, bool OUT_F32>
__global__ void __launch_bounds__(64 * kGatherWaves)
k_conv_gather(const TileHeader* __restrict__ tile_hdr, const uint16_t* __restrict__ tile_perm,
              const int32_t* __restrict__ tile_rows, int row_stride, const uint16_t* __restrict__ tile_blocks,
              int block_stride, int64_t n_items, const uint16_t* __restrict__ feat, const uint16_t* __restrict__ wp,
              int C_in, int C_out, void* __restrict__ out, bool partial) {
    typedef typename Elem<T>::vec8 vec8;
    __shared__ int32_t row_of[kGatherWaves][kMaxK3Tiled][kGroup];
    __shared__ __align__(16) int32_t out_of[kGatherWaves][kGroup];      // the block's output rows within the tile (-1: none)
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t item = (int64_t)blockIdx.x * kGatherWaves + wave;
    if (item >= n_items) return;
    const int nchunk = (C_in + kCinChunk - 1) / kCinChunk, nslice = (C_out + kCoutSlice - 1) / kCoutSlice;
    const int slice = (int)(item % nslice);
    const int64_t tg = item / nslice;
    const int g = (int)(tg % kGroupsPerTile);
    const int64_t tile = tg / kGroupsPerTile;
    const TileHeader* H = tile_hdr + tile;
    const int w = tile_wave_of(g), gi = tile_slot_of(g);
    const uint32_t gm = (uint32_t)uni((int)H->group_mask[g]);
    const uint32_t wm = (uint32_t)uni((int)H->wave_mask[w]);
    const int n = lane & 31, h = lane >> 5;
    const int n_valid = uni(H->n_out);
    if (h == 0) {
        const int local = tile_perm[tile * kTileT + g * kGroup + n];
        out_of[wave][n] = local < n_valid ? local : -1;
    }

    // (offset, voxel) -> global input row (-1: none); lane (n, h) resolves every second offset
    {
        const int flags = uni(H->flags), win_lo = uni(H->win_lo), win_n = uni(H->win_n);
        const size_t blk0 = (size_t)tile * block_stride + (uint32_t)uni((int)H->wave_block0[w]);
        const int32_t* rows = tile_rows + tile * (int64_t)row_stride;
        int rank = 0;
        for (uint32_t m = gm; m; m &= m - 1, ++rank) {
            if ((rank & 1) != h) continue;
            const int kappa = __ffs(m) - 1;
            const size_t blk = blk0 + __popc(wm & ((1u << kappa) - 1u));
            uint32_t id = tile_blocks[blk * kIdBlockElems + n * kGroupsPerWave + gi];
            if (flags & kTileLdsOffsets) id = (id / kRowBytes == (uint32_t)kRowCap) ? kNoRow : id / kRowBytes;
            int32_t r = -1;
            if (id != kNoRow) r = id < (uint32_t)win_n ? win_lo + (int32_t)id : rows[id - (uint32_t)win_n];
            row_of[wave][rank][n] = r;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // a wave's LDS accesses are processed in order
    __builtin_amdgcn_wave_barrier();

    f32x16 acc[2];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[mt][v] = 0.f;

    const int w_kappa_stride = nchunk * nslice * 4 * 64;
    const vec8* wl = reinterpret_cast<const vec8*>(wp) + lane;
    const int n_k = __popc(gm);
    const int n_steps = n_k * nchunk;            // step = (offset rank, chunk), chunk fastest
    vec8 zero;
#pragma unroll
    for (int e = 0; e < 8; ++e) zero[e] = 0;
    auto fetch = [&](vec8 (&b)[2], vec8 (&wf)[4], int step, uint32_t& rest, int& kappa) {
        const int rank = step / nchunk, c = step - rank * nchunk;
        if (c == 0) { kappa = __ffs(rest) - 1; rest &= rest - 1; }
        const int32_t r = row_of[wave][rank][n];
        b[0] = zero; b[1] = zero;
        if (r >= 0) {
            // a row that ends inside its last chunk: its last piece once more, for weights that are zero
            const uint16_t* src = feat + (int64_t)r * C_in;
            b[0] = *reinterpret_cast<const vec8*>(src + min(c * kCinChunk + h * 8, C_in - 8));
            b[1] = *reinterpret_cast<const vec8*>(src + min(c * kCinChunk + h * 8 + 16, C_in - 8));
        }
        const vec8* ws = wl + w_frag(nslice, w_kappa_stride, slice, c, kappa);
#pragma unroll
        for (int f = 0; f < 4; ++f) wf[f] = ws[f * 64];
    };
    vec8 ba[2], bb[2], wa[4], wb[4];
    uint32_t rest = gm;
    int kappa = 0;
    if (n_steps > 0) fetch(ba, wa, 0, rest, kappa);
    for (int step = 0; step < n_steps; step += 2) {
        if (step + 1 < n_steps) fetch(bb, wb, step + 1, rest, kappa);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) acc[nt] = Elem<T>::mfma(ba[ks], wa[nt * 2 + ks], acc[nt]);
        if (step + 2 < n_steps) fetch(ba, wa, step + 2, rest, kappa);
        if (step + 1 < n_steps) {       // a guard, not an early exit: one loop exit keeps one copy of the accumulators
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int nt = 0; nt < 2; ++nt) acc[nt] = Elem<T>::mfma(bb[ks], wb[nt * 2 + ks], acc[nt]);
        }
    }

    // accumulator register v of lane (n, h) is voxel 8 * (v / 4) + 4 * h + v % 4 of the block, channels 2n and 2n + 1
    // of the slice (one per n-tile): the 32 lanes of a half-wave store one whole 64-channel row slice
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const i32x4 o4 = *reinterpret_cast<const i32x4*>(&out_of[wave][8 * q + 4 * h]);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (o4[j] < 0 || slice * kCoutSlice + 2 * n >= C_out) continue;
            const int64_t at = (tile * kTileT + o4[j]) * C_out + (int64_t)slice * kCoutSlice + 2 * n;
            if (OUT_F32)
                *reinterpret_cast<f32x2*>(reinterpret_cast<float*>(out) + at) = f32x2{acc[0][4 * q + j], acc[1][4 * q + j]};
            else
                *reinterpret_cast<uint32_t*>(reinterpret_cast<uint16_t*>(out) + at) = Elem<T>::pack2(acc[0][4 * q + j], acc[1][4 * q + j]);
        }
    }
    if (partial) {
        float all = 0.f;                     // not finite if one of the sums is not
#pragma unroll
        for (int v = 0; v < 16; ++v) all += acc[0][v] + acc[1][v];
        if (__ballot(!isfinite(all))) {
            __builtin_amdgcn_s_waitcnt(0);   // the rows are stored over
            sum_pairs_again<T, OUT_F32, 2, 2>({tile_hdr, tile_perm, tile_rows, tile_blocks, row_stride, block_stride}, feat, wp, C_in, C_out, tile, g, slice, 0, out);
        }
    }
}

// ---------------------------------------------------------------------------------- gather kernel, weights in LDS
// k_conv_gather issues six vector loads per four multiplies, four of them for the weights, and
// is bound by the load path of the compute unit (one wave-wide 16-byte load occupies it for at
// least 16 cycles).  When the packed weights of one 64-channel output slice fit in LDS next to
// the row tables (K^3 * C_in * 128 bytes; 64 KB for a 2x2x2 kernel with 64 input channels), a
// persistent workgroup copies them there once, and each wave then walks column blocks with its
// weight fragments read from LDS: two vector loads per four multiplies.
// * When the weights of two adjacent slices fit together (NS = 2) a gathered fragment feeds the
//   multiplies of both and the gather is issued once per 128 output channels; that form runs twelve
//   waves with a third more registers (64 more accumulators).  With CP = 2 a step covers two
//   32-channel chunks, so its four loads use the whole 128-byte line of a 64-channel row while it
//   is in L1 instead of coming back for the second half a step later.
// * Operand roles: A = gathered rows (32 voxels x 16 input channels), B = packed weights in the
//   interleaved layout (column n of n-tile t = output channel 2n + t), so the output rows lie along
//   the accumulator registers and the channels across the lanes: a half-wave stores one output row's
//   64-channel slice as one contiguous piece.
// * What a block needs before its first gather hangs on a chain of dependent loads (tile header ->
//   id block -> row list), and so does its write-back (output permutation).  The chain is cut into
//   stages that run ahead: the header and permutation entry of block i + 2 are requested while block
//   i multiplies, the ids of block i + 1 before block i's step loop, and they are turned into the
//   row table after it.
// Workgroup b serves slice set b % (nslice / NS).  NS = output slices per workgroup, CP = 32-channel
// chunks per step, W = waves per workgroup, D = fragment sets in flight, R = offset ranks a lane half
// resolves (ceil(K^3 / 2)); PARTIAL: C_in is not a multiple of 32 (CP = 1; see sum_pairs_again).
constexpr int kGatherLdsWaves = 16;
constexpr int kGatherPairWaves = 12;

template <typename T, bool OUT_F32, int NS, int CP, int W, int D, int R, bool PARTIAL>
__global__ void __launch_bounds__(64 * W, 1)
k_conv_gather_ldsw(const TileHeader* __restrict__ tile_hdr, const uint16_t* __restrict__ tile_perm,
                   const int32_t* __restrict__ tile_rows, int row_stride, const uint16_t* __restrict__ tile_blocks,
                   int block_stride, int64_t n_blocks_total, int K3, const uint16_t* __restrict__ feat,
                   const uint16_t* __restrict__ wp, int C_in, int C_out, void* __restrict__ out) {
    typedef typename Elem<T>::vec8 vec8;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int lane = threadIdx.x & 63, wave = uni((int)(threadIdx.x >> 6));
    const int nchunk = (C_in + kCinChunk - 1) / kCinChunk, nslice = (C_out + kCoutSlice - 1) / kCoutSlice, nset = nslice / NS;
    const int npair = nchunk / CP;                                       // steps per offset (the launch checks CP | nchunk)
    const int slice = (blockIdx.x % nset) * NS;                          // first slice of this workgroup's set
    const int wg = blockIdx.x / nset, n_wg = gridDim.x / nset;           // the launch makes gridDim a multiple of nset
    unsigned char* wlds = lds_raw;                                       // [kappa][chunk][slice of the set][4 fragments][64 lanes][16 bytes]
    const int w_bytes = K3 * nchunk * NS * 4096;
    // per wave: [rank][voxel] global input rows of the current block, then [voxel] its output rows within the tile (-1: none)
    int32_t* tab = reinterpret_cast<int32_t*>(lds_raw + w_bytes) + wave * (K3 + 1) * kGroup;
    int32_t* out_of = tab + K3 * kGroup;

    for (int sl = wave; sl * 1024 < w_bytes; sl += W) {                  // 1 KB = one fragment of all lanes
        const int kc = sl / (4 * NS), sn = (sl >> 2) % NS, f = sl & 3;   // (kappa * nchunk + chunk), slice of the set, fragment
        const unsigned char* src = reinterpret_cast<const unsigned char*>(wp) + ((size_t)(kc * nslice + slice + sn) * 4 + f) * 1024 + lane * 16;
        __builtin_amdgcn_global_load_lds(src, (lds_ptr_t)(wlds + sl * 1024), 16, 0, 0);
    }

    const int n = lane & 31, h = lane >> 5;
    vec8 zero;
#pragma unroll
    for (int e = 0; e < 8; ++e) zero[e] = 0;
    const int64_t tg_stride = (int64_t)n_wg * W;
    const int64_t tg0 = (int64_t)wg * W + wave;

    struct Hdr { uint32_t gm, wm, blk0; int flags, win_lo, win_n, n_out; };
    // the header fields of block tg (uniform addresses: scalar loads)
    auto load_hdr = [&](int64_t tg) -> Hdr {
        Hdr d = {0u, 0u, 0u, 0, 0, 0, 0};
        if (tg < n_blocks_total) {
            const int g = (int)(tg % kGroupsPerTile);
            const TileHeader* H = tile_hdr + tg / kGroupsPerTile;
            const int w = tile_wave_of(g);
            d.gm = H->group_mask[g]; d.wm = H->wave_mask[w]; d.blk0 = H->wave_block0[w];
            d.flags = H->flags; d.win_lo = H->win_lo; d.win_n = H->win_n; d.n_out = H->n_out;
        }
        return d;
    };
    auto load_perm = [&](int64_t tg) -> int {
        return tg < n_blocks_total ? (int)tile_perm[tg / kGroupsPerTile * kTileT + (tg % kGroupsPerTile) * kGroup + n] : 0;
    };
    // requests the local row ids of block tg: lane (n, h) takes the offset ranks of parity h, slot j = rank / 2
    auto issue_ids = [&](int64_t tg, const Hdr& d, uint32_t (&idv)[R]) {
        const int g = (int)(tg % kGroupsPerTile);
        const int gi = tile_slot_of(g);
        const size_t blk0 = (size_t)(tg / kGroupsPerTile) * block_stride + d.blk0;
        uint32_t m = d.gm;
#pragma unroll
        for (int j = 0; j < 2 * R; ++j) {
            if (m) {
                const int kappa = __ffs(m) - 1;
                m &= m - 1;
                if ((j & 1) == h)
                    idv[j >> 1] = tile_blocks[(blk0 + __popc(d.wm & ((1u << kappa) - 1u))) * kIdBlockElems + n * kGroupsPerWave + gi];
            }
        }
    };
    // ids -> global input rows (a second load for ids outside the tile's window) and the voxels' output rows, into the
    // wave's table
    auto finish_table = [&](int64_t tg, const Hdr& d, const uint32_t (&idv)[R], int local) {
        const int32_t* rows = tile_rows + tg / kGroupsPerTile * (int64_t)row_stride;
        const int n_k = __popc(d.gm);
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int rank = 2 * j + h;
            if (rank < n_k) {
                uint32_t id = idv[j];
                if (d.flags & kTileLdsOffsets) id = (id / kRowBytes == (uint32_t)kRowCap) ? kNoRow : id / kRowBytes;
                int32_t r = -1;
                if (id != kNoRow) r = id < (uint32_t)d.win_n ? d.win_lo + (int32_t)id : rows[id - (uint32_t)d.win_n];
                tab[rank * kGroup + n] = r;
            }
        }
        if (h == 0) out_of[n] = local < d.n_out ? local : -1;
    };

    Hdr h0 = load_hdr(tg0), h1 = load_hdr(tg0 + tg_stride);
    int p0 = load_perm(tg0), p1 = load_perm(tg0 + tg_stride);
    uint32_t idv[R];
#pragma unroll
    for (int j = 0; j < R; ++j) idv[j] = kNoRow;
    if (tg0 < n_blocks_total) {
        issue_ids(tg0, h0, idv);
        finish_table(tg0, h0, idv, p0);
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();                       // the weights are in LDS

    unsigned long long odd = 0;            // PARTIAL: the wave's blocks with a sum that is not finite (bit 63: any from the 64th on)
    int nth = 0;
#pragma unroll 1
    for (int64_t tg = tg0; tg < n_blocks_total; tg += tg_stride) {
        const Hdr h2 = load_hdr(tg + 2 * tg_stride);
        const int p2 = load_perm(tg + 2 * tg_stride);
        const bool more = tg + tg_stride < n_blocks_total;
        if (more) issue_ids(tg + tg_stride, h1, idv);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // a wave's LDS accesses are processed in order
        __builtin_amdgcn_wave_barrier();

        const uint32_t gm = h0.gm;
        f32x16 acc[2 * NS];
#pragma unroll
        for (int t = 0; t < 2 * NS; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;
        const int n_steps = __popc(gm) * npair;         // step = (offset rank, CP chunks), chunks fastest
        // A fragments of step `step` into b; returns where the step's B fragments start in LDS
        // fetches come in step order: (offset rank, chunk pair) advance with them
        int f_rank = -1, f_c = npair - 1;
        auto fetch = [&](vec8 (&b)[2 * CP], int step, uint32_t& rest, int& kappa) {
            if (++f_c == npair) { f_c = 0; ++f_rank; kappa = __ffs(rest | 0x80000000u) - 1; rest &= rest - 1; }
            const int32_t r = step < n_steps ? tab[f_rank * kGroup + n] : -1;
#pragma unroll
            for (int j = 0; j < 2 * CP; ++j) b[j] = zero;
            if (r >= 0) {
                // PARTIAL: a row that ends inside its last chunk gives its last piece once more, for weights that are zero
                const uint16_t* src = feat + (int64_t)r * C_in;
#pragma unroll
                for (int j = 0; j < 2 * CP; ++j) {
                    const int at = f_c * (CP * kCinChunk) + h * 8 + 16 * j;
                    b[j] = *reinterpret_cast<const vec8*>(src + (PARTIAL ? min(at, C_in - 8) : at));
                }
            }
            return (kappa * nchunk + f_c * CP) * NS * 4096 + lane * 16;
        };
        auto multiply = [&](const vec8 (&b)[2 * CP], int w_at) {
#pragma unroll
            for (int c = 0; c < CP; ++c)
#pragma unroll
                for (int sn = 0; sn < NS; ++sn) {
                    vec8 wf[4];
#pragma unroll
                    for (int f = 0; f < 4; ++f)
                        wf[f] = *reinterpret_cast<const vec8*>(wlds + w_at + (c * NS + sn) * 4096 + f * 1024);
#pragma unroll
                    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                        for (int nt = 0; nt < 2; ++nt)
                            acc[2 * sn + nt] = Elem<T>::mfma(b[2 * c + ks], wf[nt * 2 + ks], acc[2 * sn + nt]);
                }
        };
        // D fragment sets: the gathers of the next D - 1 steps are in flight while one multiplies.  The loop has one
        // exit and guards instead of breaks: with early exits between the multiplies the compiler kept a second
        // copy of the accumulators (80 registers more).
        vec8 ring[D][2 * CP];
        int w_at[D];
        uint32_t rest = gm;
        int kappa = 0;
#pragma unroll
        for (int d = 0; d < D - 1; ++d) { w_at[d] = 0; if (d < n_steps) w_at[d] = fetch(ring[d], d, rest, kappa); }
        w_at[D - 1] = 0;
#pragma unroll 1
        for (int step = 0; step < n_steps; step += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                if (step + d + D - 1 < n_steps) w_at[(d + D - 1) % D] = fetch(ring[(d + D - 1) % D], step + d + D - 1, rest, kappa);
                if (step + d < n_steps) multiply(ring[d], w_at[d]);
            }
        }

        // accumulator register v of lane (n, h) is voxel 8 * (v / 4) + 4 * h + v % 4 of the block, channels 2n and
        // 2n + 1 of a slice (one per n-tile): the 32 lanes of a half-wave store one whole 64-channel row slice
        const int64_t row0 = tg / kGroupsPerTile * kTileT;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const i32x4 o4 = *reinterpret_cast<const i32x4*>(out_of + 8 * q + 4 * h);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (o4[j] < 0) continue;
                const int64_t at = (row0 + o4[j]) * C_out + (int64_t)slice * kCoutSlice + 2 * n;
#pragma unroll
                for (int sn = 0; sn < NS; ++sn) {
                    if ((slice + sn) * kCoutSlice + 2 * n >= C_out) continue;
                    if (OUT_F32)
                        *reinterpret_cast<f32x2*>(reinterpret_cast<float*>(out) + at + sn * kCoutSlice) =
                            f32x2{acc[2 * sn][4 * q + j], acc[2 * sn + 1][4 * q + j]};
                    else
                        *reinterpret_cast<uint32_t*>(reinterpret_cast<uint16_t*>(out) + at + sn * kCoutSlice) =
                            Elem<T>::pack2(acc[2 * sn][4 * q + j], acc[2 * sn + 1][4 * q + j]);
                }
            }
        }
        if (PARTIAL) {
            float all = 0.f;                     // not finite if one of the sums is not
#pragma unroll
            for (int t = 0; t < 2 * NS; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) all += acc[t][v];
            if (__ballot(!isfinite(all))) odd |= 1ull << min(nth, 63);
            ++nth;
        }
        __builtin_amdgcn_wave_barrier();     // the table is rewritten for the next block
        if (more) finish_table(tg + tg_stride, h1, idv, p1);
        h0 = h1; h1 = h2; p0 = p1; p1 = p2;
    }
    if constexpr (PARTIAL) {                     // after the loop, whose registers would be spilled around it
        if (odd) __builtin_amdgcn_s_waitcnt(0);  // the rows are stored over
        nth = 0;
#pragma unroll 1
        for (int64_t tg = tg0; odd && tg < n_blocks_total; tg += tg_stride, ++nth) {
            if (!((odd >> min(nth, 63)) & 1)) continue;
#pragma unroll 1
            for (int sn = 0; sn < NS; ++sn)
                sum_pairs_again<T, OUT_F32, 2, 2>({tile_hdr, tile_perm, tile_rows, tile_blocks, row_stride, block_stride}, feat, wp, C_in, C_out,
                                               tg / kGroupsPerTile, (int)(tg % kGroupsPerTile), slice + sn, 0, out);
        }
    }
}

// ---------------------------------------------------------------------------------- scalar path
// One thread per (output voxel, output channel); fp32 FMA in offset-then-channel order.  Used
// for fp32 data (true fp32 products) and for channel counts the MFMA tiling does not cover.
template <int DT, bool OUT_F32>
__global__ void k_conv_scalar(const int32_t* __restrict__ nbmap, int64_t n_out, int K3, const void* __restrict__ feat,
                              const void* __restrict__ w, int C_in, int C_out, void* __restrict__ out, int mode) {
    const int64_t total = n_out * C_out;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t o = e / C_out;
        const int co = (int)(e - o * C_out);
        float acc = 0.f;
        for (int kappa = 0; kappa < K3; ++kappa) {
            const int32_t in = nbmap[o * K3 + kappa];
            if (in < 0) continue;
            const int64_t fb = (int64_t)in * C_in;
            // plain: W[kw][ci][co]; transposed (e.g. the input gradient on a symmetric map): W[kw][co][ci]
            const int64_t kw = (mode & kWeightsFlipped) ? K3 - 1 - kappa : kappa;
            const int64_t wb = (mode & kWeightsTransposed) ? (kw * C_out + co) * C_in : kw * C_in * C_out + co;
            const int64_t ws = (mode & kWeightsTransposed) ? 1 : C_out;
            for (int ci = 0; ci < C_in; ++ci)
                acc = fmaf(load_as_float<DT>(feat, fb + ci), load_as_float<DT>(w, wb + (int64_t)ci * ws), acc);
        }
        if (OUT_F32) reinterpret_cast<float*>(out)[e] = acc;
        else if (DT == FX_F16) reinterpret_cast<uint16_t*>(out)[e] = Elem<_Float16>::from_float(acc);
        else reinterpret_cast<uint16_t*>(out)[e] = Elem<__bf16>::from_float(acc);
    }
}

// The same sum with four output channels per thread and four input channels per load (channel
// counts that are multiples of 4): one 16-byte feature load and four 16-byte
// weight loads feed 16 multiply-adds, a sixth of the loads of the kernel above.  The sum over the
// input channels of one offset keeps the order ci = 0, 1, 2, ... of the one-channel kernel.
template <int DT, bool OUT_F32>
__global__ void k_conv_scalar4(const int32_t* __restrict__ nbmap, int64_t n_out, int K3, const void* __restrict__ feat,
                               const void* __restrict__ w, int C_in, int C_out, void* __restrict__ out, int mode) {
    const int q_out = C_out / 4;
    const int64_t total = n_out * q_out;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t o = e / q_out;
        const int co = (int)(e - o * q_out) * 4;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        for (int kappa = 0; kappa < K3; ++kappa) {
            const int32_t in = nbmap[o * K3 + kappa];
            if (in < 0) continue;
            const int64_t fb = (int64_t)in * C_in;
            const int64_t kw = (mode & kWeightsFlipped) ? K3 - 1 - kappa : kappa;
            if (!(mode & kWeightsTransposed)) {
                const int64_t wb = kw * C_in * C_out + co;
                for (int ci = 0; ci < C_in; ci += 4) {
                    const f32x4 x = load4_as_float<DT>(feat, fb + ci);
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const f32x4 wr = load4_as_float<DT>(w, wb + (int64_t)(ci + j) * C_out);
#pragma unroll
                        for (int v = 0; v < 4; ++v) acc[v] = fmaf(x[j], wr[v], acc[v]);
                    }
                }
            } else {   // W[kw][co][ci]: the four contracted channels of a produced channel are adjacent
                const int64_t wb = (kw * C_out + co) * C_in;
                for (int ci = 0; ci < C_in; ci += 4) {
                    const f32x4 x = load4_as_float<DT>(feat, fb + ci);
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const f32x4 wr = load4_as_float<DT>(w, wb + (int64_t)v * C_in + ci);
#pragma unroll
                        for (int j = 0; j < 4; ++j) acc[v] = fmaf(x[j], wr[j], acc[v]);
                    }
                }
            }
        }
        const int64_t at = o * C_out + co;
        if (OUT_F32) {
            *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(out) + at) = acc;
        } else if (DT == FX_F16) {
            *reinterpret_cast<u32x2*>(reinterpret_cast<uint16_t*>(out) + at) =
                u32x2{Elem<_Float16>::pack2(acc[0], acc[1]), Elem<_Float16>::pack2(acc[2], acc[3])};
        } else {
            *reinterpret_cast<u32x2*>(reinterpret_cast<uint16_t*>(out) + at) =
                u32x2{Elem<__bf16>::pack2(acc[0], acc[1]), Elem<__bf16>::pack2(acc[2], acc[3])};
        }
    }
}

// ---------------------------------------------------------------------------------- fp32, few tiles
// fp32 over a tiled map whose tiles are too few to fill the chip with one workgroup each: one wave owns 16 voxels (half a
// column block) x 16 NT produced channels, so that ten thousand voxels at 32 channels are 1200 independent waves.  The
// voxels' input rows are resolved from the map's id blocks into LDS (four taps at a time, independent loads), taps that
// no voxel of the 16 has are dropped, and the wave walks (tap, 16 channels): one 16-byte piece of a row per lane and the
// weights straight from the caller's array, kF32Batch steps ahead of the multiplies.  v_mfma_f32_16x16x4_f32 multiplies
// in true fp32; the produced channels are its rows, so a lane ends with four adjacent channels of one voxel.  Bound by the
// latency of the gathers at small sizes, by the matrix units and weight reads from L2 beyond.  Measured against one
// scalar thread per four outputs and the dense table that took (14 us at first use): sphere of 9.9 k voxels 32 -> 32
// 53 -> 20 us, 64 -> 64 140 -> 44, 1.4 k voxels 40 -> 16, 48.8 k voxels 64 -> 64 492 -> 126 (151 before the loads of
// a stage were made unconditional, so that all of them are in flight together).
constexpr int kF32Voxels = 16;
constexpr int kF32Batch = 4;

template <int NT, bool TRANSPOSED>
__global__ void __launch_bounds__(64)
k_conv_gather_f32(const TileHeader* __restrict__ tile_hdr, const uint16_t* __restrict__ tile_perm,
                  const int32_t* __restrict__ tile_rows, int row_stride, const uint16_t* __restrict__ tile_blocks,
                  int block_stride, int K3, const float* __restrict__ feat, const float* __restrict__ w, int C_in, int C_out,
                  int n_col, float* __restrict__ out, int flipped, int vec_store) {
    __shared__ int32_t row_of[29][kF32Voxels];       // by rank of the tap among those the 16 voxels have (28: ranks they do not)
    __shared__ int32_t tap_of[29];
    const int lane = threadIdx.x, v = lane & 15, q = lane >> 4;
    const int col = (int)(blockIdx.x % n_col);
    const int64_t half = blockIdx.x / n_col;
    const int hb = (int)(half & 1), g = (int)((half >> 1) % kGroupsPerTile);
    const int64_t tile = (half >> 1) / kGroupsPerTile;
    const TileHeader* H = tile_hdr + tile;
    const int wv = tile_wave_of(g), gi = tile_slot_of(g), n = hb * kF32Voxels + v;
    const uint32_t gm = (uint32_t)uni((int)H->group_mask[g]), wm = (uint32_t)uni((int)H->wave_mask[wv]);
    const int n_valid = uni(H->n_out), flags = uni(H->flags), win_lo = uni(H->win_lo), win_n = uni(H->win_n);
    const size_t blk0 = (size_t)tile * block_stride + (uint32_t)uni((int)H->wave_block0[wv]);
    const int local = tile_perm[tile * kTileT + g * kGroup + n];
    if (__ballot(local < n_valid) == 0) return;      // the last tile's empty column blocks

    // lane (v, q) resolves the taps of rank q, q + 4, ... of the group's mask (each has an id block) for voxel v, all
    // loads of a stage unconditional so that they are in flight together
    int n_live = 0;
    if (gm) {
        const int32_t* rows = tile_rows + tile * (int64_t)row_stride;
        uint32_t id[7], mine[7];
        uint32_t m = gm;
#pragma unroll
        for (int j = 0; j < 7; ++j) {
            const uint32_t m1 = m & (m - 1), m2 = m1 & (m1 - 1), m3 = m2 & (m2 - 1);      // 0 stays 0
            mine[j] = q == 0 ? m : q == 1 ? m1 : q == 2 ? m2 : m3;
            m = m3 & (m3 - 1);
            const int kappa = __ffs(mine[j] ? mine[j] : gm) - 1;
            id[j] = tile_blocks[(blk0 + __popc(wm & ((1u << kappa) - 1u))) * kIdBlockElems + n * kGroupsPerWave + gi];
        }
        int32_t listed[7];
#pragma unroll
        for (int j = 0; j < 7; ++j) {
            if (flags & kTileLdsOffsets) id[j] = id[j] / kRowBytes == (uint32_t)kRowCap ? kNoRow : id[j] / kRowBytes;
            if (!mine[j]) id[j] = kNoRow;
            const bool far = id[j] != kNoRow && id[j] >= (uint32_t)win_n;
            listed[j] = *(far ? rows + (id[j] - (uint32_t)win_n) : reinterpret_cast<const int32_t*>(H));
        }
#pragma unroll
        for (int j = 0; j < 7; ++j) {
            const int32_t r = id[j] == kNoRow ? -1 : id[j] < (uint32_t)win_n ? win_lo + (int32_t)id[j] : listed[j];
            const uint64_t b = __ballot(r >= 0);
            int at = 28;                              // taps that none of the 16 voxels has go nowhere
#pragma unroll
            for (int s = 0; s < 4; ++s)
                if ((b >> (16 * s)) & 0xffffu) { if (q == s) at = n_live; ++n_live; }
            row_of[at][v] = r;
            tap_of[at] = __ffs(mine[j]) - 1;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // a wave's LDS accesses are processed in order
    __builtin_amdgcn_wave_barrier();

    const int nchunk = C_in >> 4, n_steps = n_live * nchunk;
    int co[NT];                                       // the channel whose weights this lane reads (columns beyond the last: dropped)
#pragma unroll
    for (int t = 0; t < NT; ++t) co[t] = min(16 * (col * NT + t) + v, C_out - 1);
    f32x4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};

    int c = 0, rank = 0;                              // the next step to fetch; past the last one the last tap is read again
    auto fetch = [&](f32x4 (&x)[kF32Batch], f32x4 (&wt)[kF32Batch][NT], bool (&has)[kF32Batch]) {
#pragma unroll
        for (int u = 0; u < kF32Batch; ++u) {
            const int32_t r = row_of[rank][v];
            const int kappa = uni(tap_of[rank]), kw = flipped ? K3 - 1 - kappa : kappa;
            const int ci = 16 * c + 4 * q;
            has[u] = r >= 0;
            x[u] = *reinterpret_cast<const f32x4*>(feat + (int64_t)max(r, 0) * C_in + ci);
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                if (TRANSPOSED) {
                    wt[u][t] = *reinterpret_cast<const f32x4*>(w + ((int64_t)kw * C_out + co[t]) * C_in + ci);
                } else {
                    const float* p = w + ((int64_t)kw * C_in + ci) * C_out + co[t];
#pragma unroll
                    for (int j = 0; j < 4; ++j) wt[u][t][j] = p[(int64_t)j * C_out];
                }
            }
            ++c;
            const bool wrap = c == nchunk;
            c = wrap ? 0 : c;
            rank = min(rank + (wrap ? 1 : 0), n_live - 1);
        }
    };
    auto multiply = [&](const f32x4 (&x)[kF32Batch], const f32x4 (&wt)[kF32Batch][NT], const bool (&has)[kF32Batch], int done) {
#pragma unroll
        for (int u = 0; u < kF32Batch; ++u) {
            if (done + u < n_steps) {                 // uniform
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float xv = has[u] ? x[u][j] : 0.f;
#pragma unroll
                    for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(wt[u][t][j], xv, acc[t], 0, 0, 0);
                }
            }
        }
    };
    if (n_steps > 0) {
        f32x4 xa[kF32Batch], xb[kF32Batch], wa[kF32Batch][NT], wb[kF32Batch][NT];
        bool ha[kF32Batch], hb2[kF32Batch];
        fetch(xa, wa, ha);
#pragma unroll 1
        for (int s = 0; s < n_steps; s += 2 * kF32Batch) {
            fetch(xb, wb, hb2);
            __builtin_amdgcn_sched_barrier(0);        // a batch is requested before the one at hand is multiplied
            multiply(xa, wa, ha, s);
            fetch(xa, wa, ha);
            __builtin_amdgcn_sched_barrier(0);
            multiply(xb, wb, hb2, s + kF32Batch);
        }
    }
    // A sum runs over the taps that a voxel has.  The multiplies give a missing one zeros, which add nothing unless a
    // weight is infinite or NaN; that leaves a sum that is not finite, and a wave with such a sum makes its sums again
    // from existing taps only.
    bool again = false;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) again |= !isfinite(acc[t][j]);
    if (__ballot(again)) {
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int s = 0; s < n_live; ++s) {
            const int32_t r = row_of[s][v];
            if (r < 0) continue;
            const int kw = flipped ? K3 - 1 - tap_of[s] : tap_of[s];
#pragma unroll 1
            for (int ci = 0; ci < C_in; ++ci) {
                const float x = feat[(int64_t)r * C_in + ci];
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int oc = min(16 * (col * NT + t) + 4 * q + j, C_out - 1);
                        acc[t][j] = fmaf(x, TRANSPOSED ? w[((int64_t)kw * C_out + oc) * C_in + ci] : w[((int64_t)kw * C_in + ci) * C_out + oc], acc[t][j]);
                    }
            }
        }
    }
    if (local >= n_valid) return;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int c0 = 16 * (col * NT + t) + 4 * q;
        float* o = out + (tile * kTileT + local) * (int64_t)C_out + c0;
        if (vec_store) {
            if (c0 < C_out) *reinterpret_cast<f32x4*>(o) = acc[t];
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (c0 + j < C_out) o[j] = acc[t][j];
        }
    }
}

template <typename T, bool OUT_F32, int NT, bool PARTIAL>
static hipError_t launch_mfma(const fx_kmap* km, const void* feat, const void* wp, int32_t* counters, int C_in, int C_out,
                              void* out, hipStream_t st) {
    const size_t lds = sizeof(ConvLds);
    hipError_t e = hipFuncSetAttribute((const void*)k_conv_mfma<T, OUT_F32, NT, PARTIAL>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    const int64_t n_work = km->n_tiles * (int64_t)((C_out + 32 * NT - 1) / (32 * NT));
    const int per_xcd = (int)((n_work + 7) / 8), grid = mfma_grid(n_work);
    k_conv_mfma<T, OUT_F32, NT, PARTIAL><<<grid, kConvThreads, lds, st>>>(km->d_tile_hdr, km->d_tile_perm, km->d_tile_rows,
                                                             km->row_stride, km->d_tile_blocks, km->block_stride, n_work,
                                                             per_xcd, counters, (const unsigned char*)feat,
                                                             (const unsigned char*)wp, C_in, C_out, out);
    return hipGetLastError();
}

// How the gather kernel with its weights in LDS would serve a map and shape: ns = 0 if it cannot (the weights of
// one 64-channel output slice and the waves' tables exceed 160 KB, or option gather_lds = 0), else the slices per
// workgroup (two when their weights fit together and option gather_lds is not 1), chunks per step, waves and the
// dynamic LDS bytes.  Maps with more than eight offsets take twelve waves (their tables are larger).
struct GatherLdsPlan { int ns, cp, waves; size_t lds; };
static GatherLdsPlan gather_lds_plan(const fx_kmap* km, int C_in, int C_out) {
    const int nslice = (C_out + kCoutSlice - 1) / kCoutSlice, nchunk = (C_in + kCinChunk - 1) / kCinChunk;
    const size_t w_slice = (size_t)km->K3 * nchunk * 4096;                   // packed weights of one output slice
    auto tables = [&](int waves) { return (size_t)waves * (km->K3 + 1) * kGroup * sizeof(int32_t); };
    GatherLdsPlan p = {0, 1, 0, 0};
    if (option(kOptGatherLds) == 0 || km->K3 > 27) return p;
    if (km->K3 <= 8 && nslice % 2 == 0 && 2 * w_slice + tables(kGatherPairWaves) <= 160 * 1024 && option(kOptGatherLds) != 1) {
        p.ns = 2; p.cp = C_in % (2 * kCinChunk) == 0 ? 2 : 1; p.waves = kGatherPairWaves;
    } else if (km->K3 <= 8 && w_slice + tables(kGatherLdsWaves) <= 160 * 1024) {
        p.ns = 1; p.waves = kGatherLdsWaves;
    } else if (km->K3 > 8 && w_slice + tables(kGatherPairWaves) <= 160 * 1024) {
        p.ns = 1; p.waves = kGatherPairWaves;
    }
    p.lds = p.ns * w_slice + tables(p.waves);
    return p;
}

template <typename T, bool OUT_F32>
static hipError_t launch_gather(const fx_kmap* km, const void* feat, const void* wp, int C_in, int C_out, void* out,
                                hipStream_t st) {
    const bool partial = C_in % kCinChunk != 0;      // see sum_pairs_again
    const GatherLdsPlan plan = gather_lds_plan(km, C_in, C_out);
    if (plan.ns) {
        const int ns = plan.ns, cp = plan.cp, waves = plan.waves;
        const int nslice = (C_out + kCoutSlice - 1) / kCoutSlice;
        const bool few = km->K3 <= 8;            // ranks per lane half: 4, else 14
        const int64_t n_blocks_total = km->n_tiles * (int64_t)kGroupsPerTile;
        // one workgroup per compute unit, a multiple of the number of slice sets, no more than there is work for
        const int nset = nslice / ns;
        int64_t grid = std::max(nset, compute_units() / nset * nset);
        grid = std::min<int64_t>(grid, (n_blocks_total + waves - 1) / waves * nset);
#define FX_GATHER_LDSW(NS_, CP_, W_, D_, R_, PARTIAL_)                                                                   \
        if (ns == NS_ && cp == CP_ && waves == W_ && few == (R_ == 4) && partial == PARTIAL_) {                          \
            hipError_t e = hipFuncSetAttribute((const void*)k_conv_gather_ldsw<T, OUT_F32, NS_, CP_, W_, D_, R_, PARTIAL_>, \
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)plan.lds);              \
            if (e != hipSuccess) return e;                                                                               \
            k_conv_gather_ldsw<T, OUT_F32, NS_, CP_, W_, D_, R_, PARTIAL_><<<(unsigned)grid, 64 * W_, plan.lds, st>>>(   \
                km->d_tile_hdr, km->d_tile_perm, km->d_tile_rows, km->row_stride, km->d_tile_blocks, km->block_stride,   \
                n_blocks_total, km->K3, (const uint16_t*)feat, (const uint16_t*)wp, C_in, C_out, out);                   \
            return hipGetLastError();                                                                                    \
        }
        // measured at config 4 (64 -> 128) before the staged look-ahead: 58 us for (2, 2, 12 waves, 3 sets), 58-59
        // for 8 waves with 2 to 4 sets, 63-64 for one chunk per step, 79-81 for one slice per workgroup
        FX_GATHER_LDSW(1, 1, kGatherLdsWaves, 4, 4, false) FX_GATHER_LDSW(1, 1, kGatherPairWaves, 2, 14, false)
        FX_GATHER_LDSW(2, 1, kGatherPairWaves, 4, 4, false) FX_GATHER_LDSW(2, 2, kGatherPairWaves, 3, 4, false)
        FX_GATHER_LDSW(1, 1, kGatherLdsWaves, 4, 4, true) FX_GATHER_LDSW(1, 1, kGatherPairWaves, 2, 14, true)
        FX_GATHER_LDSW(2, 1, kGatherPairWaves, 4, 4, true)
#undef FX_GATHER_LDSW
        return hipErrorInvalidValue;
    }
    const int64_t n_items = km->n_tiles * (int64_t)kGroupsPerTile * ((C_out + kCoutSlice - 1) / kCoutSlice);
    const unsigned grid = (unsigned)((n_items + kGatherWaves - 1) / kGatherWaves);
    k_conv_gather<T, OUT_F32><<<grid, 64 * kGatherWaves, 0, st>>>(km->d_tile_hdr, km->d_tile_perm, km->d_tile_rows,
                                                                 km->row_stride, km->d_tile_blocks, km->block_stride,
                                                                 n_items, (const uint16_t*)feat, (const uint16_t*)wp,
                                                                 C_in, C_out, out, partial);
    return hipGetLastError();
}

static hipError_t launch_gather_f32(const fx_kmap* km, const float* feat, const float* w, int C_in, int C_out, float* out,
                                    int mode, hipStream_t st) {
    const int64_t halves = km->n_tiles * (int64_t)kGroupsPerTile * 2;
    // two n-tiles per wave share the gathered rows once there are four waves for every SIMD without them
    const bool two = C_out > 16 && halves * ((C_out + 15) / 16) >= (int64_t)compute_units() * 16;
    const int n_col = two ? (C_out + 31) / 32 : (C_out + 15) / 16;
    const unsigned grid = (unsigned)(halves * n_col);
    const int flipped = (mode & kWeightsFlipped) ? 1 : 0;
    const int vec_store = C_out % 4 == 0 && ((uintptr_t)out & 15) == 0;
#define FX_GATHER_F32(NT_, TR_)                                                                                          \
    k_conv_gather_f32<NT_, TR_><<<grid, 64, 0, st>>>(km->d_tile_hdr, km->d_tile_perm, km->d_tile_rows, km->row_stride,    \
                                                     km->d_tile_blocks, km->block_stride, km->K3, feat, w, C_in, C_out,   \
                                                     n_col, out, flipped, vec_store)
    if (mode & kWeightsTransposed) { if (two) FX_GATHER_F32(2, true); else FX_GATHER_F32(1, true); }
    else { if (two) FX_GATHER_F32(2, false); else FX_GATHER_F32(1, false); }
#undef FX_GATHER_F32
    return hipGetLastError();
}

}  // namespace fx

using namespace fx;

FX_DEV_TIMING_EXPORT(fx_debug_conv_timing)



// Device memory the matrix-unit kernels need beyond inputs and outputs: the packed weights and, behind them, the
// work-list counters of the persistent kernel with its list of long tiles.
static size_t conv_scratch_bytes(int K3, int C_in, int C_out, int esize) {
    return packed_weight_bytes(K3, C_in, C_out, esize) + kConvWorkInts * sizeof(int32_t);    // the packed part is a multiple of 64 bytes
}

// The tiled map's convolution on the matrix units with that memory supplied by the caller (`scratch`, at least
// conv_scratch_bytes, 16-byte aligned): pack the weights (which also clears the counters), then the LDS-staged
// kernel or, for maps whose tiles list one row per pair, the gather kernel.  Allocates nothing.
static fx_status conv_tiles_with_scratch(const fx_kmap* km, const void* d_feat, fx_dtype in_dt, const void* d_w, int32_t C_in,
                                         int32_t C_out, void* d_out, fx_dtype out_dt, hipStream_t st, int mode, void* scratch) {
    const bool out_f32 = (out_dt == FX_F32);
    const int esize = in_dt == FX_F32 ? 4 : 2;
    void* wp = scratch;
    const size_t wbytes = packed_weight_bytes(km->K3, C_in, C_out, esize);
    int32_t* counters = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(wp) + wbytes);
    // maps whose tiles list one row per pair (strided; stride 1 back from a larger grid): the gather kernel, also where it
    // pads the last slice; others: the LDS-staged kernel.  bf16, the LDS-staged kernel / the gather kernel, us: 980 k LiDAR
    // voxels, (2,2) map 32 -> 32 92 / 31, 64 -> 96 186 / 48, (3,2) map 32 -> 32 145 / 55, 64 -> 96 360 / 168; the input gradient
    // of the map onto the padded grid 32 <- 64 1650 / 816, 96 <- 64 2610 / 1426; 3.9 k voxels, (2,2) map 32 -> 32 25 / 16
    const int fg = option(kOptConvGather);          // 0 / 1: the LDS-staged / the gather kernel on every map
    const bool gather = (fg >= 0 ? fg == 1 : !map_shares_rows(km)) && in_dt != FX_F32;
    // A work item of the tile kernel is a tile and 64 output channels, or 32 (half the multiplies, the same reads of features) where
    // that leaves no padding (up to 32 channels) or where items of 64 keep at most half of the compute units busy:
    // f16 32 -> 32 on 980 k voxels 97 -> 75 us, 317 k 45 -> 37; bf16 256 -> 256 on 13 k voxels (27 tiles, 108 items of 64)
    // 84 -> 62, 54 k voxels 64 -> 64 (106 items) 41 -> 36.  Above half of the compute units narrow items need a second round.
    const bool narrow = !gather && in_dt != FX_F32 &&
                        (C_out <= 32 || km->n_tiles * (int64_t)((C_out + kCoutSlice - 1) / kCoutSlice) <= compute_units() / 2);
    // rows that end inside a 64-byte chunk: shapes whose sums run over existing pairs only (see sum_pairs_again)
    const bool partial = in_dt != FX_F32 && C_in % kCinChunk != 0;
    PairArgs pairs = {};
    if (partial && !gather) pairs = {km->d_tile_hdr, km->d_tile_perm, km->d_tile_rows, km->d_tile_blocks, km->row_stride, km->block_stride};
    const int64_t n_work = km->n_tiles * (int64_t)(narrow ? (C_out + 31) / 32 : (C_out + 63) / 64);
    const bool list = !gather && long_tiles_first(n_work, mfma_grid(n_work));
    launch_pack_weights(d_w, wp, km->K3, C_in, C_out, esize, counters, mode, st, list ? km->d_tile_long : nullptr, km->n_tiles,
                        narrow ? 1 : 2, pairs);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && gather) {
        ProfScope ps(kProfConvGather, st);
        if (in_dt == FX_BF16)
            e = out_f32 ? launch_gather<__bf16, true>(km, d_feat, wp, C_in, C_out, d_out, st)
                        : launch_gather<__bf16, false>(km, d_feat, wp, C_in, C_out, d_out, st);
        else
            e = out_f32 ? launch_gather<_Float16, true>(km, d_feat, wp, C_in, C_out, d_out, st)
                        : launch_gather<_Float16, false>(km, d_feat, wp, C_in, C_out, d_out, st);
    } else if (e == hipSuccess) {
        ProfScope ps(kProfConvMfma, st);
#define FX_MFMA_NT(T, F32, NT)                                                                                        \
    (partial ? launch_mfma<T, F32, NT, true>(km, d_feat, wp, counters, C_in, C_out, d_out, st)                        \
             : launch_mfma<T, F32, NT, false>(km, d_feat, wp, counters, C_in, C_out, d_out, st))
#define FX_MFMA(T, F32) (narrow ? FX_MFMA_NT(T, F32, 1) : FX_MFMA_NT(T, F32, 2))
        if (in_dt == FX_F32) e = launch_mfma<float, true, 2, false>(km, d_feat, wp, counters, C_in, C_out, d_out, st);
        else if (in_dt == FX_BF16) e = out_f32 ? FX_MFMA(__bf16, true) : FX_MFMA(__bf16, false);
        else e = out_f32 ? FX_MFMA(_Float16, true) : FX_MFMA(_Float16, false);
#undef FX_MFMA
#undef FX_MFMA_NT
    }
    if (e != hipSuccess) { set_error("convolution launch failed: %s", hipGetErrorString(e)); return FX_EDEVICE; }
    return FX_OK;
}

// whether the matrix-unit kernels take this map and shape at all (the size heuristics of conv_apply aside)
static bool conv_tiles_shape_ok(const fx_kmap* km, fx_dtype in_dt, int C_in, int C_out) {
    const int esize = in_dt == FX_F32 ? 4 : 2;
    return km->n_tiles > 0 && ((int64_t)C_in * esize) % kRowBytes == 0 && C_out % 2 == 0;
}

// Partial chunks for which the scalar kernel is the faster one: few offsets make its chains short, and it needs no packing
// launch.  bf16, scalar / matrix units in us.  K = 1, whose tiles are one multiply each: 24 -> 24 94 k voxels 11 / 15, 268 k
// 15 / 31, 980 k 40 / 50; 24 -> 32 500 k 30 / 34, 980 k 51 / 47; 40 -> 24 500 k 34 / 42, 980 k 59 / 60; but 120 -> 8 268 k
// 66 / 46, 24 -> 64 94 k 19 / 15; 48 -> 48 31 k 13 / 15, 96 k 21 / 15; 40 -> 40 160 k 22 / 23, 500 k 51 / 44; 200 -> 24 12 k
// 16 / 18, 31 k 21 / 18; 24 -> 200 3.9 k 12 / 15, 12 k 25 / 15.  (2,2) map, forward, up to 24 channels in (a chain of 192
// products): 24 -> 24 3.9 k voxels 13 / 15, 67 k 15 / 15, 95 k 18 / 15; 24 -> 8 317 k 14 / 15.
static bool scalar_pays(const fx_kmap* km, int C_in, int C_out) {
    const int64_t products = km->n_in * C_in * C_out, M = 1000 * 1000;         // per offset
    if (km->K3 == 1) return products <= (C_in * C_out <= 1200 && C_in <= 72 ? 600 : C_out <= 48 ? 90 : 30) * M;
    return km->K == km->stride && km->K3 * C_in <= 192 && products <= (C_out <= 8 ? 64 : 36) * M;
}

fx_status fx::conv_apply(const fx_kmap* km, const void* d_feat, fx_dtype in_dt, const void* d_w, int32_t C_in,
                         int32_t C_out, void* d_out, fx_dtype out_dt, hipStream_t st, int mode) {
    const bool out_f32 = (out_dt == FX_F32);
    const bool force_scalar = option(kOptForceScalar) == 1;
    // Locally dense grids (Sec. 3.5 scenarios 1-2): on a 3x3x3 stride-1 map the leaf-window kernels compute the same
    // sum from the grid alone and are faster once the leaves are full enough -- the tiles of such a map need more
    // rows than the tile kernel's LDS holds twice -- and, at fp32 depths that the tile kernel does not take, almost
    // everywhere.  Option leaf_dispatch = 0 keeps the kernel-map kernels, = 1 takes the leaf kernels whenever
    // they serve the shape.
    if (km->K == 3 && km->stride == 1 && km->gin == km->gout && (mode == kWeightsForward || mode == kWeightsMirrored) &&
        leaf_shape_supported(in_dt, C_in, C_out) && !force_scalar) {
        const int ld = option(kOptLeafDispatch);
        const double occupancy = (double)km->n_in / (512.0 * (double)std::max<int64_t>(1, km->gin->hdr.n_leaf));
        // Per-leaf dispatch: a grid that mixes locally dense leaves (solid bodies) with sparse ones (thin surfaces,
        // scan lines) is split inside this one call -- the leaves with at least kDenseLeafVoxels voxels go to the
        // leaf-window kernel, the outputs of all other leaves to the tile kernel over a copy of the map that leaves
        // the dense leaves' outputs out.  Taken when the grid as a whole is too sparse for the leaf-window kernel
        // (mean occupancy below 0.40) and most of its voxels (55 %) sit in dense leaves; leaf_dispatch = 2 forces it.
        // bf16, split / tiles alone, us.  What the split gains it gains on whole solid bodies of some million voxels, with 75 % and more
        // of the voxels in them: a full cube and a thin cloud, 982 k, 90 % in the cube, 64 -> 64 303 / 318, 128 -> 128 874 / 939; a
        // ball, 979 k, 75 %, 294 / 306, 835 / 933.  Smaller grids lose by it, the more the smaller they are: its two launches run one after the other, and
        // the leaf-window kernel alone takes 33 to 40 us at 64 -> 64 and 102 to 130 at 128 -> 128 however few leaves there are (114 k, 56 % in a cube, 90 / 47, 252 / 118; 414 k,
        // 90 %, 173 / 138, 487 / 406; cubes of 24, 998 k, 90 %, 318 / 240; bodies, surfaces and scan lines, 168 k (58 %) 122 / 69, 697 k (62 %)
        // 220 / 190).  Below 55 % it lost everywhere (245 k (45 %) 118 / 84, 531 k (48 %) 190 / 128; cube, 400 k, 50 %, 383 / 379), and there it is not
        // taken any more; the line does not yet ask for the size, which is what decides above.
        // From 0.40 on the leaf-window kernel takes the whole of a small grid (below 16 k voxels), and of any from 0.60 on, from 0.54 on above
        // 2^20 voxels at up to 192 contracted channels, or 2^19 at 32 where more than 64 are produced.  Tiles / leaf window, us: random voxels of a cube, 64 -> 64, 97 k at 0.37 46 / 74, 119 k
        // at 0.45 50 / 76, 732 k at 0.52 241 / 260, 513 k at 0.58 186 / 195, 865 k at 0.62 294 / 277, 1.17 M at 0.56 460 / 426, 2.8 M at
        // 0.59 1002 / 898, 1.33 M at 0.96 464 / 340; 128 -> 128, 1.17 M at 0.56 1297 / 1221, 1.11 M at 0.53 1177 / 1172; 256 -> 256, 1.17 M at 0.56 4446 / 4745; 32 -> 192, 566 k at
        // 0.59 325 / 281, 770 k at 0.59 442 / 362, 952 k at 0.55 534 / 468 (32 -> 128 216 / 201, 318 / 260, 376 / 335), balls of 578 k at 0.56 341 / 323 (231 / 249).
        // The size decides here as well, and the line asks for it only so far: solid cubes of 33 k and 111 k 32 / 41 and 47 / 79, of 14 k 31 / 40
        // (128 -> 128 53 / 128), and just past a round of tiles up to 7 % the other way (141 k at 0.54 80 / 76).
        if (in_dt != FX_F32 && !km->is_inverse) {
            const double dense = (double)km->gin->hdr.n_voxels_dense / (double)std::max<int64_t>(1, km->n_in);
            // (a second map that a captured call built would not be there for the next call that is not replayed)
            if (ld == 2 || (ld < 0 && occupancy < 0.40 && dense >= 0.55 && (km->mixed || !stream_captures(st)))) {
                fx_kmap* kmw = const_cast<fx_kmap*>(km);
                FX_TRY(kmap_ensure_mixed(kmw, st));
                void* wp = nullptr;
                FX_TRY(dev_alloc(&wp, conv_scratch_bytes(27, C_in, C_out, 2), st));
                fx_status rc = conv_tiles_with_scratch(km->mixed, d_feat, in_dt, d_w, C_in, C_out, d_out, out_dt, st, mode, wp);
                dev_free(wp, st);
                if (rc != FX_OK) return rc;
                return leaf_apply("sparse convolution (per-leaf dispatch)", km->gin, d_feat, in_dt, d_w, C_in, C_out, d_out, out_dt, st,
                                  mode, km->mixed->d_dense_leaves, km->mixed->d_n_dense);
            }
        }
        const bool scalar_otherwise = in_dt == FX_F32 && C_in % 16 != 0;
        const int64_t large = C_in <= 32 && C_out > 64 ? 1 << 19 : 1 << 20;      // several slices of one chunk stage every row once per slice
        const double line = scalar_otherwise ? 0.08 : in_dt == FX_F32 || km->n_in < 16384 ? 0.40 : km->n_in < large || C_in > 192 ? 0.60 : 0.54;
        // Layers of one chunk or of one slice of 64 produced channels take whole rounds of either kernel's workgroups: one a compute
        // unit of the tile kernel, two of the leaf window's.  With three or four rounds of tiles but fewer of leaves (from 0.50 mean occupancy on) the
        // leaf window is faster, or as fast.  Tiles / leaf window, us: random voxels of a cube, 267 k at 0.58 (523 tiles, 900 leaves) 32 -> 64
        // 86 / 67, 32 -> 128 126 / 108, 64 -> 64 111 / 105; 302 k at 0.59 (589, 999) 87 / 70, 136 / 112, 132 / 110; 409 k at 0.55 (799, 1452)
        // 107 / 93, 164 / 155, 155 / 146; a shell of 268 k (523, 982) 91 / 88, 137 / 132, 131 / 129; a slab of 288 k (563, 1000) 83 / 83, 125 / 132,
        // 123 / 127; 96, 128, 192 -> 64 on 302 k 173 / 146, 211 / 178, 298 / 248, the slab 168 / 174, 197 / 217, 281 / 311 (64 -> 128 206 / 184 and 189 / 219,
        // even on the whole).  As many rounds of leaves: 309 k at 0.55 (605, 1100) 87 / 85, 133 / 138, 128 / 136, balls of 347 k (678, 1205) 92 / 105.  Two rounds of
        // tiles over one of leaves gain at 32 -> 64 only (55 / 55 to 56 / 52; 64 -> 64 67 / 81), five and more are uneven (balls of 578 k 146 / 157).
        const int64_t cu = compute_units(), rounds = (km->n_tiles + cu - 1) / cu, leaf_rounds = (km->gin->hdr.n_leaf + 2 * cu - 1) / (2 * cu);
        const bool fewer_rounds = in_dt != FX_F32 && (C_in <= 32 || C_out <= 64) && (rounds == 3 || rounds == 4) && leaf_rounds < rounds;
        const bool take = ld >= 0 ? ld >= 1 : occupancy >= line || fewer_rounds;
        if (take)
            return leaf_apply("sparse convolution (leaf-window kernels)", km->gin, d_feat, in_dt, d_w, C_in, C_out, d_out, out_dt,
                              st, mode);
    }
    const int esize = in_dt == FX_F32 ? 4 : 2;
    // The matrix-unit kernels take input rows in 64-byte chunks (32 channels of a 16-bit type, 16 of fp32; of a 16-bit type
    // also whole 16-byte pieces, see `pieces` below) and pad an even number of produced channels to whole slices with zero
    // weights: of 64, or 32 in the tile kernel.  Everything else is left to the low-depth and scalar kernels.
    const int64_t n_items = km->n_tiles * (int64_t)((C_out + kCoutSlice - 1) / kCoutSlice);
    // fp32 by independent waves where the tile kernel fills the chip badly (few tiles), stages rows that are used about
    // once, or pads most of its 64 channels.  Measured, waves / tiles in us: 96 items (48.8 k voxels of sheets, 64 -> 64)
    // 126 / 194, 174 items equal; 2x2x2 strided on 195 k voxels 64 -> 64 70 / 121, 3x3x3 219 / 366, on 980 k voxels 64 -> 128
    // 401 / 516; at depth on strided maps of 980 k voxels 2x2x2 128 -> 128 639 / 950, 256 -> 256 2327 / 3144, 3x3x3
    // 128 -> 128 1203 / 1973, 256 -> 256 4677 / 6772; 16 -> 16 on 980 k voxels 174 / 228; 32 -> 32 on 195 k voxels (381 items) 137 / 201, but 425 / 395 on 980 k
    // LiDAR voxels and 68 / 67 on the inverse map.  Pieces of 16 bytes need rows and weights aligned to them; the last
    // condition keeps the launch below 2^32 threads.
    const bool f32_waves = in_dt == FX_F32 && km->n_tiles > 0 && C_in % 16 == 0 && option(kOptFp32Tiles) != 1 && !force_scalar &&
                           (n_items < compute_units() / 2 || !map_shares_rows(km) ||
                            (!km->is_inverse && (C_out <= 16 || (C_out <= 32 && n_items < 2 * compute_units())))) &&
                           (((uintptr_t)d_feat | (uintptr_t)d_w) & 15) == 0 && n_items < (1 << 19);
    if (f32_waves) {
        ProfScope ps(kProfConvGather, st);
        FX_HIP_TRY(launch_gather_f32(km, (const float*)d_feat, (const float*)d_w, C_in, C_out, (float*)d_out, mode, st));
        return FX_OK;
    }
    // A 16-bit type's rows of more than 16 channels need not be whole chunks: whole 16-byte pieces do, at addresses that are
    // multiples of them (up to 16 channels: the low-depth kernels below).  Against the
    // scalar kernel, 221 k LiDAR voxels, bf16, forward / input gradient in us: 48 -> 48 778 / 2209 -> 52 / 52, 24 -> 40
    // 353 / 632 -> 46 / 43, (2,2) map 48 -> 48 108 -> 20, (3,2) map 48 -> 48 279 / 904 -> 42 / 38.
    const bool pieces = in_dt != FX_F32 && km->n_tiles > 0 && C_in > 16 && C_in % 8 == 0 && C_out % 2 == 0 &&
                        ((uintptr_t)d_feat & 15) == 0 && ((uintptr_t)d_out & 3) == 0 && !scalar_pays(km, C_in, C_out);
    const bool mfma = (conv_tiles_shape_ok(km, in_dt, C_in, C_out) || pieces) &&
                      (in_dt != FX_F32 || n_items >= compute_units() / 2 || option(kOptFp32Tiles) == 1) &&   // fp32_tiles = 1: at any size
                      !force_scalar;
    if (mfma) {
        void* wp = nullptr;
        FX_TRY(dev_alloc(&wp, conv_scratch_bytes(km->K3, C_in, C_out, esize), st));
        const fx_status rc = conv_tiles_with_scratch(km, d_feat, in_dt, d_w, C_in, C_out, d_out, out_dt, st, mode, wp);
        dev_free(wp, st);
        return rc;
    }
    FX_TRY(kmap_ensure_dense(const_cast<fx_kmap*>(km), st));
    if (!force_scalar && lowdepth_supported(in_dt, km->K3, C_in, km->n_in))
        return lowdepth_conv_on_table(km->d_nbmap, km->n_out, km->K3, d_feat, in_dt, d_w, C_in, C_out, d_out, out_dt, st, mode);
    return conv_scalar_on_table(km->d_nbmap, km->n_out, km->K3, d_feat, in_dt, d_w, C_in, C_out, d_out, out_dt, st, mode);
}

fx_status fx::conv_scalar_on_table(const int32_t* d_table, int64_t n_rows, int K3, const void* d_feat, fx_dtype in_dt,
                                   const void* d_w, int32_t C_in, int32_t C_out, void* d_out, fx_dtype out_dt, hipStream_t st,
                                   int mode) {
    const bool out_f32 = (out_dt == FX_F32);
    const bool four = C_in % 4 == 0 && C_out % 4 == 0;
    const int64_t total = n_rows * (four ? C_out / 4 : C_out);
    const size_t w_lds = sizeof(float) * (size_t)K3 * C_in * C_out;
    const bool lds_w = four && w_lds <= 32 * 1024 && total >= 8 * 1024 && option(kOptScalarLds) != 0;   // scalar_lds = 0: weights from L1
    const unsigned nb = lds_w ? (unsigned)std::max<int64_t>(1, std::min<int64_t>((total + 255) / 256, (int64_t)compute_units() * 8))
                              : (unsigned)std::max<int64_t>(1, std::min<int64_t>((total + 255) / 256, 1 << 20));
#define FX_SCALAR(DT)                                                                                            \
    do {                                                                                                         \
        if (lds_w && out_f32) k_conv_scalar4_ldsw<DT, true, 1><<<nb, 256, w_lds, st>>>(d_table, n_rows, K3, d_feat, \
                                                                                       d_w, C_in, C_out, d_out, mode); \
        else if (lds_w) k_conv_scalar4_ldsw<DT, false, 1><<<nb, 256, w_lds, st>>>(d_table, n_rows, K3, d_feat, d_w, \
                                                                                  C_in, C_out, d_out, mode);     \
        else if (four && out_f32) k_conv_scalar4<DT, true><<<nb, 256, 0, st>>>(d_table, n_rows, K3, d_feat,      \
                                                                          d_w, C_in, C_out, d_out, mode);        \
        else if (four) k_conv_scalar4<DT, false><<<nb, 256, 0, st>>>(d_table, n_rows, K3, d_feat, d_w,           \
                                                                     C_in, C_out, d_out, mode);                  \
        else if (out_f32) k_conv_scalar<DT, true><<<nb, 256, 0, st>>>(d_table, n_rows, K3, d_feat, d_w,          \
                                                                      C_in, C_out, d_out, mode);                 \
        else k_conv_scalar<DT, false><<<nb, 256, 0, st>>>(d_table, n_rows, K3, d_feat, d_w, C_in,                \
                                                          C_out, d_out, mode);                                   \
    } while (0)
    ProfScope ps(kProfConvScalar, st);
    if (in_dt == FX_F32) FX_SCALAR(FX_F32);
    else if (in_dt == FX_F16) FX_SCALAR(FX_F16);
    else FX_SCALAR(FX_BF16);
#undef FX_SCALAR
    FX_HIP_TRY(hipGetLastError());
    return FX_OK;
}

extern "C" fx_status fx_sparse_conv_fwd(const fx_kmap* km, const void* d_feat, fx_dtype in_dt, const void* d_w,
                                        int32_t C_in, int32_t C_out, void* d_out, fx_dtype out_dt, void* stream) {
    if (!km || !d_w || C_in < 1 || C_out < 1 || (km->n_in > 0 && !d_feat) || (km->n_out > 0 && !d_out)) {
        set_error("fx_sparse_conv_fwd: null pointer or non-positive channel count");
        return FX_EINVAL;
    }
    if (in_dt != FX_F32 && in_dt != FX_F16 && in_dt != FX_BF16) { set_error("unknown input dtype"); return FX_EINVAL; }
    if (out_dt != in_dt && out_dt != FX_F32) {
        set_error("output dtype must equal the input dtype or be fp32");
        return FX_EUNSUPPORTED;
    }
    if (km->n_out == 0) return FX_OK;
    return conv_apply(km, d_feat, in_dt, d_w, C_in, C_out, d_out, out_dt, (hipStream_t)stream, kWeightsForward);
}

// ---------------------------------------------------------------------------------- no allocation
// fx_sparse_conv_fwd for callers that cannot allocate device memory (under graph capture, in tight serving loops):
// the packed weights and the work-list counters live in a file-scope device array instead of an allocation.
// The array's name stands for the symbol in host code; its device address is looked up once per device and only
// that address is ever handed to kernels.
namespace {
constexpr size_t kNoAllocScratchBytes = FX_NOALLOC_MAX_WEIGHT_BYTES + 224 + kConvWorkInts * sizeof(int32_t);
__device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];
constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices];
std::atomic<bool> g_scratch_ready[kMaxDevices];
std::mutex g_scratch_mu;
}  // namespace

// Device address of the scratch array on the current device (looked up on first use per device).
fx_status fx::conv_noalloc_setup(void** out_ptr) {
    int dev = 0;
    FX_HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) { set_error("device ordinal %d out of range", dev); return FX_EDEVICE; }
    if (!g_scratch_ready[dev].load(std::memory_order_acquire)) {
        std::lock_guard<std::mutex> lock(g_scratch_mu);
        if (!g_scratch_ready[dev].load(std::memory_order_relaxed)) {
            void* ptr = nullptr;
            FX_HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
            if (!ptr) { set_error("hipGetSymbolAddress returned a null address"); return FX_EDEVICE; }
            g_scratch_ptr[dev] = ptr;
            g_scratch_ready[dev].store(true, std::memory_order_release);
        }
    }
    if (out_ptr) *out_ptr = g_scratch_ptr[dev];
    return FX_OK;
}

extern "C" fx_status fx_sparse_conv_fwd_noalloc(const fx_kmap* km, const void* d_feat, fx_dtype in_dt, const void* d_w,
                                                int32_t C_in, int32_t C_out, void* d_out, fx_dtype out_dt, void* stream) {
    if (!km || !d_w || C_in < 1 || C_out < 1 || (km->n_in > 0 && !d_feat) || (km->n_out > 0 && !d_out)) {
        set_error("fx_sparse_conv_fwd_noalloc: null pointer or non-positive channel count");
        return FX_EINVAL;
    }
    if (in_dt != FX_F32 && in_dt != FX_F16 && in_dt != FX_BF16) { set_error("unknown input dtype"); return FX_EINVAL; }
    if (out_dt != in_dt && out_dt != FX_F32) {
        set_error("output dtype must equal the input dtype or be fp32");
        return FX_EUNSUPPORTED;
    }
    if (km->n_out == 0) return FX_OK;
    if (!conv_tiles_shape_ok(km, in_dt, C_in, C_out)) {
        set_error("fx_sparse_conv_fwd_noalloc: only maps and shapes of the matrix-unit kernels (a tiled map, input rows in whole "
                  "64-byte chunks, an even number of output channels); K = %d, C_in = %d, C_out = %d is not", km->K, C_in, C_out);
        return FX_EUNSUPPORTED;
    }
    const size_t need = conv_scratch_bytes(km->K3, C_in, C_out, in_dt == FX_F32 ? 4 : 2);
    if (need > kNoAllocScratchBytes) {
        set_error("fx_sparse_conv_fwd_noalloc: the packed weights need %zu bytes, the static buffer holds %zu "
                  "(FX_NOALLOC_MAX_WEIGHT_BYTES)", need, kNoAllocScratchBytes);
        return FX_ERANGE;
    }
    void* ptr = nullptr;
    FX_TRY(conv_noalloc_setup(&ptr));
    return conv_tiles_with_scratch(km, d_feat, in_dt, d_w, C_in, C_out, d_out, out_dt, (hipStream_t)stream, kWeightsForward, ptr);
}
