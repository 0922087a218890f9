// Convolution and weight gradient of 16-bit types at up to 16 contracted channels: a network's first layers.
//
// The tile kernels contract 32 channels of one offset at a time, so at 3 or 4 input channels most of a multiply would be
// padding; these shapes used to run one scalar thread per four outputs.  Here the contracted dimension is (offset,
// channel): with the channels padded to CP = 4, 8 or 16, one v_mfma_f32_32x32x16 takes four, two or one offsets, and a
// 3x3x3 kernel at four channels is seven multiplies for 32 voxels and 32 output channels -- few enough that nothing
// is sorted or skipped: rows without a neighbour are zeros.  What remains is memory: the dense table (4 K^3 bytes per
// voxel) read once, one 8- to 32-byte row gathered per pair, the outputs written once.
#include "conv_common.h"

namespace fx {

namespace {

constexpr int kLdThreads = 256, kLdWaves = kLdThreads / 64;

inline int padded_channels(int C) { return C <= 4 ? 4 : C <= 8 ? 8 : 16; }

// N (4 or 8) channels of a row of C 16-bit channels as words (row < 0, and channels from C on: zeros).  whole: C is N and
// rows are aligned to N elements.
template <int N> struct Words;
template <> struct Words<4> { typedef u32x2 type; };
template <> struct Words<8> { typedef u32x4 type; };
template <int N>
__device__ __forceinline__ typename Words<N>::type load_channels(const uint16_t* __restrict__ p, bool has, int C, bool whole) {
    typename Words<N>::type w = {};
    if (has) {
        if (whole) {
            w = *reinterpret_cast<const typename Words<N>::type*>(p);
        } else {
            uint32_t half[N];
#pragma unroll
            for (int e = 0; e < N; ++e) half[e] = e < C ? (uint32_t)p[e] : 0u;
#pragma unroll
            for (int e = 0; e < N / 2; ++e) w[e] = half[2 * e] | (half[2 * e + 1] << 16);
        }
    }
    return w;
}

// ---------------------------------------------------------------------------------- forward
// Wave = 32 consecutive rows of the table.  The rows' K3 entries are contiguous: read coalesced, kept in LDS (a stride of
// 27 words hits all banks).  Per multiply, lane (n, h) gathers the eight (offset, channel) values of voxel n that the
// operand layout wants from it: two rows of four channels, one of eight, or half a row of sixteen.  The gathers of
// seven multiplies are in flight together.  The weights are laid out in operand order in LDS once per (persistent)
// workgroup; with two n-tiles (NT) the columns interleave, so a lane stores two adjacent channels.
// A sum runs over the offsets that a row has.  The multiplies give a missing neighbour a row of zeros, which adds nothing
// unless a weight is infinite or NaN; that leaves sums that are not finite, and a wave with such a sum makes the sums of
// its 32 rows again from existing neighbours only.  (4 -> 32 on 347 k voxels takes 25.2 us; 28.1 with a look at the weights
// as they are staged instead, whose loads then waited for each other.)
template <typename T, bool OUT_F32, int CP, int NT, bool WHOLE>
__global__ void __launch_bounds__(kLdThreads, 4)
k_conv_lowdepth(const int32_t* __restrict__ table, int64_t n_rows, int K3, const uint16_t* __restrict__ feat,
                const uint16_t* __restrict__ w, int C_in, int C_out, void* __restrict__ out, int mode) {
    typedef typename Elem<T>::vec8 vec8;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    constexpr int kTaps = 16 / CP;                                  // offsets per multiply
    constexpr int kBatch = 7;
    const int n_steps = (K3 + kTaps - 1) / kTaps;
    uint16_t* wl = reinterpret_cast<uint16_t*>(lds_raw);            // [step][n-tile][lane][8]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int32_t* nb = reinterpret_cast<int32_t*>(lds_raw + (size_t)n_steps * NT * 1024) + wave * kGroup * K3;
    const int co0 = blockIdx.y * 32 * NT;
    for (int e0 = threadIdx.x; e0 < n_steps * NT * 512; e0 += 7 * kLdThreads) {      // seven loads in flight
        uint16_t v[7];
#pragma unroll
        for (int u = 0; u < 7; ++u) {
            const int e = e0 + u * kLdThreads, el = e & 7, l = (e >> 3) & 63, nt = (e >> 9) % NT, s = (e >> 9) / NT;
            const int k = 16 * s + 8 * (l >> 5) + el, kappa = k / CP, ci = k % CP;
            const int co = co0 + (NT == 2 ? 2 * (l & 31) + nt : (l & 31));
            v[u] = 0;
            if (kappa < K3 && ci < C_in && co < C_out) {
                const int64_t kw = (mode & kWeightsFlipped) ? K3 - 1 - kappa : kappa;
                v[u] = (mode & kWeightsTransposed) ? w[(kw * C_out + co) * C_in + ci] : w[(kw * C_in + ci) * C_out + co];
            }
        }
#pragma unroll
        for (int u = 0; u < 7; ++u)
            if (e0 + u * kLdThreads < n_steps * NT * 512) wl[e0 + u * kLdThreads] = v[u];
    }
    __syncthreads();
    const int n = lane & 31, h = lane >> 5;
    const int64_t n_blocks = (n_rows + kGroup - 1) / kGroup, stride = (int64_t)gridDim.x * kLdWaves;
    for (int64_t blk = (int64_t)blockIdx.x * kLdWaves + wave; blk < n_blocks; blk += stride) {
        const int64_t row0 = blk * kGroup;
        const int valid = (int)(n_rows - row0 < kGroup ? n_rows - row0 : kGroup);
        for (int e = lane; e < kGroup * K3; e += 64) nb[e] = e < valid * K3 ? table[row0 * K3 + e] : -1;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // a wave's LDS accesses are processed in order
        __builtin_amdgcn_wave_barrier();
        f32x16 acc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;
        const int32_t* my = nb + n * K3;
        for (int s0 = 0; s0 < n_steps; s0 += kBatch) {
            u32x4 a[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int s = s0 + u;
                if (CP == 4) {
                    const int t0 = 4 * s + 2 * h;
                    const int r0 = t0 < K3 ? my[t0] : -1, r1 = t0 + 1 < K3 ? my[t0 + 1] : -1;
                    const u32x2 lo = load_channels<4>(feat + (uint32_t)r0 * (uint32_t)C_in, r0 >= 0, C_in, WHOLE);
                    const u32x2 hi = load_channels<4>(feat + (uint32_t)r1 * (uint32_t)C_in, r1 >= 0, C_in, WHOLE);
                    a[u] = u32x4{lo[0], lo[1], hi[0], hi[1]};
                } else {       // one row of eight channels, or channels 8h .. 8h + 7 of a row of sixteen
                    const int t0 = CP == 8 ? 2 * s + h : s, c0 = CP == 8 ? 0 : 8 * h;
                    const int r0 = t0 < K3 ? my[t0] : -1;
                    a[u] = load_channels<8>(feat + ((uint32_t)r0 * (uint32_t)C_in + c0), r0 >= 0, C_in - c0, WHOLE);
                }
            }
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                if (s0 + u >= n_steps) continue;      // uniform
                const vec8 av = vec8_from_words<T>(a[u]);
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const vec8 bv = *reinterpret_cast<const vec8*>(wl + ((size_t)((s0 + u) * NT + t) * 64 + lane) * 8);
                    acc[t] = Elem<T>::mfma(av, bv, acc[t]);
                }
            }
        }
        // All gathers have arrived (vmcnt 0): said here once, because the compiler cannot tell it across the skipped steps and
        // waits for every store before the next where its registers are those of a gather (8 -> 64: 51 us in place of 44).
        __builtin_amdgcn_s_waitcnt(0x0F70);
        // register v of lane (n, h): voxel 8 * (v / 4) + 4 * h + v % 4 of the block, channel(s) of column n
        const int co = co0 + (NT == 2 ? 2 * n : n);
        float all = 0.f;                              // not finite if one of the sums is not
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) all += acc[t][v];
        auto store = [&](int r, const float (&sum)[NT]) {          // the lane's channel(s) of row r of the block
            const int64_t at = (row0 + r) * C_out + co;
            if (NT == 2 && co + 1 < C_out && (C_out & 1) == 0) {
                if (OUT_F32) *reinterpret_cast<f32x2*>(reinterpret_cast<float*>(out) + at) = f32x2{sum[0], sum[NT - 1]};
                else *reinterpret_cast<uint32_t*>(reinterpret_cast<uint16_t*>(out) + at) = Elem<T>::pack2(sum[0], sum[NT - 1]);
            } else {
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    if (co + t >= C_out) continue;
                    if (OUT_F32) reinterpret_cast<float*>(out)[at + t] = sum[t];
                    else reinterpret_cast<uint16_t*>(out)[at + t] = Elem<T>::from_float(sum[t]);
                }
            }
        };
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int r = 8 * (v >> 2) + 4 * h + (v & 3);
            if (r >= valid) continue;
            float sum[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) sum[t] = acc[t][v];
            store(r, sum);
        }
        if (__ballot(!isfinite(all))) {
#pragma unroll 1
            for (int v = 0; v < 16; ++v) {
                const int r = 8 * (v >> 2) + 4 * h + (v & 3);
                if (r >= valid) continue;
                float sum[NT] = {};
#pragma unroll 1
                for (int kappa = 0; kappa < K3; ++kappa) {
                    const int32_t src = nb[r * K3 + kappa];
                    if (src < 0) continue;
                    const int64_t kw = (mode & kWeightsFlipped) ? K3 - 1 - kappa : kappa;
#pragma unroll 1
                    for (int c0 = 0; c0 < C_in; c0 += 4) {           // four channels in flight
                        float x[4], wv[4][NT];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const int ci = min(c0 + u, C_in - 1);
                            x[u] = Elem<T>::to_float(feat[(int64_t)src * C_in + ci]);
#pragma unroll
                            for (int t = 0; t < NT; ++t) {
                                const int oc = min(co + t, C_out - 1);       // columns that do not exist are not stored
                                wv[u][t] = Elem<T>::to_float((mode & kWeightsTransposed) ? w[(kw * C_out + oc) * C_in + ci] : w[(kw * C_in + ci) * C_out + oc]);
                            }
                        }
#pragma unroll
                        for (int u = 0; u < 4; ++u)
#pragma unroll
                            for (int t = 0; t < NT; ++t) sum[t] = c0 + u < C_in ? fmaf(x[u], wv[u][t], sum[t]) : sum[t];
                    }
                }
                store(r, sum);
            }
        }
        __builtin_amdgcn_wave_barrier();              // the table entries are replaced for the next block
    }
}

// ---------------------------------------------------------------------------------- weight gradient
// gw[(offset, channel)][co] = sum over voxels: rows of the product are (offset, channel) pairs, 32 per accumulator tile.
// A workgroup takes 64 voxels at a time: every (voxel, offset) row is gathered once into LDS, as row [offset][CP] of
// its voxel, next to the voxels' gout rows, and both operands are read with the transposing LDS read (voxels along k).
// The four waves split the tiles of (offset, channel) rows, MT each.  Table entries of the 64 voxels are contiguous, so
// they are read coalesced.  Rows are padded by 32 bytes: the four voxels of a transposing read then lie in different banks.
// A sum runs over the pairs that exist.  The product gives a missing pair a row of zeros, which adds nothing unless the
// voxel's gout is infinite or NaN; that leaves sums that are not finite, and the workgroup makes those again pair by pair.
// (Keeping such values out of the product as the rows are staged cost 2 of 36 us at 4 -> 32 on 347 k voxels, 14 of 99 at
// 16 -> 64.)
constexpr int kLdVoxels = 64;

template <typename T, int CP, int MT, int NT>
__global__ void __launch_bounds__(kLdThreads)
k_wgrad_lowdepth(const int32_t* __restrict__ table, int64_t n_rows, int K3, const uint16_t* __restrict__ feat,
                 const uint16_t* __restrict__ gout, int C_in, int C_out, float* __restrict__ part, int whole, int gout_whole) {
    typedef typename Elem<T>::vec8 vec8;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    constexpr int kGoStride = 64 * NT + 32;
    const int n_mt = (K3 * CP + 31) / 32, x_stride = n_mt * 64 + 32;
    unsigned char* xl = lds_raw;                                       // [voxel][offset][CP]
    unsigned char* gl = lds_raw + (size_t)kLdVoxels * x_stride;        // [voxel][32 * NT channels]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = lane & 31, h = lane >> 5, q = lane & 3, jv = (lane >> 2) & 3, g1 = (lane >> 4) & 1;
    const int co0 = blockIdx.y * 32 * NT, cols = C_out - co0 < 32 * NT ? C_out - co0 : 32 * NT;
    for (int e = tid; e < kLdVoxels * (x_stride + kGoStride) / 16; e += kLdThreads)      // offsets and channels that do not exist stay zero
        reinterpret_cast<u32x4*>(lds_raw)[e] = u32x4{0, 0, 0, 0};
    f32x16 acc[MT][NT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[m][t][v] = 0.f;
    const int64_t n_chunks = (n_rows + kLdVoxels - 1) / kLdVoxels;
    const int64_t c0 = n_chunks * blockIdx.x / gridDim.x, c1 = n_chunks * (blockIdx.x + 1) / gridDim.x;
    __syncthreads();
    for (int64_t c = c0; c < c1; ++c) {
        const int64_t row0 = c * kLdVoxels;
        const int valid = (int)(n_rows - row0 < kLdVoxels ? n_rows - row0 : kLdVoxels);
        // gather: entry e = (voxel, offset); eight entries and then eight rows in flight
        for (int e0 = tid; e0 < kLdVoxels * K3; e0 += 8 * kLdThreads) {
            int32_t in[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int e = e0 + u * kLdThreads;
                in[u] = e < valid * K3 ? table[row0 * K3 + e] : -1;
            }
            constexpr int N = CP == 4 ? 4 : 8, P = CP / N;            // words per piece, pieces per row
            typename Words<N>::type x[8][P];
#pragma unroll
            for (int u = 0; u < 8; ++u)
#pragma unroll
                for (int d = 0; d < P; ++d) x[u][d] = load_channels<N>(feat + (int64_t)in[u] * C_in + d * N, in[u] >= 0, C_in - d * N, whole);
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int e = e0 + u * kLdThreads;
                if (e >= kLdVoxels * K3) continue;
                const int v = e / K3, kappa = e - v * K3;
#pragma unroll
                for (int d = 0; d < P; ++d)
                    *reinterpret_cast<typename Words<N>::type*>(xl + (size_t)v * x_stride + kappa * (2 * CP) + d * (2 * N)) = x[u][d];
            }
        }
        // gout rows of the voxels: pieces of eight channels (rows past the end are zero)
        for (int e = tid; e < kLdVoxels * 4 * NT; e += kLdThreads) {
            const int v = e / (4 * NT), p8 = (e - v * (4 * NT)) * 8;
            u32x4 g = u32x4{0, 0, 0, 0};
            if (v < valid) {
                g = load_channels<8>(gout + (row0 + v) * C_out + co0 + p8, true, cols - p8, gout_whole && p8 + 8 <= cols);
            }
            *reinterpret_cast<u32x4*>(gl + v * kGoStride + p8 * 2) = g;
        }
        __syncthreads();
#pragma unroll
        for (int ks = 0; ks < kLdVoxels / 16; ++ks) {
            const int v = 16 * ks + 8 * h + jv;       // and v + 4
            vec8 b[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const unsigned char* src = gl + v * kGoStride + (32 * t + 16 * g1 + 4 * q) * 2;
                const u32x2 lo = tr_read4(src), hi = tr_read4(src + 4 * kGoStride);
                b[t] = vec8_from_words<T>(u32x4{lo[0], lo[1], hi[0], hi[1]});
            }
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                const int mt = wave + kLdWaves * m;
                if (mt >= n_mt) continue;             // uniform
                const unsigned char* src = xl + (size_t)v * x_stride + (32 * mt + 16 * g1 + 4 * q) * 2;
                const u32x2 lo = tr_read4(src), hi = tr_read4(src + 4 * x_stride);
                const vec8 a = vec8_from_words<T>(u32x4{lo[0], lo[1], hi[0], hi[1]});
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[m][t] = Elem<T>::mfma(a, b[t], acc[m][t]);
            }
        }
        __syncthreads();
    }
    // lane (co = n, h), register v -> row 32 mt + 8 (v / 4) + 4 h + v % 4 = (offset, channel)
    float* dst = part + (int64_t)blockIdx.x * K3 * C_in * C_out;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const int mt = wave + kLdWaves * m;
        if (mt >= n_mt) continue;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = 32 * mt + 8 * (v >> 2) + 4 * h + (v & 3), kappa = row / CP, ci = row % CP, co = 32 * t + n;
                if (kappa < K3 && ci < C_in && co < cols) dst[((int64_t)kappa * C_in + ci) * C_out + co0 + co] = acc[m][t][v];
            }
    }
    float all = 0.f;                              // not finite if one of the sums is not
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) all += acc[m][t][v];
    int* any = reinterpret_cast<int*>(lds_raw);   // the operands are no longer needed
    if (tid == 0) *any = 0;
    __syncthreads();
    if (!isfinite(all)) *any = 1;
    __syncthreads();
    if (*any == 0) return;
    __threadfence();                              // the sums as stored, by whichever thread
    __syncthreads();
    const int64_t r0 = c0 * kLdVoxels, r1 = c1 * kLdVoxels < n_rows ? c1 * kLdVoxels : n_rows;
#pragma unroll 1
    for (int e = tid; e < K3 * C_in * cols; e += kLdThreads) {
        const int co = co0 + e % cols, k = e / cols, kappa = k / C_in, ci = k - kappa * C_in;
        float* at = dst + (int64_t)k * C_out + co;
        if (isfinite(*at)) continue;
        float sum = 0.f;
#pragma unroll 1
        for (int64_t r = r0; r < r1; r += 8) {    // eight table entries, then eight pairs in flight; added in row order
            int32_t in[8];
            float x[8], g[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) in[u] = r + u < r1 ? table[(r + u) * K3 + kappa] : -1;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                x[u] = Elem<T>::to_float(feat[(int64_t)max(in[u], 0) * C_in + ci]);
                g[u] = Elem<T>::to_float(gout[min(r + u, r1 - 1) * C_out + co]);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) sum = in[u] >= 0 ? fmaf(x[u], g[u], sum) : sum;
        }
        *at = sum;
    }
}

inline size_t conv_lds(int K3, int CP, int NT) {
    const int n_steps = (K3 * CP + 15) / 16;
    return (size_t)n_steps * NT * 1024 + sizeof(int32_t) * kLdWaves * kGroup * K3;
}
inline size_t wgrad_lds(int K3, int CP, int NT) {
    const int n_mt = (K3 * CP + 31) / 32;
    return (size_t)kLdVoxels * (n_mt * 64 + 32 + 64 * NT + 32);
}

}  // namespace

// Tiles of 32 (offset, channel) rows that a wave of the weight gradient holds: 1, or for more rows one number per channel
// padding (2x2x2 and 3x3x3 at 8 channels have 2 and 7 tiles for four waves, 3x3x3 at 16 and 5x5x5 at 4 have 14 and 16).
constexpr int most_tiles_per_wave(int CP) { return CP == 8 ? 2 : 4; }

// Up to 16 contracted channels of a 16-bit type, and operands that fit the LDS of a compute unit (all kernel sizes up to 3;
// 5x5x5 at up to 4 channels).
bool lowdepth_supported(fx_dtype dt, int K3, int C_contract, int64_t n_source_rows) {
    if (dt == FX_F32 || C_contract > 16 || n_source_rows * C_contract > 0xFFFFFFFFll) return false;     // 32-bit element offsets
    const int CP = padded_channels(C_contract);
    return conv_lds(K3, CP, 2) <= 160 * 1024 && wgrad_lds(K3, CP, 2) <= 160 * 1024 && (K3 * CP + 31) / 32 <= most_tiles_per_wave(CP) * kLdWaves;
}

fx_status lowdepth_conv_on_table(const int32_t* d_table, int64_t n_rows, int K3, const void* d_feat, fx_dtype dt, const void* d_w,
                                 int32_t C_in, int32_t C_out, void* d_out, fx_dtype out_dt, hipStream_t st, int mode) {
    const int CP = padded_channels(C_in);
    const bool whole = C_in == CP && (reinterpret_cast<uintptr_t>(d_feat) & (CP == 4 ? 7 : 15)) == 0;
    const int NT = C_out > 32 ? 2 : 1;
    const size_t lds = conv_lds(K3, CP, NT);
    const int64_t n_blocks = (n_rows + kGroup - 1) / kGroup;
    // Persistent workgroups, as many as a compute unit holds at once (four by registers, fewer by LDS), no more than
    // there are blocks (7 a unit, in turn, took 42 us for 347 k voxels 4 -> 32)
    const int per_cu = (int)std::max<size_t>(1, std::min<size_t>(4, (size_t)160 * 1024 / lds));
    const int n_y = (C_out + 32 * NT - 1) / (32 * NT);
    const int64_t want = std::max<int64_t>(1, (int64_t)compute_units() * per_cu / n_y);
    const dim3 grid((unsigned)std::min<int64_t>((n_blocks + kLdWaves - 1) / kLdWaves, want), (unsigned)n_y);
    ProfScope ps(kProfConvLowdepth, st);
    hipError_t e = hipSuccess;
#define FX_LD_WHOLE(T, F32, CPV, NTV, WH)                                                                                \
    do {                                                                                                                 \
        if (lds > 64 * 1024) e = hipFuncSetAttribute((const void*)k_conv_lowdepth<T, F32, CPV, NTV, WH>,                 \
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);              \
        if (e == hipSuccess)                                                                                             \
            k_conv_lowdepth<T, F32, CPV, NTV, WH><<<grid, kLdThreads, lds, st>>>(d_table, n_rows, K3,                    \
                (const uint16_t*)d_feat, (const uint16_t*)d_w, C_in, C_out, d_out, mode);                                \
    } while (0)
#define FX_LD_NT(T, F32, CPV, NTV)                                                                                       \
    do {                                                                                                                 \
        if (whole) FX_LD_WHOLE(T, F32, CPV, NTV, true); else FX_LD_WHOLE(T, F32, CPV, NTV, false);                       \
    } while (0)
#define FX_LD_CP(T, F32, CPV) do { if (NT == 2) FX_LD_NT(T, F32, CPV, 2); else FX_LD_NT(T, F32, CPV, 1); } while (0)
#define FX_LD(T, F32) do { if (CP == 4) FX_LD_CP(T, F32, 4); else if (CP == 8) FX_LD_CP(T, F32, 8); else FX_LD_CP(T, F32, 16); } while (0)
    if (dt == FX_BF16) { if (out_dt == FX_F32) FX_LD(__bf16, true); else FX_LD(__bf16, false); }
    else { if (out_dt == FX_F32) FX_LD(_Float16, true); else FX_LD(_Float16, false); }
#undef FX_LD
#undef FX_LD_CP
#undef FX_LD_NT
#undef FX_LD_WHOLE
    if (e == hipSuccess) e = hipGetLastError();
    if (e != hipSuccess) { set_error("low-depth convolution launch failed: %s", hipGetErrorString(e)); return FX_EDEVICE; }
    return FX_OK;
}

// Two workgroups per compute unit (and column slice), at least four chunks of 64 voxels each, and at most 64 MB of partial
// sums, which the reduction reads again: 512 of them are 7 MB at 4 -> 32 channels, but 226 MB at 16 -> 256.  On 347 k
// voxels 16 -> 128 / 256 / 512 and 4 -> 512 took 195 / 431 / 874 and 215 us without the last, 169 / 325 / 636 and 195
// with it; 32 MB make 16 -> 64 141 in place of 99.
int lowdepth_wgrad_ranges(int64_t n_rows, int K3, int C_in, int C_out) {
    const int64_t chunks = (n_rows + kLdVoxels - 1) / kLdVoxels, bytes = sizeof(float) * (int64_t)K3 * C_in * C_out;
    const int64_t cu = compute_units(), n_y = C_out > 32 ? (C_out + 63) / 64 : 1;
    const int64_t round = cu * (C_in <= 4 ? 4 : 1);          // workgroups side by side: four a unit fit at four channels, one at sixteen
    int64_t most = std::min<int64_t>(2 * cu, ((int64_t)64 << 20) / bytes);
    if (most < 2 * cu && most * n_y > round) most = most * n_y / round * round / n_y;        // whole rounds
    return (int)std::max<int64_t>(1, std::min<int64_t>((chunks + 3) / 4, most));
}

fx_status lowdepth_wgrad_partial(const int32_t* d_table, int64_t n_rows, int K3, const void* d_feat, const void* d_gout, fx_dtype dt,
                                 int32_t C_in, int32_t C_out, float* part, int n_ranges, hipStream_t st) {
    const int CP = padded_channels(C_in);
    const bool whole = C_in == CP && (reinterpret_cast<uintptr_t>(d_feat) & (CP == 4 ? 7 : 15)) == 0;
    const bool gout_whole = C_out % 8 == 0 && (reinterpret_cast<uintptr_t>(d_gout) & 15) == 0;
    const int NT = C_out > 32 ? 2 : 1;
    const size_t lds = wgrad_lds(K3, CP, NT);
    const bool one_tile = (K3 * CP + 31) / 32 <= kLdWaves;               // per wave
    const dim3 grid((unsigned)n_ranges, (unsigned)((C_out + 32 * NT - 1) / (32 * NT)));
    ProfScope ps(kProfWgrad, st);
    hipError_t e = hipSuccess;
#define FX_LD_MT(T, CPV, MTV, NTV)                                                                                       \
    do {                                                                                                                 \
        if (lds > 64 * 1024) e = hipFuncSetAttribute((const void*)k_wgrad_lowdepth<T, CPV, MTV, NTV>,                    \
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);              \
        if (e == hipSuccess)                                                                                             \
            k_wgrad_lowdepth<T, CPV, MTV, NTV><<<grid, kLdThreads, lds, st>>>(d_table, n_rows, K3, (const uint16_t*)d_feat, \
                (const uint16_t*)d_gout, C_in, C_out, part, whole ? 1 : 0, gout_whole ? 1 : 0);                          \
    } while (0)
#define FX_LD_NT(T, CPV, MTV) do { if (NT == 2) FX_LD_MT(T, CPV, MTV, 2); else FX_LD_MT(T, CPV, MTV, 1); } while (0)
#define FX_LD_CP(T, CPV) do { if (one_tile) FX_LD_NT(T, CPV, 1); else FX_LD_NT(T, CPV, most_tiles_per_wave(CPV)); } while (0)
#define FX_LD(T) do { if (CP == 4) FX_LD_CP(T, 4); else if (CP == 8) FX_LD_CP(T, 8); else FX_LD_CP(T, 16); } while (0)
    if (dt == FX_BF16) FX_LD(__bf16); else FX_LD(_Float16);
#undef FX_LD
#undef FX_LD_CP
#undef FX_LD_NT
#undef FX_LD_MT
    if (e == hipSuccess) e = hipGetLastError();
    if (e != hipSuccess) { set_error("low-depth weight gradient launch failed: %s", hipGetErrorString(e)); return FX_EDEVICE; }
    return FX_OK;
}

}  // namespace fx
