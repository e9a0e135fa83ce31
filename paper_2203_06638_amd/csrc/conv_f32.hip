// conv_f32.hip -- fp32 convolution passes on gfx950 matrix cores.
//
// Forward and data-gradient passes are one implicit GEMM
//     Y[m][n] = sum_k A[m][k] * B[n][k]
// with m an output pixel (NHWC), n an output channel, and k = (r, s, c) a
// filter tap and source channel.  A is gathered on the fly from the NHWC
// source activation; B is a weight matrix whose rows are contiguous in k
// (the snapshot writes both the forward layout W_f[cout][r][s][cin] and the
// data-gradient layout W_d[cin][r][s][cout]).
//
// Matrix-core mapping (v_mfma_f32_16x16x4_f32, 64 lanes): lane l supplies
// A[row = l%16][k = l/16] and B[k = l/16][col = l%16] and holds
// D[4*(l/16) + i][l%16], i = 0..3.  Each lane loads a float4 of four
// consecutive channels for its row (pixel) and its column (filter row); the
// four components feed four successive MFMAs, so the 16 k-values a lane
// group covers per float4 are permuted identically in A and B (the sum is
// over all of them either way).
//
// Weight gradient: dW[cout][(r,s,c)] = sum over output pixels p of
// dY[p][cout] * X_im2col[p][(r,s,c)] -- a GEMM whose reduction runs over
// N*Ho*Wo pixels.  Pixel chunks of 64 are staged through LDS (dY rows and
// im2col rows as loaded, float4 along channels); each wave reduces 16 of the
// chunk's pixels; waves are summed in a fixed order and every split of the
// pixel range writes its own partial, summed in order by a second kernel.
// Convolution outputs and weight gradients use no atomics and are bitwise
// reproducible; only the batch-norm sums of the forward epilogue are merged
// across workgroups by fp64 atomic adds (bnacc.h).
#include <algorithm>
#include <cstdint>

#include "bnacc.h"
#include "kernels.h"
#include "launch.h"

namespace lpp {

typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f4 relu4(f4 v) {
    return f4{fmaxf(v[0], 0.f), fmaxf(v[1], 0.f), fmaxf(v[2], 0.f), fmaxf(v[3], 0.f)};
}

__device__ __forceinline__ f4 mfma16x16x4(float a, float b, f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Offset of source pixel (n, hs, ws) feeding output pixel (n, p, q) through
// tap (r, s), or -1 when the tap falls in the zero padding / between strides.
template <int MODE>
__device__ __forceinline__ int src_pixel(int n, int p, int q, int r, int s, const ConvGeom& g) {
    int hs, ws;
    if (MODE == CONV_FWD) {
        hs = p * g.stride - g.pad + r;
        ws = q * g.stride - g.pad + s;
    } else {
        // dX[p][q] gathers dY[(p + pad - r)/stride][(q + pad - s)/stride]
        int hn = p + g.pad - r, wn = q + g.pad - s;
        if (hn < 0 || wn < 0) return -1;
        if (g.stride != 1) {
            if ((hn % g.stride) | (wn % g.stride)) return -1;
            hn /= g.stride;
            wn /= g.stride;
        }
        hs = hn;
        ws = wn;
    }
    if (hs < 0 || hs >= g.Hs || ws < 0 || ws >= g.Ws) return -1;
    return ((n * g.Hs + hs) * g.Ws + ws) * g.Cs;
}

// WM waves along m (4/WM along n); each wave owns TM x TN tiles of 16x16.
// FAST: Cs % 16 == 0, so a group of four float4 chunks never straddles a tap.
// STATS: also form, per output channel, the mean and the sum of squared
// deviations over this workgroup's BM output rows and add the tile's share of
// the batch sums (sum y, sum y^2) into the batch-norm accumulators.
template <int MODE, int WM, int TM, int TN, bool FAST, bool STATS>
__global__ __launch_bounds__(256) void conv_igemm_f32(const float* __restrict__ src, const float* __restrict__ B,
                                                      const float* __restrict__ bias, float* __restrict__ Y,
                                                      ConvGeom g, int accumulate, BnSums sums) {
    constexpr int WN = 4 / WM;
    constexpr int BM = WM * TM * 16, BN = WN * TN * 16;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave % WM, wn = wave / WM;
    const int gi = lane >> 4, li = lane & 15;
    const int HoWo = g.Ho * g.Wo;
    const int M = g.Nb * HoWo;
    const int Ktot = g.R * g.S * g.Cs;
    const int m_base = blockIdx.x * BM + wm * TM * 16;
    const int n_base = blockIdx.y * BN + wn * TN * 16;

    int an[TM], ap[TM], aq[TM];
    bool av[TM];
#pragma unroll
    for (int t = 0; t < TM; ++t) {
        int m = m_base + t * 16 + li;
        av[t] = m < M;
        int mm = av[t] ? m : 0;
        an[t] = mm / HoWo;
        int rem = mm - an[t] * HoWo;
        ap[t] = rem / g.Wo;
        aq[t] = rem - ap[t] * g.Wo;
    }
    const float* bp[TN];
    bool bv[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t) {
        int n = n_base + t * 16 + li;
        bv[t] = n < g.Ncols;
        bp[t] = B + (long)(bv[t] ? n : 0) * Ktot;
    }
    f4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};

    if (FAST) {
        for (int r = 0; r < g.R; ++r)
            for (int s = 0; s < g.S; ++s) {
                int so[TM];
#pragma unroll
                for (int t = 0; t < TM; ++t) so[t] = av[t] ? src_pixel<MODE>(an[t], ap[t], aq[t], r, s, g) : -1;
                const int kt = (r * g.S + s) * g.Cs;
                for (int c0 = 4 * gi; c0 < g.Cs; c0 += 16) {
                    f4 a[TM], b[TN];
#pragma unroll
                    for (int t = 0; t < TM; ++t)
                        a[t] = so[t] >= 0 ? *(const f4*)(src + so[t] + c0) : f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int t = 0; t < TN; ++t)
                        b[t] = bv[t] ? *(const f4*)(bp[t] + kt + c0) : f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int x = 0; x < TM; ++x)
#pragma unroll
                            for (int y = 0; y < TN; ++y) acc[x][y] = mfma16x16x4(a[x][j], b[y][j], acc[x][y]);
                }
            }
    } else {
        const int Cq = g.Cs >> 2;   // float4 chunks per tap
        const int KC = Ktot >> 2;   // float4 chunks in all of k
        for (int kc0 = 0; kc0 < KC; kc0 += 4) {
            const int kc = kc0 + gi;
            f4 a[TM], b[TN];
#pragma unroll
            for (int t = 0; t < TM; ++t) a[t] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < TN; ++t) b[t] = f4{0.f, 0.f, 0.f, 0.f};
            if (kc < KC) {
                int tap = kc / Cq;
                int c = (kc - tap * Cq) * 4;
                int r = tap / g.S, s = tap - r * g.S;
#pragma unroll
                for (int t = 0; t < TM; ++t) {
                    int so = av[t] ? src_pixel<MODE>(an[t], ap[t], aq[t], r, s, g) : -1;
                    if (so >= 0) a[t] = *(const f4*)(src + so + c);
                }
#pragma unroll
                for (int t = 0; t < TN; ++t)
                    if (bv[t]) b[t] = *(const f4*)(bp[t] + kc * 4);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int x = 0; x < TM; ++x)
#pragma unroll
                    for (int y = 0; y < TN; ++y) acc[x][y] = mfma16x16x4(a[x][j], b[y][j], acc[x][y]);
        }
    }

#pragma unroll
    for (int y = 0; y < TN; ++y) {
        const int n = n_base + y * 16 + li;
        const float bb = (bias && n < g.Ncols) ? bias[n] : 0.f;
#pragma unroll
        for (int x = 0; x < TM; ++x)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[x][y][i] += bb;
        if (n >= g.Ncols) continue;
#pragma unroll
        for (int x = 0; x < TM; ++x)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int m = m_base + x * 16 + gi * 4 + i;
                if (m >= M) continue;
                const long o = (long)m * g.Ncols + n;
                const float v = acc[x][y][i];
                Y[o] = accumulate == kStoreAdd ? Y[o] + v : (accumulate == kStoreRelu ? fmaxf(v, 0.f) : v);
            }
    }
    if (STATS) {
        __shared__ float red[WM][3][BN];
        const auto valid = [&](int x, int i) { return m_base + x * 16 + gi * 4 + i < M; };
        const auto store = [&](int t, float n, float mu, float m2) {
            if (blockIdx.y * BN + t < g.Ncols)
                tile_moments_store(sums, (int)blockIdx.x, g.Ncols, blockIdx.y * BN + t, n, mu, m2);
        };
        if ((int)blockIdx.x * BM + BM <= M) tile_moments<TM, TN, WM, BN, true>(acc, wm, wn, valid, red, store);
        else tile_moments<TM, TN, WM, BN, false>(acc, wm, wn, valid, red, store);
    }
}

// LDS-staged variant for Cs % 16 == 0.  A k-step is one filter tap and 16
// source channels.  The workgroup's A tile (BM rows x 16) and B tile (BN rows
// x 16) are loaded cooperatively as float4 (each thread keeps the same rows in
// every k-step, so row decoding happens once), double-buffered in LDS with the
// next k-step's global loads in flight during this k-step's MFMAs; one
// barrier per k-step.  Waves form a WM x WN grid over the tile; a wave owns
// TM x TN 16x16 output tiles and reads its operands as float4 from LDS.
template <int MODE, int BM, int BN, int WM, bool STATS>
__global__ __launch_bounds__(256) void conv_lds_f32(const float* __restrict__ src, const float* __restrict__ B,
                                                    const float* __restrict__ bias, float* __restrict__ Y,
                                                    ConvGeom g, int accumulate, BnSums sums) {
    constexpr int WN = 4 / WM;
    constexpr int TM = BM / (WM * 16), TN = BN / (WN * 16);
    constexpr int LDW = 20;                                  // 16 floats + 4 pad per LDS row
    constexpr int NA = (BM * 4 + 255) / 256, NB = (BN * 4 + 255) / 256;
    __shared__ float As[2][BM][LDW];
    __shared__ float Bs[2][BN][LDW];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave % WM, wn = wave / WM;
    const int gi = lane >> 4, li = lane & 15;
    const int HoWo = g.Ho * g.Wo;
    const int M = g.Nb * HoWo;
    const int Ktot = g.R * g.S * g.Cs;
    const int CG = g.Cs >> 4;                                // 16-channel groups per tap
    const int KS = g.R * g.S * CG;                           // k-steps
    const int m0 = blockIdx.x * BM, n0 = blockIdx.y * BN;
    const int quad = tid & 3;                                // each thread's float4 within a 16-wide row

    // rows of A this thread loads: (tid + 256 i) / 4
    int an[NA], ap[NA], aq[NA];
    bool av[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int row = (tid + 256 * i) >> 2;
        const int m = m0 + row;
        av[i] = (tid + 256 * i) < BM * 4 && m < M;
        const int mm = av[i] ? m : 0;
        an[i] = mm / HoWo;
        const int rem = mm - an[i] * HoWo;
        ap[i] = rem / g.Wo;
        aq[i] = rem - ap[i] * g.Wo;
    }
    const float* brow[NB];
    bool bvld[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int row = (tid + 256 * i) >> 2;
        const int n = n0 + row;
        bvld[i] = (tid + 256 * i) < BN * 4 && n < g.Ncols;
        brow[i] = B + (long)(bvld[i] ? n : 0) * Ktot + quad * 4;
    }

    f4 ra[NA], rb[NB];
    auto gload = [&](int ks) {
        const int tap = ks / CG;
        const int cg = ks - tap * CG;
        const int r = tap / g.S, sx = tap - r * g.S;
        const int c = cg * 16 + quad * 4;
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int so = av[i] ? src_pixel<MODE>(an[i], ap[i], aq[i], r, sx, g) : -1;
            ra[i] = so >= 0 ? *(const f4*)(src + so + c) : f4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) rb[i] = bvld[i] ? *(const f4*)(brow[i] + ks * 16) : f4{0.f, 0.f, 0.f, 0.f};
    };
    auto lstore = [&](int buf) {
#pragma unroll
        for (int i = 0; i < NA; ++i)
            if ((tid + 256 * i) < BM * 4) *(f4*)&As[buf][(tid + 256 * i) >> 2][quad * 4] = ra[i];
#pragma unroll
        for (int i = 0; i < NB; ++i)
            if ((tid + 256 * i) < BN * 4) *(f4*)&Bs[buf][(tid + 256 * i) >> 2][quad * 4] = rb[i];
    };

    f4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};

    gload(0);
    lstore(0);
    __syncthreads();
    for (int ks = 0; ks < KS; ++ks) {
        const int buf = ks & 1;
        if (ks + 1 < KS) gload(ks + 1);
        f4 a[TM], b[TN];
#pragma unroll
        for (int x = 0; x < TM; ++x) a[x] = *(const f4*)&As[buf][(wm * TM + x) * 16 + li][gi * 4];
#pragma unroll
        for (int y = 0; y < TN; ++y) b[y] = *(const f4*)&Bs[buf][(wn * TN + y) * 16 + li][gi * 4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int x = 0; x < TM; ++x)
#pragma unroll
                for (int y = 0; y < TN; ++y) acc[x][y] = mfma16x16x4(a[x][j], b[y][j], acc[x][y]);
        if (ks + 1 < KS) lstore(buf ^ 1);
        __syncthreads();
    }

    const int m_base = m0 + wm * TM * 16;
    const int n_base = n0 + wn * TN * 16;
#pragma unroll
    for (int y = 0; y < TN; ++y) {
        const int n = n_base + y * 16 + li;
        const float bb = (bias && n < g.Ncols) ? bias[n] : 0.f;
#pragma unroll
        for (int x = 0; x < TM; ++x)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[x][y][i] += bb;
        if (n >= g.Ncols) continue;
#pragma unroll
        for (int x = 0; x < TM; ++x)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int m = m_base + x * 16 + gi * 4 + i;
                if (m >= M) continue;
                const long o = (long)m * g.Ncols + n;
                const float v = acc[x][y][i];
                Y[o] = accumulate == kStoreAdd ? Y[o] + v : (accumulate == kStoreRelu ? fmaxf(v, 0.f) : v);
            }
    }
    if (STATS) {
        __shared__ float red[WM][3][BN];
        const auto valid = [&](int x, int i) { return m_base + x * 16 + gi * 4 + i < M; };
        const auto store = [&](int t, float n, float mu, float m2) {
            if (n0 + t < g.Ncols) tile_moments_store(sums, (int)blockIdx.x, g.Ncols, n0 + t, n, mu, m2);
        };
        if (m0 + BM <= M) tile_moments<TM, TN, WM, BN, true>(acc, wm, wn, valid, red, store);
        else tile_moments<TM, TN, WM, BN, false>(acc, wm, wn, valid, red, store);
    }
}

template <int MODE, int BM, int BN, int WM>
static hipError_t launch_lds(const float* src, const float* B, const float* bias, float* Y, const ConvGeom& g,
                             int acc, const BnSums* stats, hipStream_t st) {
    const long M = (long)g.Nb * g.Ho * g.Wo;
    dim3 grid((unsigned)((M + BM - 1) / BM), (unsigned)((g.Ncols + BN - 1) / BN));
    if (stats)
        launch((conv_lds_f32<MODE, BM, BN, WM, true>), grid, dim3(256), 0, st, src, B, bias, Y, g,
                           (int)acc, stats ? *stats : BnSums{});
    else
        launch((conv_lds_f32<MODE, BM, BN, WM, false>), grid, dim3(256), 0, st, src, B, bias, Y, g,
                           (int)acc, stats ? *stats : BnSums{});
    return hipGetLastError();
}

// ------------------------------------------------------------------------
// spatial tiles: boxes of pixel slots over the stacked images
// ------------------------------------------------------------------------

// The images' output rows are stacked (row R = n * Hper + h).  A box is OH
// stacked rows x OW columns in OH x OWs slots (OWs >= OW); nc boxes side by
// side cover a row, and a box may reach over the end of an image, so any
// image size fills its slots.  Its input rows are rows of the padded stack,
// Hp rows an image, of which output row R reads S(R), S(R) + 1, ...,
// S(R) = n * Hp + h * step.
struct BoxGeom {
    int OH, OW, OWs, nc;        // box; boxes per row
    int rows;                   // Nb * Hper
    int Hper, Wo;               // output rows and columns of one image
    int Hp, step;               // padded rows of one image, rows between output rows
    int IH, IW;                 // staged rows and columns
    int pad_eff;                // input row of padded row hh: hh - pad_eff
    int far;                    // an activation is larger than 32-bit offsets reach
    unsigned OWs_inv, IW_inv, Hper_inv, Hp_inv, nc_inv;
};

// n / d == box_div(n, box_inv(d)) for n * d < 2^32 (checked on the host)
static unsigned box_inv(int d) { return d == 1 ? 0u : (unsigned)((0x100000000ull + d - 1) / d); }
__device__ __forceinline__ int box_div(int n, unsigned inv) { return inv ? (int)__umulhi((unsigned)n, inv) : n; }

// S(R)
__device__ __forceinline__ int box_prow(const BoxGeom& t, int R) {
    const int n = box_div(R, t.Hper_inv);
    return n * t.Hp + (R - n * t.Hper) * t.step;
}

// Tensors are read through buffer descriptors: a load at kNoLoad lies past
// every one and returns zero, so the zero padding costs no branch, and (unlike
// a pointer chosen at run time, a flat address) the loads count apart from the
// LDS accesses and stay in flight across a barrier and the MFMAs.  Offsets are
// of 32 bits: for a larger activation (BoxGeom::far) the descriptor begins at
// the box's first image or row and reaches at most to kNoLoad.  (The weight
// gradients, which form it for every box, do so in variants of their own: 50
// us on 16 x 56x56x64 without, 53 with.)
constexpr unsigned kNoLoad = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const float* p, long n) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)p, (short)0, (int)(n < 0x1fffffffL ? n * 4 : 0x7ffffffcL), 0x00020000);
}
// rows first, first + 1, ... of a tensor of `rows` rows of n floats
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const float* p, int first, long n, int rows) {
    if (first) p += first * n;
    return buf_rsrc(p, (rows - first) * n);
}
__device__ __forceinline__ f4 buf_load4(__amdgpu_buffer_rsrc_t r, unsigned off, int soff) {
    return __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(r, off, soff, 0));
}
// the workgroup's LDS accesses done, loads from memory left in flight
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Shapes boxes of `slots` slots, nc to a row, over Nb images of Hper x Wo
// outputs, each reading `ext` padded rows and columns, `step` apart; box
// columns are rounded up to a multiple of cq slots.  False when a box stages
// more than max_batches * 64 input pixels.
static bool box_shape(BoxGeom& t, int Nb, int Hper, int Wo, int ext, int step, int slots, int nc, int cq,
                      int max_batches) {
    if (nc > Wo) return false;
    t.OW = (Wo + nc - 1) / nc;
    t.OWs = cq == 1 ? t.OW : (t.OW + cq - 1) / cq * cq;
    if (t.OWs > slots) return false;
    t.nc = (Wo + t.OW - 1) / t.OW;
    t.rows = Nb * Hper;
    t.OH = std::min(slots / t.OWs, t.rows);
    // over the ends of as many images as OH rows can reach over
    const int ends = Hper % t.OH == 0 ? 0 : (t.OH + Hper - 2) / Hper;
    t.IH = (t.OH - 1) * step + ext + ends * std::max(0, ext - step);
    t.IW = (t.OWs - 1) * step + ext;
    return (t.IH * (long)t.IW + 63) / 64 <= max_batches;
}

// The rest of a shaped box's geometry.  False when an index leaves box_div's
// range.
static bool box_fill(BoxGeom& t, int Nb, int Hper, int Wo, int ext, int step, int pad_eff) {
    t.Hper = Hper;
    t.Wo = Wo;
    t.step = step;
    t.Hp = (Hper - 1) * step + ext;
    t.pad_eff = pad_eff;
    const double tiles = (double)((t.rows + t.OH - 1) / t.OH) * t.nc;
    if (((double)Nb * t.Hp + t.IH) * t.Hp >= 4294967296.0 || (double)t.rows * Hper >= 4294967296.0 ||
        tiles >= 1073741824.0 || tiles * t.nc >= 4294967296.0)
        return false;
    t.OWs_inv = box_inv(t.OWs);
    t.IW_inv = box_inv(t.IW);
    t.Hper_inv = box_inv(Hper);
    t.Hp_inv = box_inv(t.Hp);
    t.nc_inv = box_inv(t.nc);
    return true;
}
static int box_tiles(const BoxGeom& t) { return (t.rows + t.OH - 1) / t.OH * t.nc; }
// every slot of every box holds a pixel
static bool box_full(const BoxGeom& t, int slots) {
    return t.OH * t.OWs == slots && t.OWs == t.OW && t.OW * t.nc == t.Wo && t.rows % t.OH == 0;
}

// The number of boxes per row: among those within 4% of the fewest boxes, the
// one that stages the fewest batches of 64 input pixels, then the fewest
// boxes.  (At 28 columns and 64 slots 16 x 4 boxes fill all slots, 2 x 28 only
// 56; square boxes stage the smallest halo.)  Runs at every launch outside a
// graph.
static bool box_pick(BoxGeom& out, int Nb, int Hper, int Wo, int ext, int step, int pad_eff, int slots, int cq,
                     int max_batches) {
    if ((long)Nb * Hper >= (1L << 30)) return false;
    BoxGeom t;
    int nc[32], tiles[32], batches[32], n = 0, last = 0;
    long fewest = 0;
    for (int k = 1; k <= 32; ++k) {
        if ((long)k * slots < Wo || (last && (Wo + k - 1) / k == last)) continue;   // too wide; the last one's box
        if (!box_shape(t, Nb, Hper, Wo, ext, step, slots, k, cq, max_batches)) continue;
        const long b = (long)((t.rows + t.OH - 1) / t.OH) * t.nc;
        if (b >= (1L << 30)) continue;
        last = t.OW;
        nc[n] = k;
        tiles[n] = (int)b;
        batches[n++] = (t.IH * t.IW + 63) / 64;
        if (!fewest || b < fewest) fewest = b;
    }
    int best = -1;
    for (int i = 0; i < n; ++i)
        if (tiles[i] * 25L <= fewest * 26 &&
            (best < 0 || batches[i] < batches[best] || (batches[i] == batches[best] && tiles[i] < tiles[best])))
            best = i;
    return best >= 0 && box_shape(out, Nb, Hper, Wo, ext, step, slots, nc[best], cq, max_batches) &&
           box_fill(out, Nb, Hper, Wo, ext, step, pad_eff);
}

// n floats addressable with the kernels' 32-bit offsets
static bool buf_fits(double n) { return 4.0 * n < 2147483648.0; }
// so are the images that a box's staged rows may lie in (one more than its
// output rows reach over: a box ends in the padding of the next), of `image`
// floats; sets far
static bool box_fits(BoxGeom& t, int Nb, double image) {
    t.far = !buf_fits(Nb * image);
    return buf_fits(((t.OH - 1) / t.Hper + 3) * image);
}

// Epilogue of a box tile: bias, the output block through LDS, the store (set,
// add, ReLU) and the batch-norm sums (STATS).
template <int MODE, int TM, int TN, bool STATS>
__device__ __forceinline__ void box_store(f4 (&acc)[TM][TN], float* lds, const float* __restrict__ bias,
                                          float* __restrict__ Y, const ConvGeom& g, const BoxGeom& t, int accumulate,
                                          const BnSums& sums, const BnBwdSum& bs, int R0, int w0, int ohv, int owv,
                                          int n0) {
    constexpr int BN = TN * 16;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int gi = lane >> 4, li = lane & 15;
    if (bias) {
#pragma unroll
        for (int y = 0; y < TN; ++y) {
            const int n = n0 + y * 16 + li;
            const float bb = n < g.Ncols ? bias[n] : 0.f;
#pragma unroll
            for (int x = 0; x < TM; ++x)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[x][y][i] += bb;
        }
    }
    // the wave's TM*16 x TN*16 output block, transposed through LDS so that
    // every lane stores whole float4 channel quads of one pixel
    f4 bs0 = f4{0.f, 0.f, 0.f, 0.f}, bs1 = bs0;   // data gradient with STATS: sum gm, sum gm*xhat
    {
        constexpr int OP = TN * 16 + 4;           // LDS pitch of a pixel row
        float* Ot = lds + wave * (TM * 16 * OP);
#pragma unroll
        for (int x = 0; x < TM; ++x)
#pragma unroll
            for (int y = 0; y < TN; ++y)
#pragma unroll
                for (int i = 0; i < 4; ++i) Ot[(x * 16 + gi * 4 + i) * OP + y * 16 + li] = acc[x][y][i];
        __builtin_amdgcn_wave_barrier();          // a wave's LDS accesses execute in order
        constexpr int QPP = TN * 4;               // float4 quads per pixel of the block
        const int qd = lane % QPP, n = n0 + qd * 4;   // (64 % QPP == 0: a lane keeps one channel quad)
        f4 bmu{}, brs{}, bsc{}, bsh{};
        if (MODE == CONV_DGRAD && STATS && n < g.Ncols) {
            bmu = *(const f4*)(bs.aux + n);
            brs = *(const f4*)(bs.aux + g.Ncols + n);
            bsc = *(const f4*)(bs.aux + 2 * g.Ncols + n);
            bsh = *(const f4*)(bs.aux + 3 * g.Ncols + n);
        }
#pragma unroll
        for (int k = 0; k < TM * 16 * QPP / 64; ++k) {
            const int pl = (k * 64 + lane) / QPP;
            const int p = wave * TM * 16 + pl;
            const int oh = box_div(p, t.OWs_inv), ow = p - oh * t.OWs;
            if (oh < ohv && ow < owv && n < g.Ncols) {
                const long e = ((long)(R0 + oh) * t.Wo + w0 + ow) * g.Ncols + n;
                const f4 v = *(const f4*)(Ot + pl * OP + qd * 4);
                f4* o = (f4*)(Y + e);
                const f4 tot = accumulate == kStoreAdd ? *o + v : (accumulate == kStoreRelu ? relu4(v) : v);
                *o = tot;
                if (MODE == CONV_DGRAD && STATS) {
                    // gm = the stored gradient where the forward's ReLU passed
                    // (its output y > 0, or fma(x, scale, shift) > 0), xhat of the BN input
                    const f4 x = *(const f4*)(bs.x1 + e);
                    const f4 yv = bs.y ? *(const f4*)(bs.y + e) : f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const bool pass = bs.y ? yv[j] > 0.f : __builtin_fmaf(x[j], bsc[j], bsh[j]) > 0.f;
                        const float gm = pass ? tot[j] : 0.f;
                        bs0[j] += gm;
                        bs1[j] += gm * ((x[j] - bmu[j]) * brs[j]);
                    }
                }
            }
        }
    }
    if constexpr (MODE == CONV_DGRAD && STATS) {
        // lanes of one channel quad summed by a fixed xor tree, then the four waves in order
        constexpr int QPP = TN * 4;
#pragma unroll
        for (int o = QPP; o < 64; o <<= 1) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                bs0[j] += __shfl_xor(bs0[j], o);
                bs1[j] += __shfl_xor(bs1[j], o);
            }
        }
        __shared__ f4 bred[4][2][QPP];
        if (lane < QPP) {
            bred[wave][0][lane] = bs0;
            bred[wave][1][lane] = bs1;
        }
        __syncthreads();
        if (tid < 2 * BN) {
            const int k = tid / BN, cl = tid - k * BN, c = n0 + cl;
            float s = bred[0][k][cl >> 2][cl & 3];
            for (int w = 1; w < 4; ++w) s += bred[w][k][cl >> 2][cl & 3];
            if (c < g.Ncols) {
                if (sums.acc) acc_add(sums.acc, k, (int)blockIdx.x, g.Ncols, c, (double)s);
                else (k ? sums.p1 : sums.p0)[(long)blockIdx.x * g.Ncols + c] = s;
            }
        }
    }
    if constexpr (MODE == CONV_FWD && STATS) {
        __shared__ float red[4][3][BN];
        const auto store = [&](int c, float n, float mu, float m2) {
            if (n0 + c < g.Ncols) tile_moments_store(sums, (int)blockIdx.x, g.Ncols, n0 + c, n, mu, m2);
        };
        if (ohv * owv == TM * 64) {
            tile_moments<TM, TN, 4, BN, true>(acc, wave, 0, [](int, int) { return true; }, red, store);
        } else {
            // slots of this lane's accumulator rows that hold a pixel
            unsigned ok = 0;
#pragma unroll
            for (int x = 0; x < TM; ++x)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int p = (wave * TM + x) * 16 + gi * 4 + i;
                    const int oh = box_div(p, t.OWs_inv), ow = p - oh * t.OWs;
                    if (oh < ohv && ow < owv) ok |= 1u << (x * 4 + i);
                }
            tile_moments<TM, TN, 4, BN, false>(
                acc, wave, 0, [&](int x, int i) { return ((ok >> (x * 4 + i)) & 1) != 0; }, red, store);
        }
    }
}

// Spatially tiled convolution (3x3 and 1x1 passes with Cs % 4 == 0: forward
// with any stride, stride-1 data gradients; the data gradient of a stride-1
// conv is a forward conv of dY with the filter flipped and padding KS-1-pad).
// A workgroup takes one box of TM * 64 pixel slots and TN * 16 output
// channels.  Per 16 source channels the box's input rows, halo and padding
// included, and the filter slice go into LDS once and every tap runs from
// there; the next channel group's loads are in flight during this group's
// MFMAs.  At ResNet-20's sizes a pass is one round of workgroups, bound by the
// latency of its phases (loads, MFMAs, epilogue), so small boxes with several
// workgroups to a compute unit, whose phases overlap, are the fastest: 128
// slots where they still give 512 workgroups, else 64 (measured over 38
// passes within 2% of the best of 64/128/256 slots x 16/32 channels).
// 1x1 passes are bound by staging and take 32 channels where that still gives
// 512 workgroups.  Against tiles of whole rows (which took only widths that
// divide 64, 128 or 256, staged through flat loads that the compiler drained
// before the MFMAs): ResNet-20's stages 11.7 / 10.5 / 10.9 -> 10.9 / 9.5 / 9.4
// us forward; against the GEMM kernel that other widths ran on: 100 x 28x28x16
// 16.9 -> 8.9 us, 16 x 56x56x64 62 -> 43 us, 16 x 28x28x128 69 -> 43 us.
//
// INBN (forward passes): the source is the input of a training-mode batch
// norm followed by a ReLU; each staged source value becomes
// relu(fma(x, scale[c], shift[c])) (padding stays zero), with the per-channel
// coefficients derived in the prologue from the batch sums (or read from aux;
// bnacc.h).  The normalised tensor is never stored.
constexpr int kTileBatches = 6;   // staged input quads per thread and channel group, at most

template <int MODE, int KS, int TM, int TN, bool STATS, bool INBN>
__global__ __launch_bounds__(256) void conv_tile_f32(const float* __restrict__ src, const float* __restrict__ B,
                                                    const float* __restrict__ bias, float* __restrict__ Y, ConvGeom g,
                                                    BoxGeom t, int accumulate, BnSums sums, BnFwd inbn, BnBwdSum bs) {
    constexpr int BN = TN * 16, RS = KS * KS, LDW = 20;
    constexpr int NW = (BN * RS * 4 + 255) / 256;     // weight quads per thread and channel group
    extern __shared__ float lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int gi = lane >> 4, li = lane & 15, q = tid & 3;
    const int tr = box_div((int)blockIdx.x, t.nc_inv), tc = (int)blockIdx.x - tr * t.nc;
    const int R0 = tr * t.OH, w0 = tc * t.OW;
    const int ohv = min(t.OH, t.rows - R0), owv = min(t.OW, t.Wo - w0);
    const int n0 = blockIdx.y * BN;
    const int P0 = box_prow(t, R0);
    const int nx = t.IH * t.IW * 4, nxu = (nx + 255) >> 8;   // staged input quads, batches of them
    float* Xs = lds;                                  // [IH * IW][LDW]
    float* Ws = lds + t.IH * t.IW * LDW;              // [BN * RS][LDW]

    __shared__ float in_co[INBN ? 2 * kFoldMaxC : 1];   // scale | shift of the source channels
    if (INBN) bn_fwd_coeffs(inbn, g.Cs, in_co, in_co + kFoldMaxC);

    // byte offsets of this thread's quads at channel group 0
    const int n1 = t.far ? box_div(P0, t.Hp_inv) : 0;   // the descriptor's first image
    const long image = (long)g.Hs * g.Ws * g.Cs;
    const __amdgpu_buffer_rsrc_t xr = buf_rsrc(src, n1, image, g.Nb);
    const __amdgpu_buffer_rsrc_t wr = buf_rsrc(B, (long)g.Ncols * RS * g.Cs);
    unsigned xo[kTileBatches], wo[NW];
#pragma unroll
    for (int u = 0; u < kTileBatches; ++u) {
        xo[u] = kNoLoad;
        if (u < nxu) {
            const int pix = (tid + u * 256) >> 2;
            const int ih = box_div(pix, t.IW_inv), iw = pix - ih * t.IW;
            const int pr = P0 + ih;
            const int n = box_div(pr, t.Hp_inv), hh = pr - n * t.Hp;
            // a 1x1 pass stages only the pixels it reads
            const int h = (KS == 1 ? hh * g.stride : hh) - t.pad_eff;
            const int w = (KS == 1 ? (w0 + iw) * g.stride : w0 * g.stride + iw) - t.pad_eff;
            if (ih < t.IH && n < g.Nb && h >= 0 && h < g.Hs && w >= 0 && w < g.Ws)
                xo[u] = (unsigned)((((n - n1) * g.Hs + h) * g.Ws + w) * g.Cs + q * 4) * 4u;
        }
    }
#pragma unroll
    for (int u = 0; u < NW; ++u) {
        const int rest = (tid + u * 256) >> 2;
        const int nl = rest / RS, tap = rest - nl * RS;
        const int stap = MODE == CONV_FWD ? tap : RS - 1 - tap;
        wo[u] = (nl < BN && n0 + nl < g.Ncols) ? (unsigned)(((n0 + nl) * RS + stap) * g.Cs + q * 4) * 4u : kNoLoad;
    }
    f4 xv[kTileBatches], wv[NW];
    auto load = [&](int c0) {
        const unsigned bad = c0 + q * 4 < g.Cs ? 0u : kNoLoad;
#pragma unroll
        for (int u = 0; u < kTileBatches; ++u)
            if (u < nxu) xv[u] = buf_load4(xr, xo[u] | bad, c0 * 4);
#pragma unroll
        for (int u = 0; u < NW; ++u) wv[u] = buf_load4(wr, wo[u] | bad, c0 * 4);
    };
    load(0);

    // LDS offset of the input pixel each of this lane's slots reads at tap
    // (0, 0); slots outside the box's pixels read the first one's
    int abase[TM];
#pragma unroll
    for (int x = 0; x < TM; ++x) {
        const int p = (wave * TM + x) * 16 + li;
        const int oh = box_div(p, t.OWs_inv), ow = p - oh * t.OWs;
        const bool ok = oh < ohv && ow < owv;
        const int prow = ok ? box_prow(t, R0 + oh) - P0 : 0;
        abase[x] = (prow * t.IW + (ok ? ow * (KS == 1 ? 1 : g.stride) : 0)) * LDW + gi * 4;
    }
    f4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
    if (INBN) __syncthreads();

    const int sdst = (tid >> 2) * LDW + q * 4;
    for (int c0 = 0; c0 < g.Cs; c0 += 16) {
        if (INBN) {
            // relu(fma(x, scale, shift)); the zero padding stays zero
            f4 sc = f4{0.f, 0.f, 0.f, 0.f}, sh = sc;
            if (c0 + q * 4 < g.Cs) {
                sc = *(const f4*)(in_co + c0 + q * 4);
                sh = *(const f4*)(in_co + kFoldMaxC + c0 + q * 4);
            }
#pragma unroll
            for (int u = 0; u < kTileBatches; ++u)
                if (u < nxu) {
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        xv[u][k] = xo[u] == kNoLoad ? 0.f : fmaxf(__builtin_fmaf(xv[u][k], sc[k], sh[k]), 0.f);
                }
        }
#pragma unroll
        for (int u = 0; u < kTileBatches; ++u)
            if (u < nxu && tid + u * 256 < nx) *(f4*)(Xs + sdst + u * 64 * LDW) = xv[u];
#pragma unroll
        for (int u = 0; u < NW; ++u)
            if (tid + u * 256 < BN * RS * 4) *(f4*)(Ws + sdst + u * 64 * LDW) = wv[u];
        lds_barrier();
        if (c0 + 16 < g.Cs) load(c0 + 16);            // in flight during this group's MFMAs
#pragma unroll
        for (int tap = 0; tap < RS; ++tap) {
            const int toff = ((tap / KS) * t.IW + tap % KS) * LDW;
            f4 a[TM], b[TN];
#pragma unroll
            for (int x = 0; x < TM; ++x) a[x] = *(const f4*)(Xs + abase[x] + toff);
#pragma unroll
            for (int y = 0; y < TN; ++y) b[y] = *(const f4*)(Ws + ((y * 16 + li) * RS + tap) * LDW + gi * 4);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int x = 0; x < TM; ++x)
#pragma unroll
                    for (int y = 0; y < TN; ++y) acc[x][y] = mfma16x16x4(a[x][j], b[y][j], acc[x][y]);
        }
        lds_barrier();
    }

    box_store<MODE, TM, TN, STATS>(acc, lds, bias, Y, g, t, accumulate, sums, bs, R0, w0, ohv, owv, n0);
}

struct TileCfg { int tm, tn, tiles; BoxGeom t; size_t lds; };

// Box and channel tile of a pass, or false when the spatial kernel does not
// take it (the GEMM-style kernels do).
static bool pick_tile(int mode, const ConvGeom& g, TileCfg& out) {
    if (g.Cs % 4 || g.Cs < 16 || g.Ncols % 4 || g.R != g.S || (g.R != 1 && g.R != 3)) return false;
    if (mode == CONV_DGRAD && g.stride != 1) return false;
    if (!buf_fits((double)g.Ncols * g.R * g.R * g.Cs)) return false;
    static const int shapes[][2] = {{2, 2}, {2, 1}, {1, 1}};
    bool found = false;
    for (auto& sh : shapes) {
        const int tm = sh[0], tn = sh[1], bn = tn * 16;
        if (tn == 2 && (g.R != 1 || g.Ncols % 32)) continue;
        TileCfg c;
        if (!box_pick(c.t, g.Nb, g.Ho, g.Wo, g.R, g.R == 1 ? 1 : g.stride, mode == CONV_FWD ? g.pad : g.R - 1 - g.pad,
                      tm * 64, 1, kTileBatches) ||
            !box_fits(c.t, g.Nb, (double)g.Hs * g.Ws * g.Cs))
            continue;
        c.tm = tm;
        c.tn = tn;
        c.tiles = box_tiles(c.t);
        // the staged tiles; the epilogue's transpose reuses the space
        c.lds = sizeof(float) * std::max<size_t>(20 * ((size_t)c.t.IH * c.t.IW + (size_t)bn * g.R * g.R),
                                                 (size_t)4 * tm * 16 * (bn + 4));
        found = true;
        out = c;
        if ((long)c.tiles * ((g.Ncols + bn - 1) / bn) >= 512) break;
    }
    return found;
}

template <int MODE, int KS, int TM, int TN>
static hipError_t launch_tile(const float* src, const float* B, const float* bias, float* Y, const ConvGeom& g,
                              const TileCfg& c, int acc, const BnSums* stats, const BnFwd* inbn,
                              const BnBwdSum* bsv, hipStream_t st) {
    dim3 grid((unsigned)c.tiles, (unsigned)((g.Ncols + TN * 16 - 1) / (TN * 16)));
    const BnSums sm = stats ? *stats : BnSums{};
    const BnFwd ib = inbn ? *inbn : BnFwd{};
    const BnBwdSum bsum = bsv ? *bsv : BnBwdSum{};
    // a data gradient's statistics are the sums of a BN backward (bsv)
    if (MODE == CONV_DGRAD && stats && (!bsv || (acc && !bsv->y))) return hipErrorInvalidValue;
    if (inbn && (MODE != CONV_FWD || g.Cs > kFoldMaxC)) return hipErrorInvalidValue;
    if constexpr (MODE == CONV_FWD) {
        if (inbn) {
            if (stats)
                launch((conv_tile_f32<MODE, KS, TM, TN, true, true>), grid, dim3(256), c.lds, st, src, B, bias, Y, g,
                       c.t, acc, sm, ib, bsum);
            else
                launch((conv_tile_f32<MODE, KS, TM, TN, false, true>), grid, dim3(256), c.lds, st, src, B, bias, Y, g,
                       c.t, acc, sm, ib, bsum);
            return hipGetLastError();
        }
    }
    if (stats)
        launch((conv_tile_f32<MODE, KS, TM, TN, true, false>), grid, dim3(256), c.lds, st, src, B, bias, Y, g, c.t,
               acc, sm, ib, bsum);
    else
        launch((conv_tile_f32<MODE, KS, TM, TN, false, false>), grid, dim3(256), c.lds, st, src, B, bias, Y, g, c.t,
               acc, sm, ib, bsum);
    return hipGetLastError();
}

template <int MODE>
static hipError_t dispatch_tile(const float* src, const float* B, const float* bias, float* Y, const ConvGeom& g,
                                const TileCfg& c, int acc, const BnSums* stats, const BnFwd* inbn,
                                const BnBwdSum* bsv, hipStream_t st) {
    if (g.R == 3) {
        if (c.tm == 2) return launch_tile<MODE, 3, 2, 1>(src, B, bias, Y, g, c, acc, stats, inbn, bsv, st);
        return launch_tile<MODE, 3, 1, 1>(src, B, bias, Y, g, c, acc, stats, inbn, bsv, st);
    }
    if (c.tn == 2) return launch_tile<MODE, 1, 2, 2>(src, B, bias, Y, g, c, acc, stats, inbn, bsv, st);
    if (c.tm == 2) return launch_tile<MODE, 1, 2, 1>(src, B, bias, Y, g, c, acc, stats, inbn, bsv, st);
    return launch_tile<MODE, 1, 1, 1>(src, B, bias, Y, g, c, acc, stats, inbn, bsv, st);
}

// Forward pass of a stem (a source of 4 stored channels: the padded image).
// Four consecutive pixels of a row are 16 consecutive floats, so an MFMA group
// of 16 k-values is four taps of a filter row: a KS x KS filter takes
// KS * NSG groups (NSG = ceil(KS / 4); 3x3: 3, 7x7: 14) instead of one per tap
// with three quarters of the channels empty.  Taps past the filter row read a
// zero quad (and meet a zero weight).  The box's input, one quad a pixel, and
// the whole filter slice are staged once; several workgroups to a compute unit
// overlap their phases, so registers are held to what five allow (without the
// bound the compiler hoists every LDS read, two workgroups fit, and the passes
// below take 32 and 82 us).  128 x 32x32, 4 -> 96: 35 us on the gather kernel,
// 22 here; 16 x 224x224, 7x7/2, 4 -> 64: 88, 68.
template <int KS, int TN, bool STATS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5, 8))) void conv_stem_f32(const float* __restrict__ src, const float* __restrict__ B,
                                                     const float* __restrict__ bias, float* __restrict__ Y, ConvGeom g,
                                                     BoxGeom t, int accumulate, BnSums sums) {
    constexpr int TM = 2, BN = TN * 16, NSG = (KS + 3) / 4, LDW = 20;
    constexpr int WR = BN * KS * NSG;                 // LDS rows of the filter slice
    constexpr int NW = (WR * 4 + 255) / 256;
    extern __shared__ float lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int gi = lane >> 4, li = lane & 15;
    const int tr = box_div((int)blockIdx.x, t.nc_inv), tc = (int)blockIdx.x - tr * t.nc;
    const int R0 = tr * t.OH, w0 = tc * t.OW;
    const int ohv = min(t.OH, t.rows - R0), owv = min(t.OW, t.Wo - w0);
    const int n0 = blockIdx.y * BN;
    const int P0 = box_prow(t, R0);
    const int npix = t.IH * t.IW;
    float* Ws = lds;                                  // [WR][LDW]
    float* Xs = lds + WR * LDW;                       // [npix][4], then a zero quad
    const int n1 = t.far ? box_div(P0, t.Hp_inv) : 0;   // the descriptor's first image
    const long image = (long)g.Hs * g.Ws * 4;
    const __amdgpu_buffer_rsrc_t xr = buf_rsrc(src, n1, image, g.Nb);
    const __amdgpu_buffer_rsrc_t wr = buf_rsrc(B, (long)g.Ncols * KS * KS * 4);
    f4 xv[kTileBatches], wv[NW];
#pragma unroll
    for (int u = 0; u < kTileBatches; ++u)
        if (u * 256 < npix) {
            const int pix = tid + u * 256;
            const int ih = box_div(pix, t.IW_inv), iw = pix - ih * t.IW;
            const int pr = P0 + ih;
            const int n = box_div(pr, t.Hp_inv), h = pr - n * t.Hp - t.pad_eff, w = w0 * g.stride + iw - t.pad_eff;
            const bool ok = ih < t.IH && n < g.Nb && h >= 0 && h < g.Hs && w >= 0 && w < g.Ws;
            xv[u] = buf_load4(xr, ok ? (unsigned)(((n - n1) * g.Hs + h) * g.Ws + w) * 16u : kNoLoad, 0);
        }
#pragma unroll
    for (int u = 0; u < NW; ++u) {
        const int e = tid + u * 256, row = e >> 2;    // (channel, filter row, group)
        const int nl = row / (KS * NSG), rg = row - nl * (KS * NSG), r = rg / NSG;
        const int s = (rg - r * NSG) * 4 + (e & 3);
        wv[u] = buf_load4(wr, nl < BN && n0 + nl < g.Ncols && s < KS ? (unsigned)(((n0 + nl) * KS + r) * KS + s) * 16u
                                                                     : kNoLoad, 0);
    }
    int abase[TM];
#pragma unroll
    for (int x = 0; x < TM; ++x) {
        const int p = (wave * TM + x) * 16 + li;
        const int oh = box_div(p, t.OWs_inv), ow = p - oh * t.OWs;
        const bool ok = oh < ohv && ow < owv;
        abase[x] = ((ok ? box_prow(t, R0 + oh) - P0 : 0) * t.IW + (ok ? ow * g.stride : 0) + gi) * 4;
    }
#pragma unroll
    for (int u = 0; u < kTileBatches; ++u)
        if (u * 256 < npix && tid + u * 256 < npix) *(f4*)(Xs + (tid + u * 256) * 4) = xv[u];
    if (tid == 0) *(f4*)(Xs + npix * 4) = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < NW; ++u)
        if (tid + u * 256 < WR * 4) *(f4*)(Ws + ((tid + u * 256) >> 2) * LDW + (tid & 3) * 4) = wv[u];
    f4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
    __syncthreads();
#pragma unroll
    for (int r = KS - 1; r >= 0; --r)
#pragma unroll
        for (int sg = 0; sg < NSG; ++sg) {
            // lanes whose tap 4 sg + gi lies past the filter row
            const bool past = sg == NSG - 1 && (sg * 4 + gi) >= KS;
            f4 a[TM], b[TN];
#pragma unroll
            for (int x = 0; x < TM; ++x) a[x] = *(const f4*)(Xs + (past ? npix * 4 : abase[x] + (r * t.IW + sg * 4) * 4));
#pragma unroll
            for (int y = 0; y < TN; ++y)
                b[y] = *(const f4*)(Ws + (((y * 16 + li) * KS + r) * NSG + sg) * LDW + gi * 4);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int x = 0; x < TM; ++x)
#pragma unroll
                    for (int y = 0; y < TN; ++y) acc[x][y] = mfma16x16x4(a[x][j], b[y][j], acc[x][y]);
        }
    __syncthreads();
    box_store<CONV_FWD, TM, TN, STATS>(acc, lds, bias, Y, g, t, accumulate, sums, BnBwdSum{}, R0, w0, ohv, owv, n0);
}

// Box of a stem's forward pass (128 slots; 32 output channels, 16 where there
// are no more), or false when the kernel does not take it.
struct StemCfg { int tn, tiles; BoxGeom t; size_t lds; };
static bool pick_stem(const ConvGeom& g, StemCfg& c) {
    if (g.Cs != 4 || g.Ncols % 4 || g.R != g.S || (g.R != 3 && g.R != 7)) return false;
    // (box_pick counts batches of 64 pixels with a quad group each; here a batch is 256 pixels)
    if (!box_pick(c.t, g.Nb, g.Ho, g.Wo, g.R, g.stride, g.pad, 128, 1, 4 * kTileBatches) ||
        !box_fits(c.t, g.Nb, (double)g.Hs * g.Ws * 4))
        return false;
    c.tn = g.Ncols > 16 ? 2 : 1;
    c.tiles = box_tiles(c.t);
    c.lds = sizeof(float) * std::max<size_t>((size_t)c.tn * 16 * g.R * ((g.R + 3) / 4) * 20 +
                                                 ((size_t)c.t.IH * c.t.IW + 1) * 4,
                                             (size_t)4 * 32 * (c.tn * 16 + 4));
    return true;
}

template <int KS, int TN>
static hipError_t launch_stem(const float* src, const float* B, const float* bias, float* Y, const ConvGeom& g,
                              const StemCfg& c, int acc, const BnSums* stats, hipStream_t st) {
    dim3 grid((unsigned)c.tiles, (unsigned)((g.Ncols + TN * 16 - 1) / (TN * 16)));
    const BnSums sm = stats ? *stats : BnSums{};
    if (stats) launch((conv_stem_f32<KS, TN, true>), grid, dim3(256), c.lds, st, src, B, bias, Y, g, c.t, acc, sm);
    else launch((conv_stem_f32<KS, TN, false>), grid, dim3(256), c.lds, st, src, B, bias, Y, g, c.t, acc, sm);
    return hipGetLastError();
}

static hipError_t dispatch_stem(const float* src, const float* B, const float* bias, float* Y, const ConvGeom& g,
                                const StemCfg& c, int acc, const BnSums* stats, hipStream_t st) {
    if (g.R == 3) {
        if (c.tn == 2) return launch_stem<3, 2>(src, B, bias, Y, g, c, acc, stats, st);
        return launch_stem<3, 1>(src, B, bias, Y, g, c, acc, stats, st);
    }
    if (c.tn == 2) return launch_stem<7, 2>(src, B, bias, Y, g, c, acc, stats, st);
    return launch_stem<7, 1>(src, B, bias, Y, g, c, acc, stats, st);
}

// Data gradient of a stride-2 conv, split by output parity.  dX pixel
// (2i + a, 2j + b) only receives taps (r, s) with a + pad - r and b + pad - s
// even, from dY[i + (a + pad - r)/2][j + (b + pad - s)/2]: per parity class
// (a, b) this is a dense stride-1 correlation over dY with a subset of the
// taps (3x3, pad 1: 1, 2, 2 and 4 taps; 1x1, pad 0: one tap, class (0, 0)).
// A workgroup takes a box of class pixels (i, j) for all four classes, so
// every workgroup runs all taps once, the dY rows it reads are staged in LDS
// once per 16 dY channels, and no MFMA is spent on taps that fall between
// strides; odd grids leave out the last class row or column at the store.
// (The GEMM kernel that odd and non-power-of-two grids ran on spends four
// MFMAs where one counts: 16 x 28x28x128 -> 56x56x64 took 127 us, 100 x
// 14x14x32 -> 28x28x16 42 us.)
template <int KS, int PAD, int TM>
__global__ __launch_bounds__(256) void conv_dgrad_s2_f32(const float* __restrict__ dY, const float* __restrict__ B,
                                                         float* __restrict__ dX, ConvGeom g, BoxGeom t,
                                                         int accumulate) {
    constexpr int TP = TM * 64, LDW = 20, RS = KS * KS;
    constexpr int NW = (16 * RS * 4 + 255) / 256;
    extern __shared__ float lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int gi = lane >> 4, li = lane & 15, q = tid & 3;
    const int tr = box_div((int)blockIdx.x, t.nc_inv), tc = (int)blockIdx.x - tr * t.nc;
    const int R0 = tr * t.OH, w0 = tc * t.OW;
    const int ohv = min(t.OH, t.rows - R0), owv = min(t.OW, t.Wo - w0);
    const int n0 = blockIdx.y * 16;
    const int P0 = box_prow(t, R0);
    const int nx = t.IH * t.IW * 4, nxu = (nx + 255) >> 8;
    float* Xs = lds;                              // [IH * IW][LDW] dY rows
    float* Ws = lds + t.IH * t.IW * LDW;          // [16][RS][LDW]

    const int n1 = t.far ? box_div(P0, t.Hp_inv) : 0;   // the descriptor's first image
    const long image = (long)g.Hs * g.Ws * g.Cs;
    const __amdgpu_buffer_rsrc_t xr = buf_rsrc(dY, n1, image, g.Nb);
    const __amdgpu_buffer_rsrc_t wr = buf_rsrc(B, (long)g.Ncols * RS * g.Cs);
    unsigned xo[kTileBatches], wo[NW];
#pragma unroll
    for (int u = 0; u < kTileBatches; ++u) {
        xo[u] = kNoLoad;
        if (u < nxu) {
            const int pix = (tid + u * 256) >> 2;
            const int ih = box_div(pix, t.IW_inv), iw = pix - ih * t.IW;
            const int pr = P0 + ih;
            const int n = box_div(pr, t.Hp_inv), h = pr - n * t.Hp, w = w0 + iw;
            if (ih < t.IH && n < g.Nb && h < g.Hs && w < g.Ws)
                xo[u] = (unsigned)((((n - n1) * g.Hs + h) * g.Ws + w) * g.Cs + q * 4) * 4u;
        }
    }
#pragma unroll
    for (int u = 0; u < NW; ++u) {
        const int rest = (tid + u * 256) >> 2;    // (channel, tap)
        wo[u] = (rest < 16 * RS && n0 + rest / RS < g.Ncols) ? (unsigned)((n0 * RS + rest) * g.Cs + q * 4) * 4u
                                                            : kNoLoad;
    }
    f4 xv[kTileBatches], wv[NW];
    auto load = [&](int c0) {
        const unsigned bad = c0 + q * 4 < g.Cs ? 0u : kNoLoad;
#pragma unroll
        for (int u = 0; u < kTileBatches; ++u)
            if (u < nxu) xv[u] = buf_load4(xr, xo[u] | bad, c0 * 4);
#pragma unroll
        for (int u = 0; u < NW; ++u) wv[u] = buf_load4(wr, wo[u] | bad, c0 * 4);
    };
    load(0);
    int abase[TM];
#pragma unroll
    for (int x = 0; x < TM; ++x) {
        const int p = (wave * TM + x) * 16 + li;
        const int oh = box_div(p, t.OWs_inv), ow = p - oh * t.OWs;
        const bool ok = oh < ohv && ow < owv;
        abase[x] = ((ok ? box_prow(t, R0 + oh) - P0 : 0) * t.IW + (ok ? ow : 0)) * LDW + gi * 4;
    }
    f4 acc[4][TM];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int i = 0; i < TM; ++i) acc[c][i] = f4{0.f, 0.f, 0.f, 0.f};

    const int sdst = (tid >> 2) * LDW + q * 4;
    for (int c0 = 0; c0 < g.Cs; c0 += 16) {
#pragma unroll
        for (int u = 0; u < kTileBatches; ++u)
            if (u < nxu && tid + u * 256 < nx) *(f4*)(Xs + sdst + u * 64 * LDW) = xv[u];
#pragma unroll
        for (int u = 0; u < NW; ++u)
            if (tid + u * 256 < 16 * RS * 4) *(f4*)(Ws + sdst + u * 64 * LDW) = wv[u];
        lds_barrier();
        if (c0 + 16 < g.Cs) load(c0 + 16);
#pragma unroll
        for (int cls = 0; cls < 4; ++cls) {
            const int ca = cls >> 1, cb = cls & 1;
#pragma unroll
            for (int r = 0; r < KS; ++r)
#pragma unroll
                for (int sx = 0; sx < KS; ++sx) {
                    if (((ca + PAD - r) & 1) || ((cb + PAD - sx) & 1)) continue;
                    // source row i + (a + pad - r)/2, column j + (b + pad - s)/2
                    const int toff = ((ca + PAD - r) / 2 * t.IW + (cb + PAD - sx) / 2) * LDW;
                    const f4 bv = *(const f4*)(Ws + (li * RS + r * KS + sx) * LDW + gi * 4);
                    f4 av[TM];
#pragma unroll
                    for (int x = 0; x < TM; ++x) av[x] = *(const f4*)(Xs + abase[x] + toff);
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int x = 0; x < TM; ++x) acc[cls][x] = mfma16x16x4(av[x][j], bv[j], acc[cls][x]);
                }
        }
        lds_barrier();
    }

    // the four classes' pixels in LDS, then stored as float4 channel quads in
    // the order of dX's columns
    constexpr int OP = 20;
#pragma unroll
    for (int cls = 0; cls < 4; ++cls)
#pragma unroll
        for (int x = 0; x < TM; ++x)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                lds[(cls * TP + (wave * TM + x) * 16 + gi * 4 + i) * OP + li] = acc[cls][x][i];
    __syncthreads();
    const int n = n0 + q * 4;
    if (n >= g.Ncols) return;
#pragma unroll 4
    for (int e = tid >> 2; e < 4 * TP; e += 64) {
        const int b = e & 1, p = (e >> 1) & (TP - 1), a = e / (2 * TP);
        const int oh = box_div(p, t.OWs_inv), ow = p - oh * t.OWs;
        if (oh >= ohv || ow >= owv) continue;
        const int im = box_div(R0 + oh, t.Hper_inv);
        const int hr = 2 * (R0 + oh - im * t.Hper) + a, wc = 2 * (w0 + ow) + b;
        if (hr >= g.Ho || wc >= g.Wo) continue;
        const f4 v = *(const f4*)(lds + ((2 * a + b) * TP + p) * OP + q * 4);
        f4* o = (f4*)(dX + ((long)(im * g.Ho + hr) * g.Wo + wc) * g.Ncols + n);
        *o = accumulate == kStoreAdd ? *o + v : (accumulate == kStoreRelu ? relu4(v) : v);
    }
}

// Box of the parity-split stride-2 data gradient, or false when it does not
// apply.
struct S2Cfg { int tm, tiles; BoxGeom t; size_t lds; };
static bool pick_s2(const ConvGeom& g, S2Cfg& out) {
    if (g.stride != 2 || g.Cs % 4 || g.Ncols % 4) return false;
    if (!((g.R == 3 && g.S == 3 && g.pad == 1) || (g.R == 1 && g.S == 1 && g.pad == 0))) return false;
    if (!buf_fits((double)g.Ncols * g.R * g.R * g.Cs)) return false;
    const int ext = g.R == 3 ? 2 : 1;   // dY rows i, i + 1 (3x3) or i
    bool found = false;
    for (int tm : {2, 1}) {
        S2Cfg c;
        if (!box_pick(c.t, g.Nb, (g.Ho + 1) / 2, (g.Wo + 1) / 2, ext, 1, 0, tm * 64, 1, kTileBatches) ||
            !box_fits(c.t, g.Nb, (double)g.Hs * g.Ws * g.Cs))
            continue;
        c.tm = tm;
        c.tiles = box_tiles(c.t);
        c.lds = sizeof(float) * std::max<size_t>(20 * ((size_t)c.t.IH * c.t.IW + (size_t)16 * g.R * g.R),
                                                 (size_t)4 * tm * 64 * 20);
        found = true;
        out = c;
        if ((long)c.tiles * ((g.Ncols + 15) / 16) >= 512) break;
    }
    return found;
}

static hipError_t dispatch_s2(const float* dY, const float* B, float* dX, const ConvGeom& g, const S2Cfg& c, int acc,
                              hipStream_t st) {
    dim3 grid((unsigned)c.tiles, (unsigned)((g.Ncols + 15) / 16));
    if (g.R == 3 && c.tm == 2)
        launch((conv_dgrad_s2_f32<3, 1, 2>), grid, dim3(256), c.lds, st, dY, B, dX, g, c.t, acc);
    else if (g.R == 3)
        launch((conv_dgrad_s2_f32<3, 1, 1>), grid, dim3(256), c.lds, st, dY, B, dX, g, c.t, acc);
    else if (c.tm == 2)
        launch((conv_dgrad_s2_f32<1, 0, 2>), grid, dim3(256), c.lds, st, dY, B, dX, g, c.t, acc);
    else
        launch((conv_dgrad_s2_f32<1, 0, 1>), grid, dim3(256), c.lds, st, dY, B, dX, g, c.t, acc);
    return hipGetLastError();
}

template <int MODE, int WM, int TM, int TN>
static hipError_t launch_cfg(const float* src, const float* B, const float* bias, float* Y, const ConvGeom& g,
                             int acc, const BnSums* stats, hipStream_t st) {
    constexpr int BM = WM * TM * 16, BN = (4 / WM) * TN * 16;
    const long M = (long)g.Nb * g.Ho * g.Wo;
    dim3 grid((unsigned)((M + BM - 1) / BM), (unsigned)((g.Ncols + BN - 1) / BN));
    const bool fast = g.Cs % 16 == 0;
    if (stats) {
        if (fast)
            launch((conv_igemm_f32<MODE, WM, TM, TN, true, true>), grid, dim3(256), 0, st, src, B, bias,
                               Y, g, (int)acc, stats ? *stats : BnSums{});
        else
            launch((conv_igemm_f32<MODE, WM, TM, TN, false, true>), grid, dim3(256), 0, st, src, B, bias,
                               Y, g, (int)acc, stats ? *stats : BnSums{});
    } else {
        if (fast)
            launch((conv_igemm_f32<MODE, WM, TM, TN, true, false>), grid, dim3(256), 0, st, src, B, bias,
                               Y, g, (int)acc, stats ? *stats : BnSums{});
        else
            launch((conv_igemm_f32<MODE, WM, TM, TN, false, false>), grid, dim3(256), 0, st, src, B, bias,
                               Y, g, (int)acc, stats ? *stats : BnSums{});
    }
    return hipGetLastError();
}

// Tile configuration.  Cs % 16 == 0 uses the LDS kernel with (BM, BN, WM)
// by output width and rows; other passes (the padded image) the direct one.
struct ConvCfg { int lds, bm, bn, wm, tm, tn; };
static ConvCfg pick_cfg(const ConvGeom& g) {
    const long M = (long)g.Nb * g.Ho * g.Wo;
    if (g.Cs % 16 == 0) {
        if (g.Ncols <= 16) return {1, M >= 256L * 256 ? 256 : 64, 16, 4, 0, 0};
        if (g.Ncols <= 32) return {1, M >= 128L * 256 ? 128 : 64, 32, M >= 128L * 256 ? 4 : 2, 0, 0};
        if (g.Ncols <= 64) return {1, M >= 64L * 256 ? 64 : 32, 64, M >= 64L * 256 ? 2 : 1, 0, 0};
        return {1, 64, 128, 2, 0, 0};
    }
    if (g.Ncols <= 16) return {0, 128, 16, 4, 2, 1};
    if (g.Ncols <= 32) return {0, 128, 32, 4, 2, 2};
    if (g.Ncols <= 64 || M < 64L * 512) {
        if (M >= 64L * 512) return {0, 64, 64, 2, 2, 2};
        return {0, 32, 64, 2, 1, 2};
    }
    return {0, 64, 128, 2, 2, 4};
}

template <int MODE>
static hipError_t launch_mode(const float* src, const float* B, const float* bias, float* Y, const ConvGeom& g,
                              int acc, const BnSums* stats, const BnFwd* inbn, const BnBwdSum* bsv, hipStream_t st) {
    TileCfg tc;
    if (pick_tile(MODE, g, tc)) return dispatch_tile<MODE>(src, B, bias, Y, g, tc, acc, stats, inbn, bsv, st);
    if (inbn || bsv) return hipErrorInvalidValue;   // folding and backward sums need the spatial kernel
    if (MODE == CONV_FWD) {
        StemCfg sc;
        if (pick_stem(g, sc)) return dispatch_stem(src, B, bias, Y, g, sc, acc, stats, st);
    }
    if (MODE == CONV_DGRAD) {
        S2Cfg sc;
        if (pick_s2(g, sc)) return dispatch_s2(src, B, Y, g, sc, acc, st);
    }
    ConvCfg c = pick_cfg(g);
    if (c.lds) {
        if (c.bn == 16) {
            if (c.bm == 256) return launch_lds<MODE, 256, 16, 4>(src, B, bias, Y, g, acc, stats, st);
            return launch_lds<MODE, 64, 16, 4>(src, B, bias, Y, g, acc, stats, st);
        }
        if (c.bn == 32) {
            if (c.bm == 128) return launch_lds<MODE, 128, 32, 4>(src, B, bias, Y, g, acc, stats, st);
            return launch_lds<MODE, 64, 32, 2>(src, B, bias, Y, g, acc, stats, st);
        }
        if (c.bn == 64) {
            if (c.bm == 64) return launch_lds<MODE, 64, 64, 2>(src, B, bias, Y, g, acc, stats, st);
            return launch_lds<MODE, 32, 64, 1>(src, B, bias, Y, g, acc, stats, st);
        }
        return launch_lds<MODE, 64, 128, 2>(src, B, bias, Y, g, acc, stats, st);
    }
    if (c.wm == 4 && c.tn == 1) return launch_cfg<MODE, 4, 2, 1>(src, B, bias, Y, g, acc, stats, st);
    if (c.wm == 4) return launch_cfg<MODE, 4, 2, 2>(src, B, bias, Y, g, acc, stats, st);
    if (c.tn == 4) return launch_cfg<MODE, 2, 2, 4>(src, B, bias, Y, g, acc, stats, st);
    if (c.tm == 2) return launch_cfg<MODE, 2, 2, 2>(src, B, bias, Y, g, acc, stats, st);
    return launch_cfg<MODE, 2, 1, 2>(src, B, bias, Y, g, acc, stats, st);
}

TileCounts conv_tile_counts(const ConvGeom& g) {
    TileCfg c;
    if (pick_tile(CONV_FWD, g, c)) return TileCounts{c.tiles, c.t.OH, c.t.OW, c.t.nc, c.t.rows, c.t.Wo};
    StemCfg sc;
    if (pick_stem(g, sc)) return TileCounts{sc.tiles, sc.t.OH, sc.t.OW, sc.t.nc, sc.t.rows, sc.t.Wo};
    return tile_counts_rows((long)g.Nb * g.Ho * g.Wo, pick_cfg(g).bm);
}

hipError_t launch_conv_igemm(int mode, const float* src, const float* B, const float* bias, float* Y,
                             const ConvGeom& g, int accumulate, const BnSums* stats, hipStream_t st,
                             const BnFwd* inbn, const BnBwdSum* bsum) {
    if (mode == CONV_FWD) {
        if (bsum) return hipErrorInvalidValue;
        return launch_mode<CONV_FWD>(src, B, bias, Y, g, accumulate, stats, inbn, nullptr, st);
    }
    if (inbn || (bsum != nullptr) != (stats != nullptr)) return hipErrorInvalidValue;
    return launch_mode<CONV_DGRAD>(src, B, bias, Y, g, accumulate, stats, nullptr, bsum, st);
}

int conv_dgrad_sum_tiles(const ConvGeom& gd) {
    TileCfg tc;
    return pick_tile(CONV_DGRAD, gd, tc) ? tc.tiles : 0;
}

bool conv_fold_ok(const ConvGeom& g, const WgradPlan& p) {
    TileCfg tc;
    return g.Cs <= kFoldMaxC && p.tile == 1 && pick_tile(CONV_FWD, g, tc);
}

// ------------------------------------------------------------------------
// weight gradient
// ------------------------------------------------------------------------

struct WgArgs {
    int Nb, Hi, Wi, Cin_p, Ho, Wo, Cout, R, S, stride, pad, pix_per_split;
};

template <int TM, int TN>
__global__ __launch_bounds__(256) void conv_wgrad_f32(const float* __restrict__ dY, const float* __restrict__ X,
                                                      float* __restrict__ part, WgArgs a) {
    constexpr int BMw = TM * 16, BNw = TN * 16;
    constexpr int NA = 64 * (BMw / 4) / 256;   // dY quads per thread per chunk
    constexpr int NB = 64 * (BNw / 4) / 256;   // im2col quads per thread per chunk
    __shared__ float As[64][BMw + 4];
    __shared__ float Bs[64][BNw + 4];
    __shared__ float red[TM * TN * 4][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int gi = lane >> 4, li = lane & 15;
    const int HoWo = a.Ho * a.Wo;
    const int M = a.Nb * HoWo;
    const int Ktot = a.R * a.S * a.Cin_p;
    const int Cq = a.Cin_p >> 2;
    const int m0 = blockIdx.x * BMw, n0 = blockIdx.y * BNw;
    const int p_begin = blockIdx.z * a.pix_per_split;
    const int p_end = min(M, p_begin + a.pix_per_split);

    // each thread's column quad is the same in every chunk: decode it once
    const int bcq = tid % (BNw / 4);
    const int col = n0 + bcq * 4;
    const bool col_ok = col < Ktot;
    int br = 0, bs = 0, bc = 0;
    if (col_ok) {
        const int quad = col >> 2;
        const int tap = quad / Cq;
        bc = (quad - tap * Cq) * 4;
        br = tap / a.S;
        bs = tap - br * a.S;
    }
    const int acq = tid % (BMw / 4);
    const int aco = m0 + acq * 4;

    f4 ra[NA], rb[NB];
    auto load = [&](int pc) {
#pragma unroll
        for (int k = 0; k < NA; ++k) {
            const int px = (tid + 256 * k) / (BMw / 4);
            const int p = pc + px;
            ra[k] = (p < p_end && aco < a.Cout) ? *(const f4*)(dY + (long)p * a.Cout + aco) : f4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            const int px = (tid + 256 * k) / (BNw / 4);
            const int p = pc + px;
            f4 v = f4{0.f, 0.f, 0.f, 0.f};
            if (p < p_end && col_ok) {
                const int n = p / HoWo;
                const int rem = p - n * HoWo;
                const int ho = rem / a.Wo, wo = rem - ho * a.Wo;
                const int hi = ho * a.stride - a.pad + br, wi = wo * a.stride - a.pad + bs;
                if (hi >= 0 && hi < a.Hi && wi >= 0 && wi < a.Wi)
                    v = *(const f4*)(X + ((long)(n * a.Hi + hi) * a.Wi + wi) * a.Cin_p + bc);
            }
            rb[k] = v;
        }
    };

    f4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};

    if (p_begin < p_end) load(p_begin);
    for (int pc = p_begin; pc < p_end; pc += 64) {
#pragma unroll
        for (int k = 0; k < NA; ++k) *(f4*)&As[(tid + 256 * k) / (BMw / 4)][acq * 4] = ra[k];
#pragma unroll
        for (int k = 0; k < NB; ++k) *(f4*)&Bs[(tid + 256 * k) / (BNw / 4)][bcq * 4] = rb[k];
        __syncthreads();
        if (pc + 64 < p_end) load(pc + 64);   // next chunk in flight during this one's MFMAs
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int row = 16 * wave + 4 * j + gi;
            float av[TM], bv[TN];
#pragma unroll
            for (int t = 0; t < TM; ++t) av[t] = As[row][t * 16 + li];
#pragma unroll
            for (int t = 0; t < TN; ++t) bv[t] = Bs[row][t * 16 + li];
#pragma unroll
            for (int x = 0; x < TM; ++x)
#pragma unroll
                for (int y = 0; y < TN; ++y) acc[x][y] = mfma16x16x4(av[x], bv[y], acc[x][y]);
        }
        __syncthreads();
    }

    // waves 0..3 summed in order through LDS
    for (int w = 0; w < 4; ++w) {
        if (wave == w) {
#pragma unroll
            for (int x = 0; x < TM; ++x)
#pragma unroll
                for (int y = 0; y < TN; ++y)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        float* slot = &red[(x * TN + y) * 4 + i][lane];
                        *slot = (w == 0) ? acc[x][y][i] : *slot + acc[x][y][i];
                    }
        }
        __syncthreads();
    }
    if (wave == 3) {
        float* out = part + (long)blockIdx.z * a.Cout * Ktot;
#pragma unroll
        for (int x = 0; x < TM; ++x)
#pragma unroll
            for (int y = 0; y < TN; ++y) {
                const int cc = n0 + y * 16 + li;
                if (cc >= Ktot) continue;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int co = m0 + x * 16 + gi * 4 + i;
                    if (co < a.Cout) out[(long)co * Ktot + cc] = red[(x * TN + y) * 4 + i][lane];
                }
            }
    }
}

// Spatially tiled weight gradient: a workgroup takes a run of boxes of NG * 64
// pixel slots (BoxGeom; 16 output and 16 input channels) and produces the
// partial
//     dW[co][r][s][c] = sum over its boxes' pixels p of dY[p][co] * X[src(p, r, s)][c]
// for every tap.  A box's input rows (halo and padding included; for a 1x1
// conv just the pixels it reads) and its dY go into LDS once, the next box's
// loads in flight during this one's MFMAs; each wave takes NG groups of 16
// slots, keeps their dY values in registers and runs all taps over them.  The
// reduction dimension k of v_mfma_f32_16x16x4_f32 is the pixel: lane (li, gi)
// supplies dY[p][co0 + li] and X[src(p)][c0 + li] for the same four slots
// p = 16 g + 4 gi + j, consecutive in one box row (OWs % 4 == 0); slots
// without a pixel (none where FULL) hold dY = 0.  Waves are summed in a fixed
// order and every workgroup writes its own partial, summed in order by the
// reduce kernel.  What a slot without a pixel reads of X belongs to other
// outputs, and zero times an infinity there is NaN: a workgroup that finds a
// NaN among its sums forms them once more with zeros for both operands (zeros
// chosen at every MFMA cost up to 9% of a step, the look for a NaN 2% of the
// kernel).
// Bound by the staging's latency at ResNet-20's sizes (one box per workgroup)
// and by the MFMAs where several boxes pipeline.  Held to 168 registers, three
// workgroups to a compute unit (with two, 16 x 56x56x64 takes 54 us instead of
// 45, ResNet-20's stages 11.2 instead of 10.8).
// An accumulator takes at most 64 MFMAs in a row (wg_run); then the
// workgroup's sums go to fp64 and it starts again, so the error does not grow
// with the boxes of a workgroup.
constexpr int kWgBatches = 6;   // staged input quads per thread and box, at most
// Boxes between two such moments: 16 MFMAs where rows are a power of two long,
// else 64.  Root mean square error, relative, of 64 x 32x32, 128 -> 128
// channels (43 boxes): 6.6e-8, in one chain 2.2e-7, with a partial for every 16
// MFMAs 6.9e-8; of 100 x 28x28x64: 1.5e-7, in one chain 2.0e-7, the GEMM kernel
// (88 in a row) 1.8e-7.  The time follows: 16 x 56x56x64 takes 48.0 us in one
// chain, 51.6 with 16, 49.8 with 64; 87 x 38x38x44 65.8 and, with 64, 69.6.
static int wg_run(int ng, int Wo) { return std::max(1, ((Wo & (Wo - 1)) == 0 ? 16 : 64) / (4 * ng)); }

template <int RS, int NG, int ST, bool FULL, bool FAR>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 8)))
void conv_wgrad_tile_f32(const float* __restrict__ dY, const float* __restrict__ X, float* __restrict__ part, WgArgs a,
                         BoxGeom t, int tiles, int per, int run, const float* __restrict__ in_ss) {
    constexpr bool K1 = RS == 1;
    constexpr int LDW = 20;
    constexpr int JST = (K1 ? 1 : ST) * LDW;   // LDS distance between a lane's four pixels
    extern __shared__ float lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int gi = lane >> 4, li = lane & 15, q = tid & 3;
    const int co0 = blockIdx.y * 16, c0 = blockIdx.z * 16;
    const int Ktot = RS * a.Cin_p;
    const int npix = t.IH * t.IW, nx = npix * 4, nxu = (nx + 255) >> 8;
    float* Xs = lds;                         // [npix][LDW] input rows of the box
    float* Ds = lds + npix * LDW;            // [TP][LDW] dY of the box, 16 channels
    const long image = (long)a.Hi * a.Wi * a.Cin_p, row = (long)a.Wo * a.Cout;

    // the fold's scale and shift of this thread's channel quad
    f4 fsc{}, fsh{};
    if (in_ss && c0 + q * 4 < a.Cin_p) {
        fsc = *(const f4*)(in_ss + c0 + q * 4);
        fsh = *(const f4*)(in_ss + a.Cin_p + c0 + q * 4);
    }
    f4 xv[kWgBatches], dv[NG];
    unsigned valid = 0;                      // batches whose quad lies inside X
    auto load = [&](int tile) {
        const int tr = box_div(tile, t.nc_inv), tc = tile - tr * t.nc;
        const int R0 = tr * t.OH, w0 = tc * t.OW, P0 = box_prow(t, R0);
        const int ohv = min(t.OH, t.rows - R0), owv = min(t.OW, t.Wo - w0);
        const int n1 = FAR ? box_div(P0, t.Hp_inv) : 0, R1 = FAR ? R0 : 0;   // the descriptors' first image and row
        const __amdgpu_buffer_rsrc_t xr = buf_rsrc(X, n1, image, a.Nb), dr = buf_rsrc(dY, R1, row, t.rows);
        valid = 0;
#pragma unroll
        for (int u = 0; u < kWgBatches; ++u)
            if (u < nxu) {
                const int pix = (tid + u * 256) >> 2;
                const int ih = box_div(pix, t.IW_inv), iw = pix - ih * t.IW;
                const int pr = P0 + ih;
                const int n = box_div(pr, t.Hp_inv), hh = pr - n * t.Hp;
                const int h = (K1 ? hh * ST : hh) - t.pad_eff;
                const int w = (K1 ? (w0 + iw) * ST : w0 * ST + iw) - t.pad_eff;
                unsigned off = kNoLoad;
                if (ih < t.IH && n < a.Nb && h >= 0 && h < a.Hi && w >= 0 && w < a.Wi && c0 + q * 4 < a.Cin_p) {
                    off = (unsigned)((((n - n1) * a.Hi + h) * a.Wi + w) * a.Cin_p + c0 + q * 4) * 4u;
                    valid |= 1u << u;
                }
                xv[u] = buf_load4(xr, off, 0);
            }
#pragma unroll
        for (int u = 0; u < NG; ++u) {
            const int p = (tid + u * 256) >> 2;
            const int oh = box_div(p, t.OWs_inv), ow = p - oh * t.OWs;
            const bool ok = oh < ohv && ow < owv && co0 + q * 4 < a.Cout;
            dv[u] = buf_load4(dr, ok ? (unsigned)(((R0 - R1 + oh) * t.Wo + w0 + ow) * a.Cout + co0 + q * 4) * 4u : kNoLoad,
                              0);
        }
    };

    int toff[RS];
#pragma unroll
    for (int k = 0; k < RS; ++k) toff[k] = K1 ? 0 : ((k / 3) * t.IW + k % 3) * LDW;
    f4 acc[RS];
    const int t0 = blockIdx.x * per, t1 = min(tiles, t0 + per);
    const int sdst = (tid >> 2) * LDW + q * 4;
    // each wave's RS x 16 x 16 block into its own LDS slice, then the four
    // slices summed in order
    float* red = lds;   // [4][RS][16 co][16 c], then for each wave whether it met a NaN
    float all = 0.f;    // a NaN once one was among the sums
    auto waves = [&]() {
#pragma unroll
        for (int k = 0; k < RS; ++k)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                red[((wave * RS + k) * 16 + gi * 4 + i) * 16 + li] = acc[k][i];
                if (!FULL) all += acc[k][i];
            }
        if (!FULL) {
            const bool nan = __any(all != all);
            if (lane == 0) red[4 * RS * 256 + wave] = nan ? 1.f : 0.f;
        }
        lds_barrier();
    };
    auto wave_sum = [&](int k) {
        const int e = k * 256 + tid;
        return ((red[e] + red[RS * 256 + e]) + red[2 * RS * 256 + e]) + red[3 * RS * 256 + e];
    };
    // runs of `run` boxes leave their sums in fp64: entry tid of every tap in
    // thread tid, or (1x1) each lane its own four
    double tot[K1 ? 4 : RS];
    const bool chained = NG < 4 && t1 - t0 > run;
    auto leave = [&]() {
        if constexpr (K1) {
#pragma unroll
            for (int i = 0; i < 4; ++i) tot[i] += (double)acc[0][i];
            acc[0] = f4{0.f, 0.f, 0.f, 0.f};
        } else {
            waves();
#pragma unroll
            for (int k = 0; k < RS; ++k) {
                tot[k] += (double)wave_sum(k);
                acc[k] = f4{0.f, 0.f, 0.f, 0.f};
            }
            lds_barrier();
        }
    };
    auto finish = [&]() {
        if (K1 && chained) {
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[0][i] = (float)(tot[i] + (double)acc[0][i]);
        }
        waves();
        float* out = part + (long)blockIdx.x * a.Cout * Ktot;
        const int co = co0 + (tid >> 4), c = c0 + (tid & 15);
#pragma unroll
        for (int k = 0; k < RS; ++k) {
            float v = wave_sum(k);
            if (!K1 && chained) v = (float)(tot[k] + (double)v);
            if (co < a.Cout && c < a.Cin_p) out[(long)co * Ktot + k * a.Cin_p + c] = v;
        }
    };
#pragma unroll
    for (int k = 0; k < RS; ++k) acc[k] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (double& v : tot) v = 0.0;
    load(t0);
    for (int tile = t0; tile < t1; ++tile) {
        if (in_ss) {
            // X read through a folded BN + ReLU (padding stays zero)
#pragma unroll
            for (int u = 0; u < kWgBatches; ++u)
                if (u < nxu) {
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        xv[u][k] = (valid >> u) & 1 ? fmaxf(__builtin_fmaf(xv[u][k], fsc[k], fsh[k]), 0.f) : 0.f;
                }
        }
#pragma unroll
        for (int u = 0; u < kWgBatches; ++u)
            if (u < nxu && tid + u * 256 < nx) *(f4*)(Xs + sdst + u * 64 * LDW) = xv[u];
#pragma unroll
        for (int u = 0; u < NG; ++u) *(f4*)(Ds + sdst + u * 64 * LDW) = dv[u];
        // the first of each group's four consecutive slots (rows past the
        // box's, whose dY is zero, read the first)
        int boff[NG];
        {
            const int tr = box_div(tile, t.nc_inv), R0 = tr * t.OH, P0 = box_prow(t, R0);
            const int ohv = min(t.OH, t.rows - R0);
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                const int p = (wave * NG + g) * 16 + gi * 4;
                const int oh = box_div(p, t.OWs_inv), ow = p - oh * t.OWs;
                const bool ok = oh < ohv;
                boff[g] = ((ok ? box_prow(t, R0 + oh) - P0 : 0) * t.IW + (ok ? ow * (K1 ? 1 : ST) : 0)) * LDW + li;
            }
        }
        lds_barrier();
        if (tile + 1 < t1) load(tile + 1);
        // per group: the four dY values and all RS x 4 X operands are read
        // before its MFMAs, the next group's reads are issued before this
        // group's MFMAs
        float bv[2][RS][4];
        f4 av[2];
#pragma unroll
        for (int j = 0; j < 4; ++j) av[0][j] = Ds[(wave * NG * 16 + gi * 4 + j) * LDW + li];
#pragma unroll
        for (int k = 0; k < RS; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) bv[0][k][j] = Xs[boff[0] + toff[k] + j * JST];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            if (g + 1 < NG) {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    av[(g + 1) & 1][j] = Ds[(((wave * NG + g + 1) * 16) + gi * 4 + j) * LDW + li];
#pragma unroll
                for (int k = 0; k < RS; ++k)
#pragma unroll
                    for (int j = 0; j < 4; ++j) bv[(g + 1) & 1][k][j] = Xs[boff[g + 1] + toff[k] + j * JST];
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int k = 0; k < RS; ++k) acc[k] = mfma16x16x4(av[g & 1][j], bv[g & 1][k][j], acc[k]);
        }
        lds_barrier();   // the staged box is dead
        if (chained && (tile + 1 - t0) % run == 0 && tile + 1 < t1) leave();
    }

    finish();
    if (FULL) return;
    const f4 nan = *(const f4*)(red + 4 * RS * 256);
    if (nan[0] + nan[1] + nan[2] + nan[3] == 0.f) return;
    __syncthreads();
    // the same sums in the same order, zeros for both operands at slots without a pixel
#pragma unroll
    for (int k = 0; k < RS; ++k) acc[k] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (double& v : tot) v = 0.0;
#pragma unroll 1
    for (int tile = t0; tile < t1; ++tile) {
        load(tile);
        if (in_ss) {
            // X read through a folded BN + ReLU (padding stays zero)
#pragma unroll
            for (int u = 0; u < kWgBatches; ++u)
                if (u < nxu) {
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        xv[u][k] = (valid >> u) & 1 ? fmaxf(__builtin_fmaf(xv[u][k], fsc[k], fsh[k]), 0.f) : 0.f;
                }
        }
#pragma unroll
        for (int u = 0; u < kWgBatches; ++u)
            if (u < nxu && tid + u * 256 < nx) *(f4*)(Xs + sdst + u * 64 * LDW) = xv[u];
#pragma unroll
        for (int u = 0; u < NG; ++u) *(f4*)(Ds + sdst + u * 64 * LDW) = dv[u];
        __syncthreads();
#pragma unroll 1
        for (int g = 0; g < NG; ++g) {
            const int tr = box_div(tile, t.nc_inv), R0 = tr * t.OH;
            const int p = (wave * NG + g) * 16 + gi * 4;
            const int oh = box_div(p, t.OWs_inv), ow = p - oh * t.OWs;
            const bool ok = oh < min(t.OH, t.rows - R0);
            const int b0 = ok ? ((box_prow(t, R0 + oh) - box_prow(t, R0)) * t.IW + ow * (K1 ? 1 : ST)) * LDW + li : li;
            const int left = ok ? min(t.OW, t.Wo - (tile - tr * t.nc) * t.OW) - ow : 0;   // slots that hold a pixel
#pragma unroll 1
            for (int j = 0; j < 4; ++j) {
                const float d = Ds[(p + j) * LDW + li];
#pragma unroll
                for (int k = 0; k < RS; ++k) {
                    const float v = Xs[b0 + toff[k] + j * JST];
                    acc[k] = mfma16x16x4(d, j < left ? v : 0.f, acc[k]);
                }
            }
        }
        __syncthreads();
        if (chained && (tile + 1 - t0) % run == 0 && tile + 1 < t1) leave();
    }
    finish();
}

// Boxes of the spatially tiled weight gradient, or false when it does not
// apply (the GEMM-style kernel takes those passes).  Up to 384 channel blocks:
// at most 768 workgroups, one round of three to a compute unit; each takes a
// single box of 256 slots where that gives at least 512 workgroups, else a run
// of boxes of 128 slots, or of 64 where 128 leave fewer than 512 and 64 give
// more (measured over 512-1536 workgroups and all three sizes: within 4% of
// the best of 22 passes); 1x1 passes whose boxes are all full take one of 256
// slots each in up to three rounds (64 x 32x32, 32 -> 32 19.2 us in runs, 14.6
// so; 64 -> 64 at 32 x 32x32 23.9 and 18.6; ragged ones, 32 x 28x28, 64 -> 64,
// 17.2 and 18.5).  More blocks do not divide a round: up to four
// splits, at least 1536 workgroups where they suffice, even out the rounds (16
// x 14x14: 320 -> 320 channels with one split 110 us, with four 95; 448 -> 448
// 202, two 177; 768 blocks 152, two 152, three 160).
// A workgroup reads its 16 output and 16 input channels of every pixel, four
// times the traffic of the GEMM kernel's 64 x 64 tiles, which counts where taps
// do not share it.  1x1 passes of 2^28 products and more (3e8 below 32768
// pixels) take the GEMM kernel: 64 x 32x32, 64 -> 64, 2^28, 37 us and 31 there,
// 96 -> 96 65 and 44; 32 x 28x28, 320 -> 320, 299 and 93; 96 -> 96, 2.3e8, 25
// and 33; 16 x 32x32, 64 -> 256, 2.7e8, 28 and 32 (16 channels leave its tiles
// mostly empty: 100 x 64x64, 16 -> 64, 52 and 68).  So do 3x3 passes of stride 2
// from 128 blocks and 2^27 products (per tap) on: 32 x 14x14, 128 -> 256, 71 and
// 67, 320 -> 320 217 and 174; 16 x 13x13, 160 -> 320, 1.4e8, 67 and 56; 4 x
// 13x13, 144 -> 288, 2.8e7, 16 and 21; 40 x 20x20, 96 -> 192, 72 blocks, 72 and 77.
struct WgTileCfg { int ng, tiles, per, splits, run; BoxGeom t; size_t lds; };
static bool pick_wgrad_tile(int Nb, int Hi, int Wi, int Cin_p, int Ho, int Wo, int Cout, int R, int S, int stride,
                            int pad, WgTileCfg& out) {
    if (Cin_p % 4 || Cout % 4 || R != S || (R != 1 && R != 3) || (stride != 1 && stride != 2)) return false;
    if (Cin_p < 16 && Cout > 32) return false;   // mostly empty MFMA columns: the GEMM kernel is as fast
    const long blocks = (long)((Cout + 15) / 16) * ((Cin_p + 15) / 16);
    const double M = (double)Nb * Ho * Wo;
    const double products = M * Cin_p * Cout;
    if (R == 1 ? Cin_p > 16 && products >= (M >= 32768 ? 268435456.0 : 3e8)
               : stride == 2 && blocks >= 128 && products >= 134217728.0)
        return false;
    const long most = blocks <= 384 ? 768 / blocks : std::min<long>(4, (1535 + blocks) / blocks);
    bool found = false;
    for (int ng : {4, 2, 1}) {
        WgTileCfg c;
        if (!box_pick(c.t, Nb, Ho, Wo, R, R == 1 ? 1 : stride, pad, ng * 64, 4, kWgBatches) ||
            !box_fits(c.t, Nb, (double)Hi * Wi * Cin_p) || !buf_fits((double)c.t.OH * Wo * Cout))
            continue;
        c.t.far |= !buf_fits((double)Nb * Ho * Wo * Cout);
        c.ng = ng;
        c.lds = sizeof(float) *
                std::max<size_t>(((size_t)c.t.IH * c.t.IW + ng * 64) * 20, (size_t)4 * R * S * 256 + 4);
        c.tiles = box_tiles(c.t);
        const bool each = R == 1 && ng == 4 && c.tiles * blocks <= 2304 && box_full(c.t, 256);
        const long splits = each ? c.tiles : std::min<long>(c.tiles, most);
        c.per = (int)((c.tiles + splits - 1) / splits);
        c.splits = (c.tiles + c.per - 1) / c.per;
        c.run = wg_run(ng, Wo);
        if (ng == 4 && (c.per > 1 || c.splits * blocks < 512)) continue;
        if (found && c.splits <= out.splits) break;
        found = true;
        out = c;
        if (c.splits * blocks >= 512) break;
    }
    return found;
}

// Weight gradient of a stem (4 stored input channels): as conv_wgrad_tile_f32,
// with 16 MFMA columns = four taps of a filter row x 4 channels (KS * NSG
// column tiles: 3x3 three, 7x7 fourteen) read from LDS as they lie, 16
// consecutive floats from the pixel of the first tap.  Columns past the filter
// row are formed and dropped.  (128 x 32x32, 4 -> 16: 10.3 us with a column
// tile per tap, 7.4 here; 4 -> 96: 36, 22; 7x7/2, 4 -> 64: 97, 80.)
template <int KS, int NG, int ST, bool FULL, bool FAR>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(KS == 3 && (FULL || NG == 2) ? 4 : 3, 8)))
void conv_wgrad_stem_f32(const float* __restrict__ dY, const float* __restrict__ X,
                                                           float* __restrict__ part, WgArgs a, BoxGeom t, int tiles,
                                                           int per, int run) {
    constexpr int NSG = (KS + 3) / 4, RG = KS * NSG, LDW = 20, JST = ST * 4, TP = NG * 64;
    extern __shared__ float lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int gi = lane >> 4, li = lane & 15, q = tid & 3;
    const int co0 = blockIdx.y * 16;
    const int npix = t.IH * t.IW;
    float* Ds = lds;                          // [TP][LDW] dY of the box, 16 channels
    float* Xs = lds + TP * LDW;               // [npix][4] input, 16 floats of slack behind
    const long image = (long)a.Hi * a.Wi * 4, row = (long)a.Wo * a.Cout;
    f4 xv[kTileBatches], dv[NG];
    auto load = [&](int tile) {
        const int tr = box_div(tile, t.nc_inv), tc = tile - tr * t.nc;
        const int R0 = tr * t.OH, w0 = tc * t.OW, P0 = box_prow(t, R0);
        const int ohv = min(t.OH, t.rows - R0), owv = min(t.OW, t.Wo - w0);
        const int n1 = FAR ? box_div(P0, t.Hp_inv) : 0, R1 = FAR ? R0 : 0;   // the descriptors' first image and row
        const __amdgpu_buffer_rsrc_t xr = buf_rsrc(X, n1, image, a.Nb), dr = buf_rsrc(dY, R1, row, t.rows);
#pragma unroll
        for (int u = 0; u < kTileBatches; ++u)
            if (u * 256 < npix) {
                const int pix = tid + u * 256;
                const int ih = box_div(pix, t.IW_inv), iw = pix - ih * t.IW;
                const int pr = P0 + ih;
                const int n = box_div(pr, t.Hp_inv), h = pr - n * t.Hp - t.pad_eff, w = w0 * ST + iw - t.pad_eff;
                const bool ok = ih < t.IH && n < a.Nb && h >= 0 && h < a.Hi && w >= 0 && w < a.Wi;
                xv[u] = buf_load4(xr, ok ? (unsigned)(((n - n1) * a.Hi + h) * a.Wi + w) * 16u : kNoLoad, 0);
            }
#pragma unroll
        for (int u = 0; u < NG; ++u) {
            const int p = (tid + u * 256) >> 2;
            const int oh = box_div(p, t.OWs_inv), ow = p - oh * t.OWs;
            const bool ok = oh < ohv && ow < owv && co0 + q * 4 < a.Cout;
            dv[u] = buf_load4(dr, ok ? (unsigned)(((R0 - R1 + oh) * t.Wo + w0 + ow) * a.Cout + co0 + q * 4) * 4u : kNoLoad,
                              0);
        }
    };
    f4 acc[RG];
    const int t0 = blockIdx.x * per, t1 = min(tiles, t0 + per);
    // the four waves' blocks summed in order, KS rows at a time
    float* red = lds;   // [4][NSG][16 co][16], then for each wave whether it met a NaN
    float all = 0.f;    // a NaN once one was among the sums
    auto rows = [&](auto use) {
        if (!FULL) {
#pragma unroll
            for (int k = 0; k < RG; ++k) all += (acc[k][0] + acc[k][1]) + (acc[k][2] + acc[k][3]);
            const bool nan = __any(all != all);
            if (lane == 0) red[4 * NSG * 256 + wave] = nan ? 1.f : 0.f;
        }
#pragma unroll
        for (int r = 0; r < KS; ++r) {
#pragma unroll
            for (int sg = 0; sg < NSG; ++sg)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    red[((wave * NSG + sg) * 16 + gi * 4 + i) * 16 + li] = acc[r * NSG + sg][i];
            lds_barrier();
#pragma unroll
            for (int sg = 0; sg < NSG; ++sg) {
                const int e = sg * 256 + tid;
                use(r, sg, ((red[e] + red[NSG * 256 + e]) + red[2 * NSG * 256 + e]) + red[3 * NSG * 256 + e]);
            }
            lds_barrier();
        }
    };
    // 3x3: runs of `run` boxes leave their sums in fp64 (7x7: see pick_wgrad_stem)
    double tot[KS == 3 ? RG : 1];
    const bool chained = KS == 3 && t1 - t0 > run;
    auto leave = [&]() {
        rows([&](int r, int sg, float v) { tot[KS == 3 ? r * NSG + sg : 0] += (double)v; });
#pragma unroll
        for (int k = 0; k < RG; ++k) acc[k] = f4{0.f, 0.f, 0.f, 0.f};
    };
    auto finish = [&]() {
        float* out = part + (long)blockIdx.x * a.Cout * (KS * KS * 4);
        rows([&](int r, int sg, float v) {
            if (chained) v = (float)(tot[KS == 3 ? r * NSG + sg : 0] + (double)v);
            const int co = co0 + (tid >> 4), s = sg * 4 + ((tid & 15) >> 2);
            if (s < KS && co < a.Cout) out[(long)co * (KS * KS * 4) + (r * KS + s) * 4 + (tid & 3)] = v;
        });
    };
#pragma unroll
    for (int k = 0; k < RG; ++k) acc[k] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (double& v : tot) v = 0.0;
    load(t0);
    for (int tile = t0; tile < t1; ++tile) {
#pragma unroll
        for (int u = 0; u < kTileBatches; ++u)
            if (u * 256 < npix && tid + u * 256 < npix) *(f4*)(Xs + (tid + u * 256) * 4) = xv[u];
        // (the last columns' reads of the last pixels run past the input: finite values, dropped)
        if (tid < 16) Xs[npix * 4 + tid] = 0.f;
#pragma unroll
        for (int u = 0; u < NG; ++u) *(f4*)(Ds + ((tid + u * 256) >> 2) * LDW + q * 4) = dv[u];
        const int tr = box_div(tile, t.nc_inv), R0 = tr * t.OH, P0 = box_prow(t, R0);
        const int ohv = min(t.OH, t.rows - R0);
        int boff[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const int p = (wave * NG + g) * 16 + gi * 4;
            const int oh = box_div(p, t.OWs_inv), ow = p - oh * t.OWs;
            boff[g] = oh < ohv ? ((box_prow(t, R0 + oh) - P0) * t.IW + ow * ST) * 4 + li : li;
        }
        lds_barrier();
        if (tile + 1 < t1) load(tile + 1);
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            float av[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) av[j] = Ds[((wave * NG + g) * 16 + gi * 4 + j) * LDW + li];
#pragma unroll
            for (int k = 0; k < RG; ++k) {
                const int toff = ((k / NSG) * t.IW + (k % NSG) * 4) * 4;
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[k] = mfma16x16x4(av[j], Xs[boff[g] + toff + j * JST], acc[k]);
            }
        }
        lds_barrier();
        if (chained && (tile + 1 - t0) % run == 0 && tile + 1 < t1) leave();
    }
    finish();
    if (FULL) return;
    const f4 nan = *(const f4*)(red + 4 * NSG * 256);
    if (nan[0] + nan[1] + nan[2] + nan[3] == 0.f) return;
    __syncthreads();
    // the same sums in the same order, zeros for both operands at slots without a pixel
#pragma unroll
    for (int k = 0; k < RG; ++k) acc[k] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (double& v : tot) v = 0.0;
#pragma unroll 1
    for (int tile = t0; tile < t1; ++tile) {
        load(tile);
#pragma unroll
        for (int u = 0; u < kTileBatches; ++u)
            if (u * 256 < npix && tid + u * 256 < npix) *(f4*)(Xs + (tid + u * 256) * 4) = xv[u];
        // (the last columns' reads of the last pixels run past the input: finite values, dropped)
        if (tid < 16) Xs[npix * 4 + tid] = 0.f;
#pragma unroll
        for (int u = 0; u < NG; ++u) *(f4*)(Ds + ((tid + u * 256) >> 2) * LDW + q * 4) = dv[u];
        __syncthreads();
#pragma unroll 1
        for (int g = 0; g < NG; ++g) {
            const int tr = box_div(tile, t.nc_inv), R0 = tr * t.OH;
            const int p = (wave * NG + g) * 16 + gi * 4;
            const int oh = box_div(p, t.OWs_inv), ow = p - oh * t.OWs;
            const bool ok = oh < min(t.OH, t.rows - R0);
            const int b0 = ok ? ((box_prow(t, R0 + oh) - box_prow(t, R0)) * t.IW + ow * ST) * 4 + li : li;
            const int left = ok ? min(t.OW, t.Wo - (tile - tr * t.nc) * t.OW) - ow : 0;   // slots that hold a pixel
#pragma unroll 1
            for (int j = 0; j < 4; ++j) {
                const float d = Ds[(p + j) * LDW + li];
#pragma unroll
                for (int k = 0; k < RG; ++k) {
                    const float v = Xs[b0 + ((k / NSG) * t.IW + (k % NSG) * 4) * 4 + j * JST];
                    acc[k] = mfma16x16x4(d, j < left ? v : 0.f, acc[k]);
                }
            }
        }
        __syncthreads();
        if (chained && (tile + 1 - t0) % run == 0 && tile + 1 < t1) leave();
    }
    finish();
}

// Boxes of a stem's weight gradient: 256 or 128 slots, at most 1024 workgroups.
// (A 7x7 one keeps one chain: 14 sums in fp64 do not fit its registers.  16 x
// 224x224, 4 -> 64: 49 MFMAs in a row; the GEMM kernel takes 98.)
static bool pick_wgrad_stem(int Nb, int Hi, int Wi, int Cin_p, int Ho, int Wo, int Cout, int R, int S, int stride,
                            int pad, WgTileCfg& out) {
    if (Cin_p != 4 || Cout % 4 || R != S || (R != 3 && R != 7) || (stride != 1 && stride != 2)) return false;
    const long blocks = (Cout + 15) / 16;
    bool found = false;
    for (int ng : {4, 2}) {
        WgTileCfg c;
        if (!box_pick(c.t, Nb, Ho, Wo, R, stride, pad, ng * 64, 4, 4 * kTileBatches) ||
            !box_fits(c.t, Nb, (double)Hi * Wi * 4) || !buf_fits((double)c.t.OH * Wo * Cout))
            continue;
        c.t.far |= !buf_fits((double)Nb * Ho * Wo * Cout);
        c.ng = ng;
        // a column tile reads up to 16 floats past its first tap's pixel
        c.lds = sizeof(float) * std::max<size_t>((size_t)ng * 64 * 20 + ((size_t)c.t.IH * c.t.IW + 4) * 4,
                                                 (size_t)4 * ((R + 3) / 4) * 256 + 4);
        c.tiles = box_tiles(c.t);
        const long splits = std::min<long>(c.tiles, std::max<long>(1, 1024 / blocks));
        c.per = (int)((c.tiles + splits - 1) / splits);
        c.splits = (c.tiles + c.per - 1) / c.per;
        c.run = wg_run(ng, Wo);
        found = true;
        out = c;
        if (c.splits * blocks >= 512) break;
    }
    return found;
}

template <int KS, int ST, bool FULL, bool FAR>
static hipError_t launch_wg_stem(const float* dY, const float* X, float* part, const WgArgs& a, const WgTileCfg& c,
                                 hipStream_t st) {
    dim3 grid((unsigned)c.splits, (unsigned)((a.Cout + 15) / 16));
    if (c.ng == 4)
        launch((conv_wgrad_stem_f32<KS, 4, ST, FULL, FAR>), grid, dim3(256), c.lds, st, dY, X, part, a, c.t, c.tiles, c.per,
               c.run);
    else
        launch((conv_wgrad_stem_f32<KS, 2, ST, FULL, FAR>), grid, dim3(256), c.lds, st, dY, X, part, a, c.t, c.tiles, c.per,
               c.run);
    return hipGetLastError();
}

template <bool FULL, bool FAR>
static hipError_t dispatch_wg_stem(const float* dY, const float* X, float* part, const WgArgs& a, const WgTileCfg& c,
                                   hipStream_t st) {
    if (a.R == 3) {
        if (a.stride == 1) return launch_wg_stem<3, 1, FULL, FAR>(dY, X, part, a, c, st);
        return launch_wg_stem<3, 2, FULL, FAR>(dY, X, part, a, c, st);
    }
    if (a.stride == 1) return launch_wg_stem<7, 1, FULL, FAR>(dY, X, part, a, c, st);
    return launch_wg_stem<7, 2, FULL, FAR>(dY, X, part, a, c, st);
}

WgradPlan wgrad_plan(int Nb, int Hi, int Wi, int Cin_p, int Ho, int Wo, int Cout, int R, int S, int stride, int pad) {
    WgradPlan p{};
    const long M = (long)Nb * Ho * Wo;
    const int Ktot = R * S * Cin_p;
    WgTileCfg c;
    const bool stem = pick_wgrad_stem(Nb, Hi, Wi, Cin_p, Ho, Wo, Cout, R, S, stride, pad, c);
    if (stem || pick_wgrad_tile(Nb, Hi, Wi, Cin_p, Ho, Wo, Cout, R, S, stride, pad, c)) {
        p.tile = stem ? 2 : 1;
        p.splits = c.splits;
        p.part_floats = (long)p.splits * Cout * Ktot;
        return p;
    }

    p.tm = Cout <= 16 ? 1 : (Cout <= 32 ? 2 : 4);
    p.tn = 4;
    const long tiles = (long)((Cout + 16 * p.tm - 1) / (16 * p.tm)) * ((Ktot + 16 * p.tn - 1) / (16 * p.tn));
    // about 512 workgroups per pass, each over at least 512 output pixels
    long splits = (512 + tiles - 1) / tiles;
    const long max_splits = (M + 511) / 512;
    if (splits > max_splits) splits = max_splits;
    // at most 32 MFMAs in a row where rows are a power of two long (as wg_run;
    // 64 x 32x32, 160 -> 320, 1x1: 129 us instead of 124)
    if ((Wo & (Wo - 1)) == 0) splits = std::max(splits, max_splits);
    if (splits < 1) splits = 1;
    long pps = (M + splits - 1) / splits;
    pps = (pps + 63) / 64 * 64;
    p.pix_per_split = (int)pps;
    p.splits = (int)((M + pps - 1) / pps);
    p.part_floats = (long)p.splits * Cout * Ktot;
    return p;
}

template <int TM, int TN>
static hipError_t launch_wg(const float* dY, const float* X, float* part, const WgArgs& a, const WgradPlan& p,
                            hipStream_t st) {
    const int Ktot = a.R * a.S * a.Cin_p;
    dim3 grid((unsigned)((a.Cout + TM * 16 - 1) / (TM * 16)), (unsigned)((Ktot + TN * 16 - 1) / (TN * 16)),
              (unsigned)p.splits);
    launch((conv_wgrad_f32<TM, TN>), grid, dim3(256), 0, st, dY, X, part, a);
    return hipGetLastError();
}

template <int RS, int ST, bool FULL, bool FAR>
static hipError_t launch_wg_tile(const float* dY, const float* X, float* part, const WgArgs& a, const WgTileCfg& c,
                                 const float* in_ss, hipStream_t st) {
    dim3 grid((unsigned)c.splits, (unsigned)((a.Cout + 15) / 16), (unsigned)((a.Cin_p + 15) / 16));
    if (c.ng == 4)
        launch((conv_wgrad_tile_f32<RS, 4, ST, FULL, FAR>), grid, dim3(256), c.lds, st, dY, X, part, a, c.t, c.tiles, c.per,
               c.run, in_ss);
    else if (c.ng == 2)
        launch((conv_wgrad_tile_f32<RS, 2, ST, FULL, FAR>), grid, dim3(256), c.lds, st, dY, X, part, a, c.t, c.tiles, c.per,
               c.run, in_ss);
    else
        launch((conv_wgrad_tile_f32<RS, 1, ST, FULL, FAR>), grid, dim3(256), c.lds, st, dY, X, part, a, c.t, c.tiles, c.per,
               c.run, in_ss);
    return hipGetLastError();
}

template <bool FULL, bool FAR>
static hipError_t dispatch_wg_tile(const float* dY, const float* X, float* part, const WgArgs& a, const WgTileCfg& c,
                                   const float* in_ss, hipStream_t st) {
    if (a.R == 1) {
        if (a.stride == 1) return launch_wg_tile<1, 1, FULL, FAR>(dY, X, part, a, c, in_ss, st);
        return launch_wg_tile<1, 2, FULL, FAR>(dY, X, part, a, c, in_ss, st);
    }
    if (a.stride == 1) return launch_wg_tile<9, 1, FULL, FAR>(dY, X, part, a, c, in_ss, st);
    return launch_wg_tile<9, 2, FULL, FAR>(dY, X, part, a, c, in_ss, st);
}

hipError_t launch_conv_wgrad(const float* dY, const float* X, float* part, int Nb, int Hi, int Wi, int Cin_p,
                             int Ho, int Wo, int Cout, int R, int S, int stride, int pad, const WgradPlan& p,
                             hipStream_t st, const float* in_ss) {
    WgArgs a{Nb, Hi, Wi, Cin_p, Ho, Wo, Cout, R, S, stride, pad, p.pix_per_split};
    if (in_ss && p.tile != 1) return hipErrorInvalidValue;   // folding needs the spatial kernel
    if (p.tile == 2) {
        WgTileCfg c;
        if (!pick_wgrad_stem(Nb, Hi, Wi, Cin_p, Ho, Wo, Cout, R, S, stride, pad, c) || c.splits != p.splits)
            return hipErrorInvalidValue;
        if (c.t.far) return dispatch_wg_stem<false, true>(dY, X, part, a, c, st);
        return box_full(c.t, c.ng * 64) ? dispatch_wg_stem<true, false>(dY, X, part, a, c, st)
                                        : dispatch_wg_stem<false, false>(dY, X, part, a, c, st);
    }
    if (p.tile) {
        WgTileCfg c;
        if (!pick_wgrad_tile(Nb, Hi, Wi, Cin_p, Ho, Wo, Cout, R, S, stride, pad, c) || c.splits != p.splits)
            return hipErrorInvalidValue;
        if (c.t.far) return dispatch_wg_tile<false, true>(dY, X, part, a, c, in_ss, st);
        return box_full(c.t, c.ng * 64) ? dispatch_wg_tile<true, false>(dY, X, part, a, c, in_ss, st)
                                        : dispatch_wg_tile<false, false>(dY, X, part, a, c, in_ss, st);
    }
    if (p.tm == 1) return launch_wg<1, 4>(dY, X, part, a, p, st);
    if (p.tm == 2) return launch_wg<2, 4>(dY, X, part, a, p, st);
    return launch_wg<4, 4>(dY, X, part, a, p, st);
}

// Workgroup of 1024 threads on one job: L split lanes x Q = 1024 / L output
// quads.  Thread (l, q) adds the float4 partials of quad q over splits
// l, l + L, ... (eight loads issued ahead of their adds, which stay in split
// order); the L lane sums are then halved pairwise in LDS (lane i += lane
// i + h for h = L/2, L/4, ..., 1).  A wave reads 64 / min(Q, 64) runs of
// min(Q, 64) consecutive quads of one split.
__global__ __launch_bounds__(1024) void wgrad_reduce_multi_k(const WgRedTable t) {
    __shared__ f4 red[1024];
    int j = 0;
    while (j + 1 < t.n && (int)blockIdx.x >= t.job[j + 1].wg0) ++j;
    const WgRedJob& J = t.job[j];
    const int lg = J.lanes_log2, L = 1 << lg, Q = 1024 >> lg;
    const int tid = threadIdx.x, sl = tid >> (10 - lg), qi = tid & (Q - 1);
    const long nq = (long)J.Cout * J.Ktot / 4;
    const long quad = (long)(blockIdx.x - J.wg0) * Q + qi;
    f4 s = f4{0.f, 0.f, 0.f, 0.f};
    if (quad < nq) {
        const f4* p = (const f4*)J.part + quad;
        int k = sl;
        for (; k + 7 * L < J.splits; k += 8 * L) {
            f4 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = p[(long)(k + u * L) * nq];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; k < J.splits; k += L) s += p[(long)k * nq];
    }
    red[tid] = s;
    __syncthreads();
    for (int h = L >> 1; h > 0; h >>= 1) {
        if (sl < h) red[tid] = red[tid] + red[tid + h * Q];
        __syncthreads();
    }
    if (sl != 0 || quad >= nq) return;
    const f4 v = red[qi];
    const int co = (int)(quad * 4 / J.Ktot);
    const int col0 = (int)(quad * 4 - (long)co * J.Ktot);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int col = col0 + e, tap = col / J.Cin_p, c = col - tap * J.Cin_p;
        if (c < J.Cin) J.g[((long)co * J.Cin + c) * J.RS + tap] = v[e];
    }
}

bool wgred_add(WgRedTable& t, const float* part, int splits, int Cout, int Ktot, int Cin, int Cin_p, int R, int S,
               float* g) {
    if (t.n >= kWgRedMaxJobs || Ktot % 4 || Ktot != R * S * Cin_p || splits < 1 ||
        ((uintptr_t)part & 15))
        return false;
    int lg = 0;
    while (lg < 6 && (8 << lg) < splits) ++lg;   // about eight splits per lane, at most 64 lanes
    const long nq = (long)Cout * Ktot / 4;
    const long wgs = (nq + (1024 >> lg) - 1) / (1024 >> lg);
    if (t.n == 0) t.wgs = 0;
    if ((long)t.wgs + wgs > 0x7fffffffL) return false;
    t.job[t.n] = WgRedJob{part, g, splits, Cout, Ktot, Cin, Cin_p, R * S, lg, t.wgs};
    t.wgs += (int)wgs;
    ++t.n;
    return true;
}

hipError_t launch_wgrad_reduce_multi(const WgRedTable& t, hipStream_t st) {
    if (t.n == 0) return hipSuccess;
    launch(wgrad_reduce_multi_k, dim3((unsigned)t.wgs), dim3(1024), 0, st, t);
    return hipGetLastError();
}

}  // namespace lpp
