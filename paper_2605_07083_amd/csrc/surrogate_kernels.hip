// surrogate_kernels.hip -- BF16-MFMA 1D convolution network of the learned
// warm start: (emission flux, cathode temperature, bias, neutral density) ->
// (phi / V, ln(n_e / n0), ln(n_i / n0)) at the X cell centres of a diode.
//
// Net: 6 conv1d layers, kernel 5, zero padding 2, channels
// 16 -> 64 -> 64 -> 64 -> 64 -> 64 -> 39 (stored padded to 48), tanh after
// layers 1-5.  Input channels: the 4 normalised parameters and 12 functions of
// the position.  Weights are BF16 (FP32 master copies for Adam), activations
// enter every layer as BF16, all products accumulate in FP32 on
// v_mfma_f32_16x16x32_bf16.
//
// Layouts: activations and gradients channels last, act[b][x][c]: the forward
// and input-gradient GEMMs read them along K (channels) with 16-byte reads, the
// weight gradient (K = positions) reads the same tiles transposed with
// ds_read_b64_tr_b16; forward weights Wf in fragment order (see frag_at),
// transposed weights for the input gradient Wb[ci][t*Cout + co]; both padded
// with zeros to a multiple of 32 in K.
//
// MFMA 16x16x32 (bf16) lane layout: lane l supplies A[l%16][8(l/16)+i] and
// B[8(l/16)+i][l%16], i = 0..7, and receives D[4(l/16)+i][l%16], i = 0..3.
#include <hip/hip_runtime.h>
#include <limits.h>
#include <stdint.h>
#include <type_traits>

#include "net_tanh.h"

namespace sur {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;

constexpr int KS = 5;     // kernel size
constexpr int OUT = 39;   // output channels: phi / V, ln n_e / n0, ln n_i / n0, 36 velocity quantiles
constexpr int OUTP = 48;  // padded to whole 16-column matrix-core tiles

__device__ __forceinline__ bf16x8 zero8()
{
    bf16x8 z;
#pragma unroll
    for (int i = 0; i < 8; ++i) z[i] = (__bf16)0.0f;
    return z;
}

__device__ __forceinline__ bf16x8 load8(const __bf16 *p) { return *reinterpret_cast<const bf16x8 *>(p); }

__device__ __forceinline__ uint4 philox(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        uint32_t lo0 = 0xD2511F53u * c0, hi0 = __umulhi(0xD2511F53u, c0);
        uint32_t lo1 = 0xCD9E8D57u * c2, hi1 = __umulhi(0xCD9E8D57u, c2);
        uint32_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
        k0 += 0x9E3779B9u; k1 += 0xBB67AE85u;
    }
    return make_uint4(c0, c1, c2, c3);
}

// Place of forward weight (co, kappa = t*CIN + ci) in fragment order: the
// layer's weights as matrix-core fragments of 16 output channels x 32 kappa,
// output tile by output tile, each fragment's 64 lanes x 8 elements in a row.
// A wave reads a fragment as one contiguous kilobyte.
__device__ __forceinline__ int frag_at(int co, int kappa, int kp)
{
    return (((co >> 4) * (kp >> 5) + (kappa >> 5)) * 64 + ((kappa & 31) >> 3) * 16 + (co & 15)) * 8 + (kappa & 7);
}

// ---------------------------------------------------------------------------
// Input features.  params[b] = (Gamma m^-2 s^-1, T_c K, V volts, n_g m^-3) are
// mapped to [-1, 1] over the training ranges (log scale for the flux and the
// density); the position features resolve both sheaths and the interior.
// ---------------------------------------------------------------------------
// The features of position x in four parts of similar cost (PART 0..3: f0..f3,
// f6..f9, f10..f11, the rest), each written to its place of f.
template <int PART>
__device__ __forceinline__ void features_part(const float *__restrict__ p, int x, int X, __bf16 *f)
{
    const float u = ((float)x + 0.5f) / (float)X;
    if constexpr (PART == 0) {
        const float g = p[0], T = p[1], V = p[2], ng = p[3];
        f[0] = (__bf16)(2.0f * (log10f(g / 1e19f) / log10f(12.0f)) - 1.0f);
        f[1] = (__bf16)((T - 2000.0f) / 200.0f);
        f[2] = (__bf16)((V - 12.5f) / 7.5f);
        f[3] = (__bf16)(2.0f * log10f(ng / 1e21f) - 1.0f);
    } else if constexpr (PART == 1) {
        float s1, c1, s2, c2;
        sincospif(u, &s1, &c1);
        sincospif(2.0f * u, &s2, &c2);
        f[6] = (__bf16)s1;
        f[7] = (__bf16)c1;
        f[8] = (__bf16)s2;
        f[9] = (__bf16)c2;
    } else if constexpr (PART == 2) {
        float s4, c4;
        sincospif(4.0f * u, &s4, &c4);
        f[10] = (__bf16)s4;
        f[11] = (__bf16)c4;
    } else {
        f[4] = (__bf16)(2.0f * u - 1.0f);
        f[5] = (__bf16)(1.0f - 2.0f * u);
        f[12] = (__bf16)__expf(-64.0f * u);
        f[13] = (__bf16)__expf(-64.0f * (1.0f - u));
        f[14] = (__bf16)__expf(-16.0f * u);
        f[15] = (__bf16)__expf(-16.0f * (1.0f - u));
    }
}

// ---------------------------------------------------------------------------
// Weights of a layer staged in LDS once per block: rows of the padded K
// length plus 8 elements, so that the 16 rows one matrix-core fragment reads
// fall on different banks.
// ---------------------------------------------------------------------------
template <int ROWS, int KP, int THREADS>
__device__ __forceinline__ void stage_rows(__bf16 *lds, const __bf16 *__restrict__ src)
{
    constexpr int V = KP / 8;    // 16-byte vectors per row
    constexpr int N = (ROWS * V + THREADS - 1) / THREADS;
    bf16x8 r[N];                 // every load in flight before the first store
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const int v = threadIdx.x + k * THREADS;
        r[k] = v < ROWS * V ? load8(src + (size_t)(v / V) * KP + (v % V) * 8) : zero8();
    }
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const int v = threadIdx.x + k * THREADS;
        if (v < ROWS * V) *reinterpret_cast<bf16x8 *>(lds + (v / V) * (KP + 8) + (v % V) * 8) = r[k];
    }
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <int T>
__device__ __forceinline__ bf16x8 window8(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3, uint32_t w4,
                                          uint32_t w5)
{
    // elements T .. T+7 of the 12-element window w0..w5 (2 per dword, low first)
    u32x4 r;
    if constexpr (T == 0) r = (u32x4){w0, w1, w2, w3};
    else if constexpr (T == 2) r = (u32x4){w1, w2, w3, w4};
    else if constexpr (T == 4) r = (u32x4){w2, w3, w4, w5};
    else if constexpr (T == 1)
        r = (u32x4){(w0 >> 16) | (w1 << 16), (w1 >> 16) | (w2 << 16), (w2 >> 16) | (w3 << 16), (w3 >> 16) | (w4 << 16)};
    else
        r = (u32x4){(w1 >> 16) | (w2 << 16), (w2 >> 16) | (w3 << 16), (w3 >> 16) | (w4 << 16), (w4 >> 16) | (w5 << 16)};
    return __builtin_bit_cast(bf16x8, r);
}

__device__ __forceinline__ void store8(__bf16 *p, bf16x8 v) { *reinterpret_cast<bf16x8 *>(p) = v; }

// Transposed LDS read (ds_read_b64_tr_b16).  Within each group of 16 lanes,
// lane s = 4e + q passes the address of 4 consecutive 16-bit elements (row
// p_e, columns c + 4q .. c + 4q + 3 of a row-major tile); lane j of the group
// then receives the column c + j at the rows p_0 .. p_3.
__device__ __forceinline__ uint2 ldtr(const __bf16 *p)
{
    typedef short v4s __attribute__((ext_vector_type(4)));
    const v4s r = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s *)(p));
    return __builtin_bit_cast(uint2, r);
}

// ---------------------------------------------------------------------------
// Backward pass of one layer in one kernel, from the channels-last output
// gradient dZ[b][x][co] (of the pre-activation) and the layer's input:
//  * with DG (layers 2..6): the input gradient of the layer below,
//    dZprev[b][x][ci] = (sum_{t, co} W[co][t][ci] dZ[b][x-t+2][co]) (1 - y^2)
//    with y[b][x][ci] the FP32 input (the layer below's tanh output): GEMM
//    M = positions, N = CIN, K = 5 COUT, the transposed weights in LDS;
//  * the partial weight and bias gradients of the block's slice of one sample,
//    dW[co][t*CIN+ci] = sum_x dZ[x][co] in[x+t-2][ci], db[co] = sum_x dZ[x][co]
//    (in = y rounded to bfloat16, or the features for the first layer): GEMM
//    M = COUT, N = CIN per tap, K = positions.
// Block p = (sample, slice of BW_SLICE positions) writes part[p][co][kappa]
// and pbias[p][co] (k_reduce_adam sums the partials in a fixed order).  The
// slice goes through LDS in parts of BW_SUB positions plus two halo positions
// on each side (zero outside the sample), dZ and the input as channels-last
// bfloat16 tiles; the next part's global loads fly while a part is worked on.
// The input gradient reads the tiles along channels (16-byte reads); the
// weight gradient reads them transposed: a lane gets 4 consecutive positions
// of one channel per read, 8 for an A fragment (dZ^T), the 12-position window
// (two before, two after) of its 8 positions for the B fragments of the five
// taps.  The part's own FP32 inputs stay in LDS for the tanh derivative.
// Wave w of the weight gradient takes MW output x CW input channel
// tiles over every H-th run of 32-position groups; the H runs of a tile pair
// add their sums through LDS at the end; the bias is one more MFMA per output
// tile against a column of ones.  Row strides are chosen so that the four
// rows of a transposed read (32 bytes each) fall on different banks.
// ---------------------------------------------------------------------------
constexpr int BW_SLICE = 256;
constexpr int BW_SUB = 128;
constexpr int BW_THREADS = 512;
constexpr int BW_ROWS = BW_SUB + 4;        // positions -2 .. BW_SUB + 1 of a part

constexpr int bw_stride(int c) { return c == 64 ? 80 : c; }    // 160, 96 or 32 bytes per row

template <int CIN, int COUT, bool DG>
struct BwdShape {
    static constexpr int K = KS * CIN, KP = (K + 31) / 32 * 32;           // weight-gradient partial layout
    static constexpr int KD = KS * COUT, KPB = (KD + 31) / 32 * 32;       // input-gradient K
    static constexpr int MT = COUT / 16, CT = CIN / 16;
    static constexpr int MW = MT % 2 == 0 ? 2 : MT;                       // output tiles per wave
    static constexpr int CW = (MW == 2 && CT % 2 == 0) ? 2 : 1;           // input tiles per wave
    static constexpr int PAIRS = (MT / MW) * (CT / CW);
    static constexpr int WAVES = BW_THREADS / 64;
    static constexpr int H = WAVES / PAIRS;
    static constexpr int GPW = BW_SUB / 32 / H;                           // groups per wave per whole part
    static constexpr int RS = (MW * CW * KS + MW) * 4;
    static constexpr int SD = bw_stride(COUT), SI = bw_stride(CIN);
    static constexpr int DV = COUT / 8;                                   // 16-byte vectors per dZ row
    static constexpr int IV = DG ? CIN / 4 : CIN / 8;                     // float4 (y) or bf16x8 (features) per row
    static constexpr int ND = (BW_ROWS * DV + BW_THREADS - 1) / BW_THREADS;
    static constexpr int NI = (BW_ROWS * IV + BW_THREADS - 1) / BW_THREADS;
    static constexpr size_t LDS_D = (size_t)BW_ROWS * SD * 2;
    static constexpr size_t LDS_I = (size_t)BW_ROWS * SI * 2;
    static constexpr size_t LDS_W = DG ? (size_t)CIN * (KPB + 8) * 2 : 0;
    static constexpr int YS = CIN + 4;                                    // FP32 input rows of the part's own positions (DG)
    static constexpr size_t LDS_Y = DG ? (size_t)BW_SUB * YS * 4 : 0;
    static constexpr size_t LDS_OP = LDS_D + LDS_I + LDS_W + LDS_Y;
    static constexpr size_t LDS_RED = (size_t)(H - 1) * PAIRS * RS * 64 * 4;
    static constexpr size_t LDS_OUT = (size_t)COUT * (KP + 1) * 4;
    static constexpr size_t LDS_1 = LDS_OP > LDS_RED ? LDS_OP : LDS_RED;
    static constexpr size_t LDS = LDS_1 > LDS_OUT ? LDS_1 : LDS_OUT;
    static_assert(MT % MW == 0 && CT % CW == 0 && WAVES % PAIRS == 0 && H >= 1, "wave tiling");
    static_assert((BW_SUB / 32) % H == 0 && BW_SUB / 16 == WAVES, "whole groups per wave, one input-gradient tile per wave");
    static_assert(CIN % 16 == 0 && COUT % 16 == 0, "whole channel tiles");
};

template <int CIN, int COUT, bool DG>
__global__ __launch_bounds__(BW_THREADS) void k_conv_bwd(const __bf16 *__restrict__ dz, const float *__restrict__ yin,
                                                         const __bf16 *__restrict__ fin, const __bf16 *__restrict__ Wb,
                                                         __bf16 *__restrict__ dzprev, float *__restrict__ part,
                                                         float *__restrict__ pbias, int X)
{
    using S = BwdShape<CIN, COUT, DG>;
    constexpr int KP = S::KP, KPB = S::KPB, KD = S::KD, MW = S::MW, CW = S::CW, PAIRS = S::PAIRS, H = S::H;
    constexpr int RS = S::RS, SD = S::SD, SI = S::SI, GPW = S::GPW;
    __shared__ __align__(16) char lds[S::LDS];
    __bf16 *Dt = reinterpret_cast<__bf16 *>(lds);                          // dZ rows of a part
    __bf16 *It = reinterpret_cast<__bf16 *>(lds + S::LDS_D);               // input rows of a part
    __bf16 *Wl = reinterpret_cast<__bf16 *>(lds + S::LDS_D + S::LDS_I);    // transposed weights (DG)
    float *Yt = reinterpret_cast<float *>(lds + S::LDS_D + S::LDS_I + S::LDS_W);   // FP32 input, own positions (DG)
    const int slices = (X + BW_SLICE - 1) / BW_SLICE;
    const int p = blockIdx.x, b = p / slices;
    const int xb = (p - b * slices) * BW_SLICE;
    const int len = min(X, xb + BW_SLICE) - xb;          // a multiple of 64
    const int tid = threadIdx.x;
    const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = lane & 15, kb = lane >> 4;
    const int e = m >> 2, q = m & 3;                     // this lane's row and column group in a transposed read

    // one part's global loads into registers: dZ and input rows of positions xs - 2 .. xs + BW_SUB + 1
    bf16x8 rd[S::ND];
    float4 ry[DG ? S::NI : 1];
    bf16x8 rf[DG ? 1 : S::NI];
    auto load_part = [&](int xs) {
#pragma unroll
        for (int k = 0; k < S::ND; ++k) {
            const int v = tid + k * BW_THREADS, r = v / S::DV, c = (v % S::DV) * 8, x = xs - 2 + r;
            rd[k] = v < BW_ROWS * S::DV && x >= 0 && x < X ? load8(dz + ((size_t)b * X + x) * COUT + c) : zero8();
        }
#pragma unroll
        for (int k = 0; k < S::NI; ++k) {
            const int v = tid + k * BW_THREADS, r = v / S::IV, x = xs - 2 + r;
            const bool ok = v < BW_ROWS * S::IV && x >= 0 && x < X;
            if constexpr (DG) {
                const int c = (v % S::IV) * 4;
                ry[k] = ok ? *reinterpret_cast<const float4 *>(yin + ((size_t)b * X + x) * CIN + c)
                           : make_float4(0.f, 0.f, 0.f, 0.f);
            } else {
                const int c = (v % S::IV) * 8;
                rf[k] = ok ? load8(fin + ((size_t)b * X + x) * CIN + c) : zero8();
            }
        }
    };
    auto store_part = [&]() {
#pragma unroll
        for (int k = 0; k < S::ND; ++k) {
            const int v = tid + k * BW_THREADS;
            if (v < BW_ROWS * S::DV) store8(Dt + (v / S::DV) * SD + (v % S::DV) * 8, rd[k]);
        }
#pragma unroll
        for (int k = 0; k < S::NI; ++k) {
            const int v = tid + k * BW_THREADS;
            if (v >= BW_ROWS * S::IV) continue;
            if constexpr (DG) {
                bf16x4 h;
                h[0] = (__bf16)ry[k].x;
                h[1] = (__bf16)ry[k].y;
                h[2] = (__bf16)ry[k].z;
                h[3] = (__bf16)ry[k].w;
                const int r = v / S::IV, c = (v % S::IV) * 4;
                *reinterpret_cast<bf16x4 *>(It + r * SI + c) = h;
                // the FP32 values of the part's own positions for the tanh derivative
                if (r >= 2 && r < 2 + BW_SUB) *reinterpret_cast<float4 *>(Yt + (r - 2) * S::YS + c) = ry[k];
            } else {
                store8(It + (v / S::IV) * SI + (v % S::IV) * 8, rf[k]);
            }
        }
    };

    f32x4 acc[MW][CW][KS], bacc[MW];
#pragma unroll
    for (int u = 0; u < MW; ++u) {
        bacc[u] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int v = 0; v < CW; ++v)
#pragma unroll
            for (int t = 0; t < KS; ++t) acc[u][v][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    bf16x8 ones;
#pragma unroll
    for (int i = 0; i < 8; ++i) ones[i] = (__bf16)1.0f;
    const bool active = w < PAIRS * H;
    const int pair = w % PAIRS, h = w / PAIRS;
    const int mw = pair % (S::MT / MW), cw = pair / (S::MT / MW);

    load_part(xb);
    if constexpr (DG) stage_rows<CIN, KPB, BW_THREADS>(Wl, Wb);
    for (int xo = 0; xo < len; xo += BW_SUB) {
        const int xs = xb + xo, sl = min(BW_SUB, len - xo);
        store_part();
        __syncthreads();
        if (xo + BW_SUB < len) load_part(xs + BW_SUB);

        if constexpr (DG) {
            // input gradient of the 16 positions x0 .. x0 + 15 of the part (one tile per wave)
            const int x0 = w * 16;
            if (x0 < sl) {
                constexpr int NT = CIN / 16;
                f32x4 dacc[NT];
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) dacc[nt] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < KPB / 32; ++ks) {
                    const int kappa = ks * 32 + kb * 8;
                    bf16x8 a = zero8();
                    if (kappa < KD) {
                        const int t = kappa / COUT, co = kappa - t * COUT;
                        // dZ at position x0 + m - t + 2: row x0 + m - t + 4 of the part
                        a = *reinterpret_cast<const bf16x8 *>(Dt + (x0 + m - t + 4) * SD + co);
                    }
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        const bf16x8 bw = *reinterpret_cast<const bf16x8 *>(Wl + (nt * 16 + m) * (KPB + 8) + kappa);
                        dacc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bw, dacc[nt], 0, 0, 0);
                    }
                }
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    const int ci = nt * 16 + m;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int xl = x0 + kb * 4 + i;
                        const float y = Yt[xl * S::YS + ci];
                        dzprev[((size_t)b * X + xs + xl) * CIN + ci] = (__bf16)(dacc[nt][i] * (1.0f - y * y));
                    }
                }
            }
        }

        // weight and bias gradients over this wave's groups of the part
        const int g0 = h * GPW, g1 = min(g0 + GPW, sl / 32);
        if (active && g0 < g1) {
            for (int g = g0; g < g1; ++g) {
                const int r0 = g * 32 + kb * 8 + e;       // the part row of this lane's address (+2: halo)
                bf16x8 a[MW];
#pragma unroll
                for (int u = 0; u < MW; ++u) {
                    const __bf16 *pa = Dt + (r0 + 2) * SD + (mw * MW + u) * 16 + 4 * q;
                    const uint2 a0 = ldtr(pa), a1 = ldtr(pa + 4 * SD);
                    a[u] = __builtin_bit_cast(bf16x8, (u32x4){a0.x, a0.y, a1.x, a1.y});
                    bacc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u], ones, bacc[u], 0, 0, 0);
                }
#pragma unroll
                for (int v = 0; v < CW; ++v) {
                    // the window of positions 8kb - 2 .. 8kb + 9 of the group
                    const __bf16 *pb = It + r0 * SI + (cw * CW + v) * 16 + 4 * q;
                    const uint2 b0 = ldtr(pb), b1 = ldtr(pb + 4 * SI), b2 = ldtr(pb + 8 * SI);
                    const bf16x8 w0 = window8<0>(b0.x, b0.y, b1.x, b1.y, b2.x, b2.y);
                    const bf16x8 w1 = window8<1>(b0.x, b0.y, b1.x, b1.y, b2.x, b2.y);
                    const bf16x8 w2 = window8<2>(b0.x, b0.y, b1.x, b1.y, b2.x, b2.y);
                    const bf16x8 w3 = window8<3>(b0.x, b0.y, b1.x, b1.y, b2.x, b2.y);
                    const bf16x8 w4 = window8<4>(b0.x, b0.y, b1.x, b1.y, b2.x, b2.y);
#pragma unroll
                    for (int u = 0; u < MW; ++u) {
                        acc[u][v][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u], w0, acc[u][v][0], 0, 0, 0);
                        acc[u][v][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u], w1, acc[u][v][1], 0, 0, 0);
                        acc[u][v][2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u], w2, acc[u][v][2], 0, 0, 0);
                        acc[u][v][3] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u], w3, acc[u][v][3], 0, 0, 0);
                        acc[u][v][4] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u], w4, acc[u][v][4], 0, 0, 0);
                    }
                }
            }
        }
        __syncthreads();           // the part's LDS is read before the next part is stored
    }

    // the other position runs of a tile pair hand their sums to the first through LDS
    float *R = reinterpret_cast<float *>(lds);
    constexpr int NACC = MW * CW * KS;
    if (H > 1 && active && h > 0) {
        float *r = R + ((size_t)((h - 1) * PAIRS + pair) * RS) * 64 + lane;
#pragma unroll
        for (int u = 0; u < MW; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
#pragma unroll
                for (int v = 0; v < CW; ++v)
#pragma unroll
                    for (int t = 0; t < KS; ++t) r[(((u * CW + v) * KS + t) * 4 + i) * 64] = acc[u][v][t][i];
                r[((NACC + u) * 4 + i) * 64] = bacc[u][i];
            }
    }
    __syncthreads();
    if (active && h == 0) {
#pragma unroll
        for (int gg = 1; gg < H; ++gg) {
            const float *r = R + ((size_t)((gg - 1) * PAIRS + pair) * RS) * 64 + lane;
#pragma unroll
            for (int u = 0; u < MW; ++u)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
#pragma unroll
                    for (int v = 0; v < CW; ++v)
#pragma unroll
                        for (int t = 0; t < KS; ++t) acc[u][v][t][i] += r[(((u * CW + v) * KS + t) * 4 + i) * 64];
                    bacc[u][i] += r[((NACC + u) * 4 + i) * 64];
                }
        }
    }
    __syncthreads();
    // the block's partial [COUT][KP] (row stride KP + 1) in LDS, then 16-byte stores
    float *O = reinterpret_cast<float *>(lds);
    constexpr int OS = KP + 1;
    if (active && h == 0) {
#pragma unroll
        for (int u = 0; u < MW; ++u)
#pragma unroll
            for (int v = 0; v < CW; ++v)
#pragma unroll
                for (int t = 0; t < KS; ++t) {
                    const int kappa = t * CIN + (cw * CW + v) * 16 + m;
#pragma unroll
                    for (int i = 0; i < 4; ++i) O[((mw * MW + u) * 16 + kb * 4 + i) * OS + kappa] = acc[u][v][t][i];
                }
        // column n of the ones product holds the row sums: lanes n = 0
        if (cw == 0 && m == 0) {
#pragma unroll
            for (int u = 0; u < MW; ++u)
#pragma unroll
                for (int i = 0; i < 4; ++i) pbias[(size_t)p * COUT + (mw * MW + u) * 16 + kb * 4 + i] = bacc[u][i];
        }
    }
    __syncthreads();
    float *out = part + (size_t)p * COUT * KP;
    constexpr int Q = KP / 4;
    for (int ee = tid; ee < COUT * Q; ee += BW_THREADS) {
        const int r = ee / Q, c = (ee % Q) * 4;
        const float *o = O + r * OS + c;
        *reinterpret_cast<float4 *>(out + (size_t)r * KP + c) = make_float4(o[0], o[1], o[2], o[3]);
    }
}

// ---------------------------------------------------------------------------
// The gradients of every layer from their partials, then Adam on the FP32
// master weights and biases and the BF16 copies of the weights: forward Wf in
// fragment order and transposed Wb[ci][t*COUTP + co].  A block takes 64
// consecutive entries of a layer's padded weights [COUTP][KP] followed by its
// biases; wave w sums the partials w, w + 16, ... of each, and the first wave
// adds the 16 sums in wave order and updates.  One launch for all layers whose
// partials the workspace holds at once (6 x 5.5 us as a launch per layer, whose
// few hundred blocks each left the chip half empty).  In the last one, one more
// block adds the loss from the forward blocks' shares.
// ---------------------------------------------------------------------------
constexpr int RA_WAVES = 16;

struct AdamLayer {
    const float *part, *pbias;
    float *wm, *mw, *vw, *dw, *bias, *mb, *vb, *db;
    __bf16 *Wf, *Wb;
    int cin, coutp, cout_real, kp, kpb;
    int first;               // the layer's first block (INT_MAX: none)
};

struct AdamArgs {
    AdamLayer L[6];          // the launch's layers, in front
    int P;                   // partials per layer
    int blocks;              // of all layers
    const double *loss_parts;
    int nloss;
    double *loss;
    float lr, b1, b2, eps, c1, c2;
};

__global__ __launch_bounds__(RA_WAVES * 64) void k_reduce_adam(AdamArgs A)
{
    __shared__ float red[RA_WAVES][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if ((int)blockIdx.x == A.blocks) {
        if (w != 0) return;
        double sum = 0.0;
        for (int k = lane; k < A.nloss; k += 64) sum += A.loss_parts[k];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
        if (lane == 0) *A.loss = sum;
        return;
    }
    int l = 0;
#pragma unroll
    for (int k = 1; k < 6; ++k)
        if ((int)blockIdx.x >= A.L[k].first) l = k;
    const AdamLayer &L = A.L[l];
    const int kp = L.kp, coutp = L.coutp, cin = L.cin;
    const int i0 = ((int)blockIdx.x - L.first) * 64, i = i0 + lane;
    const int nw = coutp * kp;                 // a multiple of 64: a block holds weights or biases
    const bool isw = i0 < nw, inr = i < nw + coutp;
    int co, kappa = 0, stride, at;
    if (isw) {
        co = i / kp;
        kappa = i - co * kp;
        stride = nw;
        at = i;
    } else {
        co = i - nw;
        stride = coutp;
        at = co;
    }
    const bool live = inr && co < L.cout_real && (!isw || kappa < KS * cin);
    float sum = 0.0f;
    if (live) {
        const float *src = (isw ? L.part : L.pbias) + at;
#pragma unroll 4
        for (int q = w; q < A.P; q += RA_WAVES) sum += src[(size_t)q * stride];
    }
    red[w][lane] = sum;
    __syncthreads();
    if (w != 0 || !inr) return;
    float gi = 0.0f;
#pragma unroll
    for (int k = 0; k < RA_WAVES; ++k) gi += red[k][lane];
    float *wp = isw ? L.wm + i : L.bias + co, *mo = isw ? L.mw + i : L.mb + co, *ve = isw ? L.vw + i : L.vb + co;
    (isw ? L.dw[i] : L.db[co]) = gi;
    const float m1 = __builtin_fmaf(1.0f - A.b1, gi, A.b1 * *mo);
    const float v1 = __builtin_fmaf(gi, (1.0f - A.b2) * gi, A.b2 * *ve);
    *mo = m1;
    *ve = v1;
    const float nwv = *wp - A.lr * (m1 / A.c1) / (sqrtf(v1 / A.c2) + A.eps);
    *wp = nwv;
    if (isw) {
        const __bf16 v = (__bf16)(live ? nwv : 0.0f);
        L.Wf[frag_at(co, kappa, kp)] = v;
        if (kappa < KS * cin) {
            const int t = kappa / cin, ci = kappa - t * cin;
            L.Wb[(size_t)ci * L.kpb + t * coutp + co] = v;
        }
    }
}

// masters [COUTP][KP] (kappa = t*CIN + ci) -> Wf (fragment order, bf16) and
// Wb[ci][t*COUTP + co] (padded to KPB)
__global__ void k_requant(const float *__restrict__ wm, __bf16 *__restrict__ Wf, __bf16 *__restrict__ Wb, int cin,
                          int coutp, int cout_real, int kp, int kpb)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= coutp * kp) return;
    const int co = i / kp, kappa = i - co * kp;
    const bool live = co < cout_real && kappa < KS * cin;
    const __bf16 v = (__bf16)(live ? wm[i] : 0.0f);
    Wf[frag_at(co, kappa, kp)] = v;
    if (kappa < KS * cin) {
        const int t = kappa / cin, ci = kappa - t * cin;
        Wb[(size_t)ci * kpb + t * coutp + co] = v;
    }
}

// Initial weights: N(0, 1/(5*CIN)) from Philox keyed by (layer, seed).
__global__ void k_init_weights(float *__restrict__ wm, int cin, int coutp, int cout_real, int kp, uint32_t layer,
                               uint32_t seed)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= coutp * kp) return;
    const int co = i / kp, kappa = i - co * kp;
    float v = 0.0f;
    if (co < cout_real && kappa < KS * cin) {
        const uint4 r = philox((uint32_t)i, layer, 7u, 0u, seed, 0x5A11u);
        const float u1 = ((float)(r.x >> 8) + 0.5f) * (1.0f / 16777216.0f);
        const float u2 = ((float)(r.y >> 8) + 0.5f) * (1.0f / 16777216.0f);
        float s, c;
        sincospif(2.0f * u2, &s, &c);
        v = sqrtf(-2.0f * logf(u1)) * c * sqrtf(1.0f / (float)(KS * cin));
    }
    wm[i] = v;
}

// ---------------------------------------------------------------------------
// The whole forward pass in one kernel: features, the six convolutions and
// the conversion to the caller's output.
//
// A block of four waves takes T output positions of one sample.  A layer
// needs two positions more on each side than the next, so the block works on
// T + 20 <= `rows` rows, and each layer's valid rows shrink by two at both
// ends: the hidden activations never leave the block.  They live in LDS
// as bfloat16 rows of 64 channels (two buffers, a layer reads one and writes
// the other), the 16-byte groups of a row permuted by the row's low bits so
// that the 16 rows of a fragment read fall on different banks.
//
// Row r of a hidden layer is position x0 - 10 + r, stored at buffer row
// r + 2; rows outside the sample are stored as zeros (the padding of the next
// layer).  A layer is the GEMM  channels x positions, K = 5 CIN: a wave holds
// C tiles of 16 output channels, their weights for the whole K in registers
// (fragments read straight from global memory, the next layer's requested as
// soon as this layer's products are done), and walks its share of the rows,
// PB tiles of 16 positions at a time.
// The product is taken as weights x activations, so that a lane receives four
// consecutive channels of one position and stores them as one 8-byte LDS
// write; the last layer is taken the other way round, so that a lane has four
// consecutive positions of one channel, the caller's [channel][position]
// order.
//
// Bound by the vector unit (the tanh of 64 samples takes 2/3 of the cycles, the
// matrix cores 1/3), on one sample by the chain of layers.  One kernel per
// layer was bound by its launches and by every activation written and read
// again in FP32 and bfloat16.  Measured (2048 cells, the whole call, before and
// after): 1 sample 53 -> 7.7 us, 8 samples 58 -> 14.3, 64 samples 135 -> 40.3 us
// (650 TFLOP/s).
// ---------------------------------------------------------------------------
struct NetParams {
    const __bf16 *w[6];      // forward weights, fragment order
    const float *bias[6];
};

// the caller's arrays need no more than their elements' alignment
typedef float out_f32x4 __attribute__((__vector_size__(16), aligned(4)));
typedef double out_f64x2 __attribute__((__vector_size__(16), aligned(8)));

enum NetOut { NET_OUT, NET_DENSITIES, NET_STATE, NET_TRAIN };

// What the training step's forward pass keeps and computes besides.
struct NetTrain {
    float *y[5];             // tanh outputs of the hidden layers [b][x][64] (FP32, for the tanh derivative)
    __bf16 *feat;            // [b][x][16]
    const float *target;     // [b][39][x]
    __bf16 *dz;              // gradient of the loss at the output [b][x][48]
    double *loss;            // per block, its share of the loss
    int B;
};

constexpr int NET_THREADS = 256;
constexpr int NET_HALO = 20;     // rows beyond the block's outputs, both sides together

// rows: a multiple of 16 C PB; grid (tiles x samples); LDS 2 (rows + 4) x 64
// bfloat16 and 6 x 64 biases.
template <int C, int MODE>
__device__ __forceinline__ void net_block(const NetParams &np, const float *__restrict__ params,
                                          const double *__restrict__ n0, void *__restrict__ outp, const NetTrain &tr,
                                          int X, int tiles, int T, int rows)
{
    extern __shared__ __align__(16) __bf16 net_lds[];
    constexpr int FS = 24;                         // feature row stride (48 bytes)
    constexpr int PB = 2;                          // position tiles in flight
    constexpr int DEP = 2;                         // fragments in flight per position tile
    const int brows = rows + 4;                    // buffer rows: two spare ones at each end
    const int G = rows / (16 * C * PB);            // groups of PB position tiles per wave
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m = lane & 15, kb = lane >> 4;
    const int cg = w % (4 / C), rw = w / (4 / C) * (G * PB * 16);  // this wave's channel tiles and first row
    const int b = blockIdx.x / tiles;
    const int x0 = (blockIdx.x - b * tiles) * T;
    const int x1 = min(X, x0 + T);                 // the block's own positions: [x0, x1)
    const float *pb = params + (size_t)b * 4;

    bf16x8 W[C][10];                               // a layer's weights
    // unconditional (a wave without a tile in the last layer reads the last
    // one's): a load on one path of a branch would make the compiler wait for
    // every load in flight where the paths meet
    auto load_weights = [&](int l, auto nks) {
        constexpr int NKS = decltype(nks)::value;
        const __bf16 *wf = np.w[l];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int nt = min(cg * C + c, l == 5 ? OUTP / 16 - 1 : 3);
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) W[c][ks] = load8(wf + (nt * NKS + ks) * 512 + (unsigned)(lane * 8));
        }
    };
    using K3 = std::integral_constant<int, 3>;
    using K10 = std::integral_constant<int, 10>;
    load_weights(0, K3{});
    // every layer's biases in LDS: read there, they wait for no weights
    float *bias_lds = reinterpret_cast<float *>(net_lds + 2 * brows * 64);
    for (int i = threadIdx.x; i < 6 * 64; i += NET_THREADS) bias_lds[i] = i < 5 * 64 + OUTP ? np.bias[i >> 6][i & 63] : 0.0f;
    // the features of positions x0 - 12 .. (zero outside the sample), a part per wave
    __bf16 *F = net_lds + brows * 64;
    auto put_features = [&](auto part) {
        constexpr int PART = decltype(part)::value;
        for (int q = lane; q < brows; q += 64) {
            const int x = x0 - 12 + q;
            __bf16 f[16] = {};
            if (x >= 0 && x < X) features_part<PART>(pb, x, X, f);
            uint32_t *o = reinterpret_cast<uint32_t *>(F + q * FS);
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const int of = c < 2 ? 0 : c == 2 ? 3 : c < 5 ? 1 : c == 5 ? 2 : 3;
                if (of == PART) {
                    const bf16x2 v = {f[2 * c], f[2 * c + 1]};
                    o[c] = __builtin_bit_cast(uint32_t, v);
                    if (MODE == NET_TRAIN && x >= x0 && x < x1)
                        *reinterpret_cast<bf16x2 *>(tr.feat + ((size_t)b * X + x) * 16 + 2 * c) = v;
                }
            }
        }
    };
    switch (w) {
    case 0: put_features(std::integral_constant<int, 0>{}); break;
    case 1: put_features(std::integral_constant<int, 1>{}); break;
    case 2: put_features(std::integral_constant<int, 2>{}); break;
    default: put_features(std::integral_constant<int, 3>{}); break;
    }
    // element offset of the lane's 16-byte group of fragment ks in the rows from `first` on
    auto group = [&](int first, int ks) {
        const int q = first + m + (ks >> 1), g = (ks & 1) * 4 + kb;
        return q * 64 + ((g ^ (q & 7)) << 3);
    };
    int off[10];
#pragma unroll
    for (int ks = 0; ks < 10; ++ks) off[ks] = group(0, ks);
    __syncthreads();

    f32x4 bias[C];
    auto load_bias = [&](int l) {
#pragma unroll
        for (int c = 0; c < C; ++c)
            bias[c] = *reinterpret_cast<const f32x4 *>(bias_lds + l * 64 + (cg * C + c) * 16 + kb * 4);
    };
    // bias, tanh, bfloat16, into rows r + 2 of dst; zero outside the sample
    const bool inside = x0 >= 10 && x0 - 10 + rows <= X;      // the block's rows all lie in the sample
    int put[C];                                    // the lane's element offset in row m + 2
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int q = m + 2, g = (cg * C + c) * 2 + (kb >> 1);
        put[c] = q * 64 + ((g ^ (q & 7)) << 3) + (kb & 1) * 4;
    }
    auto activation = [&](int l, __bf16 *dst, const f32x4 (&acc)[C][PB], int r0) {
        __bf16 *row = dst + r0 * 64;
#pragma unroll
        for (int p = 0; p < PB; ++p) {
            const int x = x0 - 10 + r0 + p * 16 + m;
            uint2 h[C];
            if constexpr (MODE == NET_TRAIN) {
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    f32x4 y = acc[c][p] + bias[c];
#pragma unroll
                    for (int i = 0; i < 4; ++i) y[i] = tanhf(y[i]);
                    h[c] = make_uint2(pack_bf16(y[0], y[1]), pack_bf16(y[2], y[3]));
                    if (x >= x0 && x < x1)
                        *reinterpret_cast<f32x4 *>(tr.y[l] + ((size_t)b * X + x) * 64 + (cg * C + c) * 16 + kb * 4) = y;
                }
            } else {
                uint2 open[C];
                uint32_t any = 0;
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    h[c] = tanh4(acc[c][p] + bias[c], open[c]);
                    any |= open[c].x | open[c].y;
                }
                if (__builtin_expect(__any(any), 0)) {
#pragma unroll
                    for (int c = 0; c < C; ++c) tanh4_settle(acc[c][p] + bias[c], open[c], h[c]);
                }
            }
            if (!inside && (x < 0 || x >= X)) {
#pragma unroll
                for (int c = 0; c < C; ++c) h[c] = make_uint2(0u, 0u);
            }
#pragma unroll
            for (int c = 0; c < C; ++c) *reinterpret_cast<uint2 *>(row + p * 1024 + put[c]) = h[c];
        }
    };
    // the wave's groups that any output depends on
    const int groups = min(G, max(0, (T + NET_HALO - rw + PB * 16 - 1) / (PB * 16)));

    f32x4 acc[C][PB];
    auto first_products = [&](int r0) {
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int p = 0; p < PB; ++p) acc[c][p] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 3; ++ks) {
            const int kappa = ks * 32 + kb * 8;
#pragma unroll
            for (int p = 0; p < PB; ++p) {
                // row r reads the features of positions x - 2 .. x + 2: rows r .. r + 4
                const bf16x8 a = kappa < 80 ? load8(F + (r0 + p * 16 + m + (kappa >> 4)) * FS + (kappa & 15)) : zero8();
#pragma unroll
                for (int c = 0; c < C; ++c)
                    acc[c][p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[c][ks], a, acc[c][p], 0, 0, 0);
            }
        }
    };
    // K = 5 x 64 over the rows of src from r0 on: DEP fragments per position
    // tile in flight ahead of the matrix cores
    auto products = [&](const __bf16 *src, int r0) {
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int p = 0; p < PB; ++p) acc[c][p] = (f32x4){0.f, 0.f, 0.f, 0.f};
        bf16x8 a[DEP][PB];
        const __bf16 *row = src + r0 * 64;
#pragma unroll
        for (int ks = 0; ks < DEP; ++ks)
#pragma unroll
            for (int p = 0; p < PB; ++p) a[ks][p] = load8(row + p * 1024 + off[ks]);
        __builtin_amdgcn_sched_group_barrier(0x100, DEP * PB, 0);
#pragma unroll
        for (int ks = 0; ks < 10; ++ks) {
#pragma unroll
            for (int p = 0; p < PB; ++p)
#pragma unroll
                for (int c = 0; c < C; ++c)
                    acc[c][p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[c][ks], a[ks % DEP][p], acc[c][p], 0, 0, 0);
            __builtin_amdgcn_sched_group_barrier(0x8, C * PB, 0);
            if (ks + DEP < 10) {
#pragma unroll
                for (int p = 0; p < PB; ++p) a[ks % DEP][p] = load8(row + p * 1024 + off[ks + DEP]);
                __builtin_amdgcn_sched_group_barrier(0x100, PB, 0);
            }
        }
    };

    load_bias(0);
#pragma unroll 1
    for (int g = 0; g < groups - 1; ++g) {
        first_products(rw + g * PB * 16);
        activation(0, net_lds, acc, rw + g * PB * 16);
    }
    const int last = rw + max(groups - 1, 0) * PB * 16;      // the wave's last group
    first_products(last);
    load_weights(1, K10{});
    activation(0, net_lds, acc, last);
    __syncthreads();
#pragma unroll 1
    for (int l = 1; l < 5; ++l) {
        const __bf16 *src = net_lds + ((l - 1) & 1) * brows * 64;
        __bf16 *dst = net_lds + (l & 1) * brows * 64;
        load_bias(l);
#pragma unroll 1
        for (int g = 0; g < groups - 1; ++g) {
            products(src, rw + g * PB * 16);
            activation(l, dst, acc, rw + g * PB * 16);
        }
        products(src, last);
        load_weights(l + 1, K10{});      // their registers are free: the next layer's, beside the activation
        activation(l, dst, acc, last);
        __syncthreads();
    }
    // the last layer: row s is output position x0 + s, its inputs rows s + 10 .. s + 14
#pragma unroll
    for (int ks = 0; ks < 10; ++ks) off[ks] = group(10, ks);
    const double inv = MODE == NET_TRAIN ? 1.0 / ((double)OUT * (double)X * (double)tr.B) : 0.0;
    double sq = 0.0;                     // training: the lane's sum of (out - target)^2
#pragma unroll 1
    for (int g = 0; g < G; ++g) {
        const int s0 = rw + g * PB * 16;
        if (s0 >= T) break;
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int p = 0; p < PB; ++p) acc[c][p] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 10; ++ks) {
#pragma unroll
            for (int p = 0; p < PB; ++p) {
                if (s0 + p * 16 >= T) continue;      // the buffer's rows end at T + 24
                const bf16x8 a = load8(net_lds + (s0 + p * 16) * 64 + off[ks]);
#pragma unroll
                for (int c = 0; c < C; ++c)
                    if (cg * C + c < OUTP / 16) {
                        if constexpr (MODE == NET_TRAIN)     // four channels of a position per lane, as dz is laid out
                            acc[c][p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W[c][ks], a, acc[c][p], 0, 0, 0);
                        else
                            acc[c][p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, W[c][ks], acc[c][p], 0, 0, 0);
                    }
            }
        }
        if constexpr (MODE == NET_TRAIN) {
            // dz = 2 (out - target) / count in bfloat16, zero in the padding channels
#pragma unroll
            for (int p = 0; p < PB; ++p) {
                const int s = s0 + p * 16 + m, x = x0 + s;
                if (s >= T || x >= X) continue;
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    const int co = (cg * C + c) * 16 + kb * 4;
                    if (co >= OUTP) continue;
                    float dg[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        dg[i] = 0.0f;
                        if (co + i < OUT) {
                            const float d = acc[c][p][i] + bias_lds[5 * 64 + co + i] -
                                            tr.target[((size_t)b * OUT + co + i) * X + x];
                            sq += (double)d * d;
                            dg[i] = (float)(2.0 * inv) * d;
                        }
                    }
                    *reinterpret_cast<uint2 *>(tr.dz + ((size_t)b * X + x) * OUTP + co) =
                        make_uint2(pack_bf16(dg[0], dg[1]), pack_bf16(dg[2], dg[3]));
                }
            }
            continue;
        }
#pragma unroll
        for (int p = 0; p < PB; ++p) {
            const int s = s0 + p * 16 + kb * 4, x = x0 + s;     // four positions (T and X are multiples of 4)
            if (s >= T || x >= X) continue;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const int co = (cg * C + c) * 16 + m;
                if (co >= OUT) continue;
                const float bc = bias_lds[5 * 64 + co];
                const f32x4 v = acc[c][p] + (f32x4){bc, bc, bc, bc};
                if constexpr (MODE == NET_OUT) {
                    *reinterpret_cast<out_f32x4 *>(static_cast<float *>(outp) + ((size_t)b * OUT + co) * X + x) = v;
                } else {
                    // densities n0 exp(out[1]), n0 exp(out[2]); phi = V out[0]; the electron quantiles
                    // (channels 3..20) times the 1 eV electron speed sqrt(e / m_e), the ion ones (21..38)
                    // times the 1 eV ion speed sqrt(e / m_i)
                    if (MODE == NET_DENSITIES && co != 1 && co != 2) continue;
                    double d[4] = {v[0], v[1], v[2], v[3]};
                    if (co == 1 || co == 2) {
                        const double n = n0[b];
#pragma unroll
                        for (int i = 0; i < 4; ++i) d[i] = n * exp(d[i]);
                    } else {
                        const double ve = sqrt(1.602176634e-19 / 9.1093837015e-31);
                        const double vi = sqrt(1.602176634e-19 / (6.6464731e-27 - 9.1093837015e-31));
                        const double f = co == 0 ? (double)pb[2] : co < 21 ? ve : vi;
#pragma unroll
                        for (int i = 0; i < 4; ++i) d[i] *= f;
                    }
                    const int row = co == 0 ? 2 : co < 3 ? co - 1 : co, rows = MODE == NET_STATE ? OUT : 2;
                    out_f64x2 *o = reinterpret_cast<out_f64x2 *>(static_cast<double *>(outp) +
                                                                 ((size_t)b * rows + row) * X + x);
                    o[0] = (out_f64x2){d[0], d[1]};
                    o[1] = (out_f64x2){d[2], d[3]};
                }
            }
        }
    }
    if constexpr (MODE == NET_TRAIN) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) sq += __shfl_xor(sq, o, 64);
        __syncthreads();                 // the biases' place is free
        double *red = reinterpret_cast<double *>(bias_lds);
        if (lane == 0) red[w] = sq;
        __syncthreads();
        if (threadIdx.x == 0) tr.loss[blockIdx.x] = ((red[0] + red[1]) + (red[2] + red[3])) * inv;
    }
}

template <int C, int MODE>
__global__ __launch_bounds__(NET_THREADS, 3) void k_net(NetParams np, const float *__restrict__ params,
                                                        const double *__restrict__ n0, void *__restrict__ outp, int X,
                                                        int tiles, int T, int rows)
{
    net_block<C, MODE>(np, params, n0, outp, NetTrain{}, X, tiles, T, rows);
}

// The training step's forward pass.  Bound by the vector unit: the FP32 hidden
// outputs, kept for the backward pass, take tanhf itself (13 us of 50 at 32
// samples x 2048 cells; storing them 3).  With the loss inside it takes the
// place of eight launches: 83 us, every activation written twice and read once.
__global__ __launch_bounds__(NET_THREADS, 3) void k_net_train(NetParams np, const float *__restrict__ params,
                                                              NetTrain tr, int X, int tiles, int T, int rows)
{
    net_block<1, NET_TRAIN>(np, params, nullptr, nullptr, tr, X, tiles, T, rows);
}


}  // namespace sur

// ---------------------------------------------------------------------------
// Launch wrappers
// ---------------------------------------------------------------------------
using namespace sur;

// backward pass of layer `layer` (grid: batch x slices): layers 1..5 take the
// FP32 input y (the layer below's output) and write the layer below's output
// gradient dzprev; layer 0 takes the features and has no input gradient
extern "C" hipError_t surx_conv_bwd(int layer, const __bf16 *dz, const float *yin, const __bf16 *feat,
                                    const __bf16 *Wb, __bf16 *dzprev, float *part, float *pbias, int X, int B,
                                    hipStream_t s)
{
    const dim3 g((unsigned)(B * ((X + BW_SLICE - 1) / BW_SLICE))), t(BW_THREADS);
    if (layer == 0)
        hipLaunchKernelGGL((k_conv_bwd<16, 64, false>), g, t, 0, s, dz, yin, feat, Wb, dzprev, part, pbias, X);
    else if (layer < 5)
        hipLaunchKernelGGL((k_conv_bwd<64, 64, true>), g, t, 0, s, dz, yin, feat, Wb, dzprev, part, pbias, X);
    else
        hipLaunchKernelGGL((k_conv_bwd<64, OUTP, true>), g, t, 0, s, dz, yin, feat, Wb, dzprev, part, pbias, X);
    return hipGetLastError();
}

extern "C" int surx_wgrad_parts(int X, int B) { return B * ((X + BW_SLICE - 1) / BW_SLICE); }

// Adam over `layers` layers (the fields of AdamLayer but `first`, per layer)
// and, where a place for it is given, the loss from the forward blocks' shares.
extern "C" hipError_t surx_reduce_adam(int layers, const float *const *part, const float *const *pbias, int P, float *const *wm,
                                       float *const *mw, float *const *vw, float *const *dw, float *const *bias,
                                       float *const *mb, float *const *vb, float *const *db, __bf16 *const *Wf,
                                       __bf16 *const *Wb, const int *cin, const int *coutp, const int *cout_real,
                                       const int *kp, const int *kpb, const double *loss_parts, int nloss,
                                       double *loss, float lr, float b1, float b2, float eps, float c1, float c2,
                                       hipStream_t s)
{
    AdamArgs A;
    int blocks = 0;
    for (AdamLayer &L : A.L) L.first = INT_MAX;
    for (int l = 0; l < layers; ++l) {
        A.L[l] = AdamLayer{part[l], pbias[l], wm[l], mw[l], vw[l], dw[l], bias[l], mb[l], vb[l], db[l], Wf[l], Wb[l],
                           cin[l], coutp[l], cout_real[l], kp[l], kpb[l], blocks};
        blocks += (coutp[l] * kp[l] + coutp[l] + 63) / 64;
    }
    A.P = P;
    A.blocks = blocks;
    A.loss_parts = loss_parts;
    A.nloss = nloss;
    A.loss = loss;
    A.lr = lr;
    A.b1 = b1;
    A.b2 = b2;
    A.eps = eps;
    A.c1 = c1;
    A.c2 = c2;
    hipLaunchKernelGGL(k_reduce_adam, dim3(blocks + (loss ? 1 : 0)), dim3(RA_WAVES * 64), 0, s, A);
    return hipGetLastError();
}

extern "C" hipError_t surx_requant(const float *wm, __bf16 *Wf, __bf16 *Wb, int cin, int coutp, int cout_real, int kp,
                                   int kpb, hipStream_t s)
{
    const int n = coutp * kp;
    hipLaunchKernelGGL(k_requant, dim3((n + 255) / 256), dim3(256), 0, s, wm, Wf, Wb, cin, coutp, cout_real, kp, kpb);
    return hipGetLastError();
}

extern "C" hipError_t surx_init_weights(float *wm, int cin, int coutp, int cout_real, int kp, uint32_t layer,
                                        uint32_t seed, hipStream_t s)
{
    const int n = coutp * kp;
    hipLaunchKernelGGL(k_init_weights, dim3((n + 255) / 256), dim3(256), 0, s, wm, cin, coutp, cout_real, kp, layer,
                       seed);
    return hipGetLastError();
}

constexpr int NET_CUS = 256;

// Rows per block of a network launch, at most `most`: few rows give many short
// blocks, but 20 of them are halo computed again by the neighbours.  A call
// takes about the longer of a block's chain of layers, 4.5 us + 0.105 us a
// row, and the work of the most loaded CU, 5 us + 0.064 us x (rows + 8) x its
// blocks; the rows with the least of it are taken.  Measured on the forward
// pass (2048 cells; 32 / 64 / 128 / 192 rows, us): 1 sample 7.9 / 11.5 / 18 /
// 22, 8 samples 19 / 15.4 / 20 / 24, 32 samples 63 / 34 / 32 / 33, 64 samples
// 113 / 60 / 50 / 43.  160 rows give 32 samples two blocks per CU, where 128
// need three and 192 carry more halo: 28.8 against 31.2 us.
static int net_rows(int X, int B, int most)
{
    int rows = 0;
    double best = 0.0;
    for (int r : {32, 64, 96, 128, 160, 192}) {
        if (r > most) break;
        const long long blocks = (long long)((X + r - NET_HALO - 1) / (r - NET_HALO)) * B;
        const long long per_cu = (blocks + NET_CUS - 1) / NET_CUS;
        const double chain = 4.5 + 0.105 * r, work = 5.0 + 0.064 * (double)per_cu * (r + 8);
        const double t = chain > work ? chain : work;
        if (!rows || t < best) {
            rows = r;
            best = t;
        }
    }
    return rows;
}

struct NetShape {
    int rows, tiles, T;
    unsigned grid;
    size_t lds;
};

static NetShape net_shape(int X, int B, int rows)
{
    NetShape n;
    n.rows = rows;
    // equal tiles, a multiple of 4 positions each
    n.tiles = (X + rows - NET_HALO - 1) / (rows - NET_HALO);
    n.T = ((X + n.tiles - 1) / n.tiles + 3) / 4 * 4;
    n.grid = (unsigned)n.tiles * (unsigned)B;
    n.lds = (size_t)2 * (rows + 4) * 64 * sizeof(__bf16) + 6 * 64 * sizeof(float);
    return n;
}

static NetParams net_params(const __bf16 *const *wf, const float *const *bias)
{
    NetParams np;
    for (int l = 0; l < 6; ++l) {
        np.w[l] = wf[l];
        np.bias[l] = bias[l];
    }
    return np;
}

template <int C>
static hipError_t launch_net(const NetParams &np, int mode, const float *params, const double *n0, void *out, int X,
                             const NetShape &n, hipStream_t s)
{
    auto *kernel = mode == NET_OUT ? k_net<C, NET_OUT> : mode == NET_DENSITIES ? k_net<C, NET_DENSITIES>
                                                                              : k_net<C, NET_STATE>;
    hipLaunchKernelGGL(kernel, dim3(n.grid), dim3(NET_THREADS), n.lds, s, np, params, n0, out, X, n.tiles, n.T, n.rows);
    return hipGetLastError();
}

// Forward pass of B samples into the caller's output: mode 0 the network's
// channels [b][39][x] (float), 1 densities [b][2][x], 2 the loader's state
// [b][39][x] (double; n0 per sample).  192 rows take two channel tiles per
// wave, which halves the reads of the activations (with one tile per wave 10 %
// slower there, and no faster on fewer rows).
extern "C" hipError_t surx_net(const __bf16 *const *wf, const float *const *bias, int mode, const float *params,
                               const double *n0, void *out, int X, int B, hipStream_t s)
{
    const NetParams np = net_params(wf, bias);
    const NetShape n = net_shape(X, B, net_rows(X, B, 192));
    return n.rows == 192 ? launch_net<2>(np, mode, params, n0, out, X, n, s)
                         : launch_net<1>(np, mode, params, n0, out, X, n, s);
}

// blocks of the training step's forward pass at most, one share of the loss each
extern "C" int surx_net_train_blocks(int X, int B) { return (X + 32 - NET_HALO - 1) / (32 - NET_HALO) * B; }

// The training step's forward pass: hidden outputs, features, the gradient at
// the output and *blocks shares of the loss.
extern "C" hipError_t surx_net_train(const __bf16 *const *wf, const float *const *bias, const float *params,
                                     const float *target, float *const *y, __bf16 *feat, __bf16 *dz, double *loss,
                                     int *blocks, int X, int B, hipStream_t s)
{
    NetTrain tr;
    for (int l = 0; l < 5; ++l) tr.y[l] = y[l];
    tr.feat = feat;
    tr.target = target;
    tr.dz = dz;
    tr.loss = loss;
    tr.B = B;
    // one channel tile per wave throughout: with two (and 192 rows) the step of
    // 32 samples x 2048 cells took 164 us, with 128 or 160 rows and one 154
    const NetShape n = net_shape(X, B, net_rows(X, B, 128));
    *blocks = (int)n.grid;
    hipLaunchKernelGGL(k_net_train, dim3(n.grid), dim3(NET_THREADS), n.lds, s, net_params(wf, bias), params, tr, X,
                       n.tiles, n.T, n.rows);
    return hipGetLastError();
}
