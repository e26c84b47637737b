// Fused kernels of the surrogate's forward pass at its usual widths (C = 32 or
// 64, up to 16 modes).  They form the same products in the same order as the
// general GEMM path of sno.hip (BF16 operands rounded where they are staged,
// one chain of 16x16x32 MFMA over ascending k per output, FP32 in memory), so
// outputs and gradients agree with it bit for bit (the error estimates' sums
// over time run in another order); what they save is passes over memory,
// launches and idle compute units.
#pragma once
#include <hip/hip_runtime.h>

#include "sno.h"

namespace snof {

typedef short s4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f4 mma(bf8 a, bf8 b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }

__device__ __forceinline__ bf8 cvt8(float4 a, float4 b)
{
    return bf8{(__bf16)a.x, (__bf16)a.y, (__bf16)a.z, (__bf16)a.w, (__bf16)b.x, (__bf16)b.y, (__bf16)b.z, (__bf16)b.w};
}
__device__ __forceinline__ bf4 cvt4(float a, float b, float c, float d) { return bf4{(__bf16)a, (__bf16)b, (__bf16)c, (__bf16)d}; }
__device__ __forceinline__ float4 ld4(const float* p) { return *reinterpret_cast<const float4*>(p); }

// ---------------------------------------------------------------------------
// Lift: V[b][c][t] = sum_i P[c][i] A[b][i][t] + pb[c] with the lift inputs A
// (see sno.hip: position, t / T, cos and sin features, position products)
// formed where they are staged instead of in a pass of their own.  Every input
// is a factor that depends on the sample (1 or a position feature) times a
// series that does not: rows of the table tab (all ones; t / T; the cosines and
// sines), laid out once.  meta[k] = row | factor << 16 names both for channel
// k (factor 3: 1; 4: 0, the channels that fill the last slice).  A block takes
// 64 time samples of one sample; its tile of the table stays in LDS.  Aout
// (may be null) also receives A for the backward pass.  256 samples, 260
// channels to 64: 55 us (the feature pass and the product took 350 us).
struct LiftP {
    const float* X;      // [B][9]
    const float* P;      // [C][NA]
    const float* pb;     // [C]
    const float* tab;    // [rows][T]
    const int* meta;     // [NA rounded up to 32]
    float off[3], inv[3];
    int NA, rows, T, TS;
    float* Aout;         // [B][NA][TS] or null
    float* V;            // [B][C][TS]
};
constexpr int LIFT_NA = 544;   // channels at SNO_MAX_FOUR frequencies with position products, in whole slices of 32
static_assert(LIFT_NA >= (4 + 8 * SNO_MAX_FOUR + 31) / 32 * 32, "the channels' rows and factors fit LDS");

template <int C>
__global__ __launch_bounds__(256) void k_lift(LiftP p)
{
    constexpr int LD = 40;   // 32 k and 8 spare: 16-byte reads of 16 rows without bank conflicts
    __shared__ __attribute__((aligned(16))) __bf16 As[2][64][LD];
    __shared__ __attribute__((aligned(16))) __bf16 Ps[2][C][LD];
    __shared__ int rk[LIFT_NA];
    __shared__ float fk[LIFT_NA];
    extern __shared__ float tab_s[];   // [rows][64]
    const int b = blockIdx.y, t0 = blockIdx.x * 64;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int T = p.T, NA = p.NA;
    for (int e = tid; e < p.rows * 16; e += 256)
        *reinterpret_cast<float4*>(tab_s + 4 * e) = ld4(p.tab + (long)(e >> 4) * T + t0 + (e & 15) * 4);
    float px[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) px[i] = (p.X[b * 9 + i] - p.off[i]) * p.inv[i];
    for (int k = tid; k < (NA + 31) / 32 * 32; k += 256) {
        const int m = p.meta[k], a = m >> 16;
        rk[k] = (m & 0xffff) * 64;
        fk[k] = a == 0 ? px[0] : a == 1 ? px[1] : a == 2 ? px[2] : a == 3 ? 1.f : 0.f;
    }
    f4 acc[C / 16];
#pragma unroll
    for (int j = 0; j < C / 16; ++j) acc[j] = f4{0.f, 0.f, 0.f, 0.f};
    const int kq = w * 8;   // this thread's inputs: time t0 + lane, 8 channels per slice
    const int pr = tid >> 2, pk = (tid & 3) * 8;
    float4 wa, wb;
    // weights of a slice, one slice ahead.  NA is a multiple of 4: each float4
    // is inside or outside, and outside the inputs are zero
    auto load = [&](int k0) {
        if (pr < C) {
            wa = ld4(p.P + (long)pr * NA + min(k0 + pk, NA - 4));
            wb = ld4(p.P + (long)pr * NA + min(k0 + pk + 4, NA - 4));
        }
    };
    load(0);
    __syncthreads();
    int buf = 0;
    for (int k0 = 0; k0 < NA; k0 += 32, buf ^= 1) {
        float v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = fk[k0 + kq + i] * tab_s[rk[k0 + kq + i] + lane];
        if (p.Aout)
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (k0 + kq + i < NA) p.Aout[((long)b * NA + k0 + kq + i) * p.TS + t0 + lane] = v[i];
        *reinterpret_cast<bf8*>(&As[buf][lane][kq]) =
            cvt8(make_float4(v[0], v[1], v[2], v[3]), make_float4(v[4], v[5], v[6], v[7]));
        if (pr < C) {
            const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
            *reinterpret_cast<bf8*>(&Ps[buf][pr][pk]) = cvt8(k0 + pk < NA ? wa : z, k0 + pk + 4 < NA ? wb : z);
        }
        load(k0 + 32);
        __syncthreads();
        const bf8 av = *reinterpret_cast<const bf8*>(&As[buf][w * 16 + (lane & 15)][8 * (lane >> 4)]);
#pragma unroll
        for (int j = 0; j < C / 16; ++j)
            acc[j] = mma(av, *reinterpret_cast<const bf8*>(&Ps[buf][j * 16 + (lane & 15)][8 * (lane >> 4)]), acc[j]);
    }
#pragma unroll
    for (int j = 0; j < C / 16; ++j) {
        const int c = j * 16 + (lane & 15);
        const float bc = p.pb[c];
        *reinterpret_cast<float4*>(p.V + ((long)b * C + c) * p.TS + t0 + w * 16 + 4 * (lane >> 4)) =
            make_float4(acc[j][0] + bc, acc[j][1] + bc, acc[j][2] + bc, acc[j][3] + bc);
    }
}

// ---------------------------------------------------------------------------
constexpr float GELU_C = 0.7978845608028654f;   // sqrt(2 / pi)

__device__ __forceinline__ float gelu_f(float x)
{
    return 0.5f * x * (1.f + tanhf(GELU_C * (x + 0.044715f * x * x * x)));
}
__device__ __forceinline__ float gelu_d(float x)
{
    const float th = tanhf(GELU_C * (x + 0.044715f * x * x * x));
    return 0.5f * (1.f + th) + 0.5f * x * (1.f - th * th) * GELU_C * (1.f + 3.f * 0.044715f * x * x);
}

// Truncated DFT along time: Vh[b][c][q] = sum_t V[b][c][t] Ft[q][t], q < K2.
// The sum is one chain of MFMA over ascending t, so what the kernel can do is
// keep memory busy around it: a block takes 16 channels of one sample, its 256
// threads load TC time samples of V and of the transposed basis at once,
// round them into LDS in operand order, and while two waves run the chain over
// them (one per 16 columns) the next TC are on their way.  KS: k per MFMA, 32,
// or 16 where K2 < 32 (the general path's choice there).  SUM: Ft is given per
// sample, [B][K2][T], and the chain runs on over the samples to Vh[c][q] (a
// narrow weight gradient).
// 16 x 1024 by 32 columns, one sample: 4.7 us (26 us as a general 64 x 64
// tile, one block per sample, one slice in flight); 256 samples 22 us, 3 TB/s.
template <int KS, int TC, bool SUM>
__global__ __launch_bounds__(256) void k_dft(const float* __restrict__ V, const float* __restrict__ Ft, int B, int C,
                                             int T, int TS, int K2, float* __restrict__ Vh)
{
    // operand chunks of KS / 4 values (one lane's k of a slice) by 16 rows,
    // with spare bytes so that the stores of one row spread over the banks
    constexpr int CH = KS / 4, ST = 16 * CH + 8, NCH = TC / CH;
    __shared__ __attribute__((aligned(16))) __bf16 As[NCH * ST];
    __shared__ __attribute__((aligned(16))) __bf16 Bs[2][NCH * ST];
    constexpr int VA = TC / 64, VB = TC / 32;   // float4 per thread
    const int b = blockIdx.y, c0 = blockIdx.x * 16;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, r = lane & 15, g = lane >> 4;
    float4 va[VA], vb[VB];
    auto load = [&](int b, int t) {
        const long base = ((long)b * C + c0) * TS;
        const float* __restrict__ F = Ft + (SUM ? (long)b * K2 * T : 0L);
#pragma unroll
        for (int i = 0; i < VA; ++i) {
            const int e = tid + i * 256, row = e / (TC / 4), q = (e % (TC / 4)) * 4;
            va[i] = ld4(V + base + (long)row * TS + t + q);
        }
#pragma unroll
        for (int i = 0; i < VB; ++i) {
            const int e = tid + i * 256, row = e / (TC / 4), q = (e % (TC / 4)) * 4;
            vb[i] = ld4(F + (long)min(row, K2 - 1) * T + t + q);   // rows past K2 are not stored
        }
    };
    f4 acc = {0.f, 0.f, 0.f, 0.f};
    const int b_hi = SUM ? B - 1 : b;
    load(b, 0);
    for (int bb = b, t = 0; bb <= b_hi;) {   // T is a multiple of TC
        if (bb > b || t > 0) __syncthreads();
#pragma unroll
        for (int i = 0; i < VA; ++i) {
            const int e = tid + i * 256, row = e / (TC / 4), q = (e % (TC / 4)) * 4;
            *reinterpret_cast<bf4*>(As + q / CH * ST + row * CH + q % CH) = cvt4(va[i].x, va[i].y, va[i].z, va[i].w);
        }
#pragma unroll
        for (int i = 0; i < VB; ++i) {
            const int e = tid + i * 256, row = e / (TC / 4), q = (e % (TC / 4)) * 4;
            *reinterpret_cast<bf4*>(Bs[row >> 4] + q / CH * ST + (row & 15) * CH + q % CH) =
                cvt4(vb[i].x, vb[i].y, vb[i].z, vb[i].w);
        }
        t += TC;
        if (SUM && t == T) {
            t = 0;
            ++bb;
        }
        load(min(bb, b_hi), min(t, T - TC));
        if (!SUM && t == T) ++bb;
        __syncthreads();
        if (w < 2 && w * 16 < K2) {
#pragma unroll 8
            for (int s = 0; s < TC / KS; ++s) {
                const __bf16 *x = As + (s * 4 + g) * ST + r * CH, *y = Bs[w] + (s * 4 + g) * ST + r * CH;
                if constexpr (KS == 32)
                    acc = mma(*reinterpret_cast<const bf8*>(x), *reinterpret_cast<const bf8*>(y), acc);
                else
                    acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(*reinterpret_cast<const s4*>(x),
                                                                    *reinterpret_cast<const s4*>(y), acc, 0, 0, 0);
            }
        }
    }
    if (w < 2 && w * 16 + r < K2)
#pragma unroll
        for (int i = 0; i < 4; ++i) Vh[((long)b * C + c0 + 4 * g + i) * K2 + w * 16 + r] = acc[i];
}

template <int KS, bool SUM = false>
inline void launch_dft(hipStream_t st, int B, const float* V, const float* Ft, int C, int T, int TS, int K2, float* Vh)
{
    const dim3 grid(C / 16, SUM ? 1 : B);
    if (T % 512 == 0) hipLaunchKernelGGL((k_dft<KS, 512, SUM>), grid, dim3(256), 0, st, V, Ft, B, C, T, TS, K2, Vh);
    else hipLaunchKernelGGL((k_dft<KS, 128, SUM>), grid, dim3(256), 0, st, V, Ft, B, C, T, TS, K2, Vh);
}

// ---------------------------------------------------------------------------
// Per-mode complex mixing U_k = M_k V_k (HERM: the conjugate transpose), FP32,
// the sum over q ascending as one chain of FMA per output.  A block takes one
// mode, 32 output channels and MB samples, one output per thread, so that a
// batch of 16 to 64 samples fills the chip (one block per mode left all but 16
// compute units idle: 38 us for 32 samples, now 13 us for 256).  Rows of M are
// staged transposed (stride 33: no bank conflicts).
constexpr int MB = 8;

template <int C, bool HERM>
__device__ __forceinline__ void cmix_block(const float* __restrict__ Rr, const float* __restrict__ Ri,
                                           const float* __restrict__ V, int B, int K, float* __restrict__ U, int k,
                                           int b0, int c0, float* sm)
{
    float(*mr)[33] = reinterpret_cast<float(*)[33]>(sm);                 // [q][c - c0]
    float(*mi)[33] = reinterpret_cast<float(*)[33]>(sm + C * 33);
    float(*vr)[C] = reinterpret_cast<float(*)[C]>(sm + 2 * C * 33);      // [b - b0][q]
    float(*vi)[C] = reinterpret_cast<float(*)[C]>(sm + 2 * C * 33 + MB * C);
    const int tid = threadIdx.x;
    const long K2 = 2L * K;
    const int nb = min(MB, B - b0);
    const float* __restrict__ rr = Rr + (long)k * C * C;
    const float* __restrict__ ri = Ri + (long)k * C * C;
    for (int e = tid; e < 32 * C; e += 256) {
        int q, c;
        long at;
        if (HERM) {
            c = e & 31;
            q = e >> 5;
            at = (long)q * C + c0 + c;
        } else {
            q = e % C;
            c = e / C;
            at = (long)(c0 + c) * C + q;
        }
        mr[q][c] = rr[at];
        mi[q][c] = HERM ? -ri[at] : ri[at];
    }
    for (int e = tid; e < nb * C; e += 256) {
        const int b = e / C, q = e % C;
        const long row = ((long)(b0 + b) * C + q) * K2 + k;
        vr[b][q] = V[row];
        vi[b][q] = V[row + K];
    }
    __syncthreads();
    const int c = tid & 31, b = tid >> 5;
    if (b < nb) {
        float ur = 0.f, ui = 0.f;
#pragma unroll 8
        for (int q = 0; q < C; ++q) {
            const float a = mr[q][c], bb = mi[q][c];
            const float xr = vr[b][q], xi = vi[b][q];
            ur = fmaf(a, xr, fmaf(-bb, xi, ur));
            ui = fmaf(bb, xr, fmaf(a, xi, ui));
        }
        const long row = ((long)(b0 + b) * C + c0 + c) * K2 + k;
        U[row] = ur;
        U[row + K] = ui;
    }
}

template <int C>
constexpr int cmix_lds() { return 2 * C * 33 + 2 * MB * C; }

template <int C>
__global__ __launch_bounds__(256) void k_cmix_f(const float* __restrict__ Rr, const float* __restrict__ Ri,
                                                const float* __restrict__ V, int B, int K, float* __restrict__ U)
{
    __shared__ float sm[cmix_lds<C>()];
    cmix_block<C, false>(Rr, Ri, V, B, K, U, blockIdx.x, blockIdx.y * MB, blockIdx.z * 32, sm);
}

// Gradient of the mixing weights of mode k, rows c0 to c0 + DWC, summed over the
// samples (ascending, one chain of FMA per output):
// dRr[c][q] = sum_b dUr[b][c] Vr[b][q] + dUi[b][c] Vi[b][q],
// dRi[c][q] = sum_b dUi[b][c] Vr[b][q] - dUr[b][c] Vi[b][q].
constexpr int DWC = 16, DWB = 32;

template <int C>
__device__ __forceinline__ void cmix_dw_block(const float* __restrict__ dU, const float* __restrict__ V, int B, int K,
                                              float* __restrict__ dRr, float* __restrict__ dRi, int k, int c0, float* sm)
{
    float(*ur)[DWC] = reinterpret_cast<float(*)[DWC]>(sm);
    float(*ui)[DWC] = reinterpret_cast<float(*)[DWC]>(sm + DWB * DWC);
    float(*vr)[C] = reinterpret_cast<float(*)[C]>(sm + 2 * DWB * DWC);
    float(*vi)[C] = reinterpret_cast<float(*)[C]>(sm + 2 * DWB * DWC + DWB * C);
    constexpr int PER = DWC * C / 256;
    const int tid = threadIdx.x, q = tid % C, cq = tid / C * PER;
    const long K2 = 2L * K;
    float ar[PER], ai[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) ar[j] = ai[j] = 0.f;
    for (int b0 = 0; b0 < B; b0 += DWB) {
        const int nb = min(DWB, B - b0);
        __syncthreads();
        for (int e = tid; e < nb * C; e += 256) {
            const int b = e / C, r = e % C;
            const long at = ((long)(b0 + b) * C + r) * K2 + k;
            vr[b][r] = V[at];
            vi[b][r] = V[at + K];
        }
        for (int e = tid; e < nb * DWC; e += 256) {
            const int b = e / DWC, r = e % DWC;
            const long at = ((long)(b0 + b) * C + c0 + r) * K2 + k;
            ur[b][r] = dU[at];
            ui[b][r] = dU[at + K];
        }
        __syncthreads();
        for (int b = 0; b < nb; ++b) {
            const float yr = vr[b][q], yi = vi[b][q];
#pragma unroll
            for (int j = 0; j < PER; ++j) {
                const float xr = ur[b][cq + j], xi = ui[b][cq + j];
                ar[j] = fmaf(xr, yr, fmaf(xi, yi, ar[j]));
                ai[j] = fmaf(xi, yr, fmaf(-xr, yi, ai[j]));
            }
        }
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const long at = ((long)k * C + c0 + cq + j) * C + q;
        dRr[at] = ar[j];
        dRi[at] = ai[j];
    }
}

// Backward mixing: grid (K, nmix + C / DWC), the first nmix blocks of a mode
// form dV = M^H dU (as k_cmix_f), the others the weight gradients.  16 samples
// of width 64: 128 blocks instead of two launches of 16 (46 us).
template <int C>
__global__ __launch_bounds__(256) void k_cmix_b(const float* __restrict__ Rr, const float* __restrict__ Ri,
                                                const float* __restrict__ dU, const float* __restrict__ Vh, int B, int K,
                                                int nmix, float* __restrict__ dVh, float* __restrict__ dRr,
                                                float* __restrict__ dRi)
{
    constexpr int N0 = cmix_lds<C>(), N1 = 2 * DWB * (DWC + C);
    __shared__ float sm[N0 > N1 ? N0 : N1];
    const int y = blockIdx.y;
    if (y < nmix) cmix_block<C, true>(Rr, Ri, dU, B, K, dVh, blockIdx.x, y / (C / 32) * MB, y % (C / 32) * 32, sm);
    else cmix_dw_block<C>(dU, Vh, B, K, dRr, dRi, blockIdx.x, (y - nmix) * DWC, sm);
}

// ---------------------------------------------------------------------------
// Pointwise map, inverse DFT of the mixed modes and activation of one layer:
//   Z[b][c][t] = (sum_q W[c][q] V[b][q][t] + bias[c]) + sum_k Uh[b][c][k] Gt[t][k]
//   Vn = gelu(Z)
// for 64 time samples of one sample per block; either output may be null.
// pool (last layer, may be null): pool[b][blockIdx.x][c] = sum over the
// block's 64 t of Z.  TRW: W is read transposed, and Z is multiplied by
// gelu'(Zp) if Zp is given (the backward pass; Zp may be Z: a thread reads a
// value before it writes it).  Bound
// by memory (V read, Vn written): 256 samples of width 64 in 38 us, 3.5 TB/s;
// as two products and an activation pass 32 samples took 21 us.
struct ZP {
    const float *W, *bias, *V, *Uh, *Gt;
    int T, TS, K2;
    float *Z, *Vn, *pool;
    const float* Zp;
};

template <int C, bool TRW>
__global__ __launch_bounds__(256) void k_zlayer(ZP p)
{
    constexpr int LD = C + 8, LK = 40;
    __shared__ __attribute__((aligned(16))) __bf16 Ws[C][LD];
    __shared__ __attribute__((aligned(16))) __bf16 Vs[64][LD];
    __shared__ __attribute__((aligned(16))) __bf16 Us[C][LK];
    __shared__ __attribute__((aligned(16))) __bf16 Gs[64][LK];
    __shared__ float pl[4][C];
    const int b = blockIdx.y, t0 = blockIdx.x * 64;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int K2 = p.K2;
    // V tile: 4 channels x 4 samples per thread and pass, stored transposed
    float4 v[C / 64 + (C % 64 != 0)][4];
#pragma unroll
    for (int q = 0; q < C * 4; q += 256) {
        const int sb = q + tid, tq = (sb & 15) * 4, cq = (sb >> 4) * 4;
        if (sb < C * 4)
#pragma unroll
            for (int i = 0; i < 4; ++i) v[q / 256][i] = ld4(p.V + ((long)b * C + cq + i) * p.TS + t0 + tq);
    }
    // W rows: 8 values per thread and pass
#pragma unroll
    for (int e = tid; e < C * C / 8; e += 256) {
        const int r = e / (C / 8), k = (e % (C / 8)) * 8;
        if (TRW) {
            float x[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = p.W[(long)(k + i) * C + r];
            *reinterpret_cast<bf8*>(&Ws[r][k]) = cvt8(make_float4(x[0], x[1], x[2], x[3]), make_float4(x[4], x[5], x[6], x[7]));
        } else {
            *reinterpret_cast<bf8*>(&Ws[r][k]) = cvt8(ld4(p.W + (long)r * C + k), ld4(p.W + (long)r * C + k + 4));
        }
    }
    // mixed modes and inverse basis, zero past K2 (a multiple of 4, up to 32)
    for (int e = tid; e < (C + 64) * 8; e += 256) {
        const int r = e >> 3, k = (e & 7) * 4;
        float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
        if (k < K2) x = ld4(r < C ? p.Uh + ((long)b * C + r) * K2 + k : p.Gt + (long)(t0 + r - C) * K2 + k);
        *reinterpret_cast<bf4*>(r < C ? &Us[r][k] : &Gs[r - C][k]) = cvt4(x.x, x.y, x.z, x.w);
    }
#pragma unroll
    for (int q = 0; q < C * 4; q += 256) {
        const int sb = q + tid, tq = (sb & 15) * 4, cq = (sb >> 4) * 4;
        if (sb < C * 4) {
            const float4* x = v[q / 256];
            *reinterpret_cast<bf4*>(&Vs[tq + 0][cq]) = cvt4(x[0].x, x[1].x, x[2].x, x[3].x);
            *reinterpret_cast<bf4*>(&Vs[tq + 1][cq]) = cvt4(x[0].y, x[1].y, x[2].y, x[3].y);
            *reinterpret_cast<bf4*>(&Vs[tq + 2][cq]) = cvt4(x[0].z, x[1].z, x[2].z, x[3].z);
            *reinterpret_cast<bf4*>(&Vs[tq + 3][cq]) = cvt4(x[0].w, x[1].w, x[2].w, x[3].w);
        }
    }
    __syncthreads();
    // wave w: 16 time samples x C channels
    f4 acc[C / 16], acu[C / 16];
    const int r = lane & 15, g = lane >> 4;
#pragma unroll
    for (int j = 0; j < C / 16; ++j) acc[j] = acu[j] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < C; k += 32) {
        const bf8 av = *reinterpret_cast<const bf8*>(&Vs[w * 16 + r][k + 8 * g]);
#pragma unroll
        for (int j = 0; j < C / 16; ++j)
            acc[j] = mma(av, *reinterpret_cast<const bf8*>(&Ws[j * 16 + r][k + 8 * g]), acc[j]);
    }
    {
        const bf8 av = *reinterpret_cast<const bf8*>(&Gs[w * 16 + r][8 * g]);
#pragma unroll
        for (int j = 0; j < C / 16; ++j)
            acu[j] = mma(av, *reinterpret_cast<const bf8*>(&Us[j * 16 + r][8 * g]), acu[j]);
    }
#pragma unroll
    for (int j = 0; j < C / 16; ++j) {
        const int c = j * 16 + r;
        const float bc = p.bias ? p.bias[c] : 0.f;
        float z[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) z[i] = acu[j][i] + (p.bias ? acc[j][i] + bc : acc[j][i]);
        const long at = ((long)b * C + c) * p.TS + t0 + w * 16 + 4 * g;
        if (TRW && p.Zp) {
            const float4 y = ld4(p.Zp + at);
            z[0] *= gelu_d(y.x);
            z[1] *= gelu_d(y.y);
            z[2] *= gelu_d(y.z);
            z[3] *= gelu_d(y.w);
        }
        if (p.Z) *reinterpret_cast<float4*>(p.Z + at) = make_float4(z[0], z[1], z[2], z[3]);
        if (p.Vn)
            *reinterpret_cast<float4*>(p.Vn + at) = make_float4(gelu_f(z[0]), gelu_f(z[1]), gelu_f(z[2]), gelu_f(z[3]));
        if (p.pool) {
            float s = (z[0] + z[1]) + (z[2] + z[3]);
            s += __shfl_xor(s, 16, 64);
            s += __shfl_xor(s, 32, 64);
            if (g == 0) pl[w][c] = s;
        }
    }
    if (p.pool) {
        __syncthreads();
        if (tid < C)
            p.pool[((long)b * gridDim.x + blockIdx.x) * C + tid] = (pl[0][tid] + pl[1][tid]) + (pl[2][tid] + pl[3][tid]);
    }
}

// ---------------------------------------------------------------------------
// Moment-weighted output projection of every sample, for k_proj:
//   Qm[b][o][h] = sum_j m_bj Q2[(f 6 + j) O + o'][h],  bm[b][o] likewise
// (o = f O + o'), written in the order in which k_proj's waves load it: per 32
// h and 16 o the two float4 halves of an MFMA operand lane by lane, so that
// every load and store of a wave is 1 KB in a row ([b][h / 32][o / 16][half]
// [lane][4]).  A block owns one such tile, reads its six response weights once
// and applies them to every sample.
struct MixP {
    const float *Q2, *q2b, *X;
    float inv[6];        // moment feature scales
    int B, FO, O, H;
    float *Qm, *bm;
};

__global__ __launch_bounds__(128) void k_qmix_frag(MixP p)
{
    const int tid = threadIdx.x, lane = tid & 63, half = tid >> 6, r = lane & 15, g = lane >> 4;
    const int s = blockIdx.x, n16 = (p.FO + 15) / 16;
    const int h = s * 32 + g * 8 + half * 4;
    const long per = (long)n16 * 16 * p.H;
    for (int o16 = blockIdx.y; o16 < n16; o16 += gridDim.y) {
        const int fo = o16 * 16 + r, fc = min(fo, p.FO - 1);   // rows past FO repeat the last one
        const int fr = fc / p.O, o = fc - fr * p.O;
        float4 q[6];
        float qb[6];
#pragma unroll
        for (int j = 0; j < 6; ++j) {
            const long row = (long)(fr * 6 + j) * p.O + o;
            q[j] = ld4(p.Q2 + row * p.H + h);
            qb[j] = p.q2b[row];
        }
        const long slot = (((long)s * n16 + o16) * 2 + half) * 256 + lane * 4;
        for (int b = 0; b < p.B; ++b) {
            float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
            float ab = 0.f;
#pragma unroll
            for (int j = 0; j < 6; ++j) {
                const float m = p.X[b * 9 + 3 + j] * p.inv[j];
                a.x += m * q[j].x;
                a.y += m * q[j].y;
                a.z += m * q[j].z;
                a.w += m * q[j].w;
                ab += m * qb[j];
            }
            *reinterpret_cast<float4*>(p.Qm + b * per + slot) = a;
            if (s == 0 && tid < 16 && fo < p.FO) p.bm[(long)b * p.FO + fo] = ab;
        }
    }
}

// Hidden projection, activation and output projection in one kernel:
//   Yf[b][o][t] = sum_h Qm[b][o][h] gelu(sum_c Q1[h][c] V[b][c][t] + q1b[h]) + bm[b][o]
// A block owns NW RW 16 outputs x NTC 16 time samples of one sample and walks
// h in slices of 32: its waves form the slice's hidden values (MFMA, bias,
// activation), round them to BF16 where the product stages its operand (LDS,
// two buffers, one barrier per slice) and multiply them with their own rows of
// Qm, which go from memory straight to registers (no wave shares them).  The
// 1024 hidden series never reach memory: as separate passes they were written
// and read back four times over, 4 MB per sample and pass.
// What bounded it first was the vector memory path, not the products: with
// row-major operands (32-byte pieces of 16 rows per load, each wave loading Q1
// itself) 64 samples of 1024 hidden and 512 output series took 292 us; with
// every operand load 1 KB in a row per wave (Qm in the order of k_qmix_frag,
// Q1 through LDS) they take 150-160 us, 0.57 PFLOP/s, close to what the
// activations (some 45 vector instructions each) and the MFMAs need one after
// the other.  The separate passes (hidden product, activation, output product)
// took about 430 us.
// scale (may be null): the outputs are multiplied by scale[o / n_rec].
struct ProjP {
    const float *V, *Q1, *q1b, *Qm, *bm, *scale;
    int T, TS, H, FO, n_rec, nt, nm, B;   // nt time tiles, nm output tiles
    float* Y;            // [B][FO][T]
};

constexpr int XCD_COUNT = 8;

template <int C, int RW, int NTC, int NW>
__global__ __launch_bounds__(NW * 64) void k_proj(ProjP p)
{
    constexpr int N = NTC * 16, LV = C + 8, LH = 40, NTH = NW * 64;
    constexpr int HT = 2 * NTC;                     // hidden tiles (16 h x 16 t) of a slice
    constexpr int HPW = (HT + NW - 1) / NW;         // per wave
    constexpr int QPT = (8 * C + NTH - 1) / NTH;    // float4 of a Q1 slice per thread
    __shared__ __attribute__((aligned(16))) __bf16 Vs[N][LV];
    __shared__ __attribute__((aligned(16))) __bf16 Hs[2][N][LH];
    __shared__ __attribute__((aligned(16))) __bf16 Qs[2][32][LV];
    // consecutive blocks go to the chip's 8 XCDs in turn: the tiles of one
    // sample, which share its rows of Qm, are numbered 8 apart (one L2).
    // Fewer than 8 samples: tile by tile, over all XCDs
    const int per = p.nt * p.nm;
    const int L = blockIdx.x;
    const int grp = L / (XCD_COUNT * per), l = L - grp * XCD_COUNT * per;
    const bool few = p.B < XCD_COUNT;
    const int b = few ? L / per : grp * XCD_COUNT + l % XCD_COUNT, tile = few ? L % per : l / XCD_COUNT;
    if (b >= p.B) return;
    const int mt = tile / p.nt, t0 = (tile - mt * p.nt) * N;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, r = lane & 15, g = lane >> 4;
    const int T = p.T, H = p.H, n16 = (p.FO + 15) / 16;
    for (int sb = tid; sb < C / 4 * (N / 4); sb += NTH) {
        const int tq = (sb % (N / 4)) * 4, cq = (sb / (N / 4)) * 4;
        float4 x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = ld4(p.V + ((long)b * C + cq + i) * p.TS + t0 + tq);
        *reinterpret_cast<bf4*>(&Vs[tq + 0][cq]) = cvt4(x[0].x, x[1].x, x[2].x, x[3].x);
        *reinterpret_cast<bf4*>(&Vs[tq + 1][cq]) = cvt4(x[0].y, x[1].y, x[2].y, x[3].y);
        *reinterpret_cast<bf4*>(&Vs[tq + 2][cq]) = cvt4(x[0].z, x[1].z, x[2].z, x[3].z);
        *reinterpret_cast<bf4*>(&Vs[tq + 3][cq]) = cvt4(x[0].w, x[1].w, x[2].w, x[3].w);
    }
    // this wave's 16-row tiles of Qm (tiles past the last one read it again
    // and are not stored)
    const int o0 = (mt * NW + w) * RW;
    const float* __restrict__ Qb = p.Qm + (long)b * n16 * 16 * H + lane * 4;
    float4 qa[RW][2];
    auto load_q = [&](int s) {
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            const float* q = Qb + ((long)s * n16 + min(o0 + i, n16 - 1)) * 512;
            qa[i][0] = ld4(q);
            qa[i][1] = ld4(q + 256);
        }
    };
    // slice s of Q1: 32 C floats in a row
    float4 q1[QPT];
    auto load_1 = [&](int s) {
#pragma unroll
        for (int i = 0; i < QPT; ++i) {
            const int e = tid + i * NTH;
            if (8 * C % NTH == 0 || e < 8 * C) q1[i] = ld4(p.Q1 + (long)s * 32 * C + 4 * e);
        }
    };
    auto store_1 = [&](int buf) {
#pragma unroll
        for (int i = 0; i < QPT; ++i) {
            const int e = tid + i * NTH;
            if (8 * C % NTH == 0 || e < 8 * C)
                *reinterpret_cast<bf4*>(&Qs[buf][e / (C / 4)][(e % (C / 4)) * 4]) = cvt4(q1[i].x, q1[i].y, q1[i].z, q1[i].w);
        }
    };
    // hidden values of slice s from Qs[buf] into Hs[buf]
    auto hidden = [&](int s, int buf) {
#pragma unroll
        for (int i = 0; i < HPW; ++i) {
            const int ti = w + i * NW;
            if (HT % NW != 0 && ti >= HT) continue;
            const int ht = ti & 1, tt = ti >> 1;
            const float4 bq = ld4(p.q1b + s * 32 + ht * 16 + 4 * g);
            f4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < C / 32; ++k)
                a = mma(*reinterpret_cast<const bf8*>(&Qs[buf][ht * 16 + r][k * 32 + 8 * g]),
                        *reinterpret_cast<const bf8*>(&Vs[tt * 16 + r][k * 32 + 8 * g]), a);
            *reinterpret_cast<bf4*>(&Hs[buf][tt * 16 + r][ht * 16 + 4 * g]) =
                cvt4(gelu_f(a[0] + bq.x), gelu_f(a[1] + bq.y), gelu_f(a[2] + bq.z), gelu_f(a[3] + bq.w));
        }
    };
    f4 acc[RW][NTC];
#pragma unroll
    for (int i = 0; i < RW; ++i)
#pragma unroll
        for (int j = 0; j < NTC; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
    bf8 qv[RW];
    auto round_q = [&]() {
#pragma unroll
        for (int i = 0; i < RW; ++i) qv[i] = cvt8(qa[i][0], qa[i][1]);
    };
    auto product = [&](int buf) {
#pragma unroll
        for (int j = 0; j < NTC; ++j) {
            const bf8 hv = *reinterpret_cast<const bf8*>(&Hs[buf][j * 16 + r][8 * g]);
#pragma unroll
            for (int i = 0; i < RW; ++i) acc[i][j] = mma(hv, qv[i], acc[i][j]);
        }
    };
    const int ns = H / 32;
    load_1(0);
    load_q(0);
    store_1(0);
    load_1(min(1, ns - 1));
    __syncthreads();   // Vs, Qs[0]
    hidden(0, 0);
    store_1(1);
    load_1(min(2, ns - 1));
    __syncthreads();   // Hs[0], Qs[1]
    // slice s: the product of slice s, the hidden values of slice s + 1, the
    // staging of slice s + 2.  No condition in the loop body: a conditional
    // load would be waited for at the end of its own iteration
    for (int s = 0; s < ns - 1; ++s) {
        const int buf = s & 1;
        round_q();
        load_q(s + 1);
        product(buf);
        hidden(s + 1, buf ^ 1);
        store_1(buf);              // Qs[buf] was last read for slice s
        load_1(min(s + 3, ns - 1));
        __syncthreads();
    }
    round_q();
    product((ns - 1) & 1);
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        const int o = (o0 + i) * 16 + r;
        if (o >= p.FO) continue;
        const float bo = p.bm[(long)b * p.FO + o];
        const float sc = p.scale ? p.scale[o / p.n_rec] : 1.f;
        float* __restrict__ y = p.Y + ((long)b * p.FO + o) * T + t0 + 4 * g;
#pragma unroll
        for (int j = 0; j < NTC; ++j) {
            float4 v = make_float4(acc[i][j][0] + bo, acc[i][j][1] + bo, acc[i][j][2] + bo, acc[i][j][3] + bo);
            if (p.scale) v = make_float4(v.x * sc, v.y * sc, v.z * sc, v.w * sc);
            *reinterpret_cast<float4*>(y + j * 16) = v;
        }
    }
}

}  // namespace snof
