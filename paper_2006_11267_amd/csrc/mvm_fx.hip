// FP32 kernel product with entries evaluated on the fly (CIQ_F32), more than
// 16 columns, on the BF16 matrix cores.
//
// v_mfma_f32_16x16x4_f32 and vector instructions share the SIMD: at N =
// 50,000, d = 6, S = 64 the FP32 form (mvm_mfma.h) spends 2.2 ms on the
// contraction and then 2.3 ms on the entries. BF16 matrix instructions run
// beside the other waves' vector work, so here every entry and every element
// of V is split in registers into three BF16 parts of 8 bits whose sum it is,
// and
//     K V ~ Kh Vh + (Kh Vm + Km Vh) + (Km Vm + Kh Vl + Kl Vh)
// drops terms of 2^-25 of Kh Vh and less (rounding to nearest leaves 2^-9 and
// 2^-18 in the lower parts). Six v_mfma_f32_16x16x32_bf16 take 0.8 ms of matrix
// time there; the entries' evaluation and split (about 27 vector instructions,
// two of them of a quarter of the rate) are the bound. Measured, same size:
// 4.55 -> 2.9 ms; 32 columns 3.20 -> 2.20, 128 columns 9.33 -> 5.5; N = 20,000,
// 64 columns 0.82 -> 0.58. At 16 columns the FP32 form stays:
// 2.04 ms against 2.16.
//
// Range: BF16 parts hold all 24 bits of numbers of 2^-109 and more, so entries
// are scaled by 2^24 and V by 2^40: FP32's smallest normal entries and all its
// elements keep their bits. What the sums could then overflow by, elements of
// 2^56 and more, infinities among them, is left out of a chunk's pass; a chunk
// that had any takes a second pass with them alone, scaled by 2^-40. The scaling
// costs up to 2 % (Matern) and, one more instruction an entry, 3 to 5 % (RBF:
// 2.54 -> 2.62 ms at 64 columns, 1.87 -> 1.98 at 32).
//
// FP32 sums: per chunk of 64 columns the cross terms first, then the two
// Kh Vh, then to FP64. The matrix cores cut a sum of eight products off
// downwards (towards minus infinity), which adds up over the chunks (0.7 of
// the whole error at N = 50,000), so V changes its sign from chunk to chunk.
// The diagonal entry, which outweighs the rest of its chunk where lengthscales
// are short, stays out of the matrix product: 2^-60 of it takes its place (an
// infinite V[i] must still reach row i) and the epilogue adds V[i] itself.
// The lengthscale and log2(e) are one factor, rounded once, of the exponent.
// Error against 64 bits at d = 2 to 16, lengthscales 0.02 to 2, N = 300 to
// 50,000: 3e-8 to 2.2e-7, in every one of 33 cases below the FP32 form's.
//
// Block: eight waves of one 16-row tile each; per chunk of 64 columns the block
// splits V and stages it in the operand's order (16-byte units, the eight rows
// of a lane group of one column) and the points (16 bytes of padding after every
// eight: a wave reads four groups at once), double-buffered up to 64 columns:
// one barrier a chunk. One tile a wave leaves 128 registers, two
// blocks a CU (3.0 ms; two tiles a wave, one block of eight or two of four
// waves: 3.2; sixteen waves 2.9 at this size, but blocks of 256 rows). The
// 128-column form takes 250 registers and one block a CU, and still beats two
// launches of 64 (5.5 against 5.8 ms: entries are evaluated once).
#include <algorithm>

#include "bf16_parts.h"
#include "mvm_mfma.h"

namespace ciq {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
using bf16::bf16x8;
using bf16::split3;

// a value that is the same in every lane, kept in a scalar register
__device__ __forceinline__ float uniform(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x)));
}

// Entries of FP32's smallest normal size and elements below kVLarge keep all 24
// bits in their parts (2^-109 and more after the scaling), sums of 64 products
// stay below 2^126; larger elements take a pass of their own (below).
constexpr float kKScale = 0x1p24f, kVScale = 0x1p40f, kVLarge = 0x1p56f;

template <int KERNEL, int DP, int NSB, bool ARD>
__global__ __launch_bounds__(512, NSB > 4 ? 2 : 4) void mvm_fx_kernel(MvmArgs a) {
    constexpr int NT = 512;
    constexpr int S16 = NSB * 16;
    constexpr int VB = NSB * 64;                   // 16-byte units of one part of one k-step of 32 columns
    constexpr int VU = S16 * 8;                    // units of one part of a chunk of 64 columns
    constexpr int UPT = (VU + NT - 1) / NT;
    constexpr int NBUF = NSB <= 4 ? 2 : 1;
    constexpr int DPP = DP == 6 ? 8 : DP == 10 ? 12 : DP;
    constexpr int XE = 64 * DP;
    constexpr int XPT = (XE + NT - 1) / NT;
    __shared__ bf16x8 vs[NBUF][3 * VU];
    __shared__ __attribute__((aligned(16))) float xs[NBUF][64 * DPP + 32];

    if (mfma::done_now(a.done)) return;
    const int n = a.n;
    float sc[DP];
#pragma unroll
    for (int k = 0; k < DP; ++k) sc[k] = uniform((float)a.scale[k]);
    // the lengthscale (isotropic) and log2(e) are one factor of the exponent
    const double sc0 = ARD ? 1.0 : a.scale[0];
    const float ec = uniform((float)(KERNEL == CIQ_KERNEL_RBF ? -0.5 * 1.4426950408889634074 * sc0 * sc0
                                                              : -1.4426950408889634074 * sc0));
    const int split = blockIdx.y;
    const double* __restrict__ xh = static_cast<const double*>(a.xh);
    const float* __restrict__ v = static_cast<const float*>(a.v);
    double* __restrict__ y = static_cast<double*>(a.y) + (long long)split * a.ysplit;
    const int s = a.s, ldv = a.ldv, ldy = a.ldy;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row0 = (blockIdx.x * 8 + wave) * 16;
    float xi[DP];
    {
        const int i = row0 + (lane & 15);
#pragma unroll
        for (int k = 0; k < DP; ++k) xi[k] = (i < n) ? (float)xh[(long long)i * DP + k] : 0.0f;
    }

    floatx4 acc[NSB];
    double accd[NSB][4];
#pragma unroll
    for (int sb = 0; sb < NSB; ++sb)
#pragma unroll
        for (int r = 0; r < 4; ++r) accd[sb][r] = 0.0;

    const int nchunk = (n + 63) / 64;
    const int c0 = (int)(((long long)split * nchunk) / a.nsplit);
    const int c1 = (int)(((long long)(split + 1) * nchunk) / a.nsplit);

    float xreg[XPT], vreg[UPT][8];
    auto fetch = [&](int c) {
        const int j0 = c * 64;
#pragma unroll
        for (int k = 0; k < XPT; ++k) {
            const int e = tid + NT * k;
            const int j = j0 + e / DP;
            xreg[k] = (e < XE && j < n) ? (float)xh[(long long)j0 * DP + e] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < UPT; ++u) {
            const int e = tid + NT * u;
            const int cc = e % S16, j = j0 + 8 * (e / S16);
            const bool ok = e < VU && cc < s;
            const float* vp = v + (long long)j * ldv + cc;
            if (j0 + 64 <= n && S16 <= s) {
#pragma unroll
                for (int q = 0; q < 8; ++q) vreg[u][q] = (VU % NT == 0 || e < VU) ? vp[(long long)q * ldv] : 0.0f;
                continue;
            }
#pragma unroll
            for (int q = 0; q < 8; ++q) vreg[u][q] = (ok && j + q < n) ? vp[(long long)q * ldv] : 0.0f;
        }
    };
    if (c0 < c1) fetch(c0);

    __shared__ int large[NBUF];                    // the last chunk that had large elements
    if (tid < NBUF) large[tid] = -1;
    if (NBUF == 2) __syncthreads();
    bool again = false;                            // this chunk's large elements
    for (int c = c0; c < c1;) {
        const int buf = NBUF == 2 ? (c & 1) : 0;
        const float scale = ((c & 1) ? -1.0f : 1.0f) * (again ? 1.0f / kVScale : kVScale);
        if (NBUF == 1 || again) __syncthreads();
#pragma unroll
        for (int k = 0; k < XPT; ++k) {
            const int e = tid + NT * k;
            if (e < XE) xs[buf][(e / DP) * DPP + (e / DP / 8) * 4 + e % DP] = xreg[k];
        }
#pragma unroll
        for (int u = 0; u < UPT; ++u) {
            const int e = tid + NT * u;
            if (VU % NT != 0 && e >= VU) break;
            const int cc = e % S16, g = e / S16;      // column, group of eight rows of V
            bf16x8 h, m, l;
#pragma unroll
            for (int q = 0; q < 8; ++q) vreg[u][q] *= scale;
            float top = 0.0f;
#pragma unroll
            for (int q = 0; q < 8; ++q) top = fmaxf(top, fabsf(vreg[u][q]));
            if (again) {
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    if (fabsf(vreg[u][q]) < kVLarge / kVScale) vreg[u][q] = 0.0f;
            } else if (top >= kVLarge * kVScale) {
                large[buf] = c;
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    if (fabsf(vreg[u][q]) >= kVLarge * kVScale) vreg[u][q] = 0.0f;   // (not a NaN)
            }
            split3(vreg[u], h, m, l);
            if (again) bf16::only_last(vreg[u], h, m, l);
            const int at = (g >> 2) * VB + (cc >> 4) * 64 + (g & 3) * 16 + (cc & 15);
            vs[buf][at] = h;
            vs[buf][VU + at] = m;
            vs[buf][2 * VU + at] = l;
        }
        __syncthreads();
        if (c + 1 < c1) fetch(c + 1);
        bf16x8 kh[2];
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const float* xj0 = &xs[buf][(4 * kk + (lane >> 4)) * (8 * DPP + 4)];
            float kv[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                float r2 = 0.0f;
#pragma unroll
                for (int k = 0; k < DP; ++k) {
                    const float dd = xi[k] - xj0[u * DPP + k];
                    if constexpr (ARD) {
                        const float w = dd * sc[k];
                        r2 = fmaf(w, w, r2);
                    } else {
                        r2 = fmaf(dd, dd, r2);
                    }
                }
                if constexpr (KERNEL == CIQ_KERNEL_RBF) {
                    kv[u] = __builtin_amdgcn_exp2f(r2 * ec) * kKScale;
                } else {
                    // t = -rho log2(e); 1 + rho + rho^2 / 3 in t
                    constexpr double ln2 = 0.69314718055994530942;
                    const float t = __builtin_amdgcn_sqrtf(r2) * ec;
                    kv[u] = fmaf(t, fmaf(t, (float)(ln2 * ln2 / 3.0) * kKScale, (float)-ln2 * kKScale), kKScale) *
                            __builtin_amdgcn_exp2f(t);
                }
            }
            const int j0 = c * 64 + kk * 32;
            if (j0 <= row0 + 15 && row0 <= j0 + 31) {     // the diagonal (see above)
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (j0 + 8 * (lane >> 4) + u == row0 + (lane & 15)) kv[u] = (kv[u] - kKScale) + kKScale * 0x1p-60f;
            }
            bf16x8 km, kl;
            split3(kv, kh[kk], km, kl);
            const bf16x8* bp = &vs[buf][kk * VB + lane];
#pragma unroll
            for (int sb = 0; sb < NSB; ++sb) {
                const bf16x8 bh = bp[sb * 64], bm = bp[VU + sb * 64], bl = bp[2 * VU + sb * 64];
                floatx4 t = kk == 0 ? floatx4{0.f, 0.f, 0.f, 0.f} : acc[sb];
                t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kl, bh, t, 0, 0, 0);
                t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kh[kk], bl, t, 0, 0, 0);
                t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(km, bm, t, 0, 0, 0);
                t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(km, bh, t, 0, 0, 0);
                t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kh[kk], bm, t, 0, 0, 0);
                if (kk == 1) {
                    t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kh[0], vs[buf][lane + sb * 64], t, 0, 0, 0);
                    t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kh[1], bh, t, 0, 0, 0);
                }
                acc[sb] = t;
            }
        }
#pragma unroll
        for (int sb = 0; sb < NSB; ++sb)
#pragma unroll
            for (int r = 0; r < 4; ++r) accd[sb][r] = fma((double)acc[sb][r], (double)(1.0f / scale), accd[sb][r]);
        again = !again && large[buf] == c;
        if (again) fetch(c);
        else ++c;
    }

    const double o2 = a.o2, s2 = a.s2;
#pragma unroll
    for (int sb = 0; sb < NSB; ++sb) {
        const int cc = sb * 16 + (lane & 15);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = row0 + 4 * (lane >> 4) + r;
            if (i < n && cc < s) {
                double val = o2 * (1.0 / kKScale) * accd[sb][r];
                if (split == 0) val = fma(o2 + s2, (double)v[(long long)i * ldv + cc], val);
                y[(long long)i * ldy + cc] = val;
            }
        }
    }
}

template <int KERNEL, bool ARD, int DP>
hipError_t launch_fx_dp(const MvmArgs& a, int nsb, hipStream_t st) {
    const dim3 grid((a.n + kFxRows - 1) / kFxRows, a.nsplit);
    if (nsb <= 2) hipLaunchKernelGGL((mvm_fx_kernel<KERNEL, DP, 2, ARD>), grid, dim3(512), 0, st, a);
    else if (nsb <= 4) hipLaunchKernelGGL((mvm_fx_kernel<KERNEL, DP, 4, ARD>), grid, dim3(512), 0, st, a);
    else hipLaunchKernelGGL((mvm_fx_kernel<KERNEL, DP, 8, ARD>), grid, dim3(512), 0, st, a);
    return hipGetLastError();
}

template <int KERNEL, bool ARD>
hipError_t launch_fx_k(const MvmArgs& a, int nsb, hipStream_t st) {
    switch (a.dp) {
        case 4: return launch_fx_dp<KERNEL, ARD, 4>(a, nsb, st);
        case 6: return launch_fx_dp<KERNEL, ARD, 6>(a, nsb, st);
        case 8: return launch_fx_dp<KERNEL, ARD, 8>(a, nsb, st);
        case 10: return launch_fx_dp<KERNEL, ARD, 10>(a, nsb, st);
        case 12: return launch_fx_dp<KERNEL, ARD, 12>(a, nsb, st);
        default: return launch_fx_dp<KERNEL, ARD, 16>(a, nsb, st);
    }
}
}  // namespace

hipError_t launch_mvm_fx(const MvmArgs& a, int nsb, hipStream_t st) {
    static_assert(kFxRows == 128, "eight waves of 16 rows");
    if (a.wl != nullptr || nsb < 2 || nsb > 8) return hipErrorInvalidValue;
    if (a.kernel == CIQ_KERNEL_RBF)
        return a.ard ? launch_fx_k<CIQ_KERNEL_RBF, true>(a, nsb, st) : launch_fx_k<CIQ_KERNEL_RBF, false>(a, nsb, st);
    return a.ard ? launch_fx_k<CIQ_KERNEL_MATERN52, true>(a, nsb, st)
                 : launch_fx_k<CIQ_KERNEL_MATERN52, false>(a, nsb, st);
}
}  // namespace ciq
