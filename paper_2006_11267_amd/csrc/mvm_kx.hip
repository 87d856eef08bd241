// Resident FP32 kernel matrix times more than 32 columns (CIQ_F32) on the BF16
// matrix cores.
//
// v_mfma_f32_16x16x4_f32 runs at 157 TFLOP/s, so at 64 columns the FP32
// contraction, not the stream of K, bounds a product (2.84 ms at N = 50,000,
// S = 64, where reading the 10 GB matrix takes 1.6 ms). Here every FP32 entry
// is split in registers into three BF16 parts of 8 bits whose sum it is, the
// operand vector (written split by the update kernel, op3_index layout) likewise,
// and
//     K V ~ Kh Vh + (Kh Vm + Km Vh) + (Km Vm + Kh Vl + Kl Vh)
// drops terms of 2^-26 of Kh Vh and less: six v_mfma_f32_16x16x32_bf16 cost 0.9
// ms of matrix time at that size and the stream of K becomes the bound. BF16
// has FP32's range, so the parts keep all 24 bits of small entries and elements
// as well (FP16 parts take 3.5 instead of 5.5 vector instructions an entry, but
// end at 2^-38 of the outputscale: entries below 2^-15 lost bits and those below
// 2^-38 vanished); the scales that keep their lowest parts above 2^-133 are in
// ciq_internal.h.
//
// FP32 sums: per chunk of 64 columns the cross terms first, then the two Kh Vh,
// then to FP64. As in mvm_fx.hip the operand changes its sign from chunk to
// chunk, because the matrix cores cut sums off downwards, and the diagonal entry
// stays out of the matrix product: 2^-60 takes its place (an infinite V[i] must
// still reach row i) and the epilogue adds V[i] itself, in FP64. Error of one
// product against 64 bits (norms, in 2^-24; eight kernels, N = 3,000 to 20,000, d =
// 2 to 10, lengthscales 0.05 to 1): Gaussian right-hand sides 0.4 to 1.1 (0.5 to 1.7
// without the two measures and with FP16 parts, 0.5 to 2.5 on the FP32 matrix cores),
// positive ones 0.43 to 0.54 (0.45 to 0.82; 0.43 to 0.54).
//
// K is read in the layout of the FP32 form (mvm_cache.hip): lane l of a
// 16-row tile holds K[l % 16][4 st + l / 16], st = 0..15 of the chunk. The
// 16x16x32 MFMA lets the eight columns of lane group g = l / 16 be any eight,
// as long as both operands agree, so k-step ks takes the group's columns
// 32 ks + 4 m + g (m = 0..7) and the split operand is stored in that order.
//
// Block: WAVES waves of one 16-row tile each; per chunk the block stages the
// split operand (NSB column blocks x 2 k-steps x three parts, 1 KB each) in one
// of two LDS buffers, one barrier per chunk (see kt32_item). Sixteen waves
// halve the operand's L2 reads (24 KB per block and chunk against 64 KB of K)
// and fit 128 registers a wave. Measured at N = 50,000, S = 64 (the FP32 MFMA
// form: 2.86 ms with FP32 sums of 64 columns, 3.72 with sums of 16): 2.18 ms with
// sixteen waves, 4.6 TB/s of K (FP16 parts with neither alternating signs nor the
// diagonal outside, in turn with it: 2.15). Tried with those, where sixteen waves
// took 2.13: eight waves 2.20, 12 waves with two chunks of K in flight 2.23, two
// tiles a wave 2.31, 128 columns a launch 4.35 (no better than two groups of 64).
// More than 64 columns run as groups of one launch, the groups of a row block next
// to each other on one XCD so that its L2 serves K to the later ones.
#include <algorithm>
#include <cmath>

#include "bf16_parts.h"
#include "ciq_internal.h"

namespace ciq {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
using bf16::bf16x8;
using bf16::split3;

template <int NSB, int WAVES>
__global__ __launch_bounds__(64 * WAVES, 4) void mvm_kx_kernel(MvmArgs a, int groups) {
    constexpr int NT = 64 * WAVES;
    constexpr int VB = NSB * 192;                // 16-byte operand units per k-step
    constexpr int VU = 2 * VB;                   // per chunk
    constexpr int UPT = (VU + NT - 1) / NT;
    __shared__ bf16x8 vs[2 * VU];

    if (a.done != nullptr && *a.done != 0) return;
    const int nsplit = a.nsplit;
    const int split = (int)(blockIdx.x % (unsigned)nsplit);
    const int x = (int)(blockIdx.x / (unsigned)nsplit);
    const int rb = x / groups, grp = x - rb * groups;
    const int n = a.n;
    const bf16x8* __restrict__ vt = static_cast<const bf16x8*>(a.vt) + grp * VB;
    const int kstride = a.nsbt * 192;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tile = rb * WAVES + wave;
    const int tmax = (int)(((n + 127) / 128) * 8) - 1;   // last tile of the padded matrix

    const int nchunk = (n + 63) / 64;
    const int c0 = (int)(((long long)split * nchunk) / nsplit);
    const int c1 = (int)(((long long)(split + 1) * nchunk) / nsplit);

    floatx4 acc[NSB];
    double accd[NSB][4];
#pragma unroll
    for (int sb = 0; sb < NSB; ++sb)
#pragma unroll
        for (int r = 0; r < 4; ++r) accd[sb][r] = 0.0;

    // operand staging: thread offsets within a chunk are fixed, the chunk's
    // base is uniform
    bf16x8 vreg[UPT];
    int voff[UPT];
#pragma unroll
    for (int u = 0; u < UPT; ++u) {
        const int e = tid + NT * u;
        voff[u] = e + (e >= VB ? kstride - VB : 0);
    }
    auto fetch_v = [&](int c) {
        const bf16x8* base = vt + (long long)c * 2 * kstride;
#pragma unroll
        for (int u = 0; u < UPT; ++u) {
            if (VU % NT != 0 && tid + NT * u >= VU) break;
            vreg[u] = base[(unsigned)voff[u]];
        }
    };
    const float* kb = static_cast<const float*>(a.kt) + (size_t)min(tile, tmax) * a.njs * 64;
    // one chunk of K in flight per wave; half a chunk (k-step kk) of the next
    // one is requested as soon as the registers of this one's half are free
    float kq[16];
    auto fetch_k = [&](int c, int kk) {
        const floatx4* base = reinterpret_cast<const floatx4*>(kb + (size_t)c * 1024);
#pragma unroll
        for (int p = 2 * kk; p < 2 * kk + 2; ++p) {
            const floatx4 x = __builtin_nontemporal_load(base + (unsigned)(lane + 64 * p));
#pragma unroll
            for (int h = 0; h < 4; ++h) kq[4 * p + h] = x[h];
        }
    };
    auto chunk = [&](int c) {
        bf16x8* vb = vs + (c & 1) * VU;
#pragma unroll
        for (int u = 0; u < UPT; ++u) {
            const int e = tid + NT * u;
            if (VU % NT != 0 && e >= VU) break;
            vb[e] = vreg[u];
        }
        __syncthreads();
        if (c + 1 < c1) fetch_v(c + 1);
        const bool diag = c == (tile >> 2);         // the chunk holds the tile's diagonal
        bf16x8 kh[2];
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            bf16x8 km, kl;
            if (diag && kk == ((tile >> 1) & 1)) {  // row r's entry: column 16 (tile % 4) + r of the chunk
                const int r = lane & 15, step = 4 * (tile & 3) + (r >> 2);
#pragma unroll
                for (int m = 0; m < 8; ++m)
                    if (8 * kk + m == step && (r & 3) == (lane >> 4))
                        kq[8 * kk + m] = (kq[8 * kk + m] - kKxScale) + kKxScale * 0x1p-60f;
            }
            split3(kq + 8 * kk, kh[kk], km, kl);
            if (c + 1 < c1) fetch_k(c + 1, kk);
            const bf16x8* bp = vb + kk * VB + lane;
#pragma unroll
            for (int sb = 0; sb < NSB; ++sb) {
                const bf16x8 bh = bp[sb * 192], bm = bp[sb * 192 + 64], bl = bp[sb * 192 + 128];
                floatx4 t = kk == 0 ? floatx4{0.f, 0.f, 0.f, 0.f} : acc[sb];
                t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kl, bh, t, 0, 0, 0);
                t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kh[kk], bl, t, 0, 0, 0);
                t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(km, bm, t, 0, 0, 0);
                t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(km, bh, t, 0, 0, 0);
                t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kh[kk], bm, t, 0, 0, 0);
                if (kk == 1) {
                    t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kh[0], vb[sb * 192 + lane], t, 0, 0, 0);
                    t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kh[1], bh, t, 0, 0, 0);
                }
                acc[sb] = t;
            }
        }
#pragma unroll
        for (int sb = 0; sb < NSB; ++sb)
#pragma unroll
            for (int r = 0; r < 4; ++r) accd[sb][r] = fma((double)acc[sb][r], (c & 1) ? -1.0 : 1.0, accd[sb][r]);
    };
    if (c0 < c1) {
        fetch_v(c0);
        fetch_k(c0, 0);
        fetch_k(c0, 1);
    }
    for (int c = c0; c < c1; ++c) chunk(c);

    const double o2 = a.o2, dd = a.o2 * kKxScale + a.s2;   // the diagonal: entry and noise
    const double* __restrict__ v = static_cast<const double*>(a.v);
    double* __restrict__ y = static_cast<double*>(a.y) + (long long)split * a.ysplit;
    float* __restrict__ y32 = a.y32 ? a.y32 + (long long)split * a.ysplit : nullptr;
    const int s = a.s, ldv = a.ldv, ldy = a.ldy;
#pragma unroll
    for (int sb = 0; sb < NSB; ++sb) {
        const int cc = (grp * NSB + sb) * 16 + (lane & 15);
        if (cc >= s) continue;
        const double vi = a.vcol_inv ? a.vcol_inv[cc] : a.vinv;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = tile * 16 + 4 * (lane >> 4) + r;   // 16x16 accumulator layout
            if (i < n) {
                double val = o2 * (accd[sb][r] * vi);
                if (split == 0) val = fma(dd, v[(long long)i * ldv + cc], val);
                if (y32) y32[(long long)i * ldy + cc] = (float)val;
                else y[(long long)i * ldy + cc] = val;
            }
        }
    }
}

template <int NSB>
hipError_t launch_kx_nsb(const MvmArgs& a, int groups, hipStream_t st) {
    const int rows = kx_rows_per_block(a.rt);
    const dim3 grid((unsigned)((a.n + rows - 1) / rows) * groups * a.nsplit);
    if (a.rt == 1) hipLaunchKernelGGL((mvm_kx_kernel<NSB, 8>), grid, dim3(512), 0, st, a, groups);
    else hipLaunchKernelGGL((mvm_kx_kernel<NSB, 16>), grid, dim3(1024), 0, st, a, groups);
    return hipGetLastError();
}

// Column groups of a launch: blocks of 16 columns, at most four a group, as
// even as they come; the operand buffer (op16_nsbt) has room for groups * nsb.
void kx_groups(int s, int& groups, int& nsb) {
    const int nb = (s + 15) / 16;
    groups = (nb + 3) / 4;
    nsb = std::max(3, (nb + groups - 1) / groups);
}

}  // namespace

int kx_rows_per_block(int rt) { return rt == 1 ? 128 : 256; }

hipError_t launch_mvm_kx(const MvmArgs& a, hipStream_t st) {
    int groups, nsb;
    kx_groups(a.s, groups, nsb);
    if (a.rt < 1 || a.rt > 2 || a.njs * 4 != (long long)kcache_cols(a.n) || a.vt == nullptr ||
        a.nsbt < groups * nsb || a.nsplit < 1)
        return hipErrorInvalidValue;
    return nsb == 3 ? launch_kx_nsb<3>(a, groups, st) : launch_kx_nsb<4>(a, groups, st);
}

// Block form and column ranges of an n x n product with s columns whose
// partials have part_bytes per element. Modelled from the times measured at n
// = 50,000 (a CU with all its blocks resident takes 3.6 us for 256 rows x 64
// columns of K x 64 columns of V; two 128-row blocks about 4 % more, as they
// read the operand twice) and at n = 5,000 (a lone 128-row block: 2.4 us a
// chunk, bound by its loads' latency): rounds of blocks over the chip's 256
// (16 waves) or 512 (8 waves) slots, each as long as its chunks, plus writing
// and summing the partials at 4.5 TB/s (and 0.3 us a range, or a line a cycle
// where one block sums a small problem's, step_owner_kernel). Where the operand is several times an
// XCD's 4 MB L2 the ranges are 8 or 16, so that every XCD (block index mod 8)
// streams one or two of them (at N = 10,000, S = 64, where it is as large as
// the L2, six ranges in one round of blocks beat sixteen: 101 against 117 us).
void kx_plan(int n, int s, int part_bytes, int& rt, int& nsplit) {
    int groups, nsb;
    kx_groups(s, groups, nsb);
    const int chunks = (n + 63) / 64;
    const bool big = (double)n * s * 6.0 > 1.2e7;
    double best = 1e300;
    rt = 2;
    nsplit = 1;
    for (int r = 1; r <= 2; ++r) {
        const int rows = kx_rows_per_block(r), per_cu = r == 1 ? 2 : 1;
        const double blocks = (double)((n + rows - 1) / rows) * groups;
        for (int ns = 1; ns <= 16 && ns <= chunks; ++ns) {
            if (big && ns != 8 && ns != 16) continue;
            const double load = blocks * ns / (256.0 * per_cu);          // rounds
            const double chunk_us = (r == 1 ? (load <= 0.5 ? 2.4 : 3.7) : 3.6) * nsb / 4.0;
            const double us = std::ceil(load) * std::ceil((double)chunks / ns) * chunk_us +
                              ns * (std::max(0.3, n <= 1024 ? n / 2200.0 : 0.0) +
                                    (double)n * s * 2.0 * part_bytes / 4.5e6);
            if (us < best) {
                best = us;
                rt = r;
                nsplit = ns;
            }
        }
    }
}

}  // namespace ciq
