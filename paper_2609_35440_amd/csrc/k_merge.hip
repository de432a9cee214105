// Merge of a local-loss pass split over the vocabulary (few token tiles: the
// chip would idle with one workgroup per tile).  Each split left, per token,
// its unnormalised sum P_s = sum_v exp2(z_v - m_s) R_v over its part of the
// vocabulary (the target's own term left out), its running maximum m_s, its
// sum of exponentials and the target's logit.  Per token:
//
//   m = max m_s, a_s = exp2(m_s - m), the row's end from sum a_s s_s (finish_row),
//   e = (sum a_s P_s / s + (p_y - 1) R_y) / T, dhhat = tau e, and the RMSNorm
//   backward, or e to the rotate-back buffer for ROT heads.
//
// One row per wave (its mean is a wave reduction), e kept in registers between
// the two sweeps; fixed order throughout.  Bound by reading P once.
#include "mfma_common.h"

namespace solo {

namespace {

using namespace mfma;

template <typename E> __device__ __forceinline__ f32x4 ld4(const E* p) {
    typedef E EV __attribute__((ext_vector_type(4)));
    const EV v = *(const EV*)p;
    return f32x4{(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
}
template <typename E> __device__ __forceinline__ void st4(E* p, f32x4 v) {
    typedef E EV __attribute__((ext_vector_type(4)));
    *(EV*)p = EV{(E)v[0], (E)v[1], (E)v[2], (E)v[3]};
}

constexpr int kQ = 16;  // 256-column groups of the widest row (4096)

// FAM: the records the family's gradient passes read (see FusedArgs::rowrec)
template <typename E, bool F32FAM>
__global__ __launch_bounds__(256) void k_merge(FusedArgs a, int rows) {
    extern __shared__ __attribute__((aligned(16))) float pbuf[];  // [4][d] when the module trains its gain
    const int k = a.m0 + (int)blockIdx.y;
    const int tile = blockIdx.x;
    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    const int d = a.d;
    const long long KT = (long long)a.K * a.T;
    const float tau = a.tau ? a.tau[k] : 1.f;
    const E* g = (const E*)a.gain + (long long)k * a.g_stride;
    const E* Rk = k == a.K - 1 ? (const E*)a.Wt : (const E*)a.Wh + (long long)k * a.wh_stride;
    const bool want_dg = !a.ebuf && (a.dg_mode == 2 || (a.dg_mode == 1 && k == a.K - 1));
    float* pw = pbuf + w * d;
    if (want_dg)
        for (int j = lane; j < d; j += 64) pw[j] = 0.f;
    for (int tr = w; tr < rows; tr += 4) {
        const int t = tile * rows + tr;
        if (t >= a.T) break;
        const long long row = (long long)k * a.T + t;
        // lane s holds split s
        f32x4 st = {-INFINITY, 0.f, 0.f, 0.f};
        if (lane < a.nsplit) st = *(const f32x4*)(a.split_stat + 4 * (lane * KT + row));
        float m = st[0], sx, zy = st[2];
        for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
        const float al = st[0] == m ? 1.f : __builtin_amdgcn_exp2f(st[0] - m);
        sx = lane < a.nsplit ? al * st[1] : 0.f;
        for (int off = 32; off > 0; off >>= 1) {
            sx += __shfl_xor(sx, off, 64);
            zy += __shfl_xor(zy, off, 64);
        }
        const int tgt = a.targets[row];
        const bool tok = tgt >= 0 && tgt < a.V;
        const RowEnd re = finish_row(m, sx, zy, tok);
        const float r = a.rstd[row];
        if (lane == 0) {
            a.rowloss[row] = re.loss;
            if (a.rowrec) {
                const f32x4 r4 = {F32FAM ? m : re.lse2, r * tau * kLog2e, __int_as_float(tgt), re.py1};
                *(f32x4*)(a.rowrec + 4 * row) = r4;
            }
            a.lse[row] = F32FAM ? re.inv_s : re.lse2 * kLn2;
        }
        const E* hr = (const E*)a.h + row * d;
        const E* wr = Rk + (long long)(tok ? tgt : 0) * d;
        f32x4 ev[kQ];
        float c = 0.f;
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
            const int j = 256 * q + 4 * lane;
            if (256 * q >= d) break;
            f32x4 s4 = {0.f, 0.f, 0.f, 0.f};
            if (j < d) {
                const float* p = a.split_acc + row * d + j;
                for (int s = 0; s < a.nsplit; ++s) {
                    // (a lane read: lane s itself may be past the width here)
                    const float as = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(al), s));
                    const f32x4 pv = *(const f32x4*)(p + s * KT * d);
#pragma unroll
                    for (int e = 0; e < 4; ++e) s4[e] = __builtin_fmaf(as, pv[e], s4[e]);
                }
                const f32x4 wv = ld4(wr + j), gv = ld4(g + j), hv = ld4(hr + j);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    s4[e] = __builtin_fmaf(s4[e], re.inv_s, re.py1 * (tok ? wv[e] : 0.f)) * a.inv_T;
                    c = __builtin_fmaf(gv[e] * s4[e], r * hv[e], c);
                }
            }
            ev[q] = s4;
        }
        for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off, 64);
        if (a.rowdtau && lane == 0) a.rowdtau[row] = tok ? c : 0.f;
        const float cm = tau * c / (float)d;
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
            const int j = 256 * q + 4 * lane;
            if (256 * q >= d) break;
            if (j >= d) continue;
            if (a.ebuf) {
                if (F32FAM) {
                    *(f32x4*)((float*)a.ebuf + row * d + j) = ev[q];
                } else {
                    bf16x4 hi, lo;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        hi[e] = (bf16)ev[q][e];
                        lo[e] = (bf16)(ev[q][e] - (float)hi[e]);
                    }
                    bf16* er = (bf16*)a.ebuf + row * (2LL * d);
                    *(bf16x4*)(er + j) = hi;
                    *(bf16x4*)(er + d + j) = lo;
                }
                continue;
            }
            const f32x4 gv = ld4(g + j), hv = ld4(hr + j);
            f32x4 o, pv;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float dhat = tau * ev[q][e];
                const float n = r * hv[e];
                o[e] = r * (gv[e] * dhat - cm * n);
                pv[e] = dhat * n;
            }
            st4((E*)a.dh + row * d + j, o);
            if (want_dg) *(f32x4*)(pw + j) += pv;
        }
    }
    if (want_dg) {
        __syncthreads();
        float* p = a.dgain_part + ((long long)(a.dg_mode == 2 ? k : 0) * gridDim.x + tile) * d;
        for (int j = threadIdx.x; j < d; j += 256) p[j] = ((pbuf[j] + pbuf[d + j]) + pbuf[2 * d + j]) + pbuf[3 * d + j];
    }
}

template <typename E, bool F32FAM>
hipError_t launch_t(const FusedArgs& a, int nmod, int rows, hipStream_t s) {
    const size_t lds = a.dg_mode ? (size_t)16 * a.d : 0;  // at most 64 KiB
    hipLaunchKernelGGL((k_merge<E, F32FAM>), dim3((unsigned)((a.T + rows - 1) / rows), (unsigned)nmod), dim3(256), lds,
                       s, a, rows);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_merge(int dtype, bool f32fam, const FusedArgs& a, int nmod, int rows, hipStream_t s) {
    if (dtype != 0) return launch_t<float, true>(a, nmod, rows, s);
    return f32fam ? launch_t<bf16, true>(a, nmod, rows, s) : launch_t<bf16, false>(a, nmod, rows, s);
}

}  // namespace solo
