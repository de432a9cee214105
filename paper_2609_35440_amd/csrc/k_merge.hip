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
// One workgroup per row (its mean is a workgroup reduction), e kept in registers
// between the two sweeps; fixed order throughout.  For a module that trains its
// gain e goes back to the first split's part of the row, and k_merge_dgain forms
// the token tiles' partials of sum_t dhhat_t n_t from it.  Bound by reading P
// once; a row per wave with the gain partials in the same kernel left 64 rows
// of 64 splits to 16 waves (565 us at d = 2048).
//
// Measured (fp32, K=2, T=1001, d=768, V=8003: 64 tiles): 2.22 ms per training
// call with one workgroup per tile, 0.95 split.  bf16 exit evaluation of 4 x 16
// rows, d=2048, V=32000: 2.10 ms on 4 workgroups, 0.064 split.
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

constexpr int kQ = 4;  // 1024-column groups of the widest row (4096)

// What the form's gradient passes read: the record's first entry is the
// log-sum-exp (base 2), or the maximum with 1 / s in the lse array (fp32
// kernels; they scale by that array, so the exact form, whose bias gradient they
// compute, leaves ones there); e goes to the rotate-back buffer as two bf16
// planes, or in fp32.
template <typename E, int FORM>
__global__ __launch_bounds__(256) void k_merge(FusedArgs a) {
    __shared__ float red[4];
    const int k = a.m0 + (int)blockIdx.y;
    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    const int d = a.d;
    const long long KT = a.part_rows;
    const long long row = (long long)k * a.T + blockIdx.x;
    const float tau = a.tau ? a.tau[k] : 1.f;
    const E* g = (const E*)a.gain + (long long)k * a.g_stride;
    const E* Rk = k == a.K - 1 ? (const E*)a.Wt : (const E*)a.Wh + (long long)k * a.wh_stride;
    const bool want_dg = !a.ebuf && (a.dg_mode == 2 || (a.dg_mode == 1 && k == a.K - 1));
    // lane s of every wave holds split s
    f32x4 st = {-INFINITY, 0.f, 0.f, 0.f};
    if (lane < a.nsplit) st = *(const f32x4*)(a.split_stat + 4 * (lane * KT + row));
    float m = st[0], zy = st[2];
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
    const float al = st[0] == m ? 1.f : __builtin_amdgcn_exp2f(st[0] - m);
    float sx = lane < a.nsplit ? al * st[1] : 0.f;
    for (int off = 32; off > 0; off >>= 1) {
        sx += __shfl_xor(sx, off, 64);
        zy += __shfl_xor(zy, off, 64);
    }
    const int tgt = a.targets[row];
    const bool tok = tgt >= 0 && tgt < a.V;
    const RowEnd re = finish_row<FORM != MERGE_BF16>(m, sx, zy, tok);
    const float r = a.rstd[row];
    if (threadIdx.x == 0) {
        a.rowloss[row] = re.loss;
        if (a.rowrec) {
            const f32x4 r4 = {FORM == MERGE_F32 ? m : re.lse2, r * tau * kLog2e, __int_as_float(tgt), re.py1};
            *(f32x4*)(a.rowrec + 4 * row) = r4;
        }
        a.lse[row] = FORM == MERGE_F32 ? re.inv_s : (FORM == MERGE_EXACT ? 1.f : re.lse2 * kLn2);
    }
    const E* hr = (const E*)a.h + row * d;
    const E* wr = Rk + (long long)(tok ? tgt : 0) * d;
    const int j0 = 4 * threadIdx.x;
    f32x4 ev[kQ];
    float c = 0.f;
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
        const int j = 1024 * q + j0;
        if (j >= d) break;
        f32x4 s4 = {0.f, 0.f, 0.f, 0.f};
        const float* p = a.split_acc + row * d + j;
#pragma unroll 8
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
        ev[q] = s4;
    }
    for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off, 64);
    if (lane == 0) red[w] = c;
    __syncthreads();
    c = (red[0] + red[1]) + (red[2] + red[3]);
    if (a.rowdtau && threadIdx.x == 0) a.rowdtau[row] = tok ? c : 0.f;
    const float cm = tau * c / (float)d;
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
        const int j = 1024 * q + j0;
        if (j >= d) break;
        if (a.ebuf) {
            if (FORM != MERGE_BF16) {
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
        f32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = r * (gv[e] * (tau * ev[q][e]) - cm * (r * hv[e]));
        st4((E*)a.dh + row * d + j, o);
        if (want_dg) *(f32x4*)(a.split_acc + row * d + j) = ev[q];
    }
}

// The partials of dgain = sum_t tau e_t n_t over `rows` tokens each: one thread per
// four columns of a partial.  Summed in 64 bits, as the partials are later on: a chain
// of up to 64 fp32 sums would cost more bits than the unsplit passes' trees.
template <typename E>
__global__ __launch_bounds__(256) void k_merge_dgain(FusedArgs a, int rows) {
    const int k = a.m0 + (int)blockIdx.y;
    if (a.dg_mode == 1 && k != a.K - 1) return;
    const int j = 4 * (blockIdx.z * 256 + threadIdx.x);
    if (j >= a.d) return;
    const int t0 = blockIdx.x * rows;
    const int t1 = t0 + rows < a.T ? t0 + rows : a.T;
    const float tau = a.tau ? a.tau[k] : 1.f;
    double s4[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int t = t0; t < t1; ++t) {
        const long long row = (long long)k * a.T + t;
        const float r = a.rstd[row];
        const f32x4 ev = *(const f32x4*)(a.split_acc + row * a.d + j);
        const f32x4 hv = ld4((const E*)a.h + row * a.d + j);
#pragma unroll
        for (int e = 0; e < 4; ++e) s4[e] = __builtin_fma((double)(tau * ev[e]), (double)(r * hv[e]), s4[e]);
    }
    *(f32x4*)(a.dgain_part + ((long long)(a.dg_mode == 2 ? k : 0) * gridDim.x + blockIdx.x) * a.d + j) =
        (f32x4){(float)s4[0], (float)s4[1], (float)s4[2], (float)s4[3]};
}

// Exit evaluation split over the vocabulary: the row's loss and top-1 (the
// larger logit, then the lower column) from the splits' parts; one row per wave.
template <bool FINE>
__global__ __launch_bounds__(256) void k_merge_eval(FusedArgs a, long long rows) {
    const int lane = threadIdx.x & 63;
    const long long row = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    // lane l holds splits l, l + 64, ..
    float ms[kEvalSplits / 64], ss[kEvalSplits / 64], m = -INFINITY, zy = 0.f, best = -INFINITY;
    int best_v = -1;
#pragma unroll
    for (int i = 0; i < kEvalSplits / 64; ++i) {
        const int s = 64 * i + lane;
        ms[i] = -INFINITY;
        ss[i] = 0.f;
        if (s < a.nsplit) {
            const float* sp = a.split_stat + 8 * (s * a.part_rows + row);
            const f32x4 st = *(const f32x4*)sp;
            const int v = __float_as_int(sp[4]);
            ms[i] = st[0];
            ss[i] = st[1];
            zy += st[2];
            m = fmaxf(m, st[0]);
            if (st[3] > best || (st[3] == best && (unsigned)v < (unsigned)best_v)) {
                best = st[3];
                best_v = v;
            }
        }
    }
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
    float sx = 0.f;
#pragma unroll
    for (int i = 0; i < kEvalSplits / 64; ++i)
        if (64 * i + lane < a.nsplit) sx += ms[i] == m ? ss[i] : ss[i] * __builtin_amdgcn_exp2f(ms[i] - m);
    for (int off = 32; off > 0; off >>= 1) {
        sx += __shfl_xor(sx, off, 64);
        zy += __shfl_xor(zy, off, 64);
        const float ob = __shfl_xor(best, off, 64);
        const int ov = __shfl_xor(best_v, off, 64);
        if (ob > best || (ob == best && (unsigned)ov < (unsigned)best_v)) {
            best = ob;
            best_v = ov;
        }
    }
    if (lane == 0) {
        const int tgt = a.targets[row];
        a.rowloss[row] = finish_row<FINE>(m, sx, zy, tgt >= 0 && tgt < a.V).loss;
        if (a.top1) a.top1[row] = best_v;
    }
}

template <typename E, int FORM>
hipError_t launch_t(const FusedArgs& a, int nmod, int rows, hipStream_t s) {
    hipLaunchKernelGGL((k_merge<E, FORM>), dim3((unsigned)a.T, (unsigned)nmod), dim3(256), 0, s, a);
    const hipError_t e = hipGetLastError();
    // (the terminal's gain alone: only a launch that holds the terminal has partials)
    if (e != hipSuccess || a.ebuf || !a.dg_mode || (a.dg_mode == 1 && a.m0 + nmod != a.K)) return e;
    const dim3 grid((unsigned)((a.T + rows - 1) / rows), (unsigned)nmod, (unsigned)((a.d + 1023) / 1024));
    hipLaunchKernelGGL((k_merge_dgain<E>), grid, dim3(256), 0, s, a, rows);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_merge_eval(const FusedArgs& a, bool fine, long long rows, hipStream_t s) {
    const dim3 grid((unsigned)((rows + 3) / 4));
    if (fine) {
        hipLaunchKernelGGL(k_merge_eval<true>, grid, dim3(256), 0, s, a, rows);
    } else {
        hipLaunchKernelGGL(k_merge_eval<false>, grid, dim3(256), 0, s, a, rows);
    }
    return hipGetLastError();
}

hipError_t launch_merge(int dtype, MergeForm form, const FusedArgs& a, int nmod, int rows, hipStream_t s) {
    if (dtype != 0) return launch_t<float, MERGE_F32>(a, nmod, rows, s);
    return form == MERGE_BF16 ? launch_t<bf16, MERGE_BF16>(a, nmod, rows, s)
           : form == MERGE_F32 ? launch_t<bf16, MERGE_F32>(a, nmod, rows, s)
                               : launch_t<bf16, MERGE_EXACT>(a, nmod, rows, s);
}

}  // namespace solo
