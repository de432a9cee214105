// fp32 passes of the SOLO shared-readout loss on the fp32 matrix instructions
// (products and sums in fp32, on fp32 or bf16 storage).  They serve the fp32
// configuration, where the products must be true fp32 products, and the bf16
// widths that the bf16 matrix-core kernels do not tile (of those, the passes with a
// second product run in the exact form of k_mfma.hip and k_exact_wide.hip from
// d = 72 on, and exit evaluation as a product on planes, k_logits.hip).  Same passes and notation as
// k_mfma.hip (z_tv = tau_k <R_kv, hhat_t> + b_kv, hhat = g_k * r_t h_t): a tile
// of R stationary rows X, the other operand Y streamed in chunks of 256 rows,
// the T x V logits never written.
//
//   local-loss pass: X = g * h_t (r_t tau a row scale of the logits), Y = readout rows
//   exit evaluation: the same without the second product, plus the top-1
//   readout-gradient pass: X = g * R_v, Y = h_t; dR_v = g * sum_t delta_tv tau r_t h_t
//   bias-gradient pass: the same without the second product
//
// Per chunk of 256 streamed rows:
//   logits: wave w owns 32 of the chunk's rows against all R stationary rows.
//     Slabs of 128 bytes of k go buffer -> LDS directly for Y (each wave its
//     own 32 rows) and through registers for X (times the gain), both double-
//     buffered; one barrier per slab.
//   softmax: the wave's row maxima meet in LDS (the running maximum is
//     re-based only past a threshold, so all waves agree on it), each lane
//     turns its own logits into probabilities and writes them to the tile
//     G[x][y].
//   second product: wave w owns a column slice of the accumulator [R][d] and
//     contracts over the 256 rows of the chunk, its streamed operand read straight
//     from global memory (L2) in row segments.
// The fp32 matrix rate (256 flop/clk per CU, a sixteenth of bf16's) bounds
// the pass: a chunk of 256 rows is R d / 32 KiB of work per barrier pair, so
// the barriers and the exchange, which bound the bf16 passes, do not show.
// R = 32 while the accumulator fits the registers next to the streamed
// operand (d <= 2048: 128 registers at 256 columns per wave), 16 above.
//
// Measured (K=2, T=1001, d=768, V=8003, fp32): 0.95 ms per training call, 14.7
// with one thread per column on the vector ALU.
//
// Sums: a logit's k-sum is cut into pieces of 256, each summed by itself, so
// its rounding does not grow with d as one chain would.
#include "mfma_common.h"

namespace solo {

namespace {

using namespace mfma;

constexpr int NW = 8;
constexpr int NTHR = NW * 64;
constexpr int YC = 256;  // streamed rows per chunk, 32 per wave
constexpr int YW = YC / NW;

enum Mode { LOCAL = 0, RGRAD = 1, BGRAD = 2, EVAL = 3 };

typedef int i32x2 __attribute__((ext_vector_type(2)));

// R x R matrix instruction of fp32 operands: lane l holds A[m = l % R][k = l / R]
// and B[k = l / R][n = l % R]; C register i of lane l is C[row(i)][n = l % R],
// row(i) = 8 (i / 4) + 4 (l / R) + i % 4 (the first term only for R = 32).
template <int R> struct Mf;
template <> struct Mf<32> {
    typedef f32x16 C;
    static constexpr int NR = 16, KG = 2;
    static __device__ __forceinline__ C mul(float a, float b, C c) {
        return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
    }
};
template <> struct Mf<16> {
    typedef f32x4 C;
    static constexpr int NR = 4, KG = 4;
    static __device__ __forceinline__ C mul(float a, float b, C c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
};

template <typename E> struct El;
template <> struct El<float> {
    static constexpr int ES = 4, KE = 4;
    // the KE elements of a 16-byte granule
    static __device__ __forceinline__ void unpack(i32x4 g, float* o) {
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = __int_as_float(g[e]);
    }
};
template <> struct El<bf16> {
    static constexpr int ES = 2, KE = 8;
    static __device__ __forceinline__ void unpack(i32x4 g, float* o) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            o[2 * e] = __int_as_float(g[e] << 16);
            o[2 * e + 1] = __int_as_float(g[e] & (int)0xffff0000);
        }
    }
};

template <typename E> __device__ __forceinline__ float ldf(const E* p) { return (float)*p; }
__device__ __forceinline__ f32x4 ld4f(const float* p) { return *(const f32x4*)p; }
__device__ __forceinline__ f32x4 ld4f(const bf16* p) {
    const u16x4 v = *(const u16x4*)p;
    return f32x4{bf16_bits_to_f32(v[0]), bf16_bits_to_f32(v[1]), bf16_bits_to_f32(v[2]), bf16_bits_to_f32(v[3])};
}
// CW adjacent elements of a row (CW-element aligned), in fp32
template <int CW, typename E>
__device__ __forceinline__ void ldv(const E* p, float* o) {
    typedef E EV __attribute__((ext_vector_type(CW)));
    if constexpr (CW == 1) {
        o[0] = ldf(p);
    } else {
        const EV v = *(const EV*)p;
#pragma unroll
        for (int e = 0; e < CW; ++e) o[e] = (float)v[e];
    }
}
template <int CW, typename E>
__device__ __forceinline__ void stv(E* p, const float* o) {
    typedef E EV __attribute__((ext_vector_type(CW)));
    if constexpr (CW == 1) {
        p[0] = (E)o[0];
    } else {
        EV v;
#pragma unroll
        for (int e = 0; e < CW; ++e) v[e] = (E)o[e];
        *(EV*)p = v;
    }
}

// CW adjacent elements of a row through a buffer resource (zeros past its end)
template <typename E, int CW> struct Seg;
template <> struct Seg<float, 1> {
    float r;
    __device__ __forceinline__ void ld(__amdgpu_buffer_rsrc_t rs, int vo) {
        r = __int_as_float((int)__builtin_amdgcn_raw_buffer_load_b32(rs, vo, 0, 0));
    }
    __device__ __forceinline__ float get(int) const { return r; }
};
template <> struct Seg<float, 2> {
    i32x2 r;
    __device__ __forceinline__ void ld(__amdgpu_buffer_rsrc_t rs, int vo) {
        r = __builtin_bit_cast(i32x2, __builtin_amdgcn_raw_buffer_load_b64(rs, vo, 0, 0));
    }
    __device__ __forceinline__ float get(int e) const { return __int_as_float(r[e]); }
};
template <> struct Seg<float, 4> {
    i32x4 r;
    __device__ __forceinline__ void ld(__amdgpu_buffer_rsrc_t rs, int vo) {
        r = __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, vo, 0, 0));
    }
    __device__ __forceinline__ float get(int e) const { return __int_as_float(r[e]); }
};
template <> struct Seg<bf16, 1> {
    unsigned short r;
    __device__ __forceinline__ void ld(__amdgpu_buffer_rsrc_t rs, int vo) {
        r = __builtin_amdgcn_raw_buffer_load_b16(rs, vo, 0, 0);
    }
    __device__ __forceinline__ float get(int) const { return bf16_bits_to_f32(r); }
};

// The column slices of the accumulator: NG groups of R CW columns per wave
// (lane m of a group holds columns CW m .. + CW - 1); with YS > 1 only 8 / YS
// waves hold distinct columns and YS waves share each slice, a YS-th of the
// chunk's rows each (narrow rows, d <= 128).
template <typename E, int MODE, int R, int NG, int CW, int YS>
__global__ __launch_bounds__(NTHR, 1) void k_fused_f32(FusedArgs a) {
    constexpr bool LL = MODE == LOCAL || MODE == EVAL;   // X = g * h, Y = readout
    constexpr bool PC = MODE == LOCAL || MODE == RGRAD;  // second product
    using M = Mf<R>;
    using T = El<E>;
    typedef typename M::C C;
    constexpr int KG = M::KG, NR = M::NR, KE = T::KE, ES = T::ES;
    constexpr int KS = 128 / ES;     // k per slab
    constexpr int NBV = YW / R;      // R-row blocks of the wave's 32 streamed rows
    constexpr int XG = KS / 4;       // 16-byte granules of an X slab row (fp32)
    constexpr int NCG = NW / YS;     // waves with distinct columns
    constexpr int FLUSH = 256 / KS;  // slabs per piece of a logit's k-sum
    constexpr int GBUF = PC ? R * YC : 4;
    constexpr int U = NG * CW >= 24 ? 2 : (NG * CW >= 4 ? 4 : 8);
    __shared__ __attribute__((aligned(16))) char ys0[NW * YW * 128];
    __shared__ __attribute__((aligned(16))) char ys1[NW * YW * 128];
    __shared__ __attribute__((aligned(16))) float xs0[R * KS];
    __shared__ __attribute__((aligned(16))) float xs1[R * KS];
    __shared__ __attribute__((aligned(16))) float gbuf[GBUF];
    __shared__ float wred[NW * R];
    __shared__ float wred2[NW * R];
    __shared__ float sbuf[R];
    __shared__ float pybuf[R];
    __shared__ __attribute__((aligned(16))) float rec[LL ? 4 : YC * 4];
    __shared__ float recs[LL ? 1 : YC];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ln = lane % R;  // stationary row of the lane (n), or operand row (m)
    const int kq = lane / R;
    const int d = a.d;
    const int nsplit = (MODE == LOCAL) ? a.nsplit : 1;
    const int sp = (int)blockIdx.x % nsplit;  // (splits next to each other, as in k_mfma.hip)
    const int x0 = ((int)blockIdx.x / nsplit) * R;
    const int k = a.m0 + (int)blockIdx.y;
    const long long modoff = (long long)k * a.T;
    const float tau = a.tau ? a.tau[k] : 1.f;
    const E* hk = (const E*)a.h + modoff * d;
    const E* Rk = k == a.K - 1 ? (const E*)a.Wt : (const E*)a.Wh + (long long)k * a.wh_stride;
    const E* gk = (const E*)a.gain + (long long)k * a.g_stride;
    const float* bk = a.bias ? a.bias + (long long)k * a.V : nullptr;
    const E* X = LL ? hk : Rk;
    const E* Y = LL ? Rk : hk;
    const int nX = LL ? a.T : a.V;
    const int nY = LL ? a.V : a.T;
    const int nchunks = (nY + YC - 1) / YC;
    // chunks of this workgroup (the local-loss pass may be split over the vocabulary)
    const int c_lo = (int)((long long)nchunks * sp / nsplit);
    const int c_hi = (int)((long long)nchunks * (sp + 1) / nsplit);
    const int nslab = (d + KS - 1) / KS;

    const int xg = x0 + ln;  // the lane's stationary row
    const bool xok = xg < nX;
    float own_r2 = 0.f;  // LL: r_t tau log2 e
    int own_tgt = -1;
    float bx2 = 0.f;
    if (LL && xok) {
        own_r2 = a.rstd[modoff + xg] * tau * kLog2e;
        own_tgt = a.targets[modoff + xg];
    }
    if (!LL && bk && xok) bx2 = bias2(bk[xg]);

    // ---- streams
    // Y slab: instruction q writes rows 8 q + lane / 8 of the wave's 32, 16-byte
    // slot lane % 8 of a row holding granule (lane % 8) ^ (row & 7): the reads
    // of 8 rows at one granule then cover all banks
    const int ygr = (lane & 7) ^ (lane >> 3);
    const int yvo = ((YW * w + (lane >> 3)) * d) * ES + 16 * ygr;
    auto yrsrc = [&](int c) __attribute__((always_inline)) {
        const int y0 = c * YC;
        const int rows = nY - y0 < YC ? nY - y0 : YC;
        return make_rsrc(Y + (long long)y0 * d, (unsigned)rows * (unsigned)(d * ES));
    };
    LDS_AS char* const yp0 = (LDS_AS char*)(LDS_AS void*)ys0 + w * (YW * 128);
    LDS_AS char* const yp1 = (LDS_AS char*)(LDS_AS void*)ys1 + w * (YW * 128);
    LDS_AS float* const xp0 = (LDS_AS float*)(LDS_AS void*)xs0;
    LDS_AS float* const xp1 = (LDS_AS float*)(LDS_AS void*)xs1;
    const unsigned yl0 = lds_addr(yp0), yl1 = lds_addr(yp1);
    auto issue_y = [&](i32x4 rs, int s, unsigned dst) __attribute__((always_inline)) {
        // columns past d: an offset past the range, which reads as zero
        const int vo = s * KS + ygr * KE < d ? yvo + s * 128 : 0x40000000;
#pragma unroll
        for (int q = 0; q < YW / 8; ++q) buffer_load_lds16(rs, dst + q * 1024, vo + q * 8 * d * ES);
    };
    // X slab: four k of one row per thread
    const bool xthr = tid < R * XG;
    const int xr = tid / XG, xc = tid % XG;
    f32x4 xst;
    auto load_x = [&](int s) __attribute__((always_inline)) {
        xst = f32x4{0.f, 0.f, 0.f, 0.f};
        const int j = s * KS + 4 * xc;
        if (xthr && x0 + xr < nX && j < d) xst = ld4f(X + (long long)(x0 + xr) * d + j) * ld4f(gk + j);
    };
    auto store_x = [&](LDS_AS float* xs) __attribute__((always_inline)) {
        if (xthr) *(LDS_AS f32x4*)(xs + xr * KS + 4 * (xc ^ (xr & 7))) = xst;
    };

    C acc[PC ? NG : 1][PC ? CW : 1];
#pragma unroll
    for (int g = 0; g < (PC ? NG : 1); ++g)
#pragma unroll
        for (int e = 0; e < (PC ? CW : 1); ++e)
#pragma unroll
            for (int i = 0; i < NR; ++i) acc[g][e][i] = 0.f;
    const int cg = w % NCG, ysub = w / NCG;
    const int js = cg * (R * CW * NG);

    float m_run = -INFINITY, s_part = 0.f, zy_part = 0.f;
    double db_part = 0.0;  // (a sum over all tokens: four at a time in fp32, then in 64 bits)
    float best = -INFINITY;
    int best_v = -1;

    // one slab of the logit products: S += Y_slab X_slab^T for the wave's rows
    auto slab = [&](LDS_AS const char* ysw, LDS_AS const float* xs, C* S) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < KS / (KG * KE); ++t) {
            const int ga = t * KG + kq;
            float xv[KE];
#pragma unroll
            for (int p = 0; p < KE / 4; ++p) {
                const f32x4 v = *(LDS_AS const f32x4*)(xs + ln * KS + 4 * (((KE / 4) * ga + p) ^ (ln & 7)));
#pragma unroll
                for (int e = 0; e < 4; ++e) xv[4 * p + e] = v[e];
            }
#pragma unroll
            for (int b = 0; b < NBV; ++b) {
                const int row = b * R + ln;
                float yv[KE];
                T::unpack(*(LDS_AS const i32x4*)(ysw + row * 128 + 16 * (ga ^ (row & 7))), yv);
#pragma unroll
                for (int e = 0; e < KE; ++e) S[b] = M::mul(yv[e], xv[e], S[b]);
            }
        }
    };

    i32x4 yrs = yrsrc(c_lo);
    if (c_lo < c_hi) {
        issue_y(yrs, 0, yl0);
        load_x(0);
        store_x(xp0);
    }
    int par = 0;  // which slab buffer holds the next slab
    for (int c = c_lo; c < c_hi; ++c) {
        const int y0 = c * YC;
        const int rows = nY - y0 < YC ? nY - y0 : YC;
        C S[NBV], St[NBV];
#pragma unroll
        for (int b = 0; b < NBV; ++b)
#pragma unroll
            for (int i = 0; i < NR; ++i) S[b][i] = St[b][i] = 0.f;
        for (int s = 0; s < nslab; ++s) {
            wait_vm();
            lds_barrier();  // slab (c, s) is complete; the other buffer is free
            const bool last = s + 1 == nslab;
            if (!last || c + 1 < c_hi) {
                if (last) yrs = yrsrc(c + 1);
                issue_y(yrs, last ? 0 : s + 1, par ? yl0 : yl1);
                load_x(last ? 0 : s + 1);
            }
            if (!LL && s == 0 && tid < YC) {
                // the chunk's token records {m, r tau log2 e, target, p_y - 1} and 1 / s
                const int t = y0 + tid;
                f32x4 r4 = {0.f, 0.f, __int_as_float(-1), 0.f};
                float is = 0.f;
                if (t < nY) {
                    r4 = *(const f32x4*)(a.rowrec + 4 * (modoff + t));
                    is = a.lse[modoff + t];
                }
                *(f32x4*)(rec + 4 * tid) = r4;
                recs[tid] = is;
            }
            slab(par ? yp1 : yp0, par ? xp1 : xp0, S);
            if ((s + 1) % FLUSH == 0 || last) {
#pragma unroll
                for (int b = 0; b < NBV; ++b)
#pragma unroll
                    for (int i = 0; i < NR; ++i) {
                        St[b][i] += S[b][i];
                        S[b][i] = 0.f;
                    }
            }
            if (!last || c + 1 < c_hi) store_x(par ? xp0 : xp1);
            par ^= 1;
        }

        const int ylow = YW * w;  // the wave's rows of the chunk
        if (LL) {
            float zmax = -INFINITY;
#pragma unroll
            for (int b = 0; b < NBV; ++b)
#pragma unroll
                for (int i = 0; i < NR; ++i) {
                    const int yl = ylow + b * R + (R == 32 ? 8 * (i >> 2) : 0) + 4 * kq + (i & 3);
                    float zc = St[b][i] * own_r2;
                    if (bk) zc = __builtin_fmaf(St[b][i], own_r2, yl < rows ? bias2(bk[y0 + yl]) : 0.f);
                    zc = yl < rows ? zc : -INFINITY;
                    St[b][i] = zc;
                    zmax = fmaxf(zmax, zc);
                    if (MODE == EVAL && zc > best) {  // strict: the first (lowest) column keeps a tie
                        best = zc;
                        best_v = y0 + yl;
                    }
                }
#pragma unroll
            for (int off = R; off < 64; off <<= 1) zmax = fmaxf(zmax, __shfl_xor(zmax, off, 64));
            if (PC) {
                // all waves take the same decision for a row: they share the probability tile
                if (lane < R) wred[w * R + ln] = zmax;
                lds_barrier();
#pragma unroll
                for (int ww = 0; ww < NW; ++ww) zmax = fmaxf(zmax, wred[ww * R + ln]);
            }
            float alpha = 1.f;
            if (zmax > m_run + kLazyThresh2) {
                alpha = __builtin_amdgcn_exp2f(m_run - zmax);
                s_part *= alpha;
                m_run = zmax;
            }
#pragma unroll
            for (int b = 0; b < NBV; ++b)
#pragma unroll
                for (int i4 = 0; i4 < NR / 4; ++i4) {
                    const int yl = ylow + b * R + 8 * i4 + 4 * kq;
                    f32x4 g;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float zc = St[b][4 * i4 + e];
                        const bool is_y = own_tgt - y0 == yl + e;
                        float p = zc == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(zc - m_run);
                        if (is_y) {
                            // the target's term joins at the end of the row (finish_row), and its
                            // probability the input gradient in the epilogue
                            zy_part = zc;
                            p = 0.f;
                        }
                        s_part += p;
                        g[e] = p;
                    }
                    if (PC) *(f32x4*)(gbuf + ln * YC + 4 * ((yl >> 2) ^ (ln & 7))) = g;
                }
            if (PC && __any(alpha != 1.f)) {
#pragma unroll
                for (int g = 0; g < (PC ? NG : 1); ++g)
#pragma unroll
                    for (int e = 0; e < (PC ? CW : 1); ++e)
#pragma unroll
                        for (int i = 0; i < NR; ++i) acc[g][e][i] *= alpha;
            }
        } else {
            lds_barrier();  // the records
#pragma unroll
            for (int b = 0; b < NBV; ++b)
#pragma unroll
                for (int i4 = 0; i4 < NR / 4; ++i4) {
                    const int yl = ylow + b * R + 8 * i4 + 4 * kq;
                    f32x4 g, dl;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const f32x4 r4 = *(const f32x4*)(rec + 4 * (yl + e));
                        const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(St[b][4 * i4 + e], r4[1], bx2 - r4[0])) *
                                        recs[yl + e];
                        // tokens past the end are masked; the target's entry of delta is the
                        // exact p_y - 1 of the local-loss pass
                        dl[e] = yl + e < rows ? (__float_as_int(r4[2]) == xg ? r4[3] : p) : 0.f;
                        g[e] = dl[e] * (r4[1] * (kLn2 * a.inv_T));  // times r tau / T
                    }
                    db_part += (double)((dl[0] + dl[1]) + (dl[2] + dl[3]));
                    if (PC) *(f32x4*)(gbuf + ln * YC + 4 * ((yl >> 2) ^ (ln & 7))) = g;
                }
        }

        if (PC) {
            // ---- second product: acc[j][x] += sum_y Y[y][j] G[x][y]; step s takes rows
            // 4 KG s + 4 kq + i, i = 0..3
            const __amdgpu_buffer_rsrc_t ars = __builtin_amdgcn_make_buffer_rsrc(
                (void*)(Y + (long long)y0 * d), (short)0, rows * (d * ES), 0x00020000);
            const int avo = (4 * kq * d + js + CW * ln) * ES;
            // the operand segments of U rows in flight per group (a row's registers are
            // reloaded right after its products): as many as the registers hold
            Seg<E, CW> wa[U][PC ? NG : 1];
            auto load_a = [&](int slot, int row) __attribute__((always_inline)) {
#pragma unroll
                for (int g = 0; g < (PC ? NG : 1); ++g)
                    wa[slot][g].ld(ars, avo + (row * d + R * CW * g) * ES);
            };
            // steps of this wave (rows past the end read as zeros and meet zeros in the tile)
            constexpr int NS = YC / (4 * KG) / YS;
            constexpr int SU = U > 4 ? U / 4 : 1;  // steps per turn of the ring
            static_assert(NS % SU == 0, "whole turns");
            const int s_lo = ysub * NS;
            const int live = (rows + 4 * KG - 1) / (4 * KG) - s_lo;
            const int ns = js < d ? (live < NS ? live : NS) : 0;  // a slice past the width has nothing to do
            if (ns > 0) {
#pragma unroll
                for (int u = 0; u < U; ++u) load_a(u, 4 * KG * (s_lo + u / 4) + u % 4);
            }
            lds_barrier();  // the probability tile is complete
            for (int s = 0; s < ns; s += SU) {
                f32x4 gv;
#pragma unroll
                for (int u = 0; u < 4 * SU; ++u) {
                    if (u % 4 == 0)
                        gv = *(const f32x4*)(gbuf + ln * YC + 4 * ((KG * (s_lo + s + u / 4) + kq) ^ (ln & 7)));
#pragma unroll
                    for (int g = 0; g < (PC ? NG : 1); ++g)
#pragma unroll
                        for (int e = 0; e < (PC ? CW : 1); ++e)
                            acc[g][e] = M::mul(wa[u % U][g].get(e), gv[u % 4], acc[g][e]);
                    load_a(u % U, 4 * KG * (s_lo + s + (u + U) / 4) + (u + U) % 4);
                }
            }
        }
    }

    // ---- epilogues
    if (LL) {
        // row sums over the lanes and waves of a row
#pragma unroll
        for (int off = R; off < 64; off <<= 1) {
            s_part += __shfl_xor(s_part, off, 64);
            zy_part += __shfl_xor(zy_part, off, 64);
            if (MODE == EVAL) {
                const float ob = __shfl_xor(best, off, 64);
                const int ov = __shfl_xor(best_v, off, 64);
                if (ob > best || (ob == best && (unsigned)ov < (unsigned)best_v)) {
                    best = ob;
                    best_v = ov;
                }
            }
        }
        if (MODE == EVAL) {
            // every wave has its own running maximum: bring the sums to the common one
            if (lane < R) wred[w * R + ln] = m_run;
            __syncthreads();
            float m = m_run;
#pragma unroll
            for (int ww = 0; ww < NW; ++ww) m = fmaxf(m, wred[ww * R + ln]);
            if (m_run != m) s_part *= __builtin_amdgcn_exp2f(m_run - m);
            m_run = m;
            __syncthreads();
            // top-1 over the waves: larger logit, then lower column
            float* bb = (float*)ys0;
            int* bv = (int*)ys1;
            if (lane < R) {
                bb[w * R + ln] = best;
                bv[w * R + ln] = best_v;
            }
            __syncthreads();
#pragma unroll
            for (int ww = 0; ww < NW; ++ww) {
                const float ob = bb[ww * R + ln];
                const int ov = bv[ww * R + ln];
                if (ob > best || (ob == best && (unsigned)ov < (unsigned)best_v)) {
                    best = ob;
                    best_v = ov;
                }
            }
        } else {
            __syncthreads();
        }
        if (lane < R) {
            wred[w * R + ln] = s_part;
            wred2[w * R + ln] = zy_part;
        }
        __syncthreads();
        float sx = 0.f, zy = 0.f;
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) {
            sx += wred[ww * R + ln];
            zy += wred2[ww * R + ln];
        }
        if (MODE == LOCAL && nsplit > 1) {
            if (w == 0 && lane < R && xok) {
                const long long p = (long long)sp * a.part_rows + modoff + xg;
                const f32x4 st = {m_run, sx, zy, 0.f};
                *(f32x4*)(a.split_stat + 4 * p) = st;
            }
        } else if (w == 0 && lane < R) {
            const bool tok = own_tgt >= 0 && own_tgt < nY;
            const RowEnd re = finish_row<true>(m_run, sx, zy, tok);
            if (xok) {
                const long long t = modoff + xg;
                a.rowloss[t] = re.loss;
                if (MODE == EVAL && a.top1) a.top1[t] = best_v;
                if (MODE == LOCAL && a.rowrec) {
                    const f32x4 r4 = {m_run, own_r2, __int_as_float(own_tgt), re.py1};
                    *(f32x4*)(a.rowrec + 4 * t) = r4;
                    a.lse[t] = re.inv_s;
                }
            }
            sbuf[ln] = re.inv_s;
            pybuf[ln] = re.py1;
        }
    }
    if (PC && YS > 1) {
        // the waves that share a column slice: sums in wave order
        __syncthreads();
        float* red = (float*)ys0;  // NW x 64 lanes x NR floats (CW = NG = 1): 32 KiB
        static_assert(YS == 1 || (NG == 1 && CW == 1 && NW * 64 * NR * 4 <= NW * YW * 128), "slice reduction in LDS");
#pragma unroll
        for (int i = 0; i < NR; ++i) red[(w * NR + i) * 64 + lane] = acc[0][0][i];
        __syncthreads();
        if (ysub == 0) {
#pragma unroll
            for (int u = 1; u < YS; ++u)
#pragma unroll
                for (int i = 0; i < NR; ++i) acc[0][0][i] += red[((w + u * NCG) * NR + i) * 64 + lane];
        }
    }
    const bool own = ysub == 0;  // this wave's columns are its own in the epilogue
    // acc[g][e][i] is column col(g, i) + e: CW adjacent columns, all inside the
    // width or all past it (CW divides 8 and d is a multiple of 8)
    auto col = [&](int g, int i) __attribute__((always_inline)) {
        return js + R * CW * g + CW * ((R == 32 ? 8 * (i >> 2) : 0) + 4 * kq + (i & 3));
    };
    // one group of columns at a time (a scheduling barrier each: all loads at
    // once would not fit the registers next to the accumulator)
    auto each = [&](auto f) __attribute__((always_inline)) {
#pragma unroll
        for (int g = 0; g < (PC ? NG : 1); ++g)
#pragma unroll
            for (int i = 0; i < NR; ++i) {
                f(g, i, col(g, i));
                __builtin_amdgcn_sched_barrier(0);
            }
    };
    constexpr int CV = PC ? CW : 1;
    if (MODE == LOCAL && nsplit > 1) {
        // the unnormalised partial sums of this split, for the merge
        if (own && xok) {
            float* P = a.split_acc + ((long long)sp * a.part_rows + modoff + xg) * d;
            each([&](int g, int i, int j) __attribute__((always_inline)) {
                float o[CV];
#pragma unroll
                for (int e = 0; e < CV; ++e) o[e] = acc[g][e][i];
                if (j < d) stv<CV>(P + j, o);
            });
        }
        return;
    }
    if (MODE == LOCAL) {
        __syncthreads();
        const bool want_dg = a.dg_mode == 2 || (a.dg_mode == 1 && k == a.K - 1);
        const float rx = xok ? a.rstd[modoff + xg] : 0.f;
        const bool tok = xok && own_tgt >= 0 && own_tgt < nY;
        const float inv_s = sbuf[ln], py1 = pybuf[ln];
        const E* hrow = hk + (long long)(xok ? xg : 0) * d;
        const E* wrow = Rk + (long long)(tok ? own_tgt : 0) * d;
        // e = (acc / s + (p_y - 1) R_y) / T, dhhat = tau e; the row sum of e g n is both
        // d mean(dn n) / tau and the token's d loss / d tau
        float cp = 0.f;
        if (own) {
            each([&](int g, int i, int j) __attribute__((always_inline)) {
                const int jc = j < d ? j : 0;
                float wv[CV], gv[CV], hv[CV];
                ldv<CV>(wrow + jc, wv);
                ldv<CV>(gk + jc, gv);
                ldv<CV>(hrow + jc, hv);
#pragma unroll
                for (int e = 0; e < CV; ++e) {
                    float ev = __builtin_fmaf(acc[g][e][i], inv_s, py1 * (tok ? wv[e] : 0.f)) * a.inv_T;
                    ev = j < d ? ev : 0.f;
                    cp = __builtin_fmaf(gv[e] * ev, rx * hv[e], cp);
                    acc[g][e][i] = ev;
                }
            });
        }
#pragma unroll
        for (int off = R; off < 64; off <<= 1) cp += __shfl_xor(cp, off, 64);
        if (lane < R) wred[w * R + ln] = cp;
        __syncthreads();
        float csum = 0.f;
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) csum += wred[ww * R + ln];
        const float cmean = tau * csum / (float)d;
        if (a.rowdtau && w == 0 && lane < R && xok) a.rowdtau[modoff + xg] = tok ? csum : 0.f;
        if (!own) return;
        if (a.ebuf) {
            // e to the buffer; the RMSNorm backward follows the rotation back (ROT heads)
            if (!xok) return;
            float* eb = (float*)a.ebuf + (modoff + xg) * (long long)d;
            each([&](int g, int i, int j) __attribute__((always_inline)) {
                float o[CV];
#pragma unroll
                for (int e = 0; e < CV; ++e) o[e] = acc[g][e][i];
                if (j < d) stv<CV>(eb + j, o);
            });
            return;
        }
        E* out = (E*)a.dh + (modoff + (xok ? xg : 0)) * (long long)d;
        // the gain partials of the tile's groups of 8 rows
        const long long ngp = (a.T + kF32GainRows - 1) / kF32GainRows;
        float* dgp = want_dg ? a.dgain_part + ((a.dg_mode == 2 ? k : 0) * ngp + (x0 + ln) / kF32GainRows) * d : nullptr;
        each([&](int g, int i, int j) __attribute__((always_inline)) {
            const int jc = j < d ? j : 0;
            float gv[CV], hv[CV], o[CV];
            ldv<CV>(gk + jc, gv);
            ldv<CV>(hrow + jc, hv);
#pragma unroll
            for (int e = 0; e < CV; ++e) {
                const float n = rx * hv[e];
                const float dhat = tau * acc[g][e][i];
                o[e] = rx * (gv[e] * dhat - cmean * n);
                if (want_dg) {
                    // sum_t dhhat_t n_t over 8 rows (rx = 0 masks rows past the end)
                    const float t = row8_sum(dhat * n);
                    if (j < d && ln % kF32GainRows == 0 && xok) dgp[j + e] = t;
                }
            }
            if (j < d && xok) stv<CV>(out + j, o);
        });
    }
    if (!LL) {
        // bias gradient of the stationary readout rows
#pragma unroll
        for (int off = R; off < 64; off <<= 1) db_part += __shfl_xor(db_part, off, 64);
        if (lane < R) wred[w * R + ln] = (float)db_part;
        __syncthreads();
        if (a.dbias && w == 0 && lane < R && xok) {
            double db = 0.0;
#pragma unroll
            for (int ww = 0; ww < NW; ++ww) db += (double)wred[ww * R + ln];
            a.dbias[(long long)k * a.V + xg] = (float)db * a.inv_T;
        }
    }
    if (MODE == RGRAD && own && xok) {
        float* dR = ((k == a.K - 1) ? a.dWt : a.dWh + (long long)k * a.V * d) + (long long)xg * d;
        each([&](int g, int i, int j) __attribute__((always_inline)) {
            float gv[CV], o[CV];
            ldv<CV>(gk + (j < d ? j : 0), gv);
#pragma unroll
            for (int e = 0; e < CV; ++e) o[e] = gv[e] * acc[g][e][i];
            if (j < d) stv<CV>(dR + j, o);
        });
    }
}

template <typename E, int MODE, int R, int NG, int CW, int YS>
hipError_t launch_t(const FusedArgs& a, int nmod, hipStream_t s) {
    const bool ll = MODE == LOCAL || MODE == EVAL;
    const int nx = ll ? a.T : a.V;
    dim3 grid((unsigned)((nx + R - 1) / R * (MODE == LOCAL ? a.nsplit : 1)), (unsigned)nmod);
    hipLaunchKernelGGL((k_fused_f32<E, MODE, R, NG, CW, YS>), grid, dim3(NTHR), 0, s, a);
    return hipGetLastError();
}

// passes with a second product: columns per wave by width (bf16 storage up to 64:
// wider rows run in the exact form)
template <typename E, int MODE>
hipError_t launch_w(const FusedArgs& a, int nmod, hipStream_t s) {
    const int d = a.d;
    if (d <= 32) return launch_t<E, MODE, 32, 1, 1, 8>(a, nmod, s);
    if (d <= 64) return launch_t<E, MODE, 32, 1, 1, 4>(a, nmod, s);
    if constexpr (sizeof(E) == 4) {
        if (d <= 128) return launch_t<E, MODE, 32, 1, 1, 2>(a, nmod, s);
        if (d <= 256) return launch_t<E, MODE, 32, 1, 1, 1>(a, nmod, s);
        if (d <= 512) return launch_t<E, MODE, 32, 1, 2, 1>(a, nmod, s);
        if (d <= 768) return launch_t<E, MODE, 32, 3, 1, 1>(a, nmod, s);
        if (d <= 1024) return launch_t<E, MODE, 32, 1, 4, 1>(a, nmod, s);
        if (d <= 1536) return launch_t<E, MODE, 32, 3, 2, 1>(a, nmod, s);
        if (d <= 2048) return launch_t<E, MODE, 32, 2, 4, 1>(a, nmod, s);
        if (d <= 3072) return launch_t<E, MODE, 16, 6, 4, 1>(a, nmod, s);
        return launch_t<E, MODE, 16, 8, 4, 1>(a, nmod, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

int f32_rows(int d) { return d <= 2048 ? 32 : 16; }

hipError_t launch_local_loss_f32(int dtype, const FusedArgs& a, int nmod, hipStream_t s) {
    return dtype == 0 ? launch_w<bf16, LOCAL>(a, nmod, s) : launch_w<float, LOCAL>(a, nmod, s);
}
hipError_t launch_readout_grad_f32(int dtype, const FusedArgs& a, int nmod, hipStream_t s) {
    return dtype == 0 ? launch_w<bf16, RGRAD>(a, nmod, s) : launch_w<float, RGRAD>(a, nmod, s);
}
hipError_t launch_exit_eval_f32(int dtype, const FusedArgs& a, int nmod, hipStream_t s) {
    return dtype == 0 ? launch_t<bf16, EVAL, 32, 1, 1, 1>(a, nmod, s) : launch_t<float, EVAL, 32, 1, 1, 1>(a, nmod, s);
}
hipError_t launch_bias_grad_f32(int dtype, const FusedArgs& a, int nmod, hipStream_t s) {
    return dtype == 0 ? launch_t<bf16, BGRAD, 32, 1, 1, 1>(a, nmod, s)
                      : launch_t<float, BGRAD, 32, 1, 1, 1>(a, nmod, s);
}

}  // namespace solo
