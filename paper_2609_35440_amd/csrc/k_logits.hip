// Forward-only passes over many rows as a tiled product with a fused end
// (bf16 operands, fp32 accumulate): exit evaluation and the bias gradient.
// Neither needs the d-wide accumulator that fixes the row tile of the fused
// passes (k_mfma.hip), so the logits come from a plain C = Y X^T with 256 x 256
// tiles, whose operands pass through LDS once per 256 rows instead of once per
// 64, and no partial logits are exchanged between waves.
//
//   exit evaluation: Y = the readout rows v, X = the rows of bf16(g * h) (a copy);
//     a lane keeps, per row of X it owns, the online (max, sum-exp), the
//     target's logit and the top-1 over the tiles of its workgroup.
//   bias gradient: Y = the rows of bf16(g * h), X = the readout rows v;
//     db_v = sum_t (p_tv - [v = y_t]) / T from the stored log-sum-exp.
//
// A workgroup of 8 waves owns 256 rows of X and walks tiles of 256 rows of Y;
// wave (wm, wn) computes the 128 x 64 block of rows 128 wm of Y and 64 wn of X
// on 32x32x16 products (128 accumulator registers).  Steps of 64 k go
// buffer -> LDS directly into two stages of 64 KiB.  A stage's operands are
// read one 16-deep k-step ahead of their products; the barrier that hands over
// the next stage sits between the last step's products, so that the matrix
// cores have work while the next operands arrive, also across tiles and
// while a tile's end runs.  LDS rows are 128 bytes, 16-byte granule g of row r at
// g ^ (r & 7): 8 lanes of a read (8 rows, one granule) cover all banks.
//
// Workgroup order: the grid goes round-robin over the 8 XCDs; each takes an
// eighth of the (row tile, split) pairs in that order, so its 32 running
// workgroups are a few row tiles with all their splits and share both
// operands' streams in its L2.
//
// Measured (4 x 16384 rows, d = 2048, V = 32000): exit evaluation 7.1 ms, 1.2
// PFLOP/s in the product, against 8.7 ms of the fused pass; at d = 256 (4 x 8192) 0.65
// against 1.79.  On two planes (4 x 8192 x 32000, d = 640): 2.3 ms, 115 on the vector ALU.
#include "mfma_common.h"

namespace solo {

namespace {

using namespace mfma;

constexpr int NW = 8;
constexpr int NTHR = NW * 64;
constexpr int BT = 256;            // rows of a tile of either operand
constexpr int BK = 64;             // k per stage
constexpr int STAGE = BT * BK * 2; // bytes of one operand's stage
enum Mode { BGRAD = 2, EVAL = 3 };

// buffer_load_lds16 (mfma_common.h) with a scalar offset added to the address
__device__ __forceinline__ void buffer_load_lds16s(i32x4 rsrc, unsigned lds_base, int voffset, int soffset) {
    unsigned saved;
    asm volatile(
        "s_mov_b32 %0, m0\n\t"
        "s_mov_b32 m0, %1\n\t"
        "s_nop 0\n\t"
        "buffer_load_dwordx4 %2, %3, %4 offen lds\n\t"
        "s_nop 0\n\t"
        "s_mov_b32 m0, %0"
        : "=&s"(saved)
        : "s"(lds_base), "v"(voffset), "s"(rsrc), "s"(soffset)
        : "memory");
}

__device__ __forceinline__ float max3(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }

// XA: logits exact to fp32, for the bf16 widths whose calls are defined in fp32:
// one operand is the copy of g * h (16 significant bits) as two bf16 planes side by side,
// rows of 2 dp elements (dp = d rounded up to 64, zeros past d; the lower plane first,
// so that only the upper one's sums round at the logit's size), and the readout
// is read once per plane; its columns past d read as zeros.
// NI: 32-row blocks of Y per wave.  4, or 2 for XA past d = 2560: tiles of 128 rows of Y, whose
// accumulators leave room for a second set, so that the k-sum is cut into pieces of 512.
template <int MODE, bool EXT, bool XA, int NI>
__global__ __launch_bounds__(NTHR, 1) void k_logits(LogitsArgs a) {
    constexpr int BY = 64 * NI;       // rows of a tile of Y
    constexpr int WY = 32 * NI;       // rows of Y per wave
    constexpr bool CUT = NI < 4;      // the k-sum in pieces
    constexpr int STA = BY * BK * 2;  // bytes of a stage of Y
    __shared__ __attribute__((aligned(16))) char sA0[STA];
    __shared__ __attribute__((aligned(16))) char sA1[STA];
    __shared__ __attribute__((aligned(16))) char sB0[STAGE];
    __shared__ __attribute__((aligned(16))) char sB1[STAGE];
    // side data of a tile of Y, two tiles in turn: its biases (exit evaluation) or token records
    __shared__ __attribute__((aligned(16))) float side[2][MODE == BGRAD ? 4 * BT : (EXT ? BT : 4)];

    const int S = a.nsplit;
    const int pair = (int)((blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3));
    const int xt = pair / S, sp = pair % S;
    if (xt >= (a.nX + BT - 1) / BT) return;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = w >> 2, wn = w & 3;
    const int l32 = lane & 31, hi = lane >> 5;
    const int d = a.d;
    const int mod = blockIdx.y;
    const bf16* __restrict__ X = a.X + mod * a.x_stride + (mod == a.x_last ? a.x_last_off : 0);
    const bf16* __restrict__ Y = a.Y + mod * a.y_stride;
    const int x0 = xt * BT;
    const int nt = (a.nY + BY - 1) / BY;
    const int t_lo = (int)((long long)nt * sp / S), t_hi = (int)((long long)nt * (sp + 1) / S);
    // stages per tile: an even number (d % 256 == 0, or two planes)
    const int nkd = (d + BK - 1) / BK;
    const int nk = XA ? 2 * nkd : nkd;
    // row pitches: the copy of g * h is X in exit evaluation, Y in the bias gradient
    const int cp = 2 * nkd * BK;
    const int dX = XA && MODE == EVAL ? cp : d, dY = XA && MODE == BGRAD ? cp : d;

    LDS_AS char* const pA0 = (LDS_AS char*)(LDS_AS void*)sA0;
    LDS_AS char* const pA1 = (LDS_AS char*)(LDS_AS void*)sA1;
    LDS_AS char* const pB0 = (LDS_AS char*)(LDS_AS void*)sB0;
    LDS_AS char* const pB1 = (LDS_AS char*)(LDS_AS void*)sB1;

    // ---- stream: instruction i of wave w fills rows 32 w + 8 i .. + 7 of a stage of X, and
    // rows 8 NI w + 8 i .. + 7 of one of Y
    const int gr = (lane & 7) ^ (lane >> 3);  // the lane's granule of a row
    int voA[NI], voB[4];
#pragma unroll
    for (int i = 0; i < NI; ++i) voA[i] = (8 * NI * w + 8 * i + (lane >> 3)) * dY * 2 + 16 * gr;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        voB[i] = XA ? (32 * w + 8 * i + (lane >> 3)) * dX * 2 + 16 * gr : voA[i < NI ? i : 0];
    auto rows_rsrc = [&](const bf16* __restrict__ P, int n, int r0, int pitch, int most) __attribute__((always_inline)) {
        const int rows = n - r0 < most ? n - r0 : most;
        return make_rsrc(P + (long long)r0 * pitch, (unsigned)rows * (unsigned)pitch * 2u);
    };
    const i32x4 brs = rows_rsrc(X, a.nX, x0, dX, BT);
    const unsigned uA[2] = {lds_addr(pA0) + w * (STA / NW), lds_addr(pA1) + w * (STA / NW)};
    const unsigned uB[2] = {lds_addr(pB0) + w * 4096, lds_addr(pB1) + w * 4096};
    int it = t_lo, ik = 0;  // the next stage to stream
    i32x4 ars = rows_rsrc(Y, a.nY, t_lo * BY, dY, BY);
    auto issue = [&](int buf) __attribute__((always_inline)) {
        if (it >= t_hi) return;
        // XA: the readout's k of this stage, and whether the lane's granule of it is past d
        const int kr = XA && ik >= nkd ? ik - nkd : ik;
        const bool past = XA && kr * BK + 8 * gr >= d;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (i < NI) buffer_load_lds16s(ars, uA[buf] + i * 1024, MODE == EVAL && past ? 0x40000000 : voA[i < NI ? i : 0],
                               (MODE == EVAL ? kr : ik) * (BK * 2));
            buffer_load_lds16s(brs, uB[buf] + i * 1024, MODE == BGRAD && past ? 0x40000000 : voB[i],
                               (MODE == EVAL ? ik : kr) * (BK * 2));
        }
        if (ik == 1) {
            // the tile's side data, long before its end: every wave has left the
            // tile before the last by now
            const unsigned ds = lds_addr((LDS_AS char*)(LDS_AS void*)side[it & 1]);
            const int y0 = it * BY;
            const int rows = a.nY - y0 < BY ? a.nY - y0 : BY;
            if (MODE == BGRAD && w < NI)
                buffer_load_lds16(make_rsrc(a.rowrec + 4 * (mod * (long long)a.nY + y0), (unsigned)rows * 16u),
                                  ds + w * 1024, (64 * w + lane) * 16);
            if (MODE == EVAL && EXT && w < NI)
                buffer_load_lds4(make_rsrc(a.bias + y0, (unsigned)rows * 4u), ds + w * 256, (64 * w + lane) * 4);
        }
        if (++ik == nk) {
            ik = 0;
            ++it;
            if (it < t_hi) ars = rows_rsrc(Y, a.nY, it * BY, dY, BY);
        }
    };

    // ---- operands of one k-step: lane reads row l32 of each 32-row block, granule 2 s + hi
    int go[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) go[s] = l32 * 128 + 16 * ((2 * s + hi) ^ (lane & 7));
    bf16x8 fa[2][NI], fb[2][2];
    auto read = [&](LDS_AS const char* A, LDS_AS const char* B, int s, int q) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < 2; ++b) fb[q][b] = *(LDS_AS const bf16x8*)(B + (64 * wn + 32 * b) * 128 + go[s]);
#pragma unroll
        for (int b = 0; b < NI; ++b) fa[q][b] = *(LDS_AS const bf16x8*)(A + (WY * wm + 32 * b) * 128 + go[s]);
    };
    f32x16 acc[NI][2];
    f32x16 tot[CUT ? NI : 1][2];  // CUT: the sum of the pieces before this one
    auto zero = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    };
    auto add_piece = [&](bool first) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < (CUT ? NI : 1); ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) tot[i][j][e] = first ? acc[i][j][e] : tot[i][j][e] + acc[i][j][e];
    };
    // (the products of half of the blocks)
    auto mul = [&](int q, int half) __attribute__((always_inline)) {
#pragma unroll
        for (int i = half * (NI / 2); i < (half + 1) * (NI / 2); ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = mfma32(fa[q][i], fb[q][j], acc[i][j]);
    };
    // one stage in buffer `buf` (its first k-step is in the operand registers)
    auto stage = [&](int buf) __attribute__((always_inline)) {
        LDS_AS const char* A = buf ? pA1 : pA0;
        LDS_AS const char* B = buf ? pB1 : pB0;
        LDS_AS const char* An = buf ? pA0 : pA1;
        LDS_AS const char* Bn = buf ? pB0 : pB1;
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            read(A, B, s + 1, (s + 1) & 1);
            mul(s & 1, 0);
            mul(s & 1, 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        mul(1, 0);
        __builtin_amdgcn_sched_barrier(0);
        wait_vm();      // this wave's part of the next stage
        lds_barrier();  // everyone's; and everyone has read this one
        issue(buf);
        read(An, Bn, 0, 0);
        mul(1, 1);
        __builtin_amdgcn_sched_barrier(0);
    };

    // ---- per-lane state of X rows x0 + 64 wn + 32 j + l32, j = 0, 1
    float r2[2], m_run[2], sum[2], zy[2], best[2], bx2[2];
    double dsum[2] = {0.0, 0.0};  // BGRAD
    int tgt[2], best_v[2];
    long long grow[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int x = x0 + 64 * wn + 32 * j + l32;
        const bool ok = x < a.nX;
        r2[j] = bx2[j] = sum[j] = zy[j] = m_run[j] = 0.f;
        best[j] = -INFINITY;
        best_v[j] = -1;
        tgt[j] = ok ? x : -2;
        grow[j] = a.row0 + x;
        if (MODE == EVAL && ok) {
            r2[j] = a.rstd[grow[j]] * (a.tau ? a.tau[grow[j] / a.T] : 1.f) * kLog2e;
            tgt[j] = a.targets[grow[j]];
        }
        if (MODE == BGRAD && a.bias && ok) {
            const float b = a.bias[mod * (long long)a.nX + x];
            bx2[j] = XA ? bias2(b) : b * kLog2e;
        }
    }

    issue(0);
    issue(1);
    zero();
    wait_vm();
    __syncthreads();
    read(pA0, pB0, 0, 0);
    for (int t = t_lo; t < t_hi; ++t) {
#pragma nounroll
        for (int kt = 0; kt < nk; kt += 2) {
            stage(0);
            stage(1);
            if (CUT && kt % 8 == 6 && kt + 2 < nk) {
                add_piece(kt < 8);
                zero();
            }
        }
        if (CUT && nk > 8) {
#pragma unroll
            for (int i = 0; i < (CUT ? NI : 1); ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[i][j][e] += tot[i][j][e];
        }
        // ---- the tile's end.  acc[i][j][e]: row y = yb + 32 i + 8 (e / 4) + 4 hi + e % 4 of Y,
        // yb = BY t + WY wm; column: the lane's X row j
        const int yb = t * BY + WY * wm;
        const bool ragged = t * BY + BY > a.nY;  // wave-uniform
        LDS_AS const float* sd = (LDS_AS const float*)(LDS_AS void*)side[t & 1];
        if (MODE == EVAL) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                float zmax = -INFINITY;
#pragma unroll
                for (int i = 0; i < NI; ++i)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const int yl = 32 * i + 8 * g + 4 * hi;
                        f32x4 bv = {0.f, 0.f, 0.f, 0.f};
                        if (EXT) bv = *(LDS_AS const f32x4*)(sd + WY * wm + yl);
                        float z[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            z[e] = EXT ? __builtin_fmaf(acc[i][j][4 * g + e], r2[j], XA ? bias2(bv[e]) : bv[e] * kLog2e)
                                       : acc[i][j][4 * g + e] * r2[j];
                            acc[i][j][4 * g + e] = z[e];
                        }
                        zmax = max3(max3(zmax, z[0], z[1]), z[2], z[3]);
                    }
                if (ragged) {
                    // rows past the end: z = -inf
                    zmax = -INFINITY;
#pragma unroll
                    for (int i = 0; i < NI; ++i) {
                        const int left = a.nY - (yb + 32 * i + 4 * hi);
#pragma unroll
                        for (int e = 0; e < 16; ++e) {
                            if (8 * (e >> 2) + (e & 3) >= left) acc[i][j][e] = -INFINITY;
                            zmax = fmaxf(zmax, acc[i][j][e]);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                // top-1: only a lane whose maximum grew looks for its (lowest) column
                if (__any(zmax > best[j])) {
                    int at = 0;
#pragma unroll
                    for (int i = NI - 1; i >= 0; --i) {
#pragma unroll
                        for (int e = 15; e >= 0; --e)
                            at = acc[i][j][e] == zmax ? 32 * i + 8 * (e >> 2) + (e & 3) : at;
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    at += yb + 4 * hi;
                    best_v[j] = zmax > best[j] ? at : best_v[j];
                    best[j] = fmaxf(best[j], zmax);
                }
                // the running maximum is the lane's own; it is re-based past the
                // threshold, and as long as it has no term yet (selects under a branch that the
                // wave takes as one: of a lane's branch with both conditions, the compiler kept
                // only the first one's maximum past the loop in the two-block form)
                const bool none = sum[j] == 0.f;
                const bool up = (zmax > m_run[j] + kLazyThresh2) | (none & (zmax > -INFINITY));
                if (__any(up)) {
                    const float scaled = none ? 0.f : sum[j] * __builtin_amdgcn_exp2f(m_run[j] - zmax);
                    sum[j] = up ? scaled : sum[j];
                    m_run[j] = up ? zmax : m_run[j];
                }
                float s0 = 0.f, s1 = 0.f;
                const int rel = tgt[j] - yb - 4 * hi;
                if (__any(rel >= 0 && rel < WY)) {
                    // some row's target is in the tile: its term stays out of the sum (finish_row)
#pragma unroll
                    for (int i = 0; i < NI; ++i) {
#pragma unroll
                        for (int e = 0; e < 16; ++e) {
                            const bool is_y = rel == 32 * i + 8 * (e >> 2) + (e & 3);
                            if (is_y) zy[j] = acc[i][j][e];
                            const float p = __builtin_amdgcn_exp2f(acc[i][j][e] - m_run[j]);
                            s0 += is_y ? 0.f : p;
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < NI; ++i)
#pragma unroll
                        for (int e = 0; e < 16; e += 2) {
                            s0 += __builtin_amdgcn_exp2f(acc[i][j][e] - m_run[j]);
                            s1 += __builtin_amdgcn_exp2f(acc[i][j][e + 1] - m_run[j]);
                        }
                }
                sum[j] += s0 + s1;
            }
        } else {
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                // a lane's 16 tokens of a block in fp32, pairs first, then in 64 bits: one
                // chain over its T / 4 tokens lost up to 2.7 times the fp32 kernels' bits
                float blk[2] = {0.f, 0.f}, dl[2][4];
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    // record {lse log2 e, r tau log2 e, target, p_y - 1}; the target's entry
                    // of delta is the exact p_y - 1 of the local-loss pass
                    const int yl = 32 * i + 8 * (e >> 2) + 4 * hi + (e & 3);
                    const f32x4 r4 = *(LDS_AS const f32x4*)(sd + 4 * (WY * wm + yl));
                    const bool in = !ragged || yl < a.nY - yb;
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(acc[i][j][e], r4[1], bx2[j] - r4[0]));
                        dl[j][e & 3] = in ? (__float_as_int(r4[2]) == tgt[j] ? r4[3] : p) : 0.f;
                        if ((e & 3) == 3) blk[j] += (dl[j][0] + dl[j][1]) + (dl[j][2] + dl[j][3]);
                    }
                }
#pragma unroll
                for (int j = 0; j < 2; ++j) dsum[j] += (double)blk[j];
            }
        }
        zero();
    }

    // ---- the lane halves, then the two waves of a column of blocks
    __syncthreads();  // the stages are free
    float* red = (float*)sA0;  // [wm][state][256 rows of X]
    static_assert(2 * 5 * BT * 4 <= STA, "the rows' states fit a stage");
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int xl = 64 * wn + 32 * j + l32;
        if (MODE == BGRAD) {
            dsum[j] += __shfl_xor(dsum[j], 32, 64);
            if (hi == 0) red[wm * BT + xl] = (float)dsum[j];
            continue;
        }
        // a lane that saw no finite logit has no maximum
        const float mm = best[j] > -INFINITY ? m_run[j] : -INFINITY;
        const float om = __shfl_xor(mm, 32, 64), os = __shfl_xor(sum[j], 32, 64);
        const float ob = __shfl_xor(best[j], 32, 64);
        const int ov = __shfl_xor(best_v[j], 32, 64);
        zy[j] += __shfl_xor(zy[j], 32, 64);
        const float m = fmaxf(mm, om);
        const float s = sum[j] * (m == mm ? 1.f : __builtin_amdgcn_exp2f(mm - m)) +
                        os * (m == om ? 1.f : __builtin_amdgcn_exp2f(om - m));
        if (ob > best[j] || (ob == best[j] && (unsigned)ov < (unsigned)best_v[j])) {
            best[j] = ob;
            best_v[j] = ov;
        }
        if (hi == 0) {
            red[(wm * 5 + 0) * BT + xl] = m;
            red[(wm * 5 + 1) * BT + xl] = s;
            red[(wm * 5 + 2) * BT + xl] = zy[j];
            red[(wm * 5 + 3) * BT + xl] = best[j];
            red[(wm * 5 + 4) * BT + xl] = __int_as_float(best_v[j]);
        }
    }
    __syncthreads();
    if (tid >= BT) return;
    const int x = x0 + tid;
    if (x >= a.nX) return;
    if (MODE == BGRAD) {
        const float db = red[tid] + red[BT + tid];
        // the last split's part goes to the output itself
        float* const o = sp == S - 1 ? a.out : a.parts + (long long)sp * gridDim.y * a.nX;
        o[mod * (long long)a.nX + x] = S == 1 ? db * a.inv_T : db;
        return;
    }
    const float m0 = red[tid], m1 = red[5 * BT + tid];
    float sa = red[BT + tid], sb = red[6 * BT + tid];
    const float m = fmaxf(m0, m1);
    if (m0 != m) sa *= __builtin_amdgcn_exp2f(m0 - m);
    if (m1 != m) sb *= __builtin_amdgcn_exp2f(m1 - m);
    const float z = red[2 * BT + tid] + red[7 * BT + tid];
    float b0 = red[3 * BT + tid];
    int v0 = __float_as_int(red[4 * BT + tid]);
    const float b1 = red[8 * BT + tid];
    const int v1 = __float_as_int(red[9 * BT + tid]);
    if (b1 > b0 || (b1 == b0 && (unsigned)v1 < (unsigned)v0)) {
        b0 = b1;
        v0 = v1;
    }
    const long long row = a.row0 + x;
    if (S == 1) {
        const int ty = a.targets[row];
        a.rowloss[row] = finish_row<XA>(m, sa + sb, z, ty >= 0 && ty < a.nY).loss;
        if (a.top1) a.top1[row] = v0;
    } else {
        float* p = a.parts + 8 * (sp * a.part_rows + row);
        *(f32x4*)p = (f32x4){m, sa + sb, z, b0};
        *(f32x4*)(p + 4) = (f32x4){__int_as_float(v0), 0.f, 0.f, 0.f};
    }
}

// db[m][v] = sum of the splits' parts / T, the last of them in place
__global__ void k_db_sum(const float* __restrict__ parts, float* __restrict__ out, long long n, int nsplit,
                         float inv_T) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double s = out[i];
    for (int k = 0; k < nsplit - 1; ++k) s += (double)parts[k * n + i];
    out[i] = (float)s * inv_T;
}

template <int MODE, bool EXT, bool XA, int NI = 4>
hipError_t launch_t(const LogitsArgs& a, int nmod, hipStream_t s) {
    const int tiles = (a.nX + BT - 1) / BT;
    hipLaunchKernelGGL((k_logits<MODE, EXT, XA, NI>), dim3((unsigned)(((long long)tiles * a.nsplit + 7) / 8 * 8), (unsigned)nmod),
                       dim3(NTHR), 0, s, a);
    return hipGetLastError();
}

}  // namespace

// The planes' rows of Y per tile in exit evaluation.  The upper plane's chain of d / 16 sums
// rounds at the logit's size: the row losses' error (rms of 2 x 1000 rows) is 3.3e-7 at d = 2040,
// where it was 4.0e-7 on the vector ALU (4.2 at 3072), and grows with d to the same size near
// d = 3000.  Past 2560 the k-sum is therefore cut (2.8e-7 at 3072, 3.1 at 4096), on half the
// tile: 4 x 8192 x 32000 rows take 12.8 ms at 3072 and 20.1 at 4096; uncut 10.2 and 14.2.
int logits_eval_tile(bool exact, int d) { return exact && d > 2560 ? 128 : 256; }

hipError_t launch_logits_eval(const LogitsArgs& a, hipStream_t s) {
    if (logits_eval_tile(a.exact, a.d) == 128)
        return a.bias ? launch_t<EVAL, true, true, 2>(a, 1, s) : launch_t<EVAL, false, true, 2>(a, 1, s);
    if (a.exact) return a.bias ? launch_t<EVAL, true, true>(a, 1, s) : launch_t<EVAL, false, true>(a, 1, s);
    return a.bias ? launch_t<EVAL, true, false>(a, 1, s) : launch_t<EVAL, false, false>(a, 1, s);
}

hipError_t launch_logits_bgrad(const LogitsArgs& a, int nmod, hipStream_t s) {
    hipError_t e = a.exact ? launch_t<BGRAD, false, true>(a, nmod, s) : launch_t<BGRAD, false, false>(a, nmod, s);
    if (e != hipSuccess || a.nsplit == 1) return e;
    const long long n = (long long)nmod * a.nX;
    hipLaunchKernelGGL(k_db_sum, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a.parts, a.out, n, a.nsplit,
                       a.inv_T);
    return hipGetLastError();
}

}  // namespace solo
