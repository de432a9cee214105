// The exact form of the passes with a second product (see XA in k_mfma.hip: bf16
// storage, products exact to fp32 from bf16 planes) for hidden states wider
// than its 32-row tile holds, 1536 < d <= 4096.
//
// 16 stationary rows per workgroup of 8 waves; wave w owns the DS columns
// [w DS, (w+1) DS) of the accumulator (DS / 4 registers per lane) and of the
// stationary operand: two planes of g * X in registers up to DS = 384, at 512 the raw
// X, whose planes are formed from it and the gain (in LDS) at every use.
// Chunks of 16 streamed rows go buffer -> LDS directly into the wave's own
// slice, single-buffered (16 x 4096 is 128 KiB) but in two column halves: a half
// is refilled as soon as its second products' operands have been read, so it
// lands behind the other half's products and the next chunk's logits start on it.
//   logits: 16x16x32 products, rows read from the slice; partials meet in LDS
//   softmax: as in the wide tiling (k_mfma_wide.hip), the probabilities as three planes
//   second product: 16x16x16, three planes per transposed read
//
// A half-slice row has GH 16-byte granules, granule g of row r at g ^ key(r):
// with GH a multiple of 16, key = 2 (r & 7) ^ (r >> 2 & 1), which spreads 8 rows of a
// 16-byte read over 128 bytes and 8 rows of the transposing reads' 32 bytes over
// 256; at GH = 24 (rows of 384 bytes, alternately 0 and 128 mod 256) key = r & 7.
// Bound by the LDS traffic of a chunk (one write and two reads of it) and the
// half-rate 16x16x16 products; at DS = 512 also by the vector ALU that forms the
// planes (2.6 us per chunk at d = 3072, 4.8 at 4096).
//
// Measured (training, 2 x 1024 x 32000): d = 4096 7.4 ms against 19.4 on the fp32
// instructions, d = 3072 4.0.
#include "mfma_common.h"

namespace solo {

namespace {

using namespace mfma;

constexpr int NW = 8;
constexpr int NTHR = NW * 64;
constexpr int YC = 16;
constexpr int XR = 16;
constexpr int PP = 16;
enum Mode { LOCAL = 0, RGRAD = 1 };

__device__ __forceinline__ f32x4 mfma16k16(bf16x4 a, bf16x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// x * g per element (16 significant bits) as two bf16 planes: the upper 8 bits, truncated, and the rest
__device__ __forceinline__ void planes(i32x4 x, i32x4 g, bf16x8& hi, bf16x8& lo) {
    i32x4 h, l;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float p0 = __int_as_float(x[e] << 16) * __int_as_float(g[e] << 16);
        const float p1 = __int_as_float(x[e] & (int)0xffff0000) * __int_as_float(g[e] & (int)0xffff0000);
        const int u0 = __float_as_int(p0), u1 = __float_as_int(p1);
        const float r0 = p0 - __int_as_float(u0 & (int)0xffff0000);
        const float r1 = p1 - __int_as_float(u1 & (int)0xffff0000);
        h[e] = (int)__builtin_amdgcn_perm((unsigned)u1, (unsigned)u0, 0x07060302u);
        l[e] = (int)__builtin_amdgcn_perm((unsigned)__float_as_int(r1), (unsigned)__float_as_int(r0), 0x07060302u);
    }
    hi = __builtin_bit_cast(bf16x8, h);
    lo = __builtin_bit_cast(bf16x8, l);
}

template <int GH>
__device__ __forceinline__ int key(int r) {
    return GH % 16 == 0 ? (((r & 7) << 1) ^ ((r >> 2) & 1)) : (r & 7);
}

// CS (LOCAL): see kChunkSums.
template <int MODE, int DS, bool EXT, bool SPL, bool CS = false>
__global__ __launch_bounds__(NTHR, 1) void k_exact_wide(FusedArgs a) {
    constexpr bool LL = MODE == LOCAL;
    constexpr int NK = DS / 32, NB = DS / 16;
    constexpr int GH = DS / 16;            // granules per row of a half-slice
    constexpr int HALF = 16 * GH * 16;     // bytes of a half-slice
    constexpr int NI = HALF / 1024;        // direct-to-LDS instructions per half
    constexpr bool RAW = DS > 384;         // planes formed at every use
    constexpr bool BZ = LL && EXT;
    static_assert(GH % 8 == 0 && NK % 2 == 0 && NB % 2 == 0, "half-slices of whole k-steps and blocks");
    __shared__ __attribute__((aligned(16))) char ybuf[NW * 2 * HALF];
    __shared__ __attribute__((aligned(16))) float part[NW * XR * PP];
    __shared__ __attribute__((aligned(16))) bf16 gbuf[3 * XR * YC];
    __shared__ __attribute__((aligned(16))) bf16 gains[RAW ? NW * DS : 8];
    __shared__ float abuf[XR];
    __shared__ float sbuf[XR];
    __shared__ float pybuf[XR];
    __shared__ float cbuf[NW * XR];
    __shared__ __attribute__((aligned(16))) float recA[YC * 4];
    __shared__ __attribute__((aligned(16))) float recB[YC * 4];

    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int d = a.d;
    const int js = w * DS;
    // (splits next to each other: the grid goes round-robin over the XCDs, whose L2s then
    // stream a part of the vocabulary each)
    const int tile = SPL ? (int)blockIdx.x / a.nsplit : (int)blockIdx.x;
    const int sp = SPL ? (int)blockIdx.x % a.nsplit : 0;
    const int x0 = tile * XR;
    const int k = a.m0 + (int)blockIdx.y;
    const long long modoff = (long long)k * a.T;
    const float tau_k = a.tau ? a.tau[k] : 1.f;
    const bf16* __restrict__ hk = (const bf16*)a.h + modoff * d;
    const bf16* __restrict__ Rk = k == a.K - 1 ? (const bf16*)a.Wt : (const bf16*)a.Wh + (long long)k * a.wh_stride;
    const bf16* __restrict__ gk = (const bf16*)a.gain + (long long)k * a.g_stride;
    const bf16* __restrict__ X = LL ? hk : Rk;
    const bf16* __restrict__ Y = LL ? Rk : hk;
    const int nX = LL ? a.T : a.V;
    const int nY = LL ? a.V : a.T;
    const int nchunks = (nY + YC - 1) / YC;
    const int ck_lo = SPL ? (int)((long long)nchunks * sp / a.nsplit) : 0;
    const int ck_hi = SPL ? (int)((long long)nchunks * (sp + 1) / a.nsplit) : nchunks;

    LDS_AS char* const slice = (LDS_AS char*)(LDS_AS void*)ybuf + w * 2 * HALF;
    const unsigned slice_u = lds_addr(slice);
    auto chunk_rsrc = [&](int c) __attribute__((always_inline)) {
        const int rows = nY - c * YC < YC ? nY - c * YC : YC;
        return make_rsrc(Y + (long long)c * YC * d, (unsigned)rows * (unsigned)d * 2u);
    };
    // half hf of the wave's columns of a chunk: slot s of row r holds granule s ^ key(r)
    auto issue = [&](i32x4 rs, int hf) __attribute__((always_inline)) {
        const int l = lane_now();
#pragma unroll
        for (int q = 0; q < NI; ++q) {
            const int p = 64 * q + l, r = p / GH;
            const int col = js + hf * (DS / 2) + 8 * ((p - r * GH) ^ key<GH>(r));
            buffer_load_lds16(rs, slice_u + hf * HALF + q * 1024, col < d ? (r * d + col) * 2 : 0x40000000);
        }
    };
    // row-wise operand of k-step kk; transposed operand of 16-column block b
    auto row_off = [&](int kk) __attribute__((always_inline)) {
        const int r = lane & 15, hf = kk / (NK / 2);
        return hf * HALF + 16 * (r * GH + ((4 * (kk - hf * (NK / 2)) + (lane >> 4)) ^ key<GH>(r)));
    };
    auto tr_off = [&](int b) __attribute__((always_inline)) {
        const int ti = lane & 15, r = 4 * (lane >> 4) + (ti >> 2), hf = b / (NB / 2);
        return hf * HALF + 16 * (r * GH + ((2 * (b - hf * (NB / 2)) + ((ti & 3) >> 1)) ^ key<GH>(r))) + 8 * (ti & 1);
    };

    if (ck_lo < ck_hi) {
        const i32x4 rs = chunk_rsrc(ck_lo);
        issue(rs, 0);
        issue(rs, 1);
    }
    const unsigned recA_u = lds_addr((LDS_AS char*)(LDS_AS void*)recA);
    const unsigned recB_u = lds_addr((LDS_AS char*)(LDS_AS void*)recB);
    auto issue_side = [&](int y0, unsigned dst) __attribute__((always_inline)) {
        const int rows = nY - y0 < YC ? nY - y0 : YC;
        const unsigned n = rows > 0 ? (unsigned)rows : 0u;
        if (!LL && w == 0 && lane < YC) buffer_load_lds16(make_rsrc(a.rowrec + 4 * (modoff + y0), n * 16u), dst, lane * 16);
        if (BZ && w == 0 && lane < YC)
            buffer_load_lds4(make_rsrc(a.bias + (long long)k * a.V + y0, n * 4u), dst, lane * 4);
    };
    issue_side(ck_lo * YC, recA_u);

    // this lane's elementwise row (computed by lanes l and l + 32, written by l < 32) and column
    const int xo = 2 * w + ((lane >> 4) & 1);
    const bool wr = lane < 32;
    const int yy = lane & 15;
    float own_r2 = 0.f, bx2 = 0.f;
    int own_tgt = -1;
    if (LL && x0 + xo < nX) {
        own_r2 = a.rstd[modoff + x0 + xo] * tau_k * kLog2e;
        own_tgt = a.targets[modoff + x0 + xo];
    }
    if (!LL && a.bias && x0 + xo < nX) bx2 = bias2(a.bias[(long long)k * a.V + x0 + xo]);

    if (RAW) {
        for (int j = 8 * threadIdx.x; j < NW * DS; j += 8 * NTHR) {
            i32x4 v = {0, 0, 0, 0};
            if (j < d) v = *(const i32x4*)(gk + j);
            *(i32x4*)(gains + (RAW ? j : 0)) = v;
        }
    }
    // stationary operand: lane holds row lane % 16, columns js + 32 kk + 8 (lane / 16) .. + 7
    bf16x8 xhi[RAW ? 1 : NK], xlo[RAW ? 1 : NK];
    i32x4 xraw[RAW ? NK : 1];
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
        const int j0 = js + 32 * kk + 8 * (lane >> 4);
        const int xrow = x0 + (lane & 15);
        i32x4 xv = {0, 0, 0, 0}, gv = {0, 0, 0, 0};
        if (xrow < nX && j0 < d) {
            xv = *(const i32x4*)(X + (long long)xrow * d + j0);
            if (!RAW) gv = *(const i32x4*)(gk + j0);
        }
        if constexpr (RAW) {
            xraw[kk] = xv;
        } else {
            planes(xv, gv, xhi[kk], xlo[kk]);
        }
    }

    f32x4 acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = (f32x4){0.f, 0.f, 0.f, 0.f};
    float m_run = -INFINITY, s_part = 0.f, zy_part = 0.f;
    double db_part = 0.0;  // (a lane's share of a sum over all tokens)

    auto step = [&](LDS_AS float* side, unsigned side_nxt, int c) __attribute__((always_inline)) {
        const int y0 = c * YC;
        const bool more = c + 1 < ck_hi;
        f32x4 S = {0.f, 0.f, 0.f, 0.f};
        auto products = [&](int k0, int k1) __attribute__((always_inline)) {
#pragma unroll
            for (int kk = k0; kk < k1; ++kk) {
                const bf16x8 ay = *(LDS_AS bf16x8*)(slice + row_off(kk));
                if constexpr (RAW) {
                    // (opaque, or the compiler unpacks all of X once, into twice the registers)
                    asm volatile("" : "+v"(xraw[kk]));
                    bf16x8 ph, pl;
                    planes(xraw[kk], *(const i32x4*)(gains + js + 32 * kk + 8 * (lane >> 4)), ph, pl);
                    S = mfma16(ay, ph, S);
                    S = mfma16(ay, pl, S);
                    // two k-steps at a time: more operands than that do not fit the registers
                    if (kk & 1) __builtin_amdgcn_sched_barrier(0);
                } else {
                    S = mfma16(ay, xhi[kk], S);
                    S = mfma16(ay, xlo[kk], S);
                }
            }
        };
        // the first half landed before the second's NI loads; then all (vmcnt in the low bits)
        __builtin_amdgcn_s_waitcnt(0x0F70 | NI);
        asm volatile("" ::: "memory");
        products(0, NK / 2);
        wait_vm();
        products(NK / 2, NK);
        if (more) issue_side(y0 + YC, side_nxt);
        {
            const int xl = lane & 15;
            *(f32x4*)(part + (w * XR + xl) * PP + 4 * ((lane >> 4) ^ ((xl >> 1) & 3))) = S;
        }
        lds_barrier();
        {
            float q[NW];
#pragma unroll
            for (int ww = 0; ww < NW; ++ww) q[ww] = part[(ww * XR + xo) * PP + (yy ^ (4 * ((xo >> 1) & 3)))];
            const float sxy = ((q[0] + q[1]) + (q[2] + q[3])) + ((q[4] + q[5]) + (q[6] + q[7]));
            const int yg = y0 + yy;
            float gval = 0.f;
            if (LL) {
                float ymask = yg < nY ? 0.f : -INFINITY;
                if (BZ) ymask += bias2(side[yy]);
                const float zc = __builtin_fmaf(sxy, own_r2, ymask);
                float alpha = 1.f;
                if (__builtin_expect(__any(zc > m_run + kLazyThresh2), 0)) {  // wave-uniform
                    const float cmax = row16_max(zc);
                    if (cmax > m_run + kLazyThresh2) {
                        alpha = __builtin_amdgcn_exp2f(m_run - cmax);
                        s_part *= alpha;
                        m_run = cmax;
                    }
                }
                const float p = zc == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(zc - m_run);
                // the target's term joins at the end of the row (finish_row)
                gval = yg == own_tgt ? 0.f : p;
                s_part += gval;
                if (yg == own_tgt) zy_part = zc;
                if (wr) abuf[xo] = alpha;
            } else {
                // record {lse log2 e, r tau log2 e, target, p_y - 1}; padded tokens are masked
                const f32x4 r4 = *(LDS_AS f32x4*)(side + 4 * yy);
                const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(sxy, r4[1], bx2 - r4[0]));
                const float dlt = yg < nY ? (__float_as_int(r4[2]) == x0 + xo ? r4[3] : p) : 0.f;
                gval = dlt * (r4[1] * (kLn2 * a.inv_T));  // times r tau / T
                db_part += dlt;
            }
            if (wr) {
                // three planes
                bf16* gp = gbuf + xo * YC + (yy ^ (8 * ((xo >> 3) & 1)));
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) {
                    const bf16 g1 = (bf16)gval;
                    gp[pl * XR * YC] = g1;
                    gval -= (float)g1;
                }
            }
        }
        lds_barrier();
        {
            bf16x4 gf[3];
#pragma unroll
            for (int pl = 0; pl < 3; ++pl)
                gf[pl] = *(bf16x4*)(gbuf + (pl * XR + (lane & 15)) * YC + 4 * ((lane >> 4) ^ (2 * ((lane >> 3) & 1))));
            if (LL) {
                const float al = abuf[lane & 15];
                if (__any(al != 1.f)) {
#pragma unroll
                    for (int b = 0; b < NB; ++b) acc[b] *= al;
                }
            }
            const i32x4 nrs = chunk_rsrc(more ? c + 1 : c);
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) {
                if constexpr (CS) {
                    // a few blocks at a time, smallest plane first; the additions are kept here (see k_mfma.hip)
                    constexpr int FLY = DS == 256 ? 8 : (DS == 384 ? 3 : 4);
                    static_assert(NB / 2 % FLY == 0, "whole groups");
#pragma unroll
                    for (int b = hf * (NB / 2); b < (hf + 1) * (NB / 2); b += FLY) {
                        bf16x4 t[FLY];
                        f32x4 c4[FLY];
#pragma unroll
                        for (int i = 0; i < FLY; ++i) {
                            t[i] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_AS bf16x4*)(slice + tr_off(b + i)));
                            c4[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
                        }
#pragma unroll
                        for (int pl = 2; pl >= 0; --pl)
#pragma unroll
                            for (int i = 0; i < FLY; ++i) c4[i] = mfma16k16(t[i], gf[pl], c4[i]);
#pragma unroll
                        for (int i = 0; i < FLY; ++i) {
                            acc[b + i] += c4[i];
                            asm volatile("" : "+v"(acc[b + i]));
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
#pragma unroll
                for (int b = hf * (NB / 2); !CS && b < (hf + 1) * (NB / 2); ++b) {
                    const bf16x4 t = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_AS bf16x4*)(slice + tr_off(b)));
#pragma unroll
                    for (int pl = 0; pl < 3; ++pl) acc[b] = mfma16k16(t, gf[pl], acc[b]);
                    if (RAW && b % 4 == 3) __builtin_amdgcn_sched_barrier(0);
                }
                // this wave has read the half: its next rows may overwrite it
                __builtin_amdgcn_sched_barrier(0);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                if (more) issue(nrs, hf);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    wait_vm();
    __syncthreads();  // the gains, and the first side data
    for (int c = ck_lo; c < ck_hi; c += 2) {
        step((LDS_AS float*)(LDS_AS void*)recA, recB_u, c);
        if (c + 1 < ck_hi) step((LDS_AS float*)(LDS_AS void*)recB, recA_u, c + 1);
    }

    // ---- epilogues.  acc[b]: x = lane % 16, j = js + 16 b + 4 (lane / 16) + i (16-column blocks
    // past the width hold sums of zeros and are skipped; a block the width cuts has whole groups of 8)
    const int ex = lane & 15;
    const int eg = lane >> 4;
    auto each = [&](auto f) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int j = js + 16 * b + 4 * eg;
            f(b, j, j < d);
            if (b % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
    };
    if (LL) {
        const float sx = row16_sum(s_part);
        const float zy = row16_sum(zy_part);
        if (yy == 0 && wr) {
            const int xr_ = x0 + xo;
            if (SPL) {
                if (xr_ < nX)
                    *(f32x4*)(a.split_stat + 4 * ((long long)sp * a.part_rows + modoff + xr_)) =
                        (f32x4){m_run, sx, zy, 0.f};
            } else {
                const RowEnd re = finish_row<true>(m_run, sx, zy, own_tgt >= 0 && own_tgt < nY);
                if (xr_ < nX) {
                    const long long t = modoff + xr_;
                    a.lse[t] = 1.f;  // (the bias-gradient pass of these widths scales by it)
                    a.rowloss[t] = re.loss;
                    if (a.rowrec) {
                        const f32x4 rec4 = {re.lse2, own_r2, __int_as_float(own_tgt), re.py1};
                        *(f32x4*)(a.rowrec + 4 * t) = rec4;
                    }
                }
                sbuf[xo] = re.inv_s;
                pybuf[xo] = re.py1;
            }
        }
    }
    if (LL && SPL) {
        if (x0 + ex < nX) {
            float* P = a.split_acc + ((long long)sp * a.part_rows + modoff + x0 + ex) * d;
            each([&](int b, int j, bool ok) __attribute__((always_inline)) {
                if (ok) *(f32x4*)(P + j) = acc[b];
            });
        }
    }
    if (LL && !SPL) {
        __syncthreads();
        const int xg = x0 + ex;
        const bool xok = xg < nX;
        const float rx = xok ? a.rstd[modoff + xg] : 0.f;
        const int tgt = xok ? a.targets[modoff + xg] : -1;
        const bool tok = tgt >= 0 && tgt < nY;
        const float inv_s = sbuf[ex], py1 = pybuf[ex];
        const bf16* hrow = hk + (long long)(xok ? xg : 0) * d;
        const bf16* wrow = Rk + (long long)(tok ? tgt : 0) * d;
        const bool want_dg = a.dg_mode == 2 || (a.dg_mode == 1 && k == a.K - 1);
        // the gain partials of the tile's two groups of 8 rows
        const long long ngp = (a.T + kF32GainRows - 1) / kF32GainRows;
        float* dgp = want_dg ? a.dgain_part + ((a.dg_mode == 2 ? k : 0) * ngp + (x0 + ex) / kF32GainRows) * d : nullptr;
        // e = (acc / s + (p_y - 1) R_y) / T and the row sums of e g n
        float cp = 0.f;
        each([&](int b, int j, bool ok) __attribute__((always_inline)) {
            const int jc = ok ? j : 0;
            const u16x4 hv = *(const u16x4*)(hrow + jc);
            const u16x4 wv = *(const u16x4*)(wrow + jc);
            const u16x4 gv = *(const u16x4*)(gk + jc);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float wy = tok ? bf16_bits_to_f32(wv[e]) : 0.f;
                float ev = __builtin_fmaf(acc[b][e], inv_s, py1 * wy) * a.inv_T;
                ev = ok ? ev : 0.f;
                cp += bf16_bits_to_f32(gv[e]) * ev * (rx * bf16_bits_to_f32(hv[e]));
                acc[b][e] = ev;
            }
        });
        cp += __shfl_xor(cp, 16, 64);
        cp += __shfl_xor(cp, 32, 64);
        if (eg == 0) cbuf[w * XR + ex] = cp;
        __syncthreads();
        float csum = 0.f;
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) csum += cbuf[ww * XR + ex];
        const float cmean = tau_k * csum / (float)d;
        if (a.rowdtau && w == 0 && eg == 0 && xok) a.rowdtau[modoff + xg] = tok ? csum : 0.f;
        if (a.ebuf) {
            // ROT heads: e in fp32; the RMSNorm backward follows the rotation back
            float* er = (float*)a.ebuf + (modoff + (xok ? xg : 0)) * (long long)d;
            each([&](int b, int j, bool ok) __attribute__((always_inline)) {
                if (ok && xok) *(f32x4*)(er + j) = acc[b];
            });
        } else {
            bf16* dhrow = (bf16*)a.dh + (modoff + (xok ? xg : 0)) * (long long)d;
            each([&](int b, int j, bool ok) __attribute__((always_inline)) {
                const int jc = ok ? j : 0;
                const u16x4 hv = *(const u16x4*)(hrow + jc);
                const u16x4 gv = *(const u16x4*)(gk + jc);
                bf16x4 o;
                f32x4 pv;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float n = rx * bf16_bits_to_f32(hv[e]);
                    o[e] = (bf16)(rx * (tau_k * bf16_bits_to_f32(gv[e]) * acc[b][e] - cmean * n));
                    if (want_dg) pv[e] = row8_sum(tau_k * acc[b][e] * n);  // rx = 0 masks rows past the end
                }
                if (ok && xok) *(bf16x4*)(dhrow + j) = o;
                if (want_dg && ok && xok && ex % kF32GainRows == 0) *(f32x4*)(dgp + j) = pv;
            });
        }
    }
    if (!LL) {
        const float db = row16_sum((float)db_part);
        if (a.dbias && yy == 0 && wr && x0 + xo < nX) a.dbias[(long long)k * a.V + x0 + xo] = db * a.inv_T;
        const int v = x0 + ex;
        float* dwrow = ((k == a.K - 1) ? a.dWt : a.dWh + (long long)k * a.V * d) + (long long)(v < nX ? v : 0) * d;
        each([&](int b, int j, bool ok) __attribute__((always_inline)) {
            // the streamed rows were the raw h: the gain joins here
            const u16x4 gv = *(const u16x4*)(gk + (ok ? j : 0));
            f32x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = acc[b][e] * bf16_bits_to_f32(gv[e]);
            if (ok && v < nX) *(f32x4*)(dwrow + j) = o;
        });
    }
}

template <int MODE, int DS, bool EXT>
hipError_t launch_ds(const FusedArgs& a, int nmod, hipStream_t s) {
    const dim3 grid((unsigned)(((MODE == LOCAL ? a.T : a.V) + XR - 1) / XR * (MODE == LOCAL ? a.nsplit : 1)),
                    (unsigned)nmod);
    if constexpr (MODE == LOCAL) {
        if (a.nsplit > 1) {
            hipLaunchKernelGGL((k_exact_wide<MODE, DS, EXT, true>), grid, dim3(NTHR), 0, s, a);
            return hipGetLastError();
        }
        if (exact_chunk_sums(a, nmod)) {
            hipLaunchKernelGGL((k_exact_wide<MODE, DS, EXT, false, true>), grid, dim3(NTHR), 0, s, a);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((k_exact_wide<MODE, DS, EXT, false>), grid, dim3(NTHR), 0, s, a);
    return hipGetLastError();
}

template <int MODE, bool EXT>
hipError_t launch_mode(const FusedArgs& a, int nmod, hipStream_t s) {
    if (a.d <= NW * 256) return launch_ds<MODE, 256, EXT>(a, nmod, s);
    if (a.d <= NW * 384) return launch_ds<MODE, 384, EXT>(a, nmod, s);
    return launch_ds<MODE, 512, EXT>(a, nmod, s);
}

}  // namespace

int exact_wide_rows() { return XR; }
hipError_t launch_local_loss_exact_wide(const FusedArgs& a, bool ext, int nmod, hipStream_t s) {
    return ext ? launch_mode<LOCAL, true>(a, nmod, s) : launch_mode<LOCAL, false>(a, nmod, s);
}
hipError_t launch_readout_grad_exact_wide(const FusedArgs& a, int nmod, hipStream_t s) {
    return launch_mode<RGRAD, false>(a, nmod, s);
}

}  // namespace solo
