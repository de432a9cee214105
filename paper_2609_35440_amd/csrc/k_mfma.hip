// Fused matrix-core passes of the SOLO shared-readout loss (bf16 operands, fp32
// accumulate) for gfx950.
//
// Every pass has the shape "logit tile -> elementwise -> (second product)".
// Module k predicts through its readout R_k (the terminal's W for k = K-1,
// the heads' read-only copy otherwise), its gain g_k, temperature tau_k and
// bias b_k (Eq. 2 of the paper, with the bias of Algorithm 1):
//
//   z_tv = tau_k r_t <R_kv, g_k * h_t> + b_kv
//
//   local-loss pass (every module; Eq. 2 and Eq. 3):
//     stationary X = XR rows t of g_k * h_k, streamed Y = the readout rows v,
//     online (max, sum-exp) per row, and acc_t += sum_{v != y_t} exp(z_tv - m_t) R_kv,
//     so that dhhat_t = tau_k (acc_t / s_t + (p_{t,y} - 1) R_{k,y_t}) / T at the
//     end (the target's whole entry of delta in fp32, see finish_row), followed
//     by the RMSNorm backward and, for a module that trains its gain, the
//     tile's partial of dgain = sum_t dhhat_t * n_t.  The T x V logits and
//     probabilities stay on chip.
//
//   exit evaluation: the same without the second product; the top-1 of each
//     row (lowest index on ties) next to its loss.
//
//   readout-gradient pass (modules whose readout is trained):
//     stationary X = XR readout rows v, streamed Y = the rows t of g_k * h_k
//     (a copy rounded like the local-loss pass's stationary tile, so both
//     passes multiply the same operands), delta_tv = (exp(z_tv - lse_t) -
//     [v = y_t]) / T and dR_v = sum_t delta_tv tau_k r_t (g_k * h_t),
//     db_v = sum_t delta_tv.
//
//   bias-gradient pass: the readout-gradient pass without the second product,
//     for modules whose bias is trained but whose readout is not.
//
// Work split: a workgroup of 8 waves owns XR stationary rows (32, 64 or 128 where
// the register file allows it: see rows_of); wave w owns the d/8 columns
// [w d/8, (w+1) d/8).  Per chunk of 16 streamed rows, every wave multiplies
// its column slice (split-K partial of the logit tile), the partials meet in
// LDS, each wave finishes the elementwise step for XR/8 of the stationary
// rows, and every wave then accumulates its own column slice of the second
// product.  The accumulator (XR rows x d/8 columns, fp32) and the stationary
// operand stay in registers for the whole pass.
//
// Streaming: in the passes with a second product the chunk goes HBM/L2 ->
// LDS directly and is read twice from LDS: row-wise for the logit product and
// with the transposing read for the second product.  The passes without one
// (exit evaluation, bias gradient) stream the tiled copy of Y (see
// tiled_elems) straight into the registers that feed the logit product, one
// contiguous 1 KiB per wave and instruction, and need no LDS for the chunk,
// which measured faster at d = 2048.  With a second product the registers
// would still have to be written to LDS for the transposing read, and those
// ds_write_b128 measured slower than the direct-to-LDS stream and the
// row-wise reads together at d = 2048, so those passes keep the stream.
#include <type_traits>

#include "mfma_common.h"

namespace solo {

namespace {

using namespace mfma;

constexpr int NW = layout::NW;  // waves per workgroup
constexpr int NTHR = NW * 64;
constexpr int YC = layout::YC;  // streamed rows per chunk
// Partial logit tiles part[w][x][y]: rows of PP = 16 floats, the 16-byte
// group y / 4 of row x stored at (y / 4) ^ ((x >> 1) & 3), so that the 16-byte
// writes (8 rows at one group per pass) and the elementwise step's reads (4
// whole rows per wave) are both free of bank conflicts.  The probability tile
// gbuf[x][y] (bf16, rows of YC) keeps the 16-byte half y / 8 of row x at
// (y / 8) ^ ((x >> 2) & 1), for its 16-byte reads of 8 rows per pass.
constexpr int PP = 16;

enum Mode { LOCAL = 0, RGRAD = 1, BGRAD = 2, EVAL = 3 };

// Stationary rows per workgroup: 64 while the accumulator (64 rows x d/8
// columns) and the stationary operand fit the register file (d <= 1024), 32
// otherwise.  The passes without a second product (no accumulator) hold as
// many rows as 128 registers of stationary operand take: 128 up to d = 1024,
// 64 at d = 2048.  The readout streamed per flop halves with each doubling.
// The exact form (XA, see k_fused) holds two planes of the stationary operand.
template <int DS, bool PC, bool XA = false>
constexpr int rows_of() {
    if (XA) return DS <= 96 ? 64 : 32;
    return (!PC && DS <= 128) ? 128 : ((DS <= 128 || (!PC && DS <= 256)) ? 64 : 32); }

template <int DS, bool PC, bool XA = false>
struct Geo : layout::Geo<DS> {
    static constexpr int XR = rows_of<DS, PC, XA>();   // stationary rows per workgroup
    static constexpr int NXP = XA ? 2 : 1;             // planes of the stationary operand
    static constexpr int NGP = XA ? 3 : 1;             // planes of the probability tile
    static constexpr int PR = XR;                      // rows of the partial-logit exchange buffer
    static constexpr int NXB = XR / 16;                // 16-row blocks of the logit product
    static constexpr int NR = XR / 32;                 // 32-row halves of the second product
    // elementwise step: a lane takes EWC adjacent streamed columns of ER
    // stationary rows, LPR lanes share a row (64-row tiles: one row and two
    // columns per lane)
    static constexpr int EWC = XR == 64 ? 2 : 1;
    static constexpr int ER = NR / EWC;
    static constexpr int LPR = 16 / EWC;
    static constexpr int NB = DS / 32;                 // 32-column accumulator blocks per wave
    static constexpr int NK = DS / 32;                 // 32-deep k-steps of the logit product
    // one chunk buffer (all waves); the passes without a second product keep no chunk in LDS
    static constexpr int YBUF = PC ? NW * layout::Geo<DS>::SLICE : 16;
    static constexpr int GB = PC ? NGP * XR * YC : 8;  // elements of the probability tile (second product only)
    // the passes without a second product keep two exchange buffers (see k_fused)
    // from d = 512 on; at 256 their registers allow two workgroups per CU and the second
    // buffer's LDS would not (2 x 20000 x 256 x 600: 97 us with it, 84 without)
    static constexpr bool TWO = !PC && DS > 32;
    static constexpr int NPART = TWO ? 2 : 1;
    static constexpr int TOTAL = 2 * YBUF + NPART * NW * PR * PP * 4 + GB * 2 + 3 * XR * 4 + NW * XR * 4 + 4 * YC * 4;
    static_assert(TOTAL <= 160 * 1024, "LDS budget");
};

__device__ __forceinline__ const bf16* readout_of(const FusedArgs& a, int k) {
    return k == a.K - 1 ? (const bf16*)a.Wt : (const bf16*)a.Wh + (long long)k * a.wh_stride;
}

// the tiled copy of module k's readout (exit evaluation)
__device__ __forceinline__ const bf16* tiled_readout_of(const FusedArgs& a, int k) {
    return k == a.K - 1 ? (const bf16*)a.Wtt : (const bf16*)a.Wht + (long long)k * a.wht_stride;
}

// MODE LOCAL / EVAL: grid (ceil(T/XR), nmod); MODE RGRAD / BGRAD: grid
// (ceil(V/XR), nmod); module k = m0 + blockIdx.y.
// EXT (LOCAL and EVAL): the variant with per-chunk biases, launched when the call has biases.
// SPL (LOCAL and EVAL): the vocabulary of a row tile is split over a.nsplit
// workgroups, and the workgroup leaves its part of every row for the merge
// (k_merge.hip).  Exit evaluation then reads the readout row-major, 64 bytes of
// 16 rows per load: few rows read it, so it comes from memory once and a tiled
// copy would triple the traffic; and it can take the rows of all modules as one
// list (a.flat) where they share one readout and no biases.
// XA (LOCAL and RGRAD): products exact to fp32, for bf16 storage whose calls are
// defined in fp32 (the widths outside this family's own): the stationary
// operand g * h (or g * R) has 16 significant bits and is held as two bf16
// planes, a probability or delta as three, and every product of planes is exact
// in the fp32 accumulation, so the streamed bf16 operand meets the full values
// at 2 and 3 matrix instructions instead of the fp32 instructions' 16 times
// slower rate.  Y is then the raw operand (R or h; dR_v = g * the sum).  The
// width d is any multiple of 8 up to 8 DS; columns past it read as zeros and
// are not written.
// CS (XA, LOCAL): a chunk's second product summed by itself before it joins the
// accumulator (see kChunkSums).
// (at d <= 256 two workgroups share a CU: at most 128 registers, 4 waves per SIMD)
template <int MODE, int DS, bool EXT, bool SPL, bool XA = false, bool CS = false>
__global__ __launch_bounds__(NTHR, CS && DS == 32 ? 4 : 1) void k_fused(FusedArgs a) {
    constexpr bool PC = MODE == LOCAL || MODE == RGRAD;     // second product
    static_assert(!XA || PC, "the exact form is of the passes with a second product");
    static_assert(!CS || (XA && MODE == LOCAL && !SPL), "chunk sums");
    using G = Geo<DS, PC, XA>;
    constexpr int XR = G::XR;
    constexpr int NR = G::NR;
    constexpr int PR = G::PR;
    constexpr bool LL = MODE == LOCAL || MODE == EVAL;      // X = h, Y = readout
    // per-lane addresses computed anew in every step where CS leaves no registers to hold them
    constexpr bool ANEW = CS && (DS == 96 || DS == 192);
    constexpr bool RF = !PC;                                // operand registers fed from the tiled copy
    constexpr bool BZ = (MODE == LOCAL || MODE == EVAL) && EXT;  // per-chunk biases through LDS
    constexpr bool RM = RF && SPL;                               // operand registers fed row-major
    static_assert(!SPL || MODE == LOCAL || MODE == EVAL, "split over the vocabulary");
    const bool flat = RM && a.flat;
    // the stream of the next chunk: instructions [0, kDmaA) one per k-step of
    // the logit products, [kDmaA, NI) after the elementwise step.  Measured:
    // with a second product, at d = 2048 5 of 8 inside the products (3 and 8
    // are 3-5% slower, 4 and 6 within box-to-box noise), at d = 1024 2 of 4 (3%
    // faster than 3 of 4); without one (64-row tiles, twice the products per
    // chunk) all of them, 12-14% faster than 5 of 8 at d = 2048
    constexpr int kDmaA = ((DS <= 128 ? 4 : 5) * G::NI + 7) / 8;
    // Separate LDS objects, so that the compiler can tell the chunk being read
    // from the chunk being prefetched (no needless waits on the prefetch).
    __shared__ __attribute__((aligned(16))) char ybufA[G::YBUF];
    __shared__ __attribute__((aligned(16))) char ybufB[G::YBUF];
    // Exchange of the partial logits.  The wider passes without a second product take
    // turns on two buffers and need one barrier per chunk: a wave that has finished the
    // elementwise step of a chunk goes on to the products of the next one, and
    // by the barrier after those every wave has left the buffer it then reuses.
    __shared__ __attribute__((aligned(16))) float part[NW * PR * PP];
    __shared__ __attribute__((aligned(16))) float partB[G::TWO ? NW * PR * PP : 4];
    __shared__ __attribute__((aligned(16))) bf16 gbuf[G::GB];
    __shared__ float abuf[XR];
    __shared__ float sbuf[XR];
    __shared__ float pybuf[XR];
    __shared__ float cbuf[NW * XR];
    // per-chunk side data streamed next to the chunk: the per-token records
    // (readout-/bias-gradient passes) or the chunk's 16 biases (local loss)
    __shared__ __attribute__((aligned(16))) float recA[YC * 4];
    __shared__ __attribute__((aligned(16))) float recB[YC * 4];

    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    const int d = a.d;
    const int js = w * DS;
    // (splits next to each other: the grid goes round-robin over the XCDs, whose L2s then
    // stream a part of the vocabulary each)
    const int tile = SPL ? (int)blockIdx.x / a.nsplit : (int)blockIdx.x;
    const int sp = SPL ? (int)blockIdx.x % a.nsplit : 0;
    const int x0 = tile * XR;
    const int k = flat ? a.K - 1 : a.m0 + (int)blockIdx.y;
    const long long modoff = flat ? 0 : (long long)k * a.T;
    const float tau_k = a.tau ? a.tau[k] : 1.f;

    const bf16* __restrict__ hk = (const bf16*)a.h + modoff * d;
    const bf16* __restrict__ Rk = readout_of(a, k);
    const bf16* __restrict__ gk = (const bf16*)a.gain + (long long)k * a.g_stride;
    const bf16* __restrict__ X = LL ? hk : Rk;
    // the streamed rows: the readout, or the copy of g_k * h_k (row-major for
    // the direct-to-LDS stream, tiled for the register-fed passes); module
    // copies sit tiled_elems(T, d) apart either way
    const bf16* __restrict__ Y = LL ? (RF && !RM ? tiled_readout_of(a, k) : Rk)
                              : (XA ? hk : (const bf16*)a.hg + (long long)(k - a.hg_m0) * tiled_elems(a.T, d));
    const int nX = LL ? (flat ? a.K * a.T : a.T) : a.V;
    const int nY = LL ? a.V : a.T;
    const int nchunks = (nY + YC - 1) / YC;
    const int ck_lo = SPL ? (int)((long long)nchunks * sp / a.nsplit) : 0;
    const int ck_hi = SPL ? (int)((long long)nchunks * (sp + 1) / a.nsplit) : nchunks;

    LDS_AS char* sliceA = (LDS_AS char*)(LDS_AS void*)ybufA + w * G::SLICE;
    LDS_AS char* sliceB = (LDS_AS char*)(LDS_AS void*)ybufB + w * G::SLICE;

    // per-lane scalars of the rows this wave finishes in the elementwise step:
    // stationary rows xo[r] = 4 w + lane/16 + 32 r and streamed column yy of
    // the chunk, or, two columns per lane, row 8 w + lane/8 and columns yy, yy + 1
    constexpr int EWC = G::EWC, ER = G::ER, LPR = G::LPR;
    int xo[ER];
#pragma unroll
    for (int r = 0; r < ER; ++r) xo[r] = EWC == 2 ? 8 * w + (lane >> 3) : 4 * w + (lane >> 4) + 32 * r;
    const int yy = EWC == 2 ? 2 * (lane & 7) : (lane & 15);
    const int lane16 = lane & 15;  // the 16 lanes that stream a chunk's side data
    float own_r2[ER];  // LL: r_t tau_k log2 e of row xo (r_t is read again after the loop)
    // LL: target of row xo minus yy, the chunk start y0 at which this lane meets
    // it (the target itself is read again after the loop)
    int tgt_rel[ER];
    float bx2[ER];     // readout-/bias-gradient passes: bias of the stationary readout row, base 2
#pragma unroll
    for (int r = 0; r < ER; ++r) {
        own_r2[r] = 0.f;
        tgt_rel[r] = -1 - yy;
        bx2[r] = 0.f;
        if (LL && x0 + xo[r] < nX) {
            const float tau_r = flat && a.tau ? a.tau[(x0 + xo[r]) / a.T] : tau_k;
            own_r2[r] = a.rstd[modoff + x0 + xo[r]] * tau_r * kLog2e;
            tgt_rel[r] = a.targets[modoff + x0 + xo[r]] - yy;
        }
        if (!LL && a.bias && x0 + xo[r] < nX) {
            const float b = a.bias[(long long)k * a.V + x0 + xo[r]];
            bx2[r] = XA ? bias2(b) : b * kLog2e;
        }
    }
    const bool has_bias = BZ || a.bias != nullptr;  // the bias variant always has one

    ChunkStream<DS> stream;
    if (PC) stream.template init<XA>(d, js, lane);
    // first chunk in flight before the stationary operand is read
    const unsigned sliceA_u = lds_addr(sliceA), sliceB_u = lds_addr(sliceB);
    if (PC) stream.issue(Y, nY, d, ck_lo * YC, sliceA_u);
    // register-fed passes: k-step kk of chunk c of this wave's slice is NK KiB
    // into chunk c of the tiled copy plus 1 KiB kk; buffer loads over those NK
    // KiB, one lane offset shared by every load and the k-step as a scalar offset
    // (row-major: over the chunk's rows, rows past the end read as zeros)
    const bf16* __restrict__ Yw = Y + (RM ? 0 : w * (G::NK * 512));
    const int rm_off = ((lane & 15) * d + js + 8 * (lane >> 4)) * 2;
    auto rsrc_of = [&](int c) __attribute__((always_inline)) {
        const int rows = nY - c * YC < YC ? nY - c * YC : YC;
        return __builtin_amdgcn_make_buffer_rsrc((void*)(Yw + (long long)c * 16 * d), (short)0,
                                                 RM ? rows * d * 2 : G::NK * 1024, 0x00020000);
    };
    auto ld_op = [&](__amdgpu_buffer_rsrc_t rs, int kk) __attribute__((always_inline)) {
        return __builtin_bit_cast(bf16x8, RM ? __builtin_amdgcn_raw_buffer_load_b128(rs, rm_off + kk * 64, 0, 0)
                                             : __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16, kk * 1024, 0));
    };
    // operand registers of the register-fed passes: k-step kk of the current
    // chunk (lane: streamed row lane % 16, columns js + 32 kk + 8 (lane / 16) .. + 7)
    bf16x8 ay_rf[RF ? G::NK : 1];
    if (RF) {
#pragma unroll
        for (int kk = 0; kk < G::NK; ++kk) ay_rf[kk] = ld_op(rsrc_of(ck_lo), kk);
    }
    const unsigned recA_u = lds_addr((LDS_AS char*)(LDS_AS void*)recA);
    const unsigned recB_u = lds_addr((LDS_AS char*)(LDS_AS void*)recB);
    auto issue_side = [&](int y0, unsigned dst) __attribute__((always_inline)) {
        // rows of this chunk only (a range over all remaining rows could pass 2^32 bytes)
        const int rows = nY - y0 < YC ? nY - y0 : YC;
        if (!LL && w == 0 && lane < YC) {
            // the 16 per-token records of the chunk
            const unsigned rem = rows > 0 ? (unsigned)rows * 16u : 0u;
            buffer_load_lds16(make_rsrc(a.rowrec + 4 * (modoff + y0), rem), dst, lane16 * 16);
        }
        if (BZ && has_bias && w == 0 && lane < YC) {
            // the 16 biases of the chunk (zeros past the vocabulary)
            const unsigned rem = rows > 0 ? (unsigned)rows * 4u : 0u;
            buffer_load_lds4(make_rsrc(a.bias + (long long)k * a.V + y0, rem), dst, lane16 * 4);
        }
    };
    issue_side(ck_lo * YC, recA_u);

    // stationary operand (local loss and exit evaluation: times the gain,
    // rounded once): B of the 16x16x32 logit product, lane holds
    // X[x0 + 16 xb + lane%16][js + 32 kk + 8 (lane/16) .. +7]
    bf16x8 xr[G::NXB][G::NK];
    bf16x8 xlo[XA ? G::NXB : 1][G::NK];  // XA: the second plane
#pragma unroll
    for (int kk = 0; kk < G::NK; ++kk) {
        const int j0 = js + 32 * kk + 8 * (lane >> 4);
        const bool jok = !XA || j0 < d;
        bf16x8 gv = *(const bf16x8*)(gk + (jok ? j0 : 0));
#pragma unroll
        for (int xb = 0; xb < G::NXB; ++xb) {
            const int xrow = x0 + 16 * xb + (lane & 15);
            bf16x8 xv;
            if (xrow < nX && jok) {
                xv = *(const bf16x8*)(X + (long long)xrow * d + j0);
                if (flat) gv = *(const bf16x8*)((const bf16*)a.gain + (long long)(xrow / a.T) * a.g_stride + j0);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) xv[e] = (bf16)0.f;
            }
            if (XA) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float p = (float)xv[e] * (float)gv[e];  // exact: 16 bits
                    xr[xb][kk][e] = (bf16)p;
                    xlo[XA ? xb : 0][kk][e] = (bf16)(p - (float)xr[xb][kk][e]);
                }
            } else if (LL) {
#pragma unroll
                for (int e = 0; e < 8; ++e) xr[xb][kk][e] = (bf16)((float)xv[e] * (float)gv[e]);
            } else {
                xr[xb][kk] = xv;
            }
        }
    }

    // accumulator: 32-column block b of this wave's slice, 32-row half h of the tile
    f32x16 acc[PC ? G::NB : 1][NR];
#pragma unroll
    for (int b = 0; b < (PC ? G::NB : 1); ++b)
#pragma unroll
        for (int h = 0; h < NR; ++h)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[b][h][i] = 0.f;

    // online softmax state (LL, base 2), per lane and row r: row xo[r], streamed column yy
    float m_run[ER], s_part[ER], zy_part[ER];
    float best[ER];   // EVAL: largest logit seen by this lane, and its column
    int best_v[ER];
    // RGRAD / BGRAD: sum_t (p - onehot) for row xo[r] (the exact form: in 64 bits, as a lane's
    // chain of T / 8 sums in fp32 is longer than that of the fp32 kernels)
    typename std::conditional<XA && !LL, double, float>::type db_part[ER];
#pragma unroll
    for (int r = 0; r < ER; ++r) {
        m_run[r] = kNoMax;
        s_part[r] = zy_part[r] = 0.f;
        db_part[r] = 0;
        best[r] = -INFINITY;
        best_v[r] = -1;
    }

    // per-lane parts of the LDS addresses; the unrolled loops add 64 * kk or 64 * b
    const int a_off = layout::rowread_off<DS>(lane);
    const int c_lo = layout::trread_off<DS>(lane, 0);
    const int c_hi = layout::trread_off<DS>(lane, 1);

    auto step = [&](LDS_AS char* cur, unsigned nxt, LDS_AS float* prt, LDS_AS float* side, unsigned side_nxt, int c)
                    __attribute__((always_inline)) {
        const int y0 = c * YC;
        const bool more = c + 1 < ck_hi;
        const i32x4 nrs = ChunkStream<DS>::rsrc(Y, nY, d, y0 + YC);
        ChunkStream<DS> strm = stream;
        if constexpr (ANEW) strm.template init<XA>(d, js, lane_now());
        // register-fed passes reload the operand registers with the next chunk
        // (the last chunk reloads itself: no branch around the loads)
        const __amdgpu_buffer_rsrc_t yn = rsrc_of(more ? c + 1 : c);

        // ---- split-K partial of the logit tile S[y][x] over this wave's columns.
        // All operand reads go out first, ahead of the data of the next chunk,
        // whose stream is spread over the products (and the end of the
        // elementwise step), so that neither the texture unit's queue nor the
        // LDS write port sees the whole chunk at once.
        bf16x8 ay[PC ? G::NK : 1];
        if (PC) {
            // the widest slices recompute the per-lane part of the row-wise read
            // address each step (no register left to hold it)
            const int ao = DS >= 224 || ANEW ? layout::rowread_off<DS>(lane_now()) : a_off;
#pragma unroll
            for (int kk = 0; kk < G::NK; ++kk) ay[kk] = *(LDS_AS bf16x8*)(cur + ao + 64 * kk);
        }
        if (!G::TWO && more) issue_side(y0 + YC, side_nxt);
        f32x4 S[G::NXB];
#pragma unroll
        for (int xb = 0; xb < G::NXB; ++xb) S[xb] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < G::NK; ++kk) {
            if constexpr (RF) {
#pragma unroll
                for (int xb = 0; xb < G::NXB; ++xb) S[xb] = mfma16(ay_rf[kk], xr[xb][kk], S[xb]);
                ay_rf[kk] = ld_op(yn, kk);
                __builtin_amdgcn_sched_barrier(0);  // keeps the reload behind this k-step's products
            } else {
#pragma unroll
                for (int xb = 0; xb < G::NXB; ++xb) S[xb] = mfma16(ay[kk], xr[xb][kk], S[xb]);
                if constexpr (XA) {
#pragma unroll
                    for (int xb = 0; xb < G::NXB; ++xb) S[xb] = mfma16(ay[kk], xlo[XA ? xb : 0][kk], S[xb]);
                }
                if (kk < kDmaA) {
                    if (more) strm.issue_one(nrs, d, nxt, kk);
                    __builtin_amdgcn_sched_barrier(0);  // keeps the instruction between these products
                }
            }
        }
        const int ylim = nY - y0;  // columns yy >= ylim of this chunk are past the last streamed row
        // C layout: lane holds S[y = 4 (lane/16) + i][x = 16 xb + lane%16]; store as part[w][x][y]
#pragma unroll
        for (int xb = 0; xb < G::NXB; ++xb) {
            const int xl = 16 * xb + (lane & 15);
            *(LDS_AS f32x4*)(prt + (w * PR + xl) * PP + 4 * ((lane >> 4) ^ ((xl >> 1) & 3))) =
                S[xb];
        }
        lds_barrier();
        if (G::TWO && more) issue_side(y0 + YC, side_nxt);  // every wave has left the previous chunk's side data
        {
            // ---- elementwise step for rows xo[r] (lane: row xo[r], columns yy .. yy + EWC - 1)
#pragma unroll
            for (int r = 0; r < ER; ++r) {
                float q[EWC][NW];
                const int xl = xo[r];
                const int yq = yy ^ (4 * ((xl >> 1) & 3));  // (yy even for two columns: both in one group)
#pragma unroll
                for (int ww = 0; ww < NW; ++ww) {
                    if constexpr (EWC == 2) {
                        const f32x2 v = *(LDS_AS f32x2*)(prt + (ww * PR + xl) * PP + yq);
                        q[0][ww] = v[0];
                        q[EWC - 1][ww] = v[1];
                    } else {
                        q[0][ww] = prt[(ww * PR + xl) * PP + yq];
                    }
                }
                static_assert(NW == 8, "partial-sum tree");
                float sxy[EWC], gval[EWC];
#pragma unroll
                for (int e = 0; e < EWC; ++e) {
                    sxy[e] = ((q[e][0] + q[e][1]) + (q[e][2] + q[e][3])) + ((q[e][4] + q[e][5]) + (q[e][6] + q[e][7]));
                    gval[e] = 0.f;
                }
                if (LL) {
                    // columns past the end of the vocabulary get z = -inf (an additive
                    // mask rather than a branch, so the partial reads stay unconditional)
                    float zc[EWC];
                    float zmax = -INFINITY;
#pragma unroll
                    for (int e = 0; e < EWC; ++e) {
                        float ymask = (yy + e < ylim) ? 0.f : -INFINITY;
                        if (BZ && has_bias) ymask += XA ? bias2(side[yy + e]) : side[yy + e] * kLog2e;
                        zc[e] = __builtin_fmaf(sxy[e], own_r2[r], ymask);
                        zmax = fmaxf(zmax, zc[e]);
                    }
                    float alpha = 1.f;
                    if (__builtin_expect(__any(zmax > m_run[r] + kLazyThresh2), 0)) {  // wave-uniform
                        const float cmax = group_max<LPR>(zmax);
                        if (cmax > m_run[r] + kLazyThresh2) {
                            alpha = __builtin_amdgcn_exp2f(m_run[r] - cmax);
                            s_part[r] *= alpha;
                            m_run[r] = cmax;
                        }
                    }
#pragma unroll
                    for (int e = 0; e < EWC; ++e) {
                        const float p = __builtin_amdgcn_exp2f(zc[e] - m_run[r]);
                        const bool is_y = tgt_rel[r] - e == y0;
                        s_part[r] += is_y ? 0.f : p;  // the target's term joins at the end (finish_row)
                        if (is_y) zy_part[r] = zc[e];
                        if (MODE == EVAL && zc[e] > best[r]) {  // strict: the first (lowest) column keeps a tie
                            best[r] = zc[e];
                            best_v[r] = y0 + yy + e;
                        }
                        // the target's probability enters the input gradient in
                        // the epilogue, in fp32 together with its one-hot term
                        gval[e] = is_y ? 0.f : p;
                    }
                    if (MODE == LOCAL) abuf[xo[r]] = alpha;  // the lanes of a row store the same value
                } else {
                    float dsum = 0.f;
#pragma unroll
                    for (int e = 0; e < EWC; ++e) {
                        // record {lse log2 e, r tau log2 e, target, p_y - 1}; tokens past
                        // the end of the module read as zeros and are masked.  The
                        // target's entry of delta is the exact p_y - 1 of the local-loss pass.
                        const f32x4 r4 = *(LDS_AS f32x4*)(side + 4 * (yy + e));
                        const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(sxy[e], r4[1], bx2[r] - r4[0]));
                        // (a padded token's zero record would match readout row 0 as its target)
                        const float dlt =
                            (yy + e < ylim) ? (__float_as_int(r4[2]) == x0 + xo[r] ? r4[3] : p) : 0.f;
                        gval[e] = dlt * (r4[1] * (kLn2 * a.inv_T));  // times r tau / T
                        if (XA) {
                            dsum += dlt;
                        } else {
                            db_part[r] += dlt;
                        }
                    }
                    if (XA) db_part[r] += dsum;
                }
                if (PC) {
#pragma unroll
                    for (int pl = 0; pl < G::NGP; ++pl) {
                        bf16* gp = gbuf + (pl * XR + xo[r]) * YC + (yy ^ (8 * ((xo[r] >> 2) & 1)));
                        if constexpr (EWC == 2) {
                            bf16x2 g2;
                            g2[0] = (bf16)gval[0];
                            g2[1] = (bf16)gval[EWC - 1];
                            *(bf16x2*)gp = g2;
                            if (XA) {
                                gval[0] -= (float)g2[0];
                                gval[EWC - 1] -= (float)g2[1];
                            }
                        } else {
                            const bf16 g1 = (bf16)gval[0];
                            *gp = g1;
                            if (XA) gval[0] -= (float)g1;
                        }
                    }
                }
            }
        }
        if (PC && more) strm.template issue_range<kDmaA, G::NI>(nrs, d, nxt);
        if (!G::TWO) lds_barrier();

        // 64-row tiles: the second product runs at raised wave priority, so that
        // a wave's products for the next chunk do not overtake the other wave's
        // second product on the SIMD (measured 2.3% faster at d = 1024; at
        // d = 2048 with 32-row tiles it is 0.5% slower and not used)
        constexpr bool PRIO = PC && XR == 64;
        if (PRIO) __builtin_amdgcn_s_setprio(2);
        if constexpr (CS) {
            // ---- second product as below, a half of the rows at a time, and each block's sum over the
            // chunk, smallest plane first, added to the accumulator by itself.  One sum is in
            // flight: the other wave of the SIMD fills the gaps, and there are no registers for more.
            constexpr int NA = NR == 1 ? 2 : G::NB;  // transposed operands held (one half: read one block ahead)
            bf16x4 tlo[NA], thi[NA];
            const int l = ANEW ? lane_now() : lane;
            const int t_lo = ANEW ? layout::trread_off<DS>(l, 0) : c_lo;
            const int t_hi = ANEW ? layout::trread_off<DS>(l, 1) : c_hi;
            auto rd = [&](int b) __attribute__((always_inline)) {
                tlo[b % NA] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_AS bf16x4*)(cur + t_lo + 64 * b));
                thi[b % NA] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_AS bf16x4*)(cur + t_hi + 64 * b));
            };
#pragma unroll
            for (int b = 0; b < (NR == 1 ? 1 : G::NB); ++b) rd(b);
#pragma unroll
            for (int h = 0; h < NR; ++h) {
                bf16x8 gfrag[G::NGP];
                const int xg = 32 * h + (l & 31);
#pragma unroll
                for (int pl = 0; pl < G::NGP; ++pl)
                    gfrag[pl] = *(bf16x8*)(gbuf + (pl * XR + xg) * YC + 8 * ((l >> 5) ^ ((xg >> 2) & 1)));
                const float al = abuf[xg];
                if (__any(al != 1.f)) {
#pragma unroll
                    for (int b = 0; b < G::NB; ++b)
#pragma unroll
                        for (int i = 0; i < 16; ++i) acc[b][h][i] *= al;
                }
#pragma unroll
                for (int b = 0; b < G::NB; ++b) {
                    if (NR == 1 && b + 1 < G::NB) rd(b + 1);
                    bf16x8 at;
                    at[0] = tlo[b % NA][0]; at[1] = tlo[b % NA][1]; at[2] = tlo[b % NA][2]; at[3] = tlo[b % NA][3];
                    at[4] = thi[b % NA][0]; at[5] = thi[b % NA][1]; at[6] = thi[b % NA][2]; at[7] = thi[b % NA][3];
                    f32x16 t = {};
#pragma unroll
                    for (int pl = G::NGP - 1; pl >= 0; --pl) t = mfma32(at, gfrag[pl], t);
                    acc[b][h] += t;
                    // here and now (the additions would sink to the next chunk, and with them
                    // every block's sum would stay in registers)
                    asm volatile("" : "+v"(acc[b][h]));
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        } else if (PC) {
            // ---- second product: acc[j][x] += sum_y Y[y][j] G[x][y] over this wave's columns
            bf16x8 gfrag[G::NGP][NR];
#pragma unroll
            for (int pl = 0; pl < G::NGP; ++pl)
#pragma unroll
                for (int h = 0; h < NR; ++h) {
                    const int xg = 32 * h + (lane & 31);
                    gfrag[pl][h] =
                        *(bf16x8*)(gbuf + (pl * XR + xg) * YC + 8 * ((lane >> 5) ^ ((xg >> 2) & 1)));
                }
            if (MODE == LOCAL) {
#pragma unroll
                for (int h = 0; h < NR; ++h) {
                    const float al = abuf[32 * h + (lane & 31)];
                    if (__any(al != 1.f)) {
#pragma unroll
                        for (int b = 0; b < G::NB; ++b)
#pragma unroll
                            for (int i = 0; i < 16; ++i) acc[b][h][i] *= al;
                    }
                }
            }
            bf16x4 tlo[G::NB], thi[G::NB];
#pragma unroll
            for (int b = 0; b < G::NB; ++b) {
                tlo[b] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_AS bf16x4*)(cur + c_lo + 64 * b));
                thi[b] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_AS bf16x4*)(cur + c_hi + 64 * b));
            }
#pragma unroll
            for (int b = 0; b < G::NB; ++b) {
                bf16x8 at;
                at[0] = tlo[b][0]; at[1] = tlo[b][1]; at[2] = tlo[b][2]; at[3] = tlo[b][3];
                at[4] = thi[b][0]; at[5] = thi[b][1]; at[6] = thi[b][2]; at[7] = thi[b][3];
#pragma unroll
                for (int pl = 0; pl < G::NGP; ++pl)
#pragma unroll
                    for (int h = 0; h < NR; ++h) acc[PC ? b : 0][h] = mfma32(at, gfrag[pl][h], acc[PC ? b : 0][h]);
            }
        }
        if (PRIO) __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_sched_barrier(0);
        // the untracked streams: the chunk and the side data (wave 0's)
        if (PC || ((!LL || BZ) && w == 0)) wait_vm();
    };

    wait_vm();
    for (int c = ck_lo; c < ck_hi; c += 2) {
        step(sliceA, sliceB_u, (LDS_AS float*)(LDS_AS void*)part, (LDS_AS float*)(LDS_AS void*)recA, recB_u, c);
        if (c + 1 < ck_hi)
            step(sliceB, sliceA_u, (LDS_AS float*)(LDS_AS void*)(G::TWO ? partB : part),
                 (LDS_AS float*)(LDS_AS void*)recB, recA_u, c + 1);
    }

    // ---- epilogues.  acc[b][h] lane layout: x = 32 h + lane%32,
    //      j = js + 32 b + 8 (i/4) + 4 (lane/32) + i%4 for i = 0..15
    const int ex = lane & 31;
    const int ehh = lane >> 5;
    if (LL) {
        // finish the online softmax of rows xo[r]
#pragma unroll
        for (int r = 0; r < ER; ++r) {
            const int own_tgt = x0 + xo[r] < nX ? a.targets[modoff + x0 + xo[r]] : -1;
            const float sx = group_sum<LPR>(s_part[r]);
            const float zy = group_sum<LPR>(zy_part[r]);
            float bst = best[r];
            int bv = best_v[r];
            if (MODE == EVAL) {
                // argmax over the lanes of the row: larger logit, then lower column
#pragma unroll
                for (int off = 1; off < LPR; off <<= 1) {
                    const float ob = __shfl_xor(bst, off, 64);
                    const int ov = __shfl_xor(bv, off, 64);
                    if (ob > bst || (ob == bst && (unsigned)ov < (unsigned)bv)) {
                        bst = ob;
                        bv = ov;
                    }
                }
            }
            if (SPL) {
                if (lane % LPR == 0 && x0 + xo[r] < nX) {
                    constexpr int SW = MODE == EVAL ? 8 : 4;  // floats per row and split
                    float* st = a.split_stat + SW * ((long long)sp * a.part_rows + modoff + x0 + xo[r]);
                    *(f32x4*)st = (f32x4){m_run[r], sx, zy, bst};
                    if (MODE == EVAL) *(f32x4*)(st + 4) = (f32x4){__int_as_float(bv), 0.f, 0.f, 0.f};
                }
                continue;
            }
            if (lane % LPR == 0) {
                const int xr_ = x0 + xo[r];
                const bool tok = own_tgt >= 0 && own_tgt < nY;
                const RowEnd re = finish_row<XA>(m_run[r], sx, zy, tok);
                if (xr_ < nX) {
                    const long long t = modoff + xr_;
                    a.lse[t] = XA ? 1.f : re.lse2 * kLn2;  // (the fp32 family's gradient passes scale by it)
                    a.rowloss[t] = re.loss;
                    if (MODE == EVAL && a.top1) a.top1[t] = bv;
                    if (MODE == LOCAL && a.rowrec) {
                        f32x4 rec4 = {re.lse2, own_r2[r], __int_as_float(own_tgt), re.py1};
                        *(f32x4*)(a.rowrec + 4 * t) = rec4;
                    }
                }
                sbuf[xo[r]] = re.inv_s;
                // p_y - 1: the target's probability was left out of the probability tile
                if (MODE == LOCAL) pybuf[xo[r]] = re.py1;
            }
        }
    }
    if (MODE == LOCAL && SPL) {
        // the unnormalised partial sums of this split, for the merge
#pragma unroll
        for (int h = 0; h < NR; ++h) {
            const int xg = x0 + 32 * h + ex;
            if (xg >= nX) continue;
            float* P = a.split_acc + ((long long)sp * a.part_rows + modoff + xg) * d;
#pragma unroll
            for (int b = 0; b < (PC ? G::NB : 1); ++b)
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4) {
                    f32x4 o;
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = acc[b][h][4 * i4 + e];
                    if (!XA || js + 32 * b + 8 * i4 < d) *(f32x4*)(P + js + 32 * b + 8 * i4 + 4 * ehh) = o;
                }
        }
    }
    if (MODE == LOCAL && !SPL) {
        __syncthreads();
        const bool want_dg = a.dg_mode == 2 || (a.dg_mode == 1 && k == a.K - 1);
        // (XA: one partial per 8 rows, see kF32GainRows)
        const long long ngp = XA ? (a.T + kF32GainRows - 1) / kF32GainRows : gridDim.x;
        float* dgp = want_dg ? a.dgain_part + ((a.dg_mode == 2 ? k : 0) * ngp +
                                               (XA ? (x0 + ex) / kF32GainRows : blockIdx.x)) * d
                             : nullptr;
        bool xok[NR], tok[NR];
        float rx[NR];
        const bf16* hrow[NR];
        // sweep 1: acc <- e = (acc / s + (p_y - 1) R_y) / T, so that dhhat = tau e
        // (acc holds every column but the target's, whose probability term
        // joins its one-hot term here in fp32), and the row sums of e * g * n
        // (n = r h).  That row sum is both the RMSNorm backward's mean(dn * n)
        // = tau sum / d and the token's share of d loss / d tau = sum_v
        // delta_v u_v = <sum_v delta_v R_v, g * n>.
#pragma unroll
        for (int h = 0; h < NR; ++h) {
            const int xg = x0 + 32 * h + ex;
            xok[h] = xg < nX;
            rx[h] = xok[h] ? a.rstd[modoff + xg] : 0.f;
            const int tgt = xok[h] ? a.targets[modoff + xg] : -1;
            tok[h] = tgt >= 0 && tgt < nY;
            const float inv_s = sbuf[32 * h + ex];
            const float py1 = pybuf[32 * h + ex];
            hrow[h] = hk + (long long)(xok[h] ? xg : 0) * d;
            const bf16* wrow = Rk + (long long)(tok[h] ? tgt : 0) * d;
            float cp = 0.f;
#pragma unroll
            for (int b = 0; b < (PC ? G::NB : 1); ++b) {
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4) {
                    const int j = js + 32 * b + 8 * i4 + 4 * ehh;
                    // unconditional loads (the row pointers are clamped to row 0), masked
                    // afterwards: no control flow inside the sweep
                    const int jc = XA && j >= d ? 0 : j;
                    const u16x4 hv = *(const u16x4*)(hrow[h] + jc);
                    const u16x4 wv = *(const u16x4*)(wrow + jc);
                    const u16x4 gv = *(const u16x4*)(gk + jc);
                    if (XA && j >= d) {  // (columns past the width hold the streamed rows' zeros, and add none)
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[b][h][4 * i4 + e] = 0.f;
                        continue;
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float wy = tok[h] ? bf16_bits_to_f32(wv[e]) : 0.f;
                        const float ev = __builtin_fmaf(acc[b][h][4 * i4 + e], inv_s, py1 * wy) * a.inv_T;
                        cp += bf16_bits_to_f32(gv[e]) * ev * (rx[h] * bf16_bits_to_f32(hv[e]));
                        acc[b][h][4 * i4 + e] = ev;
                    }
                }
                __builtin_amdgcn_sched_barrier(0);  // one block's loads at a time
            }
            cp += __shfl_xor(cp, 32, 64);
            if (ehh == 0) cbuf[w * XR + 32 * h + ex] = cp;
        }
        __syncthreads();
        // sweep 2: dh = r (dn - c n).  The accumulator layout gives a lane 8
        // bytes of a row per store (16 contiguous bytes per row and
        // instruction), which the memory system writes back as partial lines.
        // The 32 rows of a half-tile are staged in this wave's two (now idle)
        // chunk slices instead, 16 rows each, granule g of row r at g ^ (r & SM),
        // and leave as whole row segments of the wave's columns.
        constexpr int GS = DS / 8;  // 16-byte granules per row of the wave's columns
        constexpr int SM = (GS % 16 == 0) ? 15 : ((GS % 8 == 0) ? 7 : 3);
        static_assert(GS % 4 == 0 && 16 * 2 * DS <= G::SLICE, "staging rows fit a chunk slice");
#pragma unroll
        for (int h = 0; h < NR; ++h) {
            const int xg = x0 + 32 * h + ex;
            float csum = 0.f;
#pragma unroll
            for (int ww = 0; ww < NW; ++ww) csum += cbuf[ww * XR + 32 * h + ex];
            const float cmean = tau_k * csum / (float)d;
            if (a.rowdtau && w == 0 && ehh == 0 && xok[h]) a.rowdtau[modoff + xg] = tok[h] ? csum : 0.f;
            if (a.ebuf) {
                // e to the buffer as bf16 planes hi | lo (XA: in fp32); the RMSNorm backward
                // follows the rotation back
                if (XA) {
                    if (!xok[h]) continue;
                    float* er = (float*)a.ebuf + (modoff + xg) * (long long)d;
#pragma unroll
                    for (int b = 0; b < (PC ? G::NB : 1); ++b)
#pragma unroll
                        for (int i4 = 0; i4 < 4; ++i4) {
                            const int j = js + 32 * b + 8 * i4 + 4 * ehh;
                            f32x4 o;
#pragma unroll
                            for (int e = 0; e < 4; ++e) o[e] = acc[b][h][4 * i4 + e];
                            if (j < d) *(f32x4*)(er + j) = o;
                        }
                    continue;
                }
                if (xok[h]) {
                    bf16* er = (bf16*)a.ebuf + (modoff + xg) * (long long)(2 * d);
#pragma unroll
                    for (int b = 0; b < (PC ? G::NB : 1); ++b)
#pragma unroll
                        for (int i4 = 0; i4 < 4; ++i4) {
                            const int j = js + 32 * b + 8 * i4 + 4 * ehh;
                            mfma::bf16x4 hi, lo;
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                hi[e] = (bf16)acc[b][h][4 * i4 + e];
                                lo[e] = (bf16)(acc[b][h][4 * i4 + e] - (float)hi[e]);
                            }
                            *(mfma::bf16x4*)(er + j) = hi;
                            *(mfma::bf16x4*)(er + d + j) = lo;
                        }
                }
                continue;
            }
            LDS_AS char* srow = (ex < 16 ? sliceA : sliceB) + (ex & 15) * (2 * DS);
#pragma unroll
            for (int b = 0; b < (PC ? G::NB : 1); ++b) {
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4) {
                    const int j = js + 32 * b + 8 * i4 + 4 * ehh;
                    const int jc = XA && j >= d ? 0 : j;
                    const u16x4 hv = *(const u16x4*)(hrow[h] + jc);  // row 0 for rows past the end
                    const u16x4 gv = *(const u16x4*)(gk + jc);
                    bf16x4 o;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float n = rx[h] * bf16_bits_to_f32(hv[e]);
                        o[e] = (bf16)(rx[h] * (tau_k * bf16_bits_to_f32(gv[e]) * acc[b][h][4 * i4 + e] - cmean * n));
                    }
                    *(LDS_AS bf16x4*)(srow + 16 * ((4 * b + i4) ^ (ex & SM)) + 8 * ehh) = o;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            // lane p of store q moves granule slot 64 q + p of the 32 x GS staged granules
#pragma unroll
            for (int q = 0; q < GS / 2; ++q) {
                const int sl = 64 * q + lane, row = sl / GS, g = sl % GS;
                const i32x4 v = *(LDS_AS i32x4*)((row < 16 ? sliceA : sliceB) + (row & 15) * (2 * DS) +
                                                 16 * (g ^ (row & SM)));
                const int xr = x0 + 32 * h + row;
                if (xr < nX && (!XA || js + 8 * g < d)) *(i32x4*)((bf16*)a.dh + (modoff + xr) * (long long)d + js + 8 * g) = v;
            }
        }
        // sweep 3, for a module that trains its gain: the tile's partial sums
        // of dhhat * n = tau e * n over its rows (the 16-lane row, the other row
        // of the half-wave, then the other 32-row half of the tile)
        if (want_dg && !a.ebuf) {
#pragma unroll
            for (int b = 0; b < (PC ? G::NB : 1); ++b) {
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4) {
                    const int j = js + 32 * b + 8 * i4 + 4 * ehh;
                    f32x4 pv = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int h = 0; h < NR; ++h) {
                        const u16x4 hv = *(const u16x4*)(hrow[h] + (XA && j >= d ? 0 : j));  // rx = 0 masks rows past the end
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const float n = rx[h] * bf16_bits_to_f32(hv[e]);
                            if constexpr (XA) {
                                pv[e] = row8_sum(tau_k * acc[b][h][4 * i4 + e] * n);
                            } else {
                                const float t = row16_sum(tau_k * acc[b][h][4 * i4 + e] * n);
                                pv[e] += t + __shfl_xor(t, 16, 64);
                            }
                        }
                        if (XA && j < d && xok[h] && ex % kF32GainRows == 0)
                            *(f32x4*)(dgp + 32 / kF32GainRows * h * d + j) = pv;
                    }
                    if (!XA && ex == 0) *(f32x4*)(dgp + j) = pv;
                }
            }
        }
    }
    if (!LL) {
        // bias gradient of the stationary readout rows: sum over the lanes of the row
#pragma unroll
        for (int r = 0; r < ER; ++r) {
            const float db = group_sum<LPR>((float)db_part[r]);
            if (a.dbias && lane % LPR == 0 && x0 + xo[r] < nX)
                a.dbias[(long long)k * a.V + x0 + xo[r]] = db * a.inv_T;
        }
    }
    if (MODE == RGRAD) {
        // dR_v = D_v
#pragma unroll
        for (int h = 0; h < NR; ++h) {
            const int v = x0 + 32 * h + ex;
            const bool vok = v < nX;
            float* dR = (k == a.K - 1) ? a.dWt : a.dWh + (long long)k * a.V * d;
            float* dwrow = dR + (long long)(vok ? v : 0) * d;
#pragma unroll
            for (int b = 0; b < (PC ? G::NB : 1); ++b) {
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4) {
                    const int j = js + 32 * b + 8 * i4 + 4 * ehh;
                    f32x4 o;
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = acc[b][h][4 * i4 + e];
                    if (XA) {
                        // the streamed rows were the raw h: the gain joins here
                        const u16x4 gv = *(const u16x4*)(gk + (j < d ? j : 0));
#pragma unroll
                        for (int e = 0; e < 4; ++e) o[e] *= bf16_bits_to_f32(gv[e]);
                    }
                    if (vok && (!XA || j < d)) *(f32x4*)(dwrow + j) = o;
                }
            }
        }
    }
}

template <int MODE, int DS, bool EXT>
hipError_t launch_ds(const FusedArgs& a, int nmod, hipStream_t s) {
    const bool ll = MODE == LOCAL || MODE == EVAL;
    constexpr int XR = Geo<DS, MODE == LOCAL || MODE == RGRAD>::XR;
    if constexpr (MODE == LOCAL || MODE == EVAL) {
        if (a.nsplit > 1 || a.flat) {
            const int rows = a.flat ? a.K * a.T : a.T;
            const dim3 grid((unsigned)((rows + XR - 1) / XR * a.nsplit), a.flat ? 1u : (unsigned)nmod);
            hipLaunchKernelGGL((k_fused<MODE, DS, EXT, true>), grid, dim3(NTHR), 0, s, a);
            return hipGetLastError();
        }
    }
    dim3 grid = ll ? dim3((unsigned)((a.T + XR - 1) / XR), (unsigned)nmod)
                   : dim3((unsigned)((a.V + XR - 1) / XR), (unsigned)nmod);
    hipLaunchKernelGGL((k_fused<MODE, DS, EXT, false>), grid, dim3(NTHR), 0, s, a);
    return hipGetLastError();
}

template <int MODE, int DS, bool EXT>
hipError_t launch_exact_ds(const FusedArgs& a, int nmod, hipStream_t s) {
    constexpr int XR = rows_of<DS, true, true>();
    const dim3 grid((unsigned)(((MODE == LOCAL ? a.T : a.V) + XR - 1) / XR * (MODE == LOCAL ? a.nsplit : 1)),
                    (unsigned)nmod);
    if constexpr (MODE == LOCAL) {
        if (a.nsplit > 1) {
            hipLaunchKernelGGL((k_fused<MODE, DS, EXT, true, true>), grid, dim3(NTHR), 0, s, a);
            return hipGetLastError();
        }
        if (exact_chunk_sums(a, nmod)) {
            hipLaunchKernelGGL((k_fused<MODE, DS, EXT, false, true, true>), grid, dim3(NTHR), 0, s, a);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((k_fused<MODE, DS, EXT, false, true>), grid, dim3(NTHR), 0, s, a);
    return hipGetLastError();
}

template <int MODE, bool EXT>
hipError_t launch_exact(const FusedArgs& a, int nmod, hipStream_t s) {
    switch ((a.d + NW * 32 - 1) / (NW * 32)) {
        case 1: return launch_exact_ds<MODE, 32, EXT>(a, nmod, s);
        case 2: return launch_exact_ds<MODE, 64, EXT>(a, nmod, s);
        case 3: return launch_exact_ds<MODE, 96, EXT>(a, nmod, s);
        case 4: return launch_exact_ds<MODE, 128, EXT>(a, nmod, s);
        case 5: return launch_exact_ds<MODE, 160, EXT>(a, nmod, s);
        case 6: return launch_exact_ds<MODE, 192, EXT>(a, nmod, s);
        default: return hipErrorInvalidValue;
    }
}

template <int MODE, bool EXT>
hipError_t launch_mode(const FusedArgs& a, int nmod, hipStream_t s) {
    switch (a.d / NW) {
        case 32: return launch_ds<MODE, 32, EXT>(a, nmod, s);
        case 64: return launch_ds<MODE, 64, EXT>(a, nmod, s);
        case 96: return launch_ds<MODE, 96, EXT>(a, nmod, s);
        case 128: return launch_ds<MODE, 128, EXT>(a, nmod, s);
        case 160: return launch_ds<MODE, 160, EXT>(a, nmod, s);
        case 192: return launch_ds<MODE, 192, EXT>(a, nmod, s);
        case 224: return launch_ds<MODE, 224, EXT>(a, nmod, s);
        case 256: return launch_ds<MODE, 256, EXT>(a, nmod, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

bool mfma_supported(int dtype, int d) { return dtype == 0 && d % (NW * 32) == 0 && d >= NW * 32 && d <= NW * 256; }

int mfma_eval_rows(int d) { return d <= NW * 128 ? rows_of<128, false>() : rows_of<256, false>(); }

int mfma_rows(int d) { return d <= NW * 128 ? rows_of<128, true>() : rows_of<256, true>(); }

// From d = 72 to 1536: up to 64 the fp32 kernels' narrow column slices are faster on most
// sizes (training at d = 64: 2 x 256 x 512 46 us against 66, 2 x 1001 x 8003 135 against 247,
// 20000 x 2000 0.76 ms against 1.34, but 4 x 8192 x 32000 4.5 ms against 3.6), and past 1536 two planes of 32 rows do not fit the registers
// next to the accumulator.  At 4 x 8192 x 32000 tokens, against the fp32 kernels: d =
// 640 9.2 ms against 35.8, d = 104 3.7 against 7.7 (fp32 storage).
bool exact_supported(int dtype, int d) { return dtype == 0 && d > 64 && d <= NW * 192; }
int exact_rows(int d) { return d <= NW * 96 ? rows_of<96, true, true>() : rows_of<128, true, true>(); }
hipError_t launch_local_loss_exact(const FusedArgs& a, bool ext, int nmod, hipStream_t s) {
    return ext ? launch_exact<LOCAL, true>(a, nmod, s) : launch_exact<LOCAL, false>(a, nmod, s);
}
hipError_t launch_readout_grad_exact(const FusedArgs& a, int nmod, hipStream_t s) {
    return launch_exact<RGRAD, false>(a, nmod, s);
}

hipError_t launch_local_loss_mfma(const FusedArgs& a, bool ext, int nmod, hipStream_t s) {
    return ext ? launch_mode<LOCAL, true>(a, nmod, s) : launch_mode<LOCAL, false>(a, nmod, s);
}
hipError_t launch_exit_eval_mfma(const FusedArgs& a, int nmod, hipStream_t s) {
    return a.bias ? launch_mode<EVAL, true>(a, nmod, s) : launch_mode<EVAL, false>(a, nmod, s);
}
hipError_t launch_readout_grad_mfma(const FusedArgs& a, int nmod, hipStream_t s) {
    return launch_mode<RGRAD, false>(a, nmod, s);
}
hipError_t launch_bias_grad_mfma(const FusedArgs& a, int nmod, hipStream_t s) {
    return launch_mode<BGRAD, false>(a, nmod, s);
}

}  // namespace solo
