// C ABI of the SOLO shared-readout local loss: argument checks, workspace
// layout and the launch sequence on the caller's stream.
#include <cmath>
#include <cstdint>
#include <mutex>

#include "solo_readout.h"
#include "solo_internal.h"

namespace {

constexpr size_t kAlign = 256;

size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

bool shape_ok(int K, int T, int d, int V) {
    if (K < 1 || T < 1 || V < 1) return false;
    if (d < 8 || d % 8 != 0 || d > 4096) return false;
    if (K > 65535 || T > (1 << 30) || V > (1 << 30)) return false;
    if ((long long)K * (long long)T > 2147483647LL) return false;
    return true;
}

bool flag_ok(int f) { return f == 0 || f == 1; }

// What one call launches, and where its workspace pieces sit.
struct Plan {
    bool mfma = false;         // matrix-core family (either tiling)
    bool exact = false;        // fp32 family, bf16 storage: local loss and readout gradient in the exact form (k_mfma.hip)
    bool xwide = false;        // the exact form's wide kernels (k_exact_wide.hip)
    bool planes = false;       // fp32 family, bf16 storage: forward-only products on plane copies (k_logits.hip)
    size_t eval_room = 0;      // bytes at wtile that the forms of exit evaluation without tiled copies may use
    bool wide = false;         // the 16-row wide tiling of the matrix-core family (d = 2560)
    bool eval = false;
    bool ext = false;          // local-loss variant with per-chunk biases
    int dg_mode = 0;           // 0 none, 1 terminal only, 2 every module
    int slots = 0;             // gain-gradient partial slots
    int ntiles = 0;            // token tiles of the local-loss pass
    int dg_rows = 0;           // token rows per gain-gradient partial: a tile's, or 8 outside the bf16 families
    int rg_lo = 0, rg_hi = 0;  // modules of the readout-gradient pass
    int bg_lo = 0, bg_hi = 0;  // modules of the bias-gradient pass
    int hg_lo = 0, hg_hi = 0;  // modules whose gain-scaled copy the matrix-core gradient passes stream
    int nhead_tiles = 0;       // tiled copies of the heads' readouts (0: the heads read W's copy)
    int rows = 0;              // token rows per tile of the local-loss pass
    bool rot = false;          // ROT heads: modules 0..K-2 read Wbar R_k through rotated rows
    size_t rstd = 0, lse = 0, rowloss = 0, rowrec = 0, rowdtau = 0, dgp = 0, hg = 0;
    size_t wtile = 0, whtile = 0, total = 0;
    // ROT pieces: a vector of ones (the rotated rows' gain), the rotated rows
    // u, the heads' e = sum_v delta_v Wbar_v (4 bytes per element: two bf16
    // planes, or fp32 on the fp32 family), D = e R_k (fp32), R_k^T
    size_t ones = 0, ubuf = 0, ebuf = 0, dbuf = 0, rtr = 0;
};

// Which passes stream tiled copies: every pass of the wide tiling; in the
// 16-row tiling the passes without a second product (exit evaluation, bias
// gradient), which read their operand straight into registers.  The others
// (and the fp32 family) read the row-major matrices.
bool tiled_readout(const Plan& P) { return P.wide || (P.mfma && P.eval); }
bool tiled_rgrad(const Plan& P) { return P.wide; }

// Sizes, dtype and flags only (no pointer is dereferenced).  `spare` false lays
// the workspace out without the copies that bf16 storage in fp32 can do without.
bool make_plan(const solo_readout_args& a, bool eval, Plan* P, bool spare = true) {
    *P = Plan();
    if (a.dtype != SOLO_BF16 && a.dtype != SOLO_F32) return false;
    if (!shape_ok(a.K, a.T, a.d, a.V)) return false;
    if (!flag_ok(a.gain_per_module) || !flag_ok(a.readout_per_head) || !flag_ok(a.final_module_dW) ||
        !flag_ok(a.heads_train_readout))
        return false;
    if (a.rot && a.readout_per_head) return false;
    const int K = a.K, T = a.T, d = a.d;
    P->wide = solo::mfma_wide_supported(a.dtype, d);
    P->mfma = solo::mfma_supported(a.dtype, d) || P->wide;
    P->xwide = !P->mfma && a.dtype == SOLO_BF16 && d > 1536;
    P->exact = P->xwide || (!P->mfma && solo::exact_supported(a.dtype, d));
    P->eval = eval;
    const size_t kt = (size_t)K * T;
    size_t off = 0;
    P->rstd = off;
    off = align_up(off + kt * 4);
    P->lse = off;
    off = align_up(off + kt * 4);
    P->rowloss = off;
    off = align_up(off + kt * 4);
    // bf16 storage in fp32: the product form of exit evaluation (plane copies of the
    // rows, up to 16384 at a time, and the parts of its splits)
    P->planes = spare && !P->mfma && a.dtype == SOLO_BF16 && (eval || P->exact);
    if (P->planes && eval) {
        const size_t nvt = ((size_t)a.V + 255) / 256;
        const size_t parts = kt * 32 * (nvt < solo::kEvalSplits ? nvt : solo::kEvalSplits);
        P->eval_room = (kt < 16384 ? kt : 16384) * solo::plane_pitch(d) * 2 + 512 +
                       (parts < (size_t(32) << 20) ? parts : (size_t(32) << 20));
        P->wtile = off;
        off = align_up(off + P->eval_room);
    }
    // tiled copies of the readouts the local-loss pass and exit evaluation
    // stream: the terminal's W, and the heads' own matrix or matrices
    if (tiled_readout(*P)) {
        const size_t tv = (size_t)solo::tiled_elems(a.V, d) * 2;
        P->eval_room = tv;
        P->nhead_tiles = (a.Wbar && K > 1) ? (a.readout_per_head ? K - 1 : 1) : 0;
        P->wtile = off;
        off = align_up(off + tv);
        P->whtile = off;
        off = align_up(off + tv * P->nhead_tiles);
    }
    const int rows = P->wide ? solo::kMfmaWideRows : (P->mfma ? solo::mfma_rows(d) : (P->xwide   ? solo::exact_wide_rows()
                                                                 : P->exact ? solo::exact_rows(d)
                                                                            : solo::f32_rows(d)));
    P->rows = rows;
    P->ntiles = (T + rows - 1) / rows;
    P->dg_rows = P->mfma ? rows : solo::kF32GainRows;
    P->rot = a.rot != nullptr && K > 1;
    if (P->rot) {
        const size_t es = a.dtype == SOLO_BF16 ? 2 : 4;
        const size_t htd = (size_t)(K - 1) * T * d;
        P->ones = off;
        off = align_up(off + (size_t)d * es);
        P->ubuf = off;
        off = align_up(off + htd * es);
        if (!eval) {
            P->ebuf = off;
            off = align_up(off + htd * 4);
            P->dbuf = off;
            off = align_up(off + htd * 4);
            P->rtr = off;
            off = align_up(off + (size_t)(K - 1) * d * d * es);
        }
    }
    if (eval) {
        P->total = off;
        return true;
    }
    const bool priv = a.heads_train_readout && K > 1;
    const bool fdw = a.final_module_dW;
    // readout-gradient modules: the terminal if its dW is asked for, the heads under PRIV
    P->rg_lo = priv ? 0 : K - 1;
    P->rg_hi = fdw ? K : (priv ? K - 1 : K - 1);
    if (!fdw && !priv) P->rg_lo = P->rg_hi = 0;
    // bias-gradient modules: every other module, if the bias gradient is asked for
    if (a.dbias) {
        if (P->rg_hi == P->rg_lo) {
            P->bg_lo = 0;
            P->bg_hi = K;
        } else if (P->rg_lo == 0 && P->rg_hi == K) {
            P->bg_lo = P->bg_hi = 0;
        } else if (P->rg_lo == 0) {
            P->bg_lo = K - 1;
            P->bg_hi = K;
        } else {
            P->bg_lo = 0;
            P->bg_hi = K - 1;
        }
    }
    P->ext = a.bias != nullptr;
    P->dg_mode = a.gain_per_module ? 2 : (fdw ? 1 : 0);
    P->slots = P->dg_mode == 2 ? K : (P->dg_mode == 1 ? 1 : 0);
    const bool second = P->rg_hi > P->rg_lo || P->bg_hi > P->bg_lo;
    if (P->mfma && second) {
        // the two ranges are disjoint parts of [0, K): their union is one range
        const bool rg = P->rg_hi > P->rg_lo, bg = P->bg_hi > P->bg_lo;
        P->hg_lo = rg && bg ? (P->rg_lo < P->bg_lo ? P->rg_lo : P->bg_lo) : (rg ? P->rg_lo : P->bg_lo);
        P->hg_hi = rg && bg ? (P->rg_hi > P->bg_hi ? P->rg_hi : P->bg_hi) : (rg ? P->rg_hi : P->bg_hi);
    }
    P->rowrec = off;
    off = align_up(off + (second ? kt * 16 : 0));
    P->hg = off;
    off = align_up(off + (size_t)(P->hg_hi - P->hg_lo) * (size_t)solo::tiled_elems(T, d) * 2);
    // plane copies of the bias-gradient modules' rows
    if (P->planes) off = align_up(off + (size_t)(P->bg_hi - P->bg_lo) * T * solo::plane_pitch(d) * 2);
    P->rowdtau = off;
    off = align_up(off + (a.dtau ? kt * 4 : 0));
    P->dgp = off;
    off = align_up(off + (size_t)P->slots * (((size_t)T + P->dg_rows - 1) / P->dg_rows) * d * 4);
    P->total = off;
    return true;
}

// Splits of a row tile's vocabulary over several workgroups.  These kernels run
// one workgroup per CU, so a launch of `tiles` row tiles, each cut s ways, takes
// ceil(tiles s / 256) rounds of ceil(chunks / s) chunks; the merge of the parts
// adds its launch and what it reads and writes.  The rules below take the s
// with the least of that sum, so a launch whose tiles fill whole rounds stays whole.
// Up to 1024 parts beside the whole tiles are looked at: 192 tiles (3 x 2048 x
// 2048) want 4 ways, three full rounds of a quarter: training against V = 32000
// 2.97 ms whole, 2.47 cut; 320 tiles (5 x 2048) 4.20 and 3.93; 3 x 1024 x 2560 3.40
// and 2.58; ROT of 4 x 2048 x 2048 4.05 and 3.54.  More cuts gain little more.
struct SplitCost {
    double chunk_us;    // one chunk of streamed rows of one workgroup
    double merge_us;    // the merge's launch
    double part_us;     // the parts of one split, written and read once
};

int best_split(long long tiles, long long nch, const SplitCost& c, double max_s, double* us_out = nullptr,
               int limit = solo::kMaxSplit) {
    int best = 1;
    double best_us = (double)((tiles + 255) / 256) * (double)nch * c.chunk_us;
    // (of the s with the same chunks per part the least is best: only those are looked at)
    for (long long per = nch; per > 1;) {
        const long long s = (nch + per - 2) / (per - 1);  // the least s with fewer chunks per part
        if (s > limit || s > max_s || tiles * (s - 1) >= 1024) break;
        per = (nch + s - 1) / s;
        const double us = (double)((tiles * s + 255) / 256) * (double)((nch + s - 1) / s) * c.chunk_us + c.merge_us +
                          s * c.part_us;
        if (us < best_us) {
            best = (int)s;
            best_us = us;
        }
    }
    if (us_out) *us_out = best_us;
    return best;
}

// The local-loss pass over n modules.  Its parts (a row of d fp32 sums and 4
// scalars per token and split) live in an output that the readout-gradient
// pass overwrites later, so only calls that compute one are split, as far as
// its `room` floats hold them.  Time per chunk: the fp32 family's 256 readout
// rows take 4 R d clocks at the fp32 matrix rate, 70% of it reached; a 16-row
// chunk of the bf16 kernels measured 1.15 us at 65536 elements per tile (32 x
// 2048 and 64 x 1024), of which about 0.5 us is the exchange and its barriers.
// (A call whose modules together fill the chip is split only where ROT launches
// them apart, and then has the room to itself; smaller calls share one bound
// whatever they launch apart, so that ROT with R = I cuts alike more often.)
int local_splits(const Plan& P, int n, int K, int T, int d, int V, size_t room) {
    const double td = (double)P.rows * d;
    const bool fused = P.mfma || P.exact;
    const SplitCost c = {fused ? 0.5 + 0.65 * td / 65536.0 : 4.0 * td / 1.6e3, 6.0, (double)n * T * d * 8.0 / 3e6};
    const int yc = fused ? 16 : 256;
    const double rows = (double)T * ((long long)P.ntiles * K >= 256 ? n : K);
    return best_split((long long)P.ntiles * n, ((long long)V + yc - 1) / yc, c, (double)room / (rows * (d + 4)));
}

// Exit evaluation on the matrix-core families runs in one of three forms:
//   FUSED  the fused pass over whole row tiles, streaming tiled readout copies
//          (their writing costs a read and a write of every readout);
//   SPLIT  the fused pass split over the vocabulary, reading the readouts
//          row-major: few rows, memory-bound; the parts (8 scalars per row and
//          split) take the place of the copies;
//   PROD   the tiled product (k_logits.hip): 256 x 256 tiles, so many rows; the
//          copies of bf16(g * h) it multiplies, `pass_rows` rows at a time,
//          and its parts take the place of the readout copies.
// The form with the least estimated time is taken.  Measured: 60 us per tile of
// 256 x 256 of the product at d = 2048, 10 at d = 256 (planes of wide rows, 128 x 256: 100 us at
// d = 3072, 155 at 4096); 1.05 and 1.28 us per chunk of 16
// readout rows of the fused pass at d = 2048 (64 rows per tile) and 1024 (128),
// 0.9 at d = 256 (128).  4 x 8192 x 32000 rows: product against fused pass 2.01
// against 2.55 ms at d = 1024, 0.67 against 1.79 at d = 256.
struct EvalPlan {
    enum Form { FUSED, SPLIT, PROD } form = FUSED;
    int nsplit = 1;
    long long pass_rows = 0;
};

double prod_tile_us(int d, bool planes) { return 4.0 + (planes ? 0.054 : 0.027) * d; }
double prod_eval_tile_us(int d, bool planes) {
    return solo::logits_eval_tile(planes, d) == 128 ? 2.0 + 0.036 * d : prod_tile_us(d, planes);
}
double eval_chunk_us(int rows, int d) { return 0.2 + 0.0055 * rows + 0.45 * (double)rows * d / 131072.0; }

EvalPlan plan_eval(const Plan& P, int K, int T, int d, int V, bool flat) {
    EvalPlan E;
    const int rows = P.wide ? solo::kMfmaWideEvalRows : solo::mfma_eval_rows(d);
    const long long tiles = (long long)K * ((T + rows - 1) / rows);
    const long long stiles = flat ? ((long long)K * T + rows - 1) / rows : tiles;
    const long long nch = ((long long)V + 15) / 16;
    const double chunk = eval_chunk_us(rows, d);
    double best = (double)((tiles + 255) / 256) * (double)nch * chunk +
                  (1 + P.nhead_tiles) * (4.0 + 4.0 * (double)V * d / 4e6);
    // (the fp32 kernels' pass: 32 rows against chunks of 256)
    if (P.planes)
        best = (double)(((long long)K * ((T + 31) / 32) + 255) / 256) * (double)((V + 255) / 256) * (2.0 + 0.08 * d);
    const double kt = (double)K * T;
    const double room = (double)P.eval_room;
    const double row_bytes = P.planes ? 2.0 * solo::plane_pitch(d) : 2.0 * d;
    double us = 0.0;
    // (row-major, a chunk's operand loads take 16 rows of 64 bytes each: 1.75 us at d = 2048)
    const SplitCost c = {1.05 * chunk > 0.00085 * d ? 1.05 * chunk : 0.00085 * d, 10.0, kt * 64.0 / 3e6};
    const int s = best_split(stiles, nch, c, room / (kt * 32.0), &us, solo::kEvalSplits);
    if (!P.planes && s > 1 && us < best) {
        E.form = EvalPlan::SPLIT;
        E.nsplit = s;
        best = us;
    }
    const long long lists = flat ? 1 : K, n = flat ? (long long)K * T : T;  // rows are one list, or one per module
    const int vt = solo::logits_eval_tile(P.planes, d);
    const long long nvt = ((long long)V + vt - 1) / vt;
    // (as in best_split: the least split of each number of tiles per part)
    for (long long per = nvt + 1; per > 1;) {
        const int sp = (int)((nvt + per - 2) / (per - 1));
        if (sp > solo::kEvalSplits) break;
        per = (nvt + sp - 1) / sp;
        // rows whose copies fit next to the parts, and the least number of passes over them
        const double left = room - 512.0 - (sp > 1 ? kt * 32.0 * sp : 0.0);
        const long long cap = left > 0.0 ? (long long)(left / row_bytes) : 0;
        if (cap < (n < 256 ? n : 256)) break;
        const long long np0 = (n + cap - 1) / cap;
        for (long long np = np0; np < np0 + 4; ++np) {
            const long long pr = ((n + np - 1) / np + 255) / 256 * 256;
            if ((pr < n ? pr : n) > cap) continue;
            const long long whole = n / pr, rest = n - whole * pr;
            auto rounds = [&](long long r) { return (double)(((r + 255) / 256 * sp + 255) / 256); };
            const double t = (double)lists * ((whole * rounds(pr) + (rest ? rounds(rest) : 0.0)) *
                                                  (double)((nvt + sp - 1) / sp) * prod_eval_tile_us(d, P.planes) +
                                              (double)(whole + (rest > 0)) * 8.0) +
                             10.0 + kt * d * 4.0 / 4e6 + (sp > 1 ? 5.0 + kt * 64.0 * sp / 3e6 : 0.0);
            if (t < best) {
                best = t;
                E.form = EvalPlan::PROD;
                E.nsplit = sp;
                E.pass_rows = pr;
            }
        }
    }
    return E;
}

// The rows of exit evaluation as one list (one readout, no biases); and the floats that the
// parts of split local-loss passes may use: a readout gradient, written by a later pass.
bool flat_list(const Plan& P, const solo_readout_args& x) { return !P.rot && !x.bias && !(x.Wbar && x.K > 1); }
size_t split_room(const Plan& P, const solo_readout_args& x) {
    return x.final_module_dW || P.rg_hi > P.rg_lo ? (size_t)x.V * x.d : 0;
}

// The bias-gradient pass over n modules as a tiled product (the readout rows
// against all tokens): the splits of its tokens, or 0 where the fused pass is
// estimated faster (few tokens: a tile is 256 of them; a chunk of the fused pass
// measured 1.2 times one of exit evaluation).  Its parts but the last, which
// goes to the output, take the place of the row statistics and losses (3 K T
// floats), which no later stage reads.
int prod_bgrad_splits(const Plan& P, int n, int K, int T, int d, int V) {
    // (outside the bf16 families the fused pass is the fp32 kernels': 32 rows, chunks of 256 tokens)
    const int rows = P.exact ? 32 : (P.wide ? solo::kMfmaWideEvalRows : solo::mfma_eval_rows(d));
    const double chunk = P.exact ? (2.0 + 0.08 * d) / 16.0 : 1.2 * eval_chunk_us(rows, d);
    const double fused = (double)(((((long long)V + rows - 1) / rows) * n + 255) / 256) * (double)((T + 15) / 16) * chunk;
    const SplitCost c = {prod_tile_us(d, P.exact), 4.0 + (P.exact ? (double)n * T * d * 6.0 / 4e6 : 0.0), (double)n * V * 8.0 / 3e6};
    double us = 0.0;
    const int s = best_split((((long long)V + 255) / 256) * n, ((long long)T + 255) / 256, c,
                             1.0 + 3.0 * K * T / ((double)n * V), &us);
    return us < fused ? s : 0;
}

bool aligned(const void* p, uintptr_t a) { return ((uintptr_t)p & (a - 1)) == 0; }
bool aligned_or_null(const void* p, uintptr_t a) { return !p || aligned(p, a); }

int check(const solo_readout_args& a, bool eval, Plan* P) {
    if (a.dtype != SOLO_BF16 && a.dtype != SOLO_F32) return SOLO_ERR_DTYPE;
    if (!shape_ok(a.K, a.T, a.d, a.V)) return SOLO_ERR_SHAPE;
    if (!std::isfinite(a.eps) || a.eps < 0.f) return SOLO_ERR_ARG;
    if (!flag_ok(a.gain_per_module) || !flag_ok(a.readout_per_head) || !flag_ok(a.final_module_dW) ||
        !flag_ok(a.heads_train_readout))
        return SOLO_ERR_ARG;
    if (a.readout_per_head && !a.Wbar) return SOLO_ERR_ARG;
    if (a.heads_train_readout && !a.readout_per_head) return SOLO_ERR_ARG;
    if (a.rot && a.readout_per_head) return SOLO_ERR_ARG;
    if (!a.h || !a.gain || !a.W || !a.targets || !a.losses || !a.workspace) return SOLO_ERR_NULL;
    if (!eval) {
        if (!a.dh) return SOLO_ERR_NULL;
        if (a.final_module_dW && !a.dW) return SOLO_ERR_NULL;
        if (a.heads_train_readout && a.K > 1 && !a.dWbar) return SOLO_ERR_NULL;
        if ((a.gain_per_module || a.final_module_dW) && !a.dgain) return SOLO_ERR_NULL;
    }
    if (!aligned(a.h, 16) || !aligned(a.gain, 16) || !aligned(a.W, 16) || !aligned_or_null(a.Wbar, 16) ||
        !aligned(a.targets, 4) || !aligned(a.losses, 4) || !aligned_or_null(a.row_loss, 4) ||
        !aligned_or_null(a.tau, 4) || !aligned_or_null(a.bias, 4) || !aligned_or_null(a.rot, 16) ||
        !aligned(a.workspace, kAlign))
        return SOLO_ERR_ALIGN;
    if (eval) {
        if (!aligned_or_null(a.top1, 4)) return SOLO_ERR_ALIGN;
    } else {
        if (!aligned(a.dh, 16) || !aligned_or_null(a.dtau, 4) || !aligned_or_null(a.dbias, 4))
            return SOLO_ERR_ALIGN;
        if (a.final_module_dW && !aligned(a.dW, 16)) return SOLO_ERR_ALIGN;
        if (a.heads_train_readout && a.K > 1 && !aligned(a.dWbar, 16)) return SOLO_ERR_ALIGN;
        if ((a.gain_per_module || a.final_module_dW) && !aligned(a.dgain, 4)) return SOLO_ERR_ALIGN;
    }
    if (!make_plan(a, eval, P)) return SOLO_ERR_SHAPE;
    // (a workspace without room for the plane copies still serves: the products
    // then run on the fp32 kernels, which need none)
    if (a.workspace_bytes < P->total && P->planes && !make_plan(a, eval, P, false)) return SOLO_ERR_SHAPE;
    if (a.workspace_bytes < P->total) return SOLO_ERR_WORKSPACE;
    return SOLO_OK;
}

int run(const solo_readout_args& x, bool eval) {
    Plan P;
    const int st = check(x, eval, &P);
    if (st != SOLO_OK) return st;
    const int K = x.K, T = x.T, d = x.d, V = x.V;
    hipStream_t s = (hipStream_t)x.hip_stream;
    char* ws = (char*)x.workspace;

    solo::FusedArgs a = {};
    a.K = K;
    a.T = T;
    a.d = d;
    a.V = V;
    a.m0 = 0;
    a.inv_T = (float)(1.0 / (double)T);
    a.nsplit = 1;
    a.h = x.h;
    a.Wt = x.W;
    // heads: W itself, one shared matrix, or one per head
    a.Wh = x.Wbar ? x.Wbar : x.W;
    a.wh_stride = (x.Wbar && x.readout_per_head) ? (long long)V * d : 0;
    a.Wtt = ws + P.wtile;
    a.Wht = P.nhead_tiles ? ws + P.whtile : ws + P.wtile;
    a.wht_stride = P.nhead_tiles > 1 ? solo::tiled_elems(V, d) : 0;
    a.hg = ws + P.hg;
    a.hg_m0 = P.hg_lo;
    a.gain = x.gain;
    a.g_stride = x.gain_per_module ? d : 0;
    a.tau = x.tau;
    a.bias = x.bias;
    a.targets = x.targets;
    a.rstd = (const float*)(ws + P.rstd);
    a.lse = (float*)(ws + P.lse);
    a.rowloss = x.row_loss ? x.row_loss : (float*)(ws + P.rowloss);
    a.rowrec = (!eval && (P.rg_hi > P.rg_lo || P.bg_hi > P.bg_lo)) ? (float*)(ws + P.rowrec) : nullptr;
    a.rowdtau = (!eval && x.dtau) ? (float*)(ws + P.rowdtau) : nullptr;
    a.top1 = eval ? x.top1 : nullptr;
    a.dh = eval ? nullptr : x.dh;
    a.dgain_part = P.slots ? (float*)(ws + P.dgp) : nullptr;
    a.dg_mode = eval ? 0 : P.dg_mode;
    a.dWt = (!eval && x.final_module_dW) ? x.dW : nullptr;
    a.dWh = (!eval && x.heads_train_readout) ? x.dWbar : nullptr;
    a.dbias = eval ? nullptr : x.dbias;

    auto mark = [&](int stage) -> bool {
        if (!x.stage_events || !x.stage_events[stage]) return true;
        return hipEventRecord((hipEvent_t)x.stage_events[stage], s) == hipSuccess;
    };
    const int dt = x.dtype;
    // a failure left pending by earlier work on this thread is not this call's
    (void)hipGetLastError();
    if (solo::launch_row_rstd(dt, x.h, (float*)(ws + P.rstd), (long long)K * T, d, x.eps, s) != hipSuccess)
        return SOLO_ERR_HIP;
    // exit evaluation of few rows: split over the vocabulary, no tiled copies
    const bool flat = eval && flat_list(P, x);
    const EvalPlan E = eval && (P.mfma || P.planes) ? plan_eval(P, K, T, d, V, flat) : EvalPlan();
    a.split_stat = (float*)(ws + P.wtile);
    a.part_rows = (long long)K * T;
    if (E.form == EvalPlan::SPLIT) {
        a.nsplit = E.nsplit;
        a.flat = flat;
    }
    if (tiled_readout(P) && E.form == EvalPlan::FUSED) {
        if (solo::launch_tile((const solo::bf16*)x.W, 0, nullptr, 0, (solo::bf16*)(ws + P.wtile), 1, V, d, s) !=
            hipSuccess)
            return SOLO_ERR_HIP;
        if (P.nhead_tiles && solo::launch_tile((const solo::bf16*)x.Wbar, (long long)V * d, nullptr, 0,
                                               (solo::bf16*)(ws + P.whtile), P.nhead_tiles, V, d, s) != hipSuccess)
            return SOLO_ERR_HIP;
    }
    // ROT heads: their stationary rows are u = R_k (g_k * h) (gain one from
    // then on), which the passes of the heads read in place of h
    solo::FusedArgs ah = a;
    if (P.rot) {
        if (solo::launch_fill_one(dt, ws + P.ones, d, s) != hipSuccess) return SOLO_ERR_HIP;
        if (solo::launch_rot_rows(dt, x.h, x.gain, a.g_stride, x.rot, ws + P.ubuf, K - 1, T, d, s) != hipSuccess)
            return SOLO_ERR_HIP;
        ah.h = ws + P.ubuf;
        ah.gain = ws + P.ones;
        ah.g_stride = 0;
        ah.ebuf = eval ? nullptr : (void*)(ws + P.ebuf);
    }
    if (!mark(0)) return SOLO_ERR_HIP;
    // scratch of split local-loss passes
    float* const room = eval ? nullptr : (x.final_module_dW ? x.dW : (P.rg_hi > P.rg_lo ? x.dWbar : nullptr));
    const size_t room_floats = eval ? 0 : split_room(P, x);
    // one launch over modules [m0, m0 + n) of a pass, with the arguments g
    auto pass = [&](int which, const solo::FusedArgs& g, int m0, int n) -> hipError_t {
        if (n <= 0) return hipSuccess;
        solo::FusedArgs b = g;
        b.m0 = m0;
        if (which == 1) {
            b.nsplit = local_splits(P, n, K, T, d, V, room_floats);
            if (b.nsplit > 1) {
                b.part_rows = (long long)n * T;
                b.split_acc = room - (long long)m0 * T * d;
                b.split_stat = room + b.nsplit * b.part_rows * d - 4LL * m0 * T;
            }
        }
        switch (which) {
            case 0:
                return P.wide   ? solo::launch_exit_eval_mfma_wide(b, n, s)
                       : P.mfma ? solo::launch_exit_eval_mfma(b, n, s)
                                : solo::launch_exit_eval_f32(dt, b, n, s);
            case 1: {
                const hipError_t e = P.wide    ? solo::launch_local_loss_mfma_wide(b, P.ext, n, s)
                                     : P.mfma  ? solo::launch_local_loss_mfma(b, P.ext, n, s)
                                     : P.xwide ? solo::launch_local_loss_exact_wide(b, P.ext, n, s)
                                     : P.exact ? solo::launch_local_loss_exact(b, P.ext, n, s)
                                               : solo::launch_local_loss_f32(dt, b, n, s);
                if (e != hipSuccess || b.nsplit == 1) return e;
                return solo::launch_merge(dt, P.mfma ? solo::MERGE_BF16 : (P.exact ? solo::MERGE_EXACT : solo::MERGE_F32),
                                          b, n, P.dg_rows, s);
            }
            case 2:
                return P.wide    ? solo::launch_readout_grad_mfma_wide(b, n, s)
                       : P.mfma  ? solo::launch_readout_grad_mfma(b, n, s)
                       : P.xwide ? solo::launch_readout_grad_exact_wide(b, n, s)
                       : P.exact ? solo::launch_readout_grad_exact(b, n, s)
                                 : solo::launch_readout_grad_f32(dt, b, n, s);
            default:
                return P.wide   ? solo::launch_bias_grad_mfma_wide(b, n, s)
                       : P.mfma ? solo::launch_bias_grad_mfma(b, n, s)
                                : solo::launch_bias_grad_f32(dt, b, n, s);
        }
    };
    // modules [lo, hi) of a pass: under ROT the heads and the terminal are two launches
    auto pass_range = [&](int which, int lo, int hi) -> bool {
        if (!P.rot || hi <= K - 1 || lo >= K - 1) return pass(which, P.rot && lo < K - 1 ? ah : a, lo, hi - lo) == hipSuccess;
        return pass(which, ah, lo, K - 1 - lo) == hipSuccess && pass(which, a, K - 1, hi - K + 1) == hipSuccess;
    };
    // exit evaluation as a tiled product over the rows of all modules, or of one at a time
    auto prod_eval = [&]() -> bool {
        const long long n = flat ? (long long)K * T : T;
        const size_t parts = E.nsplit > 1 ? align_up((size_t)K * T * 32 * E.nsplit) : 0;
        solo::bf16* const copy = (solo::bf16*)(ws + P.wtile + parts);
        for (int k = 0; k < (flat ? 1 : K); ++k) {
            const solo::FusedArgs& g = P.rot && k < K - 1 ? ah : a;
            solo::LogitsArgs l = {};
            l.Y = (const solo::bf16*)(flat || k == K - 1 ? a.Wt : (const void*)((const solo::bf16*)a.Wh + k * a.wh_stride));
            l.nY = V;
            l.d = d;
            l.exact = P.planes;
            l.x_last = -1;
            l.nsplit = E.nsplit;
            l.parts = a.split_stat;
            l.part_rows = (long long)K * T;
            l.bias = x.bias ? x.bias + (long long)k * V : nullptr;
            l.T = T;
            l.rstd = a.rstd;
            l.tau = a.tau;
            l.targets = a.targets;
            l.rowloss = a.rowloss;
            l.top1 = a.top1;
            for (long long r0 = 0; r0 < n; r0 += E.pass_rows) {
                const long long nr = n - r0 < E.pass_rows ? n - r0 : E.pass_rows;
                l.row0 = (flat ? 0 : (long long)k * T) + r0;
                l.nX = (int)nr;
                // the rows' products with their modules' gains
                const solo::bf16* const src = (const solo::bf16*)g.h + l.row0 * d;
                const solo::bf16* const gn = (const solo::bf16*)g.gain;
                if ((P.planes ? solo::launch_gain_planes(src, gn, g.g_stride, copy, nr, l.row0, T, d, s)
                              : solo::launch_gain_list(src, gn, g.g_stride, copy, nr, l.row0, T, d, s)) != hipSuccess)
                    return false;
                l.X = copy;
                if (solo::launch_logits_eval(l, s) != hipSuccess) return false;
            }
        }
        return true;
    };
    if (E.form == EvalPlan::PROD ? !prod_eval() : !pass_range(eval ? 0 : 1, 0, K)) return SOLO_ERR_HIP;
    if (E.nsplit > 1) {
        a.nsplit = E.nsplit;
        if (solo::launch_merge_eval(a, !P.mfma, (long long)K * T, s) != hipSuccess) return SOLO_ERR_HIP;
        a.nsplit = 1;
    }
    if (P.rot && !eval) {
        // back to the basis of h: D = e R_k = e (R_k^T)^T, then the heads' RMSNorm
        // backward (and their gain partials when every module trains its gain)
        if (solo::launch_transpose(dt, x.rot, ws + P.rtr, K - 1, d, s) != hipSuccess ||
            solo::launch_rot_back(dt, P.mfma, ws + P.ebuf, ws + P.rtr, (float*)(ws + P.dbuf), K - 1, T, d, s) !=
                hipSuccess ||
            solo::launch_rot_post(dt, (const float*)(ws + P.dbuf), x.h, x.gain, a.g_stride, (const float*)(ws + P.rstd),
                                  x.tau, x.dh, P.dg_mode == 2 ? a.dgain_part : nullptr, K - 1, T, d, P.dg_rows,
                                  s) != hipSuccess)
            return SOLO_ERR_HIP;
    }
    if (!mark(1)) return SOLO_ERR_HIP;
    if (solo::launch_module_sum(a.rowloss, x.losses, K, T, 1.0 / (double)T, s) != hipSuccess) return SOLO_ERR_HIP;
    if (a.rowdtau && solo::launch_module_sum(a.rowdtau, x.dtau, K, T, 1.0, s) != hipSuccess) return SOLO_ERR_HIP;
    if (!mark(2)) return SOLO_ERR_HIP;
    // the gain-scaled copies of h the gradient passes stream, module m at
    // hg + (m - hg_lo) tiled_elems(T, d): tiled for the register-fed passes,
    // row-major for the direct-to-LDS readout-gradient pass
    // (ROT heads: of their rotated rows, times the gain of ones)
    auto copies = [&](const solo::FusedArgs& g, int lo, int hi, bool as_tiles) -> bool {
        if (hi <= lo) return true;
        const solo::bf16* src = (const solo::bf16*)g.h + (long long)lo * T * d;
        const solo::bf16* gn = (const solo::bf16*)g.gain + (long long)lo * g.g_stride;
        solo::bf16* dst = (solo::bf16*)(ws + P.hg) + (long long)(lo - P.hg_lo) * solo::tiled_elems(T, d);
        return (as_tiles ? solo::launch_tile(src, (long long)T * d, gn, g.g_stride, dst, hi - lo, T, d, s)
                         : solo::launch_gain_rows(src, (long long)T * d, gn, g.g_stride, dst,
                                                  solo::tiled_elems(T, d), hi - lo, T, d, s)) == hipSuccess;
    };
    auto gain_copies = [&](int lo, int hi, bool as_tiles) -> bool {
        if (!P.rot || hi <= K - 1 || lo >= K - 1) return copies(P.rot && lo < K - 1 ? ah : a, lo, hi, as_tiles);
        return copies(ah, lo, K - 1, as_tiles) && copies(a, K - 1, hi, as_tiles);
    };
    const int nbg = P.bg_hi - P.bg_lo;
    const int bsplit = !eval && (P.mfma || P.planes) && nbg > 0 ? prod_bgrad_splits(P, nbg, K, T, d, V) : 0;
    if (!eval && P.mfma &&
        (!gain_copies(P.rg_lo, P.rg_hi, tiled_rgrad(P)) || !gain_copies(P.bg_lo, P.bg_hi, bsplit == 0)))
        return SOLO_ERR_HIP;
    if (P.exact && bsplit > 0) {
        // (under ROT the heads' rotated rows and the terminal's own are two lists)
        for (int m = P.bg_lo; m < P.bg_hi;) {
            const int end = P.rot && m < K - 1 && P.bg_hi == K ? K - 1 : P.bg_hi;
            const solo::FusedArgs& g = P.rot && m < K - 1 ? ah : a;
            if (solo::launch_gain_planes((const solo::bf16*)g.h + (long long)m * T * d, (const solo::bf16*)g.gain, g.g_stride,
                                         (solo::bf16*)(ws + P.hg) + (long long)(m - P.bg_lo) * T * solo::plane_pitch(d),
                                         (long long)(end - m) * T, (long long)m * T, T, d, s) != hipSuccess)
                return SOLO_ERR_HIP;
            m = end;
        }
    }
    if (!eval && !pass_range(2, P.rg_lo, P.rg_hi)) return SOLO_ERR_HIP;
    if (!mark(3)) return SOLO_ERR_HIP;
    auto prod_bgrad = [&]() -> bool {
        const int lo = P.bg_lo;
        const solo::bf16* const heads = (const solo::bf16*)a.Wh;
        const solo::bf16* const term = (const solo::bf16*)a.Wt;
        solo::LogitsArgs l = {};
        l.X = lo < K - 1 ? heads + lo * a.wh_stride : term;
        l.x_stride = lo < K - 1 ? a.wh_stride : 0;
        l.x_last = lo < K - 1 && P.bg_hi == K ? K - 1 - lo : -1;
        l.x_last_off = ((intptr_t)term - (intptr_t)(heads + (K - 1) * a.wh_stride)) / 2;
        l.exact = P.exact;
        l.y_stride = P.exact ? (long long)T * solo::plane_pitch(d) : solo::tiled_elems(T, d);
        l.Y = (const solo::bf16*)a.hg + (P.exact ? 0 : (lo - P.hg_lo) * l.y_stride);
        l.nX = V;
        l.nY = T;
        l.d = d;
        l.nsplit = bsplit;
        l.parts = (float*)(ws + P.rstd);
        l.bias = x.bias ? x.bias + (long long)lo * V : nullptr;
        l.rowrec = a.rowrec + 4LL * lo * T;
        l.out = x.dbias + (long long)lo * V;
        l.inv_T = a.inv_T;
        return solo::launch_logits_bgrad(l, nbg, s) == hipSuccess;
    };
    if (!eval && (bsplit > 0 ? !prod_bgrad() : !pass_range(3, P.bg_lo, P.bg_hi))) return SOLO_ERR_HIP;
    if (!mark(4)) return SOLO_ERR_HIP;
    if (!eval && P.slots) {
        if (solo::launch_dgain_reduce(a.dgain_part, x.dgain, P.slots, (T + P.dg_rows - 1) / P.dg_rows, d, s) != hipSuccess)
            return SOLO_ERR_HIP;
    }
    if (!mark(5)) return SOLO_ERR_HIP;
    return SOLO_OK;
}

solo_readout_args headline(int K, int T, int d, int V, int dtype, float eps, const void* h, const void* gain,
                           const void* W, const int32_t* targets, int final_module_dW, float* losses,
                           float* row_loss, void* dh, float* dW, float* dgain, void* workspace,
                           size_t workspace_bytes, void* hip_stream, void* const* stage_events) {
    solo_readout_args a = {};
    a.K = K;
    a.T = T;
    a.d = d;
    a.V = V;
    a.dtype = dtype;
    a.eps = eps;
    a.h = h;
    a.gain = gain;
    a.W = W;
    a.targets = targets;
    a.final_module_dW = final_module_dW;
    a.losses = losses;
    a.row_loss = row_loss;
    a.dh = dh;
    a.dW = dW;
    a.dgain = dgain;
    a.workspace = workspace;
    a.workspace_bytes = workspace_bytes;
    a.hip_stream = hip_stream;
    a.stage_events = stage_events;
    return a;
}

// Scratch of the entry point that allocates nothing: a file-scope device
// array, one copy per GPU, held until the process ends.  Host code never
// passes the array's name to a kernel (on the host it is a stand-in, not a
// device address): the device address is fetched once per device, with that
// device current, and kept.
constexpr size_t kScratchBytes = size_t(128) << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex scratch_mu;
void* scratch_ptr[kMaxDevices] = {};

// The current device's scratch address (nullptr on a HIP error).
void* scratch_of_current_device() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(scratch_mu);
    if (!scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
        scratch_ptr[dev] = ptr;
    }
    return scratch_ptr[dev];
}

}  // namespace

extern "C" {

size_t solo_readout_scratch_limit(void) { return kScratchBytes; }

int solo_readout_fwd_bwd_noalloc(int K, int T, int d, int V, int dtype, float eps, const void* h, const void* gain,
                                 const void* W, const int32_t* targets, int final_module_dW, float* losses,
                                 float* row_loss, void* dh, float* dW, float* dgain, void* hip_stream) {
    if (dtype != SOLO_BF16 && dtype != SOLO_F32) return SOLO_ERR_DTYPE;
    if (!shape_ok(K, T, d, V)) return SOLO_ERR_SHAPE;
    solo_readout_args a = headline(K, T, d, V, dtype, eps, h, gain, W, targets, final_module_dW, losses, row_loss,
                                   dh, dW, dgain, nullptr, 0, hip_stream, nullptr);
    Plan P;
    if (!make_plan(a, false, &P)) return SOLO_ERR_SHAPE;
    if (P.total > kScratchBytes) return SOLO_ERR_WORKSPACE;
    // every other host check before the first HIP call (a stand-in, aligned
    // workspace of the limit's size: only the scratch's address is unknown yet)
    a.workspace = (void*)(uintptr_t)kAlign;
    a.workspace_bytes = kScratchBytes;
    const int st = check(a, false, &P);
    if (st != SOLO_OK) return st;
    (void)hipGetLastError();
    void* ws = scratch_of_current_device();
    if (!ws) return SOLO_ERR_HIP;
    a.workspace = ws;
    a.workspace_bytes = kScratchBytes;
    return run(a, false);
}

int solo_readout_abi_version(void) { return SOLO_READOUT_ABI_VERSION; }

const char* solo_status_string(int status) {
    switch (status) {
        case SOLO_OK: return "ok";
        case SOLO_ERR_NULL: return "a required pointer is NULL";
        case SOLO_ERR_SHAPE: return "invalid sizes (need K,T,V >= 1, 8 <= d <= 4096, d % 8 == 0, K <= 65535, K*T < 2^31)";
        case SOLO_ERR_DTYPE: return "unknown dtype";
        case SOLO_ERR_ALIGN: return "misaligned pointer";
        case SOLO_ERR_WORKSPACE: return "workspace too small";
        case SOLO_ERR_ARG:
            return "invalid argument (eps must be finite and >= 0; flags must be 0 or 1; readout_per_head needs "
                   "Wbar; heads_train_readout needs readout_per_head; rot excludes readout_per_head)";
        case SOLO_ERR_HIP: return "HIP launch failed";
        default: return "unknown status";
    }
}

size_t solo_readout_workspace_size(int K, int T, int d, int V, int dtype, int final_module_dW) {
    const solo_readout_args a = headline(K, T, d, V, dtype, 0.f, nullptr, nullptr, nullptr, nullptr, final_module_dW,
                                         nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, 0, nullptr, nullptr);
    Plan P;
    return make_plan(a, false, &P) ? P.total : 0;
}

const char* solo_readout_kernel_family(int K, int T, int d, int V, int dtype) {
    if ((dtype != SOLO_BF16 && dtype != SOLO_F32) || !shape_ok(K, T, d, V)) return "invalid";
    if (solo::mfma_wide_supported(dtype, d)) return "mfma_wide";
    return solo::mfma_supported(dtype, d) ? "mfma" : "valu";
}

int solo_readout_fwd_bwd(int K, int T, int d, int V, int dtype, float eps, const void* h, const void* gain,
                         const void* W, const int32_t* targets, int final_module_dW, float* losses, float* row_loss,
                         void* dh, float* dW, float* dgain, void* workspace, size_t workspace_bytes,
                         void* hip_stream) {
    return solo_readout_fwd_bwd_profiled(K, T, d, V, dtype, eps, h, gain, W, targets, final_module_dW, losses,
                                         row_loss, dh, dW, dgain, workspace, workspace_bytes, hip_stream, nullptr);
}

int solo_readout_fwd_bwd_profiled(int K, int T, int d, int V, int dtype, float eps, const void* h, const void* gain,
                                  const void* W, const int32_t* targets, int final_module_dW, float* losses,
                                  float* row_loss, void* dh, float* dW, float* dgain, void* workspace,
                                  size_t workspace_bytes, void* hip_stream, void* const* stage_events) {
    if (dtype != SOLO_BF16 && dtype != SOLO_F32) return SOLO_ERR_DTYPE;
    if (!shape_ok(K, T, d, V)) return SOLO_ERR_SHAPE;
    const solo_readout_args a = headline(K, T, d, V, dtype, eps, h, gain, W, targets, final_module_dW, losses,
                                         row_loss, dh, dW, dgain, workspace, workspace_bytes, hip_stream,
                                         stage_events);
    return run(a, false);
}

size_t solo_readout_general_workspace_size(const solo_readout_args* args) {
    Plan P;
    return (args && make_plan(*args, false, &P)) ? P.total : 0;
}

int solo_readout_general(const solo_readout_args* args) {
    if (!args) return SOLO_ERR_NULL;
    return run(*args, false);
}

size_t solo_readout_exit_eval_workspace_size(const solo_readout_args* args) {
    Plan P;
    return (args && make_plan(*args, true, &P)) ? P.total : 0;
}

int solo_readout_exit_eval(const solo_readout_args* args) {
    if (!args) return SOLO_ERR_NULL;
    return run(*args, true);
}

// Which forms a call of these sizes, flags and workspace_bytes runs in, for the tests that are about
// one of them (host only; not in the public header).  Exit evaluation: route[0] the form of
// EvalPlan, route[1] its splits, route[2] the rows of one pass of the product.  Training: route[0]
// the splits of the local-loss pass (under ROT the heads'), route[1] the terminal's, route[2] the
// splits of the bias gradient's product (0: the fused pass).  SOLO_OK, or the status of such a call's sizes.
__attribute__((visibility("default"))) int solo_readout_route(const solo_readout_args* args, int exit_eval,
                                                             long long* route) {
    if (!args || !route) return SOLO_ERR_NULL;
    const solo_readout_args& x = *args;
    Plan P;
    if (!make_plan(x, exit_eval != 0, &P)) return SOLO_ERR_SHAPE;
    if (x.workspace_bytes < P.total && P.planes && !make_plan(x, exit_eval != 0, &P, false)) return SOLO_ERR_SHAPE;
    if (x.workspace_bytes < P.total) return SOLO_ERR_WORKSPACE;
    if (exit_eval) {
        const EvalPlan E = P.mfma || P.planes ? plan_eval(P, x.K, x.T, x.d, x.V, flat_list(P, x)) : EvalPlan();
        route[0] = E.form;
        route[1] = E.nsplit;
        route[2] = E.pass_rows;
        return SOLO_OK;
    }
    const size_t room = split_room(P, x);
    const int nbg = P.bg_hi - P.bg_lo;
    route[0] = local_splits(P, P.rot ? x.K - 1 : x.K, x.K, x.T, x.d, x.V, room);
    route[1] = P.rot ? local_splits(P, 1, x.K, x.T, x.d, x.V, room) : route[0];
    route[2] = (P.mfma || P.planes) && nbg > 0 ? prod_bgrad_splits(P, nbg, x.K, x.T, x.d, x.V) : 0;
    return SOLO_OK;
}

}  // extern "C"
