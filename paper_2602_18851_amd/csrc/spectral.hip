// C ABI of the per-head spectral-norm estimator and the per-layer FP8 E4M3
// scale factor for MI355X (gfx950): validation, workspace plan, context and
// the entry points of include/spectral.h.  The kernels live in gram_heads.hip
// (most calls of two or more iterations), sweeps.hip (the others), gram.hip
// (the tolerance-mode tail of the sweeps), layer_form.hip
// (spectral_step_layer) and logits_fp8.hip (spectral_logits_fp8).
//
// Method (arXiv 2602.18851, Sec. 4.1-4.2, App. E): for query head h with key
// head j = floor(h / g), one step is
//     z = K_j v,  u' = Q_h^T z (= M v),  sigma = ||u'||,
//     y = Q_h u' / sigma,  v' = K_j^T y (= M^T u),  v = v' / ||v'||,
// where Q_h, K_j are the d_h x d row blocks of the PyTorch-layout weights
// (the transposes of the paper's W^Q_h, W^K_j) and M = Q_h^T K_j is never
// formed.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "kernels.h"
#include "logits_fp8.h"
#include "spectral.h"

namespace {

using namespace sn;

thread_local std::string g_err;

int fail(int code, const std::string& msg) {
  g_err = msg;
  return code;
}

#define SN_HIP(expr)                                                                  \
  do {                                                                                \
    hipError_t e_ = (expr);                                                           \
    if (e_ != hipSuccess)                                                             \
      return fail(SN_EHIP, std::string(#expr) + " failed: " + hipGetErrorString(e_)); \
  } while (0)

enum {
  KIND_INIT = 0, KIND_Q = 1, KIND_K = 2, KIND_FIN = 3, KIND_GRAM = 4, KIND_ITER = 5, KIND_EMIT = 6,
  KIND_LROWS = 7, KIND_LCOLS = 8, KIND_LRED = 9, KIND_PROJ = 10, KIND_LOGITS = 11, KIND_TAIL = 12, KIND_N = 13
};
static_assert(KIND_N == SN_PROFILE_KINDS, "profile kinds");

// ------------------------------------------------------------------ host side

struct Plan {
  int H, g, gc, nch, vec, tile_c, n_tiles;   // W_K sweeps
  int tile_cq, n_tiles_q;                    // W_Q sweep
  bool mfma_k;  // W_K sweeps on the matrix cores
  int s_q, tps_q, s_k, tps_k;
  bool tail;    // tolerance mode on the sweeps: the heads still running after the first
                // steps are finished in d_h-space (needs d_h >= 16)
  int s_tmax;   // most strips of the tail's final W_K sweep
  int n_tiles_g;
  int g_items;  // Gram partial items of the tail
  bool layer;   // layer-level form
  int s_lq, tps_lq, s_lk, tps_lk;  // strips of the layer-form row sweeps over W_Q and W_K
  int rs_q, rbp_q, rs_k, rbp_k;    // row splits (and row blocks per split) of its column sweeps
  size_t off_zp, off_zn, off_yp, off_yn, off_sig, off_vn, off_alive, off_iters, off_fin, off_gp;
  bool fused;      // its one-pass sweeps apply
  int lf_layers, lf_ldq;                    // layers per chunk, row length of the group sums (grouped heads)
  int lf_sq, lf_tq, lf_sk, lf_tk;           // strips and tiles per strip over W_Q (or the group sums) and W_K
  size_t off_lsum, off_lx, off_lpart, off_lnp;
  size_t off_lz, off_ly, off_lvin, off_lcol, off_lu, off_lv, off_ln2, off_ln2p, off_lstat;
  size_t off_zs, off_lg, off_lk, off_kvpos, off_ctl, off_zt;
  bool heads;   // calls of two or more iterations may run the Gram form with one workgroup per head
  int h_units;  // key heads of one launch pair
  int h_sk, h_tps_k, h_sq, h_tps_q;  // column strips of their key and query matrices (h_sq 0: not split)
  size_t off_hfin, off_gk, off_gq, off_hz, off_hn;
  size_t bytes;
};

int esize(int dtype) { return dtype == SN_F32 ? 4 : 2; }

bool supported_dh(int dh) { return dh == 8 || dh == 16 || dh == 32 || dh == 64 || dh == 128; }

int validate(const sn_shape* s, const sn_params* p) {
  if (!s || !p) return fail(SN_ENULL, "shape and params must not be NULL");
  if (s->dtype != SN_F32 && s->dtype != SN_BF16) return fail(SN_EDTYPE, "dtype must be SN_F32 or SN_BF16");
  if (s->n_layers < 1 || s->d_model < 1 || s->n_q_heads < 1 || s->n_kv_heads < 1 || s->head_dim < 1)
    return fail(SN_EINVAL, "n_layers, d_model, n_q_heads, n_kv_heads and head_dim must be >= 1");
  if (s->n_q_heads % s->n_kv_heads != 0) return fail(SN_EINVAL, "n_kv_heads must divide n_q_heads");
  if (!supported_dh(s->head_dim)) return fail(SN_EINVAL, "head_dim must be one of 8, 16, 32, 64, 128");
  const int64_t ld = s->ld == 0 ? s->d_model : s->ld;
  if (ld < s->d_model) return fail(SN_EINVAL, "ld must be >= d_model");
  if ((ld * esize(s->dtype)) % 16 != 0) return fail(SN_EINVAL, "ld * element size must be a multiple of 16 bytes");
  const int64_t H = (int64_t)s->n_layers * s->n_q_heads;
  if (H * (int64_t)s->d_model > (int64_t(1) << 40) || H > (1 << 26))
    return fail(SN_EINVAL, "shape too large");
  if (!(p->alpha > 0.f) || !(p->eta_fp8 > 0.f) || !(p->r_max > 0.f) || !std::isfinite(p->alpha) ||
      !std::isfinite(p->eta_fp8) || !std::isfinite(p->r_max))
    return fail(SN_EINVAL, "alpha, eta_fp8 and r_max must be finite and > 0");
  if (!(p->tol >= 0.f) || !std::isfinite(p->tol)) return fail(SN_EINVAL, "tol must be finite and >= 0");
  if (p->q_strips < 0 || p->k_strips < 0) return fail(SN_EINVAL, "strip counts must be >= 0");
  if (p->flags & ~(SN_FLAG_VALU_K_SWEEP | SN_FLAG_GRAM | SN_FLAG_LAYER)) return fail(SN_EINVAL, "unknown flag bits");
  if ((p->flags & SN_FLAG_GRAM) && s->head_dim < 16) return fail(SN_EINVAL, "the Gram form needs head_dim >= 16");
  if ((int64_t)s->head_dim * ld * esize(s->dtype) >= (int64_t(1) << 31))
    return fail(SN_EINVAL, "head_dim * ld * element size must be below 2^31 bytes");
  return SN_OK;
}

int ceil_div(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

// Row stride of the layer form's per-unit column sums: whole 64-column tiles.
int col_stride(int d) { return ceil_div(d, 64) * 64; }

// Column strips per unit (head or KV head): the request if given, else about
// target / units (rounded up, or down when all waves should be resident at
// once), with at least kMinTilesPerStrip tiles per strip so that a wave's
// stream outweighs its prologue (which sums one partial per producer strip).
void strips(int n_tiles, int64_t units, int requested, int target, bool round_down, int* s_out, int* tps_out,
            int min_tiles = kMinTilesPerStrip) {
  const int64_t u = std::max<int64_t>(units, 1);
  int s = requested > 0 ? requested : round_down ? (int)std::max<int64_t>(1, target / u) : ceil_div(target, u);
  if (requested <= 0) s = std::min(s, std::max(1, n_tiles / min_tiles));
  s = std::max(1, std::min(s, n_tiles));
  const int tps = ceil_div(n_tiles, s);
  *tps_out = tps;
  *s_out = ceil_div(n_tiles, tps);
}

// Bytes the group sums of the layer form may take: a chunk of layers at a
// time (29 layers of the 70B GQA shape).  Smaller chunks, whose sums stay in the
// Infinity Cache, lose to their launches: that shape, five iterations 5.92 ms,
// chunks of 512, 256, 128 MiB 5.99, 6.50, 8.22 ms.
constexpr int64_t kGroupSumBytes = int64_t(1) << 30;

// The one-pass sweeps of the layer form: the rows of a layer after grouping
// have to fit the registers of one workgroup.  Strips: the fewest rounds of
// workgroups over the chip, each round costing its tiles and about half a tile
// of set-up.
void plan_fused(const sn_shape* s, Plan& pl) {
  const int dh = s->head_dim, rows = s->n_kv_heads * dh, es = esize(s->dtype), d = s->d_model;
  const int64_t ld = s->ld == 0 ? d : s->ld;
  pl.lf_ldq = ceil_div(d, 32) * 32;
  const int64_t layer = (int64_t)rows * pl.lf_ldq * 4;
  pl.fused = (int64_t)s->n_kv_heads * dh <= kLFRows && kLFRowsPerWave * std::max<int64_t>(ld * es, pl.lf_ldq * 4) < (int64_t(1) << 31) &&
             (pl.g == 1 || layer <= kGroupSumBytes);
  if (!pl.fused) return;
  pl.lf_layers = s->n_layers;
  if (pl.g > 1) {
    const int chunks = ceil_div(s->n_layers, std::max<int64_t>(1, kGroupSumBytes / layer));
    pl.lf_layers = ceil_div(s->n_layers, chunks);
  }
  const int slots = 256 * std::max(1, kLFWaves / ceil_div(rows, kLFRowsPerWave));
  auto best = [&](int tiles, int* strips_out, int* tps_out) {
    double cost = 1e30;
    for (int tps = 1; tps <= std::min(tiles, 4096); ++tps) {
      const int st = ceil_div(tiles, tps);
      const double c = (double)ceil_div((int64_t)pl.lf_layers * st, slots) * (tps + 0.5);
      if (c < cost) {
        cost = c;
        *strips_out = st;
        *tps_out = tps;
      }
    }
  };
  best(ceil_div((int64_t)d * (pl.g > 1 ? 4 : es), 128), &pl.lf_sq, &pl.lf_tq);
  best(ceil_div((int64_t)d * es, 128), &pl.lf_sk, &pl.lf_tk);
}

// Whether a layer-form call runs them: with grouped heads where forming and
// reading the fp32 group sums (4 / (g es) of W_Q's bytes) moves less than
// reading W_Q twice per iteration.
bool fused_call(const Plan& pl, int dtype, int n_iter) {
  if (!pl.fused) return false;
  if (pl.g == 1) return true;
  const double r = 4.0 / (pl.g * esize(dtype));
  return 1.0 + r * (1 + n_iter) < 2.0 * n_iter;
}

// Bytes of Gram matrices one launch pair of the one-workgroup-per-head form
// works on: half the Infinity Cache, from which every query head of a group reads
// them.  Larger shapes go through in several pairs, whose last rounds of
// workgroups leave the chip idle in turn: the 70B GQA shape (94 MB) as one pair
// 2.48 ms, as two 2.61 ms.
constexpr size_t kGkBytes = size_t(128) << 20;
constexpr int kSplitHeads = 256;     // below this many heads their query matrices are split over workgroups
constexpr int kSplitTarget = 384;    // ... into about this many (with kSplitKeys for the key heads)
constexpr int kSplitKeys = 256;
constexpr int kSplitTargetLow = 640;  // d_h <= 64: four workgroups per compute unit
constexpr int kSplitKeysLow = 384;

// Column strips of the key heads where every query head has a workgroup of its
// own: the fewest rounds of workgroups over the chip (`slots` at a time),
// against the strips' Gram matrices, which every query head reads: in units of
// streaming one head, rounds(s) / s + (query rounds) s (matrix / head bytes).
// 70B GQA shape, 640 key heads on 512 slots: one strip takes two rounds, two
// strips one and a half (the call 2.51 -> 2.48 ms).
int key_strips(int64_t units, int64_t heads, int slots, double mat_ratio, int tiles) {
  int best = 1;
  double cost = 1e30;
  for (int s = 1; s <= std::min(32, std::max(1, tiles / kMinTilesPerStrip)); ++s) {
    const double c = (double)ceil_div(units * s, slots) / s + (double)ceil_div(heads, slots) * s * mat_ratio;
    if (c < cost) {
      cost = c;
      best = s;
    }
  }
  return best;
}

// The one-workgroup-per-head form: column strips, and its buffers, which
// share the bytes of the sweeps' partials, sweep0 .. *off (a call uses one or
// the other), and go past their end where those are smaller.
// `slack`: they may add at most that many bytes to the workspace (kAnySlack: as
// many as kGkBytes allows).  The results do not depend on it, only how many key
// heads a launch pair covers: the strips and a head's order of summation are
// the same for any slack, and whether the form runs at all is make_plan's.
constexpr int64_t kAnySlack = INT64_MAX, kNoHeads = -1;

void plan_heads(const sn_shape* s, Plan& pl, size_t sweep0, int64_t slack, size_t* off) {
  const size_t H = pl.H, dh = s->head_dim, g = pl.g, n_units = (size_t)s->n_layers * s->n_kv_heads;
  const int tiles = ceil_div((int64_t)s->d_model * esize(s->dtype), 128);
  const bool split = pl.H < kSplitHeads;
  pl.h_sq = pl.h_sk = 1;
  pl.h_tps_q = pl.h_tps_k = tiles;
  const int split_q = dh <= 64 ? kSplitTargetLow : kSplitTarget, split_k = dh <= 64 ? kSplitKeysLow : kSplitKeys;
  if (split) strips(tiles, pl.H, 0, split_q, true, &pl.h_sq, &pl.h_tps_q);
  const size_t mat = (dh / 16) * (dh / 16 + 1) / 2 * 2048;  // doubles
  if (split) {
    strips(tiles, n_units, 0, split_k, true, &pl.h_sk, &pl.h_tps_k);
  } else if (g > 1) {
    const int64_t chunks = ceil_div(g, heads_per_operand(s->dtype == SN_BF16, pl.mfma_k, (int)g));
    const double ratio = (double)mat / ((double)dh * s->d_model * esize(s->dtype));
    const int want = key_strips(n_units * chunks, pl.H, dh <= 64 ? 1024 : 512, ratio, tiles);
    strips(tiles, n_units, want, 0, true, &pl.h_sk, &pl.h_tps_k);
  }
  if (!split) pl.h_sq = 0;
  const size_t fin = (H * 2 * dh * 4 + 255) & ~size_t(255);
  const size_t per_unit = split || g > 1 ? (pl.h_sk + g * pl.h_sq) * mat + g * pl.h_sk * (dh + 1) * 4 : 0;
  const size_t room = *off - sweep0;  // >= fin: the sweeps keep three or more d_h-vectors per head
  size_t most = std::max(kGkBytes, room - fin);
  if (slack != kAnySlack) most = std::min(most, room - fin + (size_t)slack);
  pl.h_units = per_unit ? (int)std::min(n_units, (most - std::min<size_t>(most, 1024)) / per_unit) : (int)n_units;
  pl.heads = pl.h_units > 0;
  if (pl.heads) pl.h_units = ceil_div(n_units, ceil_div(n_units, pl.h_units));  // pairs of equal length
  size_t o = sweep0;
  auto take = [&](size_t bytes) {
    const size_t r = o;
    o += (bytes + 255) & ~size_t(255);
    return r;
  };
  pl.off_hfin = take(fin);
  if (per_unit) {
    const size_t u = pl.h_units;
    pl.off_gk = take(u * pl.h_sk * mat);
    pl.off_gq = take(u * g * pl.h_sq * mat);
    pl.off_hz = take(u * g * pl.h_sk * dh * 4);
    pl.off_hn = take(u * g * pl.h_sk * 4);
  }
  *off = std::max(*off, o);
}

// Calls with tol > 0 and n_iter > 2 that run the one-workgroup-per-head form
// (`heads`: the plan has it).
bool heads_tolerance(const sn_shape* s, const sn_params* p, bool heads) {
  if (!heads) return false;
  if (p->flags & SN_FLAG_GRAM) return true;
  if (p->q_strips > 0 || p->k_strips > 0 || (p->flags & SN_FLAG_VALU_K_SWEEP)) return false;
  // A stop at step 2, the earliest, costs the sweeps five passes over the
  // weights and a tail for the heads still running.  Warm calls that stop
  // there for nearly every head, sweeps and tail against here: 12 GB of
  // weights (70B GQA shape) 4.18 -> 2.34 ms, 0.5 GB 387 -> 188 us, 151 MB
  // 230 -> 126 us; but 40, 32, 4.5 and 0.6 MiB 118 -> 84, 113 -> 78, 100 -> 47 and 75 ->
  // 40 us too (cold calls of up to 90 steps 256 -> 222, 175 -> 149, 175 -> 131, 159 ->
  // 124 us).  The line is not where the two meet, which they do not: it is where
  // calls stopped changing their route, and smaller ones have kept the tail.
  const int64_t bytes =
      (int64_t)s->n_layers * (s->n_q_heads + s->n_kv_heads) * s->head_dim * s->d_model * esize(s->dtype);
  return bytes >= (int64_t(64) << 20);
}

// The plan with at most `slack` bytes for the one-workgroup-per-head form
// beside the sweeps' (see plan_heads; kNoHeads: without it).  `sums`: the layer
// form may keep the sums of grouped query rows.
Plan plan_with(const sn_shape* s, const sn_params* p, int64_t slack, bool sums = true) {
  Plan pl{};
  const int dh = s->head_dim;
  pl.H = s->n_layers * s->n_q_heads;
  pl.g = s->n_q_heads / s->n_kv_heads;
  pl.gc = 1;
  while (pl.gc < pl.g && pl.gc < kMaxGC) pl.gc *= 2;
  pl.nch = ceil_div(pl.g, pl.gc);
  pl.vec = 16 / esize(s->dtype);
  pl.mfma_k = s->dtype == SN_BF16 && (dh == 64 || dh == 128) && pl.gc >= 4 &&
              !(p->flags & SN_FLAG_VALU_K_SWEEP);
  // the MFMA W_K sweep tiles 64 columns, the vector sweeps 8 chunks of 16 bytes;
  // both sweeps of a plan share one tile width (so one strip split)
  pl.tile_c = pl.mfma_k ? kMTileC : kCPL * pl.vec;
  pl.n_tiles = ceil_div(s->d_model, pl.tile_c);
  pl.tile_cq = kCPL * pl.vec;
  pl.n_tiles_q = ceil_div(s->d_model, pl.tile_cq);
  strips(pl.n_tiles_q, pl.H, p->q_strips, kQTargetItems, false, &pl.s_q, &pl.tps_q);
  strips(pl.n_tiles, (int64_t)s->n_layers * s->n_kv_heads * pl.nch, p->k_strips,
         pl.mfma_k ? kKMfmaResident : kKTargetItems, pl.mfma_k, &pl.s_k, &pl.tps_k);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off += (bytes + 255) & ~size_t(255);
    return o;
  };
  const size_t H = pl.H;
  pl.off_zn = take(2 * H * pl.s_k * 4);
  pl.off_yn = take(H * pl.s_q * 4);
  pl.off_sig = take(2 * H * 4);
  pl.off_vn = take(H * 4);
  pl.off_alive = take(2 * H * 4);
  pl.off_iters = take(H * 4);
  // the z and y partials of the sweeps
  const size_t sweep0 = off;
  pl.off_zp = take(2 * H * pl.s_k * dh * 4);
  pl.off_yp = take(H * pl.s_q * dh * 4);
  if (dh >= 16 && slack != kNoHeads) plan_heads(s, pl, sweep0, slack, &off);
  // Tolerance mode on the sweeps: after the first kTailSteps steps, the heads
  // still running are listed on the device and finished in d_h-space through
  // their Gram matrices, formed for the listed heads only; strips of those
  // launches are chosen on the device for the listed count (at most max(count,
  // target) items each).
  pl.tail = p->tol > 0.f && dh >= 16 && !(p->flags & SN_FLAG_GRAM) && !heads_tolerance(s, p, pl.heads);
  if (pl.tail) {
    const size_t nkvh = (size_t)s->n_layers * s->n_kv_heads;
    pl.s_tmax = std::max(1, pl.n_tiles / kTailMinTiles);
    pl.n_tiles_g = ceil_div((int64_t)s->d_model * esize(s->dtype), 128);
    pl.g_items = std::max<int>(H + nkvh, kGTargetItems);
    pl.off_zs = take(H * 4);
    pl.off_lg = take((H + nkvh) * 4);
    pl.off_lk = take(nkvh * pl.nch * 4);
    pl.off_kvpos = take(nkvh * 4);
    pl.off_ctl = take(TC_WORDS * 4);
    pl.off_zt = take(H * pl.s_tmax * 4);
    pl.off_fin = take(H * 2 * dh * 4);
    pl.off_gp = take((size_t)pl.g_items * (dh / 16) * (dh / 16 + 1) / 2 * 256 * 4);
  }
  pl.layer = (p->flags & SN_FLAG_LAYER) != 0;
  if (pl.layer) {
    const size_t L = s->n_layers, Hk = L * s->n_kv_heads, d = s->d_model;
    strips(pl.n_tiles_q, pl.H, 0, kQTargetItems, false, &pl.s_lq, &pl.tps_lq);
    strips(pl.n_tiles_q, (int64_t)Hk, 0, kQTargetItems, false, &pl.s_lk, &pl.tps_lk);
    pl.off_lz = take(Hk * pl.s_lk * dh * 4);
    pl.off_ly = take(H * pl.s_lq * dh * 4);
    // column sweeps: one wave per column tile and row split; rows are split
    // only as far as needed for about kQTargetItems waves
    auto rsplit = [&](int nrb, int* n_split, int* per) {
      const int64_t base = (int64_t)L * pl.n_tiles_q;
      const int want = (int)std::min<int64_t>(nrb, std::max<int64_t>(1, (kQTargetItems + base - 1) / base));
      *per = ceil_div(nrb, want);
      *n_split = ceil_div(nrb, *per);
    };
    rsplit(s->n_q_heads, &pl.rs_q, &pl.rbp_q);
    rsplit(s->n_kv_heads, &pl.rs_k, &pl.rbp_k);
    pl.off_lvin = take(H * dh * 4);
    pl.off_lcol = take(L * (size_t)std::max(pl.rs_q, pl.rs_k) * col_stride(s->d_model) * 4);
    pl.off_lu = take(L * d * 4);
    pl.off_lv = take(L * d * 4);
    pl.off_ln2 = take(3 * L * 4);
    pl.off_ln2p = take(L * (size_t)ceil_div(d, kRedThreads) * 4);
    pl.off_lstat = take(L * 4);
    if (sums || pl.g == 1) plan_fused(s, pl);
    if (pl.fused) {
      const size_t rows = (size_t)s->n_kv_heads * dh, c = pl.lf_layers, smax = std::max(pl.lf_sq, pl.lf_sk);
      if (pl.g > 1) pl.off_lsum = take(c * rows * pl.lf_ldq * 4);
      pl.off_lx = take(L * rows * 4);
      pl.off_lpart = take(c * smax * rows * 4);
      pl.off_lnp = take(c * smax * 4);
    }
  }
  pl.bytes = off;
  return pl;
}

// The static scratch of spectral_step_noalloc, and what its pointer table takes.
constexpr size_t kScratchBytes = size_t(32) << 20;
size_t table_bytes(int layers) { return ((size_t)4 * layers * sizeof(void*) + 255) & ~size_t(255); }

// The plan of a call without a context: the sweeps' workspace has to fit the
// scratch (else *need says what it takes), the rest is the heads form's.
bool plan_scratch(const sn_shape* s, const sn_params* p, Plan* pl, size_t* need) {
  sn_params q = *p;
  q.flags &= ~SN_FLAG_LAYER;  // only reserves space for spectral_step_layer
  *need = table_bytes(s->n_layers) + plan_with(s, &q, kNoHeads).bytes;
  if (*need > kScratchBytes) return false;
  *pl = plan_with(s, &q, (int64_t)(kScratchBytes - *need));
  return true;
}

// The plan of a context.  A shape whose sweeps fit the scratch while the
// matrices of even one key head do not go beside them runs the sweeps in both
// calls, which give the same bits.
Plan make_plan(const sn_shape* s, const sn_params* p, bool sums = true) {
  Plan tight{};
  size_t need = 0;
  const bool sweeps = s->head_dim >= 16 && plan_scratch(s, p, &tight, &need) && !tight.heads;
  return plan_with(s, p, sweeps ? kNoHeads : kAnySlack, sums);
}

struct ProfRec {
  int kind;
  hipEvent_t a, b;
};

// Device pointer tables are written by a kernel whose arguments carry the
// pointers: the values are taken when the launch is queued (or captured),
// with no host buffer that must outlive the call.
constexpr int kTabChunk = 256;
struct TabFill {
  const void* p[kTabChunk];
  const void** dst;
  int32_t n;
};

__global__ void table_fill_kernel(TabFill f) {
  const int i = threadIdx.x;
  if (i < f.n) f.dst[i] = f.p[i];
}

// dst[0 .. n) = src(0 .. n), in launches of up to kTabChunk pointers.
template <typename Src>
int fill_table(const void** dst, int n, Src src, hipStream_t st) {
  for (int i0 = 0; i0 < n; i0 += kTabChunk) {
    TabFill f{};
    f.dst = dst + i0;
    f.n = std::min(kTabChunk, n - i0);
    for (int i = 0; i < f.n; ++i) f.p[i] = src(i0 + i);
    table_fill_kernel<<<dim3(1), kTabChunk, 0, st>>>(f);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(SN_EHIP, std::string("table fill launch failed: ") + hipGetErrorString(e));
  }
  return SN_OK;
}

}  // namespace

// Shared with the host-side calibration helpers (calibration.cpp).
void sn_set_last_error(const char* msg) { g_err = msg; }

struct sn_ctx {
  sn_shape shape;
  sn_params params;
  Plan plan;
  hipStream_t stream = nullptr;
  int device = 0;
  char* ws = nullptr;
  bool owns_ws = true;
  Work w{};
  const void** d_tab = nullptr;  // device [2][2L]: the eager table, then the table of captured calls
  const void** tab = nullptr;    // the table the current call's launches read
  bool cache_table = true;       // eager calls skip the table write when the pointers did not change
  std::vector<const void*> cached;  // pointers in the eager table
  hipEvent_t tab_event = nullptr;
  bool prof = false;
  std::vector<ProfRec> recs;
  std::vector<hipEvent_t> pool;
};

namespace {

hipEvent_t take_event(sn_ctx* c) {
  if (!c->pool.empty()) {
    hipEvent_t e = c->pool.back();
    c->pool.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}


// Brackets one launch with profiling events when profiling is on.
template <typename F>
int timed(sn_ctx* c, int kind, F&& launch) {
  ProfRec rec{kind, nullptr, nullptr};
  if (c->prof) {
    rec.a = take_event(c);
    rec.b = take_event(c);
    if (!rec.a || !rec.b) return fail(SN_EHIP, "hipEventCreate failed");
    SN_HIP(hipEventRecord(rec.a, c->stream));
  }
  launch();
  SN_HIP(hipGetLastError());
  if (c->prof) {
    SN_HIP(hipEventRecord(rec.b, c->stream));
    c->recs.push_back(rec);
  }
  return SN_OK;
}

// Compacted launch of the tolerance-mode tail over the entries of `list`
// (query heads for a W_Q sweep, W_K units otherwise); the count and strips
// are read from `ctl` on the device, and the grid holds max_items items.
struct TailLaunch {
  const int32_t* list = nullptr;
  const int32_t* ctl = nullptr;
  int max_items = 0;
};

int run_sweep(sn_ctx* c, int ph, SweepArgs a, const TailLaunch& tl = TailLaunch{}) {
  a.ctl = tl.ctl;
  const Plan& pl = c->plan;
  const int n_units = c->shape.n_layers * c->shape.n_kv_heads * pl.nch;
  if (ph == PH_Q || ph == PH_EQ) {
    a.mats = c->tab;
    a.s_out = pl.s_q;
    a.tps = pl.tps_q;
    a.n_tiles = pl.n_tiles_q;
    a.n_items = pl.H * pl.s_q;
  } else {
    a.mats = c->tab + c->shape.n_layers;
    a.s_out = pl.s_k;
    a.tps = pl.tps_k;
    a.n_tiles = pl.n_tiles;
    a.n_items = n_units * pl.s_k;
  }
  if (tl.list) {
    a.list = tl.list;
    a.n_items = tl.max_items;
  }
  const int kind = ph == PH_INIT ? KIND_INIT : ph == PH_Q ? KIND_Q : ph == PH_K ? KIND_K : KIND_EMIT;
  return timed(c, kind, [&] {
    launch_sweep(c->shape.dtype == SN_BF16, c->shape.head_dim, ph, pl.gc, pl.mfma_k, a.n_items, c->stream, a);
  });
}


// Eq. "scale" per unit of sigma: alpha * d / sqrt(d_h) / (eta_fp8 * r_max), in double.
float scale_coef(const sn_ctx* c) {
  return (float)((double)c->params.alpha * (double)c->shape.d_model /
                 (std::sqrt((double)c->shape.head_dim) * (double)c->params.eta_fp8 * (double)c->params.r_max));
}

bool capturing(hipStream_t st) {
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  return hipStreamIsCapturing(st, &cap) == hipSuccess && cap != hipStreamCaptureStatusNone;
}

// Checks the layer pointers and the device, and points the call's launches
// at a device table of the per-layer pointers.  Eager calls share one table,
// rewritten only when the pointers change.  A call being captured into a
// graph always writes its pointers into a second table, so that every replay
// restores its own pointers whatever eager calls ran in between (graphs
// captured from one context must therefore not replay concurrently).
int update_table(sn_ctx* c, const void* const* wq_layers, const void* const* wk_layers) {
  const int L = c->shape.n_layers;
  for (int l = 0; l < L; ++l) {
    if (!wq_layers[l] || !wk_layers[l]) return fail(SN_ENULL, "a layer weight pointer is NULL");
    if ((reinterpret_cast<uintptr_t>(wq_layers[l]) | reinterpret_cast<uintptr_t>(wk_layers[l])) & 15)
      return fail(SN_EINVAL, "layer weight pointers must be 16-byte aligned");
  }
  int cur_dev = 0;
  SN_HIP(hipGetDevice(&cur_dev));
  if (cur_dev != c->device) return fail(SN_ESTATE, "the current HIP device is not the context's device");
  auto src = [&](int i) { return i < L ? wq_layers[i] : wk_layers[i - L]; };
  if (capturing(c->stream)) {
    c->tab = c->d_tab + 2 * L;
    return fill_table(c->tab, 2 * L, src, c->stream);
  }
  c->tab = c->d_tab;
  if (!c->cache_table) return fill_table(c->tab, 2 * L, src, c->stream);
  bool same = c->cached.size() == (size_t)(2 * L);
  for (int l = 0; same && l < L; ++l)
    same = c->cached[l] == wq_layers[l] && c->cached[L + l] == wk_layers[l];
  if (!same) {
    int rc = fill_table(c->tab, 2 * L, src, c->stream);
    if (rc != SN_OK) return rc;
    c->cached.assign(wq_layers, wq_layers + L);
    c->cached.insert(c->cached.end(), wk_layers, wk_layers + L);
    if (c->tab_event) SN_HIP(hipEventRecord(c->tab_event, c->stream));
  }
  return SN_OK;
}


// One layer-form sweep over W_Q (q = true) or W_K.
int layer_sweep(sn_ctx* c, bool q, int mode, LayerArgs a) {
  const Plan& pl = c->plan;
  const int L = c->shape.n_layers;
  a.mats = c->tab + (q ? 0 : L);
  a.ld = c->shape.ld;
  a.d = c->shape.d_model;
  a.n_tiles = pl.n_tiles_q;
  a.lstat = reinterpret_cast<const int32_t*>(c->ws + pl.off_lstat);
  if (mode == LM_ROWS) {
    a.units = q ? c->shape.n_q_heads : c->shape.n_kv_heads;
    a.s_out = q ? pl.s_lq : pl.s_lk;
    a.tps = q ? pl.tps_lq : pl.tps_lk;
    a.n_items = L * a.units * a.s_out;
  } else {
    a.nrb = q ? c->shape.n_q_heads : c->shape.n_kv_heads;
    a.n_rsplit = q ? pl.rs_q : pl.rs_k;
    a.rb_per = q ? pl.rbp_q : pl.rbp_k;
    a.cstride = col_stride(c->shape.d_model);
    a.n_items = L * a.n_rsplit * a.n_tiles;
  }
  return timed(c, mode == LM_ROWS ? KIND_LROWS : KIND_LCOLS, [&] {
    launch_layer_sweep(c->shape.dtype == SN_BF16, c->shape.head_dim, mode, a.n_items, c->stream, a);
  });
}

// vin of a column sweep from the previous row sweep's partials.
int layer_vin(sn_ctx* c, const float* part, int src_units, int strips, int div, int cnt, int nrb) {
  const Plan& pl = c->plan;
  LayerVinArgs v{};
  v.part = part;
  v.src_units = src_units;
  v.strips = strips;
  v.div = div;
  v.cnt = cnt;
  v.nrb = nrb;
  v.dh = c->shape.head_dim;
  v.lstat = reinterpret_cast<const int32_t*>(c->ws + pl.off_lstat);
  v.vin = reinterpret_cast<float*>(c->ws + pl.off_lvin);
  return timed(c, KIND_LRED, [&] { launch_layer_vin(c->shape.n_layers, c->stream, v); });
}

int layer_reduce(sn_ctx* c, const float* col, int units, int cstride, int mode, float* vec, float* n2) {
  const Plan& pl = c->plan;
  LayerReduceArgs r{};
  r.col = col;
  r.units = units;
  r.d = c->shape.d_model;
  r.cstride = cstride;
  r.mode = mode;
  r.vec = vec;
  r.n2 = n2;
  r.nb = ceil_div(c->shape.d_model, kRedThreads);
  r.n2part = reinterpret_cast<float*>(c->ws + pl.off_ln2p);
  r.n2_start = reinterpret_cast<float*>(c->ws + pl.off_ln2) + 2 * c->shape.n_layers;
  r.lstat = reinterpret_cast<int32_t*>(c->ws + pl.off_lstat);
  return timed(c, KIND_LRED,
               [&] { launch_layer_reduce(c->shape.n_layers, c->stream, r); });
}

// One layer-form call with one-pass sweeps: per chunk of layers the group
// sums, the first W_K sweep, then per iteration a sweep over the sums (g = 1:
// W_Q) and one over W_K, each followed by the gather of its row sums.
int run_layer_fused(sn_ctx* c, const float* v, bool want_u, int n_iter, float* lu, float* lv, float* n2) {
  const Plan& pl = c->plan;
  const sn_shape& sh = c->shape;
  const int L = sh.n_layers, rows = sh.n_kv_heads * sh.head_dim;
  const bool bf16 = sh.dtype == SN_BF16;
  float* sums = pl.g > 1 ? reinterpret_cast<float*>(c->ws + pl.off_lsum) : nullptr;
  LayerFusedArgs k{};
  k.mats = c->tab + L;
  k.ld = sh.ld;
  k.d = sh.d_model;
  k.n_tiles = ceil_div((int64_t)sh.d_model * esize(sh.dtype), 128);
  k.rows = rows;
  k.strips = pl.lf_sk;
  k.tps = pl.lf_tk;
  k.v = v;
  k.x = reinterpret_cast<float*>(c->ws + pl.off_lx);
  k.part = reinterpret_cast<float*>(c->ws + pl.off_lpart);
  k.n2part = reinterpret_cast<float*>(c->ws + pl.off_lnp);
  k.n2_start = n2 + 2 * L;
  k.lstat = reinterpret_cast<int32_t*>(c->ws + pl.off_lstat);
  LayerFusedArgs q = k;
  q.mats = c->tab;
  q.strips = pl.lf_sq;
  q.tps = pl.lf_tq;
  if (sums) {
    q.mats = nullptr;
    q.dense = sums;
    q.ld = pl.lf_ldq;
    q.n_tiles = ceil_div(sh.d_model, 32);
  }
  q.mode = 1;
  q.n2 = n2;
  k.n2 = n2 + L;
  int rc;
  for (int l0 = 0; l0 < L; l0 += pl.lf_layers) {
    const int nl = std::min(pl.lf_layers, L - l0);
    q.layer0 = k.layer0 = l0;
    auto sweep = [&](bool is_q, bool init, const LayerFusedArgs& a) {
      int e = timed(c, is_q ? KIND_LCOLS : KIND_LROWS,
                    [&] { launch_layer_fused(is_q && sums ? false : bf16, init, nl, c->stream, a); });
      if (e != SN_OK) return e;
      return timed(c, KIND_LRED, [&] { launch_layer_gather(nl, c->stream, a); });
    };
    if (sums) {
      GroupSumArgs g{c->tab, sh.ld, sh.d_model, rows, sh.head_dim, pl.g, l0, pl.lf_ldq, sums};
      if ((rc = timed(c, KIND_LRED, [&] { launch_group_sum(bf16, nl, c->stream, g); })) != SN_OK) return rc;
    }
    k.mode = 0;
    k.vec = nullptr;
    if ((rc = sweep(false, true, k)) != SN_OK) return rc;
    k.mode = 2;
    for (int i = 1; i <= n_iter; ++i) {
      q.vec = i == n_iter && want_u ? lu : nullptr;
      k.vec = i == n_iter ? lv : nullptr;
      if ((rc = sweep(true, false, q)) != SN_OK) return rc;
      if ((rc = sweep(false, false, k)) != SN_OK) return rc;
    }
  }
  return SN_OK;
}

int layer_finalize(sn_ctx* c, float* v, float* u, float* sigma, float* scale, const float* lu, const float* lv,
                   const float* n2_u) {
  const int L = c->shape.n_layers;
  LayerFinArgs f{};
  f.d = c->shape.d_model;
  f.L = L;
  f.coef = scale_coef(c);
  f.lstat = reinterpret_cast<const int32_t*>(c->ws + c->plan.off_lstat);
  f.lu = lu;
  f.lv = lv;
  f.n2_u = n2_u;
  f.n2_v = n2_u + L;
  f.n2_start = n2_u + 2 * L;
  f.v = v;
  f.u = u;
  f.sigma = sigma;
  f.scale = scale;
  return timed(c, KIND_LRED, [&] { launch_layer_finalize(L, c->stream, f); });
}

GramArgs gram_args(const sn_ctx* c) {
  const Plan& pl = c->plan;
  GramArgs g{};
  g.mats = c->tab;
  g.ld = c->shape.ld;
  g.d = c->shape.d_model;
  g.L = c->shape.n_layers;
  g.n_q = c->shape.n_q_heads;
  g.n_kv = c->shape.n_kv_heads;
  g.H = pl.H;
  g.n_tiles = pl.n_tiles_g;
  g.gp = reinterpret_cast<float*>(c->ws + pl.off_gp);
  return g;
}

IterArgs iter_args(const sn_ctx* c, const SweepArgs& a) {
  const Plan& pl = c->plan;
  IterArgs it{};
  it.H = pl.H;
  it.n_q = c->shape.n_q_heads;
  it.n_kv = c->shape.n_kv_heads;
  it.g = pl.g;
  it.s_k = pl.s_k;
  it.n_iter = a.n_iter;
  it.tol = a.tol;
  it.gp = reinterpret_cast<const float*>(c->ws + pl.off_gp);
  it.w = c->w;
  it.sigma = a.sigma;
  it.iters = a.iters;
  return it;
}

// Tolerance-mode tail after step k0 of the chain, as a fixed sequence of
// launches whatever the heads do: list the heads still running (and their
// key heads and W_K units), form the Gram matrices of the listed heads only,
// iterate each listed head in d_h-space to the tolerance or the cap, then map
// its last vectors back to v (and u) with final sweeps over the lists.  The
// iterates are those the sweep chain would compute (see gram.hip); nothing is
// read back to the host.
int run_tail(sn_ctx* c, SweepArgs a, float* u, int k0) {
  const Plan& pl = c->plan;
  const int n_units = c->shape.n_layers * c->shape.n_kv_heads * pl.nch;
  const int target_k = pl.mfma_k ? kKMfmaResident : kKTargetItems;
  TailPlan tp{pl.n_tiles_g, pl.n_tiles, pl.n_tiles_q, kGTargetItems, target_k, kQTargetItems};
  int rc = timed(c, KIND_TAIL, [&] { launch_tail_lists(a, k0 & 1, pl.gc, n_units, tp, c->stream); });
  if (rc != SN_OK) return rc;

  GramArgs g = gram_args(c);
  g.list = c->w.list_g;
  g.ctl = c->w.ctl;
  const int dh = c->shape.head_dim;
  rc = timed(c, KIND_GRAM, [&] {  // grid: at most max(listed units, target) items
    launch_gram(c->shape.dtype == SN_BF16, dh, pl.g_items, c->stream, g);
  });
  if (rc != SN_OK) return rc;

  IterArgs it = iter_args(c, a);
  it.k0 = k0;
  it.list = c->w.list_g;
  it.ctl = c->w.ctl;
  it.kvpos = c->w.kvpos;
  rc = timed(c, KIND_ITER, [&] { launch_gram_iterate(dh, pl.H, c->stream, it); });
  if (rc != SN_OK) return rc;

  SweepArgs e = a;
  e.k = 0;
  e.only = c->w.alive + (size_t)(k0 & 1) * pl.H;  // the heads running after step k0
  e.w.zn = c->w.zt;
  TailLaunch tk{c->w.list_k, c->w.ctl + TC_EK, std::max(n_units, target_k)};
  if ((rc = run_sweep(c, PH_EK, e, tk)) != SN_OK) return rc;
  if (u) {
    TailLaunch tq{c->w.list_g, c->w.ctl + TC_EQ, std::max(pl.H, kQTargetItems)};
    if ((rc = run_sweep(c, PH_EQ, e, tq)) != SN_OK) return rc;
  }
  return SN_OK;
}

// The sweeps: first W_K sweep, then n_iter x (W_Q sweep,
// W_K sweep).  In tolerance mode every W_K sweep decides, per head, whether
// the step's sigma meets the rule; a stopped head's waves leave at set-up in
// the later sweeps.  With d_h >= 16 only the first kTailSteps steps run as
// full sweeps and the tail finishes the rest (run_tail).  Nothing waits on
// the host.
int run_chain(sn_ctx* c, SweepArgs a, float* u) {
  const Plan& pl = c->plan;
  int rc;
  a.k = 0;
  if ((rc = run_sweep(c, PH_INIT, a)) != SN_OK) return rc;
  const int k_full = pl.tail ? std::min(a.n_iter, kTailSteps) : a.n_iter;
  for (int k = 1; k <= k_full; ++k) {
    a.k = k;
    a.want_vec = (u != nullptr) && (c->params.tol > 0.f || k == a.n_iter);
    if ((rc = run_sweep(c, PH_Q, a)) != SN_OK) return rc;
    a.want_vec = 0;
    if ((rc = run_sweep(c, PH_K, a)) != SN_OK) return rc;
  }
  if (pl.tail && a.n_iter > k_full) return run_tail(c, a, u, k_full);
  return SN_OK;
}

// Whether a call runs the Gram form with one workgroup per head: where it was
// asked for, and for two or more iterations of a fixed count (it reads W_K
// twice and W_Q once; the sweeps read each once per iteration, and W_K once
// more).  At one iteration both read the same and the sweeps need no Gram
// products (70B GQA shape 2.24 ms).  Two iterations, sweeps against here: 70B
// 4.0 -> 2.34 ms, Llama-2-7B 908 -> 680 us, GPT-2 XL 240 -> 178 us, one layer of
// 64 heads (8 key heads), d 8192 252 -> 152 us, of 8 heads 129 -> 130 us, GPT-2 small 74 -> 75
// us; three iterations there 173 -> 130 and 89 -> 77 us.
// Strip counts and SN_FLAG_VALU_K_SWEEP are the sweeps' own parameters.
bool heads_call(const sn_ctx* c, int n_iter) {
  const Plan& pl = c->plan;
  const sn_params& p = c->params;
  if (!pl.heads) return false;
  if (p.flags & SN_FLAG_GRAM) return true;
  if (p.q_strips > 0 || p.k_strips > 0 || (p.flags & SN_FLAG_VALU_K_SWEEP)) return false;
  if (p.tol > 0.f) return n_iter > kTailSteps && heads_tolerance(&c->shape, &p, true);
  return n_iter >= 2;
}

// The Gram form with one workgroup per head (gram_heads.hip), then the final
// sweeps, which write unit vectors: they find z / sigma, and y with its factor
// 1 / ||v'||.
int run_heads(sn_ctx* c, SweepArgs a, float* u) {
  const Plan& pl = c->plan;
  const int n_units = c->shape.n_layers * c->shape.n_kv_heads, dh = c->shape.head_dim;
  a.w.fin = reinterpret_cast<float*>(c->ws + pl.off_hfin);
  HeadArgs h{};
  h.mats = c->tab;
  h.ld = c->shape.ld;
  h.d = c->shape.d_model;
  h.L = c->shape.n_layers;
  h.n_q = c->shape.n_q_heads;
  h.n_kv = c->shape.n_kv_heads;
  h.g = pl.g;
  h.n_iter = a.n_iter;
  h.tol = a.tol;
  h.v = a.v;
  h.round_y = pl.mfma_k;
  h.sk = pl.h_sk;
  h.tps_k = pl.h_tps_k;
  h.sq = pl.h_sq;
  h.tps_q = pl.h_tps_q;
  h.gk = reinterpret_cast<double*>(c->ws + pl.off_gk);
  h.gq = reinterpret_cast<double*>(c->ws + pl.off_gq);
  h.zp = reinterpret_cast<float*>(c->ws + pl.off_hz);
  h.zn = reinterpret_cast<float*>(c->ws + pl.off_hn);
  h.w = a.w;
  h.sigma = a.sigma;
  h.iters = a.iters;
  int rc;
  for (h.unit0 = 0; h.unit0 < n_units; h.unit0 += pl.h_units) {
    h.units = std::min(pl.h_units, n_units - h.unit0);
    h.head0 = h.unit0 * pl.g;
    const bool bf16 = c->shape.dtype == SN_BF16;
    if (pl.g > 1 || h.sq > 0) {
      rc = timed(c, KIND_GRAM, [&] { launch_heads(bf16, dh, true, c->stream, h); });
      if (rc != SN_OK) return rc;
    }
    rc = timed(c, KIND_ITER, [&] { launch_heads(bf16, dh, false, c->stream, h); });
    if (rc != SN_OK) return rc;
  }
  a.k = 0;
  if (h.round_y) a.vscale = a.w.sig;
  if ((rc = run_sweep(c, PH_EK, a)) != SN_OK) return rc;
  if (u && (rc = run_sweep(c, PH_EQ, a)) != SN_OK) return rc;
  return SN_OK;
}

// Views of the workspace of a plan.
void bind_workspace(sn_ctx* c) {
  const Plan& pl = c->plan;
  char* ws = c->ws;
  c->w = Work{};
  c->w.zp = reinterpret_cast<float*>(ws + pl.off_zp);
  c->w.zn = reinterpret_cast<float*>(ws + pl.off_zn);
  c->w.yp = reinterpret_cast<float*>(ws + pl.off_yp);
  c->w.yn = reinterpret_cast<float*>(ws + pl.off_yn);
  c->w.sig = reinterpret_cast<float*>(ws + pl.off_sig);
  c->w.vnorm0 = reinterpret_cast<float*>(ws + pl.off_vn);
  c->w.alive = reinterpret_cast<int32_t*>(ws + pl.off_alive);
  c->w.iters = reinterpret_cast<int32_t*>(ws + pl.off_iters);
  if (pl.tail) c->w.fin = reinterpret_cast<float*>(ws + pl.off_fin);
  if (pl.tail) {
    c->w.zs = reinterpret_cast<int32_t*>(ws + pl.off_zs);
    c->w.list_g = reinterpret_cast<int32_t*>(ws + pl.off_lg);
    c->w.list_k = reinterpret_cast<int32_t*>(ws + pl.off_lk);
    c->w.kvpos = reinterpret_cast<int32_t*>(ws + pl.off_kvpos);
    c->w.ctl = reinterpret_cast<int32_t*>(ws + pl.off_ctl);
    c->w.zt = reinterpret_cast<float*>(ws + pl.off_zt);
  }
}

// One spectral_step call on a bound context (table already in place).
int step_body(sn_ctx* c, float* v, float* u, int32_t n_iter, float* sigma, float* scale, int32_t* iters) {
  const Plan& pl = c->plan;
  const int L = c->shape.n_layers;
  SweepArgs a{};
  a.ld = c->shape.ld;
  a.d = c->shape.d_model;
  a.n_q = c->shape.n_q_heads;
  a.n_kv = c->shape.n_kv_heads;
  a.g = pl.g;
  a.H = pl.H;
  a.s_q = pl.s_q;
  a.s_k = pl.s_k;
  a.n_tiles = pl.n_tiles;
  a.nch = pl.nch;
  a.n_iter = n_iter;
  a.tol = c->params.tol;
  a.w = c->w;
  a.v = v;
  a.u = u;
  a.sigma = sigma;
  a.iters = iters ? iters : c->w.iters;

  const bool heads = heads_call(c, n_iter);
  int rc = heads ? run_heads(c, a, u) : run_chain(c, a, u);
  if (rc != SN_OK) return rc;

  const bool tail_ran = pl.tail && !heads && n_iter > kTailSteps;
  FinArgs f{};
  f.H = pl.H;
  f.L = L;
  f.n_q = c->shape.n_q_heads;
  f.d = c->shape.d_model;
  f.s_k = pl.s_k;
  f.zs = pl.tail ? c->w.zs : nullptr;
  f.tail = tail_ran ? c->w.alive + (size_t)(kTailSteps & 1) * pl.H : nullptr;
  f.zt = c->w.zt;
  f.coef = scale_coef(c);
  f.w = c->w;
  f.v = v;
  f.u = u;
  f.sigma = sigma;
  f.scale = scale;
  f.iters = a.iters;
  return timed(c, KIND_FIN, [&] {
    if (heads)
      launch_heads_finalize(L, c->stream, f);
    else
      launch_finalize(pl.H + L, c->stream, f);
  });
}

}  // namespace

extern "C" {

SN_API const char* spectral_last_error(void) { return g_err.c_str(); }

SN_API int spectral_workspace_bytes(const sn_shape* shape, const sn_params* params, int64_t* bytes) {
  if (!bytes) return fail(SN_ENULL, "bytes must not be NULL");
  const int rc = validate(shape, params);
  if (rc != SN_OK) return rc;
  *bytes = (int64_t)make_plan(shape, params).bytes;
  return SN_OK;
}

SN_API int spectral_init(sn_ctx** ctx, const sn_shape* shape, const sn_params* params, void* hip_stream) {
  if (!ctx) return fail(SN_ENULL, "ctx must not be NULL");
  *ctx = nullptr;
  const int rc = validate(shape, params);
  if (rc != SN_OK) return rc;
  sn_ctx* c = new sn_ctx();
  c->shape = *shape;
  if (c->shape.ld == 0) c->shape.ld = shape->d_model;
  c->params = *params;
  c->plan = make_plan(&c->shape, params);
  c->stream = reinterpret_cast<hipStream_t>(hip_stream);
  auto cleanup = [&](int code) {
    spectral_destroy(c);
    return code;
  };
  if (hipGetDevice(&c->device) != hipSuccess) return cleanup(fail(SN_ESTATE, "no HIP device"));
  const size_t L = c->shape.n_layers;
  if (hipMalloc(&c->ws, c->plan.bytes + 4 * L * sizeof(void*)) != hipSuccess) {
    // short of memory: the layer form without the group sums (up to 1 GiB) reads
    // its weights twice per iteration
    (void)hipGetLastError();
    c->ws = nullptr;
    if (c->plan.fused && c->plan.g > 1) c->plan = make_plan(&c->shape, params, false);
    if (hipMalloc(&c->ws, c->plan.bytes + 4 * L * sizeof(void*)) != hipSuccess) {
      c->ws = nullptr;
      return cleanup(fail(SN_EHIP, "hipMalloc(workspace and pointer table) failed"));
    }
  }
  c->d_tab = reinterpret_cast<const void**>(c->ws + c->plan.bytes);
  if (hipEventCreateWithFlags(&c->tab_event, hipEventDisableTiming) != hipSuccess)
    return cleanup(fail(SN_EHIP, "hipEventCreate failed"));
  c->tab = c->d_tab;
  bind_workspace(c);
  *ctx = c;
  return SN_OK;
}

SN_API int spectral_set_stream(sn_ctx* c, void* hip_stream) {
  if (!c) return fail(SN_ENULL, "ctx must not be NULL");
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  // later launches share the workspace and the eager pointer table with the
  // work queued on the previous stream: order the new stream after all of it
  // (a stream being captured into a graph cannot wait on an outside event;
  // its launches run at replay)
  if (st != c->stream && !capturing(st) && !capturing(c->stream)) {
    SN_HIP(hipEventRecord(c->tab_event, c->stream));
    SN_HIP(hipStreamWaitEvent(st, c->tab_event, 0));
  }
  c->stream = st;
  return SN_OK;
}

SN_API void spectral_destroy(sn_ctx* c) {
  if (!c) return;
  if (c->stream || c->ws) (void)hipStreamSynchronize(c->stream);
  for (auto& r : c->recs) {
    if (r.a) (void)hipEventDestroy(r.a);
    if (r.b) (void)hipEventDestroy(r.b);
  }
  for (auto e : c->pool) (void)hipEventDestroy(e);
  if (c->tab_event) (void)hipEventDestroy(c->tab_event);
  if (c->owns_ws && c->ws) (void)hipFree(c->ws);
  delete c;
}

SN_API int spectral_profile(sn_ctx* c, int32_t enable) {
  if (!c) return fail(SN_ENULL, "ctx must not be NULL");
  c->prof = enable != 0;
  return SN_OK;
}

SN_API int spectral_profile_read(sn_ctx* c, double* ms, int64_t* launches) {
  if (!c || !ms || !launches) return fail(SN_ENULL, "ctx, ms and launches must not be NULL");
  for (int k = 0; k < KIND_N; ++k) {
    ms[k] = 0.0;
    launches[k] = 0;
  }
  SN_HIP(hipStreamSynchronize(c->stream));
  for (auto& r : c->recs) {
    float t = 0.f;
    SN_HIP(hipEventElapsedTime(&t, r.a, r.b));
    ms[r.kind] += t;
    launches[r.kind] += 1;
    c->pool.push_back(r.a);
    c->pool.push_back(r.b);
  }
  c->recs.clear();
  return SN_OK;
}

SN_API int spectral_step(sn_ctx* c, const void* const* wq_layers, const void* const* wk_layers, float* v,
                         float* u, int32_t n_iter, float* sigma, float* scale, int32_t* iters) {
  if (!c) return fail(SN_ENULL, "ctx must not be NULL");
  if (!wq_layers || !wk_layers || !v || !sigma || !scale)
    return fail(SN_ENULL, "wq_layers, wk_layers, v, sigma and scale must not be NULL");
  if (n_iter < 1) return fail(SN_EINVAL, "n_iter must be >= 1");
  const int rc = update_table(c, wq_layers, wk_layers);
  if (rc != SN_OK) return rc;
  return step_body(c, v, u, n_iter, sigma, scale, iters);
}

}  // extern "C"

// ---- the allocation-free variant of spectral_step
//
// Its workspace and pointer table live in `scratch`, a static device array of
// kScratchBytes that each device holds from the library's first use on it
// until the process ends.  Host code reaches a device's copy only through the
// address hipGetSymbolAddress returns on that device (the array's name in
// host code is a host-side stand-in), kept per device here.  Nothing in the
// workspace must start at zero: every buffer a kernel reads was written
// earlier in the same call (the running flags by the first sweep, partials
// by their producer sweep, the tail's lists and control block by its list
// kernel).
namespace {

constexpr int kMaxDevices = 64;

static __device__ __attribute__((aligned(256))) uint8_t scratch[kScratchBytes];

std::mutex g_scratch_mu;
char* g_scratch_ptr[kMaxDevices] = {};

// Device address of this device's scratch (the current device), looked up
// once per device.
int scratch_on_device(int dev, char** out) {
  if (dev < 0 || dev >= kMaxDevices) return fail(SN_ESTATE, "device ordinal beyond the scratch table");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    SN_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return fail(SN_EHIP, "hipGetSymbolAddress(scratch) returned NULL");
    g_scratch_ptr[dev] = static_cast<char*>(p);
  }
  *out = g_scratch_ptr[dev];
  return SN_OK;
}

}  // namespace

extern "C" {

SN_API int spectral_step_noalloc(const sn_shape* shape, const sn_params* params, const void* const* wq_layers,
                                 const void* const* wk_layers, float* v, float* u, int32_t n_iter, float* sigma,
                                 float* scale, int32_t* iters, void* hip_stream) {
  if (!wq_layers || !wk_layers || !v || !sigma || !scale)
    return fail(SN_ENULL, "wq_layers, wk_layers, v, sigma and scale must not be NULL");
  int rc = validate(shape, params);
  if (rc != SN_OK) return rc;
  if (n_iter < 1) return fail(SN_EINVAL, "n_iter must be >= 1");
  sn_ctx c;
  c.shape = *shape;
  if (c.shape.ld == 0) c.shape.ld = shape->d_model;
  c.params = *params;
  size_t need = 0;
  if (!plan_scratch(&c.shape, params, &c.plan, &need))
    return fail(SN_EINVAL, "this shape needs " + std::to_string(need) + " bytes of scratch; spectral_step_noalloc " +
                               "holds at most " + std::to_string(kScratchBytes) + " (use spectral_init / spectral_step)");
  SN_HIP(hipGetDevice(&c.device));
  char* base = nullptr;
  if ((rc = scratch_on_device(c.device, &base)) != SN_OK) return rc;
  c.stream = reinterpret_cast<hipStream_t>(hip_stream);
  c.owns_ws = false;
  c.cache_table = false;
  c.d_tab = reinterpret_cast<const void**>(base);
  c.ws = base + table_bytes(c.shape.n_layers);
  bind_workspace(&c);
  if ((rc = update_table(&c, wq_layers, wk_layers)) != SN_OK) return rc;
  return step_body(&c, v, u, n_iter, sigma, scale, iters);
}

SN_API int spectral_step_layer(sn_ctx* c, const void* const* wq_layers, const void* const* wk_layers, float* v,
                               float* u, int32_t n_iter, float* sigma, float* scale) {
  if (!c) return fail(SN_ENULL, "ctx must not be NULL");
  if (!wq_layers || !wk_layers || !v || !sigma || !scale)
    return fail(SN_ENULL, "wq_layers, wk_layers, v, sigma and scale must not be NULL");
  if (!c->plan.layer) return fail(SN_ESTATE, "the context was created without SN_FLAG_LAYER");
  if (n_iter < 1) return fail(SN_EINVAL, "n_iter must be >= 1");
  int rc = update_table(c, wq_layers, wk_layers);
  if (rc != SN_OK) return rc;
  const Plan& pl = c->plan;
  const int L = c->shape.n_layers;
  float* lz = reinterpret_cast<float*>(c->ws + pl.off_lz);
  float* ly = reinterpret_cast<float*>(c->ws + pl.off_ly);
  float* lcol = reinterpret_cast<float*>(c->ws + pl.off_lcol);
  float* lvin = reinterpret_cast<float*>(c->ws + pl.off_lvin);
  float* lu = reinterpret_cast<float*>(c->ws + pl.off_lu);
  float* lv = reinterpret_cast<float*>(c->ws + pl.off_lv);
  float* n2_u = reinterpret_cast<float*>(c->ws + pl.off_ln2);
  float* n2_v = n2_u + L;
  if (fused_call(pl, c->shape.dtype, n_iter)) {
    if ((rc = run_layer_fused(c, v, u != nullptr, n_iter, lu, lv, n2_u)) != SN_OK) return rc;
    return layer_finalize(c, v, u, sigma, scale, lu, lv, n2_u);
  }
  // start vectors: copy, squared norms, layer status
  if ((rc = layer_reduce(c, v, 1, c->shape.d_model, 0, lv, n2_v)) != SN_OK) return rc;
  for (int k = 1; k <= n_iter; ++k) {
    LayerArgs a{};
    a.xvec = lv;  // z_j = K_j v
    a.xn2 = n2_v;
    a.rowpart = lz;
    if ((rc = layer_sweep(c, false, LM_ROWS, a)) != SN_OK) return rc;
    // u' = sum_h Q_h^T z_j(h): RepeatBlocks, then one column sweep over W_Q
    if ((rc = layer_vin(c, lz, c->shape.n_kv_heads, pl.s_lk, pl.g, 1, c->shape.n_q_heads)) != SN_OK) return rc;
    a = LayerArgs{};
    a.vin = lvin;
    a.colout = lcol;
    if ((rc = layer_sweep(c, true, LM_COLS, a)) != SN_OK) return rc;
    if ((rc = layer_reduce(c, lcol, pl.rs_q, col_stride(c->shape.d_model), 1, lu, n2_u)) != SN_OK) return rc;
    a = LayerArgs{};  // y_h = Q_h u
    a.xvec = lu;
    a.xn2 = n2_u;
    a.rowpart = ly;
    if ((rc = layer_sweep(c, true, LM_ROWS, a)) != SN_OK) return rc;
    // v' = sum_j K_j^T sum_{h in j} y_h: SumGroups, then one column sweep over W_K
    if ((rc = layer_vin(c, ly, c->shape.n_q_heads, pl.s_lq, 1, pl.g, c->shape.n_kv_heads)) != SN_OK) return rc;
    a = LayerArgs{};
    a.vin = lvin;
    a.colout = lcol;
    if ((rc = layer_sweep(c, false, LM_COLS, a)) != SN_OK) return rc;
    if ((rc = layer_reduce(c, lcol, pl.rs_k, col_stride(c->shape.d_model), 2, lv, n2_v)) != SN_OK) return rc;
  }
  return layer_finalize(c, v, u, sigma, scale, lu, lv, n2_u);
}

SN_API int spectral_logits_workspace_bytes(const sn_shape* shape, int32_t seq_len, int64_t* bytes) {
  if (!shape || !bytes) return fail(SN_ENULL, "shape and bytes must not be NULL");
  if (seq_len < 1) return fail(SN_EINVAL, "seq_len must be >= 1");
  if (shape->n_layers < 1) return fail(SN_EINVAL, "n_layers must be >= 1");
  *bytes = sn_logits_workspace_bytes(shape->n_layers, seq_len, (int64_t)shape->n_q_heads * shape->head_dim,
                                     (int64_t)shape->n_kv_heads * shape->head_dim);
  return SN_OK;
}

SN_API int spectral_logits_fp8(sn_ctx* c, const void* const* x_layers, int64_t ld_x, int32_t seq_len,
                               const void* const* wq_layers, const void* const* wk_layers, const float* scale,
                               void* workspace, int64_t workspace_bytes, uint8_t* codes, float* max_abs,
                               int32_t* n_over) {
  if (!c) return fail(SN_ENULL, "ctx must not be NULL");
  if (!x_layers || !wq_layers || !wk_layers || !scale || !workspace || !max_abs || !n_over)
    return fail(SN_ENULL, "x_layers, wq_layers, wk_layers, scale, workspace, max_abs and n_over must not be NULL");
  const sn_shape& sh = c->shape;
  if (sh.dtype != SN_BF16) return fail(SN_EDTYPE, "the logit consumer needs bf16 weights and tokens");
  const int dh = sh.head_dim;
  if (dh != 16 && dh != 32 && dh != 64 && dh != 128)
    return fail(SN_EINVAL, "the logit consumer needs head_dim 16, 32, 64 or 128");
  if (seq_len < 1 || seq_len > 46340) return fail(SN_EINVAL, "seq_len must be in [1, 46340]");
  if (ld_x == 0) ld_x = sh.d_model;
  if (ld_x < sh.d_model || (ld_x * 2) % 16 != 0) return fail(SN_EINVAL, "ld_x must be >= d_model, 8-element aligned");
  const int L = sh.n_layers;
  const int64_t nq_cols = (int64_t)sh.n_q_heads * dh, nk_cols = (int64_t)sh.n_kv_heads * dh;
  if ((int64_t)seq_len * ld_x * 2 >= (int64_t(1) << 31) || (int64_t)seq_len * nq_cols * 2 >= (int64_t(1) << 31))
    return fail(SN_EINVAL, "seq_len x row bytes must stay below 2^31");
  // the projection reads a layer's weight rows through one buffer range
  if (nq_cols * sh.ld * 2 >= (int64_t(1) << 32))
    return fail(SN_EINVAL, "n_q_heads x head_dim x ld x 2 bytes (one layer's W_Q) must stay below 2^32");
  const int64_t tiles = ceil_div(seq_len, 128);
  if ((int64_t)L * sh.n_q_heads * tiles * tiles >= (int64_t(1) << 31) ||
      (int64_t)L * tiles * ceil_div(nq_cols + nk_cols, 128) >= (int64_t(1) << 31))
    return fail(SN_EINVAL, "n_layers x n_q x (seq_len / 128)^2 must stay below 2^31");
  const int64_t need = sn_logits_workspace_bytes(L, seq_len, nq_cols, nk_cols);
  if (workspace_bytes < need) return fail(SN_EINVAL, "workspace too small (spectral_logits_workspace_bytes)");
  if ((reinterpret_cast<uintptr_t>(workspace) & 255) || (reinterpret_cast<uintptr_t>(codes) & 15))
    return fail(SN_EINVAL, "workspace must be 256-byte and codes 16-byte aligned");
  for (int l = 0; l < L; ++l) {
    if (!x_layers[l] || !wq_layers[l] || !wk_layers[l]) return fail(SN_ENULL, "a layer pointer is NULL");
    if ((reinterpret_cast<uintptr_t>(x_layers[l]) | reinterpret_cast<uintptr_t>(wq_layers[l]) |
         reinterpret_cast<uintptr_t>(wk_layers[l])) & 15)
      return fail(SN_EINVAL, "layer pointers must be 16-byte aligned");
  }
  int cur_dev = 0;
  SN_HIP(hipGetDevice(&cur_dev));
  if (cur_dev != c->device) return fail(SN_ESTATE, "the current HIP device is not the context's device");

  // pointer tables at the start of the workspace, written by a kernel whose
  // arguments carry the pointers (so the call can be captured into a graph)
  const void** d_tab = reinterpret_cast<const void**>(workspace);
  int rc = fill_table(d_tab, 3 * L,
                      [&](int i) { return i < L ? x_layers[i] : i < 2 * L ? wq_layers[i - L] : wk_layers[i - 2 * L]; },
                      c->stream);
  if (rc != SN_OK) return rc;
  uint16_t* planes = reinterpret_cast<uint16_t*>(reinterpret_cast<char*>(workspace) + ((3 * L * 8 + 255) & ~255));
  const size_t qn = (size_t)L * seq_len * nq_cols, kn = (size_t)L * seq_len * nk_cols;
  ProjArgs p{};
  p.x = d_tab;
  p.wq = d_tab + L;
  p.wk = d_tab + 2 * L;
  p.ld_x = ld_x;
  p.ld_w = sh.ld;
  p.layers = L;
  p.seq = seq_len;
  p.d = sh.d_model;
  p.nq_cols = (int32_t)nq_cols;
  p.nk_cols = (int32_t)nk_cols;
  p.qh = planes;
  p.ql = planes + qn;
  p.kh = planes + 2 * qn;
  p.kl = planes + 2 * qn + kn;
  LogitArgs g{};
  g.qh = p.qh;
  g.ql = p.ql;
  g.kh = p.kh;
  g.kl = p.kl;
  g.layers = L;
  g.seq = seq_len;
  g.g = c->plan.g;
  g.nq_cols = (int32_t)nq_cols;
  g.nk_cols = (int32_t)nk_cols;
  g.tiles = ceil_div(seq_len, 128);
  g.n_heads = sh.n_q_heads;
  g.scale = scale;
  g.codes = codes;
  g.max_abs = max_abs;
  g.n_over = n_over;
  rc = timed(c, KIND_LOGITS, [&] { sn_launch_zero_stats(max_abs, n_over, L * sh.n_q_heads, c->stream); });
  if (rc != SN_OK) return rc;
  if ((rc = timed(c, KIND_PROJ, [&] { sn_launch_proj(p, c->stream); })) != SN_OK) return rc;
  return timed(c, KIND_LOGITS, [&] { sn_launch_logits(g, dh, c->stream); });
}
}  // extern "C"
