// Layer-level form of the estimator (spectral_step_layer), for MI355X
// (gfx950, wave64).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "sweep_device.h"

namespace sn {
namespace {

// ---------------------------------------------------------------------------
// Layer-level form (spectral_step_layer): the estimator as printed in App. E,
// one pair u, v in R^d per layer for the concatenated W^Q = [W^Q_1 .. W^Q_nq]
// and the key blocks repeated per group (RepeatBlocks) on the way in and
// summed per group (SumGroups) on the way back.  One step is:
//   rows(W_K, v):  z_j = K_j v                       (row sums, per key head)
//   vin:           z_j(h) for every query head h     (RepeatBlocks)
//   cols(W_Q, z):  u' = sum_h Q_h^T z_j(h)           (column sums over all rows)
//   sigma = ||u'||                                   (layer_colsum / layer_norm)
//   rows(W_Q, u):  y_h = Q_h u'/sigma
//   vin:           sum_{h in group j} y_h            (SumGroups)
//   cols(W_K, y):  v' = sum_j K_j^T (sum_{h in j} y_h)
//   ||v'||                                           (layer_colsum / layer_norm)
// A column-sweep wave owns one column tile of a layer and streams it down the
// layer's row blocks (16 KB of 128-byte row segments per block, as in the
// W_Q sweep), so its column sums are final for those rows: only one d-vector
// per layer (per row split, on small shapes) is written, not one per head.
// Per-layer status: 0 running, -1 start vector zero or not finite, -2 M v = 0.


template <typename T, int DH, int MODE>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4)))
layer_sweep_kernel(LayerArgs a) {
  constexpr int VEC = Traits<T>::VEC;
  constexpr int CPL = kCPL;
  constexpr int RPL = DH / kRG;
  constexpr int TILE_C = CPL * VEC;
  constexpr int ES = sizeof(T);
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int chunk = lane % CPL, rg = lane / CPL;
  const int item = blockIdx.x * kWaves + wv;
  const bool in_range = item < a.n_items;
  // rows: (layer, unit, strip of tiles); cols: (layer, row split, tile)
  int layer, ul = 0, strip = 0, rs = 0, tile_c = 0;
  if (MODE == LM_ROWS) {
    const int unit = in_range ? item / a.s_out : 0;
    strip = in_range ? item % a.s_out : 0;
    layer = unit / a.units;
    ul = unit % a.units;
  } else {
    tile_c = in_range ? item % a.n_tiles : 0;
    const int rest = in_range ? item / a.n_tiles : 0;
    rs = rest % a.n_rsplit;
    layer = rest / a.n_rsplit;
  }
  const bool valid = in_range && uni(a.lstat[layer]) == 0;
  if (!valid) return;

  const char* base = uni(a.mats[layer]);
  const uint32_t nrec = (uint32_t)((((int64_t)(DH - 1) * a.ld + a.d) * ES + 15) & ~int64_t(15));
  auto rsrc_of = [&](int rb) {  // the d_h x ld row block rb of this layer's matrix
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base + (int64_t)rb * DH * a.ld * ES), (short)0,
                                             (int)nrec, kRsrcWord3);
  };
  const uint32_t lane_off = (uint32_t)(((int64_t)rg * RPL * a.ld + chunk * VEC) * ES);
  const uint32_t row_bytes = (uint32_t)(a.ld * ES);
  auto load_tile = [&](u32x4 (&tile)[RPL], __amdgpu_buffer_rsrc_t rsrc, int t) {
    const uint32_t voff = lane_off + (uint32_t)(t * TILE_C * ES);
#pragma unroll
    for (int rr = 0; rr < RPL; ++rr)
      tile[rr] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff, rr * row_bytes, kStreamPolicy);
  };
  const int n_full = a.d / TILE_C;
  // zero the elements at columns >= d of the ragged last tile
  auto mask_tail = [&](u32x4 (&tile)[RPL], int t) {
    if (t < n_full) return;
    const int nval = a.d - (t * TILE_C + chunk * VEC);
    u32x4 m;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (VEC == 8)
        m[q] = (2 * q < nval ? 0x0000ffffu : 0u) | (2 * q + 1 < nval ? 0xffff0000u : 0u);
      else
        m[q] = q < nval ? 0xffffffffu : 0u;
    }
#pragma unroll
    for (int rr = 0; rr < RPL; ++rr) tile[rr] &= m;
  };

  if (MODE == LM_ROWS) {
    const __amdgpu_buffer_rsrc_t rsrc = rsrc_of(ul);
    const float* xrow = a.xvec + (size_t)layer * a.d;
    float acc[RPL];
#pragma unroll
    for (int rr = 0; rr < RPL; ++rr) acc[rr] = 0.f;
    const int t0 = strip * a.tps;
    const int t1 = min(t0 + a.tps, a.n_tiles);
    // staggered start tile and loads ahead of arithmetic, as in the W_Q sweep
    const int n_mine = t1 - t0;
    int t = t0;
    if (n_mine > 1) t += (int)(((uint32_t)item * 2654435761u) >> 16) % n_mine;
#pragma unroll 1
    for (int i = 0; i < n_mine; ++i, t = (t + 1 == t1) ? t0 : t + 1) {
      u32x4 tile[RPL];
      load_tile(tile, rsrc, t);
      __builtin_amdgcn_sched_barrier(0);
      mask_tail(tile, t);
      const int col = t * TILE_C + chunk * VEC;
      const int nval = a.d - col;  // >= VEC on full tiles
      float xv[VEC];
#pragma unroll
      for (int c = 0; c < VEC; ++c) xv[c] = c < nval ? xrow[min(col + c, a.d - 1)] : 0.f;
#pragma unroll
      for (int rr = 0; rr < RPL; ++rr) {
        float s = acc[rr];
#pragma unroll
        for (int c = 0; c < VEC; ++c) s = fmaf(elem<T>(tile[rr], c), xv[c], s);
        acc[rr] = s;
      }
    }
    const float xs_inv = 1.0f / sqrtf(a.xn2[layer]);
    float* op = a.rowpart + (((size_t)layer * a.units + ul) * a.s_out + strip) * DH + rg * RPL;
#pragma unroll
    for (int rr = 0; rr < RPL; ++rr) {
      float s = acc[rr];
#pragma unroll
      for (int m = 1; m < CPL; m <<= 1) s = xor_sum(s, m);
      if ((rr % CPL) == chunk) op[rr] = s * xs_inv;
    }
  } else {
    // one column tile down row blocks rb0 .. rb1 - 1, starting at a staggered
    // block so that the waves of neighbouring tiles read different rows
    const int rb0 = rs * a.rb_per, rb1 = min(a.nrb, rb0 + a.rb_per);
    const int n_mine = rb1 - rb0;
    int rb = rb0;
    if (n_mine > 1) rb += (int)(((uint32_t)item * 2654435761u) >> 16) % n_mine;
    const float* vl = a.vin + (size_t)layer * a.nrb * DH + rg * RPL;
    float w[VEC];
#pragma unroll
    for (int c = 0; c < VEC; ++c) w[c] = 0.f;
#pragma unroll 1
    for (int i = 0; i < n_mine; ++i, rb = (rb + 1 == rb1) ? rb0 : rb + 1) {
      u32x4 tile[RPL];
      load_tile(tile, rsrc_of(rb), tile_c);
      float z[RPL];
#pragma unroll
      for (int rr = 0; rr < RPL; ++rr) z[rr] = vl[(size_t)rb * DH + rr];
      __builtin_amdgcn_sched_barrier(0);
      mask_tail(tile, tile_c);
#pragma unroll
      for (int rr = 0; rr < RPL; ++rr)
#pragma unroll
        for (int c = 0; c < VEC; ++c) w[c] = fmaf(elem<T>(tile[rr], c), z[rr], w[c]);
    }
#pragma unroll
    for (int c = 0; c < VEC; ++c) w[c] = group_sum(w[c]);
    if (rg == 0) {  // columns past d are zero (masked) and land in the row's padding
      float* out = a.colout + ((size_t)layer * a.n_rsplit + rs) * a.cstride + tile_c * TILE_C + chunk * VEC;
#pragma unroll
      for (int c = 0; c < VEC; ++c) out[c] = w[c];
    }
  }
}

// ---------------------------------------------------------------------------
// One-pass sweeps (up to kLFRows rows per layer after grouping).  u' = Q~^T z
// needs a column's every row before y = Q~ u' can use it, so the sweeps above
// read each matrix twice per iteration.  Two changes take that to less than
// once:
//   - The heads of a group share z and their y are summed, so only the group
//     sums Q~_j = sum_h Q_h (n_kv d_h rows, fp32) enter the iteration; they
//     are formed once per call (group_sum_kernel): 10.7 GB of W_Q become
//     2.7 GB at 70B.
//   - A workgroup holds a whole column tile (every row x 128 bytes, 128 KB for
//     1024 rows) in the registers of its waves, 64 rows each: column sums are
//     reduced over the waves through LDS and used for the row sums in place.
// Bound by HBM: one tile is always in flight per wave while the previous one is
// multiplied (32 + 32 registers of tiles, 4 waves per SIMD).  70B, five
// iterations: 18.0 ms with two passes per matrix and iteration, 5.9 ms so (the
// group sums 2.27 ms at 6.0 TB/s read and written, sweeps over them 134 us per
// 27 layers at 6.8 TB/s, over W_K 77 us at 5.9 TB/s).
template <typename T, bool INIT>
__global__ void __launch_bounds__(64 * kLFWaves) layer_fused_kernel(LayerFusedArgs a) {
  constexpr int VEC = Traits<T>::VEC, ES = sizeof(T), TILE_C = kCPL * VEC, RPL = kLFRowsPerWave / kRG;
  __shared__ __attribute__((aligned(16))) float red[2][kLFWaves][TILE_C];
  const int lane = threadIdx.x & 63, wv = uni((int)(threadIdx.x >> 6)), nw = (int)blockDim.x >> 6;
  const int chunk = lane % kCPL, rg = lane / kCPL;
  const int ll = blockIdx.x / a.strips, strip = blockIdx.x % a.strips, layer = a.layer0 + ll;
  if (uni(a.lstat[layer]) != 0 && !INIT) return;  // whole workgroup
  const int r0 = kLFRowsPerWave * wv, rows = min(kLFRowsPerWave, a.rows - r0);
  const char* base = a.mats ? uni(a.mats[layer]) : reinterpret_cast<const char*>(a.dense) + (int64_t)ll * a.rows * a.ld * ES;
  const __amdgpu_buffer_rsrc_t rsrc =
      make_rsrc(base + (int64_t)r0 * a.ld * ES, (uint32_t)((((int64_t)(rows - 1) * a.ld + a.d) * ES + 15) & ~int64_t(15)));
  const uint32_t row_bytes = (uint32_t)(a.ld * ES), lane_off = (uint32_t)rg * RPL * row_bytes + chunk * 16u;
  const int n_full = a.d / TILE_C, t0 = strip * a.tps, n = min(a.tps, a.n_tiles - t0);
  const int rot = (int)((((uint32_t)blockIdx.x * 2654435761u) >> 16) % (uint32_t)n);
  auto tile_at = [&](int i) { const int u = rot + i; return t0 + (u >= n ? u - n : u); };
  auto load = [&](u32x4 (&tile)[RPL], int t) {
#pragma unroll
    for (int rr = 0; rr < RPL; ++rr)
      tile[rr] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane_off + (uint32_t)t * 128u, rr * row_bytes, kStreamPolicy);
  };
  u32x4 ta[RPL], tb[RPL];
  load(ta, tile_at(0));
  float x[RPL], acc[RPL], nrm = 0.f;
#pragma unroll
  for (int rr = 0; rr < RPL; ++rr) {
    const int r = rg * RPL + rr;
    x[rr] = !INIT && r < rows ? a.x[(size_t)layer * a.rows + r0 + r] : 0.f;
    acc[rr] = 0.f;
  }
  auto step = [&](u32x4 (&tile)[RPL], int t, int buf) {
    const int col = t * TILE_C + chunk * VEC;
    if (t >= n_full) {  // the ragged last tile: zero the elements at columns >= d
      u32x4 m;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        m[q] = VEC == 8 ? (col + 2 * q < a.d ? 0x0000ffffu : 0u) | (col + 2 * q + 1 < a.d ? 0xffff0000u : 0u)
                        : (col + q < a.d ? 0xffffffffu : 0u);
#pragma unroll
      for (int rr = 0; rr < RPL; ++rr) tile[rr] &= m;
    }
    float w[VEC];
    if constexpr (INIT) {
      const float* v = a.v + (size_t)layer * a.d;
#pragma unroll
      for (int c = 0; c < VEC; ++c) w[c] = col + c < a.d ? v[min(col + c, a.d - 1)] : 0.f;
    } else {
#pragma unroll
      for (int c = 0; c < VEC; ++c) w[c] = 0.f;
#pragma unroll
      for (int rr = 0; rr < RPL; ++rr) {
        if (rr % 2 == 0) __builtin_amdgcn_sched_barrier(0);  // no more than two rows widened to fp32 at a time
#pragma unroll
        for (int c = 0; c < VEC; ++c) w[c] = fmaf(elem<T>(tile[rr], c), x[rr], w[c]);
      }
#pragma unroll
      for (int rr = 0; rr < RPL; ++rr) reuse_fence(tile[rr]);
#pragma unroll
      for (int c = 0; c < VEC; ++c) w[c] = group_sum(w[c]);
      if (rg == 0) {
#pragma unroll
        for (int c = 0; c < VEC; c += 4)
          *reinterpret_cast<f32x4*>(&red[buf][wv][chunk * VEC + c]) = f32x4{w[c], w[c + 1], w[c + 2], w[c + 3]};
      }
      // two buffers: the next tile's sums go to the other one, and a wave can
      // be at most one tile ahead of the slowest
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
#pragma unroll
      for (int c = 0; c < VEC; c += 4) {
        f32x4 s = *reinterpret_cast<const f32x4*>(&red[buf][0][chunk * VEC + c]);
#pragma unroll 2
        for (int q = 1; q < nw; ++q) s += *reinterpret_cast<const f32x4*>(&red[buf][q][chunk * VEC + c]);
#pragma unroll
        for (int e = 0; e < 4; ++e) w[c + e] = s[e];
      }
    }
#pragma unroll
    for (int c = 0; c < VEC; ++c) nrm = fmaf(w[c], w[c], nrm);
    if (!INIT && a.vec && wv == 0 && rg == 0) {
#pragma unroll
      for (int c = 0; c < VEC; ++c)
        if (col + c < a.d) a.vec[(size_t)layer * a.d + col + c] = w[c];
    }
#pragma unroll
    for (int rr = 0; rr < RPL; ++rr) {
      if (rr % 2 == 0) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int c = 0; c < VEC; ++c) acc[rr] = fmaf(elem<T>(tile[rr], c), w[c], acc[rr]);
    }
  };
#pragma unroll 1
  for (int i = 0; i < n; i += 2) {
    if (i + 1 < n) load(tb, tile_at(i + 1));
    __builtin_amdgcn_sched_barrier(0);
    step(ta, tile_at(i), 0);
    if (i + 1 >= n) break;
    if (i + 2 < n) load(ta, tile_at(i + 2));
    __builtin_amdgcn_sched_barrier(0);
    step(tb, tile_at(i + 1), 1);
  }
  float* part = a.part + ((size_t)ll * a.strips + strip) * a.rows + r0;
#pragma unroll
  for (int rr = 0; rr < RPL; ++rr) {
    float s = acc[rr];
#pragma unroll
    for (int m = 1; m < kCPL; m <<= 1) s = xor_sum(s, m);
    const int r = rg * RPL + rr;
    if (rr == chunk && r < rows) part[r] = s;
  }
#pragma unroll
  for (int m = 1; m < kCPL; m <<= 1) nrm = xor_sum(nrm, m);
  if (wv == 0 && lane == 0) a.n2part[(size_t)ll * a.strips + strip] = nrm;
}

// The input of the next one-pass sweep, x = sum of the strips' row sums over
// the norm of the vector they were taken with, and that squared norm and the
// layer status.  Block (b, l): rows b * kRedThreads .. of layer l of the chunk.
__global__ void __launch_bounds__(kRedThreads) layer_gather_kernel(LayerFusedArgs a) {
  const int ll = blockIdx.y, layer = a.layer0 + ll;
  // the block that may write the status is the only one to look at it: the others'
  // x of a stopped layer is never read
  if (blockIdx.x == 0 && a.mode != 0 && a.lstat[layer] != 0) return;
  float n2 = 0.f;
  for (int s = 0; s < a.strips; ++s) n2 += a.n2part[(size_t)ll * a.strips + s];
  const int r = blockIdx.x * kRedThreads + (int)threadIdx.x;
  if (r < a.rows) {
    const float* p = a.part + (size_t)ll * a.strips * a.rows + r;
    float x = 0.f;
#pragma unroll 8
    for (int s = 0; s < a.strips; ++s) x += p[(size_t)s * a.rows];
    a.x[(size_t)layer * a.rows + r] = x / sqrtf(n2);
  }
  __syncthreads();  // every thread has read the status
  if (r == 0) {
    a.n2[layer] = n2;
    if (a.mode == 0) {
      a.n2_start[layer] = n2;
      a.lstat[layer] = (n2 > 0.f && isfinite(n2)) ? 0 : -1;
    } else if (a.mode == 1 && n2 == 0.f) {
      a.lstat[layer] = -2;
    }
  }
}

// Q~ of a chunk of layers: thread (row r of the layer's rows, 16-byte chunk of
// columns); the loads of eight heads are in flight at a time.  Columns past d
// become zero up to the padded row length.
template <typename T>
__global__ void __launch_bounds__(kThreads) group_sum_kernel(GroupSumArgs a) {
  constexpr int VEC = Traits<T>::VEC;
  const int cpr = a.ldq / VEC;  // chunks per row
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int ll = blockIdx.y;
  if (i >= (int64_t)a.rows * cpr) return;
  const int r = (int)(i / cpr), col = (int)(i % cpr) * VEC;
  const int j = r / a.dh, rr = r % a.dh;
  float s[VEC];
#pragma unroll
  for (int c = 0; c < VEC; ++c) s[c] = 0.f;
  if (col < a.d) {
    const char* p = static_cast<const char*>(a.wq[a.layer0 + ll]) + (((int64_t)j * a.g * a.dh + rr) * a.ld + col) * (int64_t)sizeof(T);
    const int64_t step = (int64_t)a.dh * a.ld * sizeof(T);
#pragma unroll 8
    for (int h = 0; h < a.g; ++h) {
      const u32x4 x = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p + h * step));
#pragma unroll
      for (int c = 0; c < VEC; ++c) s[c] += elem<T>(x, c);
    }
#pragma unroll
    for (int c = 0; c < VEC; ++c) s[c] = col + c < a.d ? s[c] : 0.f;
  }
  f32x4* out = reinterpret_cast<f32x4*>(a.out + ((int64_t)ll * a.rows + r) * a.ldq + col);
#pragma unroll
  for (int c = 0; c < VEC; c += 4) out[c / 4] = f32x4{s[c], s[c + 1], s[c + 2], s[c + 3]};
}

// vin of a column sweep (see LayerVinArgs): block (b, l), one thread per row.
__global__ void __launch_bounds__(64) layer_vin_kernel(LayerVinArgs v) {
  const int b = blockIdx.x, l = blockIdx.y;
  if (v.lstat[l] != 0) return;
  const float* src = v.part + ((size_t)l * v.src_units + (size_t)(b / v.div) * v.cnt) * v.strips * v.dh;
  const int n = v.cnt * v.strips;  // the cnt units' partials lie back to back
  for (int r = threadIdx.x; r < v.dh; r += 64) {
    float s = 0.f;
    for (int k = 0; k < n; ++k) s += src[(size_t)k * v.dh + r];
    v.vin[((size_t)l * v.nrb + b) * v.dh + r] = s;
  }
}


// Column sums: block (b, l) owns columns b * kRedThreads .. of layer l, one
// per thread; the units are summed in order, their loads issued eight at a
// time.
__global__ void __launch_bounds__(kRedThreads) layer_colsum_kernel(LayerReduceArgs r) {
  const int b = blockIdx.x, l = blockIdx.y, t = threadIdx.x;
  __shared__ float red[kRedThreads / 64];
  if (r.mode != 0 && r.lstat[l] != 0) return;
  const int c = b * kRedThreads + t;
  float sq = 0.f;
  if (c < r.d) {
    const float* p = r.col + (size_t)l * r.units * r.cstride + c;
    float s = 0.f;
#pragma unroll 8
    for (int u = 0; u < r.units; ++u) s += p[(size_t)u * r.cstride];
    r.vec[(size_t)l * r.d + c] = s;
    sq = s * s;
  }
  sq = wave_sum(sq);
  if ((t & 63) == 0) red[t >> 6] = sq;
  __syncthreads();
  if (t == 0) r.n2part[(size_t)l * r.nb + b] = sum_waves<kRedThreads / 64>(red);
}

// n2 of each layer from its column blocks, in block order, and the status.
__global__ void __launch_bounds__(64) layer_norm_kernel(LayerReduceArgs r) {
  const int l = blockIdx.x;
  if (threadIdx.x != 0 || (r.mode != 0 && r.lstat[l] != 0)) return;
  float n2 = 0.f;
  for (int b = 0; b < r.nb; ++b) n2 += r.n2part[(size_t)l * r.nb + b];
  r.n2[l] = n2;
  if (r.mode == 0) {
    r.n2_start[l] = n2;
    r.lstat[l] = (n2 > 0.f && isfinite(n2)) ? 0 : -1;
  } else if (r.mode == 1 && n2 == 0.f) {
    r.lstat[l] = -2;
  }
}


constexpr int kFinCols = 4 * kThreads;  // columns per workgroup (one workgroup per layer took 31 us at 70B)

__global__ void __launch_bounds__(kThreads) layer_finalize_kernel(LayerFinArgs f) {
  const int l = blockIdx.y;
  const int st = f.lstat[l];
  const float sig = st == -1 ? __builtin_nanf("") : st == -2 ? 0.f : sqrtf(f.n2_u[l]);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    f.sigma[l] = sig;
    f.scale[l] = f.coef * sig;
  }
  float* vp = f.v + (size_t)l * f.d;
  float* up = f.u ? f.u + (size_t)l * f.d : nullptr;
  const float vs = st == 0 ? 1.0f / sqrtf(f.n2_v[l]) : st == -2 ? 1.0f / sqrtf(f.n2_start[l]) : 1.f;
  const float us = st == 0 ? 1.0f / sig : 0.f;
  const int c1 = min(f.d, ((int)blockIdx.x + 1) * kFinCols);
  for (int c = blockIdx.x * kFinCols + threadIdx.x; c < c1; c += kThreads) {
    if (st == 0) vp[c] = f.lv[(size_t)l * f.d + c] * vs;
    else if (st == -2) vp[c] *= vs;
    if (up) up[c] = st == 0 ? f.lu[(size_t)l * f.d + c] * us : 0.f;
  }
}

template <typename T, int MODE>
void layer_dispatch(int dh, dim3 grid, hipStream_t st, const LayerArgs& a) {
  switch (dh) {
    case 8: layer_sweep_kernel<T, 8, MODE><<<grid, kThreads, 0, st>>>(a); break;
    case 16: layer_sweep_kernel<T, 16, MODE><<<grid, kThreads, 0, st>>>(a); break;
    case 32: layer_sweep_kernel<T, 32, MODE><<<grid, kThreads, 0, st>>>(a); break;
    case 64: layer_sweep_kernel<T, 64, MODE><<<grid, kThreads, 0, st>>>(a); break;
    default: layer_sweep_kernel<T, 128, MODE><<<grid, kThreads, 0, st>>>(a); break;
  }
}

}  // namespace

void launch_layer_sweep(bool bf16, int head_dim, int mode, int n_items, hipStream_t st, const LayerArgs& a) {
  const dim3 grid((n_items + kWaves - 1) / kWaves);
  if (bf16) {
    if (mode == LM_ROWS) layer_dispatch<uint16_t, LM_ROWS>(head_dim, grid, st, a);
    else layer_dispatch<uint16_t, LM_COLS>(head_dim, grid, st, a);
  } else {
    if (mode == LM_ROWS) layer_dispatch<float, LM_ROWS>(head_dim, grid, st, a);
    else layer_dispatch<float, LM_COLS>(head_dim, grid, st, a);
  }
}

void launch_layer_fused(bool bf16, bool init, int layers, hipStream_t st, const LayerFusedArgs& a) {
  const dim3 grid(layers * a.strips), block(64 * ((a.rows + kLFRowsPerWave - 1) / kLFRowsPerWave));
  if (bf16) {
    if (init) layer_fused_kernel<uint16_t, true><<<grid, block, 0, st>>>(a);
    else layer_fused_kernel<uint16_t, false><<<grid, block, 0, st>>>(a);
  } else {
    if (init) layer_fused_kernel<float, true><<<grid, block, 0, st>>>(a);
    else layer_fused_kernel<float, false><<<grid, block, 0, st>>>(a);
  }
}

void launch_layer_gather(int layers, hipStream_t st, const LayerFusedArgs& a) {
  layer_gather_kernel<<<dim3((a.rows + kRedThreads - 1) / kRedThreads, layers), kRedThreads, 0, st>>>(a);
}

void launch_group_sum(bool bf16, int layers, hipStream_t st, const GroupSumArgs& a) {
  const int64_t n = (int64_t)a.rows * (a.ldq / (bf16 ? 8 : 4));
  const dim3 grid((unsigned)((n + kThreads - 1) / kThreads), layers);
  if (bf16)
    group_sum_kernel<uint16_t><<<grid, kThreads, 0, st>>>(a);
  else
    group_sum_kernel<float><<<grid, kThreads, 0, st>>>(a);
}

void launch_layer_vin(int layers, hipStream_t st, const LayerVinArgs& v) {
  layer_vin_kernel<<<dim3(v.nrb, layers), 64, 0, st>>>(v);
}

void launch_layer_reduce(int layers, hipStream_t st, const LayerReduceArgs& r) {
  layer_colsum_kernel<<<dim3(r.nb, layers), kRedThreads, 0, st>>>(r);
  layer_norm_kernel<<<dim3(layers), 64, 0, st>>>(r);
}

void launch_layer_finalize(int layers, hipStream_t st, const LayerFinArgs& f) {
  layer_finalize_kernel<<<dim3((f.d + kFinCols - 1) / kFinCols, layers), kThreads, 0, st>>>(f);
}

}  // namespace sn
