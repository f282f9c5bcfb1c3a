// The Gram form with one workgroup per head (gfx950, wave64): Gram matrices
// and the whole d_h-space iteration of a head without leaving the compute
// unit, so that no query Gram matrix is ever written to memory.
//
// Per head the arithmetic is that of gram.hip (G_Q = Q Q^T, G_K = K K^T; one
// step is w = G_Q z, sigma^2 = z^T w, y = w / sigma, t = G_K y, ||v'||^2 =
// y^T t, z = t / ||v'||); what differs is where it runs.
//   units_kernel (grouped heads, or few heads): one workgroup per key head,
//     chunk of query heads and column strip reads its part of K_j once and
//     forms G_K (chunk 0) and z0 = K_j v, ||v||^2 for the heads of the chunk.
//     With fewer heads than compute units it also forms the G_Q, in column
//     strips, so that the whole chip streams.
//   heads_kernel: one workgroup per query head reads Q_h once, forms G_Q in
//     registers, loads G_K (or, with g = 1, streams K_h first and forms G_K,
//     z0 and ||v|| itself), iterates to the count or the tolerance and leaves
//     z / sigma and y of the last step with 1 / ||K^T y||, which the final sweeps
//     map to u and v, already normalised.
// Against n_iter pairs of sweeps, whole calls on one box: 70B GQA shape, 30
// iterations 56.3 -> 2.48 ms; Llama-2-7B shape 10.5 -> 0.78 ms; GPT-2 XL shape
// with u 2.56 -> 0.25 ms; GPT-2 small, 20 iterations 405 -> 70 us; 5
// iterations of 144 heads, d 3001, 261 -> 68 us.
//
// Streaming.  The workgroup's four waves share a ring of row tiles (d_h rows
// x 128 bytes) in LDS, filled by buffer loads straight to LDS; one bare
// barrier per tile says that the tile has landed and that its predecessor's
// slot is free.  The waits written here leave the loads of the next NST - 2 tiles
// in flight across it.  The compiler, which tracks loads to LDS by alias, adds a
// full wait before the LDS reads of two of the streams (the query strips of
// units_kernel and the key stream of H_OWN); the key stream of units_kernel lost
// its own with the start vectors read as the vector type of the tiles: 70B GQA
// shape 2.51 -> 2.47 ms, GPT-2 small 76 -> 74 us of two iterations.
// The upper-triangle 16 x 16 blocks of G are split over the waves by
// quadrants (waves 0 and 1: the two diagonal triangles; waves 2 and 3: halves
// of the off-diagonal square), so a wave reads at most 6 of the 8 row blocks
// of a tile (d_h = 128) and no sum over waves is needed.  The z0 products
// (slots: heads x bf16 parts of v) go to waves 2 and 3, which hold fewer
// blocks.
//
// Precision.  z^T G z rounds relative to b = sum_i z_i^2 G_ii, a sweep of Q
// relative to sqrt(b), and an error in G repeats in every step, where those of
// the sweeps differ.  So G's sums and (but for I_HALVES, below) the iteration are
// in double, with the sweeps' accuracy down to sigma^2 near b / 4.  Every step weighs
// its products against b; a head whose rows cancel further over its steps, whose
// Gram matrix is near the ends of the float range, or whose values are not
// finite is iterated again from z0 by reading Q_h and K_j directly
// (direct_sweep), in the order of the sweep form and with its stopping rules.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <type_traits>

#include "gram_device.h"

namespace sn {
namespace {

constexpr int kHThreads = 64 * kHWaves;
// How a head is iterated.  An error in G repeats in every step, where those of a
// sweep differ, so G has to be better than the sweeps' 32 bits: its sums are
// formed in double, and I_ROWS (d_h <= 64; threads hold rows of G) and I_BLOCKS
// (d_h 128; each wave holds the blocks it accumulated) iterate in double too.
// I_HALVES is I_ROWS with G and the vectors in float, for d_h 128 where the final
// W_K sweep takes vectors in two bf16 halves (2^-17), as the sweeps of such
// groups do in every step (their v errs by 6e-6).
enum { I_ROWS = 0, I_BLOCKS = 1, I_HALVES = 2 };

// An error E in G, of rows E_i. ~ eps sqrt(G_ii) (sqrt(G_jj))_j, turns w = G z by
// about eps sqrt(b tr(G)), b = sum_i z_i^2 G_ii: relative to |w| that is eps / r with
// r = sqrt(d_h / (b tr(G))) |w|, and b / sigma^2 times what the sweeps' own rounding of
// u' = Q^T z does to w.  Rows that do not cancel have r and sigma^2 / b near 1 or above.
// The errors of v add up over the products: each counts min(1 / r, b / sigma^2)^2, and
// a head whose mean over its steps passes kCancelMean is iterated on its weights, as
// is one whose reported sigma^2 (or ||v'||^2) lies below kCancelSigma b.  A product
// that cancels in passing, as the first of a random start may, costs nothing then.
// Errors of v after 20 steps at a constant r with all heads kept, against the
// sweeps: I_ROWS (d 768) r 0.55 2.1e-7 (3.3e-7), 0.25 7.4e-7 (3.5e-7), 0.08 2.9e-6
// (4.8e-7); I_BLOCKS (d 1024) 2.4e-7 (4.2e-7), 7.4e-7 (4.4e-7), 3.2e-6 (6.1e-7);
// I_HALVES (d 4096, 8 heads) 4.0e-6 (6.1e-6), 8.2e-6 (5.7e-6), 2.8e-5 (6.6e-6).
// Errors of sigma reach the sweeps' at sigma^2 / b near 0.2.
constexpr float kCancelMean = 2.f;  // one of the two matrices at r = 0.58, the other at 1
constexpr float kCancelSigma = 0.25f;
constexpr float kTinyRow = 0x1p-40f;                  // least diagonal element, of a trace in [1, 4)
constexpr float kGramMin = 1e-26f, kGramMax = 1e34f;  // trace of which the products neither under- nor overflow

template <typename T, int DH>
struct HShape {
  static constexpr int ES = sizeof(T);
  static constexpr int VEC = 16 / ES;
  static constexpr int TC = 128 / ES;               // columns per tile
  static constexpr int RB = DH / 16, NB = RB * (RB + 1) / 2;
  static constexpr int STAGE = tile_bytes(DH);
  static constexpr int VROW = TC * 4;               // bytes of one start vector's columns of a tile
  static constexpr int VCH = VROW / 16;             // ... in 16-byte chunks
  static constexpr int NR = RB > 1 ? RB / 2 : 1;    // row blocks of a diagonal triangle
  static constexpr int NC = RB >= 4 ? RB / 4 : 1;   // column blocks of an off-diagonal half
  static constexpr int NTRI = NR * (NR + 1) / 2;
  static constexpr int NACC = NTRI > NR * NC ? NTRI : NR * NC;
  static constexpr int NZ = RB >= 4 ? RB / 2 : RB;  // row blocks of z0 per wave (2 and 3, or 2 alone)
  static constexpr int P = DH + 1;                  // LDS row pitch of a whole Gram matrix
  static constexpr int MAT = NB * 256;              // elements of a Gram matrix in memory
  static constexpr int EU = DH == 128 ? 2 : 4;                 // workgroups per compute unit (waves per SIMD)
};

// The ring of a stream with VST bytes of start vectors beside each tile.
template <typename T, int DH, int VST>
struct HRing {
  using S = HShape<T, DH>;
  static constexpr int NST = ring_slots(DH, VST);  // slots
  static constexpr int BYTES = NST * (S::STAGE + VST);
};
constexpr int kVKeys = 2048;  // start vectors of a tile: 8 heads (bf16) or 16 (fp32)
constexpr int kVOwn = 1024;   // one head: one load instruction

// What a wave computes: its blocks of G and its row blocks of z0.
template <typename S>
struct Role {
  bool tri, rect;
  int r0, c0;  // triangle: first row block; off-diagonal half: rotation of its rows, first column block
  __device__ __forceinline__ explicit Role(int wv) {
    tri = wv < 2 && wv * S::NR < S::RB;
    rect = wv >= 2 && (S::RB >= 4 || (wv == 2));
    r0 = tri ? wv * S::NR : (wv - 2) * S::NC;
    c0 = S::RB >= 4 ? S::NR + (wv - 2) * S::NC : S::RB - 1;
  }
  // off-diagonal half: row block of its i-th row operand (each of the two
  // waves starts at its own share of z0)
  __device__ __forceinline__ int row(int i) const { return S::RB >= 4 ? (r0 + i) & (S::NR - 1) : 0; }
};

__device__ __forceinline__ void lds_fence() { asm volatile("" ::: "memory"); }
__device__ __forceinline__ void bare_barrier() {
  lds_fence();
  __builtin_amdgcn_s_barrier();
  lds_fence();
}

// At most N vector-memory operations outstanding and every LDS read complete.
template <int N>
__device__ __forceinline__ void wait_vm() {
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | ((N >> 4) << 14));
}

// wait_vm for a wave that requests `own` <= MAX loads per tile (wave-uniform).
template <int NST, int MAX>
__device__ __forceinline__ void wait_ahead(int own) {
  if constexpr (MAX > 0) {
    if (own < MAX) return wait_ahead<NST, MAX - 1>(own);
  }
  wait_vm<outstanding_ahead(NST, MAX)>();
}

// part + the products of one 16-byte chunk of each operand's rows.
template <typename T>
__device__ __forceinline__ f32x4 gram_mfma(const u32x4& a, const u32x4& b, const f32x4& part, int e = 0) {
  if constexpr (sizeof(T) == 2)
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), part, 0,
                                                   0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[e]), __uint_as_float(b[e]), part, 0, 0, 0);
}

__device__ __forceinline__ void add_double(const f32x4& part, double (&total)[4]) {
#pragma unroll
  for (int x = 0; x < 4; ++x) total[x] += (double)part[x];
}

// total += those products.  Every matrix-core instruction (fp32: two of 4
// columns each) starts from zero and its sums are added up in double: what is
// left of the rounding is that within them.
template <typename T>
__device__ __forceinline__ void gram_add(const u32x4& a, const u32x4& b, double (&total)[4]) {
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  if constexpr (sizeof(T) == 2) {
    add_double(gram_mfma<T>(a, b, zero), total);
  } else {
#pragma unroll
    for (int e = 0; e < 4; e += 2) add_double(gram_mfma<T>(a, b, gram_mfma<T>(a, b, zero, e), e + 1), total);
#pragma unroll
    for (int x = 0; x < 4; ++x) asm volatile("" : "+v"(total[x]));  // the additions stay by their products
  }
}

// Zeroes the elements of a 16-byte chunk at positions >= nval.
template <int ES>
__device__ __forceinline__ void mask_chunk(u32x4& x, int nval) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if constexpr (ES == 2)
      x[e] &= (2 * e < nval ? 0x0000ffffu : 0u) | (2 * e + 1 < nval ? 0xffff0000u : 0u);
    else
      x[e] &= e < nval ? 0xffffffffu : 0u;
  }
}

// The start vectors of a key stream: `heads` rows of d floats at `rows`.  Slot
// s of the z0 products is head s / np, part s % np of its bf16 split (fp32
// weights: one part, the vector itself).
struct VSlots {
  const float* rows;
  int heads, np;
};

// Streams tiles t0 .. t1 - 1 of one d_h x d row block through the ring and
// accumulates this wave's blocks of R R^T (GRAM; CHAIN: the sums of about n / 16
// tiles in float, for a G that is rounded to float in the end); with start
// vectors (VST > 0) also its row blocks of z0 and the sums of squares of its
// slot's columns.  The start vectors' columns ride in the ring beside their tile
// (chunk c of head i at slot c ^ vswz(i)), as 16-byte loads where their alignment
// allows, else as 4-byte ones.
template <typename S>
__device__ __forceinline__ int vswz(int i) {
  return S::ES == 2 ? 2 * (i & 7) : i & 7;
}

template <typename T, int DH, int VST, bool GRAM, bool CHAIN = false>
__device__ __forceinline__ void stream_block(const char* blk, int64_t ld, int d, int t0, int t1, uint32_t seed,
                                             uint8_t* ring, int wv, int lane, const Role<HShape<T, DH>>& role,
                                             const VSlots& vs, double (&acc)[HShape<T, DH>::NACC][4],
                                             double (&zacc)[HShape<T, DH>::NZ][4], float& nrm) {
  using S = HShape<T, DH>;
  using R = HRing<T, DH, VST>;
  constexpr bool Z = VST > 0;
  constexpr int OWN = tile_loads(DH, 0);
  const uint32_t nrec = (uint32_t)((((int64_t)(DH - 1) * ld + d) * S::ES + 15) & ~int64_t(15));
  const __amdgpu_buffer_rsrc_t rsrc = make_rsrc(blk, nrec);
  const uint32_t row_bytes = (uint32_t)(ld * S::ES);
  const int q = lane >> 4, s = lane & 15;
  const int n = t1 - t0;
  if (n <= 0) return;
  // whole tiles from a staggered start, as in the sweeps; the ragged last tile
  // of the block (columns past d) comes last, in a copy of the loop body
  const int n_whole = min(t1, d / S::TC) - t0;
  const int rot = n_whole > 0 ? (int)(((seed * 2654435761u) >> 16) % (uint32_t)n_whole) : 0;
  auto tile_at = [&](int i) {
    const int u = rot + i;
    return t0 + (i >= n_whole ? i : u >= n_whole ? u - n_whole : u);
  };
  const int sr = lane >> 3, p = lane & 7;
  uint8_t* vring = ring + R::NST * S::STAGE;
  const __amdgpu_buffer_rsrc_t vrsrc = make_rsrc(vs.rows, Z ? (uint32_t)vs.heads * (uint32_t)d * 4u : 0u);
  const bool vec = (d & 3) == 0 && (reinterpret_cast<uintptr_t>(vs.rows) & 15) == 0;
  const int rpi = vector_rows_per_load(S::ES, vec), nvi = Z ? vector_instructions(S::ES, vec, vs.heads) : 0;
  const int t_own = tile_loads(DH, wv), own = t_own + (Z ? vector_loads(nvi, wv) : 0);
  auto issue = [&](int i) {
    const int slot = i % R::NST, t = tile_at(i);
    if (t_own > 0) {
      uint8_t* dst = ring + slot * S::STAGE;
      const uint32_t col = (uint32_t)t * 128u;
#pragma unroll
      for (int jj = 0; jj < OWN; ++jj) {
        const int j = wv * OWN + jj;
        const uint32_t voff = (uint32_t)sr * row_bytes + col + 16u * (uint32_t)(p ^ stage_swz(8 * j + sr));
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void*)(dst + 1024 * j), 16, voff, 8u * j * row_bytes, 0,
                                                 kStreamPolicy);
      }
    }
    if constexpr (Z) {
      for (int x = vector_first(wv); x < nvi; x += kHWaves) {
        const int ln = vec ? lane : lane >> 2;  // 16-byte slot of this lane within the instruction
        const int row = x * rpi + ln / S::VCH, c = (ln % S::VCH) ^ vswz<S>(row);
        const uint32_t voff = (uint32_t)row * (uint32_t)d * 4u + (uint32_t)t * S::VROW + 16u * (uint32_t)c;
        uint8_t* dst = vring + slot * VST;
        if (vec)
          __builtin_amdgcn_raw_ptr_buffer_load_lds(vrsrc, (lds_void*)(dst + 1024 * x), 16, voff, 0, 0, 0);
        else
          __builtin_amdgcn_raw_ptr_buffer_load_lds(vrsrc, (lds_void*)(dst + 256 * x), 4, voff + 4u * (lane & 3), 0, 0,
                                                   0);
      }
    }
  };

#pragma unroll 1
  for (int i = 0; i < R::NST - 1; ++i)
    if (i < n) issue(i);
  f32x4 cur[CHAIN ? S::NACC : 1] = {};
  const int flush = (n + 15) / 16;
  int left = flush;
  auto add = [&](const u32x4& a, const u32x4& b, int i) {  // the products of block i
    if constexpr (CHAIN) {
      static_assert(S::ES == 2, "bf16 weights");
      cur[i] = gram_mfma<T>(a, b, cur[i]);
    } else {
      gram_add<T>(a, b, acc[i]);
    }
  };
  auto body = [&](int i, auto ragged_tag) {
    constexpr bool RAGGED = decltype(ragged_tag)::value;
    // this wave's part of tile i has landed (the loads of NST - 2 later tiles may be outstanding)
    if (i + R::NST - 2 < n)
      wait_ahead<R::NST, OWN + (Z ? 2 : 0)>(own);
    else
      wait_vm<0>();
    bare_barrier();  // every part of tile i, and tile i - 1 fully read
    if (i + R::NST - 1 < n) issue(i + R::NST - 1);
    const int t = tile_at(i);
    const uint8_t* tile = ring + (i % R::NST) * S::STAGE;
    auto chunk = [&](int rb, int kc) {
      u32x4 x = stage_chunk(tile, 16 * rb + s, 4 * kc + q);
      if constexpr (RAGGED) mask_chunk<S::ES>(x, d - (t * S::TC + (4 * kc + q) * S::VEC));
      return x;
    };
    if (GRAM && role.tri) {
#pragma unroll
      for (int kc = 0; kc < 2; ++kc) {
        u32x4 fr[S::NR];
        if (Z && kc == 1) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int a = 0; a < S::NR; ++a) fr[a] = chunk(role.r0 + a, kc);
#pragma unroll
        for (int a = 0; a < S::NR; ++a)
#pragma unroll
          for (int b = a; b < S::NR; ++b) add(fr[a], fr[b], tri_index<S::NR>(a, b));
      }
    }
    if (role.rect) {
#pragma unroll
      for (int kc = 0; kc < 2; ++kc) {
        u32x4 fa[S::NR], fb[S::NC];
        if (Z && kc == 1) __builtin_amdgcn_sched_barrier(0);  // keeps the two halves' operands from piling up in registers
#pragma unroll
        for (int a = 0; a < S::NR; ++a) fa[a] = chunk(role.row(a), kc);
        if constexpr (S::RB > 1) {
#pragma unroll
          for (int b = 0; b < S::NC; ++b) fb[b] = chunk(role.c0 + b, kc);
          if constexpr (GRAM) {
#pragma unroll
            for (int a = 0; a < S::NR; ++a)
#pragma unroll
              for (int b = 0; b < S::NC; ++b) add(fa[a], fb[b], a * S::NC + b);
          }
        }
        if constexpr (Z) {
          const uint8_t* vt = vring + (i % R::NST) * VST;
          const int head = s / vs.np, part = s % vs.np;
          const int cols = d - (t * S::TC + (4 * kc + q) * S::VEC);  // columns left from this chunk on
          u32x4 bv;
          if constexpr (S::ES == 2) {
            bf16x8 o;
#pragma unroll
            for (int half = 0; half < 2; ++half) {
              const f32x4 y = *reinterpret_cast<const f32x4*>(
                  vt + head * S::VROW + 16 * ((2 * (4 * kc + q) + half) ^ vswz<S>(head)));
              const float x4[4] = {y[0], y[1], y[2], y[3]};
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const float x = !RAGGED || 4 * half + e < cols ? x4[e] : 0.f;
                nrm = fmaf(x, x, nrm);
                const __bf16 h0 = (__bf16)x;
                const float x1 = x - (float)h0;
                const __bf16 h1 = (__bf16)x1;
                const __bf16 h2 = (__bf16)(x1 - (float)h1);
                o[4 * half + e] = part == 0 ? h0 : part == 1 ? h1 : h2;
              }
            }
            bv = __builtin_bit_cast(u32x4, o);
          } else {
            const f32x4 y =
                *reinterpret_cast<const f32x4*>(vt + head * S::VROW + 16 * ((4 * kc + q) ^ vswz<S>(head)));
            const float x4[4] = {y[0], y[1], y[2], y[3]};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float x = !RAGGED || e < cols ? x4[e] : 0.f;
              nrm = fmaf(x, x, nrm);
              bv[e] = __float_as_uint(x);
            }
          }
#pragma unroll
          for (int a = 0; a < S::NC; ++a) gram_add<T>(fa[a], bv, zacc[a]);
          if constexpr (S::RB > 1) {
#pragma unroll
            for (int b = 0; b < S::NC; ++b) gram_add<T>(fb[b], bv, zacc[S::NC + b]);
          }
        }
      }
    }
    if constexpr (CHAIN) {
      if (--left == 0 || i + 1 == n) {
        left = flush;
#pragma unroll
        for (int x = 0; x < S::NACC; ++x) {
          add_double(cur[x], acc[x]);
          cur[x] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
      }
    }
  };
#pragma unroll 1
  for (int i = 0; i < n_whole; ++i) body(i, std::false_type{});
  if (n_whole < n) body(n - 1, std::true_type{});
  __syncthreads();  // the ring is free again
}

// Row block of zacc[i] in wave wv.
template <typename S>
__device__ __forceinline__ int z_row_block(const Role<S>& role, int i) {
  return i < S::NC ? role.row(i) : role.c0 + i - S::NC;
}

// This wave's blocks of G into the whole symmetric matrix gl (LDS, pitch P).
template <typename T, int DH, typename N>
__device__ __forceinline__ void blocks_to_lds(const Role<HShape<T, DH>>& role,
                                              const double (&acc)[HShape<T, DH>::NACC][4], N* gl, int lane) {
  using S = HShape<T, DH>;
  const int q = lane >> 4, s = lane & 15;
  auto put = [&](int bi, int bj, int i, bool mirror) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = 16 * bi + 4 * q + e, c = 16 * bj + s;
      gl[r * S::P + c] = (N)acc[i][e];
      if (mirror) gl[c * S::P + r] = (N)acc[i][e];
    }
  };
  if (role.tri) {
#pragma unroll
    for (int a = 0; a < S::NR; ++a)
#pragma unroll
      for (int b = a; b < S::NR; ++b) put(role.r0 + a, role.r0 + b, tri_index<S::NR>(a, b), a != b);
  } else if (S::RB > 1 && role.rect) {
#pragma unroll
    for (int a = 0; a < S::NR; ++a)
#pragma unroll
      for (int b = 0; b < S::NC; ++b) put(role.row(a), role.c0 + b, a * S::NC + b, true);
  }
}

// A Gram matrix in the registers of the workgroup.  I_ROWS: TPR threads take one
// row, thread t = TPR R + C columns 2 C + 2 TPR j and their right neighbours (d_h
// 16: column C).  I_HALVES: thread t = 16 R + C rows 8 R .. + 7 and columns C, C +
// 16, ..  I_BLOCKS: each wave its blocks (36 of 64: G is symmetric), as they left
// the matrix cores, a lane's four elements of a block in the order e ^ (s mod 4);
// whole rows of doubles would not fit.
template <typename T, int DH, int MODE>
struct Iter {
  using S = HShape<T, DH>;
  static constexpr bool BLOCKS = MODE == I_BLOCKS;
  using Num = std::conditional_t<MODE == I_HALVES, float, double>;
  static constexpr int TPR = BLOCKS ? 1 : MODE == I_HALVES ? 16 : kHThreads / DH;  // threads per row of a product
  static constexpr int ROWS = MODE == I_HALVES ? DH / 16 : 1, COLS = DH / TPR;
  using Mat = std::conditional_t<BLOCKS, double[S::NACC][4], Num[ROWS][BLOCKS ? 1 : COLS]>;
  // LDS bytes of a whole G, or of a product's partials
  static constexpr int GL = BLOCKS ? 4 * DH * 8 : DH * S::P * (int)sizeof(Num);
  __device__ static __forceinline__ int col(int C, int j) {
    return MODE == I_HALVES ? C + 16 * j : COLS > 1 ? 2 * C + 2 * TPR * (j >> 1) + (j & 1) : C;
  }
};

// This thread's part of the whole matrix in gl; thread t < DH also takes its
// diagonal element.
template <typename T, int DH, int MODE>
__device__ __forceinline__ void lds_to_regs(const typename Iter<T, DH, MODE>::Num* gl, float* diag,
                                            typename Iter<T, DH, MODE>::Mat& reg) {
  using I = Iter<T, DH, MODE>;
  constexpr int P = DH + 1;
  const int t = threadIdx.x, R = t / I::TPR, C = t % I::TPR;
  if (t < DH) diag[t] = (float)gl[t * P + t];
#pragma unroll
  for (int i = 0; i < I::ROWS; ++i)
#pragma unroll
    for (int j = 0; j < I::COLS; ++j) reg[i][j] = gl[(I::ROWS * R + i) * P + I::col(C, j)];
  __syncthreads();  // gl is read out
}

// The diagonal of the matrix whose blocks the waves hold, and each lane's order of
// a block's elements (I_BLOCKS).
template <typename S>
__device__ __forceinline__ void blocks_diag(const Role<S>& role, double (&g)[S::NACC][4], float* diag, int lane) {
  const int q = lane >> 4, s = lane & 15;
  const bool b0 = s & 1, b1 = s & 2;
#pragma unroll
  for (int i = 0; i < S::NACC; ++i) {
    const double y[4] = {b0 ? g[i][1] : g[i][0], b0 ? g[i][0] : g[i][1], b0 ? g[i][3] : g[i][2], b0 ? g[i][2] : g[i][3]};
#pragma unroll
    for (int e = 0; e < 4; ++e) g[i][e] = b1 ? y[e ^ 2] : y[e];
  }
  if (role.tri && (s >> 2) == q) {
#pragma unroll
    for (int a = 0; a < S::NR; ++a) diag[16 * (role.r0 + a) + s] = (float)g[tri_index<S::NR>(a, a)][0];
  }
  __syncthreads();
}

// keep + (give of the lane that CTRL names)
template <int CTRL>
__device__ __forceinline__ double dpp_take(double keep, double give) {
  const uint64_t b = __builtin_bit_cast(uint64_t, give);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xF, 0xF, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xF, 0xF, true);
  return keep + __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
template <int CTRL>
__device__ __forceinline__ double dpp_add(double x) {
  return dpp_take<CTRL>(x, x);
}

// Where lane s of a DPP row holds y[j] of row j ^ (s mod 4): the sum of row s mod
// 4 over the 16 lanes.  Each of the first two steps halves what a lane carries.
__device__ __forceinline__ double row16_sums_of_4(const double (&y)[4]) {
  double x = dpp_take<0x4E>(dpp_take<0xB1>(y[0], y[1]), dpp_take<0xB1>(y[2], y[3]));
  x = dpp_add<0x128>(x);  // rotations by 8 and 4 keep s mod 4
  return dpp_add<0x124>(x);
}

// Sum over the four lanes s, s + 16, s + 32, s + 48.
__device__ __forceinline__ double rows4_sum(double x) {
  // swapped with itself, a register gives both halves (rows) everywhere
  auto swap_sum = [](double x, auto swap) {
    const uint64_t b = __builtin_bit_cast(uint64_t, x);
    const auto lo = swap((uint32_t)b), hi = swap((uint32_t)(b >> 32));
    return __builtin_bit_cast(double, (uint64_t)hi[0] << 32 | lo[0]) +
           __builtin_bit_cast(double, (uint64_t)hi[1] << 32 | lo[1]);
  };
  x = swap_sum(x, [](uint32_t r) { return __builtin_amdgcn_permlane16_swap(r, r, false, false); });
  return swap_sum(x, [](uint32_t r) { return __builtin_amdgcn_permlane32_swap(r, r, false, false); });
}

// out: this thread's rows of G x, for x in LDS.  I_ROWS and I_HALVES: complete in
// every thread of a row.  I_BLOCKS: row t in thread t < d_h, with one barrier
// inside; each block G_IJ off the diagonal gives to the rows of I and, transposed,
// to those of J, and the waves' partials meet in pp[4][DH], of which the places
// that no wave writes are zero.
template <typename T, int DH, int MODE>
__device__ __forceinline__ void product(const typename Iter<T, DH, MODE>::Mat& g,
                                        const typename Iter<T, DH, MODE>::Num* x, double* pp,
                                        const Role<HShape<T, DH>>& role, int wv, int lane,
                                        typename Iter<T, DH, MODE>::Num (&out)[Iter<T, DH, MODE>::ROWS]) {
  using S = HShape<T, DH>;
  using I = Iter<T, DH, MODE>;
  if constexpr (MODE == I_HALVES) {
    const int C = threadIdx.x % I::TPR;
    float xv[I::COLS];
#pragma unroll
    for (int j = 0; j < I::COLS; ++j) xv[j] = x[I::col(C, j)];
#pragma unroll
    for (int i = 0; i < I::ROWS; ++i) {
      float a = 0.f;
#pragma unroll
      for (int j = 0; j < I::COLS; ++j) a = fmaf(g[i][j], xv[j], a);
      out[i] = row16_sum(a);
    }
  } else if constexpr (MODE == I_ROWS) {
    const int C = threadIdx.x % I::TPR;
    double a0 = 0., a1 = 0.;
#pragma unroll
    for (int j = 0; j < I::COLS; j += 2) {
      a0 = fma(g[0][j], x[I::col(C, j)], a0);
      if constexpr (I::COLS > 1) a1 = fma(g[0][j + 1], x[I::col(C, j + 1)], a1);
    }
    double a = a0 + a1;  // the steps of row16_sum, as many as TPR lanes take
    a = dpp_add<0xB1>(a);
    a = dpp_add<0x4E>(a);
    if constexpr (I::TPR > 4) a = dpp_add<0x141>(a);
    if constexpr (I::TPR > 8) a = dpp_add<0x140>(a);
    out[0] = a;
  } else {
    asm volatile("" : "+v"(lane));  // addresses formed here, not kept in registers across the iteration
    const int q = lane >> 4, s = lane & 15;
    auto rows_of = [&](int bi, double (&xr)[4]) {
#pragma unroll
      for (int e = 0; e < 4; ++e) xr[e] = x[16 * bi + 4 * q + (e ^ (s & 3))];
    };
    if (role.tri) {  // pp[0]: row sums, pp[1]: column sums
      double yc[S::NR] = {};
#pragma unroll
      for (int a = 0; a < S::NR; ++a) {
        double xr[4], yr[4] = {};
        rows_of(role.r0 + a, xr);
#pragma unroll
        for (int b = a; b < S::NR; ++b) {
          const double xc = x[16 * (role.r0 + b) + s];
          const double(&m)[4] = g[tri_index<S::NR>(a, b)];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            yr[e] = fma(m[e], xc, yr[e]);
            if (b > a) yc[b] = fma(m[e], xr[e], yc[b]);
          }
        }
        const double y = row16_sums_of_4(yr);
        if (s < 4) pp[16 * (role.r0 + a) + 4 * q + s] = y;
      }
#pragma unroll
      for (int b = 1; b < S::NR; ++b) {
        const double y = rows4_sum(yc[b]);
        if (q == b) pp[DH + 16 * (role.r0 + b) + s] = y;
      }
    } else {  // pp[2], pp[3]: row sums of waves 2 and 3; their column sums lie in the other half of pp[2]
      double yc[S::NC] = {};
#pragma unroll
      for (int a = 0; a < S::NR; ++a) {
        double xr[4], yr[4] = {};
        rows_of(role.row(a), xr);
#pragma unroll
        for (int b = 0; b < S::NC; ++b) {
          const double xc = x[16 * (role.c0 + b) + s];
          const double(&m)[4] = g[a * S::NC + b];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            yr[e] = fma(m[e], xc, yr[e]);
            yc[b] = fma(m[e], xr[e], yc[b]);
          }
        }
        const double y = row16_sums_of_4(yr);
        if (s < 4) pp[wv * DH + 16 * role.row(a) + 4 * q + s] = y;
      }
#pragma unroll
      for (int b = 0; b < S::NC; ++b) {
        const double y = rows4_sum(yc[b]);
        if (q == b) pp[2 * DH + 16 * (role.c0 + b) + s] = y;
      }
    }
    __syncthreads();
    const int t = threadIdx.x;
    out[0] = t < DH ? (pp[t] + pp[DH + t]) + (pp[2 * DH + t] + pp[3 * DH + t]) : 0.;
  }
}

template <int CTRL>
__device__ __forceinline__ float dpp_take(float keep, float give) {
  return keep + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, give), CTRL, 0xF, 0xF, true));
}

// Sum over the lanes of a wave that are equal mod MOD (4, 8 or 16).
template <int MOD>
__device__ __forceinline__ float lanes_sum(float x) {
  if constexpr (MOD < 16) x = dpp_take<0x128>(x, x);  // rotations by 8 and 4
  if constexpr (MOD < 8) x = dpp_take<0x124>(x, x);
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// One pass over a d_h x d row block R by the workgroup: w = R^T x, out = R w
// (unnormalised, in LDS) and ||w||^2, as in a fused sweep.  x, out and part
// are LDS arrays of d_h, d_h and kHWaves * d_h floats.  What a head that
// cannot be iterated in d_h-space costs: with every head such a one, 20 steps
// against the sweeps, 70B GQA shape 67 vs 36 ms (each query head reads its own K_j),
// Llama-2-7B 7.3 vs 7.1 ms, GPT-2 small 0.33 vs 0.42 ms, 8 heads of d 8192, d_h
// 128 1.83 vs 0.93 ms (2.72 without the loads one tile ahead; one workgroup draws
// about 45 GB/s).
template <typename T, int DH>
__device__ __forceinline__ float direct_sweep(const char* blk, int64_t ld, int d, const float* x, float* out,
                                              float* part, float* npart, int wv, int lane) {
  using S = HShape<T, DH>;
  constexpr int RPL = DH / kRG;
  const uint32_t nrec = (uint32_t)((((int64_t)(DH - 1) * ld + d) * S::ES + 15) & ~int64_t(15));
  const __amdgpu_buffer_rsrc_t rsrc = make_rsrc(blk, nrec);
  const uint32_t row_bytes = (uint32_t)(ld * S::ES);
  const int chunk = lane & 7, rg = lane >> 3;
  const int n = (d + S::TC - 1) / S::TC, n_full = d / S::TC;
  const uint32_t lane_off = (uint32_t)(((int64_t)rg * RPL * ld + chunk * S::VEC) * S::ES);
  float xr[RPL], acc[RPL], nrm = 0.f;
#pragma unroll
  for (int rr = 0; rr < RPL; ++rr) {
    xr[rr] = x[rg * RPL + rr];
    acc[rr] = 0.f;
  }
  auto load = [&](u32x4 (&tile)[RPL], int t) {  // past the last tile: later rows or zeros, never used
#pragma unroll
    for (int rr = 0; rr < RPL; ++rr)
      tile[rr] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, lane_off + (uint32_t)t * 128u, rr * row_bytes, kStreamPolicy);
  };
  u32x4 next[RPL];
  load(next, wv);
#pragma unroll 1
  for (int t = wv; t < n; t += kHWaves) {
    u32x4 tile[RPL];
#pragma unroll
    for (int rr = 0; rr < RPL; ++rr) tile[rr] = next[rr];
    load(next, t + kHWaves);  // in flight while this tile is multiplied
    __builtin_amdgcn_sched_barrier(0);
    if (t >= n_full) {
#pragma unroll
      for (int rr = 0; rr < RPL; ++rr) mask_chunk<S::ES>(tile[rr], d - (t * S::TC + chunk * S::VEC));
    }
    float w[S::VEC];
#pragma unroll
    for (int c = 0; c < S::VEC; ++c) w[c] = 0.f;
#pragma unroll
    for (int rr = 0; rr < RPL; ++rr)
#pragma unroll
      for (int c = 0; c < S::VEC; ++c) w[c] = fmaf(elem<T>(tile[rr], c), xr[rr], w[c]);
#pragma unroll
    for (int rr = 0; rr < RPL; ++rr) reuse_fence(tile[rr]);
#pragma unroll
    for (int c = 0; c < S::VEC; ++c) {
      w[c] = group_sum(w[c]);
      nrm = fmaf(w[c], w[c], nrm);
    }
#pragma unroll
    for (int rr = 0; rr < RPL; ++rr)
#pragma unroll
      for (int c = 0; c < S::VEC; ++c) acc[rr] = fmaf(elem<T>(tile[rr], c), w[c], acc[rr]);
  }
#pragma unroll
  for (int m = 1; m < 8; m <<= 1) nrm = xor_sum(nrm, m);
  if (lane == 0) npart[wv] = nrm;
#pragma unroll
  for (int rr = 0; rr < RPL; ++rr) {
    float a = acc[rr];
#pragma unroll
    for (int m = 1; m < 8; m <<= 1) a = xor_sum(a, m);
    if ((rr & 7) == chunk) part[wv * DH + rg * RPL + rr] = a;
  }
  __syncthreads();
  if ((int)threadIdx.x < DH) {
    float a = 0.f;
#pragma unroll
    for (int w = 0; w < kHWaves; ++w) a += part[w * DH + threadIdx.x];
    out[threadIdx.x] = a;
  }
  const float n2 = sum_waves<kHWaves>(npart);
  __syncthreads();
  return n2;
}

// Sums the parts of each head's z0 slot (slots of head i: i np .. + np - 1)
// from zacc through LDS (16 slots x d_h doubles at zl) and the squared norms of
// the start vectors into nv[0 .. 16).
template <typename T, int DH>
__device__ __forceinline__ void z0_to_lds(const Role<HShape<T, DH>>& role, const double (&zacc)[HShape<T, DH>::NZ][4],
                                          float nrm, int wv, int lane, int np, double* zl, float* nv) {
  using S = HShape<T, DH>;
  const int q = lane >> 4, s = lane & 15;
  if (role.rect) {
#pragma unroll
    for (int i = 0; i < S::NZ; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) zl[s * DH + 16 * z_row_block(role, i) + 4 * q + e] = zacc[i][e];
  }
  if (wv == 2) {  // both z0 waves read every column; the q lanes of a slot hold disjoint ones
    nrm += __shfl_xor(nrm, 16);
    nrm += __shfl_xor(nrm, 32);
    if (q == 0 && s % np == 0) nv[s / np] = nrm;
  }
  __syncthreads();
}

// f(block of the upper triangle, index into the wave's accumulators) for each of
// the wave's blocks.  The index is the same in every wave, so that the
// accumulators stay in registers.
template <typename T, int DH, typename F>
__device__ __forceinline__ void each_block(const Role<HShape<T, DH>>& role, F&& f) {
  using S = HShape<T, DH>;
#pragma unroll
  for (int x = 0; x < S::NR; ++x)
#pragma unroll
    for (int y = x; y < S::NR; ++y) {
      const int i = tri_index<S::NR>(x, y);
      const bool in_rect = S::RB > 1 && i < S::NR * S::NC && role.rect;
      if (role.tri || in_rect)
        f(role.tri ? tri_index<S::RB>(role.r0 + x, role.r0 + y)
                   : tri_index<S::RB>(role.row(i / S::NC), role.c0 + i % S::NC),
          i);
    }
  static_assert(S::NTRI >= S::NR * S::NC, "the triangle's indices cover the other half's");
}

// This wave's blocks of G to memory, in the block order and lane layout of
// tri_index and the matrix-core output.
template <typename T, int DH>
__device__ __forceinline__ void blocks_to_memory(const Role<HShape<T, DH>>& role,
                                                 const double (&acc)[HShape<T, DH>::NACC][4], double* dst, int lane) {
  each_block<T, DH>(role, [&](int b, int i) {
    double* out = dst + (b * 64 + lane) * 4;
#pragma unroll
    for (int e = 0; e < 4; ++e) out[e] = acc[i][e];
  });
}

// The sum of `strips` Gram matrices written by blocks_to_memory: this wave's
// blocks of it (d_h 128), or a whole symmetric matrix in LDS.
template <typename T, int DH>
__device__ __forceinline__ void memory_to_blocks(const Role<HShape<T, DH>>& role, const double* src, int strips,
                                                 double (&g)[HShape<T, DH>::NACC][4], int lane) {
  using S = HShape<T, DH>;
  each_block<T, DH>(role, [&](int b, int i) {
    const double* in = src + (b * 64 + lane) * 4;
#pragma unroll
    for (int e = 0; e < 4; ++e) g[i][e] = in[e];
  });
#pragma unroll 1
  for (int st = 1; st < strips; ++st) {
    each_block<T, DH>(role, [&](int b, int i) {
      const double* in = src + (size_t)st * S::MAT + (b * 64 + lane) * 4;
#pragma unroll
      for (int e = 0; e < 4; ++e) g[i][e] += in[e];
    });
  }
}
template <typename T, int DH, typename N>
__device__ __forceinline__ void memory_to_lds(const double* src, int strips, N* gl) {
  using S = HShape<T, DH>;
  for (int x = threadIdx.x; x < S::NB * 64; x += kHThreads) {
    const int b = x >> 6, ln = x & 63;
    int bi = 0, start = 0;
    while (b >= start + (S::RB - bi)) {  // upper-triangle block b -> (bi, bj)
      start += S::RB - bi;
      ++bi;
    }
    const int bj = bi + (b - start);
    double y[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = src[x * 4 + e];
#pragma unroll 4
    for (int st = 1; st < strips; ++st) {
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e] += src[(size_t)st * S::MAT + x * 4 + e];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = 16 * bi + 4 * (ln >> 4) + e, c = 16 * bj + (ln & 15);
      gl[r * S::P + c] = (N)y[e];
      if (bi != bj) gl[c * S::P + r] = (N)y[e];
    }
  }
  __syncthreads();
}

// Where a head's (or key head and chunk's) strip starts in its tiles: by its
// place in the model, not in the launch, so that the order of its sums does not
// depend on how many key heads a launch pair covers.
__device__ __forceinline__ uint32_t tile_seed(int head, int strips, int strip) {
  return (uint32_t)head * (uint32_t)strips + (uint32_t)strip;
}

// Items: (key head, chunk of query heads, column strip) for the key heads of
// the launch, then (query head, column strip) where the query matrices are
// split over workgroups too (a.sq > 0).
template <typename T, int DH>
__global__ void __launch_bounds__(kHThreads) __attribute__((amdgpu_waves_per_eu(HShape<T, DH>::EU)))
units_kernel(HeadArgs a) {
  using S = HShape<T, DH>;
  constexpr int RING = HRing<T, DH, kVKeys>::BYTES > HRing<T, DH, 0>::BYTES ? HRing<T, DH, kVKeys>::BYTES
                                                                            : HRing<T, DH, 0>::BYTES;
  static_assert(RING >= 16 * DH * 8, "the z0 slots fit the ring");
  __shared__ __attribute__((aligned(16))) uint8_t big[RING];
  __shared__ float nv[16];
  const int lane = threadIdx.x & 63, wv = uni((int)(threadIdx.x >> 6));
  const Role<S> role(wv);
  const int n_tiles = (a.d + S::TC - 1) / S::TC;
  double acc[S::NACC][4] = {}, zacc[S::NZ][4] = {};
  float nrm = 0.f;
  const int item = blockIdx.x, n_key = a.units * a.nch * a.sk;
  if (item >= n_key) {
    const int hl = (item - n_key) / a.sq, strip = (item - n_key) % a.sq;
    const int h = a.head0 + hl;
    const char* blk = uni(a.mats[h / a.n_q]) + (int64_t)(h % a.n_q) * DH * a.ld * S::ES;
    const int t0 = strip * a.tps_q, t1 = min(t0 + a.tps_q, n_tiles);
    stream_block<T, DH, 0, true>(blk, a.ld, a.d, t0, t1, tile_seed(h, a.sq, strip), big, wv, lane, role, VSlots{nullptr, 0, 1},
                                 acc, zacc, nrm);
    blocks_to_memory<T, DH>(role, acc, a.gq + (size_t)(hl * a.sq + strip) * S::MAT, lane);
    return;
  }
  const int strip = item % a.sk, ch = item / a.sk % a.nch, ul = item / (a.sk * a.nch);
  const int unit = a.unit0 + ul, layer = unit / a.n_kv, j = unit % a.n_kv;
  const int hin = ch * a.hps, nvalid = min(a.hps, a.g - hin);
  const int h0 = ul * a.g + hin;  // first query head, counted from the launch's
  const char* blk = uni(a.mats[a.L + layer]) + (int64_t)j * DH * a.ld * S::ES;
  const VSlots vs{a.v + (size_t)(a.head0 + h0) * a.d, nvalid, a.np};
  const int t0 = strip * a.tps_k, t1 = min(t0 + a.tps_k, n_tiles);
  const uint32_t seed = tile_seed(unit * a.nch + ch, a.sk, strip);
  if (ch == 0) {
    stream_block<T, DH, kVKeys, true>(blk, a.ld, a.d, t0, t1, seed, big, wv, lane, role, vs, acc, zacc, nrm);
    blocks_to_memory<T, DH>(role, acc, a.gk + (size_t)(ul * a.sk + strip) * S::MAT, lane);
  } else {
    stream_block<T, DH, kVKeys, false>(blk, a.ld, a.d, t0, t1, seed, big, wv, lane, role, vs, acc, zacc, nrm);
  }
  double* zl = reinterpret_cast<double*>(big);
  z0_to_lds<T, DH>(role, zacc, nrm, wv, lane, a.np, zl, nv);
  for (int x = threadIdx.x; x < nvalid * DH; x += kHThreads) {
    const int i = x / DH, r = x % DH;
    double z = 0.;
    for (int p = 0; p < a.np; ++p) z += zl[(i * a.np + p) * DH + r];
    const size_t o = (size_t)(h0 + i) * a.sk + strip;
    a.zp[o * DH + r] = (float)z;
    if (r == 0) a.zn[o] = nv[i];
  }
}

// SRC: where a head's Gram matrices come from.  H_OWN (g = 1): the workgroup
// streams K_h, then Q_h.  H_KEYS: G_K and z0 from units_kernel, Q_h streamed
// here.  H_SPLIT: both from units_kernel.
enum { H_OWN = 0, H_KEYS = 1, H_SPLIT = 2 };

template <typename T, int DH, int SRC, int MODE>
__global__ void __launch_bounds__(kHThreads) __attribute__((amdgpu_waves_per_eu(HShape<T, DH>::EU)))
heads_kernel(HeadArgs a) {
  using S = HShape<T, DH>;
  using I = Iter<T, DH, MODE>;
  using Num = typename I::Num;
  constexpr int RING0 = HRing<T, DH, 0>::BYTES, RINGV = HRing<T, DH, kVOwn>::BYTES;
  constexpr int RING = SRC == H_SPLIT ? 0 : SRC == H_OWN && RINGV > RING0 ? RINGV : RING0;
  __shared__ __attribute__((aligned(16))) uint8_t big[RING > I::GL ? RING : I::GL];
  __shared__ float z0[DH], tb[DH], wb[DH], dq[DH], dk[DH], nv[16], red[2][3][kHWaves];
  __shared__ __attribute__((aligned(16))) Num vec[2][DH];
  Num *tv = vec[0], *yv = vec[1];  // the iteration's t and w (last step: y)
  Num* gl = reinterpret_cast<Num*>(big);
  double* pp = reinterpret_cast<double*>(big);
  const int t = threadIdx.x, lane = t & 63, wv = uni(t >> 6);
  const bool own = I::BLOCKS ? t < DH : t % I::TPR == 0;  // has rows row0 .. of a product
  const int row0 = I::BLOCKS ? t : I::ROWS * (t / I::TPR);
  const int hl = blockIdx.x, h = a.head0 + hl;
  const int layer = h / a.n_q, hq = h % a.n_q, j = hq / a.g;
  const char* qblk = uni(a.mats[layer]) + (int64_t)hq * DH * a.ld * S::ES;
  const char* kblk = uni(a.mats[a.L + layer]) + (int64_t)j * DH * a.ld * S::ES;
  const int n_tiles = (a.d + S::TC - 1) / S::TC;
  const Role<S> role(wv);
  double acc[S::NACC][4], zacc[S::NZ][4];
  typename I::Mat gq, gk;
  float nrm = 0.f, n2v = 0.f;
  double zr = 0.;  // ||v||^2 and, in thread r < d_h, z0[r] ||v||
  auto clear = [](auto& m) {
#pragma unroll
    for (auto& b : m)
#pragma unroll
      for (double& x : b) x = 0.;
  };
  // the matrix whose blocks acc holds, in registers, and its diagonal
  auto take = [&](typename I::Mat& g, float* diag) {
    if constexpr (!I::BLOCKS) {
      blocks_to_lds<T, DH>(role, acc, gl, lane);
      __syncthreads();
      lds_to_regs<T, DH, MODE>(gl, diag, g);
    } else {
#pragma unroll
      for (int i = 0; i < S::NACC; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) g[i][e] = acc[i][e];
      blocks_diag<S>(role, g, diag, lane);
    }
  };
  auto load = [&](const double* src, int strips, typename I::Mat& g, float* diag) {
    if constexpr (!I::BLOCKS) {
      memory_to_lds<T, DH>(src, strips, gl);
      lds_to_regs<T, DH, MODE>(gl, diag, g);
    } else {
      memory_to_blocks<T, DH>(role, src, strips, g, lane);
      blocks_diag<S>(role, g, diag, lane);
    }
  };
  if constexpr (SRC == H_OWN) {
    clear(zacc);
    clear(acc);
    stream_block<T, DH, kVOwn, true>(kblk, a.ld, a.d, 0, n_tiles, tile_seed(h, 1, 0), big, wv, lane, role,
                                     VSlots{a.v + (size_t)h * a.d, 1, a.np}, acc, zacc, nrm);
    z0_to_lds<T, DH>(role, zacc, nrm, wv, lane, a.np, pp, nv);
    n2v = nv[0];
    if (t < DH)
      for (int p = 0; p < a.np; ++p) zr += pp[p * DH + t];
    __syncthreads();
    take(gk, dk);
  } else {
    for (int st = 0; st < a.sk; ++st) n2v += a.zn[(size_t)hl * a.sk + st];
    if (t < DH)
      for (int st = 0; st < a.sk; ++st) zr += (double)a.zp[((size_t)hl * a.sk + st) * DH + t];
  }
  const float vn = sqrtf(n2v);
  if (t == 0) a.w.vnorm0[h] = vn;
  if (!(vn > 0.f) || !isfinite(vn)) {  // zero or non-finite start vector
    if (t == 0) {
      a.sigma[h] = __builtin_nanf("");
      a.iters[h] = -1;
    }
    return;
  }
  zr /= (double)vn;
  if (t < DH) z0[t] = (float)zr;
  if constexpr (SRC != H_SPLIT) {
    clear(acc);
    stream_block<T, DH, 0, true, MODE == I_HALVES>(qblk, a.ld, a.d, 0, n_tiles, tile_seed(h, 1, 0), big, wv, lane, role,
                                 VSlots{nullptr, 0, 1}, acc, zacc, nrm);
    take(gq, dq);
  } else {
    load(a.gq + (size_t)hl * a.sq * S::MAT, a.sq, gq, dq);
  }
  if constexpr (SRC != H_OWN)
    load(a.gk + (size_t)(layer * a.n_kv + j - a.unit0) * a.sk * S::MAT, a.sk, gk, dk);

  // The iteration runs on G_Q / fq^2 and G_K / fk^2, fq and fk powers of two
  // that take the traces (trq, trk) to [1, 4): its values then stay in range
  // whatever the weights' size.
  auto scale_of = [&](const float* diag, float* f, float* tr) {
    float x = diag[lane % DH];
    if constexpr (DH > 64) x += diag[lane + 64];
    const float sum = c0_lanes_sum(row16_sum(x)) * (DH < 64 ? DH / 64.f : 1.f);
    *f = 1.f;
    if (!(sum >= kGramMin && sum <= kGramMax)) return false;
    const int e = ilogbf(sum) >> 1;
    *f = ldexpf(1.f, e);
    *tr = ldexpf(sum, -2 * e);
    return true;
  };
  float fq, fk, trq = 0.f, trk = 0.f;
  bool in_range = scale_of(dq, &fq, &trq);
  in_range = scale_of(dk, &fk, &trk) && in_range;

  float* fin = a.w.fin + (size_t)h * 2 * DH;
  auto finish = [&](int k, float sig, const auto* z, float zs, const auto* y, float ys, float rn) {
    if (t < DH) {
      fin[t] = (float)(z[t] * zs);
      fin[DH + t] = a.round_y ? (float)(y[t] * ys) : (float)(y[t] * ys * rn);
    }
    if (t == 0) {
      a.sigma[h] = sig;
      a.iters[h] = k;
      a.w.sig[h] = rn;  // read by the final W_K sweep with round_y
    }
  };
  // y = w / sigma of the last step, in place; with round_y as the final W_K
  // sweep will take it, so that ||K^T y|| is the norm of what that sweep writes
  auto last_y = [&](auto* w, float inv) {
    if (t < DH) {
      const float y = (float)(w[t] * inv);
      const float hi = (float)(__bf16)y;
      w[t] = a.round_y ? hi + (float)(__bf16)(y - hi) : y;
    }
    __syncthreads();
  };
  auto stop = [&](int k, float sig, float prev) {
    return k >= a.n_iter || (a.tol > 0.f && k >= 2 && fabsf(sig - prev) <= a.tol * sig);
  };

  if (in_range) {
    const Num sq = (Num)1 / ((Num)fq * (Num)fq), sk = (Num)1 / ((Num)fk * (Num)fk);
#pragma unroll
    for (auto& b : gq)
#pragma unroll
      for (Num& x : b) x *= sq;
#pragma unroll
    for (auto& b : gk)
#pragma unroll
      for (Num& x : b) x *= sk;
    // Three sums over the rows follow each product: z^T w (lanes with C mod 4 = 0),
    // the rounding bound z_i^2 G_ii (1) and w^2 (2), each lane adding up its own.
    const int c = lane & 3;
    float dqr[I::ROWS], dkr[I::ROWS];
#pragma unroll
    for (int i = 0; i < I::ROWS; ++i) {
      const bool mine = I::BLOCKS ? t < DH : c == 1;
      dqr[i] = mine ? fmaxf(dq[row0 + i] * (float)sq, kTinyRow) : 1.f;
      dkr[i] = mine ? fmaxf(dk[row0 + i] * (float)sk, kTinyRow) : 1.f;
    }
    if (t < DH) tv[t] = (Num)(zr / fk);
    if constexpr (I::BLOCKS) {
      for (int i = t; i < 4 * DH; i += kHThreads) pp[i] = 0.;
    }
    __syncthreads();
    float prev = 0.f, zscale = 1.f;
    Num out[I::ROWS];
    // After a product out of the vector x (LDS), both times `by`: its rows to y
    // (unless null), and the sums over the wave's rows.
    auto sums = [&](int to, const Num* x, Num* y, float by, const float (&diag)[I::ROWS]) {
      float sum = 0.f;
      if constexpr (I::BLOCKS) {
        if (own) {
          const Num w = out[0] * by, z = x[row0] * by;
          const float wf = (float)w, zf = (float)z;
          const float v[3] = {zf * wf, zf * zf * diag[0], wf * wf};
          // v[j ^ c] at j, so that a lane keeps v[c] and gives the others away
          const bool b0 = c & 1, b1 = c & 2;
          const float p[4] = {b0 ? v[1] : v[0], b0 ? v[0] : v[1], b0 ? 0.f : v[2], b0 ? v[2] : 0.f};
          const float lo = dpp_take<0xB1>(b1 ? p[2] : p[0], b1 ? p[3] : p[1]);
          const float hi = dpp_take<0xB1>(b1 ? p[0] : p[2], b1 ? p[1] : p[3]);
          sum = dpp_take<0x4E>(lo, hi);
          if (y) y[row0] = w;
        }
        sum = lanes_sum<4>(sum);
      } else {
#pragma unroll
        for (int i = 0; i < I::ROWS; ++i) {
          const Num w = out[i] * by, z = x[row0 + i] * by;
          const float wf = (float)w, zf = (float)z;
          sum = fmaf((c == 2 ? wf : zf) * diag[i], c == 1 ? zf : wf, sum);
          if (own && y) y[row0 + i] = w;
        }
        sum = lanes_sum<I::TPR>(sum);
      }
      if (lane < 3) red[to][lane][wv] = sum;
    };
    auto dot_of = [&](int from) { return sum_waves<kHWaves>(red[from][0]); };
    // Adds what the product just summed up counts (see kCancelMean); its bound b.
    float cancel = 0.f;
    auto weigh = [&](int from, float tr, float dot) {
      const float bound = sum_waves<kHWaves>(red[from][1]), ww = sum_waves<kHWaves>(red[from][2]);
      const float x = bound * __builtin_amdgcn_rcpf(dot);
      cancel += fminf(x * x, bound * tr * __builtin_amdgcn_rcpf(DH * ww));
      return bound;
    };
    // Each product is formed on the unscaled vector before the sums of the
    // step that made it are looked at: their way through LDS, the square root
    // and the division run beside it.  In steps that cannot be the last only
    // the scale of the vectors depends on those two, and an instruction's 1 ulp
    // is enough.
    auto may_end = [&](int k) { return a.tol > 0.f || k >= a.n_iter; };
#pragma unroll 1
    for (int k = 1;; ++k) {
      // w = G_Q z with z = zscale * tv
      product<T, DH, MODE>(gq, tv, pp, role, wv, lane, out);
      if (k > 1) {
        const float n2 = dot_of(1);
        if (!(n2 > 0.f)) break;
        weigh(1, trk, n2);
        zscale = may_end(k) ? 1.0f / sqrtf(n2) : __builtin_amdgcn_rsqf(n2);
      }
      sums(0, tv, yv, zscale, dqr);
      __syncthreads();
      // t = G_K y with y = w / sigma
      product<T, DH, MODE>(gk, yv, pp, role, wv, lane, out);
      const float s2 = dot_of(0);
      if (!(s2 > 0.f)) break;
      const float bound = weigh(0, trq, s2);
      float sig = 0.f, inv_sig;
      bool last = false;
      if (may_end(k)) {
        sig = sqrtf(s2);
        inv_sig = 1.0f / sig;
        last = stop(k, sig, prev);
      } else {
        inv_sig = __builtin_amdgcn_rsqf(s2);
      }
      if (last) {
        __syncthreads();
        last_y(yv, inv_sig);
        product<T, DH, MODE>(gk, yv, pp, role, wv, lane, out);
      }
      sums(1, yv, last ? nullptr : tv, last ? 1.f : inv_sig, dkr);
      __syncthreads();
      if (last) {
        const float n2 = dot_of(1);
        if (!(n2 > 0.f)) break;
        const float bound_k = weigh(1, trk, n2);
        if (!(s2 >= kCancelSigma * bound && n2 >= kCancelSigma * bound_k && cancel <= 2 * k * kCancelMean)) break;
        finish(k, sig * fq * fk, tv, zscale * inv_sig / fq, yv, fq, 1.0f / (sqrtf(n2) * fq * fk));
        return;
      }
      prev = sig;
    }
    __syncthreads();
  }

  // the head's rows cancel, or its values leave the range of the Gram
  // products: iterate by reading the weights, from z0
  float* part = reinterpret_cast<float*>(big);
  if (t < DH) tb[t] = z0[t];
  __syncthreads();
  float prev = 0.f;
#pragma unroll 1
  for (int k = 1;; ++k) {
    const float s2 = direct_sweep<T, DH>(qblk, a.ld, a.d, tb, wb, part, red[0][0], wv, lane);
    const float sig = sqrtf(s2);
    if (s2 == 0.f) {  // M v = 0
      if (t == 0) {
        a.sigma[h] = 0.f;
        a.iters[h] = -2;
      }
      return;
    }
    const bool last = stop(k, sig, prev);
    const float inv = 1.0f / sig;
    if (last) {
      last_y(wb, inv);
    } else {
      if (t < DH) wb[t] *= inv;
      __syncthreads();
    }
    const float n2 = direct_sweep<T, DH>(kblk, a.ld, a.d, wb, dq, part, red[0][0], wv, lane);
    const float rn = 1.0f / sqrtf(n2);
    if (last) {
      finish(k, sig, tb, inv, wb, 1.f, rn);
      return;
    }
    if (t < DH) tb[t] = dq[t] * rn;
    __syncthreads();
    prev = sig;
  }
}

// Layer scales, and the vectors of the heads that took no step (the others
// leave the final sweeps normalised): block l.
__global__ void __launch_bounds__(kThreads) heads_finalize_kernel(FinArgs f) {
  const int l = blockIdx.x;
  __shared__ float red[kThreads / 64];
  __shared__ int nan_seen;
  if (threadIdx.x == 0) nan_seen = 0;
  __syncthreads();
  float m = 0.f;
  for (int i = threadIdx.x; i < f.n_q; i += kThreads) {
    const float s = f.sigma[(size_t)l * f.n_q + i];
    if (isnan(s)) nan_seen = 1;
    m = fmaxf(m, s);
  }
#pragma unroll
  for (int x = 32; x >= 1; x >>= 1) m = fmaxf(m, __shfl_xor(m, x));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 1; w < kThreads / 64; ++w) m = fmaxf(m, red[w]);
    f.scale[l] = nan_seen ? __builtin_nanf("") : f.coef * m;
  }
  __shared__ int list[kThreads], n_list;
  for (int i0 = 0; i0 < f.n_q; i0 += kThreads) {
    if (threadIdx.x == 0) n_list = 0;
    __syncthreads();
    const int i = i0 + (int)threadIdx.x;
    if (i < f.n_q && f.iters[l * f.n_q + i] <= 0) list[atomicAdd(&n_list, 1)] = l * f.n_q + i;
    __syncthreads();
    for (int x = 0; x < n_list; ++x) {  // rare, and independent of the order of the list
      const int h = list[x];
      const bool scale_v = f.iters[h] == -2;
      const float vs = 1.0f / f.w.vnorm0[h];
      for (int c = threadIdx.x; c < f.d; c += kThreads) {
        if (scale_v) f.v[(size_t)h * f.d + c] *= vs;
        if (f.u) f.u[(size_t)h * f.d + c] = 0.f;
      }
    }
    __syncthreads();
  }
}

template <typename T, int DH, int MODE>
void launch_mode(const HeadArgs& a, int heads, hipStream_t st) {
  if (a.sq > 0)
    heads_kernel<T, DH, H_SPLIT, MODE><<<dim3(heads), kHThreads, 0, st>>>(a);
  else if (a.g > 1)
    heads_kernel<T, DH, H_KEYS, MODE><<<dim3(heads), kHThreads, 0, st>>>(a);
  else if constexpr (MODE != I_HALVES)
    heads_kernel<T, DH, H_OWN, MODE><<<dim3(heads), kHThreads, 0, st>>>(a);
}

template <typename T, int DH>
void launch_dh(const HeadArgs& a, bool units, hipStream_t st) {
  const int heads = a.units * a.g;
  if (units) {
    units_kernel<T, DH><<<dim3(a.units * a.nch * a.sk + heads * a.sq), kHThreads, 0, st>>>(a);
    return;
  }
  if constexpr (sizeof(T) == 2 && DH == 128) {
    if (a.round_y) {
      launch_mode<T, DH, I_HALVES>(a, heads, st);
      return;
    }
  }
  launch_mode<T, DH, DH <= 64 ? I_ROWS : I_BLOCKS>(a, heads, st);
}

template <typename T>
void launch_t(int dh, const HeadArgs& a, bool units, hipStream_t st) {
  switch (dh) {
    case 16: launch_dh<T, 16>(a, units, st); break;
    case 32: launch_dh<T, 32>(a, units, st); break;
    case 64: launch_dh<T, 64>(a, units, st); break;
    default: launch_dh<T, 128>(a, units, st); break;
  }
}

}  // namespace

void launch_heads(bool bf16, int head_dim, bool units, hipStream_t st, HeadArgs a) {
  a.hps = heads_per_operand(bf16, a.round_y != 0, a.g);
  a.np = !bf16 ? 1 : a.hps == 8 ? 2 : 3;
  a.nch = (a.g + a.hps - 1) / a.hps;
  if (bf16)
    launch_t<uint16_t>(head_dim, a, units, st);
  else
    launch_t<float>(head_dim, a, units, st);
}

void launch_heads_finalize(int layers, hipStream_t st, const FinArgs& f) {
  heads_finalize_kernel<<<dim3(layers), kThreads, 0, st>>>(f);
}

}  // namespace sn
