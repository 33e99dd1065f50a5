// SSBA block-sparse attention forward in fp32 (fp32 inputs, products,
// accumulation and output) for gfx950 -- the full-precision path.
//
// Same decomposition and key order as the bf16 kernels (Algorithm 1, attend
// step; masked blocks are never read).  Both products run on the fp32 matrix
// instructions (2 K flops per 32 cycles, 157 TFLOP/s on the chip), which bound
// the kernel: a 32-query x 32-key unit at D 64 costs 4096 matrix cycles
// against ~200 cycles of softmax and ~100 of LDS reads, so neither needs to be
// clever.  Two ways to feed them, chosen per workgroup:
//
//   block_rows  64 query rows of one 8x8 block (or a quarter of a 16x16 one,
//               or 64 natural-order rows of the dense control): four waves =
//               two query halves x two 32-key streams over 64-key chunks that
//               all four share through LDS, with v_mfma_f32_32x32x2.  K and V
//               have one buffer each: chunk c's V is requested before its
//               scores and chunk c + 1's K before chunk c's value product, so
//               each load has half a chunk (2048 matrix cycles per wave, four
//               workgroups to a CU) to arrive.
//   wave_rows   16 query rows per wave, K and V straight from memory into
//               registers with v_mfma_f32_16x16x4, no LDS: a 4x4 block has
//               only 16 queries to share a key with.  Text rows use it too,
//               their keys dealt to the four waves of a workgroup: a text row
//               sees every key, and 64 rows walking them as one chain would
//               end long after the image blocks.
//
// Measured at B 1, H 16, 64x64 tokens, 8x8 blocks, keep 10, D 64 against the
// one-row-per-thread vector kernel it replaced (the launch alone): 1590 -> 99 us,
// 109 TFLOP/s (a large fp32 matrix product reaches 154 on this card); at 16x16
// tokens, 4x4 blocks, 2 heads, keep 4 (two steps per wave): 66 -> 7.2 us.
// Relative error against 64 bits at the first size: 6.5e-7 -> 4.3e-7.
//
// Register layouts (lane l):
//   32x32x2  A[i][k]: i = l % 32, k = l / 32; B[k][j]: j = l % 32, k = l / 32;
//            D: col l % 32, rows 8 (r / 4) + 4 (l / 32) + r % 4 (r = 0..15)
//   16x16x4  A[i][k]: i = l % 16, k = l / 16; B likewise;
//            D: col l % 16, rows 4 (l / 16) + r (r = 0..3)
// Scores are formed transposed (S^T = K Q^T), so a lane holds its own query's
// probabilities and they are the value product's B operand as they stand:
// step r contracts exactly the keys that register r of the lanes holds.
// Channels are dealt to the k index in runs of four so every operand is a
// 16-byte read; fp32 tensors are only 4-byte aligned, which global 16-byte
// loads accept, and the LDS copies are aligned.
#include <hip/hip_runtime.h>

#include "ssba_common.h"

namespace ssba {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));   // in memory: 4-byte aligned

constexpr int KC = 64;   // keys per chunk of block_rows
// Floats per K row in LDS: four more than D, so that the 16 rows that one
// pass of a 16-byte read takes lie on different banks.
template <int D>
constexpr int kRow = D + 4;

__device__ __forceinline__ floatx4 load4(const float* p) { return *reinterpret_cast<const floatx4u*>(p); }
__device__ __forceinline__ void store4(float* p, floatx4 v) { *reinterpret_cast<floatx4u*>(p) = v; }

__device__ __forceinline__ float exp2_f(float x) { return __builtin_amdgcn_exp2f(x); }

// Max / sum over lanes l, l ^ 32 and (quad) also l ^ 16.
__device__ __forceinline__ float pair_max(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float pair_sum(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float quad_max(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return pair_max(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}
__device__ __forceinline__ float quad_sum(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return pair_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}

// A run of keys: slots of one image block from block row y0 on, or sequence
// rows in order (then `base` is the first and `width` the block side, so the
// same arithmetic counts them off).  Slots hi and up do not exist.
struct Keys {
  int base, y0, x0, width, hi;
};

__device__ __forceinline__ int key_row(const Frame& f, const Keys& k, int slot) {
  int y = k.y0 + (slot >> f.tile_log2), x = k.x0 + (slot & ((1 << f.tile_log2) - 1));
  y += y < 0 ? f.grid_h : 0;
  x += x < 0 ? f.grid_w : 0;
  return k.base + y * k.width + x;
}

// `rows` slots of block j from slot `first` on; an id outside the grid has none.
__device__ __forceinline__ Keys image_keys(const AttnArgs& a, int j, int first, int rows) {
  Keys k;
  const int jj = (unsigned)j < (unsigned)a.n_tiles ? j : 0;
  const int ty = jj / a.f.nx;
  k.base = a.f.n_text;
  k.y0 = (ty << a.f.tile_log2) - a.f.sy + (first >> a.f.tile_log2);
  k.x0 = ((jj - ty * a.f.nx) << a.f.tile_log2) - a.f.sx;
  k.width = a.f.grid_w;
  k.hi = jj == j ? rows : 0;
  return k;
}

__device__ __forceinline__ Keys linear_keys(const AttnArgs& a, int first, int end, int rows) {
  Keys k;
  k.base = first;
  k.y0 = k.x0 = 0;
  k.width = 1 << a.f.tile_log2;
  k.hi = min(max(end - first, 0), rows);
  return k;
}

// The kept list of one query block, read through the scalar cache: an entry
// costs no vector register and is requested a step before it is used.
struct List {
  const __attribute__((address_space(4))) int32_t* ids;
  int count;
  __device__ __forceinline__ void open(const AttnArgs& a, int64_t bh, int block) {
    ids = (const __attribute__((address_space(4))) int32_t*)(a.index + (bh * a.n_tiles + block) * (a.n_tiles + 1));
    count = min(max(ids[0], 0), a.n_tiles);
  }
  __device__ __forceinline__ int at(int e) const { return e < count ? ids[1 + e] : -1; }
};

// 64 query rows per workgroup (see the file comment).  `group`: image group
// (block, then quarter of a 16x16 block), or 64 natural-order rows.
template <int D>
__device__ __forceinline__ void block_rows(const AttnArgs& a, int64_t bh, int64_t off, int group, float* kbuf,
                                           float* vbuf) {
  constexpr int PR = D / 4;            // 16-byte pieces per row
  constexpr int RPI = 256 / PR;        // rows per staging round
  constexpr int NF = KC / RPI;         // staging rounds per chunk
  constexpr int NQ = D / 8;            // 16-byte pieces of a row per lane half
  constexpr int NDB = D / 32;          // 32-channel tiles of O
  const float* qbase = static_cast<const float*>(a.q) + off;
  const float* kbase = static_cast<const float*>(a.k) + off;
  const float* vbase = static_cast<const float*>(a.v) + off;
  float* obase = static_cast<float*>(a.o) + off;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int qh = w & 1, sk = w >> 1, hw = lane >> 5, l32 = lane & 31;
  const int part = threadIdx.x % PR, srow = threadIdx.x / PR;   // staging: 16 bytes of row srow + RPI i
  const int cl = 2 * a.f.tile_log2 - 6;                         // log2 of 64-row chunks per block

  int qrow, n_img = 0, n;
  List list{nullptr, 0};
  if (a.dense) {
    const int q = 64 * group + 32 * qh + l32;
    qrow = q < a.seq ? q : -1;
    n = (a.seq + KC - 1) / KC;
  } else {
    const int i = group >> cl;
    qrow = frame_row(a.f, i, 64 * (group - (i << cl)) + 32 * qh + l32);
    list.open(a, bh, i);
    n_img = list.count << cl;
    n = n_img + (a.f.n_text + KC - 1) / KC;
  }
  auto entry_of = [&](int c) { return a.dense ? -1 : list.at(c >> cl); };
  auto keys_of = [&](int c, int entry) {
    if (a.dense) return linear_keys(a, c * KC, a.seq, KC);
    if (c >= n_img) return linear_keys(a, (c - n_img) * KC, a.f.n_text, KC);
    return image_keys(a, entry, (c & ((1 << cl) - 1)) * KC, KC);
  };
  auto fetch = [&](const float* base, const Keys& ks, floatx4 (&r)[NF]) {
    if (ks.hi == KC) {
#pragma unroll
      for (int i = 0; i < NF; ++i)
        r[i] = load4(base + (int64_t)key_row(a.f, ks, srow + RPI * i) * a.st + 4 * part);
    } else {   // rows that do not exist are zeros: their probability is zero
#pragma unroll
      for (int i = 0; i < NF; ++i) {
        r[i] = floatx4{};
        if (srow + RPI * i < ks.hi) r[i] = load4(base + (int64_t)key_row(a.f, ks, srow + RPI * i) * a.st + 4 * part);
      }
    }
  };
  auto put_k = [&](const floatx4 (&r)[NF]) {
#pragma unroll
    for (int i = 0; i < NF; ++i) *reinterpret_cast<floatx4*>(kbuf + (srow + RPI * i) * kRow<D> + 4 * part) = r[i];
  };
  auto put_v = [&](const floatx4 (&r)[NF]) {
#pragma unroll
    for (int i = 0; i < NF; ++i) *reinterpret_cast<floatx4*>(vbuf + (srow + RPI * i) * D + 4 * part) = r[i];
  };

  floatx4 qf[NQ];   // channels 8 i + 4 hw + [0, 4) of the lane's query
#pragma unroll
  for (int i = 0; i < NQ; ++i) qf[i] = load4(qbase + (int64_t)max(qrow, 0) * a.st + 8 * i + 4 * hw);

  floatx16 o[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) o[db] = floatx16{};
  float m_run = -INFINITY, l_run = 0.f;
  const float c2 = a.scale_log2;

  floatx4 stage[NF];
  Keys cur = linear_keys(a, 0, 0, 0);
  if (n > 0) {
    cur = keys_of(0, entry_of(0));
    fetch(kbase, cur, stage);
    put_k(stage);
  }
  __syncthreads();
  const float* krow = kbuf + (32 * sk + l32) * kRow<D> + 4 * hw;
  const float* vcol = vbuf + 32 * sk * D + NDB * l32;
  for (int c = 0; c < n; ++c) {
    const int entry = entry_of(c + 1);
    fetch(vbase, cur, stage);
    floatx16 sc = floatx16{};
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      const floatx4 kf = *reinterpret_cast<const floatx4*>(krow + 8 * i);
#pragma unroll
      for (int e = 0; e < 4; ++e) sc = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[e], qf[i][e], sc, 0, 0, 0);
    }
    if (cur.hi < KC) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (32 * sk + 8 * (r >> 2) + 4 * hw + (r & 3) >= cur.hi) sc[r] = -INFINITY;
    }
    put_v(stage);
    __syncthreads();   // V is there, and every wave is past chunk c's K
    const bool more = c + 1 < n;
    if (more) {
      cur = keys_of(c + 1, entry);
      fetch(kbase, cur, stage);
    }
    // Online softmax in log2 units; -inf stands for "no key yet".
    float mx = sc[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, sc[r]);
    const float m_new = fmaxf(m_run, pair_max(mx) * c2);
    const float m_use = m_new == -INFINITY ? 0.f : m_new;
    if (__any(m_new > m_run)) {
      const float alpha = exp2_f(m_run - m_use);
      l_run *= alpha;
#pragma unroll
      for (int db = 0; db < NDB; ++db) o[db] *= alpha;
      m_run = m_new;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) sc[r] = exp2_f(__builtin_fmaf(sc[r], c2, -m_use));
    float s0 = 0.f, s1 = 0.f;
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
      s0 += sc[r];
      s1 += sc[r + 1];
    }
    l_run += s0 + s1;
    // O^T[NDB i + db] += V^T P^T: step r takes key 8 (r / 4) + 4 hw + r % 4.
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float* v = vcol + (8 * (r >> 2) + 4 * hw + (r & 3)) * D;
      float vf[NDB];
#pragma unroll
      for (int db = 0; db < NDB; ++db) vf[db] = v[db];
#pragma unroll
      for (int db = 0; db < NDB; ++db) o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(vf[db], sc[r], o[db], 0, 0, 0);
    }
    if (more) put_k(stage);
    __syncthreads();   // chunk c + 1's K is there, and every wave is past chunk c's V
  }

  // Merge the two key streams: stream 1 leaves (O, m, l) in LDS.
  static_assert(2 * 16 * NDB * 64 <= KC * D, "O of both query halves fits the K buffer");
  float* xo = kbuf + qh * 16 * NDB * 64 + lane;
  float* xm = vbuf + 128 * qh + lane;
  if (sk == 1) {
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) xo[(16 * db + r) * 64] = o[db][r];
    xm[0] = m_run;
    xm[64] = l_run;
  }
  __syncthreads();
  if (sk == 1) return;
  const float m1 = xm[0], mm = fmaxf(m_run, m1), mu = mm == -INFINITY ? 0.f : mm;
  const float a0 = exp2_f(m_run - mu), a1 = exp2_f(m1 - mu);
  const float l = pair_sum(l_run * a0 + xm[64] * a1);
  const float inv = l > 0.f ? 1.0f / l : 0.f;
  const bool none = mm == -INFINITY;   // no score above -inf: a row of zeros
  if (qrow < 0) return;
  float* orow = obase + (int64_t)qrow * a.st;
#pragma unroll
  for (int g = 0; g < 4; ++g) {   // rows 8 g + 4 hw + [0, 4) of every tile: 4 NDB channels in a row
    float x[4 * NDB];
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int db = 0; db < NDB; ++db)
        x[NDB * e + db] = none ? 0.f : (o[db][4 * g + e] * a0 + xo[(16 * db + 4 * g + e) * 64] * a1) * inv;
#pragma unroll
    for (int u = 0; u < NDB; ++u)
      store4(orow + NDB * (8 * g + 4 * hw) + 4 * u, floatx4{x[4 * u], x[4 * u + 1], x[4 * u + 2], x[4 * u + 3]});
  }
}

// 16 query rows per wave (see the file comment): the wave's own 4x4 block
// (`block`), or, with block < 0, 16 text rows from q0 on, whose keys the four
// waves of the workgroup share out and merge through `xbuf`.
template <int D>
__device__ __forceinline__ void wave_rows(const AttnArgs& a, int64_t bh, int64_t off, int block, int q0, float* xbuf) {
  constexpr int KB = D == 64 ? 2 : 1;   // 16-key runs per step (K and V of a step stay in registers)
  constexpr int NQ = D / 16;            // 16-byte pieces of a row per lane
  constexpr int NU = D / 64;            // 16-byte pieces of a V row per lane
  const float* qbase = static_cast<const float*>(a.q) + off;
  const float* kbase = static_cast<const float*>(a.k) + off;
  const float* vbase = static_cast<const float*>(a.v) + off;
  float* obase = static_cast<float*>(a.o) + off;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, l16 = lane & 15;
  const bool text = block < 0;

  int qrow, n_img = 0, runs;
  List list{nullptr, 0};
  if (text) {
    qrow = q0 + l16 < a.f.n_text ? q0 + l16 : -1;
    runs = (a.seq + 15) / 16;
  } else {
    qrow = frame_row(a.f, block, l16);
    list.open(a, bh, block);
    n_img = list.count;
    runs = n_img + (a.f.n_text + 15) / 16;
  }
  const int steps = (runs + KB - 1) / KB;
  const int first = text ? w : 0, stride = text ? 4 : 1;
  auto entries_of = [&](int step, int (&entry)[KB]) {
#pragma unroll
    for (int b = 0; b < KB; ++b) entry[b] = text ? -1 : list.at(KB * step + b);
  };
  auto keys_of = [&](int step, const int (&entry)[KB], Keys (&ks)[KB]) {
#pragma unroll
    for (int b = 0; b < KB; ++b) {
      const int r = KB * step + b;
      if (text) ks[b] = linear_keys(a, 16 * r, a.seq, 16);
      else if (r < n_img) ks[b] = image_keys(a, entry[b], 0, 16);
      else ks[b] = linear_keys(a, 16 * (r - n_img), a.f.n_text, 16);
    }
  };
  auto fetch_k = [&](const Keys (&ks)[KB], floatx4 (&kr)[KB][NQ]) {   // channels 16 i + 4 g + [0, 4) of key l16
#pragma unroll
    for (int b = 0; b < KB; ++b) {
      const float* p = kbase + (int64_t)key_row(a.f, ks[b], l16 < ks[b].hi ? l16 : 0) * a.st + 4 * g;
      if (ks[b].hi == 0) p = kbase;   // no such run: any row (masked)
#pragma unroll
      for (int i = 0; i < NQ; ++i) kr[b][i] = load4(p + 16 * i);
    }
  };

  floatx4 qf[NQ];
#pragma unroll
  for (int i = 0; i < NQ; ++i) qf[i] = load4(qbase + (int64_t)max(qrow, 0) * a.st + 16 * i + 4 * g);
  floatx4 o[4 * NU];   // [4 u + e]: channels 64 u + 4 i + e of query l16, i = 4 g + r
#pragma unroll
  for (int t = 0; t < 4 * NU; ++t) o[t] = floatx4{};
  float m_run = -INFINITY, l_run = 0.f;
  const float c2 = a.scale_log2;

  Keys ks[KB];
  floatx4 kr[KB][NQ];
  int entry[KB];
  if (first < steps) {
    entries_of(first, entry);
    keys_of(first, entry, ks);
    fetch_k(ks, kr);
  }
  for (int step = first; step < steps; step += stride) {
    entries_of(step + stride, entry);
    floatx4 vr[KB][4][NU];   // key 4 g + r, channels 64 u + 4 l16 + [0, 4)
    bool whole = true;
#pragma unroll
    for (int b = 0; b < KB; ++b) whole = whole && ks[b].hi == 16;
    int hi[KB];
#pragma unroll
    for (int b = 0; b < KB; ++b) {
      hi[b] = ks[b].hi;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int s = 4 * g + r;
        const float* p = vbase + (int64_t)key_row(a.f, ks[b], s < hi[b] ? s : 0) * a.st + 4 * l16;
        if (hi[b] == 0) p = vbase + 4 * l16;
#pragma unroll
        for (int u = 0; u < NU; ++u) vr[b][r][u] = load4(p + 64 * u);
      }
    }
    floatx4 sc[KB];
#pragma unroll
    for (int b = 0; b < KB; ++b) {
      sc[b] = floatx4{};
#pragma unroll
      for (int i = 0; i < NQ; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) sc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(kr[b][i][e], qf[i][e], sc[b], 0, 0, 0);
    }
    if (step + stride < steps) {
      keys_of(step + stride, entry, ks);
      fetch_k(ks, kr);
    }
    if (!whole) {
#pragma unroll
      for (int b = 0; b < KB; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (4 * g + r >= hi[b]) {
            sc[b][r] = -INFINITY;
#pragma unroll
            for (int u = 0; u < NU; ++u) vr[b][r][u] = floatx4{};
          }
    }
    float mx = sc[0][0];
#pragma unroll
    for (int b = 0; b < KB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) mx = fmaxf(mx, sc[b][r]);
    const float m_new = fmaxf(m_run, quad_max(mx) * c2);
    const float m_use = m_new == -INFINITY ? 0.f : m_new;
    if (__any(m_new > m_run)) {
      const float alpha = exp2_f(m_run - m_use);
      l_run *= alpha;
#pragma unroll
      for (int t = 0; t < 4 * NU; ++t) o[t] *= alpha;
      m_run = m_new;
    }
#pragma unroll
    for (int b = 0; b < KB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        sc[b][r] = exp2_f(__builtin_fmaf(sc[b][r], c2, -m_use));
        l_run += sc[b][r];
      }
#pragma unroll
    for (int b = 0; b < KB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            o[4 * u + e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vr[b][r][u][e], sc[b][r], o[4 * u + e], 0, 0, 0);
  }

  float l = l_run;
  if (text) {   // waves 1..3 leave (O, m, l), wave 0 merges them in order
    constexpr int VALS = 16 * NU + 2;
    static_assert(3 * VALS * 64 <= KC * D, "three streams fit the K buffer");
    if (w > 0) {
      float* x = xbuf + (w - 1) * VALS * 64 + lane;
#pragma unroll
      for (int t = 0; t < 4 * NU; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) x[(4 * t + r) * 64] = o[t][r];
      x[(VALS - 2) * 64] = m_run;
      x[(VALS - 1) * 64] = l_run;
    }
    __syncthreads();
    if (w > 0) return;
    for (int s = 0; s < 3; ++s) {
      const float* x = xbuf + s * VALS * 64 + lane;
      const float m1 = x[(VALS - 2) * 64], mm = fmaxf(m_run, m1), mu = mm == -INFINITY ? 0.f : mm;
      const float a0 = exp2_f(m_run - mu), a1 = exp2_f(m1 - mu);
      l = l * a0 + x[(VALS - 1) * 64] * a1;
      m_run = mm;
#pragma unroll
      for (int t = 0; t < 4 * NU; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) o[t][r] = o[t][r] * a0 + x[(4 * t + r) * 64] * a1;
    }
  }
  l = quad_sum(l);
  const float inv = l > 0.f ? 1.0f / l : 0.f;
  if (m_run == -INFINITY) {   // no score above -inf: a row of zeros
#pragma unroll
    for (int t = 0; t < 4 * NU; ++t) o[t] = floatx4{};
  }
  if (qrow < 0) return;
  float* orow = obase + (int64_t)qrow * a.st;
#pragma unroll
  for (int u = 0; u < NU; ++u)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      store4(orow + 64 * u + 16 * g + 4 * r, floatx4{o[4 * u][r], o[4 * u + 1][r], o[4 * u + 2][r], o[4 * u + 3][r]} * inv);
}

template <int D>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(D == 64 ? 4 : 2))) k_attn_f32(AttnArgs a) {
  __shared__ __attribute__((aligned(16))) float kbuf[KC * kRow<D>];
  __shared__ __attribute__((aligned(16))) float vbuf[KC * D];
  // (batch, head) and group: consecutive hardware ids go round-robin over the
  // 8 XCDs; when the (batch, head) count divides by 8 each XCD gets whole
  // heads, so their K and V stay in its L2.  Text groups (every key) first.
  const int bid = blockIdx.x, nbh = a.batch * a.heads, nt = a.n_text_groups, ni = a.groups_per_bh - nt;
  int bh, r;
  if ((nbh & 7) == 0) {
    const int xcd = bid & 7, s = bid >> 3, hpx = nbh >> 3;
    const bool t = s < hpx * nt;
    const int s2 = t ? s : s - hpx * nt, d = t ? nt : ni;
    bh = xcd * hpx + s2 / d;
    r = (t ? 0 : nt) + s2 % d;
  } else {
    bh = bid / a.groups_per_bh;
    r = bid - bh * a.groups_per_bh;
  }
  const int b = bh / a.heads, h = bh - b * a.heads;
  const int64_t off = (int64_t)b * a.sb + (int64_t)h * a.sh;
  if (r < nt) {
    __builtin_amdgcn_s_setprio(2);   // the longest chains of the launch
    wave_rows<D>(a, bh, off, -1, 16 * r, kbuf);
  } else if (!a.dense && a.f.tile_log2 == 2) {
    const int block = 4 * (r - nt) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (block < a.n_tiles) wave_rows<D>(a, bh, off, block, 0, nullptr);
  } else {
    block_rows<D>(a, bh, off, r - nt, kbuf, vbuf);
  }
}

template <int D>
hipError_t launch_t(const AttnArgs& a0, int tile, hipStream_t s) {
  AttnArgs a = a0;
  if (a.dense) {   // 64 natural-order rows per group
    a.n_text_groups = 0;
    a.groups_per_bh = (a.seq + 63) / 64;
  } else {         // 16 text rows, then four 4x4 blocks, one 8x8 block or a quarter of a 16x16 block
    a.n_text_groups = (a.f.n_text + 15) / 16;
    a.groups_per_bh = a.n_text_groups + (tile == 4 ? (a.n_tiles + 3) / 4 : tile == 8 ? a.n_tiles : 4 * a.n_tiles);
  }
  // One launch, but for millions of (batch, head) pairs: whole batch elements,
  // or heads of one, as many as a launch has threads for.
  int64_t per = kMaxGroups256 / a.groups_per_bh;
  if (per < 1) per = 1;
  const int64_t nb = per / a0.heads > 0 ? per / a0.heads : 1, nh = per < a0.heads ? per : a0.heads;
  for (int64_t b = 0; b < a0.batch; b += nb)
    for (int64_t h = 0; h < a0.heads; h += nh) {
      const int64_t off = b * a.sb + h * a.sh;
      a.batch = (int)(a0.batch - b < nb ? a0.batch - b : nb);
      a.heads = (int)(a0.heads - h < nh ? a0.heads - h : nh);
      a.q = static_cast<const float*>(a0.q) + off;
      a.k = static_cast<const float*>(a0.k) + off;
      a.v = static_cast<const float*>(a0.v) + off;
      a.o = static_cast<float*>(a0.o) + off;
      if (!a.dense) a.index = a0.index + (b * a0.heads + h) * a.n_tiles * (a.n_tiles + 1);
      const int64_t total = (int64_t)a.batch * a.heads * a.groups_per_bh;
      hipLaunchKernelGGL(k_attn_f32<D>, dim3((unsigned)total), dim3(256), 0, s, a);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
  return hipSuccess;
}

}  // namespace

hipError_t launch_attn_f32(const AttnArgs& a, int head_dim, int tile, hipStream_t s) {
  if (head_dim == 64) return launch_t<64>(a, tile, s);
  return launch_t<128>(a, tile, s);
}

}  // namespace ssba
