// SSBA attention forward, bf16, head_dim 64 or 128, 4x4-token blocks: one wave
// per query block.
//
// Computes the attend step of Algorithm 1 like the other attention kernels
// (image queries of a block attend to the image keys of its kept blocks and to
// every text key; text queries attend to every key).
//
// What bounds it: a block has 16 queries, so each kept key's K and V rows are
// used for only 16 queries and come from the L2 again for the next block
// (16 flops per byte at any head_dim).  So the work is laid out for loads in
// flight, not for reuse:
//   * a wave owns one query block and shares nothing: no barrier, and five
//     workgroups (D 64) keep 20 waves a CU, each with 4 to 8 KB under way;
//   * a step is two units of 16 keys (a kept block or 16 text rows).  K and V
//     rows go by DMA into the wave's own LDS, whole rows to consecutive lanes:
//     read straight into the operand order of the products, in which
//     consecutive lanes hold different rows, the same rows arrive at
//     9.7 TB/s over the chip instead of 32.  K comes back as the rows of
//     v_mfma_f32_16x16x32_bf16 (ds_read_b128), V transposed
//     (ds_read_b64_tr_b16).  Each buffer is single: the next step's copy is
//     issued as soon as the operands are in registers, so K's is under way
//     during the softmax and the second product, V's during the next first
//     product and softmax;
//   * S^T = K Q^T leaves each lane 4 keys of one query, which is the operand
//     order of O^T += V^T P^T, so P stays in registers;
//   * the softmax takes no maximum until a lane's step sum exceeds 2^20 (the
//     running max grew); the scale stays in the fp32 scores.
// Text queries see every key, 16 rows to a workgroup: its four waves take the
// steps in turn and merge at the end (one wave a group would run several times
// as long as an image block and finish alone).
// Measured at 60x92 tokens + 77 text, 12 heads, D 64, keep 54 of 345 (17.3
// GFLOP, about 1 GB through the L2), the launch alone: the generic kernel
// 565 us, this one 52 us (20 TB/s through the L2, which gives plain copies 32).
//
// LDS layout of a unit: 16 keys of 2 D bytes, 16-byte chunk c of key k at
//   K, D 64:  c ^ ((k >> 1) & 7)     V, D 64:  c ^ 2 ((k >> 1) & 3)
//   K, D 128: c ^ (k & 15)           V, D 128: c ^ 2 (k & 7)
// so that 16 lanes' K reads (16 keys at one chunk) and a half wave's
// transposing V read (8 keys x 32 bytes) hit every bank once.
#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>
#include <type_traits>

#include "ssba_common.h"

namespace ssba {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t u16;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef __attribute__((address_space(3))) void lds_void;

constexpr int kWaves = 4;                 // per workgroup
constexpr float kSumLimit = 1048576.0f;   // 2^20: redo a step above this lane sum
constexpr float kNoMax = -0.99e30f;       // a running max below this: no score seen yet
// s_waitcnt immediate (vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8):
// at most n vector memory operations left.
constexpr int wait_vm(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }
constexpr int kRawBufferFlags = 0x00020000;
// Byte offset of a row that is not there: past every slice this kernel takes
// (below 2^31 bytes), so loads of it return zeros.
constexpr unsigned kNoRow = 0x80000000u;

template <int D>
struct Shape4 {
  static constexpr int ROWB = 2 * D;          // bytes per row
  static constexpr int CPR = D / 8;           // 16-byte chunks per row
  static constexpr int KPI = 1024 / ROWB;     // keys per copy instruction
  static constexpr int NI = 16 / KPI;         // copy instructions per unit (of K, and of V)
  static constexpr int NKS = D / 32;          // 32-channel steps of Q K^T
  static constexpr int NDB = D / 16;          // 16-channel tiles of O
  static constexpr int UNIT = 16 * ROWB;      // LDS bytes of a unit's K or V
};

__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{lo, hi}, bf16x2));
}
// Over the four lanes that hold one query.
__device__ __forceinline__ float xmax4(float v) {
  v = fmaxf(v, __shfl_xor(v, 16));
  return fmaxf(v, __shfl_xor(v, 32));
}
__device__ __forceinline__ float xsum4(float v) {
  v += __shfl_xor(v, 16);
  return v + __shfl_xor(v, 32);
}

// Logical id of hardware workgroup `bid` of `n`: hardware ids go round-robin
// over the 8 XCDs; each gets one contiguous range of logical ids, so the
// groups of a head share one L2.
__device__ __forceinline__ int xcd_range(int bid, int n) {
  const int xcd = bid & 7, slot = bid >> 3, per = n >> 3, rem = n & 7;
  return xcd * per + min(xcd, rem) + slot;
}

template <int D>
__device__ __forceinline__ void attn_tile4(const AttnArgs& a) {
  using S = Shape4<D>;
  constexpr int NKS = S::NKS, NDB = S::NDB, NI = S::NI;
  // K and V of a step, a part per wave.  Two variables, each named statically
  // by every access, so that the compiler can tell a read of one from the copy
  // into the other.
  __shared__ __attribute__((aligned(16))) char kbuf[kWaves * 2 * S::UNIT];
  __shared__ __attribute__((aligned(16))) char vbuf[kWaves * 2 * S::UNIT];

  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lq = lane & 15, lg = lane >> 4;
  const int nbh = a.batch * a.heads;

  // Text groups first (a multiple of 8 of them, the last ones empty, so that
  // the image groups start on XCD 0), then four image blocks a group.
  const int n_text_wg = (nbh * a.n_text_groups + 7) & ~7;
  const bool text = (int)blockIdx.x < n_text_wg;
  int bh, i = 0, row0 = 0;
  if (text) {
    const int id = blockIdx.x;
    if (id >= nbh * a.n_text_groups) return;
    bh = id / a.n_text_groups;
    row0 = 16 * (id - bh * a.n_text_groups);
  } else {
    const int id = xcd_range((int)blockIdx.x - n_text_wg, (int)gridDim.x - n_text_wg);
    bh = id / a.groups_per_tile;                      // image groups per (batch, head)
    i = kWaves * (id - bh * a.groups_per_tile) + w;
    if (i >= a.n_tiles) return;
  }
  const int b = bh / a.heads, h = bh - b * a.heads;
  const int64_t off = (int64_t)b * a.sb + (int64_t)h * a.sh;
  const u16* qbase = static_cast<const u16*>(a.q) + off;
  const int W = a.f.grid_w, st = (int)a.st;
  const unsigned st2 = 2u * (unsigned)st;

  const int qrow = !text ? frame_row(a.f, i, lq) : row0 + lq < a.f.n_text ? row0 + lq : -1;
  bf16x8 qf[NKS];   // Q^T operand: query lq, channels 32 ks + 8 lg + [0, 8)
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks)
    qf[ks] = *reinterpret_cast<const bf16x8*>(qbase + (int64_t)max(qrow, 0) * st + 32 * ks + 8 * lg);

  // Units: the kept blocks in list order, then 16 natural rows each of
  // [0, end).  Steps of two units; a text group's waves take them in turn.
  const int32_t* list = a.index + (bh * (int64_t)a.n_tiles + i) * (a.n_tiles + 1);
  const int count = text ? 0 : __builtin_amdgcn_readfirstlane(min(max(list[0], 0), a.n_tiles));
  const int end = text ? a.seq : a.f.n_text;
  const int n = (count + (end + 15) / 16 + 1) / 2;
  const int first = text ? w : 0, stride = text ? kWaves : 1;
  if (text) __builtin_amdgcn_s_setprio(3);   // the longest waves of the launch

  const unsigned slice_bytes = 2u * (unsigned)((a.seq - 1) * st + D);
  const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<u16*>(static_cast<const u16*>(a.k) + off), (short)0, (int)slice_bytes, kRawBufferFlags);
  const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<u16*>(static_cast<const u16*>(a.v) + off), (short)0, (int)slice_bytes, kRawBufferFlags);

  // Frame origin of 64 list entries at a time, one per lane.
  int orig_y = 0, orig_x = 0, ok = 0;
  auto load_list = [&](int e0) {
    const int ent = e0 + lane < count ? list[1 + e0 + lane] : -1;
    ok = (unsigned)ent < (unsigned)a.n_tiles ? 1 : 0;
    const int j = ok ? ent : 0, ty = j / a.f.nx;
    orig_y = 4 * ty - a.f.sy;
    orig_x = 4 * (j - ty * a.f.nx) - a.f.sx;
  };
  if (count > 0) load_list(0);
  // Q arrives with the list: were it first waited for inside the loop, that
  // wait would drain the copies under way on every step.
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) asm volatile("" : "+v"(qf[ks]));

  // Copy instruction m of a unit fills key KPI m + lane / CPR, physical chunk
  // lane % CPR, with the chunk that the LDS layout wants there.  `at` is the
  // key's row within a block (instruction m: m more row steps below it).
  const unsigned line = (unsigned)W * st2;
  const int ckey = lane / S::CPR, cch = lane % S::CPR;
  const unsigned at = (unsigned)(ckey >> 2) * line + (unsigned)(ckey & 3) * st2;
  const unsigned rstep = (unsigned)(S::KPI / 4) * line;
  unsigned kcol[NI], vcol[NI];
#pragma unroll
  for (int m = 0; m < NI; ++m) {
    const int key = S::KPI * m + ckey;
    kcol[m] = 16u * (unsigned)(cch ^ (D == 64 ? (key >> 1) & 7 : key & 15));
    vcol[m] = 16u * (unsigned)(cch ^ (D == 64 ? 2 * ((key >> 1) & 3) : 2 * (key & 7)));
  }
  // Byte offsets of the lane's rows in the copies of unit u; returns its
  // number of keys.
  auto rows_of = [&](int u, unsigned (&ro)[NI]) {
    int hi;
    if (u < count) {
      if (u > 0 && (u & 63) == 0) load_list(u);   // units are taken in order
      const int e = u & 63;
      const int y0 = __builtin_amdgcn_readlane(orig_y, e), x0 = __builtin_amdgcn_readlane(orig_x, e);
      hi = __builtin_amdgcn_readlane(ok, e) ? 16 : 0;
      const unsigned base = (unsigned)(a.f.n_text + y0 * W + x0) * st2;
#pragma unroll
      for (int m = 0; m < NI; ++m) ro[m] = base + (unsigned)m * rstep + at;
      if ((y0 | x0) < 0) {   // a block on the seam: rows and columns past it wrap
        const unsigned grid = (unsigned)a.f.grid_h * line;
#pragma unroll
        for (int m = 0; m < NI; ++m)
          ro[m] += (y0 + ((S::KPI * m + ckey) >> 2) < 0 ? grid : 0u) + (x0 + (ckey & 3) < 0 ? line : 0u);
      }
    } else {   // 16 rows in natural order
      const int row = 16 * (u - count);
      hi = min(max(end - row, 0), 16);
#pragma unroll
      for (int m = 0; m < NI; ++m) ro[m] = (unsigned)(row + S::KPI * m + ckey) * st2;
    }
    if (hi < 16) {   // the text's last rows, an odd last unit, an invalid id
#pragma unroll
      for (int m = 0; m < NI; ++m) ro[m] = S::KPI * m + ckey < hi ? ro[m] : kNoRow;
    }
    return __builtin_amdgcn_readfirstlane(hi);
  };
  unsigned ro0[NI], ro1[NI];   // rows of the step being copied
  int hi0 = 0, hi1 = 0;        // ... and its valid keys
  auto copy = [&](const __amdgpu_buffer_rsrc_t& rs, const unsigned (&col)[NI], char* dst) {
#pragma unroll
    for (int m = 0; m < NI; ++m)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)(dst + 1024 * m), 16, ro0[m] + col[m], 0u, 0, 0);
#pragma unroll
    for (int m = 0; m < NI; ++m)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)(dst + S::UNIT + 1024 * m), 16, ro1[m] + col[m], 0u, 0,
                                               0);
  };

  // K operand reads: key lq, chunk 4 ks + lg.
  int koff[NKS];
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) {
    const int c = 4 * ks + lg;
    koff[ks] = lq * S::ROWB + 16 * (c ^ (D == 64 ? (lq >> 1) & 7 : lq));
  }
  // V transposing reads: lane i = lane % 16 of group lg reads key 4 lg + i / 4,
  // channels 16 db + 4 (i % 4) .. + 3, and receives channel 16 db + i of the
  // four keys 4 lg .. + 3.
  int voff[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) {
    const int key = 4 * lg + (lq >> 2);
    const int sw = D == 64 ? (key >> 1) & 3 : key & 7;
    voff[db] = key * S::ROWB + 32 * (db ^ sw) + 8 * (lq & 3);
  }

  floatx4 oacc[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) oacc[db] = floatx4{};
  float m_run = -1e30f, l_run = 0.f;   // running max of the scaled scores (log2 units), lane's sum
  float nm = 0.f;                      // -m_run, 0 while unset

  // P of a step's scores as bf16 pairs, O and l rescaled where the max grew.
  auto softmax = [&](const floatx4& s0, const floatx4& s1, int h0, int h1, uint32_t (&pk)[4]) {
    float sc[8];   // keys 4 lg + e of unit 0, then of unit 1
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      sc[e] = __builtin_fmaf(s0[e], a.scale_log2, nm);
      sc[4 + e] = __builtin_fmaf(s1[e], a.scale_log2, nm);
    }
    if (min(h0, h1) < 16) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (4 * lg + e >= h0) sc[e] = -INFINITY;
        if (4 * lg + e >= h1) sc[4 + e] = -INFINITY;
      }
    }
    float ls;
    auto probs = [&](float shift, bool shifted) {
      float l0 = 0.f, l1 = 0.f;
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const float x0 = shifted ? sc[2 * p] - shift : sc[2 * p];
        const float x1 = shifted ? sc[2 * p + 1] - shift : sc[2 * p + 1];
        const float p0 = __builtin_amdgcn_exp2f(x0), p1 = __builtin_amdgcn_exp2f(x1);
        pk[p] = pack2(p0, p1);
        l0 += p0;   // (v_dot2 on the packed pair would queue with the products: 59 us against 52)
        l1 += p1;
      }
      ls = l0 + l1;
    };
    probs(0.f, false);
    // The max grew, or there is none yet: take the step's, rescale, redo.
    if (__any(!(ls <= kSumLimit) || m_run < kNoMax)) {
      float mx = sc[0];
#pragma unroll
      for (int e = 1; e < 8; ++e) mx = fmaxf(mx, sc[e]);
      float mb = m_run > kNoMax ? m_run : 0.f;   // the offset in sc
      // Where the max is more than 2^10 from the offset, sc was rounded to
      // worse than 2^-14: again from the scores, against an offset near it.
      if (__any(fabsf(mx) > 1024.f && mx > -INFINITY)) {
        const float by = xmax4(mx);
        mb += by > -INFINITY ? by : 0.f;
        int g0 = h0, g1 = h1;   // (opaque, or the tests of h0 and h1 are kept for here)
        asm volatile("" : "+s"(g0), "+s"(g1));
        mx = -INFINITY;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          sc[e] = 4 * lg + e < g0 ? __builtin_fmaf(s0[e], a.scale_log2, -mb) : -INFINITY;
          sc[4 + e] = 4 * lg + e < g1 ? __builtin_fmaf(s1[e], a.scale_log2, -mb) : -INFINITY;
          mx = fmaxf(mx, fmaxf(sc[e], sc[4 + e]));
        }
      }
      const float mabs = mb + xmax4(mx);
      if (mabs > m_run) {
        const float alpha = __builtin_amdgcn_exp2f(m_run - mabs);   // 0 while unset
        m_run = mabs;
        l_run *= alpha;
#pragma unroll
        for (int db = 0; db < NDB; ++db) oacc[db] *= alpha;
      }
      const float mnew = m_run > kNoMax ? m_run : 0.f;
      probs(mnew - mb, true);
      nm = -mnew;
    }
    l_run += ls;
  };
  auto values = [&](const char* vt, const uint32_t (&pk)[4]) {
    const bf16x8 pb = __builtin_bit_cast(bf16x8, u32x4{pk[0], pk[1], pk[2], pk[3]});
#pragma unroll
    for (int db = 0; db < NDB; ++db) {
      const s16x4 x0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(vt + voff[db]));
      const s16x4 x1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(vt + S::UNIT + voff[db]));
      const s16x8 v8 = {x0[0], x0[1], x0[2], x0[3], x1[0], x1[1], x1[2], x1[3]};
      oacc[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, v8), pb, oacc[db], 0, 0, 0);
    }
  };

  char* const kt = kbuf + 2 * S::UNIT * w;
  char* const vt = vbuf + 2 * S::UNIT * w;
  constexpr int OPS = 2 * NI;   // vector memory operations of a step's K copy, and of its V copy
  if (first < n) {
    hi0 = rows_of(2 * first, ro0);
    hi1 = rows_of(2 * first + 1, ro1);
    copy(rk, kcol, kt);
    copy(rv, vcol, vt);
  }
  // Step c; `more`: the wave has another.  (A template, and the last step
  // apart, so that every path around the loop issues the same copies: the
  // compiler's own waits then count like these.)
  auto step = [&](int c, auto more) {
    const int h0 = hi0, h1 = hi1;
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(wait_vm(OPS));   // K has landed, V may be under way
    __builtin_amdgcn_sched_barrier(0);
    floatx4 s0 = floatx4{}, s1 = floatx4{};
    {
      bf16x8 kf[2 * NKS];
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        kf[ks] = *reinterpret_cast<const bf16x8*>(kt + koff[ks]);
        kf[NKS + ks] = *reinterpret_cast<const bf16x8*>(kt + S::UNIT + koff[ks]);
      }
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[ks], qf[ks], s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[NKS + ks], qf[ks], s1, 0, 0, 0);
      }
    }
    // The products have their operands: the next K may land in the buffer.
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (more.value) {
      hi0 = rows_of(2 * (c + stride), ro0);
      hi1 = rows_of(2 * (c + stride) + 1, ro1);
      copy(rk, kcol, kt);
    }
    __builtin_amdgcn_sched_barrier(0);
    uint32_t pk[4];
    softmax(s0, s1, h0, h1, pk);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(wait_vm(more.value ? OPS : 0));   // V has landed, the next K is under way
    __builtin_amdgcn_sched_barrier(0);
    values(vt, pk);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (more.value) copy(rv, vcol, vt);
  };
  int c = first;
  for (; c + stride < n; c += stride) step(c, std::true_type());
  if (c < n) step(c, std::false_type());

  u16* orow = static_cast<u16*>(a.o) + off + (int64_t)max(qrow, 0) * st;
  auto store = [&](int db, const floatx4& o, float inv) {
    *reinterpret_cast<uint2*>(orow + 16 * db + 4 * lg) =
        make_uint2(pack2(o[0] * inv, o[1] * inv), pack2(o[2] * inv, o[3] * inv));
  };
  if (!text) {
    const float l = xsum4(l_run);
    const float inv = l > 0.f ? 1.0f / l : 0.f;
#pragma unroll
    for (int db = 0; db < NDB; ++db) store(db, oacc[db], inv);
    return;
  }

  // Text group: each wave leaves (m, l, O) in LDS, then wave w merges and
  // stores the channel tiles w, w + 4, ...
  static_assert(NDB * 64 * 16 <= 2 * S::UNIT && 2 * 64 * 4 <= 2 * S::UNIT, "a wave's state fits its parts");
#pragma unroll
  for (int db = 0; db < NDB; ++db) *reinterpret_cast<floatx4*>(kt + 1024 * db + 16 * lane) = oacc[db];
  *reinterpret_cast<floatx2*>(vt + 8 * lane) = floatx2{m_run, l_run};
  __syncthreads();
  float m[kWaves], l[kWaves], mm = -1e30f;
#pragma unroll
  for (int x = 0; x < kWaves; ++x) {
    const floatx2 ml = *reinterpret_cast<const floatx2*>(vbuf + 2 * S::UNIT * x + 8 * lane);
    m[x] = ml[0];
    l[x] = ml[1];
    mm = fmaxf(mm, m[x]);
  }
  float lsum = 0.f;
#pragma unroll
  for (int x = 0; x < kWaves; ++x) {
    m[x] = __builtin_amdgcn_exp2f(m[x] - mm);   // the wave's weight
    lsum += l[x] * m[x];
  }
  lsum = xsum4(lsum);
  const float inv = lsum > 0.f ? 1.0f / lsum : 0.f;
  for (int db = w; db < NDB; db += kWaves) {
    floatx4 o = floatx4{};
#pragma unroll
    for (int x = 0; x < kWaves; ++x)
      o += *reinterpret_cast<const floatx4*>(kbuf + 2 * S::UNIT * x + 1024 * db + 16 * lane) * m[x];
    if (qrow >= 0) store(db, o, inv);
  }
}

template <int D>
__global__ void __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(D == 64 ? 5 : 2)))
k_attn_tile4(AttnArgs a) {
  attn_tile4<D>(a);
}

}  // namespace

hipError_t launch_attn_tile4(const AttnArgs& a0, int head_dim, hipStream_t s) {
  AttnArgs a = a0;
  if (a.dense || a.f.tile_log2 != 2 || (head_dim != 64 && head_dim != 128)) return hipErrorInvalidValue;
  a.n_text_groups = (a.f.n_text + 15) / 16;
  a.groups_per_tile = (a.n_tiles + kWaves - 1) / kWaves;
  const int64_t total = tile4_groups(a);
  if (total <= 0) return hipSuccess;
  if (total > kMaxGroups256) return hipErrorInvalidValue;
  const dim3 grid((unsigned)total), block(64 * kWaves);
  if (head_dim == 64) hipLaunchKernelGGL((k_attn_tile4<64>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((k_attn_tile4<128>), grid, block, 0, s, a);
  return hipGetLastError();
}

}  // namespace ssba
