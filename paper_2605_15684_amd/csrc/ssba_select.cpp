// Host-side kernel selection: which attention and backward kernels a
// descriptor's shape is served by, and their names as profilers show them.
// Host code only (no kernels), so the argument-checking and dispatch layer
// can also be built and exercised on a CPU.
#include "ssba_common.h"

namespace ssba {

namespace {
constexpr int kMfmaChunk = 64;   // keys per chunk of the MFMA attention kernels
}  // namespace

const char* mfma_kernel_name(int head_dim, int tile, bool dense, bool gated) {
  static const char* const names[2][2][2] = {
      {{"k_attn_mfma<64, 3, false, false>", "k_attn_mfma<64, 3, true, false>"},
       {"k_attn_mfma<64, 4, false, false>", "k_attn_mfma<64, 4, true, false>"}},
      {{"k_attn_mfma<128, 3, false, false>", "k_attn_mfma<128, 3, true, false>"},
       {"k_attn_mfma<128, 4, false, false>", "k_attn_mfma<128, 4, true, false>"}}};
  if (gated && !dense) return head_dim == 64 ? "k_attn_mfma<64, 3, false, true>" : "k_attn_mfma<128, 3, false, true>";
  // The dense control runs natural-order rows only; it uses the 8x8 shape.
  const int ti = (!dense && tile == 16) ? 1 : 0;
  return names[head_dim == 64 ? 0 : 1][ti][dense ? 1 : 0];
}

bool mfma_supported(int head_dim, int tile, bool dense, int n_tiles, int seq, int64_t span) {
  // 32-bit byte offsets inside one (batch, head); at most 64 kept blocks;
  // natural-order chunks need at least one full chunk of rows.
  return (head_dim == 64 || head_dim == 128) && (dense || ((tile == 8 || tile == 16) && n_tiles <= 64)) &&
         seq >= kMfmaChunk && 2 * span < ((int64_t)1 << 32);
}

bool mfma_long_supported(int head_dim, int tile, int n_tiles, int seq, int64_t span) {
  // As mfma_supported, with a list that passes through the lanes in parts, and
  // offsets that also reach the rows past the last that a ragged chunk names.
  return (head_dim == 64 || head_dim == 128) && (tile == 8 || tile == 16) && n_tiles > 64 && seq >= kMfmaChunk &&
         2 * (span + span / seq * kMfmaChunk) < ((int64_t)1 << 32);
}

int64_t tile4_groups(const AttnArgs& a) {
  // 16 text rows a group (a multiple of 8 of them), or four blocks.
  const int64_t pairs = (int64_t)a.batch * a.heads;
  return ((pairs * ((a.f.n_text + 15) / 16) + 7) & ~(int64_t)7) + pairs * ((a.n_tiles + 3) / 4);
}

bool tile4_supported(const AttnArgs& a, int head_dim, int tile) {
  // Byte offsets inside one (batch, head) below 2^31: the next value up marks
  // a row that is not there.  Its groups of few blocks or rows take up to four
  // times the threads of the generic kernel, which keeps what passes a launch.
  return (head_dim == 64 || head_dim == 128) && tile == 4 && !a.dense &&
         2 * (int64_t)a.seq * a.st < ((int64_t)1 << 31) && tile4_groups(a) <= kMaxGroups256;
}

const char* attn_kernel_name(const AttnArgs& a, int head_dim, int tile, int dtype) {
  if (dtype == SSBA_DT_F32) return head_dim == 64 ? "k_attn_f32<64>" : "k_attn_f32<128>";
  if (mfma_supported(head_dim, tile, a.dense != 0, a.n_tiles, a.seq, (int64_t)a.seq * a.st))
    return mfma_kernel_name(head_dim, tile, a.dense != 0, a.gated != 0);
  if (!a.dense && mfma_long_supported(head_dim, tile, a.n_tiles, a.seq, (int64_t)a.seq * a.st)) {
    static const char* const longs[2][2] = {{"k_attn_mfma_long<64, 3>", "k_attn_mfma_long<64, 4>"},
                                            {"k_attn_mfma_long<128, 3>", "k_attn_mfma_long<128, 4>"}};
    return longs[head_dim == 64 ? 0 : 1][tile == 16 ? 1 : 0];
  }
  if (tile4_supported(a, head_dim, tile)) return head_dim == 64 ? "k_attn_tile4<64>" : "k_attn_tile4<128>";
  static const char* const names[2][3] = {
      {"k_attn_bf16<64, 2>", "k_attn_bf16<64, 3>", "k_attn_bf16<64, 4>"},
      {"k_attn_bf16<128, 2>", "k_attn_bf16<128, 3>", "k_attn_bf16<128, 4>"}};
  return names[head_dim == 64 ? 0 : 1][tile == 4 ? 0 : tile == 8 ? 1 : 2];
}

bool bwd_supported(int head_dim, int tile, int n_tiles, int dtype) {
  return dtype == SSBA_DT_BF16 && (head_dim == 64 || head_dim == 128) && (tile == 8 || tile == 16) &&
         n_tiles <= 64;
}

}  // namespace ssba
