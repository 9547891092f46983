// Split plan and workspace layout of the decode path, and the choice between
// its kernels: the table kernels (decode_lut.hip, decode_lut64.hip) and, for
// the head counts and layouts outside them, decode_vq.hip.
#include <algorithm>

#include "nova_kv_internal.h"

namespace novakv {

namespace {

// Split count that sizes the workspace: it covers every plan below, and stays
// what it was, so a workspace sized for a shape keeps serving it.
int workspace_splits(int batch, int num_kv_heads, int max_seq_len) {
  int c = 1024;
  auto splits = [&](int cc) { return (max_seq_len + cc - 1) / cc; };
  while (c > 64 && static_cast<long long>(batch) * num_kv_heads * splits(c) < 2048) c /= 2;
  return splits(c);
}

// Splits of decode_vq: one workgroup fills a CU, so the launch takes
// ceil(units * splits / 256) rounds of (setup + chunk).  The setup and tail of
// a workgroup cost about as much as 2000 tokens, and one more split adds about
// 40 tokens' time to the combine.  With a band a split's partial takes two rows
// of the workspace: at most `limit` splits where there are several.
void plan_vq(long long units, int span, int limit, int *n_split, int *chunk) {
  long long best = 0;
  const long long most = std::min<long long>(limit, 512 / units + 1);  // past two rounds of one unit's share nothing is gained
  for (int ns = 1; ns <= most; ++ns) {
    const int ch = ((span + ns - 1) / ns + 63) & ~63;
    const int n = (span + ch - 1) / ch;
    const long long cost = (units * n + 255) / 256 * (2000 + ch) + 40 * n;
    if (ns == 1 || cost < best) {
      best = cost;
      *n_split = n;
      *chunk = ch;
    }
  }
}

}  // namespace

DecodePlan plan_decode(int batch, int num_q_heads, int num_kv_heads, int head_dim,
                       int max_seq_len, int block_size, int window) {
  DecodePlan p{};
  const int gqa = num_q_heads / num_kv_heads;
  // Splits tile the attended span: the last `window` tokens, or all of them.
  const int span = window > 0 && window < max_seq_len ? window : max_seq_len;
  // Workspace bound over every window: the split count above, and the table
  // plan's split target (its split count never exceeds it).
  const int ns_full = workspace_splits(batch, num_kv_heads, max_seq_len);
  const long long units = static_cast<long long>(batch) * num_kv_heads;
  const int lut_bound = static_cast<int>((256 + units - 1) / units);
  const int max_split = ns_full > lut_bound ? ns_full : lut_bound;
  p.n_split = 1;
  p.chunk = span;
  if (block_size > 0) {
    p.use_lut = lut_path_eligible(head_dim, gqa, block_size) ? 1 : 0;
    if (p.use_lut)
      plan_lut(batch, num_kv_heads, span, &p.n_split, &p.chunk);
    else
      plan_vq(units, span, max_split / 2 > 1 ? max_split / 2 : 1, &p.n_split, &p.chunk);
  }
  auto align = [](size_t x) { return (x + 255) & ~static_cast<size_t>(255); };
  const size_t rows = static_cast<size_t>(batch) * num_q_heads;
  // groups of the two-level combine, at most, over every split count up to the bound
  int max_group = 1;
  for (int n = 1; n <= max_split; ++n) {
    const int gs = plan_group_size(n), ng = (n + gs - 1) / gs;
    if (ng > max_group) max_group = ng;
  }
  p.off_cnt = 0;
  // the gap after the counters held the pre-transformed queries and sink
  // logits of a separate launch; a workspace keeps its size and layout
  const size_t gap = align(align(static_cast<size_t>(units) * (1 + max_group) * sizeof(int)) + rows * head_dim * sizeof(float));
  p.off_ml = align(gap + rows * sizeof(float));
  p.off_acc = align(p.off_ml + rows * max_split * 2 * sizeof(float));
  p.off_new = align(p.off_acc + rows * max_split * head_dim * sizeof(float));
  p.off_xch = align(p.off_new + static_cast<size_t>(batch) * num_kv_heads * 8 * 32 * sizeof(float));
  p.off_xnew = align(p.off_xch + units * max_split * kXchSlotWords * sizeof(uint64_t));
  p.off_xgrp = align(p.off_xnew + static_cast<size_t>(units) * 8 * 32 * sizeof(uint64_t));
  p.total = align(p.off_xgrp + units * max_group * kXchSlotWords * sizeof(uint64_t));
  return p;
}

hipError_t launch_decode(const DecodeArgs &a, int use_lut, hipStream_t stream) {
  if (!use_lut) return launch_decode_vq(a, stream);
  return a.head_dim == 128 ? launch_decode_lut(a, stream) : launch_decode_lut64(a, stream);
}

}  // namespace novakv
