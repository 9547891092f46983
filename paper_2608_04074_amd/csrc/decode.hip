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

// Splits per (sequence, KV head).  A workgroup of any decode kernel fills a CU,
// so a launch takes ceil(units * splits / 256) rounds, and each round costs its
// setup and tail beside the chunk; every split adds to the combine.  All in
// tokens' time of the kernel:
//   cost = rounds * (setup + chunk) + splits * split (+ levels, two-level combine)
// A last round that is nearly empty so loses to fewer, longer splits: 12
// sequences of 8192 tokens (96 units) take 36.8 us in 3 splits (288 workgroups),
// 23.9 us in 2; 40 of 16384 tokens (320 units) 110 us in 1, 103 us in 2 (3
// rounds); 24 of 2000 tokens 29.4 us in 2, 17.2 us in 1.
//
// A step adds its token's encode, the cheapest of:
//   workgroups  where units * (splits + 1..) fit the CUs (step_encode.h): next to
//               nothing (a step of 2000 tokens, 8 KV heads: 15.2 us, against 19.6
//               by teams and 18.4 in two launches; in the deployed format
//               with a band 22.9 against 31.0);
//   teams       the splits encode between them, beside their token loops: about
//               2.5 us and 3 us per item that the loop does not hide (head_dim
//               128 without a scaled format, or any format with a band);
//   two launches  4.5 us, 11 us in the scaled formats.
struct SplitCost {
  int setup, split, levels;
  int launch, launch_scaled, team, item, item_scaled;  // a step's encode
  int teams;                              // encoder teams of an encoder workgroup
  int even;                               // tokens of one round per wave (0: no such rule)
  int row;                                // a band row, where the splits share the band
};

struct Splits {
  int n_split, chunk, enc_per_unit;
  StepMode step;
};

Splits plan_splits(const SplitCost &c, const int units, const int span, const int limit, const int band_rows,
                   const StepFormat *step, const bool teams_ok, const bool one_split_ok, const bool workgroups_ok) {
  constexpr int kCUs = 256, kMinChunk = 192;
  const int most = std::min(limit, std::max(1, 4 * kCUs / units));
  Splits best{1, span, 0, kStepTwoLaunches};
  long long best_cost = -1;
  // Where one launch round has room for splits of one 64-token round per wave,
  // only such are taken: every round then has a softmax reference of its own,
  // and the result does not depend on how the span is split.
  const int one_round = std::min(limit, kCUs / units);
  const bool even = c.even > 0 && one_round > 0 && ((span - 1) / one_round + 64) / 64 * 64 <= c.even;
  auto consider = [&](const int ns) {
    const int ch = std::max(((span - 1) / ns + 64) & ~63, kMinChunk);
    const int n = (span - 1) / ch + 1;
    if (even && ch > c.even) return;
    const long long rounds = (units * n + kCUs - 1) / kCUs;
    long long cost = rounds * (c.setup + ch) + n * c.split + (n > kXchBatch + 1 ? c.levels : 0) + band_rows * c.row / n;
    Splits s{n, ch, 0, kStepTwoLaunches};
    if (step) {
      long long extra = step->scaled ? c.launch_scaled : c.launch;
      if (teams_ok && (n > 1 || one_split_ok)) {
        const int items = (step->tasks + n - 1) / n;
        const long long t = c.team + std::max(0, items * (step->scaled ? c.item_scaled : c.item) - ch);
        if (t < extra) {
          extra = t;
          s.step = kStepTeams;
        }
      }
      const int free = kCUs / units - n;  // workgroups a unit may add within the round
      const int want = workgroups_ok ? (step->tasks + c.teams - 1) / c.teams : 0;
      if (want > 0 && free >= 1) {
        extra = 0;
        s.step = kStepWorkgroups;
        s.enc_per_unit = std::min(free, want);
      }
      cost += extra;
    }
    if (best_cost < 0 || cost < best_cost) {
      best_cost = cost;
      best = s;
    }
  };
  for (int ns = 1; ns <= most; ns += std::max(1, ns / 8)) consider(ns);
  if (one_round > 1) consider(one_round);  // every CU
  return best;
}
// head_dim 128: 2.7 ns a token and CU, 12.5 us a round; head_dim 64: 1.9 ns and 12
// us, decode_vq: 4 ns and 16 us, both with splits that wait for their stores
// (0.35 and 0.4 us each in the combine).
constexpr SplitCost kCost128 = {4600, 30, 650, 1700, 4000, 900, 1100, 2500, 3, 12 * 64, 7},
                    kCost64 = {6300, 180, 0, 2400, 5700, 1200, 0, 0, 4, 16 * 64, 0},
                    kCostVq = {4000, 100, 0, 0, 0, 0, 0, 0, 0, 0, 3};

}  // namespace

bool lut_path_eligible(int head_dim, int gqa, int block_size) {
  return block_size % 16 == 0 && ((head_dim == 128 && gqa <= 4) || (head_dim == 64 && gqa <= 8));
}

// Sequences per block of the table kernels' workgroup order: the largest
// divisor of batch that leaves about two KV heads (all their splits) in each
// XCD's eighth of the grid.  Same-box timing at B=8, 8 KV heads, 4 splits:
// two KV heads per XCD beat both one (32 CUs of one L2 request the same
// parameter lines at once) and eight (every L2 fetches every KV head's
// parameters).
// One combine reads up to kXchBatch other slots in one round trip; above
// that the splits are merged in groups of about sqrt(n_split) splits (a power
// of two, at most 32) first.
int plan_group_size(int n_split) {
  if (n_split <= kXchBatch + 1) return n_split > 0 ? n_split : 1;
  int gs = 2;
  while (gs < 32 && gs * gs < n_split) gs *= 2;
  return gs;
}

int plan_b_chunk(int batch, int num_kv_heads, int n_split) {
  const long long grid = static_cast<long long>(batch) * num_kv_heads * n_split;
  const long long per_xcd = grid / 8 > 0 ? grid / 8 : 1;
  long long target = per_xcd / (2LL * n_split);
  if (target < 1) target = 1;
  int bc = 1;
  for (int d = 1; d <= batch && d <= target; ++d)
    if (batch % d == 0) bc = d;
  return bc;
}

DecodePlan plan_decode(int batch, int num_q_heads, int num_kv_heads, int head_dim,
                       int max_seq_len, int block_size, int window, int band_rows, const StepFormat *step) {
  DecodePlan p{};
  const int gqa = num_q_heads / num_kv_heads;
  // Splits tile the attended span: the last `window` tokens, or all of them.
  const int span = window > 0 && window < max_seq_len ? window : max_seq_len;
  // Workspace bound over every window, which also bounds the plan.
  const int ns_full = workspace_splits(batch, num_kv_heads, max_seq_len);
  const long long units = static_cast<long long>(batch) * num_kv_heads;
  const int lut_bound = static_cast<int>((256 + units - 1) / units);
  const int max_split = ns_full > lut_bound ? ns_full : lut_bound;
  p.n_split = 1;
  p.chunk = span;
  if (block_size > 0) {
    p.use_lut = lut_path_eligible(head_dim, gqa, block_size) ? 1 : 0;
    const SplitCost &cost = !p.use_lut ? kCostVq : (head_dim == 128 ? kCost128 : kCost64);
    // with a band a split's partial of decode_vq takes two rows of the workspace
    const int limit = p.use_lut ? max_split : std::max(1, max_split / 2);
    // Teams: with the token in the band, any format; without a band at head_dim
    // 128, unscaled, over several splits.  The head_dim-64 kernel encodes in the
    // first split to arrive, the head_dim-128 one on a contiguous cache also in
    // an only split.
    const bool teams_ok = p.use_lut && step && (step->in_band || (step->no_band && head_dim == 128 && !step->scaled));
    const bool one_split_ok = step && step->in_band && (head_dim == 64 || !step->paged);
    const bool workgroups_ok = p.use_lut && step && (step->no_band || step->in_band);
    const Splits s =
        plan_splits(cost, static_cast<int>(units), span, limit, band_rows, step, teams_ok, one_split_ok, workgroups_ok);
    p.n_split = s.n_split;
    p.chunk = s.chunk;
    p.step = s.step;
    p.enc_per_unit = s.enc_per_unit;
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
  // The counters must be zero between calls, also where one workspace serves
  // calls of several shapes: no call may store anything else where another's
  // counters lie.  Plans with several splits have at most 384 units, so those of
  // the kernels with plain partials end before kCounterBytes (3072 in the
  // head_dim-128 table kernel, whose partials are far from there).  The partials
  // start past them as far as the two gaps allow, which held the queries of a
  // separate launch and a step's results, and keep a workspace's size and the
  // exchange's place what they were.
  constexpr size_t kCounterBytes = 3072;
  const size_t gap = align(align(static_cast<size_t>(units) * (1 + max_group) * sizeof(int)) + rows * head_dim * sizeof(float));
  const size_t gap2_bytes = static_cast<size_t>(units) * 8 * 32 * sizeof(float);
  const size_t ml0 = align(gap + rows * sizeof(float));
  p.off_ml = std::max(ml0, std::min(kCounterBytes, ml0 + gap2_bytes));
  const size_t after_ml = align(rows * max_split * 2 * sizeof(float));
  p.off_acc = p.off_ml + after_ml;
  const size_t gap2 = align(ml0 + after_ml + rows * max_split * head_dim * sizeof(float));
  p.off_xch = align(gap2 + static_cast<size_t>(batch) * num_kv_heads * 8 * 32 * sizeof(float));
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
