// Greedy tree verification and top-k tree drafting of ONE sequence (Sec. 3.2.2, Appendix A.1) as device
// functions: the bodies of the two stand-alone kernels and of the fused tail of the LM head.  Lane i of a
// wavefront owns tree node i (T <= 64).
#pragma once
#include "ss_common.h"

namespace ss {

// Template of the next tree, passed by value when the caller gives per-level branching.
struct TemplateArg {
  int8_t parent[SS_MAX_T];
  int8_t rank[SS_MAX_T];
};

// The high words first; the low words only of the lanes that tie.
SS_DEV uint64_t wave_max_u64(uint64_t v) {
  const uint32_t hi = (uint32_t)(v >> 32), top = wave_max_u32(hi);
  const uint64_t tied = __ballot(hi == top);
  const uint32_t lo = (tied & (tied - 1)) == 0 ? (uint32_t)__builtin_amdgcn_readlane((int)v, (int)__builtin_ctzll(tied))
                                               : wave_max_u32(hi == top ? (uint32_t)v : 0u);
  return ((uint64_t)top << 32) | lo;
}
SS_DEV uint64_t max_u64(uint64_t a, uint64_t b) { return a > b ? a : b; }

// Acceptance is a property of a node's whole root path: every edge on it must match.  One wavefront, lane i = node i with
// its parent p, token my_tok, ancestors `anc` (reach max_depth + 1), the main stream's arg-max a_own at the node and
// a_parent at its parent: a node is accepted iff its ancestors-or-self hold no node whose edge fails.  The deepest accepted
// node wins, ties go to the lowest index.  A parent has a lower index than its child, so node i's depth is its rank among
// its ancestors and the lanes on the winner's path write their own slots.  Every wavefront of a workgroup may make the
// call; those that `write` store the results.
SS_DEV void verify_sequence(int i, int b, int my_tok, uint64_t anc, int a_own, int a_parent, int T, int max_depth,
                            bool write, int32_t* __restrict__ n_accept, int32_t* __restrict__ last, int32_t* __restrict__ bonus,
                            int32_t* __restrict__ path, int32_t* __restrict__ out_tokens, int& last_node, int& bonus_tok) {
  const bool node = i < T;
  const uint64_t fails = __ballot(node && i > 0 && my_tok != a_parent);
  const int depth = __popcll(anc) - 1;
  // key: depth * 64 + (63 - i) for accepted nodes; the root (always accepted) gives key >= 63
  const uint32_t mine = node && depth <= max_depth && (anc & fails) == 0 ? (uint32_t)(depth * 64 + (63 - i)) : 0u;
  const uint32_t key = wave_max_u32(mine);
  const int best = 63 - (int)(key & 63), best_depth = (int)(key >> 6);
  last_node = best;
  bonus_tok = __builtin_amdgcn_readlane(a_own, best);
  if (!write) return;
  if (i == 0) {
    n_accept[b] = best_depth;
    last[b] = best;
    bonus[b] = bonus_tok;
  }
  int32_t* pb = path + (size_t)b * (max_depth + 1);
  int32_t* ob = out_tokens + (size_t)b * (max_depth + 1);
  const uint64_t on_path = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(anc >> 32), best) << 32) |
                           (uint32_t)__builtin_amdgcn_readlane((int)anc, best);
  if (node && ((on_path >> i) & 1)) {
    pb[depth] = i;
    if (depth > 0) ob[depth - 1] = my_tok;
  }
  if (i <= max_depth && i >= best_depth) {
    ob[i] = i == best_depth ? bonus_tok : -1;
    if (i > best_depth) pb[i] = -1;
  }
}

// The next tree: node i of the template takes the token of rank `rank[i]` of stream `level(i)` of the
// last accepted node; the root takes the bonus token.  `topk_of_node[(j-1) * K + r]` is the token of
// rank r of stream j of that node (global memory or LDS).  One wavefront, lane i = template node i.
// `p` (clamped), `rank`: template entry i; `level` from template_level.
SS_DEV void draft_load(int i, const int32_t* __restrict__ tmpl_parent, const int32_t* __restrict__ tmpl_rank,
                       const TemplateArg& targ, int& p, int& rank) {
  if (tmpl_parent) {
    p = tmpl_parent[i];
    rank = tmpl_rank[i];
  } else {
    p = targ.parent[i];
    rank = targ.rank[i];
  }
}
SS_DEV int template_level(int i, int p, int T2, int gamma) { return __popcll(ancestors(i, p, T2, gamma + 1)) - 1; }

SS_DEV void draft_sequence(int i, int b, int p, int rank, int level, const int32_t* topk_of_node, int K, int bonus_tok,
                           int gamma, int T2, int32_t* __restrict__ next_tok, int32_t* __restrict__ next_parent) {
  if (i >= T2) return;
  int t;
  if (i == 0) t = bonus_tok;
  else if (level >= 1 && level <= gamma && rank >= 0 && rank < K) t = topk_of_node[(size_t)(level - 1) * K + rank];
  else t = -1;
  next_tok[(size_t)b * T2 + i] = t;
  if (next_parent && b == 0) next_parent[i] = p;
}

// Host: the template argument of a draft call from per-level branching (checks it against K and T2).
int draft_template_from_branching(const char* fn, const int32_t* branching, int gamma, int K, int T2, TemplateArg* targ);

}  // namespace ss
