// Shared declarations of the multi-stream attention kernels (a2).
#pragma once

#include "ss_common.h"

namespace ss {

// Everything a workgroup needs; passed by value.
struct MsaArgs {
  const void* q;
  const void* k_new;
  const void* v_new;
  const void* k_cache;
  const void* v_cache;
  const int32_t* block_table;
  const int32_t* seq_lens;
  const int32_t* parent;
  const int32_t* n_nodes;  // [B] kept nodes per sequence after pruning (rows of the others are not computed), or NULL
  void* out;
  float* part_o;    // [rows,D]  per-split outputs, already divided by their own sum (part_row_of: which row)
  float* part_lse;  // [rows]    log2-domain log-sum-exp of each split
  int B, T, gamma, R, H, Hkv, g, D;
  int page, page_shift, max_pages, num_pages;
  int split_keys;  // cached tokens per split (multiple of 32; of 64 for the fp32 kernel)
  int split0_keys; // cached tokens of split 0 (MFMA path: shorter, that split also scans the step's own rows)
  int n_splits;    // S: upper bound on splits per sequence
  int n_qc;        // query-row chunks per (sequence, KV head) (MFMA path)
  int groups;      // wave groups per workgroup the plan asks for (MFMA path)
  int stages;      // ring stages per wave group the plan asks for (MFMA path)
  unsigned int* arrive;  // MFMA path, splits merged inside the kernel (two, or a few of few rows): arrival counters
                         // [B,Hkv,n_qc,kArriveTiles] in the workspace (zero before the call, zero again after it), else NULL
  float scale_log2;  // softmax scale times log2(e)
  uint32_t flags;
  int n_groups, n_stages;  // what the launch has of `groups` and `stages`
  int n_extra;             // stages per wave group for more blocks of the step's own rows (MFMA path)
  int by_split;            // whether the split is the slowest index of the workgroups (MFMA path)
  // last, so that kernels that do not cut read no more of the arguments than they need
  int2* cut_table;  // [B] adaptive calls: splits and first slot of every sequence, which workgroup 0 of the attention
                    // kernel leaves in the workspace for the merge kernel; else NULL
  int adaptive;    // 1: a batch the host's split lengths do not fit is cut anew on the device (plan_uneven)
  int even_len;    // 7/8 of the capacity, in tokens
  int even_work;   // 7/8 of the whole plan's blocks times row chunks, or 0: not looked at (plan_is_even)
  int new_units;   // blocks' worth of time that scanning the step's own rows costs split 0
  int max_n;       // most splits per sequence plan_uneven may make (2: merged in the kernel; else 0 = no limit)
  int min_units;   // shortest split plan_uneven considers, in blocks
  int chunk_rows;  // folded query rows per row chunk (MFMA path)
  int xcd_slots;   // workgroups an XCD holds at a time
  float cut_fixed, cut_piece;  // what a round and a piece cost beside their blocks, in blocks (cut_cost)
};

// A sequence of L cached tokens has active_splits(L) splits; every sequence has at least one (split 0, which
// also scans the step's new keys).  Split 0 takes the tokens [0, min(L, split0_keys)), split s > 0 the
// tokens [split_begin(s), min(L, split_begin(s) + split_keys)).
SS_HD int clamp_len(int L, const MsaArgs& a) { return min(max(L, 0), a.max_pages * a.page); }
SS_HD int active_splits(int L, const MsaArgs& a) {
  return L <= a.split0_keys ? 1 : 1 + (L - a.split0_keys + a.split_keys - 1) / a.split_keys;
}
// Kept nodes of sequence b: all T unless the call passes n_nodes (clamped to [1,T]).
SS_DEV int kept_nodes(int b, const MsaArgs& a) { return a.n_nodes ? min(max(a.n_nodes[b], 1), a.T) : a.T; }
SS_DEV int split_begin(int s, const MsaArgs& a) { return s == 0 ? 0 : a.split0_keys + (s - 1) * a.split_keys; }
SS_DEV int split_len(int s, const MsaArgs& a) { return s == 0 ? a.split0_keys : a.split_keys; }

// Row of the partial results of (sequence, split, query head, query row).  The splits of a sequence's head lie together,
// [B,H,S,R].  Where the device cuts the sequences (below) it deals out the B*S slots, a sequence's from slot0 on, and
// they lie by slot, [B*S,H,R].
template <bool CUTS>
SS_DEV size_t part_row_of(const MsaArgs& a, int b, int slot0, int s, int h, int r) {
  return CUTS ? ((size_t)(slot0 + s) * a.H + h) * a.R + r : (((size_t)b * a.H + h) * a.n_splits + s) * a.R + r;
}

// ---- splits cut on the device.  The host plans from the capacity of the block table; what the sequences really
// hold (and, after pruning, how many row chunks they have) is known on the device only.  Where the
// host's cut stands (plan_is_even) it is used as it is.  Otherwise the lengths are chosen here, by one wavefront, from 64
// candidates: the one with the least (rounds of the workgroups an XCD holds) x (blocks per workgroup + a fixed cost) + what
// the pieces' partial results cost, among those whose splits fit the B x S slots of the workspace.  16 rows per wave, 32
// workgroups: a fixed cost of 4 (0, 2, 8, 16 instead: 20 random batches of fewer than 256 items within 0.2 %, four of 320
// items +2.4, 0, -1.4, -3.3 %).  32 rows per wave, 64 workgroups: 8, and a fiftieth per piece (two sequences of 9005 and
// 3001 tokens in a table of 1.8 times the capacity, 8 KV heads, 384 rows: 47.3 us with 4 and nothing per piece, 44.6; four
// sequences 67.2 and 61.9).  Lane b holds sequence b, so this is for B <= kAdaptiveMaxB.
// Measured with the merge kernel, host's cut against this: two sequences of 9005 and 3001 tokens (8 KV heads of 4 query
// heads, 24 nodes) in a table of 1.8 times the capacity 59.7 and 43.3 us; eight of 2000..8192 tokens with a third to two
// thirds of 32 nodes kept 179 and 135 us; three of 16000, 9005 and 3001 with 4 KV heads 126 and 77 us (84 with the pieces
// of a sequence rounded up to whole eights).
constexpr int kAdaptiveMaxB = 64;
SS_HD int len_units(int L, const MsaArgs& a) { return (clamp_len(L, a) + 31) >> 5; }
SS_HD bool seq_is_even(const MsaArgs& a, int len, int kept) { return len >= a.even_len && kept == a.T; }
SS_DEV int wave_sum(int v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
SS_DEV int wave_scan(int v, int lane) {  // inclusive
  for (int off = 1; off < 64; off <<= 1) {
    const int o = __shfl_up(v, off, 64);
    if (lane >= off) v += o;
  }
  return v;
}
// The arithmetic of a cut, the same on the device (a lane per candidate) and in ss_msa_plan_splits (one after the other).
// Blocks' worth of time that a sequence of U cached blocks takes; at least one, for an empty sequence has a split 0 and
// so a slot too, also where the step's own rows are set to count for nothing.
SS_HD int cut_load(const MsaArgs& a, int U) { return max(U + a.new_units, 1); }
SS_HD int cut_chunks(const MsaArgs& a, int kept) { return (a.g * kept * (1 + a.gamma) + a.chunk_rows - 1) / a.chunk_rows; }
// Shortest and longest split that is considered, from the sum and the largest of the loads.  Rounding the sum down keeps
// every candidate worth a look; what does not fit the slots is dropped by its cost (of launches that are cut the attention
// kernel merges two splits of a sequence at most).
struct CutRange {
  int lo, hi;
};
SS_HD CutRange cut_range(const MsaArgs& a, int sum, int most) {
  const int fill = (int)((float)sum / (float)(a.B * a.n_splits)), floor2 = a.max_n == 2 ? (most + 1) / 2 : 1;
  const int lo = max(max(a.min_units, fill), floor2);
  return CutRange{lo, max(most, lo)};
}
// Candidate j of 64: geometric steps from lo to hi; the last leaves every sequence whole, which always fits.
SS_HD int cut_candidate(const MsaArgs& a, int j, CutRange r) {
#ifdef __HIP_DEVICE_COMPILE__
  const float up = __builtin_amdgcn_exp2f(__log2f((float)r.hi / (float)r.lo) * ((float)j * (1.f / 63.f)));
#else
  const float up = exp2f(log2f((float)r.hi / (float)r.lo) * ((float)j * (1.f / 63.f)));
#endif
  const int c = j == 63 ? r.hi : min(r.hi, (int)((float)r.lo * up));
  return (max(c, r.lo) + a.groups - 1) / a.groups * a.groups;
}
// Cost of splits of c blocks; load(i), chunks(i): of sequence i.
template <class Load, class Chunks>
SS_HD float cut_cost(const MsaArgs& a, int c, Load load, Chunks chunks) {
  const float rc = 1.f / (float)c;
  int slots = 0, xcd0 = 0, all = 0;
  for (int i = 0; i < a.B; ++i) {
    const int up = load(i) + c - 1;
    int q = (int)((float)up * rc);  // off by one at most
    const int rem = up - q * c;
    q += (rem >= c) - (rem < 0);
    const int before = slots * a.Hkv, after = before + q * a.Hkv;  // pieces, dealt to the XCDs in turn
    slots += q;
    xcd0 += (((after + 7) >> 3) - ((before + 7) >> 3)) * chunks(i);
    all += (after - before) * chunks(i);
  }
  // Rounds of the workgroups an XCD holds, on the XCD with the most: XCD 0 has as many pieces as any, and where the
  // sequences' row chunks differ at least the average.
  const int rounds = (max(xcd0, (all + 7) >> 3) + a.xcd_slots - 1) >> (a.xcd_slots == 32 ? 5 : 6);
  return slots <= a.B * a.n_splits ? (float)rounds * ((float)c + a.cut_fixed) + (float)all * a.cut_piece : INFINITY;
}
// Of one sequence: cached blocks of split 0 and of the others, number of splits, row chunks with kept rows.
struct SeqCut {
  int split0, split, n, chunks;
};
SS_HD SeqCut cut_of(const MsaArgs& a, int cut, int U, int chunks) {
  const int x = cut_load(a, U), q = max(1, (x + cut - 1) / cut), even = (x + q - 1) / q;
  SeqCut r;
  r.split = max((even + a.groups - 1) / a.groups, 1) * a.groups;
  r.split0 = max(0, r.split - a.new_units);
  r.n = U <= r.split0 ? 1 : 1 + (U - r.split0 + r.split - 1) / r.split;  // <= q
  r.chunks = chunks;
  return r;
}
// The host's cut stands when every sequence fills 7/8 of the capacity and no node was removed.  With 256 items or more
// also when what there is to do, blocks times row chunks over all sequences, is 7/8 of what the host planned for: each
// round of workgroups pays 2.6 us for cutting anew, and only that much less work makes up for it (eight sequences of up to
// 8192 tokens, 160 rows, 320 items in 5 rounds, us with the host's and with the device's cut: all full 246 and 259, at 9/10
// 237 and 241, at 7/8 236 and 235, at 0.7 234 and 209; one of them at 1/2, the others full 240 and 253).  With fewer items
// the device's cut is the better one full or not (48 items over 16384 tokens 112 and 75, 96 over 8192 114 and 86; one
// of two sequences at 0.8 105 and 72): the host's plan does not count rounds there.
// Every wave comes to this before it knows its piece, so the sum is the scalar unit's (a lane read and an add per sequence)
// and the division by the chunk's rows one by a constant.
template <int CHUNK_ROWS>
SS_DEV bool plan_is_even(const MsaArgs& a, int lane, int len, int kept) {
  if (__all(lane >= a.B || seq_is_even(a, len, kept))) return true;
  if (a.even_work == 0) return false;
  const int work = len_units(len, a) * ((a.g * kept * (1 + a.gamma) + CHUNK_ROWS - 1) / CHUNK_ROWS);
  int sum = 0;
  for (int i = 0; i < a.B; ++i) sum += __builtin_amdgcn_readlane(work, i);
  return sum >= a.even_work;
}
SS_DEV SeqCut plan_uneven(const MsaArgs& a, int lane, int U, int kept) {
  const bool mine = lane < a.B;
  const int x = mine ? cut_load(a, U) : 0, chunks = mine ? cut_chunks(a, kept) : 0;
  int x_max = x;
  for (int off = 32; off > 0; off >>= 1) x_max = max(x_max, __shfl_xor(x_max, off, 64));
  const int c = cut_candidate(a, lane, cut_range(a, wave_sum(x), x_max));
  const float cost = cut_cost(a, c, [&](int i) { return __builtin_amdgcn_readlane(x, i); },
                              [&](int i) { return __builtin_amdgcn_readlane(chunks, i); });
  float best = cost;
  for (int off = 32; off > 0; off >>= 1) best = fminf(best, __shfl_xor(best, off, 64));
  const int win = 63 - __builtin_clzll(__ballot(cost == best));  // the longest splits among equals
  SeqCut r = cut_of(a, __builtin_amdgcn_readlane(c, win), U, chunks);
  if (!mine) r.n = 0;
  return r;
}

// Arrival counters of the in-kernel split merge: one per (sequence, KV head, row chunk, query tile of at most
// kArriveTiles per chunk).
// They lie in front of the workspace, in a region of the same size for every shape: they have to be zero when a call
// begins, so no shape may leave anything else where another shape looks for them.  8192 (sequence, KV head, row chunk)
// items fit, 32 rounds of workgroups; calls of more take the merge kernel (same bits).
constexpr int kArriveTiles = 8;
constexpr size_t kArriveRegionBytes = (size_t)8192 * kArriveTiles * sizeof(unsigned int);

// MFMA path (bf16, D = 64 or 128).  Returns SS_OK or an error code.
int launch_msa_bf16(const MsaArgs& a, hipStream_t stream);
// Query rows per workgroup chunk the MFMA path uses for F = g*R folded rows.
int msa_bf16_rows_per_chunk(int F);
// The launch of that kernel: workgroups, wave groups of each, ring stages per group, stages per group for more of the step's
// own rows, waves and bytes of LDS per workgroup; whether the split is the slowest index of the workgroups.
struct MsaLaunch {
  long wgs;
  int groups, stages, extra, waves;
  bool by_split;
  size_t lds;
};
MsaLaunch msa_bf16_launch(const MsaArgs& a);

// The same with 32 query rows per wave (D = 128, more than 80 folded rows).
constexpr int kWideSlots = 512;  // workgroups the chip holds at a time: two per compute unit
MsaLaunch msa_bf16_wide_launch(const MsaArgs& a);
int launch_msa_bf16_wide(const MsaArgs& a, hipStream_t stream);
int msa_bf16_wide_rows(int F);

}  // namespace ss
