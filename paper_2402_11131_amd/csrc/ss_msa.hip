// a2: multi-stream attention (Eq. 1 main rows, Eq. 2 stream rows) over a paged
// KV cache.  This file holds the entry point, the split planning, the fp32
// kernel and the kernel that merges the per-split partial results.
#include <math.h>
#include <stdlib.h>

#include <atomic>
#include <mutex>

#include "ss_msa.h"

namespace ss {

// ------------------------------------------------------------------ fp32 kernel
//
// One workgroup = (row chunk of 4*RW rows, split, sequence, head); wave w owns RW of the rows.  Keys are taken 64 at a
// time: the K tile sits in LDS token-major, the V tile feature-major, rows padded by 16 bytes (16-byte reads of 16
// lanes then meet 64 different banks); in the score phase a lane owns a key, in the P.V phase it owns output features.
// Softmax is the usual running max / running sum in the log2 domain.
//
// Small problems are all latency: a tile's values are fetched into registers while the tile before is computed, with
// one page lookup per lane (the wave's other lanes' rows come by lane reads); the queries are asked for before the first
// lookup is waited for.  A tile's maximum is taken by register moves and a row's sum once, at the end (by lane shuffles, and
// each tile: 10 us of 40 rows' 15).  Operands leave LDS four steps at a time, two with heads of 128: the code of more of them
// is fetched cold by every launch (eight: 11.9 -> 14.4 us).  RW = 8, 2 or 1 (see the launch).  Before and after, one layer:
// 4 heads of 64, 128 cached tokens, 40 rows 15.0 -> 9.8 us; 8 heads of 64, 4 sequences of 500..1000 tokens, 192 rows (RW = 8)
// 109 -> 92; 16 heads of 128, 8000 tokens, 40 rows 202 -> 150; 32 of 128 on 8, 4 sequences of 500..1000, 80 rows 331 -> 245.
template <int D, int RW>
__global__ __launch_bounds__(256) void msa_f32_kernel(MsaArgs a) {
  constexpr int RC = 4 * RW, KT = 64, DL = D / 64;
  constexpr int NL = KT * D / 256;  // values of a K (or V) tile per thread
  __shared__ __attribute__((aligned(16))) float Qs[RC][D];
  __shared__ __attribute__((aligned(16))) float Ks[KT][D + 4];
  __shared__ __attribute__((aligned(16))) float Vs[D][KT + 4];
  __shared__ __attribute__((aligned(16))) float Ps[4][RW][KT];

  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int chunk = blockIdx.x, s = blockIdx.y;
  const int b = blockIdx.z / a.H, h = blockIdx.z % a.H, hk = h / a.g;
  const int L = clamp_len(a.seq_lens[b], a);
  const int n_active = active_splits(L, a);
  if (s >= n_active) return;
  const bool is_last = (s == n_active - 1);
  const int k0 = split_begin(s, a);
  const int n_prefix = max(0, min(L, k0 + split_len(s, a)) - k0);
  const int n_new = is_last ? a.R : 0;
  const int total = n_prefix + n_new;
  const int r0 = chunk * RC;
  const int R = a.R, T = a.T;
  const int n_kept = kept_nodes(b, a);

  const float* q = (const float*)a.q;
  const float* k_new = (const float*)a.k_new;
  const float* v_new = (const float*)a.v_new;
  const float* k_cache = (const float*)a.k_cache;
  const float* v_cache = (const float*)a.v_cache;

  const int par = a.parent[(size_t)b * T + min(lane, T - 1)];
  float qv[RC * D / 256];  // asked for before, and put down after, the first tile's page lookup is waited for
#pragma unroll
  for (int i = 0; i < RC * D / 256; ++i) {
    const int r = (tid + 256 * i) / D, d = (tid + 256 * i) % D;
    qv[i] = q[(((size_t)b * R + min(r0 + r, R - 1)) * a.H + h) * D + d];
  }

  // Tile t0's values on their way to registers.  Of K a wave takes whole rows (or halves), of V whole features of the
  // 64 tokens.  Keys past the end repeat the last one; their scores are masked, and their V becomes zero.
  float kv[NL], vv[NL];
  const int w_u = __builtin_amdgcn_readfirstlane(w);
  auto fetch = [&](int t0) {
    const int u = min(t0 + lane, total - 1);  // this lane's key
    const float *kp, *vp;
    int vstride;
    if (u < n_prefix) {
      const int tok = k0 + u;
      int pg = a.block_table[(size_t)b * a.max_pages + (tok >> a.page_shift)];
      pg = min(max(pg, 0), a.num_pages - 1);
      const size_t head = ((size_t)pg * a.Hkv + hk) * a.page * D;
      const int at = tok & (a.page - 1);
      kp = k_cache + head + (size_t)at * D;
      vp = v_cache + head + at;
      vstride = a.page;
    } else {
      const size_t row = (((size_t)b * R + (u - n_prefix)) * a.Hkv + hk) * D;
      kp = k_new + row;
      vp = v_new + row;
      vstride = 1;
    }
    const uint64_t kbits = (uint64_t)kp;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int kk = (w_u + 4 * i) / DL, d = ((w_u + 4 * i) % DL) * 64 + lane;
      const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)kbits, kk), hi = __builtin_amdgcn_readlane((uint32_t)(kbits >> 32), kk);
      kv[i] = reinterpret_cast<const float*>(((uint64_t)hi << 32) | lo)[d];
    }
#pragma unroll
    for (int i = 0; i < NL; ++i) vv[i] = vp[(size_t)(w_u + 4 * i) * vstride];
  };
  if (total > 0) fetch(0);
#pragma unroll
  for (int i = 0; i < RC * D / 256; ++i) Qs[(tid + 256 * i) / D][(tid + 256 * i) % D] = qv[i];

  RowVis vis[RW];
  float m[RW], l[RW], o[RW][DL];
#pragma unroll
  for (int i = 0; i < RW; ++i) {
    int node, strm;
    row_split(min(r0 + w * RW + i, R - 1), T, a.gamma, node, strm);
    vis[i] = make_row_vis(node, strm, ancestors_of(node, lane < T ? clamp_parent(par, lane) : -1), T, a.gamma, (a.flags & SS_STREAM_EXCLUDE_SELF) != 0);
    m[i] = -1e30f;
    l[i] = 0.f;
#pragma unroll
    for (int dd = 0; dd < DL; ++dd) o[i][dd] = 0.f;
  }

  for (int t0 = 0; t0 < total; t0 += KT) {
    __syncthreads();  // the previous tile has been consumed
#pragma unroll
    for (int i = 0; i < NL; ++i) Ks[(w_u + 4 * i) / DL][((w_u + 4 * i) % DL) * 64 + lane] = kv[i];
#pragma unroll
    for (int i = 0; i < NL; ++i) Vs[w_u + 4 * i][lane] = t0 + lane < total ? vv[i] : 0.f;
    __syncthreads();
    if (t0 + KT < total) fetch(t0 + KT);

    // scores of this lane's key against the wave's rows
    float sc[RW];
#pragma unroll
    for (int i = 0; i < RW; ++i) sc[i] = 0.f;
#pragma unroll (D == 128 ? 2 : 4)
    for (int d = 0; d < D; d += 4) {
      const floatx4 kd = *reinterpret_cast<const floatx4*>(&Ks[lane][d]);
#pragma unroll
      for (int i = 0; i < RW; ++i) {
        const floatx4 qd = *reinterpret_cast<const floatx4*>(&Qs[w * RW + i][d]);
#pragma unroll
        for (int e = 0; e < 4; ++e) sc[i] = fmaf(qd[e], kd[e], sc[i]);
      }
    }
    const int u = t0 + lane;
#pragma unroll
    for (int i = 0; i < RW; ++i) {
      bool vis_ok = u < total;
      if (u >= n_prefix) vis_ok = vis_ok && row_sees(vis[i], u - n_prefix, T);
      const float sv = vis_ok ? sc[i] * a.scale_log2 : -INFINITY;
      const float m_new = fmaxf(m[i], wave_max_f32(sv));
      const float alpha = exp2f(m[i] - m_new);
      const float p = exp2f(sv - m_new);
      l[i] = l[i] * alpha + p;  // this lane's keys; the lanes are summed at the end
      m[i] = m_new;
#pragma unroll
      for (int dd = 0; dd < DL; ++dd) o[i][dd] *= alpha;
      Ps[w][i][lane] = p;
    }
    // P.V: a lane owns output features lane, lane+64; the probabilities of the wave's
    // rows are read back from LDS (same address for all lanes: a broadcast)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll (D == 128 ? 2 : 4)
    for (int kk = 0; kk < KT; kk += 4) {
      floatx4 vk[DL];
#pragma unroll
      for (int dd = 0; dd < DL; ++dd) vk[dd] = *reinterpret_cast<const floatx4*>(&Vs[lane + 64 * dd][kk]);
#pragma unroll
      for (int i = 0; i < RW; ++i) {
        const floatx4 pk = *reinterpret_cast<const floatx4*>(&Ps[w][i][kk]);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int dd = 0; dd < DL; ++dd) o[i][dd] = fmaf(pk[e], vk[dd][e], o[i][dd]);
      }
    }
  }

#pragma unroll
  for (int i = 0; i < RW; ++i) {
    const int row = r0 + w * RW + i;
    if (row >= R) continue;
    if ((row < T ? row : (row - T) / max(a.gamma, 1)) >= n_kept) continue;  // rows of removed nodes are not written
    for (int off = 32; off > 0; off >>= 1) l[i] += __shfl_xor(l[i], off, 64);
    const float inv = l[i] > 0.f ? 1.f / l[i] : 0.f;
    if (a.n_splits == 1) {
      float* out = (float*)a.out + (((size_t)b * R + row) * a.H + h) * D;
#pragma unroll
      for (int dd = 0; dd < DL; ++dd) out[lane + 64 * dd] = o[i][dd] * inv;
    } else {
      const size_t pr = part_row_of<false>(a, b, 0, s, h, row);
#pragma unroll
      for (int dd = 0; dd < DL; ++dd) a.part_o[pr * D + lane + 64 * dd] = o[i][dd] * inv;
      if (lane == 0) a.part_lse[pr] = m[i] + log2f(l[i]);
    }
  }
}

// ------------------------------------------------------------------ merge of splits
//
// out = sum_s w_s * o_s with w_s = 2^(lse_s - max) / sum.  One thread per (sequence, row, head,
// 4 features).  The partial outputs are fetched four splits at a time without waiting for the
// log-sum-exps (their addresses do not depend on them) and folded in with a running maximum, so the
// kernel is one round of independent loads deep for each four splits.  CUTS: after an attention kernel that may have
// cut the batch anew; the table of cuts tells.
template <bool BF16, bool CUTS>
__global__ __launch_bounds__(256) void msa_combine_kernel(MsaArgs a) {
  const int dq = a.D >> 2;  // threads per row
  const long t = (long)blockIdx.x * 256 + threadIdx.x;
  const long item = t / dq;
  const int d0 = (int)(t % dq) * 4;
  if (item >= (long)a.B * a.R * a.H) return;
  const int h = item % a.H;
  const int r = (item / a.H) % a.R;
  const int b = item / ((long)a.H * a.R);
  if ((r < a.T ? r : (r - a.T) / max(a.gamma, 1)) >= kept_nodes(b, a)) return;  // rows of removed nodes: no partials, not written
  // the rows of part_row_of: the sequence's first, or where the table of cuts tells the slots the workspace's first
  const size_t stride = CUTS ? (size_t)a.H * a.R : a.R, row0 = CUTS ? (size_t)h * a.R + r : part_row_of<false>(a, b, 0, 0, h, r);
  floatx4 v[4];
  float l[4];
  auto fetch = [&](int slot0, int s0, int n) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const size_t row = (size_t)(slot0 + min(s0 + i, n - 1)) * stride + row0;
      v[i] = *reinterpret_cast<const floatx4*>(a.part_o + row * a.D + d0);
      l[i] = a.part_lse[row];
    }
  };
  // The first four splits are fetched where the host's cut puts them, before it is known whether that stands and how many
  // the sequence has: one round of loads less to wait for (0.2 us of 4.8; what lies in the place of a split that the
  // sequence does not have is not used).  The empty asm keeps the compiler from moving the loads behind the test.
  fetch(CUTS ? b * a.n_splits : 0, 0, a.n_splits);
  int n_active, slot0 = 0;
  if (CUTS) {
    const int2 cut = a.cut_table[b];
    n_active = min(max(cut.x, 1), a.B * a.n_splits);  // clamped: whatever the workspace holds, what is read lies in it
    slot0 = min(max(cut.y, 0), a.B * a.n_splits - n_active);
  } else {
    n_active = active_splits(clamp_len(a.seq_lens[b], a), a);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(v[i]), "+v"(l[i]));
  if (CUTS && (slot0 != b * a.n_splits || n_active > a.n_splits)) fetch(slot0, 0, n_active);
  float m = -INFINITY, wsum = 0.f;
  floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < n_active; s0 += 4) {
    if (s0 > 0) fetch(slot0, s0, n_active);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (s0 + i < n_active && l[i] > -INFINITY) {
        const float m_new = fmaxf(m, l[i]);
        const float keep = exp2f(m - m_new), w = exp2f(l[i] - m_new);
        acc = merge_step(acc, keep, v[i], w);
        wsum = __builtin_fmaf(wsum, keep, w);
        m = m_new;
      }
    }
  }
  const float inv = wsum > 0.f ? 1.f / wsum : 0.f;
  acc *= inv;
  const size_t oidx = (((size_t)b * a.R + r) * a.H + h) * a.D + d0;
  if (BF16) {
    *reinterpret_cast<uintx2*>((uint16_t*)a.out + oidx) = uintx2{pack_bf16x2(acc[0], acc[1]), pack_bf16x2(acc[2], acc[3])};
  } else {
    *reinterpret_cast<floatx4*>((float*)a.out + oidx) = acc;
  }
}

// ------------------------------------------------------------------ planning (host)

static std::atomic<int> g_split_keys_override{0};
static std::atomic<int> g_merge_in_kernel{1};

// Scratch memory of ss_msa_attention_static: it takes a shape whose partial results need at most the first with one of the
// shape's two plans (MsaPlan.scratch_bytes); with its own plan they find room in the second.
constexpr size_t kStaticScratchBytes = (size_t)32 << 20, kStaticArrayBytes = (size_t)64 << 20;

struct MsaPlan {
  int split_keys, split0_keys, n_splits, n_qc, groups, stages;
  int adaptive, new_units, min_units, chunk_rows;
  bool wide;              // MFMA path: the kernel with 32 query rows per wave
  size_t arrive_bytes;    // arrival counters of this shape (front of the workspace); 0 = not merged in the attention kernel
  size_t part_o_at, part_lse_at, table_at, total_bytes;  // places in the workspace
  size_t scratch_bytes;   // what counts against the limit of ss_msa_attention_static
};

// Chooses the split length from the shape alone (sequence lengths live on the device).  Every split
// costs a workgroup set-up and fp32 partial results that are read back, so the plan uses as few as fill
// the chip; no split is shorter than 256 cached tokens.
//   fp32 kernel: splits for about 512 workgroups.
//   MFMA kernel: with 512 or more (sequence, KV head, row chunk) items one workgroup of one wave group
//   each with a two-stage ring, three resident per compute unit (measured best when lengths vary: the
//   hardware evens them out); with fewer, two wave groups per workgroup (the prefix split again inside the
//   workgroup and merged through LDS) with three ring stages each, and splits for about 256 workgroups;
//   three wave groups when a sequence has several row chunks (long GQA trees: the kernel is then bound by
//   the matrix cores and more waves hide more latency).  Split 0 also scans the step's own rows and gets
//   that much less of the prefix.
// Tuning aid: blocks' worth of time, beyond its ceil(R/32) blocks, that scanning the step's own rows costs
// split 0 (SS_MSA_SPLIT0_EXTRA, read once).
static int split0_extra_blocks() {
  static const int v = []() {
    const char* e = getenv("SS_MSA_SPLIT0_EXTRA");
    const int x = e ? atoi(e) : 2;
    return x < -64 ? -64 : (x > 64 ? 64 : x);
  }();
  return v;
}

// Whether the kernel with 32 query rows per wave takes the call.  It halves the LDS reads and barriers per score, but its
// workgroups take 96 or 128 rows and start up more slowly, so it is the better one where that pads few rows and where there
// is much to do: from 75 blocks of 32 tokens per workgroup that the chip holds on, by the block table.  Measured, us per
// layer with 16 and with 32 rows per wave (8 KV heads of 128, 640 rows): 8 x 32768 tokens 818 and 725, 8 x 8192 250 and 219,
// 4 x 16384 290 and 200, 4 x 8192 (80 blocks) 162 and 115, 8 x 4096 (80) 160 and 133; 384 rows: 8 x 8192 (96) 165 and 146,
// 2 x 16209 (47; 9005 and 3001 of them used) 46 and 45, 2 x 8000 (640 rows, 4 heads: 20) 41 and 44; 96 rows, one chunk
// instead of two of 48: 16 x 32 heads x 4096 (128) 275 and 241, a quarter of that 60 and 59.  320 rows (384 with padding)
// 8 x 8192 128 and 136; 120 rows, a single chunk either way, 260 and 263.  Heads of 64 have half the products per
// exponential and gain nothing: 400 rows 8 x 8192 128 and 125, 16384 214 and 226.
static bool wide_fits(int B, int R, int H, int Hkv, int D, int len) {
  const int F = (H / Hkv) * R;
  if (D != 128 || F <= 80 || (F > 96 && F <= 128) || H >= (1 << 20)) return false;
  const int rows = msa_bf16_wide_rows(F), chunks = ceil_div(F, rows);
  const int rows16 = msa_bf16_rows_per_chunk(F), pad16 = ceil_div(F, rows16) * rows16;
  return 10L * chunks * rows <= 11L * pad16 && (double)B * Hkv * chunks * ceil_div(len, 32) >= 75.0 * kWideSlots;
}

// Three or four splits are merged inside the attention kernel where the wave that finds itself last has little to read: few
// rows of few features.  The merge kernel and its launch are saved, all of it for sequences of one split.  Us per layer with
// the merge kernel and without (32 heads of 64, 5 rows, two sequences): in a table of four times their 411 and 777 tokens
// 15.0 and 12.4, full tables of 2048 tokens 15.3 and 14.0, of 3100 18.0 and 17.5.  Beyond 512 values it loses or draws:
// heads of 128, 5 rows 16.2 and 16.6, 38.7 and 40.0; 15 rows 22.3 and 23.9; eight splits 16.3 and 17.8, fourteen 17.5 and 33.5.
static bool merges_few_rows(int F, int D, int n_splits) { return F * D <= 512 && n_splits <= 4; }

// What a launch of 256 and more items with several row chunks costs in n splits, in blocks: rounds of the 32 compute units of
// an XCD, which gets whole (sequence, KV head, split) groups, times the blocks of a split and 8 for its start, and what the
// partial results cost (a fiftieth per workgroup, as in cut_cost, and the merge kernel).  With 32 rows per wave it says where
// whole rounds of 256 workgroups want too many splits: they are kept if that costs at most 3 % more (of batches that are cut
// on the device more splits are finer pieces).  Measured on 90 shapes (2 to 16 sequences of 2300 to 32000 tokens, 450 to 2700
// rows per KV head), against the best of 1 to 8 splits: 3 % lost on average, 9 to 12 % by whole rounds alone, with which
// shorter sequences were slower than with 16 rows per wave (us: 13 x 4416 tokens, 1296 rows, 4 splits 548, unsplit 375;
// 10 x 5248, 480 rows, 5 splits 187, unsplit 146, with 16 rows 151; 16 x 2368, 1410 rows, 2 splits 419, unsplit 314, 377).
// Where that kernel's chunks are 80 rows (15 waves) the two costs compare as the times do, and it keeps what it does as well in
// one split (a cost at most 7 % higher): 9 x 4288 tokens, 780 rows, 3 rounds either way, 188 and with 32 rows 207; 12 x 5312,
// 2072 rows, 5 rounds, 389 and 408; 8 x 4288 of which a twelfth to a quarter is used, 960 rows, 72 and 92.  (Its chunks of 48
// or 64 rows take 1.2 to 2.3 times as long, those of 128 1.1 to 1.5.)
static double launch_cost(int groups, int chunks, int len, int n) {
  const long per_xcd = ((long)groups * n + 7) / 8 * chunks;
  return (double)((per_xcd + 31) / 32) * (ceil_div(ceil_div(len, 32), n) + 8) + (n > 1 ? 0.16 * (double)per_xcd + 16.0 : 0.0);
}

static MsaPlan make_plan(int B, int R, int H, int Hkv, int D, int max_len, int dtype, bool allow_wide = true) {
  MsaPlan p;
  const int g = H / Hkv;
  p.wide = allow_wide && dtype == SS_BF16 && wide_fits(B, R, H, Hkv, D, max_len);
  int base;
  p.groups = 1;
  p.stages = 2;
  if (dtype == SS_BF16) {
    const int rows = p.wide ? msa_bf16_wide_rows(g * R) : msa_bf16_rows_per_chunk(g * R);
    p.n_qc = ceil_div(g * R, rows);
    base = B * Hkv * p.n_qc;
  } else {
    p.n_qc = ceil_div(R, 32);
    base = B * H * p.n_qc;
  }
  if (base < 1) base = 1;
  const int len = max_len < 1 ? 1 : max_len;
  const int unit = dtype == SS_BF16 ? 32 : 64;  // the MFMA kernel works in 32-key blocks, the fp32 kernel in 64-key tiles
  int split_keys = g_split_keys_override.load();
  const bool overridden = split_keys > 0;
  int want_wgs = 512;
  if (dtype == SS_BF16 && !p.wide) {
    if (base < 512) {
      p.groups = 2;
      p.stages = 3;
      want_wgs = 256;
    } else if (p.n_qc > 1) {
      p.groups = 3;
      p.stages = 3;
    }
    if (p.n_qc > 1) p.groups = msa_bf16_rows_per_chunk(g * R) == 128 ? 2 : 3;  // 16 or 15 waves per workgroup
  }
  if (split_keys <= 0) {
    // (32 rows per wave: two workgroups fit a compute unit, and one more than that makes a second round)
    int n = p.wide ? (kWideSlots / base < 1 ? 1 : kWideSlots / base) : ceil_div(want_wgs, base);
    const int n_cap = len / 256 < 1 ? 1 : len / 256;
    if (n > n_cap) n = n_cap;
    if (dtype == SS_BF16 && p.n_qc > 1 && base >= 256) {
      // Several row chunks, one workgroup per compute unit: whole rounds of 256 workgroups matter more than
      // anything else.  The fewest splits (of at least 1024 tokens) that waste the least of the last round:
      // 320 items -> 4 splits = 5 rounds exactly (c5: 845 us; unsplit, in 2 rounds of which the second is a
      // quarter full: 1120 us).
      int best_n = 1;
      double best_waste = 0.0;
      for (int cand = 1; cand <= 8 && (cand == 1 || len / cand >= 1024); ++cand) {
        const double wgs = (double)base * cand, waste = ceil(wgs / 256.0) * 256.0 / wgs;
        if (cand == 1 || waste < best_waste - 1e-9) {
          best_n = cand;
          best_waste = waste;
        }
      }
      n = best_n;
      if (p.wide) {
        for (int cand = best_n - 1; cand >= 1; --cand)
          if (launch_cost(B * Hkv, p.n_qc, len, cand) <= launch_cost(B * Hkv, p.n_qc, len, n)) n = cand;
        if (launch_cost(B * Hkv, p.n_qc, len, best_n) <= 1.03 * launch_cost(B * Hkv, p.n_qc, len, n)) n = best_n;
        if (msa_bf16_rows_per_chunk(g * R) == 80) {
          const MsaPlan q = make_plan(B, R, H, Hkv, D, max_len, dtype, false);
          if (q.n_splits == 1 && launch_cost(B * Hkv, q.n_qc, len, 1) <= 1.07 * launch_cost(B * Hkv, p.n_qc, len, n)) return q;
        }
      }
    }
    split_keys = ceil_div(ceil_div(len, unit), n) * unit;
  }
  split_keys = (int)align_up((size_t)(split_keys < 64 ? 64 : split_keys), unit);
  p.split_keys = p.split0_keys = split_keys;
  p.n_splits = ceil_div(len, split_keys);
  if (dtype == SS_BF16 && p.n_splits > 1 && !overridden) {
    // Split 0 also scans the step's own rows: masked blocks with transposing reads, about `extra` blocks'
    // worth of time.  It gets that much less of the prefix; the others take whole iterations of all wave
    // groups where that leaves split 0 something.  Where it does not they take what they must (one sequence of 2048 tokens
    // with 80 rows in 8 splits: one block and 7 x 9 instead of 8 x 8, 20.5 -> 20.0 us; 16 heads 19.9 -> 18.7, heads of 64
    // 16.3 -> 15.5), with one block of `extra` less: with as many, 40 rows got splits of 9 blocks too, 18.0 -> 18.6 us.  This
    // only if split 0 then has fewer blocks than in equal splits (39 shapes against equal splits, means over tables that are a
    // quarter to all full: 0.4 to 8 % faster where it has less, 1 to 3 % slower with one block more, 5 to 8 % with two and
    // more; 16 heads, 8320 tokens, 60 rows 20.8 us with 17 in each, 22.3 with 20 and 15 x 16).
    const int nu = ceil_div(len, 32), n = p.n_splits, extra = ceil_div(R, 32) + split0_extra_blocks();
    int rest = (nu + extra + n / 2) / n, most = nu;  // blocks of the others, most of split 0
    const int whole = (rest + p.groups / 2) / p.groups * p.groups;
    if (nu - (n - 1) * whole >= 1) {
      rest = whole;
    } else {
      rest = (nu + extra - 1 + n / 2) / n;
      most = split_keys / 32 - 1;
    }
    const int rest0 = nu - (n - 1) * rest;
    if (rest >= 2 && rest0 >= 1 && rest0 <= most) {
      p.split_keys = 32 * rest;
      p.split0_keys = 32 * rest0;
    }
  }
  // Cutting on the device needs slots to deal out and a lane per sequence; a caller's split length stays.  With one
  // row chunk a launch is so short that waiting for the lengths costs 1 us of 16 even where the host's cut stands
  // (one sequence of 2048 tokens, 32 heads; 2 % of a step), so those keep the host's cut.  So do launches whose
  // splits are short by the host's plan: cutting anew takes 2 to 4 us (splits of 300 tokens: 10 to 15 % lost, from
  // 1024 tokens on 5 to 20 % gained).
  p.adaptive = dtype == SS_BF16 && p.n_qc > 1 && p.n_splits > 1 && p.split_keys >= 1024 && !overridden && B <= kAdaptiveMaxB;
  p.new_units = ceil_div(R, 32) + split0_extra_blocks();
  if (p.new_units < 0) p.new_units = 0;
  // The more rounds a launch has, the less a short split gains it: one sequence of 848 tokens 22 us with splits of 8 blocks
  // and 25 with 16; batches of fewer than 256 items 0.5 % between the two and 5 % slower with 32; four batches of 320
  // items the same with 8 and 16 and 5 % faster with 32 (two of them; the others the same).
  p.min_units = base >= 256 ? 16 : 8;
  p.chunk_rows = dtype != SS_BF16 ? 32 : p.wide ? msa_bf16_wide_rows(g * R) : msa_bf16_rows_per_chunk(g * R);
  // Workspace: arrival counters (their region is there for every split shape) | partial outputs | log-sum-exps | cuts
  p.arrive_bytes = 0;
  p.part_o_at = p.part_lse_at = p.table_at = 0;
  p.total_bytes = p.scratch_bytes = 256;  // to align the start
  if (p.n_splits > 1) {
    // Merged in the attention kernel: two splits, or a few of few rows (merges_few_rows)
    const bool merged = dtype == SS_BF16 && !p.wide && (p.n_splits == 2 || merges_few_rows(g * R, D, p.n_splits));
    const size_t counters = merged
                                ? align_up((size_t)B * Hkv * p.n_qc * kArriveTiles * sizeof(unsigned int), 256) : 0;
    if (counters <= kArriveRegionBytes) p.arrive_bytes = counters;
    const size_t rows = (size_t)B * H * p.n_splits * R;
    p.part_o_at = kArriveRegionBytes;
    p.part_lse_at = p.part_o_at + align_up(rows * D * sizeof(float), 256);
    p.table_at = p.part_lse_at + align_up(rows * sizeof(float), 256);
    p.total_bytes += p.table_at + (p.adaptive ? kAdaptiveMaxB * sizeof(int2) : 0);
    p.scratch_bytes += p.table_at - kArriveRegionBytes + (p.n_splits == 2 ? counters : 0);
  }
  // ss_msa_attention_static and ss_msa_attention have one plan.  This kernel's splits may be twice the other's, so a shape
  // counts there as what the smaller needs, and the other kernel takes it, in both calls, if this one's do not fit the array.
  // (It taking all shapes whose 32 MiB only it keeps to cost 5 to 12 %: 4 x 9600 tokens, 512 rows 110 and 124 us.)
  if (p.wide && p.scratch_bytes > kStaticScratchBytes) {
    const MsaPlan q = make_plan(B, R, H, Hkv, D, max_len, dtype, false);
    if (q.scratch_bytes <= kStaticScratchBytes) {
      if (p.scratch_bytes > kStaticArrayBytes) return q;
      p.scratch_bytes = q.scratch_bytes;
    }
  }
  return p;
}

// The plan of a call with a workspace of that size: one that only the other kernel's splits fit stays good.
static MsaPlan plan_for(int B, int R, int H, int Hkv, int D, int max_len, int dtype, size_t workspace_bytes) {
  const MsaPlan p = make_plan(B, R, H, Hkv, D, max_len, dtype);
  if (p.wide && p.n_splits > 1 && workspace_bytes < p.total_bytes) return make_plan(B, R, H, Hkv, D, max_len, dtype, false);
  return p;
}

// The shape and the plan of a call, as the kernels read them.
static void set_plan(MsaArgs& a, const MsaPlan& plan, int B, int T, int gamma, int H, int Hkv, int D, int max_len, int dtype) {
  a.B = B; a.T = T; a.gamma = gamma; a.R = T * (1 + gamma); a.H = H; a.Hkv = Hkv; a.g = H / Hkv; a.D = D;
  a.split_keys = plan.split_keys; a.split0_keys = plan.split0_keys; a.n_splits = plan.n_splits; a.n_qc = plan.n_qc; a.groups = plan.groups; a.stages = plan.stages;
  a.max_n = plan.n_splits == 2 && dtype == SS_BF16 && !plan.wide ? 2 : 0;  // also where the merge kernel does it: the same cut either way
  a.even_len = max_len - max_len / 8;
  const double whole = (double)B * ceil_div(max_len, 32) * plan.n_qc;
  a.even_work = (long)B * Hkv * plan.n_qc >= 256 && whole < INT_MAX ? (int)ceil(0.875 * whole) : 0;
  a.adaptive = plan.adaptive; a.new_units = plan.new_units; a.min_units = plan.min_units; a.chunk_rows = plan.chunk_rows;
  a.xcd_slots = plan.wide ? kWideSlots / 8 : 32; a.cut_fixed = plan.wide ? 8.f : 4.f; a.cut_piece = plan.wide ? 0.02f : 0.f;
}

// Whether a full call folds its splits inside the attention kernel (see msa_run).
static bool merges_in_kernel(const MsaPlan& plan) {
  return g_merge_in_kernel.load() && plan.arrive_bytes > 0;
}

static int check_shape(const char* fn, int B, int T, int gamma, int H, int Hkv, int D, int dtype) {
  SS_REQUIRE(B >= 0, SS_ERR_INVALID_ARG, "%s: B=%d", fn, B);
  SS_REQUIRE(T >= 1 && T <= SS_MAX_T, SS_ERR_UNSUPPORTED, "%s: T=%d outside [1,%d]", fn, T, SS_MAX_T);
  SS_REQUIRE(gamma >= 0 && gamma <= SS_MAX_GAMMA, SS_ERR_UNSUPPORTED, "%s: gamma=%d outside [0,%d]", fn, gamma,
             SS_MAX_GAMMA);
  SS_REQUIRE(H >= 1 && Hkv >= 1 && H % Hkv == 0, SS_ERR_INVALID_ARG, "%s: H=%d must be a multiple of Hkv=%d", fn, H,
             Hkv);
  SS_REQUIRE(D == 64 || D == 128, SS_ERR_UNSUPPORTED, "%s: head dim %d not in {64,128}", fn, D);
  SS_REQUIRE(dtype == SS_F32 || dtype == SS_BF16, SS_ERR_UNSUPPORTED, "%s: dtype %d", fn, dtype);
  return SS_OK;
}

// Zero fill by a kernel (a memset node must not be recorded into a captured graph): 16 bytes per thread over
// the aligned middle, thread 0 also takes the unaligned ends.
__global__ __launch_bounds__(256) void zero_bytes_kernel(unsigned char* p, size_t head, size_t chunks, size_t tail) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < chunks) reinterpret_cast<uintx4*>(p + head)[i] = uintx4{0u, 0u, 0u, 0u};
  if (i == 0) {
    for (size_t j = 0; j < head; ++j) p[j] = 0;
    for (size_t j = 0; j < tail; ++j) p[head + 16 * chunks + j] = 0;
  }
}
static int zero_bytes(unsigned char* p, size_t bytes, hipStream_t st, const char* fn) {
  if (bytes == 0) return SS_OK;
  size_t head = (16 - ((uintptr_t)p & 15)) & 15;
  if (head > bytes) head = bytes;
  const size_t chunks = (bytes - head) / 16, tail = bytes - head - 16 * chunks;
  const size_t blocks = chunks / 256 + 1;
  SS_REQUIRE(blocks <= 0x7fffffffUL, SS_ERR_UNSUPPORTED, "%s: %zu bytes are too many for one fill", fn, bytes);
  hipLaunchKernelGGL(zero_bytes_kernel, dim3((unsigned)blocks), dim3(256), 0, st, p, head, chunks, tail);
  return check_launch(fn);
}

// Scratch memory of ss_msa_attention_static: the per-split partial results and the arrival counters of a
// call, for callers that cannot provide a workspace: the counters' region, kStaticArrayBytes of partial rows and
// the table of cuts.  Every GPU the library runs on holds its own copy of
// the array; host code reaches it only through the address hipGetSymbolAddress reports for the device that
// is current, looked up once per device.
static __device__ __align__(256) unsigned char g_msa_scratch[kArriveRegionBytes + kStaticArrayBytes + kAdaptiveMaxB * sizeof(int2)];
constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mutex;
static void* g_scratch_ptr[kMaxDevices];  // guarded by g_scratch_mutex

static int static_scratch(const char* fn, void** ptr) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) SS_FAIL(SS_ERR_HIP, "%s: hipGetDevice: %s", fn, hipGetErrorString(e));
  SS_REQUIRE(dev >= 0 && dev < kMaxDevices, SS_ERR_UNSUPPORTED, "%s: device %d outside [0,%d)", fn, dev, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(g_msa_scratch));
    if (e != hipSuccess || p == nullptr)
      SS_FAIL(SS_ERR_HIP, "%s: hipGetSymbolAddress: %s", fn, hipGetErrorString(e));
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return SS_OK;
}

// The body of ss_msa_attention and ss_msa_attention_static.  `library_scratch`: the workspace is the library's
// own array, whose size is a limit of the call (not a caller's mistake) and whose arrival counters are cleared
// here on every call.
static int msa_run(const char* fn, const void* q, const void* k_new, const void* v_new, const void* k_cache,
                   const void* v_cache, const int32_t* block_table, int max_pages_per_seq, int num_pages,
                   const int32_t* seq_lens, const int32_t* parent, const int32_t* n_nodes, int B, int T, int gamma, int H,
                   int Hkv, int D, int page_size, float scale, int dtype, uint32_t flags, void* out, void* workspace,
                   size_t workspace_bytes, bool library_scratch, void* stream) {
  if (int rc = check_shape(fn, B, T, gamma, H, Hkv, D, dtype)) return rc;
  SS_REQUIRE(B == 0 || (q && k_new && v_new && k_cache && v_cache && block_table && seq_lens && parent && out),
             SS_ERR_INVALID_ARG, "%s: NULL tensor argument", fn);
  SS_REQUIRE(page_size == 16 || page_size == 32 || page_size == 64, SS_ERR_UNSUPPORTED,
             "%s: page_size %d not in {16,32,64}", fn, page_size);
  SS_REQUIRE(max_pages_per_seq >= 1 && num_pages >= 1, SS_ERR_INVALID_ARG, "%s: max_pages_per_seq=%d num_pages=%d", fn,
             max_pages_per_seq, num_pages);
  SS_REQUIRE((long)max_pages_per_seq * page_size <= (1L << 30), SS_ERR_UNSUPPORTED, "%s: sequence capacity too large",
             fn);
  // the MFMA kernel keeps a page's offset in units of 256 bytes in 32 bits
  SS_REQUIRE(dtype != SS_BF16 || (double)num_pages * Hkv * page_size * D * 2.0 <= 1099511627776.0, SS_ERR_UNSUPPORTED,
             "%s: a cache of more than 1 TiB per tensor (num_pages=%d)", fn, num_pages);
  SS_REQUIRE(scale > 0.f && isfinite(scale), SS_ERR_INVALID_ARG, "%s: scale must be positive and finite", fn);
  SS_REQUIRE((flags & ~(SS_STREAM_EXCLUDE_SELF | SS_MSA_PARTIALS_ONLY | SS_MSA_MERGE_ONLY)) == 0, SS_ERR_INVALID_ARG,
             "%s: unknown flags 0x%x", fn, flags);
  SS_REQUIRE((flags & (SS_MSA_PARTIALS_ONLY | SS_MSA_MERGE_ONLY)) != (SS_MSA_PARTIALS_ONLY | SS_MSA_MERGE_ONLY),
             SS_ERR_INVALID_ARG, "%s: SS_MSA_PARTIALS_ONLY and SS_MSA_MERGE_ONLY exclude each other", fn);
  if (B == 0) return SS_OK;

  const int R = T * (1 + gamma);
  const int max_len = max_pages_per_seq * page_size;
  const MsaPlan plan = library_scratch ? make_plan(B, R, H, Hkv, D, max_len, dtype)
                                       : plan_for(B, R, H, Hkv, D, max_len, dtype, workspace == nullptr ? 0 : workspace_bytes);
  if (library_scratch) {
    SS_REQUIRE(plan.scratch_bytes <= workspace_bytes, SS_ERR_UNSUPPORTED,
               "%s: this shape needs %zu bytes of scratch memory, the library's array holds %zu; use "
               "ss_msa_attention with a workspace", fn, plan.scratch_bytes, workspace_bytes);
  } else {
    SS_REQUIRE(plan.n_splits == 1 || (workspace != nullptr && workspace_bytes >= plan.total_bytes), SS_ERR_WORKSPACE,
               "%s: workspace of %zu bytes needed, %zu given", fn, plan.total_bytes, workspace_bytes);
  }

  MsaArgs a;
  a.q = q; a.k_new = k_new; a.v_new = v_new; a.k_cache = k_cache; a.v_cache = v_cache;
  a.block_table = block_table; a.seq_lens = seq_lens; a.parent = parent; a.n_nodes = n_nodes; a.out = out;
  char* ws = (char*)(((uintptr_t)workspace + 255) & ~(uintptr_t)255);
  a.part_o = (float*)(ws + plan.part_o_at);
  a.part_lse = (float*)(ws + plan.part_lse_at);
  set_plan(a, plan, B, T, gamma, H, Hkv, D, max_len, dtype);
  a.page = page_size; a.page_shift = page_size == 16 ? 4 : (page_size == 32 ? 5 : 6);
  a.max_pages = max_pages_per_seq; a.num_pages = num_pages;
  a.scale_log2 = scale * 1.4426950408889634f;
  // In-kernel merge (MFMA path, 16 rows per wave; two splits, or three and four of few rows: merges_few_rows): the last split
  // of a (sequence, head) to finish adds the others' partial rows to its own and writes the output, which saves the merge kernel
  // and its kernel boundary.  With more to fetch for one wave the merge kernel is faster.
  a.arrive = nullptr;
  if (merges_in_kernel(plan) && !(flags & SS_MSA_MERGE_ONLY))
    a.arrive = (unsigned int*)ws;
  a.cut_table = plan.adaptive ? (int2*)(ws + plan.table_at) : nullptr;
  a.flags = flags;
  hipStream_t st = (hipStream_t)stream;

  if (library_scratch && a.arrive != nullptr)
    if (int rc = zero_bytes((unsigned char*)a.arrive, plan.arrive_bytes, st, fn)) return rc;
  if (flags & SS_MSA_MERGE_ONLY) {
    // the attention kernel ran in an earlier call with SS_MSA_PARTIALS_ONLY
  } else if (dtype == SS_F32) {
    // Rows per workgroup of the fp32 kernel, by the workgroups that are really made.  D = 64: 32 from 512 workgroups of 32
    // rows and splits on, where reading K and V four times as often costs more than the latency that smaller workgroups
    // hide (us with 8 and with 32 rows, first measured as 384: 67 and 81, 512: 75 and 71 or 124 and 113, 768: 174 and 129);
    // 4 while workgroups of 8 are at most 256 (us with 4 and with 8 rows; 20: 9.8 and 11.9, 120: 12.4 and 15.1, 160: 15.0
    // and 15.5, 240: 15.3 and 15.7, 320: 19.0 and 18.8, 480: 32.2 and 29.5); else 8.  D = 128: always 8, two workgroups per
    // compute unit (75 KB of LDS) where of 32 rows (93 KB) only one fits (256: 99 and 119, 512: 184 and 236).
    const bool few = D == 128 || (long)B * H * plan.n_qc * plan.n_splits < 512;
    const bool fewest = D == 64 && few && (long)B * H * ceil_div(R, 8) * plan.n_splits <= 256;
    dim3 grid(fewest ? ceil_div(R, 4) : few ? ceil_div(R, 8) : plan.n_qc, plan.n_splits, B * H);
    SS_REQUIRE((long)B * H <= 65535 && plan.n_splits <= 65535, SS_ERR_UNSUPPORTED, "%s: grid too large", fn);
    auto kern = D == 128 ? msa_f32_kernel<128, 2> : fewest ? msa_f32_kernel<64, 1> : few ? msa_f32_kernel<64, 2> : msa_f32_kernel<64, 8>;
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, st, a);
    if (int rc = check_launch(fn)) return rc;
  } else {
    if (int rc = plan.wide ? launch_msa_bf16_wide(a, st) : launch_msa_bf16(a, st)) return rc;
  }
  if (plan.n_splits > 1 && !(flags & SS_MSA_PARTIALS_ONLY) && a.arrive == nullptr) {
    const long threads = (long)B * R * H * (D / 4);
    dim3 grid((unsigned)((threads + 255) / 256));
    auto kern = dtype == SS_F32 ? msa_combine_kernel<false, false> : plan.adaptive ? msa_combine_kernel<true, true> : msa_combine_kernel<true, false>;
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, st, a);
    if (int rc = check_launch(fn)) return rc;
  }
  return SS_OK;
}

}  // namespace ss

extern "C" {

int ss_msa_set_split_keys(int split_keys) {
  return ss::g_split_keys_override.exchange(split_keys > 0 ? split_keys : 0);
}

int ss_msa_set_merge_in_kernel(int on) { return ss::g_merge_in_kernel.exchange(on ? 1 : 0); }

int ss_msa_plan(int B, int T, int gamma, int H, int Hkv, int D, int max_seq_len, int dtype, int* n_splits,
                int* n_kernels) {
  ss::clear_error();
  if (int rc = ss::check_shape("ss_msa_plan", B, T, gamma, H, Hkv, D, dtype)) return rc;
  if (max_seq_len < 0) max_seq_len = 0;
  const ss::MsaPlan plan = ss::make_plan(B, T * (1 + gamma), H, Hkv, D, max_seq_len, dtype);
  if (n_splits) *n_splits = plan.n_splits;
  if (n_kernels) *n_kernels = (plan.n_splits > 1 && !ss::merges_in_kernel(plan)) ? 2 : 1;
  return SS_OK;
}

int ss_msa_plan_launch(int B, int T, int gamma, int H, int Hkv, int D, int max_seq_len, size_t workspace_bytes, int32_t* launch) {
  using namespace ss;
  clear_error();
  const char* fn = "ss_msa_plan_launch";
  if (int rc = check_shape(fn, B, T, gamma, H, Hkv, D, SS_BF16)) return rc;
  SS_REQUIRE(launch != nullptr, SS_ERR_INVALID_ARG, "%s: NULL launch", fn);
  if (max_seq_len < 0) max_seq_len = 0;
  const MsaPlan plan = plan_for(B, T * (1 + gamma), H, Hkv, D, max_seq_len, SS_BF16, workspace_bytes);
  SS_REQUIRE(plan.n_splits == 1 || workspace_bytes >= plan.total_bytes, SS_ERR_WORKSPACE, "%s: workspace of %zu bytes needed, %zu given", fn,
             plan.total_bytes, workspace_bytes);
  MsaArgs a = {};
  set_plan(a, plan, B, T, gamma, H, Hkv, D, max_seq_len, SS_BF16);
  const MsaLaunch l = plan.wide ? msa_bf16_wide_launch(a) : msa_bf16_launch(a);
  SS_REQUIRE(l.wgs <= 0x7fffffffL, SS_ERR_UNSUPPORTED, "%s: grid too large", fn);
  launch[0] = plan.wide ? 32 : 16;
  launch[1] = plan.chunk_rows;
  launch[2] = plan.n_splits;
  launch[3] = (int32_t)l.wgs;
  launch[4] = l.waves;
  launch[5] = (int32_t)l.lds;
  return SS_OK;
}

int ss_msa_plan_splits(int B, int T, int gamma, int H, int Hkv, int D, int max_seq_len, int dtype,
                       const int32_t* seq_lens, const int32_t* n_nodes, int* where, int32_t* n_splits) {
  using namespace ss;
  clear_error();
  const char* fn = "ss_msa_plan_splits";
  if (int rc = check_shape(fn, B, T, gamma, H, Hkv, D, dtype)) return rc;
  SS_REQUIRE(B == 0 || seq_lens != nullptr, SS_ERR_INVALID_ARG, "%s: NULL seq_lens", fn);
  if (max_seq_len < 0) max_seq_len = 0;
  MsaArgs a = {};
  set_plan(a, make_plan(B, T * (1 + gamma), H, Hkv, D, max_seq_len, dtype), B, T, gamma, H, Hkv, D, max_seq_len, dtype);
  a.max_pages = max_seq_len; a.page = 1;  // clamp_len
  int load[kAdaptiveMaxB], chunks[kAdaptiveMaxB], units[kAdaptiveMaxB];
  bool even = true;
  int work = 0;  // at most the whole plan's, which even_work is set for only where it fits
  int sum = 0, most = 0;
  for (int b = 0; a.adaptive && b < B; ++b) {
    const int kept = n_nodes ? min(max(n_nodes[b], 1), T) : T;
    even = even && seq_is_even(a, seq_lens[b], kept);
    units[b] = len_units(seq_lens[b], a);
    load[b] = cut_load(a, units[b]);
    chunks[b] = cut_chunks(a, kept);
    if (a.even_work > 0) work += units[b] * chunks[b];
    sum += load[b];
    most = max(most, load[b]);
  }
  even = even || (a.even_work > 0 && work >= a.even_work);
  if (where) *where = !a.adaptive ? 0 : (even ? 1 : 2);
  if (!n_splits) return SS_OK;
  if (!a.adaptive || even) {
    for (int b = 0; b < B; ++b) n_splits[b] = active_splits(clamp_len(seq_lens[b], a), a);
    return SS_OK;
  }
  float best = INFINITY;
  int cut = 0;
  for (int j = 0; j < 64; ++j) {
    const int c = cut_candidate(a, j, cut_range(a, sum, most));
    const float cost = cut_cost(a, c, [&](int i) { return load[i]; }, [&](int i) { return chunks[i]; });
    if (cost <= best) {
      best = cost;
      cut = c;
    }
  }
  for (int b = 0; b < B; ++b) n_splits[b] = cut_of(a, cut, units[b], chunks[b]).n;
  return SS_OK;
}

size_t ss_msa_workspace_bytes(int B, int T, int gamma, int H, int Hkv, int D, int max_seq_len, int dtype) {
  ss::clear_error();
  if (ss::check_shape("ss_msa_workspace_bytes", B, T, gamma, H, Hkv, D, dtype) != SS_OK) return 0;
  if (max_seq_len < 0) max_seq_len = 0;
  return ss::make_plan(B, T * (1 + gamma), H, Hkv, D, max_seq_len, dtype).total_bytes;
}

int ss_msa_workspace_init(void* workspace, size_t workspace_bytes, void* stream) {
  ss::clear_error();
  SS_REQUIRE(workspace != nullptr || workspace_bytes == 0, SS_ERR_INVALID_ARG, "ss_msa_workspace_init: NULL workspace");
  return ss::zero_bytes((unsigned char*)workspace, workspace_bytes, (hipStream_t)stream, "ss_msa_workspace_init");
}

int ss_msa_attention(const void* q, const void* k_new, const void* v_new, const void* k_cache, const void* v_cache,
                     const int32_t* block_table, int max_pages_per_seq, int num_pages, const int32_t* seq_lens,
                     const int32_t* parent, int B, int T, int gamma, int H, int Hkv, int D, int page_size, float scale,
                     int dtype, uint32_t flags, void* out, void* workspace, size_t workspace_bytes, void* stream) {
  ss::clear_error();
  return ss::msa_run("ss_msa_attention", q, k_new, v_new, k_cache, v_cache, block_table, max_pages_per_seq, num_pages,
                     seq_lens, parent, nullptr, B, T, gamma, H, Hkv, D, page_size, scale, dtype, flags, out, workspace,
                     workspace_bytes, false, stream);
}

int ss_msa_attention_pruned(const void* q, const void* k_new, const void* v_new, const void* k_cache,
                            const void* v_cache, const int32_t* block_table, int max_pages_per_seq, int num_pages,
                            const int32_t* seq_lens, const int32_t* parent, const int32_t* n_nodes, int B, int T,
                            int gamma, int H, int Hkv, int D, int page_size, float scale, int dtype, uint32_t flags,
                            void* out, void* workspace, size_t workspace_bytes, void* stream) {
  ss::clear_error();
  SS_REQUIRE(B == 0 || n_nodes != nullptr, SS_ERR_INVALID_ARG, "ss_msa_attention_pruned: NULL n_nodes");
  return ss::msa_run("ss_msa_attention_pruned", q, k_new, v_new, k_cache, v_cache, block_table, max_pages_per_seq,
                     num_pages, seq_lens, parent, n_nodes, B, T, gamma, H, Hkv, D, page_size, scale, dtype, flags, out,
                     workspace, workspace_bytes, false, stream);
}

size_t ss_msa_static_scratch_bytes(void) { return ss::kStaticScratchBytes; }

int ss_msa_attention_static(const void* q, const void* k_new, const void* v_new, const void* k_cache,
                            const void* v_cache, const int32_t* block_table, int max_pages_per_seq, int num_pages,
                            const int32_t* seq_lens, const int32_t* parent, int B, int T, int gamma, int H, int Hkv,
                            int D, int page_size, float scale, int dtype, uint32_t flags, void* out, void* stream) {
  using namespace ss;
  clear_error();
  const char* fn = "ss_msa_attention_static";
  void* scratch = nullptr;
  if (int rc = static_scratch(fn, &scratch)) return rc;
  return msa_run(fn, q, k_new, v_new, k_cache, v_cache, block_table, max_pages_per_seq, num_pages, seq_lens, parent,
                 nullptr, B, T, gamma, H, Hkv, D, page_size, scale, dtype, flags, out, scratch, kStaticScratchBytes, true, stream);
}

}  // extern "C"
