// a2, bf16 path for large problems with many query rows per KV head (wide_fits in ss_msa.hip): multi-stream attention
// (Eq. 1 / Eq. 2) with 32 query rows per wave on v_mfma_f32_32x32x16_bf16: the kernel and its launch, instantiated in
// ss_msa_bf16.hip.
//
// What binds these launches is arithmetic: K and V of a KV head are wanted by several row chunks and come from the L2.  With
// 16 rows per wave (ss_msa_bf16.hip) sixteen waves read every K and V tile out of LDS for 16 rows each and meet at one
// barrier per 32 tokens; with 32 rows per wave the operand reads and the barriers per score are halved, and two workgroups of
// three or four waves per compute unit, which share no barrier, fill each other's waits.  A wave has up to 256 registers, so
// a block's operands are read a stage ahead (K under the P.V products of the block before, V under the scores and the
// softmax), and the probabilities are formed without their maximum (see `softmax`).  8 sequences of 32768 tokens, 8 KV heads
// of 4 query heads, 160 rows: 818 -> 725 us (838 -> 950 TFLOP/s).  The matrix cores are busy 55 % of the cycles (44 %), but
// the chip then grants 1.65 instead of 1.97 GHz: a quarter fewer cycles are a ninth less time.  Wave priorities raised
// around the matrix instructions or around the softmax: no change (733 against 751 and 745 us).
//
// Scores are computed transposed, S^T = K Q^T, so that a lane holds 16 tokens of one query row; which token a row of the
// score tile holds is chosen so that they are the k-slots the lane must supply to O^T += V^T P^T (wide_key).
#pragma once
#include <mutex>

#include "ss_msa_mfma.h"

namespace ss {

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;

// Token (0..31) of a block that row m of the score tile holds: a lane then ends up with 8 consecutive tokens per half of
// the block (registers 8*t .. 8*t+7: tokens 16*t + 8*lh + 0..7), the k-slots it must supply to P.V.
SS_DEV int wide_key(int m) { return 16 * (m >> 4) + 8 * ((m >> 2) & 1) + 4 * ((m >> 3) & 1) + (m & 3); }
// XOR swizzle of a K row's 16-byte chunks: an operand read takes one chunk of 16 consecutive rows per LDS cycle.
SS_DEV int wide_swz(int row) { return row & 15; }

// NW waves of 32 query rows each.  STREAM, CUTS: as in msa_bf16_kernel (ss_msa_bf16.hip), and so are the pieces of work,
// the trip of first loads, the cut on the device and how blocks reach the ring of NS stages in LDS.
template <int D, int NW, bool STREAM, bool CUTS>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2, 2))) void msa_bf16_wide_kernel(MsaArgs args) {
  constexpr int KS = D / 16, DT = D / 32;
  constexpr int NS = NW;                       // ring stages: the waves' output tiles take their place at the end
  constexpr int LW = NW == 4 ? 4 : 2;          // waves that move data
  using Slots = BlockSlots<D, LW>;
  constexpr int K_BYTES = Slots::kKBytes, STAGE = Slots::kStage, K_SLOTS = Slots::kSlots, KJ = Slots::KJ, LPB = Slots::kLoads;
  constexpr int CPR = Slots::kPieces, ROWS_PER_SLOT = Slots::kRowsPerSlot, V_DBLK = Slots::kVBlocks, VHALF = Slots::kVHalf;
  constexpr int ROWS = 32 * NW;

  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];  // [NS][STAGE] | cut
  int* cut = reinterpret_cast<int*>(smem + NS * STAGE);  // [8]: this workgroup's piece where the device cuts the sequences

  const int tid = threadIdx.x, lane = tid & 63, lq = lane & 31, lh = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool loader = w < LW;
  const int wl = w & (LW - 1);
  const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
  const int n_new_units = (args.R + 31) >> 5;
  // The ring's blocks are the step's own ones (split 0), then those of the prefix, of which block i takes stage i % NS.
  const int new0 = NS * SS_MAX_GAMMA * 4 - n_new_units;  // stage of own block u: (new0 + u) % NS

  int b, hk, s, qc, n_active = 0, slot0, split0_keys, split_keys, k0;
  uint32_t tab_a = 0, tab_b = 0;
  const int32_t* my_table;
  const uint32_t page_units = (uint32_t)((size_t)args.Hkv * args.page * D / 128);
  const int key_cap = max(args.max_pages * args.page - 32, 0) & ~31;
  auto load_pages = [&](const MsaArgs& a, int jbase) {
    const int kb = min(k0 + 32 * (jbase + lane), key_cap);
    tab_a = (uint32_t)my_table[kb >> a.page_shift];
    tab_b = (uint32_t)my_table[min((kb + 16) >> a.page_shift, a.max_pages - 1)];
  };
  auto page_offsets = [&](const MsaArgs& a) {
    tab_a = (uint32_t)min(max((int)tab_a, 0), a.num_pages - 1) * page_units;
    tab_b = (uint32_t)min(max((int)tab_b, 0), a.num_pages - 1) * page_units;
  };
  int L_raw, n_kept, R_kept, par_v, q_r, q_h;
  bool f_valid;
  uintx4 Qraw[KS];

  auto swz = [](int row) { return wide_swz(row); };
  auto dma_new = [&](const MsaArgs& a, int c0, uint32_t st_addr) { move_own<D, LW>(a, b, hk, c0, wl, lane, st_addr, swz); };

  const int G = args.B * args.Hkv * args.n_splits;
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  qc = slot % args.n_qc;
  int group = (slot / args.n_qc) * 8 + xcd;
  const bool spare = group >= G;  // has a piece at most where the device cuts the sequences
  if (spare && !CUTS) return;
  if (CUTS) group = min(group, G - 1);
  s = group % args.n_splits;
  hk = (group / args.n_splits) % args.Hkv;
  b = group / (args.n_splits * args.Hkv);
  split0_keys = args.split0_keys;
  split_keys = args.split_keys;
  slot0 = b * args.n_splits;

  auto first_trip = [&](const MsaArgs& a) {
    k0 = s == 0 ? 0 : split0_keys + (s - 1) * split_keys;
    my_table = a.block_table + (size_t)b * a.max_pages;
    load_pages(a, 0);
    L_raw = a.seq_lens[b];
    n_kept = kept_nodes(b, a);
    par_v = a.parent[(size_t)b * a.T + min(lane, a.T - 1)];
    R_kept = n_kept * (1 + a.gamma);
  };
  auto load_queries = [&](const MsaArgs& a) {
    const int f = qc * ROWS + 32 * w + lq;
    f_valid = f < a.g * R_kept;
    const int f_head = f_valid ? fast_div(f, R_kept) : 0, f_row = f_valid ? f - f_head * R_kept : 0;
    q_r = f_row < n_kept ? f_row : a.T + (f_row - n_kept);
    q_h = hk * a.g + f_head;
    const uint16_t* qp = (const uint16_t*)a.q + (((size_t)b * a.R + q_r) * a.H + q_h) * D + lh * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) Qraw[ks] = ld16(qp + 16 * ks);
  };
  int lane_len = 0, lane_kept = args.T;  // CUTS: of the lane's sequence
  if (CUTS && lane < args.B) {
    lane_len = args.seq_lens[lane];
    lane_kept = kept_nodes(lane, args);
  }
  first_trip(args);
  if (!CUTS && qc * ROWS >= args.g * R_kept) return;
  load_queries(args);

  const MsaArgs& a = reread_args<CUTS>(args);
  const int R = a.R, T = a.T;
  const float c = a.scale_log2;
  const uint16_t *k_head, *v_head;
  const int pmask = a.page - 1;

  const int ril = lane / CPR, pch = lane % CPR;
  uint32_t k_voff[KJ], v_voff[KJ];
  bool second[KJ];
#pragma unroll
  for (int j = 0; j < KJ; ++j) {
    const int sl = wl + LW * j, r0 = ROWS_PER_SLOT * sl;
    second[j] = sl >= K_SLOTS / 2;
    k_voff[j] = 2u * (uint32_t)((r0 & 15) * D + ril * D + ((pch ^ wide_swz(r0 + ril)) * 8));
    v_voff[j] = 2u * (uint32_t)((sl % V_DBLK) * 32 * a.page + (lane >> 1) * a.page + (((lane & 1) ^ ((lane >> 4) & 1)) * 8));
  }
  auto dma_main = [&](int u, uint32_t pg_a, uint32_t pg_b, uint32_t st_addr) {
    const int kb = k0 + 32 * u;
    const uint32_t o_a = (uint32_t)(kb & pmask), o_b = (uint32_t)((kb + 16) & pmask);
    const size_t g_a = (size_t)pg_a << 8, g_b = (size_t)pg_b << 8;  // bytes
    const char* ka = (const char*)k_head + g_a + o_a * (2 * D);
    const char* kb2 = (const char*)k_head + g_b + o_b * (2 * D);
    const char* va = (const char*)v_head + g_a + 2 * o_a;
    const char* vb = (const char*)v_head + g_b + 2 * o_b;
    const uint32_t slot_addr = st_addr + (uint32_t)wl * 1024;
#pragma unroll
    for (int j = 0; j < KJ; ++j) dma16<STREAM>(second[j] ? kb2 : ka, k_voff[j], slot_addr + LW * j * 1024);
#pragma unroll
    for (int j = 0; j < KJ; ++j) dma16<STREAM>(second[j] ? vb : va, v_voff[j], slot_addr + K_BYTES + LW * j * 1024);
  };
  uintx4 stg[LPB];
  auto load_ragged = [&](int base, int last) { load_ragged_block<D, LW>(a, my_table, k_head, v_head, base, last, wl, lane, stg, swz); };
  auto store_ragged = [&](unsigned char* st) { store_ragged_block<D, LW>(st, wl, lane, stg); };

  bool has_new = s == 0 && !spare && qc * ROWS < a.g * R_kept;
  const int n_new_pre = min(n_new_units, NS - 1);
  auto start_new = [&](const MsaArgs& a) {
    if (has_new && loader)
      for (int u = 0; u < n_new_pre; ++u) dma_new(a, 32 * u, lds0 + (uint32_t)((new0 + u) % NS) * STAGE);
  };
  start_new(a);

  if constexpr (CUTS) {
    if (plan_is_even<ROWS>(a, lane, lane_len, lane_kept)) {
      if (blockIdx.x == 0 && w == 0 && lane < a.B)
        a.cut_table[lane] = make_int2(active_splits(clamp_len(lane_len, a), a), lane * a.n_splits);
      if (spare) return;
    } else {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // nothing of the abandoned trip is under way to LDS
      if (w == 0) find_piece(reread_args<CUTS>(args), xcd, slot, lane, lane_len, lane_kept, cut);
      __syncthreads();
      b = __builtin_amdgcn_readfirstlane(cut[0]);
      if (b >= 64) return;
      s = __builtin_amdgcn_readfirstlane(cut[1]);
      hk = __builtin_amdgcn_readfirstlane(cut[2]);
      qc = __builtin_amdgcn_readfirstlane(cut[3]);
      n_active = __builtin_amdgcn_readfirstlane(cut[4]);
      split0_keys = __builtin_amdgcn_readfirstlane(cut[5]);
      split_keys = __builtin_amdgcn_readfirstlane(cut[6]);
      slot0 = __builtin_amdgcn_readfirstlane(cut[7]);
      const MsaArgs& a = reread_args<CUTS>(args);
      first_trip(a);
      load_queries(a);
      has_new = s == 0 && qc * ROWS < a.g * R_kept;
      start_new(a);
    }
  }
  k_head = (const uint16_t*)a.k_cache + (size_t)hk * a.page * D;
  v_head = (const uint16_t*)a.v_cache + (size_t)hk * a.page * D;
  const int L = clamp_len(L_raw, a);
  if (CUTS && qc * ROWS >= a.g * R_kept) return;
  if (n_active == 0) {
    n_active = active_splits(L, a);
    if (s >= n_active) return;
  }
  const int k1 = max(k0, min(L, k0 + (s == 0 ? split0_keys : split_keys)));
  const int n_full = (k1 - k0) >> 5;
  const int tail = (k1 - k0) & 31;

  asm volatile("s_waitcnt vmcnt(0)" : "+v"(tab_a), "+v"(tab_b), "+v"(par_v)::"memory");
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(Qraw[ks]));
  page_offsets(a);
  bf16x8 Q[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) Q[ks] = as_bf16x8(f_valid ? Qraw[ks] : uintx4{0u, 0u, 0u, 0u});

  const int n_own = has_new ? n_new_units : 0, n_blocks = n_own + n_full;  // blocks of this workgroup
  auto fetch = [&](int jl, uint32_t st_addr) {
    if ((jl & 63) == 0 && jl > 0) {
      load_pages(a, jl);
      page_offsets(a);
    }
    dma_main(jl, __builtin_amdgcn_readlane(tab_a, jl & 63), __builtin_amdgcn_readlane(tab_b, jl & 63), st_addr);
  };
  if (loader)
    for (int i = n_own; i < min(n_blocks, NS - 1); ++i) fetch(i - n_own, lds0 + (uint32_t)(i - n_own) * STAGE);

  floatx16 O[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) O[dt][e] = 0.f;
  float m_run = -1e30f, nmc_run = 1e30f * c, l_run = 0.f;
  bf16x2 ones2;
  ones2[0] = ones2[1] = (__bf16)1.0f;

  // operand reads: K row wide_key(lq), chunk 2*ks + lh; V: feature 32*dt + lq, tokens 16*t + 8*lh ..
  const int kr = wide_key(lq);
  const uint32_t k_rd = (uint32_t)(kr * (2 * D) + ((lh ^ wide_swz(kr)) * 16));
  const uint32_t v_rd = (uint32_t)(K_BYTES + lq * 32 + ((lh ^ ((lq >> 3) & 1)) * 16));

  // Probabilities (log2 domain, bf16) of a block's scores, and their sum.  The running maximum only moves when the sum of
  // a lane's 16 probabilities exceeds 2^16 (each of them is then at most that where it does not), so no maximum is formed
  // in the common case; the sums are those of the rounded probabilities that enter P.V.
  auto softmax = [&](const floatx16& S, bf16x8 (&P)[2]) {
    float sum;
    auto probs = [&]() {
      float sp[2] = {0.f, 0.f};
#pragma unroll
      for (int t = 0; t < 2; ++t) {
#pragma unroll
        for (int i = 0; i < 8; ++i) P[t][i] = (__bf16)__builtin_amdgcn_exp2f(fmaf(S[8 * t + i], c, nmc_run));
#pragma unroll
        for (int i = 0; i < 8; i += 2) {
          bf16x2 pp;
          pp[0] = P[t][i];
          pp[1] = P[t][i + 1];
          sp[t] = __builtin_amdgcn_fdot2_f32_bf16(pp, ones2, sp[t], false);
        }
      }
      sum = sp[0] + sp[1];
    };
    probs();
    if (__any(sum > 65536.f)) {
      float mx = S[0];
#pragma unroll
      for (int e = 1; e < 16; ++e) mx = fmaxf(mx, S[e]);
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      const float m_new = fmaxf(m_run, mx);
      const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * c);
      l_run *= alpha;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) O[dt][e] *= alpha;
      m_run = m_new;
      nmc_run = -(m_new * c);
      probs();
    }
    l_run += sum;
  };
  // A masked block out of an LDS stage: the ragged block of the prefix, or (is_new) rows c0.. of the step's own block, of
  // which `vis` tells what this lane's query row may see.  The lane id is laundered so that none of its arithmetic is kept
  // in registers across the main loop.
  auto compute = [&](bool is_new, int c0, const unsigned char* st, const RowVis& vis) {
    int ln = lane;
    asm volatile("" : "+v"(ln));
    floatx16 S;
#pragma unroll
    for (int e = 0; e < 16; ++e) S[e] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const uintx4 kop = *reinterpret_cast<const uintx4*>(st + (k_rd ^ (uint32_t)(32 * ks)));
      S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kop), Q[ks], S, 0, 0, 0);
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int off = 16 * (e >> 3) + 8 * (ln >> 5) + (e & 7);
      const bool see_tail = off < tail;
      const bool see_new = (c0 + off < R) & row_sees(vis, c0 + off, T);
      const float sv = S[e];
      S[e] = (is_new ? see_new : see_tail) ? sv : -INFINITY;
    }
    bf16x8 P[2];
    softmax(S, P);
    if (!is_new) {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int nv = min(max(tail - (16 * t + 8 * (ln >> 5)), 0), 8);  // how many of this lane's 8 tokens exist
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
          uintx4 vv = *reinterpret_cast<const uintx4*>(st + v_rd + t * VHALF + dt * 1024);
#pragma unroll
          for (int e = 0; e < 4; ++e) vv[e] &= nv >= 2 * e + 2 ? 0xffffffffu : (nv == 2 * e + 1 ? 0x0000ffffu : 0u);
          O[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(vv), P[t], O[dt], 0, 0, 0);
        }
      }
    } else {
      const unsigned char* vb = st + K_BYTES;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
          uintx2 half[2];
#pragma unroll
          for (int hh = 0; hh < 2; ++hh) {
            const int row = 16 * t + 8 * (ln >> 5) + 4 * hh + ((ln & 15) >> 2);
            const int ch = 4 * dt + 2 * ((ln >> 4) & 1) + ((ln & 3) >> 1);
            half[hh] = lds_read_tr16(vb + row * (2 * D) + ((ch ^ (2 * (row & 3))) * 16) + (ln & 1) * 8);
          }
          const uintx4 vv = uintx4{half[0][0], half[0][1], half[1][0], half[1][1]};
          O[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(vv), P[t], O[dt], 0, 0, 0);
        }
    }
  };

  // ---- the step's own rows (split 0): iteration u waits for its block, its barrier publishes it and frees the stage of
  // the one before, which block u + NS - 1 is sent to.
  if (has_new) {
    const int stream_row = q_r - T;
    const int node = stream_row < 0 ? q_r : fast_div(stream_row, a.gamma), strm = stream_row < 0 ? 0 : stream_row - node * a.gamma + 1;
    const uint64_t anc = ancestors_of(node, lane < T ? clamp_parent(par_v, lane) : -1);
    const RowVis vis = make_row_vis(node, strm, anc, T, a.gamma, (a.flags & SS_STREAM_EXCLUDE_SELF) != 0);
    for (int u = 0; u < n_own; ++u) {
      if (loader) wait_vm_units<LPB>(min(n_blocks - 1 - u, NS - 2));
      __syncthreads();
      const int v = u + NS - 1;
      if (loader && v < n_own) dma_new(a, 32 * v, lds0 + (uint32_t)((new0 + v) % NS) * STAGE);
      else if (loader && v < n_blocks) fetch(v - n_own, lds0 + (uint32_t)((v - n_own) % NS) * STAGE);
      compute(true, 32 * u, smem + (size_t)((new0 + u) % NS) * STAGE, vis);
    }
  }

  // ---- main loop over full blocks of the prefix, software-pipelined: block it's scores come from K operands read during
  // block it - 1, its V operands are read under them and the softmax.  The barrier behind the softmax publishes block
  // it + 1 (this wave's older loads have landed) and frees block it's stage, which block it + NS is sent to; block
  // it + 1's K operands are read under the P.V products.
  if (n_full > 0) {
    uintx4 Kr[KS], Vr[2 * DT];
    auto read_k = [&](const unsigned char* st) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) Kr[ks] = *reinterpret_cast<const uintx4*>(st + (k_rd ^ (uint32_t)(32 * ks)));
    };
    if (loader) wait_vm_units<LPB>(min(n_full - 1, NS - 2));
    __syncthreads();
    if (loader && NS - 1 < n_full) fetch(NS - 1, lds0 + (uint32_t)(NS - 1) * STAGE);
    read_k(smem);
    for (int it0 = 0; it0 < n_full; it0 += NS) {
#pragma unroll
      for (int st = 0; st < NS; ++st) {
        const int it = it0 + st;
        if (it >= n_full) break;
        const unsigned char* cur = smem + (size_t)st * STAGE;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int dt = 0; dt < DT; ++dt) Vr[t * DT + dt] = *reinterpret_cast<const uintx4*>(cur + v_rd + t * VHALF + dt * 1024);
        floatx16 S;
#pragma unroll
        for (int e = 0; e < 16; ++e) S[e] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(Kr[ks]), Q[ks], S, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        bf16x8 P[2];
        softmax(S, P);
        __builtin_amdgcn_sched_barrier(0);
        if (it + 1 < n_full) {
          if (loader) {
            if (it + NS <= n_full) wait_vmcnt<(NS - 2) * LPB>();
            else wait_vmcnt<0>();
          }
          __syncthreads();
          if (loader && it + NS < n_full) fetch(it + NS, lds0 + (uint32_t)st * STAGE);
          read_k(smem + (size_t)((st + 1) % NS) * STAGE);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int dt = 0; dt < DT; ++dt)
            O[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(Vr[t * DT + dt]), P[t], O[dt], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  if (tail != 0) {
    __syncthreads();  // the stages are free
    if (loader) {
      load_ragged(k0 + 32 * n_full, k1 - 1);
      store_ragged(smem);
    }
    __syncthreads();
    compute(false, 0, smem, RowVis{0, 0, 0});
  }

  // ---- normalise, turn the tile round through LDS (each wave its own 32 rows) and store whole rows.
  __syncthreads();  // the stages are free
  const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
  const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  const float my_lse = m_run * c + __log2f(l_tot);
  unsigned char* ot = smem + (size_t)w * (32 * D * 4);
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const floatx4 v = floatx4{O[dt][4 * q] * inv, O[dt][4 * q + 1] * inv, O[dt][4 * q + 2] * inv, O[dt][4 * q + 3] * inv};
      *reinterpret_cast<floatx4*>(ot + lq * (4 * D) + (((8 * dt + 2 * q + lh) ^ (lq & 15)) * 16)) = v;
    }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const int where = f_valid ? (q_h << 10 | q_r) : -1;  // q_r < 64 * 9
  const bool split_launch = a.n_splits > 1;
  if (!split_launch) {
    constexpr int PL = D / 8;  // lanes per row
#pragma unroll
    for (int i = 0; i < 32; i += 64 / PL) {
      const int row = i + lane / PL, j = lane % PL;
      const int at = __shfl(where, row, 64);
      const floatx4 lo = *reinterpret_cast<const floatx4*>(ot + row * (4 * D) + (((2 * j) ^ (row & 15)) * 16));
      const floatx4 hi = *reinterpret_cast<const floatx4*>(ot + row * (4 * D) + (((2 * j + 1) ^ (row & 15)) * 16));
      if (at >= 0)
        *reinterpret_cast<uintx4*>((uint16_t*)a.out + (((size_t)b * R + (at & 1023)) * a.H + (at >> 10)) * D + 8 * j) =
            uintx4{pack_bf16x2(lo[0], lo[1]), pack_bf16x2(lo[2], lo[3]), pack_bf16x2(hi[0], hi[1]), pack_bf16x2(hi[2], hi[3])};
    }
    return;
  }
  constexpr int PL = D / 4;
#pragma unroll
  for (int i = 0; i < 32; i += 64 / PL) {
    const int row = i + lane / PL, j = lane % PL;
    const int at = __shfl(where, row, 64);
    const floatx4 v = *reinterpret_cast<const floatx4*>(ot + row * (4 * D) + ((j ^ (row & 15)) * 16));
    if (at >= 0) *reinterpret_cast<floatx4*>(a.part_o + part_row_of<CUTS>(a, b, slot0, s, at >> 10, at & 1023) * D + 4 * j) = v;
  }
  if (f_valid && lh == 0) a.part_lse[part_row_of<CUTS>(a, b, slot0, s, q_h, q_r)] = my_lse;
}

template <int D, int NW, bool STREAM, bool CUTS>
static int launch_wide_dns(const MsaArgs& a, hipStream_t stream) {
  const MsaLaunch l = msa_bf16_wide_launch(a);
  SS_REQUIRE(l.wgs <= 0x7fffffffL, SS_ERR_UNSUPPORTED, "ss_msa_attention: grid too large");
  auto kern = msa_bf16_wide_kernel<D, NW, STREAM, CUTS>;
  static std::once_flag attr_once;
  static hipError_t attr_err = hipSuccess;
  std::call_once(attr_once, [&]() {
    attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)l.lds);
  });
  if (attr_err != hipSuccess)
    SS_FAIL(SS_ERR_HIP, "ss_msa_attention: hipFuncSetAttribute: %s", hipGetErrorString(attr_err));
  hipLaunchKernelGGL(kern, dim3((unsigned)l.wgs), dim3(64 * NW), l.lds, stream, a);
  return check_launch("ss_msa_attention");
}

template <int D, int NW>
static int launch_wide_dn(const MsaArgs& a, hipStream_t stream) {
  if constexpr (NW == 3)
    if (a.n_qc == 1) return launch_wide_dns<D, NW, true, false>(a, stream);
  return a.adaptive ? launch_wide_dns<D, NW, false, true>(a, stream) : launch_wide_dns<D, NW, false, false>(a, stream);
}

}  // namespace ss
