// Device helpers shared by the two bf16 attention kernels (16 and 32 query rows per wave).
#pragma once

#include "ss_msa.h"

namespace ss {

// Stores and loads that are coherent at device scope by themselves (the sc1 bit: written through to, read from,
// the level all XCDs share), for the partial results the in-kernel split merge hands from one workgroup to
// another: no cache-wide write-back or invalidate is then needed around the arrival counter.
SS_DEV void st16_device(float* p, floatx4 v) { asm volatile("global_store_dwordx4 %0, %1, off sc1" ::"v"(p), "v"(v) : "memory"); }
SS_DEV void st4_device(float* p, float v) { asm volatile("global_store_dword %0, %1, off sc1" ::"v"(p), "v"(v) : "memory"); }
// lse and DT 16-byte pieces (64 bytes apart) of one partial row, as relaxed device-scope loads of 8 bytes each:
// the compiler knows them as loads, so they can be issued early and are waited for at their first use.
template <int DT>
SS_DEV void ld_row_device(const float* lse_p, const float* o_p, float& lse, floatx4 (&o)[DT]) {
  lse = __uint_as_float(__hip_atomic_load(reinterpret_cast<const unsigned int*>(lse_p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) {
    const unsigned long long* p8 = reinterpret_cast<const unsigned long long*>(o_p + 16 * dt);
    const unsigned long long lo = __hip_atomic_load(p8, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long hi = __hip_atomic_load(p8 + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    o[dt] = floatx4{__uint_as_float((unsigned int)lo), __uint_as_float((unsigned int)(lo >> 32)),
                    __uint_as_float((unsigned int)hi), __uint_as_float((unsigned int)(hi >> 32))};
  }
}
// Arrival counter of the in-kernel split merge, read and written at device scope.
SS_DEV unsigned int ld_counter_device(const unsigned int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
SS_DEV void st_counter_device(unsigned int* p, unsigned int v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Maximum as one instruction: the median of (a, b, +inf).  fmaxf() on matrix-core results costs an extra
// instruction per operand (the compiler first quiets signalling NaNs), a fifth of all vector work in the softmax
// of a 32-key block.  `pinf` is +inf in a register the compiler cannot see through (it would turn the median back
// into that maximum).  A compiler builtin, not inline assembly: the wait states between a matrix instruction or a
// row swap and the first reader of its result are inserted by the compiler only for instructions it knows.
SS_DEV float vmax2(float a, float b, float pinf) { return __builtin_amdgcn_fmed3f(a, b, pinf); }
// Maximum over the four lanes l, l^16, l^32, l^48 (the lanes that share a query row), left in all four, by
// the row-swap instructions: rows of 16 lanes [r0 r1 r2 r3] and a copy become [r0 r0 r2 r2] and [r1 r1 r3 r3],
// then halves of 32 lanes likewise.  No trip through LDS, unlike a general lane shuffle.
SS_DEV float max_over_lane_groups(float x, float pinf) {
  const unsigned int u = __float_as_uint(x);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const unsigned int v = __float_as_uint(vmax2(__uint_as_float(a[0]), __uint_as_float(a[1]), pinf));
  const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return vmax2(__uint_as_float(b[0]), __uint_as_float(b[1]), pinf);
}

SS_DEV bf16x8 as_bf16x8(uintx4 u) { return __builtin_bit_cast(bf16x8, u); }
SS_DEV uintx4 ld16(const uint16_t* p) { return *reinterpret_cast<const uintx4*>(p); }
// The same with the streaming hint: the K/V cache is read once per call and should not displace anything in
// the L2 and the memory-side cache (measured: 9 % less kernel time on the 4096-token workloads).
template <bool STREAM>
SS_DEV uintx4 ld16_cache(const uint16_t* p) {
  if constexpr (STREAM) return __builtin_nontemporal_load(reinterpret_cast<const uintx4*>(p));
  else return *reinterpret_cast<const uintx4*>(p);
}

// LDS transpose read.  Within each group of 16 lanes, lane j passes the address of 4 consecutive
// 16-bit elements In[j][0..3]; lane i receives Out[i][e] = In[4*e + (i >> 2)][i & 3].  With lane
// (i = feature, group) pointing at row (i >> 2) and columns 4*(i & 3).. of a row-major tile, it
// receives feature i of rows 0..3: four consecutive keys of one feature.
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short shortx4;
SS_DEV uintx2 lds_read_tr16(const unsigned char* p) {
  const shortx4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((shortx4 __attribute__((address_space(3)))*)(p));
  return __builtin_bit_cast(uintx2, v);
}

// 16 bytes per lane from (sbase + voff) straight into LDS: lane l's piece lands at lds_addr + 16*l.  No
// staging register and no LDS store instruction; the load counts in the issuing wave's vector-memory
// counter and completes in issue order.  STREAM adds the streaming hint (data no other workgroup asks for).
template <bool STREAM>
SS_DEV void dma16(const void* sbase, uint32_t voff, uint32_t lds_addr) {
  if constexpr (STREAM)
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %0 nt" ::"s"(sbase), "v"(voff), "s"(lds_addr) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %0" ::"s"(sbase), "v"(voff), "s"(lds_addr) : "memory", "m0");
}
// Waits until at most `units` blocks' worth of this wave's direct-to-LDS loads (LPB per block) are outstanding.
// The counter has 6 bits; a smaller number than asked for only waits longer.
template <int N>
SS_DEV void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N < 63 ? N : 63) : "memory");
}
template <int LPB>
SS_DEV void wait_vm_units(int units) {
  switch (units) {
    case 0: wait_vmcnt<0>(); break;
    case 1: wait_vmcnt<LPB>(); break;
    case 2: wait_vmcnt<2 * LPB>(); break;
    case 3: wait_vmcnt<3 * LPB>(); break;
    case 4: wait_vmcnt<4 * LPB>(); break;
    case 5: wait_vmcnt<5 * LPB>(); break;
    case 6: wait_vmcnt<6 * LPB>(); break;
    case 7: wait_vmcnt<7 * LPB>(); break;
    case 8: wait_vmcnt<8 * LPB>(); break;
    case 9: wait_vmcnt<9 * LPB>(); break;
    case 10: wait_vmcnt<10 * LPB>(); break;
    case 11: wait_vmcnt<11 * LPB>(); break;
    case 12: wait_vmcnt<12 * LPB>(); break;
    case 13: wait_vmcnt<13 * LPB>(); break;
    case 14: wait_vmcnt<14 * LPB>(); break;
    default: wait_vmcnt<15 * LPB>(); break;
  }
}
// The kernel's arguments, to be read from memory again from here on.  Kept in scalar registers from the start of the
// kernel to its end, over the code that cuts a batch anew, they do not fit, and what is pushed out there is paid for
// by every launch, also where the host's cut stands (1.5 us).
template <bool YES>
SS_DEV const MsaArgs& reread_args(const MsaArgs& args) {
  if constexpr (!YES) return args;
  auto p = __builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const MsaArgs*)p;
}


// ---- how blocks of 32 tokens reach an LDS stage.  A block is moved in 1 KB slots, one direct-to-LDS load each: K slot sl
// holds rows kRowsPerSlot*sl + lane/kPieces, the lane at piece position p = lane%kPieces fetching piece p ^ swz(row).  The V
// tile consists of two halves of 16 keys, each D feature rows of 32 bytes; V slot s2 holds features dblk*32 + lane/2 of half
// s2 / kVBlocks (dblk = s2 % kVBlocks), the lane at position lane&1 fetching the 8-key piece (lane&1) ^ ((feature >> 3) & 1),
// which makes the 16-lane operand reads (16 features x 16 bytes) hit 64 different banks.  In a feature-major page a slot is
// one contiguous KB.  LW waves move the data: wave wl of them takes K slots and V slots wl + LW*j.  The full blocks of the
// prefix are moved by the kernels' own code: through a function that both call, the compiler's schedule of the 16-row kernel's
// main loop came out slower (two sequences of 8000 and 3001 tokens, 384 rows 38.9 -> 39.8 us).
template <int D, int LW>
struct BlockSlots {
  static constexpr int kKBytes = 32 * D * 2;        // K rows of a block (V takes the same)
  static constexpr int kStage = 2 * kKBytes;
  static constexpr int kSlots = kKBytes / 1024;     // of K (V: as many)
  static constexpr int KJ = kSlots / LW;            // K slots per loading wave, and V slots per loading wave
  static constexpr int kLoads = 2 * KJ;             // loads per block and loading wave
  static constexpr int kPieces = D / 8;             // 16-byte pieces per K row
  static constexpr int kRowsPerSlot = 64 / kPieces;
  static constexpr int kVBlocks = kSlots / 2;       // 32-feature blocks per 16-key half of the V tile
  static constexpr int kVHalf = D * 32;             // bytes of one 16-key half of the V tile
};

// Rows c0 .. c0+31 of the step's own block -> the stage at st_addr: K rows as above, V rows token-major (row r at 2*D*r, piece
// position p holding piece p ^ 2*(r&3)) for the transposing operand read.  Rows past R repeat the last one (they are masked).
// The lane id is laundered, here and below, so that none of this arithmetic is kept in registers across the main loop.
template <int D, int LW, typename Swz>
SS_DEV void move_own(const MsaArgs& a, int b, int hk, int c0, int wl, int lane, uint32_t st_addr, Swz swz) {
  using S = BlockSlots<D, LW>;
  asm volatile("" : "+v"(lane));
  const int ril = lane / S::kPieces, pch = lane % S::kPieces;
  const size_t head0 = ((size_t)b * a.R * a.Hkv + hk) * D;  // elements to row 0 of this sequence and head
  const uint16_t* kn = (const uint16_t*)a.k_new + head0;
  const uint16_t* vn = (const uint16_t*)a.v_new + head0;
#pragma unroll
  for (int j = 0; j < S::KJ; ++j) {
    const int sl = wl + LW * j;
    const int rr = S::kRowsPerSlot * sl + ril;
    const uint32_t row_off = (uint32_t)min(c0 + rr, a.R - 1) * (uint32_t)(a.Hkv * D * 2);
    dma16<false>(kn, row_off + (uint32_t)((pch ^ swz(rr)) * 16), st_addr + sl * 1024);
    dma16<false>(vn, row_off + (uint32_t)((pch ^ (2 * (rr & 3))) * 16), st_addr + S::kKBytes + sl * 1024);
  }
}
// The ragged last block of the prefix goes through registers (per-lane page lookups, clamped to existing keys; what is read in
// excess is masked).  base = its first cached token, last = the last one.
template <int D, int LW, typename Swz>
SS_DEV void load_ragged_block(const MsaArgs& a, const int32_t* my_table, const uint16_t* k_head, const uint16_t* v_head, int base,
                              int last, int wl, int lane, uintx4 (&stg)[BlockSlots<D, LW>::kLoads], Swz swz) {
  using S = BlockSlots<D, LW>;
  const size_t page_stride = (size_t)a.Hkv * a.page * D;  // elements per physical page (K and V alike)
  const int pmask = a.page - 1;
  asm volatile("" : "+v"(lane));
  const int ril = lane / S::kPieces, pch = lane % S::kPieces;
#pragma unroll
  for (int j = 0; j < S::KJ; ++j) {
    const int sl = wl + LW * j;
    const int rr = S::kRowsPerSlot * sl + ril;
    const int key = min(base + rr, last);
    const int pg = min(max(my_table[key >> a.page_shift], 0), a.num_pages - 1);
    const uint16_t* ksrc = k_head + (size_t)pg * page_stride + (size_t)(key & pmask) * D;
    const int half = sl / S::kVBlocks, dblk = sl % S::kVBlocks;
    const int vkey = min(base + 16 * half + (lane & 1) * 8, last & ~7);
    const int vpg = min(max(my_table[vkey >> a.page_shift], 0), a.num_pages - 1);
    const uint16_t* vsrc = v_head + (size_t)vpg * page_stride + (size_t)(dblk * 32 + (lane >> 1)) * a.page + (vkey & pmask);
    stg[j] = ld16(ksrc + ((pch ^ swz(rr)) * 8));
    stg[S::KJ + j] = ld16(vsrc);
  }
}
template <int D, int LW>
SS_DEV void store_ragged_block(unsigned char* st, int wl, int lane, const uintx4 (&stg)[BlockSlots<D, LW>::kLoads]) {
  using S = BlockSlots<D, LW>;
  asm volatile("" : "+v"(lane));
#pragma unroll
  for (int j = 0; j < S::KJ; ++j) {
    const int sl = wl + LW * j;
    *reinterpret_cast<uintx4*>(st + sl * 1024 + lane * 16) = stg[j];
    const int half = sl / S::kVBlocks, fr = (sl % S::kVBlocks) * 32 + (lane >> 1);
    *reinterpret_cast<uintx4*>(st + S::kKBytes + half * S::kVHalf + fr * 32 + (((lane & 1) ^ ((fr >> 3) & 1)) * 16)) = stg[S::KJ + j];
  }
}

// One wavefront cuts a batch anew and finds the piece of the workgroup in `slot` of XCD `xcd`; lane b holds sequence b's length
// and kept nodes.  Pieces keep the order of the host's cut: those of one sequence together, the splits of a head next to each
// other, the live row chunks of a (sequence, KV head, split) on one XCD.  Workgroup 0 leaves the table of cuts.
// cut [8]: sequence (64: no piece), split, KV head, row chunk, splits of the sequence, tokens of split 0 and of the others,
// the sequence's first slot.
SS_DEV void find_piece(const MsaArgs& a, int xcd, int slot, int lane, int lane_len, int lane_kept, int* cut) {
  const SeqCut r = plan_uneven(a, lane, len_units(lane_len, a), lane_kept);
  const int slots = wave_scan(r.n, lane), groups0 = (slots - r.n) * a.Hkv;  // pieces of earlier sequences
  const int skip = (groups0 + 7 - xcd) >> 3;    // this XCD takes the pieces that are xcd mod 8
  const int here = (((slots * a.Hkv + 7 - xcd) >> 3) - skip) * r.chunks;
  const int upto = wave_scan(here, lane);
  const int bb = __popcll(__ballot(upto <= slot));
  if (blockIdx.x == 0 && lane < a.B) a.cut_table[lane] = make_int2(r.n, slots - r.n);
  if (lane == 0) cut[0] = bb;  // 64: none
  if (lane == bb) {
    const int at = slot - (upto - here);
    const int piece = 8 * (skip + at / r.chunks) + xcd - groups0;
    cut[1] = piece % r.n;
    cut[2] = piece / r.n;
    cut[3] = at % r.chunks;
    cut[4] = r.n;
    cut[5] = 32 * r.split0;
    cut[6] = 32 * r.split;
    cut[7] = slots - r.n;
  }
}

}  // namespace ss
