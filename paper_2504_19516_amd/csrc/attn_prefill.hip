// Causal flash-style attention for prefill chunks on gfx950, reading K and V from the paged
// cache (the chunk's own K,V are written there first, so a chunk appended after p cached
// tokens needs no separate path).
//
// A workgroup of 4 waves owns 128 consecutive query rows of one head of one sequence, each
// wave 32 of them with its Q operands in registers, and walks 64-key tiles (four pages). Tiles go global -> LDS directly,
// two stages deep: wave w fetches page w of the tile after this one (8 KiB: 16 K rows and the transposed V page) while this one
// is consumed, so a tile costs one barrier and no staging registers. Per tile:
//   S^T[key, q] = K[key, :] . Q[q, :]          v_mfma_f32_32x32x16_bf16, A = K rows, B = Q rows
//   online softmax down the key axis: a lane holds one query column (16 keys per 32x32
//   block per lane half), so the running max/sum need one cross-half exchange only
//   O^T[dd, q] += V^T[dd, key] . P^T[key, q]   A = V^T rows (token-contiguous in a page),
//   B = P^T taken straight from the S^T accumulator registers (no LDS round trip).
// Row m of a 16-row group of the K operand holds token (m & 3) | ((m >> 3) & 1) << 2 | ((m >> 2) & 1) << 3 of its page: the
// eight S^T registers a lane half holds for a page are then its tokens 8 half .. 8 half + 7, which is how V^T lies in
// memory, so V pages are copied as they are and an operand read is 1 KiB of consecutive LDS. K rows are unpadded; the 16-byte
// chunk c of a row sits at slot c ^ swizzle(row), applied on the global side, so the operand reads are conflict free.
//
// Bound by issue: per tile a wave has 32 matrix-core instructions (1024 cycles) and about as many cycles of exponentials,
// maxima and conversions, which only a second wave on the SIMD can overlap; LDS holds two workgroups per CU. Tiles staged through
// registers, two barriers a tile and Q read from LDS took 658 us for 8192 rows of 32 heads (0.84 PFLOP/s), this form 505 (1.09); 2048
// rows on 224 CUs 68 -> 54, 301 rows 14.2 -> 10.4. Where a launch has only one workgroup per CU (1024 new tokens over 15 000 cached
// ones: 256) long key ranges are cut into parts (attn_prefill_plan), at the price of fp32 partial outputs. Launches of many and long
// ranges take two heads of a KV group in one workgroup (attn_prefill_pair_kernel).
#include <algorithm>
#include <functional>
#include <numeric>
#include <queue>

#include "kernels.h"

namespace sts {

constexpr int BQ = 128, BKV = 64;

constexpr float RESCALE_LOG2 = 8.f;
constexpr int AP_LDS_BASE = 1024;                 // buffers filled by direct-to-LDS loads stay clear of address 0
template <int D>
constexpr int attn_prefill_lds() { return AP_LDS_BASE + 2 * 2 * BKV * D * 2; }   // two stages of a K and a V^T tile

// max over a lane and its partner 32 lanes away (v_permlane32_swap: the upper half of the first
// operand trades places with the lower half of the second)
__device__ __forceinline__ float half_swap_max(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// The output of a wave's 32 query rows (lane l: row l % 32, columns 32 b + 8 r4 + 4 (l / 32) ..) through LDS, so that a store writes whole
// rows: straight from the registers it takes 16 or 32 bytes of each of 32 rows, four or two times the stores (8192 rows of 32 heads 516 ->
// 504 us with one head per workgroup, 1024 rows over 15 000 cached ones 255 -> 246). `buf` is this wave's, 32 rows of D elements of T; rows
// from n_rows on are left out. Returns NaN where an output is not finite.
template <int D, typename T>
__device__ __forceinline__ float store_rows(unsigned char* buf, int lane, const f32x16 (&o)[D / 32], float factor, int n_rows, T* dst, int ld) {
  constexpr int ROWB = D * (int)sizeof(T), CPR = ROWB / 16, RPI = 64 / CPR, SW = CPR < 16 ? CPR : 16;   // 16-byte chunks, swizzled by row
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(lane));                         // addresses are made here, not kept in registers from earlier on
#endif
  const int l32 = lane & 31, lh = lane >> 5;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
  for (int b = 0; b < D / 32; b++)
#pragma unroll
    for (int r4 = 0; r4 < 4; r4++) {
      const int c0 = sizeof(T) == 4 ? b * 8 + 2 * r4 + lh : b * 4 + r4;
      unsigned char* p = buf + l32 * ROWB + (c0 ^ (l32 % SW)) * 16;
      if constexpr (sizeof(T) == 4) {
        *reinterpret_cast<f32x4*>(p) = f32x4{o[b][4 * r4] * factor, o[b][4 * r4 + 1] * factor, o[b][4 * r4 + 2] * factor, o[b][4 * r4 + 3] * factor};
      } else {
        bf16x4 v;
#pragma unroll
        for (int e = 0; e < 4; e++) v[e] = f2bf(o[b][4 * r4 + e] * factor);
        *reinterpret_cast<bf16x4*>(p + 8 * lh) = v;
      }
    }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  float over = 0.f;
#pragma unroll
  for (int b = 0; b < D / 32; b++)
#pragma unroll
    for (int r = 0; r < 16; r++) over = fmaf(o[b][r], 0.f, over);
  const int r0 = lane / CPR, c = lane % CPR;
  u32x4 v[32 / RPI];
#pragma unroll
  for (int i = 0; i < 32 / RPI; i++) v[i] = *reinterpret_cast<const u32x4*>(buf + (i * RPI + r0) * ROWB + (c ^ ((i * RPI + r0) % SW)) * 16);
  unsigned char* p = reinterpret_cast<unsigned char*>(dst + (size_t)r0 * ld) + c * 16;
#pragma unroll
  for (int i = 0; i < 32 / RPI; i++, p += (size_t)RPI * ld * sizeof(T))
    if (i * RPI + r0 < n_rows) *reinterpret_cast<u32x4*>(p) = v[i];
  return over;
}

// One head of one query tile.
template <int D>
__device__ __forceinline__ void attn_prefill_head(unsigned char* smem, const bf16* __restrict__ qkv, int ld, bf16* __restrict__ out, int ldo, const PrefillSeq& sq,
                                                  const AttnItem& it, int head, const int* __restrict__ block_tables, const bf16* __restrict__ pool,
                                                  const KvGeom& geo, int n_q, float scale_log2e, float* __restrict__ part_ws) {
  constexpr int KSTEPS = D / 16, DB = D / 32;
  constexpr int ROWB = D * 2, CPR = D / 8, RPI = 64 / CPR, IPP = 16 / RPI;     // K row bytes, 16-byte chunks, rows per load, loads per page
  constexpr int PAGE = 16 * ROWB, TILE = 4 * PAGE, STAGE = 2 * TILE;           // bytes of a K (or V^T) page, tile; of a stage
  const int kvh = head / (n_q / geo.n_kv);
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int* bt = block_tables + sq.bt_off;

  const int qloc = it.q0 + wave * 32 + l32;              // row inside the chunk
  const int qpos = sq.p + qloc;                          // absolute position (causal limit)
  const int wave_min_qpos = sq.p + it.q0 + wave * 32;
  const int wave_max_qpos = wave_min_qpos + 31;
  const int k_end = sq.p + min(it.q0 + BQ, sq.sl);       // keys [0, k_end) are needed by these query rows
  const int kt_end = min(it.kt1, (k_end + BKV - 1) / BKV);
  const int last_page = min(sq.n_pages, (k_end + 15) / 16) - 1;

  // Q operands (rows past the chunk repeat its last row)
  bf16x8 qf[KSTEPS];
  {
    const bf16* q = qkv + (size_t)(sq.row0 + min(qloc, sq.sl - 1)) * ld + head * D + 8 * lh;
#pragma unroll
    for (int j = 0; j < KSTEPS; j++) qf[j] = *reinterpret_cast<const bf16x8*>(q + 16 * j);
  }

  // This wave's page of tile kt; past the last page it repeats that page: what is fetched for positions beyond the context is
  // causally masked (the pool only ever holds finite values, so 0 * V stays 0).
  const size_t page_stride = (size_t)geo.n_kv * geo.head_elems();
  const bf16* pool_h = pool + (size_t)kvh * geo.head_elems();
  auto page_id = [&](int kt) { return bt[min(kt * 4 + wave, last_page)]; };
  unsigned k_off[IPP];
#pragma unroll
  for (int j = 0; j < IPP; j++) {
    const int row = j * RPI + lane / CPR, swz = D == 128 ? row : (row >> 1) & 7;
    k_off[j] = (unsigned)row * ROWB + (unsigned)((lane % CPR) ^ swz) * 16u;
  }
  unsigned char* arena = smem + AP_LDS_BASE;
  auto issue = [&](int stage, int page) {
    const bf16* pb = pool_h + (size_t)__builtin_amdgcn_readfirstlane(page) * page_stride;
    unsigned char* dst = arena + stage * STAGE + wave * PAGE;
#pragma unroll
    for (int j = 0; j < IPP; j++) lds_dma16(pb, k_off[j], dst + j * 1024);
#pragma unroll
    for (int j = 0; j < IPP; j++) lds_dma16(pb + (size_t)16 * D, (unsigned)(j * 1024 + lane * 16), dst + TILE + j * 1024);
  };
  // K operand of this lane: token tok of page l32 >> 4 of a 32-key block
  const int tok = (l32 & 3) | (((l32 >> 3) & 1) << 2) | (((l32 >> 2) & 1) << 3);
  const int k_row = (l32 >> 4) * PAGE + tok * ROWB;
  int k_slot[KSTEPS];
#pragma unroll
  for (int j = 0; j < KSTEPS; j++) k_slot[j] = k_row + ((2 * j + lh) ^ (D == 128 ? tok : (tok >> 1) & 7)) * 16;
  const int v_lane = TILE + l32 * 32 + lh * 16;          // V^T operand: d row l32 of a 32-row block, tokens 8 lh .. of a page

  f32x16 o[DB];
#pragma unroll
  for (int b = 0; b < DB; b++)
#pragma unroll
    for (int r = 0; r < 16; r++) o[b][r] = 0.f;
  float m_ref = -INFINITY, l_run = 0.f;

  if (it.kt0 < kt_end) issue(it.kt0 & 1, page_id(it.kt0));
  int next_page = it.kt0 + 1 < kt_end ? page_id(it.kt0 + 1) : 0;
  for (int kt = it.kt0; kt < kt_end; kt++) {
    // this tile has landed (every wave waits for its own page), and nobody reads the other stage any more
    wait_vmem<0>();
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);
    if (kt + 1 < kt_end) {
      issue((kt + 1) & 1, next_page);
      next_page = page_id(kt + 2);
    }
    if (kt * BKV > wave_max_qpos) continue;               // wave-uniform: every key of the tile is masked
    const unsigned char* st = arena + (kt & 1) * STAGE;

    // ---- S^T = K Q^T (two 32-key blocks); operands of step j+1 are read from LDS while the MFMAs of step j run
    f32x16 s[2];
#pragma unroll
    for (int kb = 0; kb < 2; kb++)
#pragma unroll
      for (int r = 0; r < 16; r++) s[kb][r] = 0.f;
    __builtin_amdgcn_sched_barrier(0);
    {
      bf16x8 kf[2][2];
#pragma unroll
      for (int kb = 0; kb < 2; kb++) kf[0][kb] = *reinterpret_cast<const bf16x8*>(st + kb * 2 * PAGE + k_slot[0]);
#pragma unroll
      for (int j = 0; j < KSTEPS; j++) {
        const int c = j & 1, n = c ^ 1;
        if (j + 1 < KSTEPS) {
#pragma unroll
          for (int kb = 0; kb < 2; kb++) kf[n][kb] = *reinterpret_cast<const bf16x8*>(st + kb * 2 * PAGE + k_slot[j + 1]);
        }
#pragma unroll
        for (int kb = 0; kb < 2; kb++) s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[c][kb], qf[j], s[kb], 0, 0, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
#pragma unroll
      for (int j = 0; j + 1 < KSTEPS; j++) {
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    // first V^T operands: in flight during the softmax arithmetic
    bf16x8 vf[2][DB];
#pragma unroll
    for (int b = 0; b < DB; b++) vf[0][b] = *reinterpret_cast<const bf16x8*>(st + v_lane + b * 1024);
    __builtin_amdgcn_sched_barrier(0);
    // ---- causal mask and online softmax on the raw scores; the scale rides in the exponent's
    // fused multiply-add. The reference maximum m_ref is only moved when the tile maximum
    // exceeds it by more than 2^RESCALE_LOG2 (probabilities then stay below that factor, far
    // inside fp32/bf16 range), so the rescale of O and l is skipped on most tiles.
    if (kt * BKV + BKV - 1 > wave_min_qpos) {
#pragma unroll
      for (int kb = 0; kb < 2; kb++)
#pragma unroll
        for (int r = 0; r < 16; r++) {
          const int key = kt * BKV + kb * 32 + 16 * (r >> 3) + 8 * lh + (r & 7);
          if (key > qpos) s[kb][r] = -INFINITY;
        }
    }
    float mx = -INFINITY;
#pragma unroll
    for (int kb = 0; kb < 2; kb++)
#pragma unroll
      for (int r = 0; r < 16; r++) mx = fmaxf(mx, s[kb][r]);
    mx = half_swap_max(mx);
    const bool grow = (mx - m_ref) * scale_log2e > RESCALE_LOG2;     // false when both are -inf (NaN)
    if (__any(grow)) {                                               // wave-uniform
      const float m_upd = grow ? mx : m_ref;
      const float corr = (m_upd == -INFINITY) ? 1.f : __builtin_amdgcn_exp2f((m_ref - m_upd) * scale_log2e);
      m_ref = m_upd;
      l_run *= corr;
#pragma unroll
      for (int b = 0; b < DB; b++)
#pragma unroll
        for (int r = 0; r < 16; r++) o[b][r] *= corr;
    }
    const float nm = (m_ref == -INFINITY) ? 0.f : -m_ref * scale_log2e;
    float rs = 0.f;
#pragma unroll
    for (int kb = 0; kb < 2; kb++)
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const float p = __builtin_amdgcn_exp2f(fmaf(s[kb][r], scale_log2e, nm));
        s[kb][r] = p;
        rs += p;
      }
    l_run += rs;                                                      // this half's keys; halves are added at the end

    // ---- O^T += V^T P^T, a page (16 keys) at a time; the next page's V^T operands are read while the current one's MFMAs run
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int g = 0; g < 4; g++) {
      const int c = g & 1, n = c ^ 1;
      if (g + 1 < 4) {
#pragma unroll
        for (int b = 0; b < DB; b++) vf[n][b] = *reinterpret_cast<const bf16x8*>(st + v_lane + (g + 1) * PAGE + b * 1024);
      }
      bf16x8 pb;
#pragma unroll
      for (int e = 0; e < 8; e++) pb[e] = f2bf(s[g >> 1][8 * (g & 1) + e]);
#pragma unroll
      for (int b = 0; b < DB; b++) o[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[c][b], pb, o[b], 0, 0, 0);
    }
#pragma unroll
    for (int g = 0; g + 1 < 4; g++) {
      __builtin_amdgcn_sched_group_barrier(0x100, DB, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, DB, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, DB, 0);
    __builtin_amdgcn_sched_barrier(0);
  }

  l_run += __shfl_xor(l_run, 32, 64);
  __syncthreads();                                       // LDS now takes the output
  unsigned char* buf = arena + wave * (32 * D * 4);
  const int row0 = it.q0 + wave * 32;
  if (it.part >= 0) {
    // one part of the key range: unnormalised output, reference maximum (scaled) and sum of each query row
    float* po = part_ws + ((size_t)it.part * n_q + head) * BQ * (D + 2);
    if (lh == 0) *reinterpret_cast<f32x2*>(po + (size_t)BQ * D + (wave * 32 + l32) * 2) = f32x2{m_ref * scale_log2e, l_run};
    store_rows<D, float>(buf, lane, o, 1.f, 32, po + (size_t)wave * 32 * D, D);
  } else {
    store_rows<D, bf16>(buf, lane, o, 1.f / l_run, sq.sl - row0, out + (size_t)(sq.row0 + row0) * ldo + head * D, ldo);
  }
}

template <int D>
__global__ void __launch_bounds__(256, 2) attn_prefill_kernel(const bf16* __restrict__ qkv, int ld, bf16* __restrict__ out, int ldo,
                                                           const PrefillSeq* __restrict__ seqs, const AttnItem* __restrict__ items,
                                                           const int* __restrict__ block_tables, const bf16* __restrict__ pool,
                                                           KvGeom geo, int n_q, float scale_log2e, float* __restrict__ part_ws) {
  extern __shared__ __align__(16) unsigned char smem[];
  const AttnItem it = items[blockIdx.x / n_q];
  const PrefillSeq sq = seqs[it.seq];
  attn_prefill_head<D>(smem, qkv, ld, out, ldo, sq, it, blockIdx.x % n_q, block_tables, pool, geo, n_q, scale_log2e, part_ws);
}

// ---- two heads of a KV group per workgroup, one wave per SIMD (d = 128) ---------------------------------------------
// The kernel above is bound by issue: each of a SIMD's two waves multiplies, then makes its probabilities, and what overlaps is what the
// two happen to offer each other (about 1.05 PFLOP/s). Here a wave holds 32 query rows of two heads that share K and V, and every matrix
// instruction has a fixed piece of the rest placed behind it: one probability (exponential, fused multiply-add, sum, half a conversion),
// an LDS read, a piece of the copy of the tile after the next. A K or V^T operand read from LDS feeds two products instead of one. An LDS
// read stands right behind a product: ahead of it, it holds up the wave's vector instructions and with them the next product (44 cycles a
// product against 34). The reference maximum of a row, a chain from a tile's scores to its probabilities, moves by the rule of the kernel
// above, but the first half of a tile's probabilities is made before all of its scores are known: where a score outgrows the reference,
// which is rare, that half is made again. Products and sums run in the order of the kernel above, so both give the same bits.
// 8192 rows of 32 heads 521 us with one head per workgroup, 486 with two; 1024 over 15 000 cached ones 260 / 234, 256 over 15 000 84 / 76, 4096 over
// 8000 616 / 550. A reference that never moves saved the maxima (468, 230, 75, 535) but cost precision in rows that a late key dominates:
// there the moved one makes that key's probability exactly 1. What is left beside the loop, 5 to 6 us a workgroup, is its start (the
// first tiles' way from memory, their scores) and its output, which no second workgroup on the CU hides.
// o += a * b with o in accumulation registers; s = a * b + (FIRST ? 0 : s) with b in accumulation registers. In assembly so that the
// 128 accumulators stay in place and the scores come out in the registers the vector ALUs can read.
__device__ __forceinline__ void mma32_acc(f32x16& o, const bf16x8& a, const bf16x8& b) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(o) : "v"(a), "v"(b));
#endif
}
template <bool FIRST>
__device__ __forceinline__ void mma32_scores(f32x16& s, const bf16x8& a, const bf16x8& b) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (FIRST) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(s) : "v"(a), "a"(b));
  else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(s) : "v"(a), "a"(b));
#endif
}
// The compiler does not know that these take time: wait before other instructions touch their results, and after others wrote them.
__device__ __forceinline__ void mma32_settle() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#endif
}
__device__ __forceinline__ void mma32_operand_idle() {   // between a vector-ALU write and the product that reads it
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_nop 1");
#endif
}
// In assembly: the compiler would first quiet the operands, which it does not know.
__device__ __forceinline__ float max3(float a, float b, float c) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm("v_max3_f32 %0, %0, %1, %2" : "+v"(a) : "v"(b), "v"(c));
#endif
  return a;
}
__device__ __forceinline__ void pin_f32(float& x) {      // the sum is made here, not where the compiler would sink it to
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(x));
#endif
}
__device__ __forceinline__ unsigned pin_pair(float a, float b) {
  bf16x2 v; v[0] = f2bf(a); v[1] = f2bf(b);
  unsigned w = __builtin_bit_cast(unsigned, v);
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(w));
#endif
  return w;
}
__device__ __forceinline__ void mma32_tie(f32x16& s) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(s));
#endif
}
__device__ __forceinline__ void mma32_tie_acc(f32x16& s) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+a"(s));
#endif
}
constexpr int PAIR_STAGES = 4;
constexpr int attn_pair_lds() { return AP_LDS_BASE + PAIR_STAGES * 2 * BKV * 128 * 2; }

__global__ void __launch_bounds__(256, 1) attn_prefill_pair_kernel(const bf16* __restrict__ qkv, int ld, bf16* __restrict__ out, int ldo,
                                                                   const PrefillSeq* __restrict__ seqs, const AttnItem* __restrict__ items,
                                                                   const int* __restrict__ block_tables, const bf16* __restrict__ pool,
                                                                   KvGeom geo, int n_q, float scale_log2e, float* __restrict__ part_ws) {
  constexpr int D = 128, KSTEPS = D / 16, DB = D / 32, NS = PAIR_STAGES;
  constexpr int ROWB = D * 2, CPR = D / 8, RPI = 64 / CPR, IPP = 16 / RPI;     // K row bytes, 16-byte chunks, rows per load, loads per page
  constexpr int PAGE = 16 * ROWB, TILE = 4 * PAGE, STAGE = 2 * TILE;           // bytes of a K (or V^T) page, tile; of a stage
  constexpr int LOADS = 2 * IPP;                                               // of a wave per tile
  extern __shared__ __align__(16) unsigned char smem[];
  typedef const __attribute__((address_space(3))) unsigned char* lds_cptr;

  const int pairs = n_q >> 1, head0 = (blockIdx.x % pairs) * 2;
  const AttnItem it = items[blockIdx.x / pairs];
  const PrefillSeq sq = seqs[it.seq];
  const int kvh = head0 / (n_q / geo.n_kv);
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int* bt = block_tables + sq.bt_off;

  // Rows past the chunk are its last row once more, with that row's keys: what a page holds behind the context, left by another
  // sequence, must not decide whether the rows are taken again (below).
  const int row_first = it.q0 + wave * 32, row_last = sq.sl - 1;
  const int qloc = min(row_first + l32, row_last);       // row inside the chunk
  const int qpos = sq.p + qloc;                          // absolute position (causal limit)
  const int wave_min_qpos = sq.p + min(row_first, row_last);
  const int wave_max_qpos = sq.p + min(row_first + 31, row_last);
  const int k_end = sq.p + min(it.q0 + BQ, sq.sl);       // keys [0, k_end) are needed by these query rows
  const int kt_end = min(it.kt1, (k_end + BKV - 1) / BKV);
  const int wave_end = min(kt_end, wave_max_qpos / BKV + 1);                   // tiles past it are masked for all of this wave's rows
  const int last_page = min(sq.n_pages, (k_end + 15) / 16) - 1;

  // Q operands of both heads, in accumulation registers
  bf16x8 qf[2][KSTEPS];
#pragma unroll
  for (int x = 0; x < 2; x++) {
    const bf16* q = qkv + (size_t)(sq.row0 + qloc) * ld + (head0 + x) * D + 8 * lh;
#pragma unroll
    for (int j = 0; j < KSTEPS; j++) qf[x][j] = *reinterpret_cast<const bf16x8*>(q + 16 * j);
  }

  // A wave fetches one page per tile; past the last page it repeats that page: what is fetched for positions beyond the context is
  // causally masked (the pool only ever holds finite values, so 0 * V stays 0). The ids of its pages of 64 tiles, one per lane.
  const size_t page_stride = (size_t)geo.n_kv * geo.head_elems();
  const bf16* pool_h = pool + (size_t)kvh * geo.head_elems();
  int ids = 0, ids_kt = 0;
  auto fetch_ids = [&](int kt) { ids_kt = kt; ids = bt[min((kt + lane) * 4 + wave, last_page)]; };
  auto page_base = [&](int kt) -> const bf16* {
    return pool_h + (size_t)__builtin_amdgcn_readlane(ids, __builtin_amdgcn_readfirstlane(kt - ids_kt)) * page_stride;
  };
  unsigned k_off[IPP];
#pragma unroll
  for (int j = 0; j < IPP; j++) {
    const int row = j * RPI + lane / CPR;
    k_off[j] = (unsigned)row * ROWB + (unsigned)((lane % CPR) ^ row) * 16u;
  }
  const unsigned v_off = (unsigned)lane * 16u;
  unsigned char* arena = smem + AP_LDS_BASE;
  const unsigned dma_base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)arena + wave * PAGE;
  auto dma_first = [&](auto j_c, unsigned stage) {       // operation j of a tile: K rows, then V^T
    constexpr int j = decltype(j_c)::value;
    dma_m0<(j < IPP ? j * 1024 : TILE + (j - IPP) * 1024)>(stage);
  };
  auto dma_second = [&](auto j_c, const bf16* pb) {
    constexpr int j = decltype(j_c)::value;
    if constexpr (j < IPP) dma_load(reinterpret_cast<const unsigned char*>(pb), k_off[j]);
    else dma_load(reinterpret_cast<const unsigned char*>(pb) + PAGE + (j - IPP) * 1024, v_off);
  };
  // K operand of this lane: token tok of page l32 >> 4 of a 32-key block
  const int tok = (l32 & 3) | (((l32 >> 3) & 1) << 2) | (((l32 >> 2) & 1) << 3);
  const int k_row = (l32 >> 4) * PAGE + tok * ROWB;
  int k_slot[KSTEPS];
#pragma unroll
  for (int j = 0; j < KSTEPS; j++) k_slot[j] = k_row + ((2 * j + lh) ^ tok) * 16;
  const int v_lane = TILE + l32 * 32 + lh * 16;          // V^T operand: d row l32 of a 32-row block, tokens 8 lh .. of a page
  const lds_cptr lds0 = (lds_cptr)arena;
  auto lds16 = [](lds_cptr p) { return *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(p); };

  f32x16 o[2][DB];
#pragma unroll
  for (int x = 0; x < 2; x++)
#pragma unroll
    for (int b = 0; b < DB; b++)
#pragma unroll
      for (int r = 0; r < 16; r++) o[x][b][r] = 0.f;
  float nm[2] = {0.f, 0.f}, m_ref[2] = {-INFINITY, -INFINITY}, l_run[2] = {0.f, 0.f}, l_tile[2] = {0.f, 0.f};
  f32x16 s[2][2];                                        // scores of a tile: [head][32-key block]
  u32x4 pb[2][4];                                        // probabilities: [head][page], bf16 pairs
#pragma unroll
  for (int x = 0; x < 2; x++)
#pragma unroll
    for (int g = 0; g < 4; g++) pb[x][g] = u32x4{0u, 0u, 0u, 0u};
  auto mask = [&](auto kb_c, int kt) {
    constexpr int kb = decltype(kb_c)::value;
#pragma unroll
    for (int x = 0; x < 2; x++)
#pragma unroll
      for (int r = 0; r < 16; r++) {
        const int key = kt * BKV + kb * 32 + 16 * (r >> 3) + 8 * lh + (r & 7);
        if (key > qpos) s[x][kb][r] = -INFINITY;
      }
  };
  const int unmasked = min(wave_end, (wave_min_qpos + 1) / BKV);               // tiles before it need no mask
  // Probability q of the stream: block q / 32 ^ 1 (the second block of a tile, then the first of the next), page q / 16 % 2 of it, head
  // q / 8 % 2. Its exponent is made with the exponential of the one before, and it is added up and rounded with that of the next: no
  // instruction waits for the one before it.
  float y_next = 0.f, p_last = 0.f, p_even = 0.f;
  auto finish = [&](auto q_c) {
    constexpr int q = decltype(q_c)::value, kb = q / 32 ^ 1, g = q / 16 % 2, x = q / 8 % 2, e = q % 8;
    // this half's keys, tile by tile as the kernel above adds them; halves are added at the end
    if constexpr (kb == 0 && g == 0 && e == 0) l_tile[x] = p_last; else l_tile[x] += p_last;
    if constexpr (kb == 1 && g == 1 && e == 7) { l_run[x] += l_tile[x]; pin_f32(l_run[x]); } else pin_f32(l_tile[x]);
    if constexpr (e & 1) pb[x][2 * kb + g][e / 2] = pin_pair(p_even, p_last);
    else p_even = p_last;
  };
  auto exponent = [&](auto q_c) {
    constexpr int q = decltype(q_c)::value % 64, kb = q / 32 ^ 1, g = q / 16 % 2, x = q / 8 % 2, e = q % 8;
    y_next = fmaf(s[x][kb][8 * g + e], scale_log2e, nm[x]);
  };
  auto score = [&](auto q_c) {                           // exponential of q, exponent of q + 1, the rest of q - 1
    constexpr int q = decltype(q_c)::value % 64;
    const float y = y_next;
    exponent(std::integral_constant<int, q + 1>{});
    const float p = __builtin_amdgcn_exp2f(y);
    finish(std::integral_constant<int, (q + 63) % 64>{});
    p_last = p;
  };
  auto first_block = [&]() {                             // the first block's probabilities but the last five
    exponent(std::integral_constant<int, 32>{});
    static_for<27>([&](auto q_c) {
      constexpr int q = 32 + decltype(q_c)::value;
      if constexpr (q == 32) {
        const float y = y_next;
        exponent(std::integral_constant<int, 33>{});
        p_last = __builtin_amdgcn_exp2f(y);
      } else score(std::integral_constant<int, q>{});
    });
  };
  bf16x8 kf[4], vf[2][DB];
  // Largest score of the tile after the one in hand, of this lane half, before the causal mask of its second block: where it does not
  // outgrow the reference, no score does that counts.
  float mx[2];
  const float reach = RESCALE_LOG2 * 0.999f / scale_log2e;
  auto max_of = [&](auto x_c, auto kb_c, auto r_c) {
    constexpr int x = decltype(x_c)::value, kb = decltype(kb_c)::value, r = decltype(r_c)::value;
    mx[x] = max3(mx[x], s[x][kb][r], s[x][kb][r + 1]);
  };

  if (it.kt0 < kt_end) {
    fetch_ids(it.kt0);
    for (int i = 0; i < 2; i++) {
      const bf16* page = page_base(it.kt0 + i);
      static_for<LOADS>([&](auto j_c) {
        dma_first(j_c, dma_base + ((it.kt0 + i) % NS) * STAGE);
        dma_m0_idle();
        dma_second(j_c, page);
      });
    }
    wait_vmem<0>();                                      // the first two tiles have landed
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    // the first one's scores, the reference maxima and the first block's probabilities but the last five
    const lds_cptr kst = lds0 + (it.kt0 % NS) * STAGE, vst = kst + v_lane;
    static_for<KSTEPS>([&](auto j_c) {
      constexpr int j = decltype(j_c)::value;
#pragma unroll
      for (int kb = 0; kb < 2; kb++) kf[kb] = lds16(kst + k_slot[j] + kb * 2 * PAGE);
#pragma unroll
      for (int kb = 0; kb < 2; kb++)
#pragma unroll
        for (int x = 0; x < 2; x++) mma32_scores<(j == 0)>(s[x][kb], kf[kb], qf[x][j]);
    });
#pragma unroll
    for (int b = 0; b < DB; b++) vf[0][b] = lds16(vst + 2 * PAGE + b * 1024);
    mma32_settle();
    static_for<4>([&](auto q) { mma32_tie(s[decltype(q)::value / 2][decltype(q)::value % 2]); });
    if (it.kt0 >= unmasked) { mask(std::integral_constant<int, 0>{}, it.kt0); mask(std::integral_constant<int, 1>{}, it.kt0); }
#pragma unroll
    for (int x = 0; x < 2; x++) {
      float m = -INFINITY;
#pragma unroll
      for (int kb = 0; kb < 2; kb++)
#pragma unroll
        for (int r = 0; r < 16; r++) m = fmaxf(m, s[x][kb][r]);
      m_ref[x] = half_swap_max(m);
      nm[x] = -m_ref[x] * scale_log2e;
    }
    first_block();
    if (it.kt0 + 1 < wave_end) {                         // K operands of the next tile's first steps
#pragma unroll
      for (int j = 0; j < 2; j++) kf[j] = lds16(lds0 + ((it.kt0 + 1) % NS) * STAGE + k_slot[j]);
    }
  }
  // One iteration, 64 products, turn by turn (but for the last four of the scores a product depends on the fourth one before it at the
  // nearest), a probability between any two:
  //   O += pages 2 and 3 of tile kt - 1, scores of the first 32 keys of kt + 1;   probabilities of the second 32 keys of tile kt
  //   O += pages 0 and 1 of tile kt, scores of the second 32 keys of kt + 1;      probabilities of the first 32 keys of tile kt + 1
  // The probabilities run five products behind: then a score is read well after its last product and before the next tile's first
  // overwrites it, and a page's probabilities are written after the products of the page before have read theirs.
  auto product_o = [&](auto i_c, auto g0_c) {            // product i of pages g0 and g0 + 1
    constexpr int i = decltype(i_c)::value, g0 = decltype(g0_c)::value, x = i / 4 % 2, b = i % 4;
    mma32_acc(o[x][b], vf[i / 8][b], __builtin_bit_cast(bf16x8, pb[x][g0 + i / 8]));
  };
  // product i of 16 of a run of scores: head 0 two steps ahead of head 1
  static constexpr int SX[16] = {0, 0, 1, 0, 1, 0, 1, 0, 1, 0, 1, 0, 1, 0, 1, 1}, SJ[16] = {0, 1, 0, 2, 1, 3, 2, 4, 3, 5, 4, 6, 5, 7, 6, 7};
  // O and scores in turns; at the end the last four of the scores first, and the maxima of what they finish beside the last of O, so
  // that the tile's maxima are known when the iteration ends. (No product of O may come later than that: the probabilities of the
  // next tile take the place of the ones it reads.)
  static constexpr auto is_score = [](int u) { return u < 56 ? u % 2 == 1 : u < 60; };
  static constexpr auto number = [](int u) { return u < 56 ? u % 32 / 2 : u < 60 ? u - 44 : u - 48; };
  int kt = it.kt0;
  const bf16* page = nullptr;
  for (; kt + 1 < wave_end; kt++) {
    const lds_cptr vprev = lds0 + ((kt > it.kt0 ? kt - 1 : kt) % NS) * STAGE + v_lane, vst = lds0 + (kt % NS) * STAGE + v_lane;
    const lds_cptr kst = lds0 + ((kt + 1) % NS) * STAGE, knext = lds0 + ((kt + 2) % NS) * STAGE;
    const unsigned stage = dma_base + ((kt + 2) % NS) * STAGE;
    if (kt + 2 - ids_kt >= 64) fetch_ids(kt + 2);
    page = page_base(kt + 2);
    static_for<64>([&](auto u_c) {
      constexpr int u = decltype(u_c)::value, half = u / 32, i = number(u);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (u == 54) {
        wait_vmem<0>();                                  // tile kt + 2 has landed
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
      }
      // this wave's page of tile kt + 2
      if constexpr (u < 16 && u % 2 == 1) dma_first(std::integral_constant<int, u / 2>{}, stage);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (!is_score(u)) product_o(std::integral_constant<int, i>{}, std::integral_constant<int, half ? 0 : 2>{});
      else mma32_scores<(SJ[i] == 0)>(s[SX[i]][half], kf[SJ[i] % 4], qf[SX[i]][SJ[i]]);
      __builtin_amdgcn_sched_barrier(0);
      // LDS reads: V^T operands of a page once the page before is through, K operands of a step (head 0 takes it first) five to seven
      // products ahead
      if constexpr (u >= 4 && u < 12 && u % 2 == 0) vf[1][u / 2 - 2] = lds16(vprev + 3 * PAGE + (u / 2 - 2) * 1024);
      if constexpr (u >= 18 && u < 26 && u % 2 == 0) vf[0][u / 2 - 9] = lds16(vst + (u / 2 - 9) * 1024);
      if constexpr (u >= 34 && u < 42 && u % 2 == 0) vf[1][u / 2 - 17] = lds16(vst + PAGE + (u / 2 - 17) * 1024);
      if constexpr (u >= 48 && u < 56 && u % 2 == 0) vf[0][u / 2 - 24] = lds16(vst + 2 * PAGE + (u / 2 - 24) * 1024);
      // step j of a run is read where the run stands at product KU[j] (KV[j] in the second half): steps 0 and 1 before it begins
      constexpr int KU[8] = {-6, -4, 1, 5, 9, 13, 17, 21}, KV[8] = {-6, -4, 1, 5, 9, 13, 17, 19};
      static_for<8>([&](auto j_c) {
        constexpr int j = decltype(j_c)::value;
        if constexpr (KV[j] + 32 == u) kf[j % 4] = lds16(kst + k_slot[j] + 2 * PAGE);                       // second block
        else if constexpr (KU[j] + 64 == u) kf[j % 4] = lds16(knext + k_slot[j]);                           // the tile after, first block
        else if constexpr (KU[j] == u) kf[j % 4] = lds16(kst + k_slot[j]);
      });
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (u < 16 && u % 2 == 1) dma_second(std::integral_constant<int, u / 2>{}, page);
      score(std::integral_constant<int, (u + 59) % 64>{});
      if constexpr (u == 36) mx[0] = mx[1] = -INFINITY;
      if constexpr (u >= 37 && u < 53) max_of(std::integral_constant<int, (u - 37) / 8>{}, std::integral_constant<int, 0>{}, std::integral_constant<int, (u - 37) % 8 * 2>{});
      if constexpr (u >= 60)                               // head 0, then head 1: their scores are done with u = 57 and 59
        static_for<4>([&](auto r_c) { max_of(std::integral_constant<int, u / 62>{}, std::integral_constant<int, 1>{}, std::integral_constant<int, u % 2 * 8 + decltype(r_c)::value * 2>{}); });
      if constexpr (u == 31 || u == 63) {
        __builtin_amdgcn_sched_barrier(0);
        if (kt + 1 >= unmasked) {
          mma32_settle();
          static_for<2>([&](auto x_c) { mma32_tie(s[decltype(x_c)::value][u / 32]); });
          mask(std::integral_constant<int, u / 32>{}, kt + 1);
        }
      }
    });
    __builtin_amdgcn_sched_barrier(0);
    if (__any(mx[0] - m_ref[0] > reach || mx[1] - m_ref[1] > reach)) {
      // A score of tile kt + 1 outgrows a reference: what is left of tile kt is added, then the references move, O and the sums are
      // scaled, and the probabilities already made of tile kt + 1 are made again.
      float corr[2];
      bool moved = false;
#pragma unroll
      for (int x = 0; x < 2; x++) {
        float m = -INFINITY;
#pragma unroll
        for (int kb = 0; kb < 2; kb++)
#pragma unroll
          for (int r = 0; r < 16; r++) m = fmaxf(m, s[x][kb][r]);
        m = half_swap_max(m);
        const bool grow = (m - m_ref[x]) * scale_log2e > RESCALE_LOG2;
        const float m_upd = grow ? m : m_ref[x];
        corr[x] = grow ? __builtin_amdgcn_exp2f((m_ref[x] - m_upd) * scale_log2e) : 1.f;
        m_ref[x] = m_upd;
        moved |= grow;
      }
      if (__any(moved)) {
#pragma unroll
        for (int b = 0; b < DB; b++) vf[1][b] = lds16(vst + 3 * PAGE + b * 1024);
        __builtin_amdgcn_sched_barrier(0);
        static_for<16>([&](auto i_c) { product_o(i_c, std::integral_constant<int, 2>{}); });
        mma32_settle();
        static_for<2 * DB>([&](auto q) {
          constexpr int x = decltype(q)::value / DB, b = decltype(q)::value % DB;
          mma32_tie_acc(o[x][b]);
#pragma unroll
          for (int r = 0; r < 16; r++) o[x][b][r] *= corr[x];
          mma32_tie_acc(o[x][b]);
        });
#pragma unroll
        for (int x = 0; x < 2; x++) {
          l_run[x] *= corr[x];
          nm[x] = -m_ref[x] * scale_log2e;
          pb[x][2] = pb[x][3] = u32x4{0u, 0u, 0u, 0u};
        }
        first_block();
        mma32_settle();
      }
    }
  }
  if (it.kt0 < kt_end) {                                 // what is left of the wave's last tile
    const lds_cptr vprev = lds0 + ((kt > it.kt0 ? kt - 1 : kt) % NS) * STAGE + v_lane, vst = lds0 + (kt % NS) * STAGE + v_lane;
    static_for<16>([&](auto u_c) {
      constexpr int u = decltype(u_c)::value;
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (u < 4) vf[1][u] = lds16(vprev + 3 * PAGE + u * 1024);
      __builtin_amdgcn_sched_barrier(0);
      product_o(u_c, std::integral_constant<int, 2>{});
      __builtin_amdgcn_sched_barrier(0);
      score(std::integral_constant<int, (u + 59) % 64>{});
    });
    static_for<21>([&](auto t_c) { score(std::integral_constant<int, 11 + decltype(t_c)::value>{}); });
    finish(std::integral_constant<int, 31>{});
#pragma unroll
    for (int h = 0; h < 2; h++) {
#pragma unroll
      for (int g = 0; g < 2; g++)
#pragma unroll
        for (int b = 0; b < DB; b++) vf[g][b] = lds16(vst + (2 * h + g) * PAGE + b * 1024);
      __builtin_amdgcn_sched_barrier(0);
      mma32_operand_idle();
      static_for<16>([&](auto i_c) { if (h == 0) product_o(i_c, std::integral_constant<int, 0>{}); else product_o(i_c, std::integral_constant<int, 2>{}); });
      __builtin_amdgcn_sched_barrier(0);
    }
    kt++;
  }
  for (kt = kt - 1; kt + 1 < kt_end; kt++) {             // nothing left for this wave's rows: its pages for the others
    if (kt + 2 - ids_kt >= 64) fetch_ids(kt + 2);
    page = page_base(kt + 2);
    static_for<LOADS>([&](auto j_c) {
      dma_first(j_c, dma_base + ((kt + 2) % NS) * STAGE);
      dma_m0_idle();
      dma_second(j_c, page);
    });
    wait_vmem<0>();
    __builtin_amdgcn_s_barrier();
  }
  wait_vmem<0>();                                        // pieces on their way to LDS
  mma32_settle();
  static_for<2 * DB>([&](auto q) { mma32_tie_acc(o[decltype(q)::value / DB][decltype(q)::value % DB]); });

  float l_all[2];
#pragma unroll
  for (int x = 0; x < 2; x++) l_all[x] = l_run[x] + __shfl_xor(l_run[x], 32, 64);
  float over = 0.f;                                      // NaN where an output is not finite
  __syncthreads();                                       // LDS now takes the output
  unsigned char* buf = arena + wave * (32 * D * 4);
  const int row0 = it.q0 + wave * 32;
  if (it.part >= 0) {
    // one part of the key range: unnormalised output, reference maximum (scaled) and sum of each query row
#pragma unroll
    for (int x = 0; x < 2; x++) {
      float* po = part_ws + ((size_t)it.part * n_q + head0 + x) * BQ * (D + 2);
      if (lh == 0) *reinterpret_cast<f32x2*>(po + (size_t)BQ * D + (wave * 32 + l32) * 2) = f32x2{m_ref[x] * scale_log2e, l_all[x]};
      over += store_rows<D, float>(buf, lane, o[x], 1.f, 32, po + (size_t)wave * 32 * D, D);
    }
  } else {
#pragma unroll
    for (int x = 0; x < 2; x++)
      over += store_rows<D, bf16>(buf, lane, o[x], 1.f / l_all[x], sq.sl - row0, out + (size_t)(sq.row0 + row0) * ldo + (head0 + x) * D, ldo);
  }
  // An infinity or a NaN in Q, K or V, times a probability of zero here and left out there, may show in other rows than above. Then the
  // workgroup takes its query tile again, head by head, and a wave writes its rows once more. After the output, so that no
  // accumulator has to live through it (in scratch: 10 us a workgroup).
  if (__syncthreads_or(!(l_all[0] < INFINITY) || !(l_all[1] < INFINITY) || over != 0.f))
    for (int x = 0; x < 2; x++) {
      __syncthreads();
      attn_prefill_head<D>(smem, qkv, ld, out, ldo, sq, it, head0 + x, block_tables, pool, geo, n_q, scale_log2e, part_ws);
    }
}

// Adds up the parts of one query tile's key range: out = sum_c o_c 2^(m_c - m) / sum_c l_c 2^(m_c - m), parts in order. One thread
// per four elements; bound by the fp32 parts it reads. Every row sees keys of every part (attn_prefill_plan), so m is finite.
template <int D>
__global__ void __launch_bounds__(256) attn_prefill_merge_kernel(bf16* __restrict__ out, int ldo, const PrefillSeq* __restrict__ seqs,
                                                                 const AttnMerge* __restrict__ merges, int n_q, const float* __restrict__ part_ws) {
  const int head = blockIdx.x % n_q;
  const AttnMerge mg = merges[blockIdx.x / n_q];
  const PrefillSeq sq = seqs[mg.seq];
  const int e = blockIdx.y * 256 + threadIdx.x, r = e / (D / 4), dd = e % (D / 4) * 4;
  if (mg.q0 + r >= sq.sl) return;
  const size_t stride = (size_t)n_q * BQ * (D + 2);
  const float* p = part_ws + ((size_t)mg.part0 * n_q + head) * BQ * (D + 2);
  const float* ml = p + (size_t)BQ * D + r * 2;
  float m = -INFINITY;
  for (int c = 0; c < mg.parts; c++) m = fmaxf(m, ml[c * stride]);
  float l = 0.f;
  f32x4 o = {0.f, 0.f, 0.f, 0.f};
  for (int c = 0; c < mg.parts; c++) {
    const f32x2 v = *reinterpret_cast<const f32x2*>(ml + c * stride);
    const f32x4 x = *reinterpret_cast<const f32x4*>(p + c * stride + (size_t)r * D + dd);
    const float w = __builtin_amdgcn_exp2f(v[0] - m);
    l += v[1] * w;
#pragma unroll
    for (int i = 0; i < 4; i++) o[i] += x[i] * w;
  }
  bf16x4 y;
#pragma unroll
  for (int i = 0; i < 4; i++) y[i] = f2bf(o[i] / l);
  *reinterpret_cast<bf16x4*>(out + (size_t)(sq.row0 + mg.q0 + r) * ldo + head * D + dd) = y;
}

int attn_prefill_tile_q() { return BQ; }
size_t attn_prefill_part_floats(int n_q, int d) { return (size_t)n_q * BQ * (d + 2); }

// The launch's work: query tiles of every sequence, longest key range first (the tail of the launch is then made of short
// ones). A key range is cut into the number of parts (up to 8) that brings them nearest to what one workgroup slot of the
// partition (two per CU) gets of an even deal, or to 32 tiles (2048 keys: a part costs fp32 outputs written and read back, about
// an eighth of that work) where that is less; a part has at least 24 tiles, more keys than a query tile has rows. So ranges
// are cut only where a few long ones leave slots empty: 1024 new tokens over 15 000 cached ones, 32 heads on 256 CUs, two parts
// (406 -> 274 + 10 us a layer); a 2048-token prompt or 8192 rows on their own are not. At most `max_extra` items more than query tiles and
// `max_parts` parts.
// `pairs` says that two heads per workgroup is estimated the faster form. In units of a CU's time for 64 keys of two heads: pairs, one
// workgroup per CU, take the busiest CU's tiles and 3 units beside them for each workgroup, which nothing hides; single heads,
// two workgroups per CU, 1.12 times the mean of an even deal and the busiest slot's tiles (a workgroup that is alone on its CU runs faster),
// and 3 units. Measured one / two heads per workgroup, us, 32 heads (estimated quotient of two and one in brackets):
// 256 CUs: 8192 rows 521 / 486 (0.92), 4096 147 / 132 (0.93), 3000 86 / 85 (0.99), 2048 50 / 57 (1.14), 1024 over 15 000 cached 260 / 234 (0.91), over 4000
// 92 / 89 (0.94), over 2000 66 / 76 (1.21), 8 x 512 over 700 86 / 81 (0.97), 4 x 2048 150 / 157 (1.01), 3 x 1500 73 / 81 (1.09), six ragged prompts 53 / 58
// (1.09). 224 CUs: 8192 547 / 532 (0.94), 1024 over 15 000 334 / 356 (1.14: 256 workgroups), 8 x 512 over 700 92 / 97 (1.10). 64 CUs: 8192 1481 / 1434 (0.93), 2048
// 114 / 125 (1.01), 1024 over 15 000 741 / 631 (0.90), 4 x 2048 454 / 469 (1.04). The faster form in all 34 launches measured.
// Tiles of the busiest of `slots` slots where `n` workgroups of each item, of its tiles and `extra` units, go to the slot that is free first.
static double busiest_slot(const std::vector<AttnItem>& items, int n, int slots, double extra) {
  const int same = std::gcd(n, slots);               // so many slots and workgroups of an item at a time do alike
  std::priority_queue<double, std::vector<double>, std::greater<double>> free_at(std::greater<double>(), std::vector<double>(slots / same, 0.0));
  double end = 0.0;
  for (const AttnItem& it : items)
    for (int i = 0; i < n / same; i++) {
      const double t = free_at.top() + (it.kt1 - it.kt0) + extra;
      free_at.pop();
      free_at.push(t);
      end = std::max(end, t);
    }
  return end;
}
AttnPlan attn_prefill_plan(int n_seqs, const int* lens, const int* priors, int n_q, int slots, int max_extra, long long max_parts) {
  AttnPlan plan;
  struct Tile { int seq, q0, tiles; };
  std::vector<Tile> tiles;
  long long total = 0;
  for (int i = 0; i < n_seqs; i++)
    for (int q0 = 0; q0 < lens[i]; q0 += BQ) {
      tiles.push_back({i, q0, (priors[i] + std::min(q0 + BQ, lens[i]) + BKV - 1) / BKV});
      total += tiles.back().tiles;
    }
  const double share = std::max(32.0, (double)total * n_q / std::max(1, slots));
  for (const Tile& t : tiles) {
    int parts = std::max(1, std::min(8, (int)(t.tiles / share + 0.5)));
    if (parts - 1 > max_extra || plan.parts + parts > max_parts) parts = 1;
    for (int z = 0; z < parts; z++)
      plan.items.push_back(AttnItem{t.seq, t.q0, (int)((long long)t.tiles * z / parts), (int)((long long)t.tiles * (z + 1) / parts), parts > 1 ? plan.parts + z : -1});
    if (parts > 1) { plan.merges.push_back(AttnMerge{t.seq, t.q0, plan.parts, parts}); plan.parts += parts; max_extra -= parts - 1; }
  }
  std::stable_sort(plan.items.begin(), plan.items.end(), [](const AttnItem& a, const AttnItem& b) { return a.kt1 - a.kt0 > b.kt1 - b.kt0; });
  if (n_q % 2 == 0 && slots >= 2) {
    const double deal = (double)total * n_q / slots;
    plan.pairs = busiest_slot(plan.items, n_q / 2, slots / 2, 3.0) < 1.12 * (0.5 * (deal + busiest_slot(plan.items, n_q, slots, 0.0)) + 3.0);
  }
  return plan;
}

// Heads per workgroup of a launch whose plan wants `pairs` or not: two need d = 128 and an even group.
int attn_prefill_heads(bool pairs, int n_q, int n_kv, int d) { return pairs && d == 128 && (n_q / n_kv) % 2 == 0 ? 2 : 1; }

// qkv: packed [rows, ld] with Q of head h at columns [h*d, (h+1)*d), already rotated.
// out: [rows, ldo], head h at the same columns. items: query tiles (sequence, first row, key tiles, part or -1);
// one workgroup per (item, `heads` heads of a KV group, 1 or 2: attn_prefill_heads). merges: the query tiles whose key range was cut. part_ws:
// attn_prefill_part_floats(n_q, d) per part.
// Requires page_tokens == 16 and d in {64, 128}.
hipError_t attn_prefill(hipStream_t s, const bf16* qkv, int ld, bf16* out, int ldo, const PrefillSeq* seqs,
                        const AttnItem* items, int n_items, int heads, const AttnMerge* merges, int n_merges, const int* block_tables, const bf16* pool,
                        KvGeom geo, int n_q, float* part_ws) {
  if (n_items == 0) return hipSuccess;
  if (heads < 1 || heads > attn_prefill_heads(true, n_q, geo.n_kv, geo.d)) return hipErrorInvalidValue;
  if (geo.page_tokens != 16 || n_q % geo.n_kv != 0 || (n_merges > 0 && (!merges || !part_ws))) return hipErrorInvalidValue;
  const float scale_log2e = 1.4426950408889634f / sqrtf((float)geo.d);
  auto launch = [&](auto d_c) {
    constexpr int D = decltype(d_c)::value;
    auto run = [&](auto* kernel, hipError_t attr, int lds) {
      if (attr == hipSuccess)
        hipLaunchKernelGGL(kernel, dim3((unsigned)n_items * (n_q / heads)), dim3(256), lds, s, qkv, ld, out, ldo, seqs, items, block_tables, pool, geo, n_q, scale_log2e, part_ws);
      return attr;
    };
    hipError_t e;
    if (D == 128 && heads == 2) {
      static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_prefill_pair_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, attn_pair_lds());
      e = run(&attn_prefill_pair_kernel, attr, attn_pair_lds());
    } else {
      static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_prefill_kernel<D>), hipFuncAttributeMaxDynamicSharedMemorySize, attn_prefill_lds<D>());
      e = run(&attn_prefill_kernel<D>, attr, attn_prefill_lds<D>());
    }
    if (e != hipSuccess) return e;
    if (n_merges > 0)
      hipLaunchKernelGGL(attn_prefill_merge_kernel<D>, dim3((unsigned)n_merges * n_q, BQ * D / 1024), dim3(256), 0, s, out, ldo, seqs, merges, n_q, part_ws);
    return hipGetLastError();
  };
  if (geo.d == 128) return launch(std::integral_constant<int, 128>{});
  if (geo.d == 64) return launch(std::integral_constant<int, 64>{});
  return hipErrorInvalidValue;
}

}  // namespace sts
