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
// registers, two barriers a tile and Q read from LDS took 658 us for 8192 rows of 32 heads (0.84 PFLOP/s), this form 539 (1.02); 2048
// rows on 224 CUs 68 -> 54, 301 rows 14.2 -> 10.4. Where a launch has only one workgroup per CU (1024 new tokens over 15 000 cached
// ones: 256) long key ranges are cut into parts (attn_prefill_plan), at the price of fp32 partial outputs.
#include <algorithm>

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

template <int D>
__global__ void __launch_bounds__(256, 2) attn_prefill_kernel(const bf16* __restrict__ qkv, int ld, bf16* __restrict__ out, int ldo,
                                                           const PrefillSeq* __restrict__ seqs, const AttnItem* __restrict__ items,
                                                           const int* __restrict__ block_tables, const bf16* __restrict__ pool,
                                                           KvGeom geo, int n_q, float scale_log2e, float* __restrict__ part_ws) {
  constexpr int KSTEPS = D / 16, DB = D / 32;
  constexpr int ROWB = D * 2, CPR = D / 8, RPI = 64 / CPR, IPP = 16 / RPI;     // K row bytes, 16-byte chunks, rows per load, loads per page
  constexpr int PAGE = 16 * ROWB, TILE = 4 * PAGE, STAGE = 2 * TILE;           // bytes of a K (or V^T) page, tile; of a stage
  extern __shared__ __align__(16) unsigned char smem[];

  const int head = blockIdx.x % n_q;
  const AttnItem it = items[blockIdx.x / n_q];
  const PrefillSeq sq = seqs[it.seq];
  const int kvh = head / (n_q / geo.n_kv);
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, lh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int* bt = block_tables + sq.bt_off;

  const int qloc = it.q0 + wave * 32 + l32;              // row inside the chunk
  const bool q_valid = qloc < sq.sl;
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
  if (it.part >= 0) {
    // one part of the key range: unnormalised output, reference maximum (scaled) and sum of each query row
    float* po = part_ws + ((size_t)it.part * n_q + head) * BQ * (D + 2);
    float* row = po + (size_t)(wave * 32 + l32) * D + 4 * lh;
#pragma unroll
    for (int b = 0; b < DB; b++)
#pragma unroll
      for (int r4 = 0; r4 < 4; r4++) *reinterpret_cast<f32x4*>(row + b * 32 + 8 * r4) = f32x4{o[b][4 * r4], o[b][4 * r4 + 1], o[b][4 * r4 + 2], o[b][4 * r4 + 3]};
    if (lh == 0) *reinterpret_cast<f32x2*>(po + (size_t)BQ * D + (wave * 32 + l32) * 2) = f32x2{m_ref * scale_log2e, l_run};
    return;
  }
  if (!q_valid) return;
  const float inv_l = 1.f / l_run;
  bf16* orow = out + (size_t)(sq.row0 + qloc) * ldo + head * D + 4 * lh;
#pragma unroll
  for (int b = 0; b < DB; b++)
#pragma unroll
    for (int r4 = 0; r4 < 4; r4++) {
      bf16x4 v;
#pragma unroll
      for (int e = 0; e < 4; e++) v[e] = f2bf(o[b][4 * r4 + e] * inv_l);
      *reinterpret_cast<bf16x4*>(orow + b * 32 + 8 * r4) = v;
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
  return plan;
}

// qkv: packed [rows, ld] with Q of head h at columns [h*d, (h+1)*d), already rotated.
// out: [rows, ldo], head h at the same columns. items: query tiles (sequence, first row, key tiles, part or -1);
// one workgroup per (item, head). merges: the query tiles whose key range was cut. part_ws: attn_prefill_part_floats(n_q, d) per part.
// Requires page_tokens == 16 and d in {64, 128}.
hipError_t attn_prefill(hipStream_t s, const bf16* qkv, int ld, bf16* out, int ldo, const PrefillSeq* seqs,
                        const AttnItem* items, int n_items, const AttnMerge* merges, int n_merges, const int* block_tables, const bf16* pool,
                        KvGeom geo, int n_q, float* part_ws) {
  if (n_items == 0) return hipSuccess;
  if (geo.page_tokens != 16 || n_q % geo.n_kv != 0 || (n_merges > 0 && (!merges || !part_ws))) return hipErrorInvalidValue;
  const float scale_log2e = 1.4426950408889634f / sqrtf((float)geo.d);
  auto launch = [&](auto d_c) {
    constexpr int D = decltype(d_c)::value;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_prefill_kernel<D>), hipFuncAttributeMaxDynamicSharedMemorySize, attn_prefill_lds<D>());
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(attn_prefill_kernel<D>, dim3((unsigned)n_items * n_q), dim3(256), attn_prefill_lds<D>(), s, qkv, ld, out, ldo, seqs, items, block_tables, pool, geo, n_q, scale_log2e, part_ws);
    if (n_merges > 0)
      hipLaunchKernelGGL(attn_prefill_merge_kernel<D>, dim3((unsigned)n_merges * n_q, BQ * D / 1024), dim3(256), 0, s, out, ldo, seqs, merges, n_q, part_ws);
    return hipGetLastError();
  };
  if (geo.d == 128) return launch(std::integral_constant<int, 128>{});
  if (geo.d == 64) return launch(std::integral_constant<int, 64>{});
  return hipErrorInvalidValue;
}

}  // namespace sts
