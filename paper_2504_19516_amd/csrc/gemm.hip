// bf16 MFMA GEMM for gfx950:  C[M,N] (+)= A[M,K] * W[N,K]^T, fp32 accumulation.
//
// Both operands are K-contiguous, which is the layout v_mfma_f32_32x32x16_bf16 wants: a lane
// holds 8 consecutive k of one A row (or one W row). A workgroup owns a BM x BN tile and each of
// its waves accumulates a (BM/WGM) x (BN/WGN) sub-tile in 32x32 MFMA blocks.
//
// Main loops. gemm_rows_kernel: the prefill tiles of 256 columns and any multiple of 32 rows up to 256 (4 waves); only
// the activation tile goes through LDS, the W operands go from the packed weight layout straight into registers.
// gemm_dl_kernel: K tiles of 64 of both operands go global -> LDS directly (no
// staging registers, no LDS store instructions): activations into 128-byte rows whose 16-byte chunks
// are XOR-swizzled so that the 16-byte operand reads are bank-conflict free, packed weights as the
// operand-order blocks they are in memory; two or three LDS stages;
// operand reads of the next 16-wide step are slotted between the MFMAs of the current one. It runs
// the 128x128 tiles with 4 waves (two workgroups per CU) for prefill, the 64x128 (4 waves, two per
// CU) and 64x256 (8 waves) tiles with split-K for decode batches, and row-major W of callers that
// bring their own weights.
// gemm_skinny_kernel: decode batches of up to 64 rows -- tiles of 256 to 512 columns, the W operands three K tiles deep in
// registers.
// Epilogues: bf16 store, fp32 store (split-K partial sums), fp32 residual add, SwiGLU on interleaved
// gate/up rows.
//
// Wave quantisation (paper Section 2.2.1) is met in the launch: the tiles of a partly filled last
// wave of workgroups are cut along K into pieces that fill the partition (gemm_tail_plan), the
// pieces leave fp32 partial tiles, and gemm_tail_fixup sums them in a fixed order and applies the
// epilogue.
//
// Lane layout of the 32x32 accumulator block (register r of lane l):
//   row = 8*(r/4) + 4*(l/32) + r%4,  col = l%32.
// gemm_rows_kernel uses the 16x16 block with W as the first operand: register r of lane l is column 4*(l/16) + r, row l%16.
#include <atomic>
#include <type_traits>
#include <utility>

#include "kernels.h"

namespace sts {

constexpr int GEMM_DL_LDS_BASE = 1024;   // the direct-to-LDS arena stays clear of LDS address 0
#ifndef GEMM_SKINNY_PD
#define GEMM_SKINNY_PD 3                 // K tiles of W operands a wave of gemm_skinny_kernel keeps in flight
#endif

struct GemmArgs {
  const bf16* A; const bf16* W; void* C;
  int lda, ldw, ldc;
  int M, N, K;
  int w_packed;               // W in the packed block layout (weight_packed_index) instead of row-major
  int stream_nt;              // skinny tiles: fetch W with the non-temporal hint
  int tiles_m, tiles_n, group_m;
  int k_per_split;            // K range handled by one blockIdx.y
  long long split_stride;     // elements between consecutive split-K partial outputs
  // Tail splitting. Tiles [0, n_full) are computed whole. The remaining tiles -- the last,
  // partly filled wave of workgroups on the partition -- are cut along K into tail_f pieces each,
  // so that wave takes 1/tail_f of a tile time; pieces leave fp32 partial tiles in tail_ws and a
  // second small kernel adds them up in a fixed order and applies the epilogue.
  int n_full, full_per_xcd, tail_f, n_pieces, piece_per_xcd;
  int piece_stride;           // floats between consecutive partial tiles
  float* tail_ws;
  int row_blocks;             // gemm_rows_kernel: 32-row blocks of M, dealt evenly to tiles_m row tiles, or (tile_blocks > 0)
  int tile_blocks;            // tile_blocks to each and the rest to the last
  QkvOut qkv;                 // EPI_QKV
};

// tile index -> tile coordinates: tiles are walked in groups of group_m tile rows so that
// workgroups resident together share operand rows in L2
__device__ __forceinline__ void tile_coords(const GemmArgs& g, int v, int* tm, int* tn) {
  const int gsz = g.group_m * g.tiles_n;
  const int first_m = (v / gsz) * g.group_m;
  const int gm = min(g.tiles_m - first_m, g.group_m);
  *tm = first_m + (v % gsz) % gm;
  *tn = (v % gsz) / gm;
}

// Workgroups are dealt round-robin to the 8 XCDs, in order: each XCD first gets a contiguous
// run of whole tiles (neighbours share operands in its L2), then its share of the tail pieces.
// Returns false for a padding workgroup. piece < 0 for a whole tile.
template <int BK>
__device__ __forceinline__ bool block_work(const GemmArgs& g, int* v, int* kbeg, int* kend, int* piece) {
  const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3;
  *piece = -1;
  if (local < g.full_per_xcd) {
    *v = xcd * g.full_per_xcd + local;
    if (*v >= g.n_full) return false;
    *kbeg = blockIdx.y * g.k_per_split;
    *kend = min(g.K, *kbeg + g.k_per_split);
  } else {
    *piece = xcd * g.piece_per_xcd + (local - g.full_per_xcd);
    if (*piece >= g.n_pieces) return false;
    *v = g.n_full + *piece / g.tail_f;
    const int z = *piece % g.tail_f, ksteps = g.K / BK;
    *kbeg = (int)((long long)ksteps * z / g.tail_f) * BK;
    *kend = (int)((long long)ksteps * (z + 1) / g.tail_f) * BK;
  }
  return true;
}

// Epilogue of one workgroup tile (or the partial-tile store of a tail piece).
template <int BM, int BN, int WGM, int WGN, int EPI>
__device__ __forceinline__ void store_tile(const GemmArgs& g, f32x16 (&acc)[BM / WGM / 32][BN / WGN / 32], int m0, int n0, int piece,
                                           int wm, int wn, int l32, int lh) {
  constexpr int WTM = BM / WGM, WTN = BN / WGN, TM = WTM / 32, TN = WTN / 32;
  // a tail piece stores its partial tile, row-major [BM][BN]
  if (piece >= 0) {
    float* part = g.tail_ws + (size_t)piece * (BM * BN) + (size_t)(wm * WTM + 4 * lh) * BN + wn * WTN + l32;
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int r = 0; r < 16; r++)
#pragma unroll
        for (int j = 0; j < TN; j++) part[(size_t)(i * 32 + 8 * (r >> 2) + (r & 3)) * BN + j * 32] = acc[i][j][r];
    return;
  }

  // ---- epilogue
  const int rbase = m0 + wm * WTM + 4 * lh;
  const int cbase = n0 + wn * WTN + l32;
#pragma unroll
  for (int i = 0; i < TM; i++) {
#pragma unroll
    for (int r = 0; r < 16; r++) {
      const int row = rbase + i * 32 + 8 * (r >> 2) + (r & 3);
      if (row >= g.M) continue;
      if constexpr (EPI == EPI_SWIGLU_BF16) {
        bf16* out = reinterpret_cast<bf16*>(g.C) + (size_t)row * g.ldc + ((n0 + wn * WTN) >> 1) + l32;
#pragma unroll
        for (int j = 0; j < TN; j += 2) {
          const float gate = acc[i][j][r], up = acc[i][j + 1][r];
          out[(j >> 1) * 32] = f2bf(swiglu(gate, up));
        }
      } else {
#pragma unroll
        for (int j = 0; j < TN; j++) {
          const size_t idx = (size_t)row * g.ldc + cbase + j * 32;
          if constexpr (EPI == EPI_BF16) reinterpret_cast<bf16*>(g.C)[idx] = f2bf(acc[i][j][r]);
          else if constexpr (EPI == EPI_F32)
            reinterpret_cast<float*>(g.C)[(size_t)blockIdx.y * g.split_stride + idx] = acc[i][j][r];
          else reinterpret_cast<float*>(g.C)[idx] += acc[i][j][r];
        }
      }
    }
  }
}

// ---- direct-to-LDS main loop ---------------------------------------------------------------
// Tiles go global -> LDS without passing through registers (no staging VGPRs, no LDS store
// instructions). A tile row is 128 bytes (BK = 64) and unpadded; the 16-byte K-chunk c of row r
// is stored at slot c ^ ((r >> 1) & 7), which keeps the 16-byte operand reads bank-conflict
// free. One wave instruction fills 64 consecutive slots (8 rows), so the swizzle is applied on
// the global side: each lane fetches the chunk that belongs in its slot.
//
// Schedule of one K tile (four 16-wide steps): steps 0-2 run from the current LDS buffer; then
// the wave waits for its own loads of the next tile and meets the others at the barrier, which
// both publishes the next tile and retires the current buffer (the operands of step 3 are
// already in registers); the loads of the tile after next go out right behind the barrier, a
// whole iteration ahead of their use; step 3 runs while the first operands of the next tile
// are read. The LDS arena starts 1 KB above address 0.
template <int BM, int BN, int WGM, int WGN, int EPI, int NS, bool WPACK = true>
__global__ void __launch_bounds__(WGM* WGN * 64) gemm_dl_kernel(GemmArgs g) {
  constexpr int BK = 64, NT = WGM * WGN * 64;
  static_assert(NS >= 2 && (NS - 2) * (BM + BN) * 8 / NT < 64, "stages: at least two, outstanding loads within vmcnt's range");
  constexpr int WTM = BM / WGM, WTN = BN / WGN, TM = WTM / 32, TN = WTN / 32;
  constexpr int ROWB = BK * 2;                               // bytes per tile row
  constexpr int A_CH = BM * 8 / NT, B_CH = BN * 8 / NT;      // 16-byte chunks per thread
  constexpr int STAGE = (BM + BN) * ROWB;
  static_assert(BM * 8 % NT == 0 && BN * 8 % NT == 0, "tile/thread mismatch");
  static_assert(EPI != EPI_SWIGLU_BF16 || TN % 2 == 0, "swiglu needs gate/up block pairs");
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* arena = smem + GEMM_DL_LDS_BASE;

  int v, kbeg, kend, piece;
  if (!block_work<BK>(g, &v, &kbeg, &kend, &piece)) return;
  int tm, tn;
  tile_coords(g, v, &tm, &tn);
  const int m0 = tm * BM, n0 = tn * BN;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, lh = lane >> 5;
  const int wm = wave / WGN, wn = wave % WGN;

  // slot q = j * NT + tid of a tile: row q / 8, holds K-chunk (q % 8) ^ ((row >> 1) & 7). A lane keeps
  // the 32-bit byte offset of its chunk from the tile's first row; the tile bases are wave-uniform
  // and advance along K in scalar registers, and so do the LDS destinations (the wave index is read
  // into a scalar once): queuing a load takes no vector ALU work and sends 4 address bytes per lane.
  const int swave = __builtin_amdgcn_readfirstlane(wave);
  const unsigned char* a_base = reinterpret_cast<const unsigned char*>(g.A + (size_t)m0 * g.lda);
  // W: row-major (its tile is laid out in LDS like the A tile), or (WPACK) 32 x 64 blocks of 4 KiB in matrix-core operand
  // order (weight_packed_index), copied to LDS as they are.
  const unsigned char* b_base = WPACK ? reinterpret_cast<const unsigned char*>(g.W) + (size_t)(n0 >> 5) * (g.K >> 6) * 4096
                                      : reinterpret_cast<const unsigned char*>(g.W + (size_t)n0 * g.ldw);
  unsigned a_off[A_CH], b_off[B_CH];
#pragma unroll
  for (int j = 0; j < A_CH; j++) {
    const int q = j * NT + tid, row = q >> 3, ch = (q & 7) ^ ((row >> 1) & 7);
    a_off[j] = (unsigned)(min(m0 + row, g.M - 1) - m0) * (unsigned)g.lda * 2u + ch * 16;
  }
#pragma unroll
  for (int j = 0; j < B_CH; j++) {
    const int q = j * NT + tid, row = q >> 3, ch = (q & 7) ^ ((row >> 1) & 7);
    // packed: slot q is the q-th 16-byte piece of the tile's 4 KiB blocks for this K step, so a wave's load reads 1 KiB of
    // consecutive memory
    b_off[j] = WPACK ? (unsigned)(q >> 8) * (unsigned)(g.K >> 6) * 4096u + (unsigned)(q & 255) * 16u
                     : (unsigned)row * (unsigned)g.ldw * 2u + ch * 16;
  }
  auto issue_a = [&](int stage, int k) {
    unsigned char* sa = arena + stage * STAGE + swave * 1024;
    const unsigned char* ak = a_base + (size_t)k * 2;
#pragma unroll
    for (int j = 0; j < A_CH; j++) lds_dma16(ak, a_off[j], sa + j * NT * 16);
  };
  auto issue_b = [&](int stage, int k) {
    unsigned char* sb = arena + stage * STAGE + swave * 1024 + BM * ROWB;
    const unsigned char* bk = b_base + (WPACK ? (size_t)(k >> 6) * 4096 : (size_t)k * 2);
#pragma unroll
    for (int j = 0; j < B_CH; j++) lds_dma16(bk, b_off[j], sb + j * NT * 16);
  };
  auto issue = [&](int stage, int k) { issue_a(stage, k); issue_b(stage, k); };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[i][j][r] = 0.f;

  // byte offset of this lane's operand chunk inside its row, for each of the four K steps
  // and of its W operand: the same for a row-major W tile; a packed W tile is in LDS what it is in memory, 1 KiB per
  // 32-row block and step with lane l's operand at byte 16 l
  int koff[4], kboff[4];
#pragma unroll
  for (int kk = 0; kk < 4; kk++) {
    koff[kk] = ((kk * 2 + lh) ^ ((l32 >> 1) & 7)) * 16;
    kboff[kk] = WPACK ? kk * 1024 : koff[kk];
  }
  const int a_row = (wm * WTM + l32) * ROWB;
  const int b_row = BM * ROWB + (WPACK ? wn * WTN * ROWB + lane * 16 : (wn * WTN + l32) * ROWB);

  constexpr int MPR = (TM * TN) / (TM + TN) > 0 ? (TM * TN) / (TM + TN) : 1;       // MFMAs per LDS read
  constexpr int REST = TM * TN > MPR * (TM + TN) ? TM * TN - MPR * (TM + TN) : 0;

  // NS LDS stages: tile t lives in stage t % NS; while tile t is consumed, tiles t+1 .. t+NS-1
  // are landing or on their way.
  constexpr int LOADS = A_CH + B_CH;                         // loads per thread and tile
  const int nk = (kend - kbeg) / BK;
#pragma unroll
  for (int t = 0; t < NS; t++)
    if (t < nk) issue(t, kbeg + t * BK);
  if (nk >= NS) wait_vmem<(NS - 1) * LOADS>(); else wait_vmem<0>();
  __syncthreads();
  bf16x8 af[2][TM], bfr[2][TN];
#pragma unroll
  for (int i = 0; i < TM; i++) af[0][i] = *reinterpret_cast<const bf16x8*>(arena + a_row + i * 32 * ROWB + koff[0]);
#pragma unroll
  for (int j = 0; j < TN; j++) bfr[0][j] = *reinterpret_cast<const bf16x8*>(arena + b_row + j * 32 * ROWB + kboff[0]);

  int cur = 0;                                               // stage of tile t
  for (int t = 0; t < nk; t++) {
    const int nxt = cur + 1 == NS ? 0 : cur + 1;
    const unsigned char* Ac = arena + cur * STAGE + a_row;
    const unsigned char* Bc = arena + cur * STAGE + b_row;
    const unsigned char* An = arena + nxt * STAGE + a_row;
    const unsigned char* Bn = arena + nxt * STAGE + b_row;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kk = 0; kk < 3; kk++) {
#pragma unroll
      for (int i = 0; i < TM; i++) af[(kk + 1) & 1][i] = *reinterpret_cast<const bf16x8*>(Ac + i * 32 * ROWB + koff[kk + 1]);
#pragma unroll
      for (int j = 0; j < TN; j++) bfr[(kk + 1) & 1][j] = *reinterpret_cast<const bf16x8*>(Bc + j * 32 * ROWB + kboff[kk + 1]);
#pragma unroll
      for (int i = 0; i < TM; i++)
#pragma unroll
        for (int j = 0; j < TN; j++)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[kk & 1][i], bfr[kk & 1][j], acc[i][j], 0, 0, 0);
    }
#pragma unroll
    for (int kk = 0; kk < 3; kk++) {
#pragma unroll
      for (int x = 0; x < TM + TN; x++) {
        __builtin_amdgcn_sched_group_barrier(0x008, MPR, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      if (REST > 0) __builtin_amdgcn_sched_group_barrier(0x008, REST, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    // tile t+1 must have landed; the NS-2 tiles issued after it may still be in flight
    if (t + NS - 1 < nk) wait_vmem<(NS - 2) * LOADS>(); else wait_vmem<0>();
    __syncthreads();
    // the tile after the ones in flight goes into the stage just retired
    if (t + NS < nk) issue(cur, kbeg + (t + NS) * BK);
    __builtin_amdgcn_sched_barrier(0);
    if (t + 1 < nk) {
#pragma unroll
      for (int i = 0; i < TM; i++) af[0][i] = *reinterpret_cast<const bf16x8*>(An + i * 32 * ROWB + koff[0]);
#pragma unroll
      for (int j = 0; j < TN; j++) bfr[0][j] = *reinterpret_cast<const bf16x8*>(Bn + j * 32 * ROWB + kboff[0]);
    }
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[1][i], bfr[1][j], acc[i][j], 0, 0, 0);
#pragma unroll
    for (int x = 0; x < TM + TN; x++) {
      __builtin_amdgcn_sched_group_barrier(0x008, MPR, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    if (REST > 0) __builtin_amdgcn_sched_group_barrier(0x008, REST, 0);
    __builtin_amdgcn_sched_barrier(0);
    cur = nxt;
  }
  store_tile<BM, BN, WGM, WGN, EPI>(g, acc, m0, n0, piece, wm, wn, l32, lh);
}

// ---- W operands straight from global memory into registers ------------------------------------------
// The loads are written in assembly, so the compiler does not know when their registers are valid; the wait names them as
// in/out operands, which keeps every use behind it.
template <bool NT = false>
__device__ __forceinline__ void load_w16(bf16x8& dst, const unsigned char* base, unsigned lane_off, int step) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (NT) {   // the same loads with the non-temporal hint
    switch (step) {
      case 0: asm volatile("global_load_dwordx4 %0, %1, %2 nt" : "=v"(dst) : "v"(lane_off), "s"(base) : "memory"); break;
      case 1: asm volatile("global_load_dwordx4 %0, %1, %2 offset:1024 nt" : "=v"(dst) : "v"(lane_off), "s"(base) : "memory"); break;
      case 2: asm volatile("global_load_dwordx4 %0, %1, %2 offset:2048 nt" : "=v"(dst) : "v"(lane_off), "s"(base) : "memory"); break;
      default: asm volatile("global_load_dwordx4 %0, %1, %2 offset:3072 nt" : "=v"(dst) : "v"(lane_off), "s"(base) : "memory"); break;
    }
    return;
  }
  switch (step) {   // the step's 1 KiB piece is addressed by the instruction's immediate offset
    case 0: asm volatile("global_load_dwordx4 %0, %1, %2" : "=v"(dst) : "v"(lane_off), "s"(base) : "memory"); break;
    case 1: asm volatile("global_load_dwordx4 %0, %1, %2 offset:1024" : "=v"(dst) : "v"(lane_off), "s"(base) : "memory"); break;
    case 2: asm volatile("global_load_dwordx4 %0, %1, %2 offset:2048" : "=v"(dst) : "v"(lane_off), "s"(base) : "memory"); break;
    default: asm volatile("global_load_dwordx4 %0, %1, %2 offset:3072" : "=v"(dst) : "v"(lane_off), "s"(base) : "memory"); break;
  }
#endif
}
// Wait until at most N vector-memory operations of this wave are outstanding; a and b are valid afterwards.
template <int N>
__device__ __forceinline__ void wait_vmem_for(bf16x8& a, bf16x8& b) {
#if defined(__HIP_DEVICE_COMPILE__)
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
  asm volatile("s_waitcnt vmcnt(%2)" : "+v"(a), "+v"(b) : "n"(N) : "memory");
#endif
}

// ---- decode batches (up to 64 rows per tile): weights streamed through registers, several K tiles deep ----
// A decode GEMM reads every weight byte once and runs at the rate at which its CUs pull bytes from memory; what
// a workgroup reads beside its weights -- the 64 activation rows of its K range, again for every workgroup --
// comes out of that rate. A workgroup here is 4 to 8 waves (the launch's block size; a tile is 64 columns per
// wave wide), so that a width can be chosen that divides N into whole rounds of workgroups on the partition
// while the activation tile is shared by as many waves as possible. A wave reads the W operands of its 64
// columns (two 32-row blocks of the packed layout) straight into registers and keeps PD K tiles of them -- 8 PD
// loads of 1 KiB -- under way. Only the activation tile passes through LDS (PD + 2 stages of 8 KB, fetched by
// the first four waves as in the loops above).
//
// Order of a wave's vector-memory operations (they complete in order): iteration t queues the A loads of
// tile t + PD + 1 (2), then after each step kk the two W loads of (tile t + PD, step kk) into the registers
// that step just used; the prologue queues A(0) and then, for s < PD, A(s + 1) and W(s) in the same order.
// When step kk of tile t waits for its operands, 10 PD - 2 operations were queued after them (the W loads
// of the later steps of tile t: 6 - 2 kk; A and W of the PD - 1 tiles between: 10 each; this iteration's A
// loads: 2; its W loads so far: 2 kk), in every iteration: the last ones re-read the last K tile into
// registers and stages nobody uses. A(t + 1) was queued before the operands step 3 of tile t waits for, so
// it has landed at the barrier there, which also retires the stage of tile t for the A loads of iteration
// t + 1.
template <int EPI, int PD, bool NT>
__global__ void __launch_bounds__(512, 2) gemm_skinny_kernel(GemmArgs g) {
  constexpr int BM = 64, BK = 64, NS = PD + 2, DUTY = 4;     // DUTY waves load the A tile
  constexpr int TM = 2, TN = 2, ROWB = BK * 2, A_CH = BM * 8 / (DUTY * 64), STAGE = BM * ROWB;
  constexpr int WAIT = 10 * PD - 2;
  static_assert(A_CH == 2 && WAIT < 64, "the waits count 2 A loads per tile and 2 W loads per step, within vmcnt's range");
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* arena = smem + GEMM_DL_LDS_BASE;

  int v, kbeg, kend, piece;
  if (!block_work<BK>(g, &v, &kbeg, &kend, &piece)) return;
  int tm, tn;
  tile_coords(g, v, &tm, &tn);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, lh = lane >> 5;
  const int swave = __builtin_amdgcn_readfirstlane(wave);
  const int wn = swave;
  const int m0 = tm * BM, n0 = tn * (int)(blockDim.x >> 6) * 64;     // a tile is 64 columns per wave wide

  const unsigned char* a_base = reinterpret_cast<const unsigned char*>(g.A + (size_t)m0 * g.lda);
  // The first DUTY waves fetch the A tile. The others queue as many 16-byte loads of the tile's first bytes into a
  // spare KB behind the stages, so that every wave's queue has the same shape and the waits below count alike.
  const bool duty = swave < DUTY;
  unsigned a_off[A_CH];
#pragma unroll
  for (int j = 0; j < A_CH; j++) {
    const int q = j * (DUTY * 64) + (tid & (DUTY * 64 - 1)), row = q >> 3, ch = (q & 7) ^ ((row >> 1) & 7);
    a_off[j] = duty ? (unsigned)(min(m0 + row, g.M - 1) - m0) * (unsigned)g.lda * 2u + ch * 16 : 0u;
  }
  auto issue_a = [&](int stage, int k) {
    unsigned char* sa = duty ? arena + stage * STAGE + swave * 1024 : arena + NS * STAGE;
    const unsigned char* ak = a_base + (size_t)k * 2;
#pragma unroll
    for (int j = 0; j < A_CH; j++) lds_dma16(ak, a_off[j], duty ? sa + j * (DUTY * 64) * 16 : sa);
  };
  const size_t wrow = (size_t)(g.K >> 6) * 4096;
  const unsigned char* w_base = reinterpret_cast<const unsigned char*>(g.W) + (size_t)((n0 >> 5) + wn * TN) * wrow;
  const unsigned w_lane = (unsigned)lane * 16u;
  bf16x8 w[PD][TN][4];
#pragma unroll
  for (int s = 0; s < PD; s++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int kk = 0; kk < 4; kk++)
#pragma unroll
        for (int e = 0; e < 8; e++) w[s][j][kk][e] = 0;

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int r = 0; r < 16; r++) acc[i][j][r] = 0.f;

  int koff[4];
#pragma unroll
  for (int kk = 0; kk < 4; kk++) koff[kk] = ((kk * 2 + lh) ^ ((l32 >> 1) & 7)) * 16;
  const int a_row = l32 * ROWB;

  const int nk = (kend - kbeg) / BK;
  auto tile_k = [&](int t) { return kbeg + min(t, nk - 1) * BK; };
  issue_a(0, tile_k(0));
#pragma unroll
  for (int s = 0; s < PD; s++) {
    issue_a(s + 1, tile_k(s + 1));
    const unsigned char* wk = w_base + (size_t)(tile_k(s) >> 6) * 4096;
#pragma unroll
    for (int kk = 0; kk < 4; kk++)
#pragma unroll
      for (int j = 0; j < TN; j++) load_w16<NT>(w[s][j][kk], wk + j * wrow, w_lane, kk);
  }
  wait_vmem<10 * PD>();                                      // A(0) has landed
  __syncthreads();
  bf16x8 af[2][TM];
#pragma unroll
  for (int i = 0; i < TM; i++) af[0][i] = *reinterpret_cast<const bf16x8*>(arena + a_row + i * 32 * ROWB + koff[0]);

  int cur = 0;                                               // stage of tile t
  int ahead = PD + 1;                                        // stage of tile t + PD + 1
  for (int t0 = 0; t0 < nk; t0 += PD) {
    auto tile = [&](auto s_c) {
      constexpr int s = decltype(s_c)::value;                // register set of tile t: t % PD
      const int t = t0 + s;
      const bool live = t < nk;                              // the surplus tiles of the last round only keep the queue's shape
      const int nxt = cur + 1 == NS ? 0 : cur + 1;
      const unsigned char* Ac = arena + cur * STAGE + a_row;
      const unsigned char* An = arena + nxt * STAGE + a_row;
      const unsigned char* wk = w_base + (size_t)(tile_k(t + PD) >> 6) * 4096;
      __builtin_amdgcn_sched_barrier(0);
      issue_a(ahead, tile_k(t + PD + 1));
      auto step = [&](auto kk_c) {
        constexpr int kk = decltype(kk_c)::value;
        __builtin_amdgcn_sched_barrier(0);
        wait_vmem_for<WAIT>(w[s][0][kk], w[s][1][kk]);
        if constexpr (kk == 3) {
          __syncthreads();
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int i = 0; i < TM; i++) af[0][i] = *reinterpret_cast<const bf16x8*>(An + i * 32 * ROWB + koff[0]);
        } else {
#pragma unroll
          for (int i = 0; i < TM; i++) af[(kk + 1) & 1][i] = *reinterpret_cast<const bf16x8*>(Ac + i * 32 * ROWB + koff[kk + 1]);
        }
        if (live) {
#pragma unroll
          for (int i = 0; i < TM; i++)
#pragma unroll
            for (int j = 0; j < TN; j++)
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[kk & 1][i], w[s][j][kk], acc[i][j], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < TN; j++) load_w16<NT>(w[s][j][kk], wk + j * wrow, w_lane, kk);
      };
      step(std::integral_constant<int, 0>{});
      step(std::integral_constant<int, 1>{});
      step(std::integral_constant<int, 2>{});
      step(std::integral_constant<int, 3>{});
      cur = nxt;
      ahead = ahead + 1 == NS ? 0 : ahead + 1;
    };
    tile(std::integral_constant<int, 0>{});
    if constexpr (PD > 1) tile(std::integral_constant<int, 1>{});
    if constexpr (PD > 2) tile(std::integral_constant<int, 2>{});
    if constexpr (PD > 3) tile(std::integral_constant<int, 3>{});
    if constexpr (PD > 4) tile(std::integral_constant<int, 4>{});
    if constexpr (PD > 5) tile(std::integral_constant<int, 5>{});
  }
  // the surplus loads of the last iterations must not land in registers the epilogue reuses
#pragma unroll
  for (int s = 0; s < PD; s++)
#pragma unroll
    for (int kk = 0; kk < 4; kk++) wait_vmem_for<0>(w[s][0][kk], w[s][1][kk]);
  // a wave's 64 x 64 block: the tile store of a four-wave row, placed by the wave's index
  store_tile<BM, 256, 1, 4, EPI>(g, acc, m0, n0, piece, 0, wn, l32, lh);
}

// Four consecutive columns c .. c + 3 of a tail tile's row: its pieces (stride floats apart, p in the first) added in piece order,
// then the epilogue. n0: the tile's first column.
template <int EPI>
__device__ __forceinline__ void store_fixed_up(const GemmArgs& g, const float* p, int stride, int row, int n0, int c) {
  f32x4 sum = *reinterpret_cast<const f32x4*>(p), up = {0.f, 0.f, 0.f, 0.f};
  if (EPI == EPI_SWIGLU_BF16) up = *reinterpret_cast<const f32x4*>(p + 32);
  for (int z = 1; z < g.tail_f; z++) {
    sum += *reinterpret_cast<const f32x4*>(p + (size_t)z * stride);
    if (EPI == EPI_SWIGLU_BF16) up += *reinterpret_cast<const f32x4*>(p + (size_t)z * stride + 32);
  }
  const int col = n0 + c;
  if constexpr (EPI == EPI_SWIGLU_BF16) {
    bf16x4 o;
#pragma unroll
    for (int i = 0; i < 4; i++) o[i] = f2bf(swiglu(sum[i], up[i]));
    const int ocol = ((n0 + (c & ~63)) >> 1) + (c & 31);
    *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16*>(g.C) + (size_t)row * g.ldc + ocol) = o;
  } else if constexpr (EPI == EPI_BF16) {
    bf16x4 o;
#pragma unroll
    for (int i = 0; i < 4; i++) o[i] = f2bf(sum[i]);
    *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16*>(g.C) + (size_t)row * g.ldc + col) = o;
  } else {
    f32x4* dst = reinterpret_cast<f32x4*>(reinterpret_cast<float*>(g.C) + (size_t)row * g.ldc + col);
    if constexpr (EPI == EPI_RESID_F32) *dst += sum;
    else *dst = sum;
  }
}

// Adds the tail pieces of each split tile in piece order and applies the epilogue. One thread per
// four consecutive columns.
template <int BM, int BN, int EPI>
__global__ void __launch_bounds__(256) gemm_tail_fixup(GemmArgs g) {
  const int t = blockIdx.x;                                   // tail tile
  const int e = blockIdx.y * 256 + threadIdx.x;
  const int r = e / (BN / 4), c = (e % (BN / 4)) * 4;
  int tm, tn;
  tile_coords(g, g.n_full + t, &tm, &tn);
  const int row = tm * BM + r;
  if (row >= g.M) return;
  if (EPI == EPI_SWIGLU_BF16 && ((c >> 5) & 1)) return;      // "up" columns are consumed by their gate thread
  store_fixed_up<EPI>(g, g.tail_ws + (size_t)t * g.tail_f * (BM * BN) + (size_t)r * BN + c, BM * BN, row, tn * BN, c);
}

// ---- the 256-column prefill tiles: row tiles of any multiple of 32 rows up to 256 -----------------------------------
// A launch's rows are cut into `tiles_m` row tiles of nearly equal height in blocks of 32 (row_range), and a workgroup runs
// the loop compiled for its height: nothing is computed for padding beyond the last block, and the number of row tiles is
// free to make whole waves of workgroups (Section 2.2.1): 2048 x 4096 outputs on 224 CUs are 14 x 16 tiles of at most 160 rows,
// one per CU, where 256-row tiles leave 96 CUs idle or cut along K. T = 301 rows run as two tiles of 160.
//
// Four waves, one per SIMD, each all rows x 64 columns in 16 x 16 matrix-core blocks. Only the activation tile goes through LDS
// (four stages, read by every wave); a wave reads its own columns' W operands from the packed layout straight into registers, two
// K tiles ahead, so no W byte is loaded twice. A wave has the SIMD's 512 registers: 256 of sums, 64 of W operands, 32 of row blocks.
//
// What bounds it: nothing stands in for a wave that waits, so everything but the matrix instructions has to fit into
// their shadow. They take 16 cycles each and 4 to issue, so one other instruction fits behind each, not a run of them: a K tile is
// dealt out in units of one row block (four matrix instructions) with that unit's LDS read, at most one vector-memory
// operation and the pointer arithmetic each between two of them (RowsPlan). 256 rows: 2160 to 2220 cycles per K tile of 2048 matrix-core
// cycles; with the reads and loads of four row blocks in a run 2670, with eight waves of 32 columns, whose LDS reads are
// twice as many, 68 % busy. The clock falls as the matrix cores get busier (1.7 GHz at 256 rows on a full GPU: power), so the rate gains
// less than the cycles. Against eight waves, 256 CUs: 8192 x 28672 x 4096 1424 -> 1263 us (1.52 PFLOP/s), 8192 x 4096 x 14336 756 -> 657, 3980 x 28672 x
// 4096 730 -> 638, 700 x 57344 x 8192 588 -> 513; two row tiles of 28672 x 4096 at heights 32 / 96 / 128 / 160 / 192 / 256, launched over and over with the
// weights in the memory-side cache: 36 / 48 / 59 / 74 / 84 / 109 us before, 36 / 43 / 49 / 63 / 73 / 93 now. Inside a layer, weights from HBM, 51 / 69 / 73 / 79 /
// 84 / 95: up to about 160 rows such a launch waits for its weights, and 301 rows gained 1 us of 79. The W block is the first operand, so a lane holds four consecutive output columns: fp32
// results leave in 16-byte pieces. The 32 x 32 x 16 instruction gives the same bits but moves twice the accumulator registers per
// product, which costs clock.
//
// Order of a wave's vector-memory operations (they complete in order): the first half of tile t queues the step-1 W operands of
// tile t + 1 and the first pieces of the A tile t + 2, the second half the step-0 W operands of tile t + 2 and the other pieces, in
// every iteration (the last ones re-read the last K tile into stages and registers nobody uses). RowsPlan counts
// what was queued behind the operands a step waits for (WAIT0, WAIT1), and behind the A pieces of tile t + 1 at the barrier that publishes
// them (WAITB). Pieces go into the stage that tile t - 2 left: its operands were multiplied, hence read, before the last barrier.
// A number of K tiles that SETS does not divide starts with null tiles (zero operands add nothing), so that the loop has one exit.
constexpr int ROWS_LDS = 136 * 1024;              // A stages of a gemm_rows_kernel workgroup (or its output image)
__device__ __forceinline__ void row_range(const GemmArgs& g, int tm, int* row0, int* blocks) {
  const int b0 = g.tile_blocks ? tm * g.tile_blocks : (int)((long long)tm * g.row_blocks / g.tiles_m);
  const int b1 = g.tile_blocks ? min(b0 + g.tile_blocks, g.row_blocks) : (int)((long long)(tm + 1) * g.row_blocks / g.tiles_m);
  *row0 = b0 * 32; *blocks = b1 - b0;
}

// One product of the 256-column tiles. Written in assembly so that the sum stays where it is: left to itself the compiler gives
// the result a register quad of its own and copies 256 accumulators per K tile. AG: the sum lives in an accumulation register.
template <bool AG>
__device__ __forceinline__ void mma16(f32x4& c, const bf16x8& a, const bf16x8& b) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (AG) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
  else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
#endif
}
// The compiler does not know that mma16 takes time: before the sums are read otherwise, wait, then tie every one of them to that point.
__device__ __forceinline__ void mma16_settle() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_nop 15\n\ts_nop 7" ::: "memory");
#endif
}
template <bool AG>
__device__ __forceinline__ void mma16_settled(f32x4& c) {
#if defined(__HIP_DEVICE_COMPILE__)
  if constexpr (AG) asm volatile("" : "+a"(c)); else asm volatile("" : "+v"(c));
#endif
}
// Wait until at most N vector-memory operations of this wave are outstanding; the four operands are valid afterwards.
template <int N>
__device__ __forceinline__ void wait_vmem_for4(bf16x8 (&w)[4]) {
#if defined(__HIP_DEVICE_COMPILE__)
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
  asm volatile("s_waitcnt vmcnt(%4)" : "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3]) : "n"(N) : "memory");
#endif
}
template <int OFF>
__device__ __forceinline__ void load_w_off(bf16x8& dst, const unsigned char* base, unsigned lane_off) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("global_load_dwordx4 %0, %1, %2 offset:%3" : "=v"(dst) : "v"(lane_off), "s"(base), "n"(OFF) : "memory");
#endif
}
// A K tile of one wave: U units of one 16-row block each. A half of the units is one 32-wide step; its vector-memory operations -- four W
// loads and its share of the A pieces, alternating -- are dealt over its units.
template <int TM>
struct RowsPlan {
  static constexpr int SETS = 2;                                          // K tiles of W operands in registers
  static constexpr int AGPR_BLOCKS = 13;                                  // of 16; the rest leaves the register allocator room
  static constexpr int RB = 2 * TM, U = 2 * RB;                           // row blocks of a step, units of a K tile
  static constexpr int ACH = TM, D0 = ACH / 2, D1 = ACH - D0;             // A pieces a wave queues per K tile, and in each half of it
  static constexpr int PER = ACH + 8;                                     // vector-memory operations of a K tile
  static constexpr int R = 8, D = U - 2 < 6 ? 2 : 6;                      // row blocks in registers, and how many units ahead one is read
  static constexpr int after_w(int nd) { return nd > 3 ? nd - 3 : 0; }    // DMAs of a half behind its last W load
  static constexpr int after_d(int nd) { return nd < 4 ? 4 - nd : 0; }    // W loads of a half behind its last DMA
  // operation k of a half with nd DMAs: W load (true) or DMA, and its number among its kind
  static constexpr bool is_w(int k, int nd) { return k < 2 * nd && k < 8 ? k % 2 == 0 : (nd < 4 ? true : false); }
  static constexpr int num(int k, int nd) { int n = 0; for (int i = 0; i < k; i++) n += is_w(i, nd) == is_w(k, nd); return n; }
  static constexpr int unit_of(int k, int nd) { return k * RB / (4 + nd); }   // unit of the half it goes out in
  static constexpr int upto(int u, int nd) { int n = 0; for (int k = 0; k < 4 + nd; k++) n += unit_of(k, nd) < u; return n; }
  // operations queued behind the W operands of step 0 and of step 1 when that step begins, and behind the last A piece of the next
  // tile at the barrier
  static constexpr int WAIT0 = after_w(D1) + (SETS - 1) * PER, WAIT1 = after_w(D0) + (SETS - 1) * PER;
  static constexpr int UB = U - D;                                        // the barrier stands before the reads of this unit
  static constexpr int WAITB = after_d(D1) + (SETS - 2) * PER + (UB >= RB ? 4 + D0 + upto(UB - RB, D1) : upto(UB, D0));
  static_assert(WAIT0 < 64 && WAIT1 < 64 && WAITB < 64 && WAITB >= 0, "vmcnt is a 6-bit counter");
  static_assert(SETS * U % R == 0 && D + 2 <= R && D <= RB * 2 - 2, "the row blocks' registers turn over whole within the loop");
};

typedef const __attribute__((address_space(3))) unsigned char* lds_cptr;
__device__ __forceinline__ bf16x8 lds_read16(lds_cptr p) { return *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(p); }
// Output of one tile of the QKV projection, from its bf16 image [rows][256 + padding]: what rope_kv_prefill_kernel does, without the
// pass over memory (8192 rows of 32 + 8 + 8 heads 59 us, 2048 on 224 CUs 17, 301 5.8). A tile is 256 / d whole heads of any kind.
// Q and K: 16 threads a row, eight rotation pairs each. V: a thread per column; eight rows that fill half a page row leave as 16 bytes.
template <int RS>
__device__ __forceinline__ void store_qkv_image(const GemmArgs& g, const bf16* img, int m0, int n0, int rows) {
  constexpr int BATCH = 4;                                   // rows of a thread under way
  const QkvOut& o = g.qkv;
  const int tid = threadIdx.x, lane = tid & 63, d = o.geo.d, half = d >> 1, head0 = n0 / d;
  {
    const int per_head = d >> 4, hd = head0 + (tid & 15) / per_head, i0 = (tid & 15) % per_head * 8, c0 = (hd - head0) * d + i0;
    if (hd < o.n_q + o.geo.n_kv) {
      const bool is_k = hd >= o.n_q;
      for (int r0 = tid >> 4; r0 < rows; r0 += 16 * BATCH) {
        f32x4 cs[BATCH][2], sn[BATCH][2];
        int place[BATCH];
#pragma unroll
        for (int p = 0; p < BATCH; p++) {                    // rows past the tile's repeat its last one
          const int row = min(r0 + 16 * p, rows - 1);
          const float* t = o.rot + (size_t)(m0 + row) * d + i0;
#pragma unroll
          for (int q = 0; q < 2; q++) {
            cs[p][q] = *reinterpret_cast<const f32x4*>(t + 4 * q);
            sn[p][q] = *reinterpret_cast<const f32x4*>(t + half + 4 * q);
          }
          place[p] = is_k ? o.place[m0 + row] : 0;
        }
#pragma unroll
        for (int p = 0; p < BATCH; p++) {
          const int row = r0 + 16 * p;
          const bf16* im = img + (size_t)min(row, rows - 1) * RS + c0;
          const bf16x8 a = *reinterpret_cast<const bf16x8*>(im), b = *reinterpret_cast<const bf16x8*>(im + half);
          bf16x8 ya, yb;
#pragma unroll
          for (int e = 0; e < 8; e++) {
            float ra, rb;
            rotate_pair(bf2f(a[e]), bf2f(b[e]), cs[p][e >> 2][e & 3], sn[p][e >> 2][e & 3], &ra, &rb);
            ya[e] = f2bf(ra);
            yb[e] = f2bf(rb);
          }
          bf16* dst = is_k ? o.pool + ((size_t)(place[p] >> 4) * o.geo.n_kv + (hd - o.n_q)) * o.geo.head_elems() + (size_t)(place[p] & 15) * d + i0
                           : reinterpret_cast<bf16*>(g.C) + (size_t)(m0 + row) * g.ldc + n0 + c0;
          if (row < rows) {
            *reinterpret_cast<bf16x8*>(dst) = ya;
            *reinterpret_cast<bf16x8*>(dst + half) = yb;
          }
        }
      }
    }
  }
  const int hv = head0 + tid / d - o.n_q - o.geo.n_kv;       // this column's V head
  if (__any(hv >= 0)) {
    bf16* vt = o.pool + (size_t)max(hv, 0) * o.geo.head_elems() + (size_t)16 * d + (size_t)(tid % d) * 16;
    const bf16* col = img + tid;
    for (int r0 = 0; r0 < rows; r0 += 64) {
      const int cnt = min(64, rows - r0), mine = o.place[m0 + r0 + min(lane, cnt - 1)];   // a row's place per lane
      for (int r = 0; r < cnt;) {
        const int place = __builtin_amdgcn_readlane(mine, r);
        bf16* dst = vt + (size_t)(place >> 4) * o.geo.page_elems() + (place & 15);
        if ((place & 7) == 0 && r + 8 <= cnt && __builtin_amdgcn_readlane(mine, min(r + 7, 63)) == place + 7) {   // places of a sequence follow each other
          bf16x8 v;
#pragma unroll
          for (int e = 0; e < 8; e++) v[e] = col[(size_t)(r0 + r + e) * RS];
          if (hv >= 0) *reinterpret_cast<bf16x8*>(dst) = v;
          r += 8;
        } else {
          if (hv >= 0) *dst = col[(size_t)(r0 + r) * RS];
          r++;
        }
      }
    }
  }
}

template <int EPI, int TM>
__device__ __forceinline__ void gemm_rows_body(const GemmArgs& g, unsigned char* arena, int m0, int n0, int kbeg, int kend, int piece) {
  using P = RowsPlan<TM>;
  constexpr int BM = 32 * TM, BN = 256, BK = 64, NT = 256, TN = 4, RB = P::RB, U = P::U, D = P::D, R = P::R, SETS = P::SETS;
  constexpr int NS = SETS + 2;                               // A stages
  constexpr int ROWB = BK * 2, STAGE = BM * ROWB, ACH = TM;
  static_assert(NS * STAGE <= ROWS_LDS, "the stages fit the launch's LDS");
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lq = lane >> 4;
  const int swave = __builtin_amdgcn_readfirstlane(tid >> 6);

  unsigned a_off[ACH];
#pragma unroll
  for (int j = 0; j < ACH; j++) {
    const int q = (j * 4 + swave) * 64 + lane, row = q >> 3, ch = (q & 7) ^ ((row >> 1) & 7);
    a_off[j] = (unsigned)(min(m0 + row, g.M - 1) - m0) * (unsigned)g.lda * 2u + ch * 16;
  }
  // A wave's 64 columns are two neighbouring 32-column blocks -- a gate block and its up block in the SwiGLU form -- in halves of 16.
  // Operand of a half, step s: 256 bytes out of each quarter of a 2 KiB half of the block's 4 KiB.
  const unsigned wrow = (unsigned)(g.K >> 6) * 4096u;
  const unsigned w_lane0 = (unsigned)((lq >> 1) * 1024 + (lq & 1) * 512 + l16 * 16), w_lane1 = w_lane0 + wrow;
  bf16x8 w[SETS][2][TN];
#pragma unroll
  for (int z = 0; z < SETS; z++)
#pragma unroll
    for (int s = 0; s < 2; s++)
#pragma unroll
      for (int j = 0; j < TN; j++)
#pragma unroll
        for (int e = 0; e < 8; e++) w[z][s][j][e] = 0;
  // the loop takes a multiple of SETS tiles: `lead` null tiles (zero operands) first
  const int nk = (kend - kbeg) / BK, lead = (SETS - nk % SETS) % SETS, nt = nk + lead;
  const unsigned char* ap = reinterpret_cast<const unsigned char*>(g.A + (size_t)m0 * g.lda) + (size_t)kbeg * 2;   // A of the tile whose pieces are queued
  const unsigned char* wp = reinterpret_cast<const unsigned char*>(g.W) + (size_t)((n0 >> 5) + swave * 2) * wrow + (size_t)(kbeg >> 6) * 4096;
  const unsigned arena_lds = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)arena + swave * 1024;
  // operation k of half h of a tile: W operands (set z, step 1 - h) or a piece of A; in two parts, the first sets m0
  auto vm_first = [&](auto h_c, auto k_c, unsigned stage) {
    constexpr int h = decltype(h_c)::value, k = decltype(k_c)::value, nd = h ? P::D1 : P::D0, n = P::num(k, nd);
    if constexpr (!P::is_w(k, nd)) { constexpr int j = h ? P::D0 + n : n; dma_m0<j * 4096>(stage); }
  };
  auto vm_op = [&](auto h_c, auto k_c, auto z_c) {
    constexpr int h = decltype(h_c)::value, k = decltype(k_c)::value, z = decltype(z_c)::value, nd = h ? P::D1 : P::D0, s = 1 - h;
    constexpr int n = P::num(k, nd);
    if constexpr (P::is_w(k, nd)) load_w_off<(n & 1) * 256 + s * 2048>(w[z][s][n], wp, n >> 1 ? w_lane1 : w_lane0);
    else { constexpr int j = h ? P::D0 + n : n; dma_load(ap, a_off[j]); }
  };

  f32x4 acc[RB][TN];
#pragma unroll
  for (int i = 0; i < RB; i++)
#pragma unroll
    for (int j = 0; j < TN; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // queue the first SETS tiles in the loop's order
  static_for<SETS>([&](auto z_c) {
    constexpr int z = decltype(z_c)::value;
    const unsigned stage = arena_lds + z * STAGE;
    static_for<4 + P::D0>([&](auto k_c) {
      constexpr int k = decltype(k_c)::value;
      if constexpr (z > 0 || !P::is_w(k, P::D0)) {
        vm_first(std::integral_constant<int, 0>{}, k_c, stage);
        dma_m0_idle();
        vm_op(std::integral_constant<int, 0>{}, k_c, std::integral_constant<int, (z + SETS - 1) % SETS>{});
      }
    });
    if (z > lead) wp += 4096;
    static_for<4 + P::D1>([&](auto k_c) {
      vm_first(std::integral_constant<int, 1>{}, k_c, stage);
      dma_m0_idle();
      vm_op(std::integral_constant<int, 1>{}, k_c, z_c);
    });
    if (z >= lead) ap += z - lead + 1 < nk ? 128 : 0;
  });
  if (lead > 0) {                                            // the null tiles' operands and stages
    wait_vmem<0>();
    __syncthreads();                                         // every wave's pieces have landed
    static_for<SETS>([&](auto z_c) {
      constexpr int z = decltype(z_c)::value;
      static_for<2>([&](auto s_c) { constexpr int s = decltype(s_c)::value; wait_vmem_for4<0>(w[z][s]); });
      if (z < lead) {
#pragma unroll
        for (int s = 0; s < 2; s++)
#pragma unroll
          for (int j = 0; j < TN; j++)
#pragma unroll
            for (int e = 0; e < 8; e++) w[z][s][j][e] = 0;
        for (int c = tid; c < STAGE / 16; c += NT) *reinterpret_cast<u32x4*>(arena + z * STAGE + c * 16) = u32x4{0u, 0u, 0u, 0u};
      }
    });
  }
  wait_vmem<P::after_d(P::D1) + (SETS - 1) * P::PER>();      // A(0) has landed
  __syncthreads();
  const int koff0 = (lq ^ ((l16 >> 1) & 7)) * 16;            // step 1's chunk: koff0 ^ 64
  lds_cptr base0 = (lds_cptr)(arena + l16 * ROWB + koff0), base1 = (lds_cptr)(arena + l16 * ROWB + (koff0 ^ 64));
  bf16x8 af[R];
  static_for<D>([&](auto u_c) {
    constexpr int u = decltype(u_c)::value;
    af[u] = lds_read16((u / RB ? base1 : base0) + (u % RB) * 16 * ROWB);
  });
  // a unit per row block: its four products, between them the read of the block D units ahead and a vector-memory operation
  unsigned cur = 0, into = SETS * STAGE;                     // stages of the tile in hand and of the tile whose pieces are queued (bytes)
  lds_cptr rd0 = base0, rd1 = base1;
  auto tile = [&](int t, auto z_c) {
    constexpr int z = decltype(z_c)::value, zp = (z + SETS - 1) % SETS;
    lds_cptr nx0 = rd0, nx1 = rd1;
    const unsigned stage = arena_lds + into;
    static_for<U>([&](auto u_c) {
      constexpr int u = decltype(u_c)::value, s = u / RB, i = u % RB, nd = s ? P::D1 : P::D0;
      constexpr std::integral_constant<int, s> s_c{};
      constexpr std::integral_constant<int, s ? z : zp> zz{};
      constexpr int n_ops = P::upto(i + 1, nd) - P::upto(i, nd), k0 = P::upto(i, nd);
      constexpr bool AG = i < P::AGPR_BLOCKS;
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (u == 0) wait_vmem_for4<P::WAIT0>(w[z][0]);
      if constexpr (u == RB) wait_vmem_for4<P::WAIT1>(w[z][1]);
      if constexpr (u == P::UB) {
        wait_vmem<P::WAITB>();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
      }
      mma16<AG>(acc[i][0], w[z][s][0], af[(z * U + u) % R]);
      __builtin_amdgcn_sched_barrier(0);
      constexpr int un = (u + D) % U;
      af[(z * U + u + D) % R] = lds_read16((u + D >= U ? (un / RB ? nx1 : nx0) : (un / RB ? rd1 : rd0)) + (un % RB) * 16 * ROWB);
      __builtin_amdgcn_sched_barrier(0);
      mma16<AG>(acc[i][1], w[z][s][1], af[(z * U + u) % R]);
      if constexpr (n_ops > 0) vm_first(s_c, std::integral_constant<int, k0>{}, stage);
      mma16<AG>(acc[i][2], w[z][s][2], af[(z * U + u) % R]);
      if constexpr (n_ops > 0) vm_op(s_c, std::integral_constant<int, k0>{}, zz);
      mma16<AG>(acc[i][3], w[z][s][3], af[(z * U + u) % R]);
      __builtin_amdgcn_sched_barrier(0);
      static_for<n_ops>([&](auto k_c) {
        constexpr int k = k0 + decltype(k_c)::value;
        if constexpr (k > k0) {
          vm_first(s_c, std::integral_constant<int, k>{}, stage);
          dma_m0_idle();
          vm_op(s_c, std::integral_constant<int, k>{}, zz);
        }
      });
      if constexpr (u == RB - 1) wp += t + SETS < nt ? 4096 : 0;                // W of tile t + SETS from here on
      if constexpr (u == U - 1) ap += t + SETS + 1 < nt ? 128 : 0;
      if constexpr (u == P::UB - 2) cur = cur + STAGE == NS * STAGE ? 0 : cur + STAGE;
      if constexpr (u == P::UB - 1) { nx0 = base0 + cur; nx1 = base1 + cur; }
      if constexpr (u == U - 1) into = into + STAGE == NS * STAGE ? 0 : into + STAGE;
    });
    rd0 = nx0; rd1 = nx1;
  };
  for (int t = 0; t < nt; t += SETS) static_for<SETS>([&](auto z_c) { tile(t + decltype(z_c)::value, z_c); });
  mma16_settle();
  static_for<RB * TN>([&](auto q) {
    constexpr int i = decltype(q)::value / TN, j = decltype(q)::value % TN;
    mma16_settled<(i < P::AGPR_BLOCKS)>(acc[i][j]);
  });
  // the surplus loads of the last iterations must not land in registers or stages the epilogue reuses
#pragma unroll
  for (int z = 0; z < SETS; z++)
#pragma unroll
    for (int s = 0; s < 2; s++) wait_vmem_for4<0>(w[z][s]);

  // ---- outputs: lane (lq, l16) holds columns 4 lq .. + 4 of 16-column block j, rows 16 i + l16 of its wave tile. They leave
  // through the (now free) A stages as a [rows][columns] image, so that rows go out whole.
  const int rloc = l16, cloc = swave * 64 + 4 * lq;          // column block j: + 16 j
  // A row block's sums are read where they are stored, not earlier: all at once, or ahead of a branch, the compiler spills.
  auto take_row_block = [&](auto i_c) {
    constexpr int i = decltype(i_c)::value;
    __builtin_amdgcn_sched_barrier(0);
    mma16_settled<(i < P::AGPR_BLOCKS)>(acc[i][0]);
    mma16_settled<(i < P::AGPR_BLOCKS)>(acc[i][1]);
    mma16_settled<(i < P::AGPR_BLOCKS)>(acc[i][2]);
    mma16_settled<(i < P::AGPR_BLOCKS)>(acc[i][3]);
  };
  // fp32 rows, up to 128 at a time: each wave takes a quarter of them, a row (1 KiB) per instruction. ADD: to what is there, the rows of
  // the next eight under way. Bound by memory, all workgroups of a wave of them at once: 256 rows of the residual stream 45 us straight
  // from the accumulators (64 bytes of a row in each of 16 rows per instruction), 24 this way; the projection of 8192 x 4096 x 4096 231 -> 220 us,
  // 8192 x 4096 x 14336 663 -> 649, 3980 x 4096 x 4096 108 -> 103, 2048 rows on tiles of 128 62 -> 57.
  auto store_f32 = [&](auto add_c, float* out, int ld, int rows) {
    constexpr bool ADD = decltype(add_c)::value;
    constexpr int HB = RB < 8 ? RB : 8, RSF = BN + 4;        // row blocks of a pass; floats of an image row
    static_assert(HB * 16 * RSF * 4 <= ROWS_LDS, "the image fits the stages");
    float* img = reinterpret_cast<float*>(arena);
    float* col = out + lane * 4;
    static_for<(RB + HB - 1) / HB>([&](auto h_c) {
      constexpr int h = decltype(h_c)::value, cnt = RB - h * HB < HB ? RB - h * HB : HB, RPW = cnt * 4;
      const int r0 = h * HB * 16 + swave * RPW;              // this wave's rows of the pass
      f32x4 old[8];
      auto fetch = [&](int q) {
#pragma unroll
        for (int i = 0; i < 8; i++) old[i] = *reinterpret_cast<const f32x4*>(col + (size_t)min(r0 + q + i, rows - 1) * ld);
      };
      if constexpr (ADD) fetch(0);
      __syncthreads();                                       // the stage reads of the main loop, or of the pass before, are done
      static_for<cnt>([&](auto i_c) {
        constexpr int i = decltype(i_c)::value;
        take_row_block(std::integral_constant<int, h * HB + i>{});
#pragma unroll
        for (int j = 0; j < TN; j++) *reinterpret_cast<f32x4*>(img + (i * 16 + rloc) * RSF + cloc + j * 16) = acc[h * HB + i][j];
      });
      __syncthreads();
      for (int q = 0; q < RPW; q += 8) {
        f32x4 v[8];
#pragma unroll
        for (int i = 0; i < 8; i++) v[i] = *reinterpret_cast<const f32x4*>(img + (swave * RPW + q + i) * RSF + lane * 4);
        if constexpr (ADD) {
#pragma unroll
          for (int i = 0; i < 8; i++) v[i] = old[i] + v[i];
          if (q + 8 < RPW) fetch(q + 8);
        }
#pragma unroll
        for (int i = 0; i < 8; i++)
          if (r0 + q + i < rows) *reinterpret_cast<f32x4*>(col + (size_t)(r0 + q + i) * ld) = v[i];
      }
    });
  };
  if (piece >= 0) {                                          // a tail piece leaves its partial tile, row-major [height][256]
    store_f32(std::integral_constant<bool, false>{}, g.tail_ws + (size_t)piece * g.piece_stride, BN, BM);
    return;
  }
  if constexpr (EPI == EPI_F32 || EPI == EPI_RESID_F32) {
    float* out = reinterpret_cast<float*>(g.C) + (EPI == EPI_F32 ? (size_t)blockIdx.y * g.split_stride : 0) + (size_t)m0 * g.ldc + n0;
    store_f32(std::integral_constant<bool, EPI == EPI_RESID_F32>{}, out, g.ldc, min(BM, g.M - m0));
  } else {
    constexpr bool SW = EPI == EPI_SWIGLU_BF16;
    constexpr int OC = SW ? BN / 2 : BN, RS = OC + 16;
    // whole 128-byte lines of bf16; 32 bytes of padding per row spread the 8-byte writes of 16 rows over the banks
    static_assert(BM * RS * 2 <= ROWS_LDS, "the image fits the stages");
    bf16* img = reinterpret_cast<bf16*>(arena);
    bf16* outp = reinterpret_cast<bf16*>(g.C) + (SW ? (n0 >> 1) : n0);
    __syncthreads();                                         // the stage reads of the main loop are done
    bf16* dst = img + (size_t)rloc * RS + (SW ? swave * 32 + 4 * lq : cloc);
    static_for<RB>([&](auto i_c) {
      constexpr int i = decltype(i_c)::value;
      take_row_block(i_c);
#pragma unroll
      for (int j = 0; j < (SW ? 2 : TN); j++) {
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; e++) {
          if constexpr (SW) {
            o[e] = f2bf(swiglu(acc[i][j][e], acc[i][j + 2][e]));
          } else {
            o[e] = f2bf(acc[i][j][e]);
          }
        }
        *reinterpret_cast<bf16x4*>(dst + (size_t)i * 16 * RS + j * 16) = o;
      }
    });
    __syncthreads();
    if constexpr (EPI == EPI_QKV) {
      store_qkv_image<RS>(g, img, m0, n0, min(BM, g.M - m0));
      return;
    }
    constexpr int CPRW = OC / 8;
#pragma unroll
    for (int c = 0; c < BM * CPRW / NT; c++) {
      const int q = c * NT + tid, row = q / CPRW, cc = q % CPRW;
      const int grow = m0 + row;
      if (grow < g.M)
        *reinterpret_cast<u32x4*>(outp + (size_t)grow * g.ldc + cc * 8) = *reinterpret_cast<const u32x4*>(img + (size_t)row * RS + cc * 8);
    }
  }
}

template <int EPI>
__global__ void __launch_bounds__(256, 1) gemm_rows_kernel(GemmArgs g) {
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* arena = smem + GEMM_DL_LDS_BASE;
  int v, kbeg, kend, piece, tm, tn, m0, blocks;
  if (!block_work<64>(g, &v, &kbeg, &kend, &piece)) return;
  tile_coords(g, v, &tm, &tn);
  row_range(g, tm, &m0, &blocks);
  const int n0 = tn * 256;
  switch (blocks) {                                          // workgroup-uniform
    case 1: gemm_rows_body<EPI, 1>(g, arena, m0, n0, kbeg, kend, piece); break;
    case 2: gemm_rows_body<EPI, 2>(g, arena, m0, n0, kbeg, kend, piece); break;
    case 3: gemm_rows_body<EPI, 3>(g, arena, m0, n0, kbeg, kend, piece); break;
    case 4: gemm_rows_body<EPI, 4>(g, arena, m0, n0, kbeg, kend, piece); break;
    case 5: gemm_rows_body<EPI, 5>(g, arena, m0, n0, kbeg, kend, piece); break;
    case 6: gemm_rows_body<EPI, 6>(g, arena, m0, n0, kbeg, kend, piece); break;
    case 7: gemm_rows_body<EPI, 7>(g, arena, m0, n0, kbeg, kend, piece); break;
    case 8: gemm_rows_body<EPI, 8>(g, arena, m0, n0, kbeg, kend, piece); break;
    default: break;
  }
}

// ---- the same tiles with row-major W (callers that bring their own weights; fp32 store), many of them ---------------
// Both operands through LDS in two stages, waves of 128 x 64, and the 16 x 16 x 32 instruction, whose chain along K gives bit for
// bit what the 32 x 32 x 16 one gives. It holds a higher clock where the chip is full for long (see gemm_rows_kernel) but waits
// for a whole stage at each barrier: gemm_dl_kernel's tiles are faster where every CU has one (launch_rowmajor256). A step's
// operands are taken in two groups of four row blocks.
template <int WGM>
__global__ void __launch_bounds__(WGM * 256, 2) gemm_rowmajor256_kernel(GemmArgs g) {
  constexpr int BM = WGM * 128, BN = 256, BK = 64, NT = WGM * 256, ROWB = BK * 2, STAGE = (BM + BN) * ROWB;
  constexpr int A_CH = BM * 8 / NT, B_CH = BN * 8 / NT;
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* arena = smem + GEMM_DL_LDS_BASE;
  int v, kbeg, kend, piece, tm, tn;
  if (!block_work<BK>(g, &v, &kbeg, &kend, &piece)) return;
  tile_coords(g, v, &tm, &tn);
  const int m0 = tm * BM, n0 = tn * BN;
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lq = lane >> 4;
  const int swave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = swave >> 2, wn = swave & 3;

  const unsigned char* a_base = reinterpret_cast<const unsigned char*>(g.A + (size_t)m0 * g.lda);
  const unsigned char* b_base = reinterpret_cast<const unsigned char*>(g.W + (size_t)n0 * g.ldw);
  unsigned a_off[A_CH], b_off[B_CH];
#pragma unroll
  for (int j = 0; j < A_CH; j++) {
    const int q = j * NT + tid, row = q >> 3, ch = (q & 7) ^ ((row >> 1) & 7);
    a_off[j] = (unsigned)(min(m0 + row, g.M - 1) - m0) * (unsigned)g.lda * 2u + ch * 16;
  }
#pragma unroll
  for (int j = 0; j < B_CH; j++) {
    const int q = j * NT + tid, row = q >> 3, ch = (q & 7) ^ ((row >> 1) & 7);
    b_off[j] = (unsigned)row * (unsigned)g.ldw * 2u + ch * 16;
  }
  auto issue = [&](int stage, int k) {
    unsigned char* sa = arena + stage * STAGE + swave * 1024;
#pragma unroll
    for (int j = 0; j < A_CH; j++) lds_dma16(a_base + (size_t)k * 2, a_off[j], sa + j * NT * 16);
#pragma unroll
    for (int j = 0; j < B_CH; j++) lds_dma16(b_base + (size_t)k * 2, b_off[j], sa + BM * ROWB + j * NT * 16);
  };
  f32x4 acc[8][4];
#pragma unroll
  for (int i = 0; i < 8; i++)
#pragma unroll
    for (int j = 0; j < 4; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  int koff[2];
#pragma unroll
  for (int s = 0; s < 2; s++) koff[s] = ((s * 4 + lq) ^ ((l16 >> 1) & 7)) * 16;
  const int a_row = (wm * 128 + l16) * ROWB, b_row = BM * ROWB + (wn * 64 + l16) * ROWB;

  const int nk = (kend - kbeg) / BK;
  issue(0, kbeg);
  if (nk > 1) issue(1, kbeg + BK);
  if (nk > 1) wait_vmem<A_CH + B_CH>(); else wait_vmem<0>();
  __syncthreads();
  bf16x8 af[2][4], wf[2][4];
#pragma unroll
  for (int i = 0; i < 4; i++) {
    af[0][i] = *reinterpret_cast<const bf16x8*>(arena + a_row + i * 16 * ROWB + koff[0]);
    wf[0][i] = *reinterpret_cast<const bf16x8*>(arena + b_row + i * 16 * ROWB + koff[0]);
  }
  for (int t = 0; t < nk; t++) {
    const unsigned char* cur = arena + (t & 1) * STAGE;
    const unsigned char* nxt = arena + ((t + 1) & 1) * STAGE;
    static_for<4>([&](auto p_c) {
      constexpr int p = decltype(p_c)::value, s = p >> 1, h = p & 1, pn = (p + 1) & 3, sn = pn >> 1, hn = pn & 1;
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (pn == 0) {
        // tile t + 1 has landed and this one's operands are in registers: its stage takes tile t + 2
        wait_vmem<0>();
        __syncthreads();
        if (t + 2 < nk) issue(t & 1, kbeg + (t + 2) * BK);
        __builtin_amdgcn_sched_barrier(0);
      }
      const unsigned char* src = pn == 0 ? nxt : cur;          // (after the last tile: a stage nobody uses the operands of)
#pragma unroll
      for (int i = 0; i < 4; i++) af[pn & 1][i] = *reinterpret_cast<const bf16x8*>(src + a_row + (hn * 4 + i) * 16 * ROWB + koff[sn]);
      if constexpr (hn == 0) {
#pragma unroll
        for (int j = 0; j < 4; j++) wf[sn][j] = *reinterpret_cast<const bf16x8*>(src + b_row + j * 16 * ROWB + koff[sn]);
      }
#pragma unroll
      for (int i = 0; i < 4; i++)
#pragma unroll
        for (int j = 0; j < 4; j++)
          acc[h * 4 + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[s][j], af[p & 1][i], acc[h * 4 + i][j], 0, 0, 0);
      constexpr int NR = hn == 0 ? 8 : 4;
#pragma unroll
      for (int x = 0; x < NR; x++) {
        __builtin_amdgcn_sched_group_barrier(0x008, 16 / NR, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  }
  const int rloc = wm * 128 + l16, cloc = wn * 64 + 4 * lq;
  float* out = piece >= 0 ? g.tail_ws + (size_t)piece * g.piece_stride + cloc
                          : reinterpret_cast<float*>(g.C) + (size_t)blockIdx.y * g.split_stride + (size_t)m0 * g.ldc + n0 + cloc;
  const int ld = piece >= 0 ? BN : g.ldc, rows = piece >= 0 ? BM : g.M - m0;
#pragma unroll
  for (int i = 0; i < 8; i++) {
    const int row = rloc + i * 16;
    if (row >= rows) continue;
#pragma unroll
    for (int j = 0; j < 4; j++) *reinterpret_cast<f32x4*>(out + (size_t)row * ld + j * 16) = acc[i][j];
  }
}

// store_fixed_up of the QKV projection: a thread whose columns are of a head's first half takes their rotation partners too.
__device__ __forceinline__ void store_fixed_up_qkv(const GemmArgs& g, const float* p, int stride, int row, int col) {
  const QkvOut& o = g.qkv;
  const int d = o.geo.d, half = d >> 1, hd = col / d, i0 = col % d;
  const bool rotated = hd < o.n_q + o.geo.n_kv;
  if (rotated && i0 >= half) return;
  f32x4 a = *reinterpret_cast<const f32x4*>(p), b = {0.f, 0.f, 0.f, 0.f};
  if (rotated) b = *reinterpret_cast<const f32x4*>(p + half);
  for (int z = 1; z < g.tail_f; z++) {
    a += *reinterpret_cast<const f32x4*>(p + (size_t)z * stride);
    if (rotated) b += *reinterpret_cast<const f32x4*>(p + (size_t)z * stride + half);
  }
  const int place = hd >= o.n_q ? o.place[row] : 0;
  if (!rotated) {
    bf16* v = o.pool + (size_t)(place >> 4) * o.geo.page_elems() + (size_t)(hd - o.n_q - o.geo.n_kv) * o.geo.head_elems() + (size_t)16 * d + (place & 15);
#pragma unroll
    for (int e = 0; e < 4; e++) v[(size_t)(i0 + e) * 16] = f2bf(a[e]);
    return;
  }
  const f32x4 cs = *reinterpret_cast<const f32x4*>(o.rot + (size_t)row * d + i0), sn = *reinterpret_cast<const f32x4*>(o.rot + (size_t)row * d + half + i0);
  bf16x4 ya, yb;
#pragma unroll
  for (int e = 0; e < 4; e++) {
    float ra, rb;
    rotate_pair(bf2f(f2bf(a[e])), bf2f(f2bf(b[e])), cs[e], sn[e], &ra, &rb);   // the projection's result is rounded to bf16 first
    ya[e] = f2bf(ra);
    yb[e] = f2bf(rb);
  }
  bf16* dst = hd < o.n_q ? reinterpret_cast<bf16*>(g.C) + (size_t)row * g.ldc + col
                         : o.pool + ((size_t)(place >> 4) * o.geo.n_kv + (hd - o.n_q)) * o.geo.head_elems() + (size_t)(place & 15) * d + i0;
  *reinterpret_cast<bf16x4*>(dst) = ya;
  *reinterpret_cast<bf16x4*>(dst + half) = yb;
}

// Adds the tail pieces of each split tile of gemm_rows_kernel in piece order and applies the epilogue. One thread per four
// consecutive columns; blocks past the tile's height leave.
template <int EPI>
__global__ void __launch_bounds__(256) gemm_rows_fixup(GemmArgs g) {
  constexpr int BN = 256;
  const int t = blockIdx.x;                                   // tail tile
  const int e = blockIdx.y * 256 + threadIdx.x;
  const int r = e / (BN / 4), c = (e % (BN / 4)) * 4;
  int tm, tn, m0, blocks;
  tile_coords(g, g.n_full + t, &tm, &tn);
  row_range(g, tm, &m0, &blocks);
  const int row = m0 + r;
  if (r >= blocks * 32 || row >= g.M) return;
  if (EPI == EPI_SWIGLU_BF16 && ((c >> 5) & 1)) return;      // "up" columns are consumed by their gate thread
  const float* p = g.tail_ws + (size_t)t * g.tail_f * g.piece_stride + (size_t)r * BN + c;
  if constexpr (EPI == EPI_QKV) store_fixed_up_qkv(g, p, g.piece_stride, row, tn * BN + c);
  else store_fixed_up<EPI>(g, p, g.piece_stride, row, tn * BN, c);
}

// gemm_rows_fixup of a residual GEMM and the RMSNorm of the rows it finishes, in one pass: a workgroup takes a row, adds the
// pieces of its split tiles to the residual stream in the same order, keeps the row in registers and normalises it as
// rmsnorm_kernel does. Bound by memory: the pieces and the row in, the row twice out; the pair of kernels reads the residual once more
// and waits twice for a launch to fill the chip. Measured, the pair and this one, mean over the O and down projections: 301 rows
// of 4096 in 3 and 8 pieces 12.5 -> 9.2 us, 1024 rows 21.7 -> 17.0. Rows of 8192 take the pair: 704 rows in 8 pieces 25.8 us, 26.7 with
// eight loads a piece and thread here.
constexpr int FIXUP_NORM_MAX_N = 4096;
__global__ void __launch_bounds__(256) gemm_rows_fixup_norm(GemmArgs g, bf16* out, const float* gain, float eps) {
  constexpr int PER = FIXUP_NORM_MAX_N / 1024;
  __shared__ float red[4];
  const int row = blockIdx.x, b = row / 32;
  const int tm = g.tile_blocks ? b / g.tile_blocks : (int)(((long long)(b + 1) * g.tiles_m - 1) / g.row_blocks);   // row_range's inverse
  int m0, blocks;
  row_range(g, tm, &m0, &blocks);
  const int first_m = tm / g.group_m * g.group_m, gm = min(g.tiles_m - first_m, g.group_m);
  const int v0 = first_m * g.tiles_n + tm - first_m;          // index of the row's first tile; the next ones are gm apart (tile_coords)
  float* x = reinterpret_cast<float*>(g.C) + (size_t)row * g.ldc;
  const float* p = g.tail_ws + (size_t)(row - m0) * 256 + (threadIdx.x * 4) % 256;
  f32x4 v[PER], sum[PER];
  const float* src[PER];                                      // the first piece of each four elements; those of a whole tile have none
  size_t stride[PER];                                         // and read the row again (no branch between the loads), unused
  bool cut[PER];                                              // wave-uniform: a wave's load is one tile wide
#pragma unroll
  for (int i = 0; i < PER; i++) {
    const int c = min(threadIdx.x * 4 + i * 1024, g.N - 4), t = v0 + c / 256 * gm - g.n_full;
    cut[i] = t >= 0 && threadIdx.x * 4 + i * 1024 < g.N;
    src[i] = cut[i] ? p + (size_t)t * g.tail_f * g.piece_stride : x + c;
    stride[i] = cut[i] ? g.piece_stride : 0;
    v[i] = *reinterpret_cast<const f32x4*>(x + c);
    sum[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  for (int z0 = 0; z0 < g.tail_f; z0 += 4) {
    f32x4 q[4][PER];
#pragma unroll
    for (int z = 0; z < 4; z++)
#pragma unroll
      for (int i = 0; i < PER; i++) q[z][i] = *reinterpret_cast<const f32x4*>(src[i] + min(z0 + z, g.tail_f - 1) * stride[i]);
#pragma unroll
    for (int z = 0; z < 4; z++)
      if (z0 + z < g.tail_f) {
#pragma unroll
        for (int i = 0; i < PER; i++) sum[i] = z0 + z == 0 ? q[z][i] : sum[i] + q[z][i];
      }
  }
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < PER; i++) {
    if (cut[i]) { v[i] += sum[i]; *reinterpret_cast<f32x4*>(x + threadIdx.x * 4 + i * 1024) = v[i]; }
    if (threadIdx.x * 4 + i * 1024 >= g.N) v[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    ss += v[i][0] * v[i][0] + v[i][1] * v[i][1] + v[i][2] * v[i][2] + v[i][3] * v[i][3];
  }
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  const float inv = rsqrtf((red[0] + red[1] + red[2] + red[3]) / (float)g.N + eps);
#pragma unroll
  for (int i = 0; i < PER; i++) {
    const int c = threadIdx.x * 4 + i * 1024;
    if (c >= g.N) break;
    const f32x4 w = *reinterpret_cast<const f32x4*>(gain + c);
    bf16x4 o;
#pragma unroll
    for (int j = 0; j < 4; j++) o[j] = f2bf(v[i][j] * inv * w[j]);
    *reinterpret_cast<bf16x4*>(out + (size_t)row * g.N + c) = o;
  }
}

// How the tiles of one launch are divided when the partition holds `slots` workgroups of this
// configuration at once: n_full tiles run whole (complete waves), the `rest` tiles of the last
// wave are cut into f pieces (f = 1: no cut). rest * f pieces take ceil(rest * f / slots) rounds
// of 1/f tile time each; every piece also pays a fixed start-up and partial-store cost, taken as
// 3 % of a tile time. The cut is made only if it saves at least a tenth of a tile time.
void gemm_tail_plan(int tiles, int ksteps, int slots, long long max_pieces, int* n_full, int* f) {
  *n_full = tiles; *f = 1;
  if (slots <= 0) return;
  const int full = tiles / slots * slots, rest = tiles - full;
  if (rest == 0) return;
  int best = 1; double best_t = 1.0;
  for (int cut = 2; cut <= std::min(ksteps / 4, 16); cut++) {
    if ((long long)rest * cut > max_pieces) break;               // partial tiles must fit the scratch buffer
    const int rounds = (rest * cut + slots - 1) / slots;
    const double t = rounds * (1.0 / cut + 0.03);
    if (t < best_t - 1e-9) { best_t = t; best = cut; }
  }
  if (best_t > 0.9) return;
  *n_full = full; *f = best;
}

// Whole tiles, tail pieces (stride floats each) and slices along K of a launch; returns the number of slices (gridDim.y).
static int plan_launch(GemmArgs* g, int tiles, int splits, const GemmTail* tail, int piece_floats) {
  constexpr int BK = 64;
  g->group_m = 8;
  const int ksteps = g->K / BK;
  g->n_full = tiles; g->tail_f = 1; g->n_pieces = 0; g->piece_per_xcd = 0; g->tail_ws = nullptr; g->piece_stride = piece_floats;
  if (tail && tail->ws && splits == 1 && g->ldc % 4 == 0) {
    int n_full, f;
    gemm_tail_plan(tiles, ksteps, tail->slots, (long long)(tail->ws_bytes / (piece_floats * sizeof(float))), &n_full, &f);
    if (f > 1) {
      g->n_full = n_full; g->tail_f = f; g->n_pieces = (tiles - n_full) * f;
      g->piece_per_xcd = (g->n_pieces + 7) / 8;
      g->tail_ws = tail->ws;
    }
  }
  g->full_per_xcd = (g->n_full + 7) / 8;
  const int per = (ksteps + splits - 1) / splits;
  g->k_per_split = per * BK;
  return (ksteps + per - 1) / per;
}

// NS: LDS stages of the main loop.
template <int BM, int BN, int WGM, int WGN, int EPI, int NS>
static hipError_t launch_cfg(hipStream_t s, GemmArgs g, int splits, const GemmTail* tail) {
  constexpr int NT = WGM * WGN * 64, BK = 64;
  constexpr size_t lds_dl = GEMM_DL_LDS_BASE + NS * (size_t)(BM + BN) * BK * sizeof(bf16);
  // decode batches: 64-row tiles, 64 columns per wave, the W operands GEMM_SKINNY_PD tiles deep in registers
  constexpr bool SKINNY = BM == 64 && WGM == 1 && BN == WGN * 64;
  constexpr size_t lds_skinny = GEMM_DL_LDS_BASE + (size_t)(GEMM_SKINNY_PD + 2) * BM * BK * sizeof(bf16) + 1024;
  void (*kern)(GemmArgs) = nullptr;
  void (*kern_rowmajor)(GemmArgs) = nullptr;       // row-major W: the fp32-store epilogue only (callers that bring their own weights)
  if constexpr (SKINNY) kern = g.stream_nt ? gemm_skinny_kernel<EPI, GEMM_SKINNY_PD, true> : gemm_skinny_kernel<EPI, GEMM_SKINNY_PD, false>;
  else kern = gemm_dl_kernel<BM, BN, WGM, WGN, EPI, NS>;
  if constexpr (EPI == EPI_F32 && !SKINNY) kern_rowmajor = gemm_dl_kernel<BM, BN, WGM, WGN, EPI, NS, false>;
  if (!g.w_packed && !kern_rowmajor) return hipErrorInvalidValue;
  constexpr size_t lds_packed = SKINNY ? lds_skinny : lds_dl;
  const size_t lds = !g.w_packed ? lds_dl : lds_packed;
  static std::atomic<bool> attr_set{false};        // the two phases' control threads may launch the same shape
  if (!attr_set.load()) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_packed);
    if constexpr (SKINNY) {      // both forms of the kernel, whichever this call takes
      void (*other)(GemmArgs) = g.stream_nt ? gemm_skinny_kernel<EPI, GEMM_SKINNY_PD, false> : gemm_skinny_kernel<EPI, GEMM_SKINNY_PD, true>;
      if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(other), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_packed);
    }
    if (e == hipSuccess && kern_rowmajor) e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern_rowmajor), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_dl);
    if (e != hipSuccess) return e;
    attr_set.store(true);
  }
  g.tiles_m = (g.M + BM - 1) / BM;
  g.tiles_n = g.N / BN;
  const int tiles = g.tiles_m * g.tiles_n;
  const int ny = plan_launch(&g, tiles, splits, tail, BM * BN);
  if (!g.w_packed) kern = kern_rowmajor;
  hipLaunchKernelGGL(kern, dim3((g.full_per_xcd + g.piece_per_xcd) * 8, ny), dim3(NT), lds, s, g);
  if constexpr (!SKINNY) {
    if (g.n_pieces > 0)
      hipLaunchKernelGGL((gemm_tail_fixup<BM, BN, EPI>), dim3(tiles - g.n_full, BM * BN / 1024), dim3(256), 0, s, g);
  }
  return hipGetLastError();
}

// gemm_rows_kernel: the rows in row_tiles tiles of nearly equal height (0: as few as 256 rows allow).
template <int EPI>
static hipError_t launch_rows(hipStream_t s, GemmArgs g, int splits, const GemmTail* tail, int row_tiles, int tile_blocks) {
  constexpr size_t lds = GEMM_DL_LDS_BASE + ROWS_LDS;
  static std::atomic<bool> attr_set{false};        // the two phases' control threads may launch the same shape
  if (!attr_set.load()) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_rows_kernel<EPI>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    attr_set.store(true);
  }
  g.row_blocks = (g.M + 31) / 32;
  g.tile_blocks = row_tiles > 0 ? 0 : tile_blocks;
  g.tiles_m = row_tiles > 0 ? row_tiles : (g.row_blocks + tile_blocks - 1) / tile_blocks;
  g.tiles_n = g.N / 256;
  const int height = row_tiles > 0 ? (g.row_blocks + row_tiles - 1) / row_tiles : std::min(tile_blocks, g.row_blocks);   // blocks of the tallest tile
  if (height > 8 || g.tiles_m > g.row_blocks) return hipErrorInvalidValue;
  const int tiles = g.tiles_m * g.tiles_n;
  // row_tiles == 0: pieces of whole tiles, so that the cut is that of the row-major form
  const int ny = plan_launch(&g, tiles, splits, tail, (row_tiles > 0 ? height : tile_blocks) * 32 * 256);
  hipLaunchKernelGGL((gemm_rows_kernel<EPI>), dim3((g.full_per_xcd + g.piece_per_xcd) * 8, ny), dim3(256), lds, s, g);
  if (EPI == EPI_RESID_F32 && g.n_pieces > 0 && tail->norm && g.N <= FIXUP_NORM_MAX_N) {
    ResidNorm& r = *tail->norm;
    hipLaunchKernelGGL(gemm_rows_fixup_norm, dim3(g.M), dim3(256), 0, s, g, r.out, r.gain, r.eps);
    r.done = true;
  } else if (g.n_pieces > 0)
    hipLaunchKernelGGL((gemm_rows_fixup<EPI>), dim3(tiles - g.n_full, height * 8), dim3(256), 0, s, g);
  return hipGetLastError();
}

// Row-major W with a 256-column tile (fp32 store). Fewer workgroups than a GPU has CUs: gemm_dl_kernel; else gemm_rowmajor256_kernel,
// if its 16-byte stores are aligned. Both give the same bits. 520 x 4096 x 4096 77 us against 83, 223 rows in four slices 30 against 35,
// 2048 x 4096 x 14336 (128 tiles) 314 against 316; 2048 x 4096 x 4096 in 256 tiles of 128 rows 66.7 against 65.3, 4096 x 28672 x 4096
// (1792 tiles) 798 against 757.
template <int WGM>
static hipError_t launch_rowmajor256(hipStream_t s, GemmArgs g, int splits, const GemmTail* tail) {
  constexpr int BM = WGM * 128, BN = 256;
  constexpr size_t lds = GEMM_DL_LDS_BASE + 2 * (size_t)(BM + BN) * 64 * sizeof(bf16);
  void (*const few)(GemmArgs) = gemm_dl_kernel<BM, BN, WGM, 4, EPI_F32, 2, false>;
  void (*const many)(GemmArgs) = gemm_rowmajor256_kernel<WGM>;
  static std::atomic<bool> attr_set{false};
  if (!attr_set.load()) {
    for (void (*k)(GemmArgs) : {few, many}) {
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
    }
    attr_set.store(true);
  }
  g.tiles_m = (g.M + BM - 1) / BM;
  g.tiles_n = g.N / BN;
  const int tiles = g.tiles_m * g.tiles_n;
  const int ny = plan_launch(&g, tiles, splits, tail, BM * BN);
  const bool aligned = reinterpret_cast<uintptr_t>(g.C) % 16 == 0 && g.ldc % 4 == 0 && g.split_stride % 4 == 0;
  const bool full = (long long)g.n_full * ny + g.n_pieces >= 256;
  hipLaunchKernelGGL(full && aligned ? many : few, dim3((g.full_per_xcd + g.piece_per_xcd) * 8, ny), dim3(WGM * 256), lds, s, g);
  if (g.n_pieces > 0)
    hipLaunchKernelGGL((gemm_tail_fixup<BM, BN, EPI_F32>), dim3(tiles - g.n_full, BM * BN / 1024), dim3(256), 0, s, g);
  return hipGetLastError();
}

template <int EPI>
static hipError_t launch_epi(hipStream_t s, int cfg, const GemmArgs& g, int splits, const GemmTail* tail, int row_tiles) {
  if (cfg == GEMM_256x256 || cfg == GEMM_128x256) {
    if (g.w_packed) return launch_rows<EPI>(s, g, splits, tail, cfg == GEMM_256x256 ? row_tiles : 0, cfg == GEMM_256x256 ? 8 : 4);
    if constexpr (EPI == EPI_F32) return cfg == GEMM_256x256 ? launch_rowmajor256<2>(s, g, splits, tail) : launch_rowmajor256<1>(s, g, splits, tail);
    return hipErrorInvalidValue;
  }
  switch (cfg) {
    case GEMM_128x128: return launch_cfg<128, 128, 2, 2, EPI, 2>(s, g, splits, tail);
    case GEMM_64x256: if constexpr (EPI != EPI_SWIGLU_BF16) return launch_cfg<64, 256, 1, 8, EPI, 3>(s, g, splits, tail); else break;
    case GEMM_64x128:     // SwiGLU: wave tiles of 32 x 64, one gate/up pair
      if constexpr (EPI == EPI_SWIGLU_BF16) return launch_cfg<64, 128, 2, 2, EPI, 3>(s, g, splits, tail);
      else return launch_cfg<64, 128, 1, 4, EPI, 3>(s, g, splits, tail);
    case GEMM_64x256S: return launch_cfg<64, 256, 1, 4, EPI, 3>(s, g, splits, nullptr);
    case GEMM_64x320S: return launch_cfg<64, 320, 1, 5, EPI, 3>(s, g, splits, nullptr);
    case GEMM_64x384S: return launch_cfg<64, 384, 1, 6, EPI, 3>(s, g, splits, nullptr);
    case GEMM_64x448S: return launch_cfg<64, 448, 1, 7, EPI, 3>(s, g, splits, nullptr);
    case GEMM_64x512S: return launch_cfg<64, 512, 1, 8, EPI, 3>(s, g, splits, nullptr);
    default: break;
  }
  return hipErrorInvalidValue;
}

int gemm_tile_n(int cfg) {
  if (cfg >= GEMM_64x256S && cfg <= GEMM_64x512S) return 256 + 64 * (cfg - GEMM_64x256S);
  return cfg == GEMM_256x256 || cfg == GEMM_64x256 || cfg == GEMM_128x256 ? 256 : 128;
}
int gemm_tile_m(int cfg) { return cfg == GEMM_256x256 ? 256 : cfg == GEMM_128x128 || cfg == GEMM_128x256 ? 128 : 64; }
// Workgroups per CU the launch plan counts: the 8-wave tiles and the 256-column ones (by their LDS) fill a CU, the other 4-wave
// tiles share it in pairs.
int gemm_wgs_per_cu(int cfg) { return cfg == GEMM_256x256 || cfg == GEMM_64x256 || cfg == GEMM_128x256 || cfg > GEMM_64x256S ? 1 : 2; }

// C = A * W^T with the chosen tile configuration and epilogue. Requirements (checked):
// K % 64 == 0, N % tile_n == 0, leading dimensions multiples of 8 elements, M >= 1; W packed (ldw == K) or,
// for the fp32-store epilogue, row-major.
// With splits > 1 (EPI_F32 only) partial sums go to C + z * split_stride. With `tail` (splits == 1)
// the tiles of the last, partly filled wave of workgroups are cut along K (see GemmArgs). row_tiles: row tiles of a 256x256
// launch (0: as few as 256 rows allow).
hipError_t gemm_bf16(hipStream_t s, int cfg, int epi, const bf16* A, int lda, const bf16* W, int ldw,
                     void* C, int ldc, int M, int N, int K, int splits, long long split_stride, const GemmTail* tail, bool w_packed, bool stream_nt,
                     int row_tiles, const QkvOut* qkv) {
  if (M < 1 || K % 64 != 0 || N % gemm_tile_n(cfg) != 0 || lda % 8 != 0 || ldw % 8 != 0) return hipErrorInvalidValue;
  if (w_packed && ldw != K) return hipErrorInvalidValue;          // packed blocks are addressed by K alone
  if (splits < 1 || (splits > 1 && epi != EPI_F32)) return hipErrorInvalidValue;
  // 16-byte output stores
  if (w_packed && (cfg == GEMM_256x256 || cfg == GEMM_128x256) && ldc % (epi == EPI_BF16 || epi == EPI_SWIGLU_BF16 || epi == EPI_QKV ? 8 : 4) != 0) return hipErrorInvalidValue;
  if (epi == EPI_QKV && (!qkv || cfg != GEMM_256x256 || !w_packed || (qkv->geo.d != 64 && qkv->geo.d != 128) || qkv->geo.page_tokens != 16 ||
                         N != (qkv->n_q + 2 * qkv->geo.n_kv) * qkv->geo.d)) return hipErrorInvalidValue;
  if (epi == EPI_SWIGLU_BF16 && cfg == GEMM_64x256) return hipErrorInvalidValue;   // its wave tile is one 32-column block, not a gate/up pair
  if (epi == EPI_SWIGLU_BF16 && cfg == GEMM_128x256) return hipErrorInvalidValue;  // not offered (the engine itself never takes this shape: its row tiles have any height)
  GemmArgs g{};
  g.A = A; g.W = W; g.C = C; g.lda = lda; g.ldw = ldw; g.ldc = ldc; g.M = M; g.N = N; g.K = K;
  if (qkv) g.qkv = *qkv;
  g.split_stride = split_stride; g.w_packed = w_packed ? 1 : 0; g.stream_nt = stream_nt ? 1 : 0;
  switch (epi) {
    case EPI_BF16: return launch_epi<EPI_BF16>(s, cfg, g, splits, tail, row_tiles);
    case EPI_F32: return launch_epi<EPI_F32>(s, cfg, g, splits, tail, row_tiles);
    case EPI_RESID_F32: return launch_epi<EPI_RESID_F32>(s, cfg, g, splits, tail, row_tiles);
    case EPI_SWIGLU_BF16: return launch_epi<EPI_SWIGLU_BF16>(s, cfg, g, 1, tail, row_tiles);
    case EPI_QKV: return launch_rows<EPI_QKV>(s, g, 1, tail, row_tiles, 8);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace sts
