// GEMMs of 1 to 256 rows, gfx950: a workgroup takes all the rows and 128 columns, so that every weight byte is asked for once. For decode steps of 17
// rows and more on large partitions (fewer take gemm_kslice.hip) and prefill batches on the whole GPU.
//
// What bounds them is what a CU pulls: about 256 lines of 128 bytes are under way at a time, whatever instruction asks for them, which
// is 57 GB/s of lines that come from HBM (63 with the non-temporal hint), 103 from the memory-side cache and 140 from L2, and lines
// come back in their order, so that activations from L2 wait behind weights from HBM. A CU's time therefore is its rows plus its
// columns times K. Tiles of 256 columns in two row tiles ask for every weight line twice, and may not use the hint, because the
// second reader wants the line in L2. Operand loads alone, 28672 x 4096 on 224 CUs: two tiles of 160 rows 69 us, one of 320 rows x 128
// columns 60; two of 128 rows 68, one of 224 rows 52, of 128 rows 46, of 64 rows 40 (HBM: 36).
//
// Four waves, one per SIMD, 32 columns each (16 gate and their 16 up columns in the SwiGLU form). Activations go global -> LDS directly
// (rows of 128 bytes, 16-byte chunks swizzled as in gemm.hip), W from the packed layout straight into registers, both PD K tiles ahead with
// one wait and one barrier a K tile. Loads go through buffer descriptors: rows past M and tiles past the range lie behind the
// descriptor's end, return zero and fetch nothing, so that every iteration queues the same number of operations and the waits need no cases.
// How deep PD is hardly matters (2 to 6 within 3 %), because the lines under way are the limit.
//
// A row's sum keeps the order of the split GEMM: the chain along a slice of K, the slices added in their order. A workgroup either owns
// one slice and leaves its fp32 partial sums, as the tiles of gemm.hip do, or (SwiGLU) goes through all slices and adds them up in registers:
// no partial sums and no kernel that reads them. Both give the same bits as the tiles.
//
// In the engine, 256 CUs, hidden 4096, tiles / this: gate/up with SwiGLU 64 rows 52 / 40 us (HBM floor 36), 96 rows 69 / 45, 128 rows 74 / 50, 160 rows
// 68 / 52, 223 rows 78 / 61, 256 rows 81 / 67; down 64 rows 26.0 / 25.4, 96 rows 34 / 28, 192 rows 39 / 35; hidden 8192: down of 24 rows 80 / 70 us (470 MB),
// gate/up of 96 rows 202 / 161.
#include "kernels.h"

namespace sts {

namespace {

struct ColsArgs {
  const bf16* A; const bf16* W; void* C;
  int lda, ldc, M, K;
  int per, slices;            // K tiles of a slice, slices of the whole K
  long long split_stride;
};

// Buffer descriptor of `bytes` bytes from p on: loads past them return zero and read nothing.
__device__ __forceinline__ u32x4 buffer_of(const void* p, unsigned bytes) {
  const unsigned long long a = (unsigned long long)p;
  u32x4 r = {(unsigned)a, (unsigned)(a >> 32) & 0xffffu, bytes, 0x00020000u};
#pragma unroll
  for (int i = 0; i < 4; i++) r[i] = (unsigned)__builtin_amdgcn_readfirstlane((int)r[i]);
  return r;
}
constexpr unsigned PAST_END = 0x80000000u;     // PAST_END / 2 and PAST_END, alone, added up or with an offset inside a buffer, lie behind every buffer here
template <int OFF>
__device__ __forceinline__ void buf_load_nt(bf16x8& dst, u32x4 rsrc, unsigned off) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("buffer_load_dwordx4 %0, %1, %2, 0 offen offset:%3 nt" : "=v"(dst) : "v"(off), "s"(rsrc), "n"(OFF) : "memory");
#endif
}
__device__ __forceinline__ void buf_to_lds(u32x4 rsrc, unsigned off, unsigned lds) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds" ::"v"(off), "s"(rsrc), "s"(lds) : "memory");
#endif
}
template <int N>
__device__ __forceinline__ void wait_for4(bf16x8& a, bf16x8& b, bf16x8& c, bf16x8& d) {
#if defined(__HIP_DEVICE_COMPILE__)
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
  asm volatile("s_waitcnt vmcnt(%4)" : "+v"(a), "+v"(b), "+v"(c), "+v"(d) : "n"(N) : "memory");
#endif
}

// K tiles ahead. By LDS and registers (98 to 126 of them up to 96 rows) a CU holds four workgroups that leave partial sums up to 32 rows, three up to 96, two up to
// 192 and one of more; which of that pays is the engine's to decide.
constexpr int cols_pd(int tm) { return tm <= 2 ? 4 : tm <= 4 ? 3 : 2; }
constexpr int COLS_BASE = 1024;                // buffers filled by direct-to-LDS loads stay clear of address 0
constexpr int cols_lds(int tm) { return COLS_BASE + (cols_pd(tm) + 1) * tm * 4096; }
static_assert(2 * cols_lds(6) <= 160 * 1024 && cols_lds(8) <= 160 * 1024, "workgroups of a CU");

// Order of a wave's vector-memory operations (they complete in order): iteration t queues the TM pieces of A of tile t + PD behind the barrier, and
// the W operands of tile t + PD, a step's two behind the products that used their registers. When tile t begins, those of the PD - 1 tiles
// after it may be under way. A(t + PD) goes into the stage of tile t - 1, whose reads every wave has used in products before that barrier.
template <int TM, int EPI>
__global__ void __launch_bounds__(256, EPI == EPI_F32 ? 2 : 1) gemm_cols_kernel(ColsArgs g) {
  constexpr int PD = cols_pd(TM), NS = PD + 1, RB = 2 * TM, STAGE = TM * 4096, PER_TILE = TM + 4;
  constexpr bool SW = EPI == EPI_SWIGLU_BF16;
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* arena = smem + COLS_BASE;
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ksteps = g.K >> 6;
  const int tiles = (int)gridDim.x / (SW ? 1 : g.slices);
  const int v = gridDim.x % 8 == 0 ? xcd_contiguous(blockIdx.x, gridDim.x >> 3) : (int)blockIdx.x;   // slice by slice, neighbouring columns on one XCD
  const int z = SW ? 0 : v / tiles, tn = SW ? v : v % tiles;
  const int k0 = z * g.per, nk = (SW ? ksteps : min(ksteps, k0 + g.per)) - k0;

  // W: four 32-row blocks of the packed layout
  const unsigned wrow = (unsigned)ksteps * 4096u;
  const u32x4 wbuf = buffer_of(reinterpret_cast<const unsigned char*>(g.W) + (size_t)tn * 4 * wrow, 4 * wrow);
  const u32x4 abuf = buffer_of(g.A, (unsigned)g.M * (unsigned)g.lda * 2u);
  unsigned w_off[2], a_off[TM];
#pragma unroll
  for (int j = 0; j < 2; j++) {
    const unsigned blk = SW ? 2 * (wave >> 1) + j : wave, half = SW ? wave & 1 : j;
    w_off[j] = blk * wrow + (unsigned)k0 * 4096u + (unsigned)((lq >> 1) * 1024 + (lq & 1) * 512) + (half * 16 + l16) * 16u;
  }
#pragma unroll
  for (int j = 0; j < TM; j++) {
    const int q = (j * 4 + wave) * 64 + lane, row = q >> 3, ch = (q & 7) ^ ((row >> 1) & 7);
    a_off[j] = row < g.M ? (unsigned)row * (unsigned)g.lda * 2u + (unsigned)k0 * 128u + ch * 16u : PAST_END;
  }
  const unsigned arena_lds = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)arena + wave * 1024;

  bf16x8 w[PD][2][2];
#pragma unroll
  for (int s = 0; s < PD; s++)
#pragma unroll
    for (int kk = 0; kk < 2; kk++)
#pragma unroll
      for (int j = 0; j < 2; j++)
#pragma unroll
        for (int e = 0; e < 8; e++) w[s][kk][j][e] = 0;
  // The tile that is being fetched: its K tile of the workgroup's range, or past the end of everything. A slice is rounded up to PD
  // tiles, the surplus ones fetch nothing and are not multiplied.
  const int my_slices = SW ? g.slices : 1, pad = (min(g.per, nk) + PD - 1) / PD * PD;
  int f_tile = 0, f_left = min(g.per, nk), f_slot = 0;       // next K tile, tiles left of its slice, place in the rounded slice
  auto fetched = [&] {                                       // on to the next one
    f_tile += f_left > 0; f_left--;
    if (++f_slot == pad) { f_slot = 0; f_left = min(g.per, nk - f_tile); }
  };
  auto load_a = [&](unsigned stage) {
    const unsigned k = f_left > 0 ? (unsigned)f_tile * 128u : PAST_END / 2;
#pragma unroll
    for (int j = 0; j < TM; j++) buf_to_lds(abuf, a_off[j] + k, arena_lds + stage + j * 4096);
  };
  auto load_w = [&](auto kk_c, bf16x8 (&dst)[2]) {
    constexpr int kk = decltype(kk_c)::value;
    const unsigned k = f_left > 0 ? (unsigned)f_tile * 4096u : PAST_END / 2;
#pragma unroll
    for (int j = 0; j < 2; j++) buf_load_nt<kk * 2048>(dst[j], wbuf, w_off[j] + k);
  };
  f32x4 acc[RB][2], tot[SW ? RB : 1][2];
  auto clear = [&] {
#pragma unroll
    for (int i = 0; i < RB; i++)
#pragma unroll
      for (int j = 0; j < 2; j++) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  clear();
  if constexpr (SW) {
#pragma unroll
    for (int i = 0; i < RB; i++)
#pragma unroll
      for (int j = 0; j < 2; j++) tot[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  static_for<PD>([&](auto s_c) {
    constexpr int s = decltype(s_c)::value;
    load_a(s * STAGE);
    load_w(std::integral_constant<int, 0>{}, w[s][0]);
    load_w(std::integral_constant<int, 1>{}, w[s][1]);
    fetched();
  });
  const int koff0 = (lq ^ ((l16 >> 1) & 7)) * 16;
  const unsigned char* rd0 = arena + l16 * 128 + koff0;
  const unsigned char* rd1 = arena + l16 * 128 + (koff0 ^ 64);
  unsigned cur = 0, into = PD * STAGE;
  for (int sl = 0; sl < my_slices; sl++) {
    const int len = min(g.per, nk - sl * g.per);
    for (int t0 = 0; t0 < pad; t0 += PD) {
      static_for<PD>([&](auto s_c) {
        constexpr int s = decltype(s_c)::value;
        const int t = t0 + s;
        __builtin_amdgcn_sched_barrier(0);
        wait_for4<(PD - 1) * PER_TILE>(w[s][0][0], w[s][0][1], w[s][1][0], w[s][1][1]);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        load_a(into);
        __builtin_amdgcn_sched_barrier(0);
        static_for<2>([&](auto kk_c) {
          constexpr int kk = decltype(kk_c)::value;
          if (t < len) {
            const unsigned char* p = (kk ? rd1 : rd0) + cur;
            bf16x8 af[RB];
#pragma unroll
            for (int i = 0; i < RB; i++) af[i] = *reinterpret_cast<const bf16x8*>(p + i * 2048);
#pragma unroll
            for (int i = 0; i < RB; i++)
#pragma unroll
              for (int j = 0; j < 2; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[s][kk][j], af[i], acc[i][j], 0, 0, 0);
            // four reads ahead of the products
            constexpr int AHEAD = RB < 4 ? RB : 4;
            __builtin_amdgcn_sched_group_barrier(0x100, AHEAD, 0);
#pragma unroll
            for (int i = 0; i < RB - AHEAD; i++) {
              __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
              __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
            __builtin_amdgcn_sched_group_barrier(0x008, 2 * AHEAD, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
          load_w(kk_c, w[s][kk]);
          __builtin_amdgcn_sched_barrier(0);
        });
        fetched();
        cur = cur + STAGE == NS * STAGE ? 0 : cur + STAGE;
        into = into + STAGE == NS * STAGE ? 0 : into + STAGE;
      });
    }
    if constexpr (SW) {                                      // a slice is complete: its sum joins those before it
#pragma unroll
      for (int i = 0; i < RB; i++)
#pragma unroll
        for (int j = 0; j < 2; j++) tot[i][j] += acc[i][j];
      clear();
    }
  }
  // nothing of the surplus loads may land in what the epilogue uses
#pragma unroll
  for (int s = 0; s < PD; s++) wait_for4<0>(w[s][0][0], w[s][0][1], w[s][1][0], w[s][1][1]);

  if constexpr (SW) {
    constexpr int RS = 64 + 8;
    bf16* img = reinterpret_cast<bf16*>(arena);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < RB; i++) {
      bf16x4 o;
#pragma unroll
      for (int e = 0; e < 4; e++) o[e] = f2bf(swiglu(tot[i][0][e], tot[i][1][e]));
      *reinterpret_cast<bf16x4*>(img + (i * 16 + l16) * RS + wave * 16 + lq * 4) = o;
    }
    __syncthreads();
    bf16* out = reinterpret_cast<bf16*>(g.C) + (size_t)tn * 64;
#pragma unroll
    for (int c = 0; c < TM; c++) {
      const int q = c * 256 + tid, row = q >> 3, cc = q & 7;
      if (row < g.M) *reinterpret_cast<u32x4*>(out + (size_t)row * g.ldc + cc * 8) = *reinterpret_cast<const u32x4*>(img + row * RS + cc * 8);
    }
  } else {
    // a row block at a time through a piece of LDS of the wave's own, so that whole 128-byte lines are stored
    constexpr int RS = 32 + 4;
    float* img = reinterpret_cast<float*>(arena) + wave * 2 * 16 * RS;
    float* out = reinterpret_cast<float*>(g.C) + (size_t)z * g.split_stride + (size_t)tn * 128 + wave * 32 + (lane & 7) * 4;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < RB; i++) {
      float* im = img + (i & 1) * 16 * RS;
#pragma unroll
      for (int j = 0; j < 2; j++) *reinterpret_cast<f32x4*>(im + l16 * RS + j * 16 + lq * 4) = acc[i][j];
#pragma unroll
      for (int h = 0; h < 2; h++) {
        const int r = h * 8 + (lane >> 3), row = i * 16 + r;
        const f32x4 v = *reinterpret_cast<const f32x4*>(im + r * RS + (lane & 7) * 4);
        if (row < g.M) *reinterpret_cast<f32x4*>(out + (size_t)row * g.ldc) = v;
      }
    }
  }
}

template <int TM, int EPI>
hipError_t launch_cols(hipStream_t s, const ColsArgs& g, int grid) {
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_cols_kernel<TM, EPI>), hipFuncAttributeMaxDynamicSharedMemorySize, cols_lds(TM));
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL((gemm_cols_kernel<TM, EPI>), dim3(grid), dim3(256), cols_lds(TM), s, g);
  return hipGetLastError();
}
template <int EPI>
hipError_t launch_cols_rows(hipStream_t s, const ColsArgs& g, int grid) {
  switch ((g.M + 31) / 32) {
    case 1: return launch_cols<1, EPI>(s, g, grid);
    case 2: return launch_cols<2, EPI>(s, g, grid);
    case 3: return launch_cols<3, EPI>(s, g, grid);
    case 4: return launch_cols<4, EPI>(s, g, grid);
    case 5: return launch_cols<5, EPI>(s, g, grid);
    case 6: return launch_cols<6, EPI>(s, g, grid);
    case 7: return launch_cols<7, EPI>(s, g, grid);
    case 8: return launch_cols<8, EPI>(s, g, grid);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

// A [M, lda] row-major, W [N, K] packed. EPI_F32: C + z * split_stride = the partial sums of slice z, `splits` slices of K as
// gemm_bf16 makes them (fewer where K has not as many tiles). EPI_SWIGLU_BF16: C[M, N / 2] = silu(gate) * up of the slices' sums.
hipError_t gemm_cols(hipStream_t s, int epi, const bf16* A, int lda, const bf16* W, void* C, int ldc, int M, int N, int K, int splits, long long split_stride) {
  if (!A || !W || !C || M < 1 || M > COLS_MAX_ROWS || N < 128 || N % 128 != 0 || K < 64 || K % 64 != 0 || lda < K || lda % 8 != 0 || splits < 1) return hipErrorInvalidValue;
  if ((epi != EPI_F32 && epi != EPI_SWIGLU_BF16) || ldc % (epi == EPI_F32 ? 4 : 8) != 0 || (epi == EPI_F32 && splits > 1 && split_stride % 4 != 0)) return hipErrorInvalidValue;
  if ((unsigned long long)M * lda * 2 >= PAST_END / 4 || (unsigned long long)K * 256 >= PAST_END / 4) return hipErrorInvalidValue;      // 32-bit byte offsets
  ColsArgs g{};
  g.A = A; g.W = W; g.C = C; g.lda = lda; g.ldc = ldc; g.M = M; g.K = K; g.split_stride = split_stride;
  const int ksteps = K / 64;
  g.per = (ksteps + splits - 1) / splits;
  g.slices = (ksteps + g.per - 1) / g.per;
  return epi == EPI_F32 ? launch_cols_rows<EPI_F32>(s, g, N / 128 * g.slices) : launch_cols_rows<EPI_SWIGLU_BF16>(s, g, N / 128);
}

}  // namespace sts
