// Decode GEMMs that finish their own output, for up to 16 rows on a large partition, gfx950.
//
// A decode GEMM streams its weights once. Cutting K over workgroups to keep a large partition busy leaves fp32
// partial sums in memory and a second kernel to add them up; at a few rows those kernels (4 to 6 us each: launch and
// memory latency) were a fifth of a layer. Here K is cut over the waves of ONE workgroup: it owns 16 or 32 columns and
// the whole K, wave w takes the 64-wide K tiles w, w + NW, ..., and the waves' accumulators meet in LDS. The workgroup
// then has its columns' results and finishes them itself: residual add, SwiGLU, rotary embedding and KV append, logits.
// 16 columns make 256 workgroups of a 4096-wide output (one per CU), which 32-column tiles leave half idle.
//
// RMSNorm needs whole rows, which no workgroup has. The residual epilogue therefore leaves the row scaled by the
// gains only, bf16(x * g), and each workgroup's share of the row's sum of squares; the next GEMM's workgroups add the shares
// (in a fixed order) while their first weights are on the way and multiply their results by 1 / rms: a row factor
// commutes with the product.
//
// Bound by memory: both operands go straight to registers, PD K tiles deep (W from the packed layout with the non-temporal
// hint; the activations as 16-byte pieces of row-major rows, which stay in L2). What limits the shape's range is what a CU
// can pull (58 GB/s): every workgroup reads the activations of the whole K for 16 or 32 columns, so above 16 rows, or on a
// small partition, the wide tiles of gemm.hip move fewer bytes per CU (decode_layer_plan in engine.hip has the estimate).
// One row on 256 CUs, weights from HBM, against the split GEMM (without its reduce kernel): 6144 x 4096 9.6 us (11.7),
// 4096 x 4096 7.4 (8.4), 28672 x 4096 37.1 (40.0, 6.3 TB/s), 4096 x 14336 19.1 (21.7), 1024 x 4096 5.7 (33 unsplit).
#include "kernels.h"

namespace sts {

namespace {

struct KsArgs {
  const bf16* A; const bf16* W;
  int lda, M, N, K;
  const float* ssq; int ssq_parts; float eps;        // row factor 1 / sqrt(sum of the shares / K + eps); no factor if ssq is null
  // outputs, by epilogue
  void* C; int ldc;                                  // logits (fp32) or MLP hidden (bf16)
  float* X; const float* gain; bf16* Xg; float* ssq_out;
  const int* place; const float* rot; bf16* q_out; bf16* pool; KvGeom geo; int n_q;
};

// CB: 16-column blocks per workgroup; NW waves; PD K tiles in flight per wave.
template <int CB, int NW, int PD, int EPI>
__global__ void __launch_bounds__(NW * 64, 4) gemm_kslice_kernel(KsArgs g) {
  constexpr int ROWS = 16, COLS = CB * 16, NT = NW * 64, RS = COLS + 4;
  constexpr int RPW = (ROWS + NW - 1) / NW;                  // rows whose sums of squares a wave adds up
  __shared__ __align__(16) float red[NW][ROWS][RS];
  __shared__ float inv_rms[ROWS];
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, lq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int blk = blockIdx.x;
  const int nk = g.K >> 6;

  // what the epilogue reads beside the sums is requested first
  constexpr int CPR = COLS / 4, CHUNKS = ROWS * CPR, XCH = EPI == KS_RESID ? (CHUNKS + NT - 1) / NT : 1;
  f32x4 xr[XCH], gr;
  if constexpr (EPI == KS_RESID) {
    static_assert(CHUNKS % NT == 0 || CHUNKS < NT, "whole passes of column chunks, or one");
#pragma unroll
    for (int i = 0; i < XCH; i++) {
      const int c = tid + i * NT, row = min(c / CPR, g.M - 1);
      xr[i] = *reinterpret_cast<const f32x4*>(g.X + (size_t)row * g.N + blk * COLS + c % CPR * 4);
    }
    gr = *reinterpret_cast<const f32x4*>(g.gain + blk * COLS + tid % CPR * 4);
  }
  float sq[RPW];
  if (g.ssq) {
#pragma unroll
    for (int i = 0; i < RPW; i++) {
      const float* p = g.ssq + (size_t)min(wave * RPW + i, g.M - 1) * g.ssq_parts;
      float s = 0.f;
      for (int c0 = 0; c0 < g.ssq_parts; c0 += 256) {        // four loads in flight
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; e++) v[e] = c0 + e * 64 + lane < g.ssq_parts ? p[c0 + e * 64 + lane] : 0.f;
        s += (v[0] + v[1]) + (v[2] + v[3]);
      }
      sq[i] = s;
    }
  }

  // A 64-wide K tile is two matrix-core steps of 32; lane (lq, l16) of step s holds k 32 s + 8 lq .. + 8 of row or column l16: in
  // the packed layout piece 2 s + lq / 2, half lq % 2. The QKV form's two column blocks are 16 rotation pairs of one
  // head: 16 elements of its first half and their partners half a head further.
  unsigned w_off[CB];
#pragma unroll
  for (int j = 0; j < CB; j++) {
    int col;
    if constexpr (EPI == KS_QKV) {
      const int d = g.geo.d, per = d >> 5;
      col = blk / per * d + 16 * (blk % per) + j * (d >> 1) + l16;
    } else if constexpr (EPI == KS_SWIGLU) {
      col = (blk >> 1) * 64 + j * 32 + (blk & 1) * 16 + l16;  // gate and up rows alternate in blocks of 32
    } else {
      col = blk * COLS + j * 16 + l16;
    }
    w_off[j] = (unsigned)(col >> 5) * (unsigned)nk * 4096u + (unsigned)((lq >> 1) * 1024 + (lq & 1) * 512 + (col & 31) * 16);
  }
  const unsigned a_off = ((unsigned)min(l16, g.M - 1) * (unsigned)g.lda + lq * 8) * 2u;

  u32x4 w[PD][CB][2], a[PD][2];
  auto load = [&](int s, int t) {                            // operands of this wave's t-th K tile
    const size_t kt = wave + (size_t)t * NW;
    const unsigned char* wb = reinterpret_cast<const unsigned char*>(g.W) + kt * 4096;
    const unsigned char* ab = reinterpret_cast<const unsigned char*>(g.A) + kt * 128;
#pragma unroll
    for (int j = 0; j < CB; j++)
#pragma unroll
      for (int kk = 0; kk < 2; kk++) w[s][j][kk] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(wb + w_off[j] + kk * 2048));
#pragma unroll
    for (int kk = 0; kk < 2; kk++) a[s][kk] = *reinterpret_cast<const u32x4*>(ab + a_off + kk * 64);
  };
  f32x4 acc[CB];
#pragma unroll
  for (int j = 0; j < CB; j++) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](int s) {
#pragma unroll
    for (int kk = 0; kk < 2; kk++)
#pragma unroll
      for (int j = 0; j < CB; j++)
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[s][kk]), __builtin_bit_cast(bf16x8, w[s][j][kk]), acc[j], 0, 0, 0);
  };
  auto row_factors = [&] {
    if (g.ssq) {
#pragma unroll
      for (int i = 0; i < RPW; i++) {
        const float s = wave_sum(sq[i]);
        if (lane == 0 && wave * RPW + i < ROWS) inv_rms[wave * RPW + i] = rsqrtf(s / (float)g.K + g.eps);
      }
    } else if (tid < ROWS) {
      inv_rms[tid] = 1.f;
    }
  };

  const int cnt = wave < nk ? (nk - wave + NW - 1) / NW : 0;  // this wave's K tiles
  if (cnt >= PD) {
#pragma unroll
    for (int s = 0; s < PD; s++) load(s, s);
    __builtin_amdgcn_sched_barrier(0);
    row_factors();
    int t = 0;
    for (; t + 2 * PD <= cnt; t += PD) {
#pragma unroll
      for (int s = 0; s < PD; s++) {
        compute(s);
        __builtin_amdgcn_sched_barrier(0);
        load(s, t + s + PD);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    const int rest = cnt - t - PD;                            // tiles not requested yet, fewer than PD
#pragma unroll
    for (int s = 0; s < PD; s++) {
      compute(s);
      if (s < rest) load(s, t + s + PD);
    }
#pragma unroll
    for (int s = 0; s < PD - 1; s++)
      if (s < rest) compute(s);
  } else {
    row_factors();
#pragma unroll
    for (int s = 0; s < PD - 1; s++)
      if (s < cnt) load(s, s);
#pragma unroll
    for (int s = 0; s < PD - 1; s++)
      if (s < cnt) compute(s);
  }

  // ---- the waves' sums meet in LDS and are added up in order
#pragma unroll
  for (int j = 0; j < CB; j++)
#pragma unroll
    for (int r = 0; r < 4; r++) red[wave][4 * lq + r][j * 16 + l16] = acc[j][r];
  __syncthreads();
  auto sum4 = [&](int row, int col) {
    f32x4 v = *reinterpret_cast<const f32x4*>(&red[0][row][col]);
#pragma unroll
    for (int z = 1; z < NW; z++) v += *reinterpret_cast<const f32x4*>(&red[z][row][col]);
    return v * inv_rms[row];
  };

  if constexpr (EPI == KS_F32) {
    for (int c = tid; c < CHUNKS; c += NT) {
      const int row = c / CPR, col = c % CPR * 4;
      if (row < g.M) *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(g.C) + (size_t)row * g.ldc + blk * COLS + col) = sum4(row, col);
    }
  } else if constexpr (EPI == KS_RESID) {
#pragma unroll
    for (int i = 0; i < XCH; i++) {
      const int c = tid + i * NT, row = c / CPR, col = c % CPR * 4;
      if (c >= CHUNKS) break;                                // whole waves
      const f32x4 x = xr[i] + sum4(row, col);
      float s = x[0] * x[0] + x[1] * x[1] + x[2] * x[2] + x[3] * x[3];
#pragma unroll
      for (int o = 1; o < CPR; o <<= 1) s += __shfl_xor(s, o, 64);
      if (row < g.M) {
        const size_t at = (size_t)row * g.N + blk * COLS + col;
        *reinterpret_cast<f32x4*>(g.X + at) = x;
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; e++) o[e] = f2bf(x[e] * gr[e]);
        *reinterpret_cast<bf16x4*>(g.Xg + at) = o;
        if (col == 0) g.ssq_out[(size_t)row * gridDim.x + blk] = s;
      }
    }
  } else if constexpr (EPI == KS_SWIGLU) {
    for (int c = tid; c < ROWS * 4; c += NT) {
      const int row = c >> 2, col = (c & 3) * 4;
      if (row >= g.M) continue;
      const f32x4 gate = sum4(row, col), up = sum4(row, COLS - 16 + col);
      bf16x4 o;
#pragma unroll
      for (int e = 0; e < 4; e++) o[e] = f2bf(swiglu(gate[e], up[e]));
      *reinterpret_cast<bf16x4*>(reinterpret_cast<bf16*>(g.C) + (size_t)row * g.ldc + blk * 16 + col) = o;
    }
  } else {
    const int d = g.geo.d, half = d >> 1, per = d >> 5, head = blk / per, u = blk % per;
    for (int c = tid; c < ROWS * 4; c += NT) {
      const int row = c >> 2, i0 = (c & 3) * 4, e0 = 16 * u + i0;
      if (row >= g.M) continue;
      const f32x4 a4 = sum4(row, i0), b4 = sum4(row, 16 + i0);
      const int place = head < g.n_q ? 0 : g.place[row], page = place >> 4, slot = place & 15;
      if (head >= g.n_q + g.geo.n_kv) {
        bf16* v = g.pool + ((size_t)page * g.geo.n_kv + (head - g.n_q - g.geo.n_kv)) * g.geo.head_elems() + (size_t)g.geo.page_tokens * d;
#pragma unroll
        for (int e = 0; e < 4; e++) {
          v[(size_t)(e0 + e) * g.geo.page_tokens + slot] = f2bf(a4[e]);
          v[(size_t)(half + e0 + e) * g.geo.page_tokens + slot] = f2bf(b4[e]);
        }
        continue;
      }
      const f32x4 cs = *reinterpret_cast<const f32x4*>(g.rot + (size_t)row * d + e0), sn = *reinterpret_cast<const f32x4*>(g.rot + (size_t)row * d + half + e0);
      bf16x4 ya, yb;
#pragma unroll
      for (int e = 0; e < 4; e++) {
        // the projection's result is rounded to bf16 before the rotation, as in the prefill path
        float ra, rb;
        rotate_pair(bf2f(f2bf(a4[e])), bf2f(f2bf(b4[e])), cs[e], sn[e], &ra, &rb);
        ya[e] = f2bf(ra);
        yb[e] = f2bf(rb);
      }
      bf16* dst = head < g.n_q ? g.q_out + (size_t)row * g.n_q * d + head * d
                               : g.pool + ((size_t)page * g.geo.n_kv + (head - g.n_q)) * g.geo.head_elems() + (size_t)slot * d;
      *reinterpret_cast<bf16x4*>(dst + e0) = ya;
      *reinterpret_cast<bf16x4*>(dst + half + e0) = yb;
    }
  }
}

template <int CB, int NW, int PD, int EPI>
hipError_t launch_ks(hipStream_t s, const KsArgs& g, int grid) {
  hipLaunchKernelGGL((gemm_kslice_kernel<CB, NW, PD, EPI>), dim3(grid), dim3(NW * 64), 0, s, g);
  return hipGetLastError();
}

// Byte offsets into W and the activations are 32 bits wide; a workgroup reads rows up to M - 1 of A only.
bool fill(KsArgs* g, const KsliceIn& in) {
  if (!in.A || !in.W || in.M < 1 || in.M > KSLICE_MAX_ROWS || in.N < 64 || in.N % 64 != 0 || in.K < 64 || in.K % 64 != 0 || in.lda % 8 != 0 || in.lda < in.K) return false;
  if (!kslice_covers(in.N, in.K) || (in.scale.ssq && in.scale.parts < 1)) return false;
  *g = KsArgs{};
  g->A = in.A; g->W = in.W; g->lda = in.lda; g->M = in.M; g->N = in.N; g->K = in.K;
  g->ssq = in.scale.ssq; g->ssq_parts = in.scale.parts; g->eps = in.scale.eps;
  return true;
}

}  // namespace

// Columns per workgroup: 16 while 32-column tiles would leave CUs without a workgroup, else 32 (half the activation reads).
// The QKV and SwiGLU forms take 32 (16 rotation pairs, 16 gate/up pairs).
int kslice_cols(int epi, int n, int cus) { return epi == KS_QKV || epi == KS_SWIGLU || n / 32 >= cus ? 32 : 16; }

// C[M, ldc] (fp32) = A W^T, rows scaled.
hipError_t kslice_f32(hipStream_t s, const KsliceIn& in, int cus, float* C, int ldc) {
  KsArgs g;
  if (!fill(&g, in) || !C || ldc % 4 != 0 || ldc < in.N) return hipErrorInvalidValue;
  g.C = C; g.ldc = ldc;
  return kslice_cols(KS_F32, in.N, cus) == 16 ? launch_ks<1, 16, 3, KS_F32>(s, g, in.N / 16) : launch_ks<2, 16, 2, KS_F32>(s, g, in.N / 32);
}
// X[M, N] += A W^T; Xg = bf16(X * gain); ssq_out[row][N / kslice_cols(..)]: the workgroups' shares of the rows' sums of squares.
hipError_t kslice_resid(hipStream_t s, const KsliceIn& in, int cus, float* X, const float* gain, bf16* Xg, float* ssq_out) {
  KsArgs g;
  if (!fill(&g, in) || !X || !gain || !Xg || !ssq_out) return hipErrorInvalidValue;
  g.X = X; g.gain = gain; g.Xg = Xg; g.ssq_out = ssq_out;
  return kslice_cols(KS_RESID, in.N, cus) == 16 ? launch_ks<1, 8, 4, KS_RESID>(s, g, in.N / 16) : launch_ks<2, 16, 3, KS_RESID>(s, g, in.N / 32);
}
// H[M, N / 2] = silu(gate) * up; gate and up rows of W alternate in blocks of 32.
hipError_t kslice_swiglu(hipStream_t s, const KsliceIn& in, bf16* H) {
  KsArgs g;
  if (!fill(&g, in) || !H) return hipErrorInvalidValue;
  g.C = H; g.ldc = in.N / 2;
  return launch_ks<2, 8, 2, KS_SWIGLU>(s, g, in.N / 32);
}
// The QKV projection of one new token per request, rotated (rot: [M][d / 2 cosines | d / 2 sines] of the requests' positions), q to
// q_out, k and v appended to the requests' pages.
hipError_t kslice_qkv(hipStream_t s, const KsliceIn& in, const int* place, const float* rot, bf16* q_out, bf16* pool, KvGeom geo, int n_q) {
  KsArgs g;
  if (!fill(&g, in) || (geo.d != 64 && geo.d != 128) || in.N != (n_q + 2 * geo.n_kv) * geo.d || geo.page_tokens != 16) return hipErrorInvalidValue;
  g.place = place; g.rot = rot; g.q_out = q_out; g.pool = pool; g.geo = geo; g.n_q = n_q;
  return launch_ks<2, 16, 2, KS_QKV>(s, g, in.N / 32);
}

}  // namespace sts
