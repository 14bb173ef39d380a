// Memory-bound kernels between the contractions: weight generation, embedding, RMSNorm,
// rotary embedding + KV page writes, split-K reductions fused with residual/norm/SwiGLU,
// greedy argmax, and the copy kernel used as the bandwidth probe.
#include <type_traits>

#include "kernels.h"

namespace sts {

// ------------------------------------------------------------------ counter-based generator
// Twelve-term Irwin-Hall approximation of a normal deviate from three 64-bit hashes of
// (seed, tensor id, element index): integer arithmetic plus one fp32 multiply, so a host
// implementation of the same recipe reproduces every value exactly.
__host__ __device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z += 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
__device__ __forceinline__ int irwin_hall12(uint64_t base, uint64_t i) {
  int s = 0;
#pragma unroll
  for (int j = 0; j < 3; j++) {
    uint64_t r = mix64(base ^ (4 * i + j));
    s += (int)(r & 0xFFFF) + (int)((r >> 16) & 0xFFFF) + (int)((r >> 32) & 0xFFFF) + (int)(r >> 48);
  }
  return s - 393210;
}

__device__ __forceinline__ int phys_row(int r, int row_offset, int ib, int phase) {
  return ib > 0 ? (r / ib) * 2 * ib + phase * ib + r % ib : row_offset + r;
}

// Where element (physical row r, column c) of a weight matrix with ld columns lives. Row-major, or the
// packed layout of the GEMM weights (weight_packed_index in kernels.h).
__device__ __forceinline__ size_t weight_elem(int r, int c, int ld, int packed) {
  return packed ? weight_packed_index(r, c, ld) : (size_t)r * ld + c;
}

__global__ void init_weight_kernel(bf16* dst, int ld, uint64_t base, int rows, int cols, int row_offset, int ib, int phase, int packed) {
  size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i >= (size_t)rows * cols) return;
  int r = (int)(i / cols), c = (int)(i % cols);
  float w = (float)irwin_hall12(base, i) * 0.02f * 1.52587890625e-05f;   // * 2^-16, exact
  dst[weight_elem(phys_row(r, row_offset, ib, phase), c, ld, packed)] = f2bf(w);
}
hipError_t init_weight(hipStream_t s, bf16* dst, int ld, uint64_t seed, uint64_t tensor_id, int rows, int cols,
                       int row_offset, int ib, int phase, int packed) {
  size_t n = (size_t)rows * cols;
  uint64_t base = mix64(seed ^ mix64(tensor_id));
  hipLaunchKernelGGL(init_weight_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, dst, ld, base, rows, cols, row_offset, ib, phase, packed);
  return hipGetLastError();
}

__global__ void convert_weight_kernel(bf16* dst, int ld, const float* src, int rows, int cols, int row_offset, int ib, int phase, int packed) {
  size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i >= (size_t)rows * cols) return;
  int r = (int)(i / cols), c = (int)(i % cols);
  dst[weight_elem(phys_row(r, row_offset, ib, phase), c, ld, packed)] = f2bf(src[i]);
}
hipError_t convert_weight(hipStream_t s, bf16* dst, int ld, const float* src, int rows, int cols, int row_offset, int ib, int phase, int packed) {
  size_t n = (size_t)rows * cols;
  hipLaunchKernelGGL(convert_weight_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, dst, ld, src, rows, cols, row_offset, ib, phase, packed);
  return hipGetLastError();
}
__global__ void export_weight_kernel(float* dst, const bf16* src, int ld, int rows, int cols, int row_offset, int ib, int phase, int packed) {
  size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i >= (size_t)rows * cols) return;
  int r = (int)(i / cols), c = (int)(i % cols);
  dst[i] = bf2f(src[weight_elem(phys_row(r, row_offset, ib, phase), c, ld, packed)]);
}
hipError_t export_weight(hipStream_t s, float* dst, const bf16* src, int ld, int rows, int cols, int row_offset, int ib, int phase, int packed) {
  size_t n = (size_t)rows * cols;
  hipLaunchKernelGGL(export_weight_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, dst, src, ld, rows, cols, row_offset, ib, phase, packed);
  return hipGetLastError();
}

__global__ void fill_f32_kernel(float* dst, float v, size_t n) {
  size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i < n) dst[i] = v;
}
hipError_t fill_f32(hipStream_t s, float* dst, float v, size_t n) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(fill_f32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, dst, v, n);
  return hipGetLastError();
}

// ------------------------------------------------------------------ embedding
__global__ void embed_kernel(float* X, const bf16* emb, const int* tokens, int h) {
  const int row = blockIdx.x;
  const bf16* e = emb + (size_t)tokens[row] * h;
  for (int c = threadIdx.x * 8; c < h; c += blockDim.x * 8) {
    bf16x8 v = *reinterpret_cast<const bf16x8*>(e + c);
    float* o = X + (size_t)row * h + c;
#pragma unroll
    for (int j = 0; j < 8; j++) o[j] = bf2f(v[j]);
  }
}
hipError_t embed_rows(hipStream_t s, float* X, const bf16* emb, const int* tokens, int n, int h) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(embed_kernel, dim3(n), dim3(256), 0, s, X, emb, tokens, h);
  return hipGetLastError();
}

// ------------------------------------------------------------------ RMSNorm
__device__ __forceinline__ float block_sum(float v, float* red) {   // red: one float per wave (<= 16)
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  float t = 0.f;
  for (int w = 0; w < (int)(blockDim.x >> 6); w++) t += red[w];
  __syncthreads();
  return t;
}

// A workgroup normalises R rows at once: all their loads are issued before the first reduction, so
// the launch is one round of latency-bound workgroups instead of two. Rows of up to 4096 * PER / 4
// elements stay in registers between the sum of squares and the scaling (PER 16-byte loads per
// thread and row); longer rows are read a second time.
template <int R, int PER>
__global__ void __launch_bounds__(256) rmsnorm_kernel(bf16* out, const float* X, const float* gain, float eps, int h, int n, const int* idx) {
  __shared__ float red[R][16];
  const int row0 = blockIdx.x * R;
  auto src_row = [&](int r) { const int q = min(r, n - 1); return idx ? idx[q] : q; };
  const bool in_regs = h <= 1024 * PER;
  f32x4 v[R][PER];
  float ss[R];
#pragma unroll
  for (int r = 0; r < R; r++) {
    ss[r] = 0.f;
    const float* x = X + (size_t)src_row(row0 + r) * h;
    if (in_regs) {
#pragma unroll
      for (int i = 0; i < PER; i++) {
        const int c = threadIdx.x * 4 + i * 1024;
        v[r][i] = c < h ? *reinterpret_cast<const f32x4*>(x + c) : f32x4{0.f, 0.f, 0.f, 0.f};
      }
    }
  }
#pragma unroll
  for (int r = 0; r < R; r++) {
    if (in_regs) {
#pragma unroll
      for (int i = 0; i < PER; i++) ss[r] += v[r][i][0] * v[r][i][0] + v[r][i][1] * v[r][i][1] + v[r][i][2] * v[r][i][2] + v[r][i][3] * v[r][i][3];
    } else {
      const float* x = X + (size_t)src_row(row0 + r) * h;
      for (int c = threadIdx.x * 4; c < h; c += 1024) {
        const f32x4 t = *reinterpret_cast<const f32x4*>(x + c);
        ss[r] += t[0] * t[0] + t[1] * t[1] + t[2] * t[2] + t[3] * t[3];
      }
    }
  }
  // block sums of the R rows with one pair of barriers
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int r = 0; r < R; r++) {
    const float w = wave_sum(ss[r]);
    if (lane == 0) red[r][wave] = w;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; r++) {
    if (row0 + r >= n) break;
    const float tot = red[r][0] + red[r][1] + red[r][2] + red[r][3];
    const float inv = rsqrtf(tot / (float)h + eps);
    const float* x = X + (size_t)src_row(row0 + r) * h;
    bf16* o_row = out + (size_t)(row0 + r) * h;
    if (in_regs) {
#pragma unroll
      for (int i = 0; i < PER; i++) {
        const int c = threadIdx.x * 4 + i * 1024;
        if (c < h) {
          const f32x4 g = *reinterpret_cast<const f32x4*>(gain + c);
          bf16x4 o;
#pragma unroll
          for (int j = 0; j < 4; j++) o[j] = f2bf(v[r][i][j] * inv * g[j]);
          *reinterpret_cast<bf16x4*>(o_row + c) = o;
        }
      }
    } else {
      for (int c = threadIdx.x * 4; c < h; c += 1024) {
        const f32x4 t = *reinterpret_cast<const f32x4*>(x + c);
        const f32x4 g = *reinterpret_cast<const f32x4*>(gain + c);
        bf16x4 o;
#pragma unroll
        for (int j = 0; j < 4; j++) o[j] = f2bf(t[j] * inv * g[j]);
        *reinterpret_cast<bf16x4*>(o_row + c) = o;
      }
    }
  }
}
// The rotation angles of a launch's rows are written once for all layers: cosines and sines of row's position, [row][d].
__device__ __forceinline__ void write_rotation(float* table, int row, int pos, const double* inv_freq, int half) {
  for (int i = threadIdx.x; i < half; i += blockDim.x) {
    double sv, cv;
    sincos((double)pos * inv_freq[i], &sv, &cv);
    table[(size_t)row * 2 * half + i] = (float)cv;
    table[(size_t)row * 2 * half + half + i] = (float)sv;
  }
}
__global__ void rotation_kernel(RowRotation rot) { write_rotation(rot.table, blockIdx.x, rot.pos[blockIdx.x], rot.inv_freq, rot.d >> 1); }
hipError_t row_rotation(hipStream_t s, const RowRotation& rot, int n) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(rotation_kernel, dim3(n), dim3(64), 0, s, rot);
  return hipGetLastError();
}
// Metadata from pinned host memory, read over the bus by the kernel itself: a runtime copy of these few KB left the stream idle
// for 15 to 30 us around it.
__global__ void __launch_bounds__(256) copy_in_kernel(MetaCopy meta) {
  const int i = (blockIdx.x * 256 + threadIdx.x) * 16;
  if (i < meta.bytes) *reinterpret_cast<u32x4*>(meta.dst + i) = *reinterpret_cast<const u32x4*>(meta.src + i);
}
hipError_t copy_in(hipStream_t s, const MetaCopy& meta) {
  if (meta.bytes == 0) return hipSuccess;
  hipLaunchKernelGGL(copy_in_kernel, dim3((meta.bytes + 4095) / 4096), dim3(256), 0, s, meta);
  return hipGetLastError();
}
// Embedding rows and the first layer's RMSNorm in one pass: the row is in registers anyway, so the residual stream
// (fp32) and its normalised bf16 copy are written together and the stream is not read back. One workgroup per row,
// 8 elements per thread and 2048-column slab, rows of up to 8192 elements.
__global__ void __launch_bounds__(256) embed_norm_kernel(float* X, bf16* out, const bf16* emb, const int* tokens, const float* gain, float eps, int h, int n,
                                                         RowRotation rot, MetaCopy meta) {
  constexpr int PER = 4;
  __shared__ float red[4];
  const int row = blockIdx.x;
  if (row >= n) {                                            // the blocks behind the rows copy the metadata for the kernels after this one
    const int i = ((row - n) * 256 + threadIdx.x) * 16;
    if (i < meta.bytes) *reinterpret_cast<u32x4*>(meta.dst + i) = *reinterpret_cast<const u32x4*>(meta.src + i);
    return;
  }
  const bf16* e = emb + (size_t)tokens[row] * h;
  bf16x8 v[PER];
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < PER; i++) {
    const int c = threadIdx.x * 8 + i * 2048;
    if (c < h) {
      v[i] = *reinterpret_cast<const bf16x8*>(e + c);
#pragma unroll
      for (int j = 0; j < 8; j++) { const float f = bf2f(v[i][j]); ss += f * f; }
    }
  }
  write_rotation(rot.table, row, rot.pos[row], rot.inv_freq, rot.d >> 1);      // while the row is on its way
  const float w = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = w;
  __syncthreads();
  const float inv = rsqrtf((red[0] + red[1] + red[2] + red[3]) / (float)h + eps);
#pragma unroll
  for (int i = 0; i < PER; i++) {
    const int c = threadIdx.x * 8 + i * 2048;
    if (c < h) {
      float* x = X + (size_t)row * h + c;
      const f32x4 g0 = *reinterpret_cast<const f32x4*>(gain + c), g1 = *reinterpret_cast<const f32x4*>(gain + c + 4);
      f32x4 x0, x1;
      bf16x8 o;
#pragma unroll
      for (int j = 0; j < 4; j++) {
        x0[j] = bf2f(v[i][j]); x1[j] = bf2f(v[i][j + 4]);
        o[j] = f2bf(x0[j] * inv * g0[j]); o[j + 4] = f2bf(x1[j] * inv * g1[j]);
      }
      *reinterpret_cast<f32x4*>(x) = x0;
      *reinterpret_cast<f32x4*>(x + 4) = x1;
      *reinterpret_cast<bf16x8*>(out + (size_t)row * h + c) = o;
    }
  }
}
hipError_t embed_norm_rows(hipStream_t s, float* X, bf16* out, const bf16* emb, const int* tokens, const float* gain, float eps, int n, int h,
                           const RowRotation& rot, const MetaCopy& meta) {
  if (n == 0) return hipSuccess;
  if (h > 8192 || h % 8 != 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(embed_norm_kernel, dim3(n + (meta.bytes + 4095) / 4096), dim3(256), 0, s, X, out, emb, tokens, gain, eps, h, n, rot, meta);
  return hipGetLastError();
}

hipError_t rmsnorm_rows(hipStream_t s, bf16* out, const float* X, const float* gain, float eps, int n, int h, const int* idx) {
  if (n == 0) return hipSuccess;
  if (n >= 1024) hipLaunchKernelGGL((rmsnorm_kernel<2, 4>), dim3((n + 1) / 2), dim3(256), 0, s, out, X, gain, eps, h, n, idx);
  else hipLaunchKernelGGL((rmsnorm_kernel<1, 8>), dim3(n), dim3(256), 0, s, out, X, gain, eps, h, n, idx);
  return hipGetLastError();
}

// ------------------------------------------------------------------ rotary + KV page write (prefill)
// One workgroup per token row; rot: the rows' cosines and sines (computed in double:
// positions reach tens of thousands of radians). Q is rotated in
// place; K is rotated and scattered to its page; V is scattered transposed (page_tokens = 16).
__global__ void __launch_bounds__(256) rope_kv_prefill_kernel(bf16* qkv, int ld, const PrefillSeq* seqs, int n_seqs,
                                                              const int* block_tables, const float* rot,
                                                              bf16* pool, KvGeom geo, int n_q) {
  const int row = blockIdx.x, d = geo.d, half = d >> 1;
  int si = 0;
  while (si + 1 < n_seqs && row >= seqs[si + 1].row0) si++;
  const PrefillSeq sq = seqs[si];
  const int pos = sq.p + (row - sq.row0);
  const float* cs = rot + (size_t)row * d;
  const float* sn = cs + half;
  const int page = block_tables[sq.bt_off + pos / geo.page_tokens], slot = pos % geo.page_tokens;
  bf16* r = qkv + (size_t)row * ld;
  // eight rotation pairs (two 16-byte loads, two 16-byte stores) per work item
  const int per_head = half >> 3, n_rot = (n_q + geo.n_kv) * per_head;
  for (int t = threadIdx.x; t < n_rot; t += blockDim.x) {
    const int hd = t / per_head, i0 = (t % per_head) * 8;
    const bf16x8 a = *reinterpret_cast<const bf16x8*>(r + hd * d + i0);
    const bf16x8 b = *reinterpret_cast<const bf16x8*>(r + hd * d + i0 + half);
    f32x4 c4[2], s4[2];
#pragma unroll
    for (int q = 0; q < 2; q++) {
      c4[q] = *reinterpret_cast<const f32x4*>(cs + i0 + 4 * q);
      s4[q] = *reinterpret_cast<const f32x4*>(sn + i0 + 4 * q);
    }
    bf16x8 ya, yb;
#pragma unroll
    for (int e = 0; e < 8; e++) {
      float ra, rb;
      rotate_pair(bf2f(a[e]), bf2f(b[e]), c4[e >> 2][e & 3], s4[e >> 2][e & 3], &ra, &rb);
      ya[e] = f2bf(ra);
      yb[e] = f2bf(rb);
    }
    bf16* dst = hd < n_q ? r + hd * d : pool + ((size_t)page * geo.n_kv + (hd - n_q)) * geo.head_elems() + (size_t)slot * d;
    *reinterpret_cast<bf16x8*>(dst + i0) = ya;
    *reinterpret_cast<bf16x8*>(dst + i0 + half) = yb;
  }
  // V^T: a page row holds 16 tokens of one (head, dd). Where the chunk covers a whole group of 8
  // tokens, the workgroup of the group's first row writes all 8 at once (one 16-byte store per
  // (head, dd), the 8 values gathered from the 8 rows with lane-contiguous loads) and the other
  // seven rows write nothing; a group the chunk covers only partly is written element by element.
  const bf16* vsrc = r + (n_q + geo.n_kv) * d;
  const int g0 = pos & ~7;                                  // first position of this row's group of 8
  const bool whole_group = g0 >= sq.p && g0 + 8 <= sq.p + sq.sl;
  if (whole_group) {
    if (pos != g0) return;
    for (int t = threadIdx.x; t < geo.n_kv * d; t += blockDim.x) {
      const int hd = t / d, dd = t % d;
      bf16x8 pack;
#pragma unroll
      for (int e = 0; e < 8; e++) pack[e] = vsrc[(size_t)e * ld + t];
      bf16* v = pool + ((size_t)page * geo.n_kv + hd) * geo.head_elems() + (size_t)geo.page_tokens * d;
      *reinterpret_cast<bf16x8*>(v + (size_t)dd * geo.page_tokens + slot) = pack;
    }
    return;
  }
  for (int t = threadIdx.x; t < geo.n_kv * d; t += blockDim.x) {
    const int hd = t / d, dd = t % d;
    bf16* v = pool + ((size_t)page * geo.n_kv + hd) * geo.head_elems() + (size_t)geo.page_tokens * d;
    v[(size_t)dd * geo.page_tokens + slot] = vsrc[t];
  }
}
hipError_t rope_kv_write_prefill(hipStream_t s, bf16* qkv, int ld, const PrefillSeq* seqs, int n_seqs,
                                 const int* block_tables, const float* rot, bf16* pool, KvGeom geo,
                                 int n_rows, int n_q) {
  if (n_rows == 0) return hipSuccess;
  hipLaunchKernelGGL(rope_kv_prefill_kernel, dim3(n_rows), dim3(256), 0, s, qkv, ld, seqs, n_seqs, block_tables,
                     rot, pool, geo, n_q);
  return hipGetLastError();
}

// Partial sums z = 0 .. S - 1 of four consecutive elements, added in that order onto v. S is a template argument of the
// kernels below: with the count known all the loads are under way before the first is used, and these kernels are bound by the
// latency of that chain (a loop over a runtime count waits for each load in turn).
template <int S>
__device__ __forceinline__ f32x4 add_partials(f32x4 v, const float* p, long long split_stride) {
  f32x4 q[S];
#pragma unroll
  for (int z = 0; z < S; z++) q[z] = *reinterpret_cast<const f32x4*>(p + z * split_stride);
#pragma unroll
  for (int z = 0; z < S; z++) v += q[z];
  return v;
}
// Launches with the split count (1 .. 8) as a compile-time constant S.
template <typename F>
hipError_t by_splits(int splits, F&& launch) {
  switch (splits) {
    case 1: launch(std::integral_constant<int, 1>{}); break;
    case 2: launch(std::integral_constant<int, 2>{}); break;
    case 3: launch(std::integral_constant<int, 3>{}); break;
    case 4: launch(std::integral_constant<int, 4>{}); break;
    case 5: launch(std::integral_constant<int, 5>{}); break;
    case 6: launch(std::integral_constant<int, 6>{}); break;
    case 7: launch(std::integral_constant<int, 7>{}); break;
    case 8: launch(std::integral_constant<int, 8>{}); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------ decode: QKV finish
// Sums the split-K partials of the QKV projection, rotates q and k (rot: the step's angles), stores q
// (bf16) for the attention kernel and appends k and v to the request's last page.
template <int S>
__global__ void __launch_bounds__(256) decode_qkv_finish_kernel(const float* partials, long long split_stride, int ld, const int* places,
                                                                const float* rot, bf16* q_out, bf16* pool,
                                                                KvGeom geo, int n_q) {
  // blockIdx.x = request, blockIdx.y = group of 8 head slots out of n_q (Q) + n_kv (K) + n_kv (V)
  const int row = blockIdx.x, d = geo.d, half = d >> 1;
  const int slot0 = blockIdx.y * 8, n_slots = n_q + 2 * geo.n_kv, slot1 = min(n_slots, slot0 + 8);
  const int place = places[row], page = place >> 4, slot = place & 15;
  const float* pr = partials + (size_t)row * ld;
  // a work item is four consecutive rotation pairs of a Q or K head, or four consecutive elements of a V head
  const int per_rot = half >> 2, per_v = d >> 2;
  const int n_rot_slots = max(0, min(slot1, n_q + geo.n_kv) - slot0), n_v_slots = (slot1 - slot0) - n_rot_slots;
  const int n_items = n_rot_slots * per_rot + n_v_slots * per_v;
  for (int t = threadIdx.x; t < n_items; t += blockDim.x) {
    if (t < n_rot_slots * per_rot) {
      const int hd = slot0 + t / per_rot, i0 = (t % per_rot) * 4;
      const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
      const f32x4 a = add_partials<S>(zero, pr + hd * d + i0, split_stride), b = add_partials<S>(zero, pr + hd * d + i0 + half, split_stride);
      const f32x4 cs = *reinterpret_cast<const f32x4*>(rot + (size_t)row * d + i0), sn = *reinterpret_cast<const f32x4*>(rot + (size_t)row * d + half + i0);
      bf16x4 ya, yb;
#pragma unroll
      for (int e = 0; e < 4; e++) {
        // the projection's result is rounded to bf16 before the rotation, as in the prefill path
        float ra, rb;
        rotate_pair(bf2f(f2bf(a[e])), bf2f(f2bf(b[e])), cs[e], sn[e], &ra, &rb);
        ya[e] = f2bf(ra);
        yb[e] = f2bf(rb);
      }
      bf16* dst = hd < n_q ? q_out + (size_t)row * n_q * d + hd * d
                           : pool + ((size_t)page * geo.n_kv + (hd - n_q)) * geo.head_elems() + (size_t)slot * d;
      *reinterpret_cast<bf16x4*>(dst + i0) = ya;
      *reinterpret_cast<bf16x4*>(dst + i0 + half) = yb;
    } else {
      const int tv = t - n_rot_slots * per_rot;
      const int hd = slot0 + n_rot_slots + tv / per_v, dd0 = (tv % per_v) * 4;
      const int vh = hd - n_q - geo.n_kv;
      const f32x4 a = add_partials<S>(f32x4{0.f, 0.f, 0.f, 0.f}, pr + hd * d + dd0, split_stride);
      bf16* v = pool + ((size_t)page * geo.n_kv + vh) * geo.head_elems() + (size_t)geo.page_tokens * d;
#pragma unroll
      for (int e = 0; e < 4; e++) v[(size_t)(dd0 + e) * geo.page_tokens + slot] = f2bf(a[e]);
    }
  }
}
hipError_t decode_qkv_finish(hipStream_t s, const float* partials, int splits, long long split_stride, int ld,
                             const int* place, const float* rot, bf16* q_out, bf16* pool, KvGeom geo, int n, int n_q) {
  if (n == 0) return hipSuccess;
  if (geo.page_tokens != 16) return hipErrorInvalidValue;
  return by_splits(splits, [&](auto S) {
    hipLaunchKernelGGL((decode_qkv_finish_kernel<decltype(S)::value>), dim3(n, (n_q + 2 * geo.n_kv + 7) / 8), dim3(256), 0, s, partials, split_stride, ld, place, rot, q_out,
                       pool, geo, n_q);
  });
}

// ------------------------------------------------------------------ split-K reductions
// X[row] += sum of partials; optionally out = rmsnorm(X[row]) * gain (bf16).
template <int S>
__global__ void __launch_bounds__(1024) reduce_resid_norm_kernel(float* X, const float* partials, long long split_stride,
                                                                 bf16* out, const float* gain, float eps, int h) {
  __shared__ float red[16];
  float* x = X + (size_t)blockIdx.x * h;
  const float* p = partials + (size_t)blockIdx.x * h;
  const int step = blockDim.x * 4;
  float ss = 0.f;
  for (int c = threadIdx.x * 4; c < h; c += step) {
    const f32x4 v = add_partials<S>(*reinterpret_cast<const f32x4*>(x + c), p + c, split_stride);
    *reinterpret_cast<f32x4*>(x + c) = v;
    ss += v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
  }
  if (out == nullptr) return;
  const float inv = rsqrtf(block_sum(ss, red) / (float)h + eps);
  for (int c = threadIdx.x * 4; c < h; c += step) {
    f32x4 v = *reinterpret_cast<const f32x4*>(x + c);     // this thread wrote these itself
    f32x4 g = *reinterpret_cast<const f32x4*>(gain + c);
    bf16x4 o;
#pragma unroll
    for (int j = 0; j < 4; j++) o[j] = f2bf(v[j] * inv * g[j]);
    *reinterpret_cast<bf16x4*>(out + (size_t)blockIdx.x * h + c) = o;
  }
}
hipError_t reduce_resid_norm(hipStream_t s, float* X, const float* partials, int splits, long long split_stride,
                             bf16* out_norm, const float* gain, float eps, int n, int h) {
  if (n == 0) return hipSuccess;
  const int threads = h >= 4096 ? 1024 : (h >= 2048 ? 512 : 256);      // one float4 per thread where the row allows
  return by_splits(splits, [&](auto S) {
    hipLaunchKernelGGL((reduce_resid_norm_kernel<decltype(S)::value>), dim3(n), dim3(threads), 0, s, X, partials, split_stride, out_norm, gain, eps, h);
  });
}

// H[row][j] = silu(sum gate_j) * sum up_j; gate/up columns are interleaved in blocks of 32.
template <int S>
__global__ void __launch_bounds__(256) reduce_swiglu_kernel(bf16* H, const float* partials, long long split_stride, int mlp) {
  const int row = blockIdx.y;
  const int j = (blockIdx.x * blockDim.x + threadIdx.x) * 4;         // four consecutive outputs, inside one block of 32
  if (j >= mlp) return;
  const float* p = partials + (size_t)row * 2 * mlp + (j >> 5) * 64 + (j & 31);
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  const f32x4 g = add_partials<S>(zero, p, split_stride), u = add_partials<S>(zero, p + 32, split_stride);
  bf16x4 o;
#pragma unroll
  for (int e = 0; e < 4; e++) o[e] = f2bf(swiglu(g[e], u[e]));
  *reinterpret_cast<bf16x4*>(H + (size_t)row * mlp + j) = o;
}
hipError_t reduce_swiglu(hipStream_t s, bf16* H, const float* partials, int splits, long long split_stride, int n, int mlp) {
  if (n == 0) return hipSuccess;
  if (mlp % 32 != 0 || split_stride % 4 != 0) return hipErrorInvalidValue;
  return by_splits(splits, [&](auto S) {
    hipLaunchKernelGGL((reduce_swiglu_kernel<decltype(S)::value>), dim3((mlp / 4 + 255) / 256, n), dim3(256), 0, s, H, partials, split_stride, mlp);
  });
}

__global__ void reduce_f32_kernel(float* out, const float* partials, int splits, long long split_stride, size_t n) {
  size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i >= n) return;
  float a = 0.f;
  for (int z = 0; z < splits; z++) a += partials[z * split_stride + i];
  out[i] = a;
}
hipError_t reduce_f32(hipStream_t s, float* out, const float* partials, int splits, long long split_stride, size_t n) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(reduce_f32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, out, partials, splits, split_stride, n);
  return hipGetLastError();
}

// ------------------------------------------------------------------ greedy sampling
// A row is dealt to `parts` workgroups of 1024 threads (16-byte loads, four in flight per thread), and the host takes the best of their
// maxima (in order, so that the first of equal values wins here as well): a thread scans its indices in ascending order and the lower index is kept
// on equal values. Bound by what one workgroup loads and, with `copy` (pinned host memory, the logits again), by the bus: the pass that reads them stores
// them there too (a runtime copy leaves the stream idle for about 15 us), and one workgroup a row asks for too little of either.
// A step of one layer with tokens alone, 128256 columns, one workgroup a row / in parts: 1 row 266 / 260 us, 8 rows 275 / 269, 64 rows 349 / 335.
__global__ void __launch_bounds__(1024) argmax_kernel(ArgBest* out, const float* logits, int vocab, int width, float* copy) {
  __shared__ ArgBest wave_best[16];
  const int tid = threadIdx.x, c0 = blockIdx.x * width, c1 = min(vocab, c0 + width);
  const float* l = logits + (size_t)blockIdx.y * vocab;
  float best = -INFINITY; int idx = 0x7FFFFFFF;
  auto take = [&](float v, int c) { if (v > best) { best = v; idx = c; } };
  if ((vocab & 3) == 0) {
    const f32x4* l4 = reinterpret_cast<const f32x4*>(l);
    f32x4* to = copy ? reinterpret_cast<f32x4*>(copy + (size_t)blockIdx.y * vocab) : nullptr;
    const int n4 = c1 >> 2;
    auto use = [&](const f32x4& v, int q) {
#pragma unroll
      for (int e = 0; e < 4; e++) take(v[e], 4 * q + e);
      if (to) to[q] = v;
    };
    int q = (c0 >> 2) + tid;
    for (; q + 3 * 1024 < n4; q += 4 * 1024) {
      const f32x4 a = l4[q], b = l4[q + 1024], c = l4[q + 2048], d = l4[q + 3072];
      use(a, q); use(b, q + 1024); use(c, q + 2048); use(d, q + 3072);
    }
    for (; q < n4; q += 1024) use(l4[q], q);
  } else {
    for (int c = c0 + tid; c < c1; c += 1024) take(l[c], c);
  }
  auto join = [&](float v, int i) { if (v > best || (v == best && i < idx)) { best = v; idx = i; } };
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) join(__shfl_xor(best, o, 64), __shfl_xor(idx, o, 64));
  if ((tid & 63) == 0) wave_best[tid >> 6] = ArgBest{best, idx};
  __syncthreads();
  if (tid >= 64) return;
  best = wave_best[tid & 15].value; idx = wave_best[tid & 15].index;
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) join(__shfl_xor(best, o, 64), __shfl_xor(idx, o, 64));
  if (tid == 0) out[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = ArgBest{best, idx};
}
// Parts of a row: one load of every thread or more each, about two workgroups a CU in all.
int argmax_parts(int n, int vocab) { return std::max(1, std::min({(vocab + 4095) / 4096, 512 / std::max(n, 1), ARGMAX_MAX_PARTS})); }
// out: n x argmax_parts(n, vocab), pinned host memory
hipError_t argmax_rows(hipStream_t s, ArgBest* out, const float* logits, int n, int vocab, float* copy) {
  if (n == 0) return hipSuccess;
  if (copy && vocab % 4 != 0) return hipErrorInvalidValue;
  const int parts = argmax_parts(n, vocab), width = ((vocab + parts - 1) / parts + 3) / 4 * 4;
  hipLaunchKernelGGL(argmax_kernel, dim3(parts, n), dim3(1024), 0, s, out, logits, vocab, width, copy);
  return hipGetLastError();
}

// ------------------------------------------------------------------ bandwidth probe
__global__ void __launch_bounds__(256) copy_kernel(uint4* __restrict__ dst, const uint4* __restrict__ src, size_t n) {
  size_t i = blockIdx.x * (size_t)256 + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * 256;
  for (; i + 3 * stride < n; i += 4 * stride) {
    uint4 a = src[i], b = src[i + stride], c = src[i + 2 * stride], d = src[i + 3 * stride];
    dst[i] = a; dst[i + stride] = b; dst[i + 2 * stride] = c; dst[i + 3 * stride] = d;
  }
  for (; i < n; i += stride) dst[i] = src[i];
}
// The read half of the copy alone: what a partition pulls from memory when nothing is written back. The loads carry the
// non-temporal hint (every byte is used once); `sink` receives a word only if the data's XOR hits one particular value,
// which keeps the loads alive.
__global__ void __launch_bounds__(256) read_kernel(const u32x4* __restrict__ src, size_t n, unsigned* __restrict__ sink) {
  size_t i = blockIdx.x * (size_t)256 + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * 256;
  u32x4 acc = {0u, 0u, 0u, 0u};
  for (; i + 7 * stride < n; i += 8 * stride) {
    u32x4 v[8];
#pragma unroll
    for (int u = 0; u < 8; u++) v[u] = __builtin_nontemporal_load(src + i + u * stride);
#pragma unroll
    for (int u = 0; u < 8; u++) acc ^= v[u];
  }
  for (; i < n; i += stride) acc ^= src[i];
  if ((acc[0] ^ acc[1] ^ acc[2] ^ acc[3]) == 0x5a17c0deu) *sink = 1u;
}
hipError_t read_probe(hipStream_t s, const void* src, size_t bytes, unsigned* sink, int grid) {
  hipLaunchKernelGGL(read_kernel, dim3(grid), dim3(256), 0, s, (const u32x4*)src, bytes / 16, sink);
  return hipGetLastError();
}
hipError_t copy_probe(hipStream_t s, void* dst, const void* src, size_t bytes, int grid) {
  hipLaunchKernelGGL(copy_kernel, dim3(grid), dim3(256), 0, s, (uint4*)dst, (const uint4*)src, bytes / 16);
  return hipGetLastError();
}

// ------------------------------------------------------------------ KV pool access (tests, synthetic contexts)
__device__ __forceinline__ void kv_addr(const KvGeom& geo, const int* bt, int pos, int hd, int dd, size_t& ki, size_t& vi) {
  const int page = bt[pos / geo.page_tokens], slot = pos % geo.page_tokens;
  const size_t base = ((size_t)page * geo.n_kv + hd) * geo.head_elems();
  ki = base + (size_t)slot * geo.d + dd;
  vi = base + (size_t)geo.page_tokens * geo.d + (size_t)dd * geo.page_tokens + slot;
}
// Element (pos, head, dd) of K (V) is deviate number ((pos*n_kv + head)*d + dd) of the stream
// keyed by tensor id 0x4B000000 + 2*layer (+1 for V): unit variance, rounded to bf16.
__global__ void kv_fill_kernel(bf16* pool, KvGeom geo, const int* bt, int pos0, int n, uint64_t kbase, uint64_t vbase) {
  size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  const size_t per = (size_t)geo.n_kv * geo.d;
  if (i >= (size_t)n * per) return;
  const int pos = pos0 + (int)(i / per), hd = (int)(i % per) / geo.d, dd = (int)(i % per) % geo.d;
  const uint64_t e = (uint64_t)pos * per + (i % per);
  size_t ki, vi; kv_addr(geo, bt, pos, hd, dd, ki, vi);
  pool[ki] = f2bf((float)irwin_hall12(kbase, e) * 1.52587890625e-05f);
  pool[vi] = f2bf((float)irwin_hall12(vbase, e) * 1.52587890625e-05f);
}
hipError_t kv_fill_random(hipStream_t s, bf16* pool, KvGeom geo, const int* bt, int pos0, int n, uint64_t seed, int layer) {
  size_t tot = (size_t)n * geo.n_kv * geo.d;
  if (tot == 0) return hipSuccess;
  const uint64_t kb = mix64(seed ^ mix64(0x4B000000ull + 2 * (uint64_t)layer)), vb = mix64(seed ^ mix64(0x4B000000ull + 2 * (uint64_t)layer + 1));
  hipLaunchKernelGGL(kv_fill_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, pool, geo, bt, pos0, n, kb, vb);
  return hipGetLastError();
}
__global__ void kv_write_kernel(bf16* pool, KvGeom geo, const int* bt, int pos0, int n, const float* k, const float* v) {
  size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  const size_t per = (size_t)geo.n_kv * geo.d;
  if (i >= (size_t)n * per) return;
  const int pos = pos0 + (int)(i / per), hd = (int)(i % per) / geo.d, dd = (int)(i % per) % geo.d;
  size_t ki, vi; kv_addr(geo, bt, pos, hd, dd, ki, vi);
  pool[ki] = f2bf(k[i]); pool[vi] = f2bf(v[i]);
}
hipError_t kv_write_tokens(hipStream_t s, bf16* pool, KvGeom geo, const int* bt, int pos0, int n, const float* k, const float* v) {
  size_t tot = (size_t)n * geo.n_kv * geo.d;
  if (tot == 0) return hipSuccess;
  hipLaunchKernelGGL(kv_write_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, pool, geo, bt, pos0, n, k, v);
  return hipGetLastError();
}
__global__ void kv_read_kernel(const bf16* pool, KvGeom geo, const int* bt, int pos0, int n, float* k, float* v) {
  size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  const size_t per = (size_t)geo.n_kv * geo.d;
  if (i >= (size_t)n * per) return;
  const int pos = pos0 + (int)(i / per), hd = (int)(i % per) / geo.d, dd = (int)(i % per) % geo.d;
  size_t ki, vi; kv_addr(geo, bt, pos, hd, dd, ki, vi);
  k[i] = bf2f(pool[ki]); v[i] = bf2f(pool[vi]);
}
hipError_t kv_read_tokens(hipStream_t s, const bf16* pool, KvGeom geo, const int* bt, int pos0, int n, float* k, float* v) {
  size_t tot = (size_t)n * geo.n_kv * geo.d;
  if (tot == 0) return hipSuccess;
  hipLaunchKernelGGL(kv_read_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, pool, geo, bt, pos0, n, k, v);
  return hipGetLastError();
}

}  // namespace sts
