// Internal (C++) interface between the engine and the gfx950 kernels. Not part of the C ABI.
#pragma once
#include <vector>

#include "common.h"

namespace sts {

// ---- GEMM -------------------------------------------------------------------------------
enum GemmEpilogue { EPI_BF16 = 0, EPI_F32 = 1, EPI_RESID_F32 = 2, EPI_SWIGLU_BF16 = 3, EPI_QKV = 4 };
// the same numbering as STS_GEMM_* in sts.h
enum GemmConfig { GEMM_128x128 = 0, GEMM_64x256 = 1, GEMM_64x128 = 2, GEMM_256x256 = 3, GEMM_128x256 = 4, GEMM_64x256S = 5, GEMM_64x320S = 6, GEMM_64x384S = 7,
                  GEMM_64x448S = 8, GEMM_64x512S = 9, GEMM_NCFG = 10 };
int gemm_tile_m(int cfg);
int gemm_tile_n(int cfg);
int gemm_wgs_per_cu(int cfg);                       // resident workgroups per CU of this configuration
// Tail splitting: `slots` = workgroups the stream's CU partition holds at once, `ws` = fp32 scratch.
// norm: RMSNorm wanted of the finished rows of C (out: [M, N] bf16); `done` is set if the launch's last kernel writes it.
struct ResidNorm { bf16* out; const float* gain; float eps; bool done; };
// EPI_QKV (256x256, packed W): columns are n_q query heads, then n_kv K and n_kv V heads of geo.d. Q is rotated into C, K rotated and V
// transposed into the rows' places in the KV pool; C's K and V columns are not written. rot: each row's angles; place: page *
// page_tokens + slot of each row.
struct QkvOut;
struct GemmTail { int slots; float* ws; size_t ws_bytes; ResidNorm* norm = nullptr; };
void gemm_tail_plan(int tiles, int ksteps, int slots, long long max_pieces, int* n_full, int* f);
// W is either row-major [N, ldw] or (w_packed, the engine's weights; needs ldw == K) in
// the packed layout below. The row-major form exists for the fp32-store epilogue only.
hipError_t gemm_bf16(hipStream_t s, int cfg, int epi, const bf16* A, int lda, const bf16* W, int ldw,
                     void* C, int ldc, int M, int N, int K, int splits, long long split_stride,
                     const GemmTail* tail = nullptr, bool w_packed = true, bool stream_nt = false, int row_tiles = 0, const QkvOut* qkv = nullptr);

// Packed GEMM weights: blocks of 32 rows x 64 columns (4 KiB), stored one after the other along K, then
// along N. A block is laid out the way the matrix cores take a W operand: four pieces of 1 KiB, one per
// 16-column step, each holding for lane l = 32 * h + n of a wave the 8 consecutive elements
// W[row n][16 * step + 8 * h .. + 8). A wave therefore loads an operand straight into registers with one
// 16-byte load per lane from 1 KiB of consecutive memory (the large prefill tile does that, and keeps W
// out of LDS), and the direct-to-LDS loads of the other tiles gather the same bytes in whole 128-byte
// pieces (8 rows of one half-step). A tile's share of a K step is whole 4 KiB blocks instead of one
// 128-byte piece out of each of its rows (rows are K * 2 bytes apart), which is what HBM-bound decode
// GEMMs want. N must be a multiple of 32 and K of 64.
__host__ __device__ __forceinline__ size_t weight_packed_index(int row, int col, int ld) {
  const size_t block = (size_t)(row >> 5) * (ld >> 6) + (col >> 6);
  return block * 2048 + (size_t)((col & 63) >> 4) * 512 + (size_t)((((col >> 3) & 1) << 5) + (row & 31)) * 8 + (col & 7);
}

// ---- paged KV layout ----------------------------------------------------------------------
// One layer's pool is [n_pages][n_kv_heads][ K: page_tokens x d | V^T: d x page_tokens ] bf16.
// V is kept transposed inside a page so that the P*V contraction (over tokens) reads
// token-contiguous operands, as the MFMA operand layout wants.
struct KvGeom {
  int n_kv, d, page_tokens;
  __host__ __device__ size_t head_elems() const { return (size_t)2 * page_tokens * d; }
  __host__ __device__ size_t page_elems() const { return head_elems() * n_kv; }
};

struct QkvOut { const float* rot; const int* place; bf16* pool; KvGeom geo; int n_q; };

// Per-sequence metadata of one prefill launch (device array, one entry per sequence).
struct PrefillSeq {
  int row0;        // first row of this sequence in the packed activation buffers
  int sl;          // new tokens
  int p;           // tokens already cached (positions 0..p-1)
  int bt_off;      // offset of this sequence's block table in the block-table buffer
  int n_pages;     // valid entries in that block table
};
// One query tile of one sequence (rows from q0), or one part of its key range: 64-key tiles [kt0, kt1). part: where its partial
// output goes, -1 if the tile is finished by its workgroup.
struct AttnItem { int seq, q0, kt0, kt1, part; };
struct AttnMerge { int seq, q0, part0, parts; };   // a query tile whose key range was cut: parts part0 .. part0 + parts - 1

// Per-request metadata of one decode step.
struct DecodeSeq {
  int cl;          // tokens already cached; the new token sits at position cl
  int bt_off;
  int n_pages;     // pages covering positions 0..cl
};

// One context chunk of one decode request, with what its workgroup needs to start: a single
// 16-byte load instead of a chain through the per-request record.
struct DecodeItem { int seq; int chunk; int cl; int bt_off; };
struct DecodeMerge { int seq; int chunks; };           // a request whose context has more than one chunk

// ---- element-wise / small kernels ---------------------------------------------------------
hipError_t init_weight(hipStream_t s, bf16* dst, int ld, uint64_t seed, uint64_t tensor_id, int rows, int cols,
                       int row_offset, int interleave_block, int interleave_phase, int packed);
hipError_t convert_weight(hipStream_t s, bf16* dst, int ld, const float* src, int rows, int cols,
                          int row_offset, int interleave_block, int interleave_phase, int packed);
hipError_t export_weight(hipStream_t s, float* dst, const bf16* src, int ld, int rows, int cols,
                         int row_offset, int interleave_block, int interleave_phase, int packed);
hipError_t fill_f32(hipStream_t s, float* dst, float v, size_t n);
hipError_t embed_rows(hipStream_t s, float* X, const bf16* emb, const int* tokens, int n, int h);
// Rotation angles of a launch's rows, written to table [row][d / 2 cosines | d / 2 sines]. pos: each row's position (device or pinned
// host memory: one read a row).
struct RowRotation { float* table; const int* pos; const double* inv_freq; int d; };
hipError_t row_rotation(hipStream_t s, const RowRotation& rot, int n);
// Metadata in pinned host memory to the device (bytes rounded up to 16 must be readable and writable).
struct MetaCopy { const unsigned char* src; unsigned char* dst; int bytes; };
hipError_t copy_in(hipStream_t s, const MetaCopy& meta);
// embedding rows into the fp32 residual stream X and, in the same pass, their RMSNorm into out (bf16); h <= 8192; the rows'
// rotation angles; and the metadata copy (bytes 0: none)
hipError_t embed_norm_rows(hipStream_t s, float* X, bf16* out, const bf16* emb, const int* tokens, const float* gain, float eps, int n, int h,
                           const RowRotation& rot, const MetaCopy& meta);
// rows idx[i] of X if idx is given
hipError_t rmsnorm_rows(hipStream_t s, bf16* out, const float* X, const float* gain, float eps, int n, int h, const int* idx = nullptr);
hipError_t rope_kv_write_prefill(hipStream_t s, bf16* qkv, int ld, const PrefillSeq* seqs, int n_seqs,
                                 const int* block_tables, const float* rot, bf16* pool, KvGeom geo,
                                 int n_rows, int n_q);
// place: page * page_tokens + slot of each row's K and V (also in kslice_qkv)
hipError_t decode_qkv_finish(hipStream_t s, const float* partials, int splits, long long split_stride, int ld,
                             const int* place, const float* rot, bf16* q_out, bf16* pool, KvGeom geo, int n, int n_q);
hipError_t reduce_resid_norm(hipStream_t s, float* X, const float* partials, int splits, long long split_stride,
                             bf16* out_norm, const float* gain, float eps, int n, int h);
hipError_t reduce_swiglu(hipStream_t s, bf16* H, const float* partials, int splits, long long split_stride,
                         int n, int mlp);
hipError_t reduce_f32(hipStream_t s, float* out, const float* partials, int splits, long long split_stride, size_t n);
// Largest value of a part of a row and its first index; index 0x7FFFFFFF: no value above -inf.
struct ArgBest { float value; int index; };
constexpr int ARGMAX_MAX_PARTS = 32;
int argmax_parts(int n, int vocab);
// copy: the logits again (pinned host memory), or null
hipError_t argmax_rows(hipStream_t s, ArgBest* out, const float* logits, int n, int vocab, float* copy = nullptr);
hipError_t copy_probe(hipStream_t s, void* dst, const void* src, size_t bytes, int grid);
hipError_t read_probe(hipStream_t s, const void* src, size_t bytes, unsigned* sink, int grid);    // the read half alone; sink: 4 bytes of device memory
hipError_t kv_fill_random(hipStream_t s, bf16* pool, KvGeom geo, const int* block_table, int pos0, int n,
                          uint64_t seed, int layer);
hipError_t kv_write_tokens(hipStream_t s, bf16* pool, KvGeom geo, const int* block_table, int pos0, int n,
                           const float* k, const float* v);
hipError_t kv_read_tokens(hipStream_t s, const bf16* pool, KvGeom geo, const int* block_table, int pos0, int n,
                          float* k, float* v);

// ---- attention ----------------------------------------------------------------------------
hipError_t attn_prefill(hipStream_t s, const bf16* qkv, int ld, bf16* out, int ldo, const PrefillSeq* seqs,
                        const AttnItem* items, int n_items, int heads, const AttnMerge* merges, int n_merges, const int* block_tables, const bf16* pool,
                        KvGeom geo, int n_q, float* part_ws);
int attn_prefill_tile_q();
struct AttnPlan { std::vector<AttnItem> items; std::vector<AttnMerge> merges; int parts = 0; bool pairs = false; };
AttnPlan attn_prefill_plan(int n_seqs, const int* lens, const int* priors, int n_q, int slots, int max_extra, long long max_parts);
int attn_prefill_heads(bool pairs, int n_q, int n_kv, int d);
size_t attn_prefill_part_floats(int n_q, int d);   // of one part
size_t attn_decode_ws_floats(int n, int n_q, int d, int max_chunks);
hipError_t attn_decode(hipStream_t s, const bf16* q, bf16* out, const DecodeSeq* seqs, const DecodeItem* items, int n_items, const DecodeMerge* multi, int n_multi,
                       const int* block_tables, const bf16* pool, KvGeom geo, int n, int n_q, int chunk_pages, int max_chunks, float* ws,
                       bool stream_nt = false);
int attn_decode_max_chunk_tokens();

// ---- decode GEMMs that finish their own output (gemm_kslice.hip) ----------------------------
enum KsliceEpilogue { KS_F32 = 0, KS_RESID = 1, KS_SWIGLU = 2, KS_QKV = 3 };
constexpr int KSLICE_MAX_ROWS = 16;
// Sizes the form takes: its byte offsets into W are 32 bits wide. A plan asks before it compares times.
inline bool kslice_covers(int n, int k) { return (unsigned long long)n * k * 2 < (1ull << 32); }
// Row factor of a GEMM's activations: 1 / sqrt(sum of `parts` shares of the row's sum of squares / K + eps); none if ssq is null.
struct RowScale { const float* ssq; int parts; float eps; };
// A [M, lda] row-major, W [N, K] in the packed layout.
struct KsliceIn { const bf16* A; int lda; RowScale scale; const bf16* W; int M, N, K; };
int kslice_cols(int epi, int n, int cus);
hipError_t kslice_f32(hipStream_t s, const KsliceIn& in, int cus, float* C, int ldc);
hipError_t kslice_resid(hipStream_t s, const KsliceIn& in, int cus, float* X, const float* gain, bf16* Xg, float* ssq_out);
hipError_t kslice_swiglu(hipStream_t s, const KsliceIn& in, bf16* H);
hipError_t kslice_qkv(hipStream_t s, const KsliceIn& in, const int* place, const float* rot, bf16* q_out, bf16* pool, KvGeom geo, int n_q);

// ---- GEMMs of up to 256 rows that read their weights once (gemm_cols.hip) --------------------
constexpr int COLS_MAX_ROWS = 256;
hipError_t gemm_cols(hipStream_t s, int epi, const bf16* A, int lda, const bf16* W, void* C, int ldc, int M, int N, int K, int splits, long long split_stride);

}  // namespace sts
