// Concurrent execution engine: owns weights, the shared paged KV pool, the per-phase
// workspaces and the CU-masked streams, and drives the kernels of a prefill layer slice and of
// a decode step (paper Sections 3.4 and 3.5). Everything here is host code; the kernels live in
// gemm.hip, attn_prefill.hip, attn_decode.hip and elementwise.hip.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "kernels.h"
#include "sts.h"

using namespace sts;

static std::atomic<int> g_hip_err{0};   // either phase's control thread may record an error
#define HIPCK(x)                                                 \
  do {                                                           \
    hipError_t e_ = (x);                                         \
    if (e_ != hipSuccess) { g_hip_err = (int)e_; return STS_EHIP; } \
  } while (0)
#define STSCK(x) do { int r_ = (x); if (r_ != STS_OK) return r_; } while (0)

extern "C" const char* sts_strerror(int code) {
  switch (code) {
    case STS_OK: return "ok";
    case STS_EINVAL: return "invalid argument";
    case STS_ENOMEM: return "KV page pool or workspace exhausted";
    case STS_ESTATE: return "call out of order for the current state";
    case STS_EHIP: return "HIP runtime error (see sts_last_hip_error)";
    case STS_EIO: return "file or parse error";
    default: return "unknown error";
  }
}
extern "C" int sts_last_hip_error(void) { return g_hip_err.load(); }

static const char* kKernelNames[STS_K_COUNT] = {"embed", "norm", "qkv", "rope", "attn", "attn_merge", "o", "gateup",
                                                "swiglu", "down", "reduce", "head", "sample"};
extern "C" const char* sts_kernel_name(int32_t kind) { return (kind >= 0 && kind < STS_K_COUNT) ? kKernelNames[kind] : "?"; }

namespace {

struct LayerW { bf16 *wqkv, *wo, *wgu, *wd; float *g1, *g2; };

struct Seq { bool used = false; int len = 0; std::vector<int> pages; };

struct Phase {
  int side = 0;
  int cus = 0;
  hipStream_t stream = nullptr;
  hipEvent_t ev0 = nullptr, ev1 = nullptr;
  bool ran = false;
  // device workspace
  float* X = nullptr; bf16* Xn = nullptr; bf16* QKV = nullptr; bf16* A = nullptr; bf16* H = nullptr;
  float* part = nullptr; size_t part_floats = 0; float* attn_ws = nullptr; bf16* Q = nullptr;
  float* rot = nullptr; float* ssq = nullptr;                 // rotation angles of the launch's rows; decode: shares of the rows' sums of squares
  float* tail_ws = nullptr; size_t tail_ws_bytes = 0;         // prefill: GEMM tail pieces, partial attention outputs, head partial sums
  int max_attn_extra = 0;
  bf16* Xlast_n = nullptr; float* logits = nullptr;
  // Per-call metadata (sequence records, block tables, work items, token ids, positions) is packed into one pinned
  // block, which a kernel copies to the device (the embedding kernel on the side, or copy_in); the pointers below are views
  // into the two blocks, laid out afresh by every launch.
  unsigned char* h_meta = nullptr; unsigned char* d_meta = nullptr; size_t meta_bytes = 0, meta_used = 0;
  int* d_tokens = nullptr; int* d_pos = nullptr; int* d_place = nullptr; int* d_bt = nullptr; int* d_rows = nullptr;
  PrefillSeq* d_pseq = nullptr; DecodeSeq* d_dseq = nullptr; AttnItem* d_items = nullptr; DecodeItem* d_ditems = nullptr;
  // pinned staging
  int* h_tokens = nullptr; int* h_pos = nullptr; int* h_place = nullptr; int* h_bt = nullptr; int* h_rows = nullptr;
  PrefillSeq* h_pseq = nullptr; DecodeSeq* h_dseq = nullptr; AttnItem* h_items = nullptr; DecodeItem* h_ditems = nullptr;
  float* h_logits = nullptr; ArgBest* h_best = nullptr;
  int rows = 0;                               // rows of the last call
  bool alone = false;                         // neither queued together with the other phase nor while a launched step of it was in flight (blocking calls of two threads do not see each other)
  // per-kernel timing
  std::vector<hipEvent_t> kev; std::vector<int> kkind; size_t kused = 0;
  int64_t kns[STS_K_COUNT] = {0}, kcnt[STS_K_COUNT] = {0};
  int fail_after = -1;                        // sts_fail_launch: launches until one is reported as failed, -1: none
};

}  // namespace

struct sts_ctx {
  sts_model_desc d;
  sts_init_params p;
  int n_cu = 0;
  int qd = 0, kvd = 0, qkvn = 0;
  KvGeom geo;
  bf16 *emb = nullptr, *lm = nullptr; float* gf = nullptr;
  std::vector<LayerW> layers;
  bf16* pool = nullptr; size_t pool_layer_elems = 0;
  double* inv_freq = nullptr;
  std::mutex alloc_mu;                         // serialises page allocation / release
  std::mutex state_mu;                         // guards the in-flight prefill batch description
  std::mutex part_mu;                          // serialises repartitioning (one control thread per phase may call it)
  std::vector<int> free_pages; std::vector<char> page_used;
  std::vector<Seq> seqs;
  Phase ph[2];
  int part_cus[2] = {0, 0};
  bool ktiming = false;
  // in-flight layer-sliced prefill batch
  bool pf_active = false; int pf_next_layer = 0; std::vector<int> pf_seqs, pf_lens;
  int64_t last_wall_ns = 0;
  // launches whose finish call is still due (non-blocking API)
  std::atomic<bool> pend_prefill{false}, pend_decode{false};    // a launch of that phase is in flight (each set by its own control thread)
  std::vector<int> pend_pseqs, pend_plens, pend_dseqs; int pend_le = 0;
  void* probe_src = nullptr; void* probe_dst = nullptr; size_t probe_bytes = 0;
  std::vector<void*> allocs;
  std::vector<hipStream_t> used_streams;       // every pooled stream this ctx ever selected (guarded by part_mu)
  // what the choice of GEMM tiles assumes about the part (sts_set_tile_model): TFLOP/s per busy CU of the 128x128
  // tiles (two workgroups per CU) and of the 256x256 tiles (one), bytes/s per CU for partial tiles
  double rate_128 = 3.5, rate_256 = 4.8, partial_bw = 20e9;
  double stream_bw_cu = 59e9, stream_bw_gpu = 6.4e12;          // read-only streams: bytes/s per CU of a 32-CU partition, bytes/s of the whole GPU
};

namespace {

template <typename T>
int dev_alloc(sts_ctx* c, T** out, size_t count) {
  void* p = nullptr;
  HIPCK(hipMalloc(&p, std::max<size_t>(count, 1) * sizeof(T)));
  c->allocs.push_back(p);
  *out = reinterpret_cast<T*>(p);
  return STS_OK;
}
// Next 256-byte aligned view of `count` elements in a phase's metadata blocks.
template <typename T>
void meta_take(Phase& ph, T** host, T** dev, size_t count);

template <typename T>
int host_alloc(T** out, size_t count) {
  void* p = nullptr;
  // coherent: kernels read metadata from it and store results to it, the host sees those once the stream is done
  HIPCK(hipHostMalloc(&p, std::max<size_t>(count, 1) * sizeof(T), hipHostMallocMapped | hipHostMallocCoherent));
  *out = reinterpret_cast<T*>(p);
  return STS_OK;
}

template <typename T>
void meta_take(Phase& ph, T** host, T** dev, size_t count) {
  const size_t off = (ph.meta_used + 255) & ~(size_t)255;
  *host = reinterpret_cast<T*>(ph.h_meta + off);
  *dev = reinterpret_cast<T*>(ph.d_meta + off);
  ph.meta_used = off + count * sizeof(T);
}

// CU-masked streams are a process-wide pool: one stream per (side, CU count), created on first
// use and kept until the process ends. Repartitioning is then a pointer switch, engines that
// come and go reuse the same hardware queues, and no masked queue is ever torn down.
std::mutex g_stream_mu;
std::map<std::pair<int, int>, hipStream_t> g_streams;
std::atomic<int> g_live_ctx{0};            // engines alive in this process (sts_release_streams refuses while any is)
std::atomic<bool> g_streams_released{false};   // set by sts_release_streams: the process is ending, no further engine is created

void trace(const char* what) {
  static const bool on = std::getenv("STS_TRACE") != nullptr;
  if (on) { std::fprintf(stderr, "[sts] %s\n", what); std::fflush(stderr); }
}

int get_stream(sts_ctx* c, int side, int cus, hipStream_t* out) {
  std::lock_guard<std::mutex> g(g_stream_mu);
  auto key = std::make_pair(side, cus);
  auto it = g_streams.find(key);
  if (it != g_streams.end()) { *out = it->second; return STS_OK; }
  // A mask that leaves some XCD without a CU makes stream creation fail (and crashes some
  // runtime versions): contiguous runs of >= 8 bits always cover all 8 XCDs because mask bit i
  // belongs to XCD i % 8.
  if (cus < 8 || cus > c->n_cu || cus % 8 != 0) return STS_EINVAL;
  const int words = (c->n_cu + 31) / 32;
  std::vector<uint32_t> mask(words, 0);
  const int lo = side == 0 ? 0 : c->n_cu - cus;
  for (int b = lo; b < lo + cus; b++) mask[b / 32] |= 1u << (b % 32);
  hipStream_t s = nullptr;
  HIPCK(hipExtStreamCreateWithCUMask(&s, words, mask.data()));
  g_streams[key] = s;
  *out = s;
  return STS_OK;
}

// Caller holds part_mu (or is the only user of the ctx).
void remember_stream(sts_ctx* c, hipStream_t s) {
  if (s && std::find(c->used_streams.begin(), c->used_streams.end(), s) == c->used_streams.end()) c->used_streams.push_back(s);
}

int select_streams(sts_ctx* c) {
  for (int side = 0; side < 2; side++) {
    Phase& ph = c->ph[side];
    if (c->part_cus[side] == 0) { ph.stream = nullptr; ph.cus = 0; continue; }
    STSCK(get_stream(c, side, c->part_cus[side], &ph.stream));
    remember_stream(c, ph.stream);
    ph.cus = c->part_cus[side];
  }
  return STS_OK;
}

// ---- per-kernel timing
int k_begin(sts_ctx* c, Phase& ph, int kind) {
  if (ph.fail_after >= 0 && ph.fail_after-- == 0) { g_hip_err = (int)hipErrorLaunchFailure; return STS_EHIP; }
  if (!c->ktiming) return STS_OK;
  if (ph.kused + 2 > ph.kev.size()) {
    for (int i = 0; i < 256; i++) { hipEvent_t e; HIPCK(hipEventCreate(&e)); ph.kev.push_back(e); }
  }
  ph.kkind.push_back(kind);
  HIPCK(hipEventRecord(ph.kev[ph.kused], ph.stream));
  return STS_OK;
}
int k_end(sts_ctx* c, Phase& ph) {
  if (!c->ktiming) return STS_OK;
  HIPCK(hipEventRecord(ph.kev[ph.kused + 1], ph.stream));
  ph.kused += 2;
  return STS_OK;
}
int k_collect(sts_ctx* c, Phase& ph) {
  if (!c->ktiming) return STS_OK;
  for (size_t i = 0; i < ph.kkind.size(); i++) {
    float ms = 0.f;
    HIPCK(hipEventElapsedTime(&ms, ph.kev[2 * i], ph.kev[2 * i + 1]));
    ph.kns[ph.kkind[i]] += (int64_t)(ms * 1e6);
    ph.kcnt[ph.kkind[i]] += 1;
  }
  ph.kkind.clear(); ph.kused = 0;
  return STS_OK;
}
#define KL(ph, kind, expr)                \
  do {                                    \
    STSCK(k_begin(c, ph, kind));          \
    HIPCK(expr);                          \
    STSCK(k_end(c, ph));                  \
  } while (0)

int pick_cfg(int m, int n, int k, int cus) {
  // up to 64 rows: 64x128 tiles, two workgroups (8 waves) per CU streaming weights (decode GEMMs whose N allows
  // it take the skinny tiles instead, see pick_decode_gemm)
  if (m <= 64) return GEMM_64x128;
  // up to 128 rows: one row of 128x128 tiles, two workgroups per CU. Above that both shapes compute
  // 256 rows and the 256x256 tile's larger wave tiles run the MFMAs faster; a large decode batch
  // on a small partition is compute-bound (Section 2.1). One 256x256 workgroup fills a CU, so the
  // shape is taken only when its tiles times the deepest split-K still cover the partition.
  const bool covers = (long long)(n / 256) * std::min(8, std::max(1, k / 512)) >= cus;
  return (m <= 128 || n % 256 != 0 || !covers) ? GEMM_128x128 : GEMM_256x256;
}
// Prefill GEMM tile choice for a partition of `cus` CUs: the candidate with the smallest
// estimated time, which is where wave quantisation (paper Section 2.2.1) enters -- complete
// waves of workgroups at the tile's busy-CU rate, then the last wave, whole or cut along K.
// Rates are measured busy-CU throughputs in TFLOP/s per CU: 128x128 tiles run two workgroups
// per CU, the 256-column tiles one; rate_256 is that of the tallest. The latter come in heights of 32 to 256 rows: the rows
// are dealt to any number of row tiles, so that they fill whole waves of workgroups.
struct PrefillGemm { int cfg = GEMM_64x128, row_tiles = 0; double est_s = 0.0; };
// Time of a 256-column tile of 32 (h + 1) rows against one of 256 (a short tile still streams its 256 columns of weights). Measured inside a
// layer on 256 CUs at heights 32 / 64 / 96 / 128 / 160 / 192 / 224: 16 row tiles of 4096 x 4096 0.41 / 0.47 / 0.52 / 0.60 / 0.70 / 0.76 / 0.88, of 4096 x
// 14336 0.42 / 0.48 / 0.52 / 0.59 / 0.67 / 0.77 / 0.88; two of 28672 x 4096, which wait for their weights, 0.54 / 0.66 / 0.72 / 0.77 / 0.83 / 0.88 / 0.93. It
// serves smaller partitions too: on 32 to 256 CUs, 96 to 4096 rows, the choice made with it and with the profiles' rates is within
// 3 % of the fastest candidate in 243 of 288 launches, within 8 % in 268; the worst, 14336-deep tiles of 256 rows on 32 CUs, takes 184 us for 142
// because those rates are of slower tiles (4.97 TFLOP/s per CU for 5.52 now). They stay because they also decide where K is cut.
constexpr double TILE_HEIGHT_COST[8] = {0.40, 0.43, 0.52, 0.59, 0.70, 0.78, 0.91, 1.0};
PrefillGemm pick_prefill_gemm(const sts_ctx* ctx, int m, int n, int k, int cus, size_t tail_ws_bytes) {
  PrefillGemm best;
  if (m <= 64) return best;
  double best_cost = 1e300;
  const int c = std::max(cus, 8), blocks = (m + 31) / 32;
  // in units of the candidate's tile time: complete waves, then the last wave -- whole, or in rounds of 1/f with a start-up
  // charge per round, plus the partial tiles written and read back (4 bytes out, 4 in per element and piece, at the
  // measured per-CU rate)
  auto consider = [&](int cfg, int row_tiles, int tiles, int slots, int tile_elems, double tile_s) {
    int n_full, f;
    gemm_tail_plan(tiles, k / 64, slots, (long long)(tail_ws_bytes / (tile_elems * sizeof(float))), &n_full, &f);
    double t;
    if (f > 1) {
      const int rest = tiles - n_full, rounds = (rest * f + slots - 1) / slots;
      t = (n_full / slots + rounds * (1.0 / f + 0.03)) * tile_s + (double)rest * f * tile_elems * 8.0 / (c * ctx->partial_bw) + 6e-6;
    } else {
      t = (double)((tiles + slots - 1) / slots) * tile_s;
    }
    if (t < best_cost) { best_cost = t; best = PrefillGemm{cfg, row_tiles, t}; }
  };
  consider(GEMM_128x128, 0, ((m + 127) / 128) * (n / 128), 2 * c, 128 * 128, 2.0 * 128 * 128 * k / (ctx->rate_128 * 1e12 / 2));
  if (n % 256 == 0) {
    const double tall_s = 2.0 * 256 * 256 * k / (ctx->rate_256 * 1e12);
    const int least = (blocks + 7) / 8;
    for (int t = least; t <= std::min(blocks, 2 * least + 2); t++) {       // beyond that a tile is mostly its weights
      const int h = (blocks + t - 1) / t;
      consider(GEMM_256x256, t, t * (n / 256), c, h * 32 * 256, TILE_HEIGHT_COST[h - 1] * tall_s);
    }
  }
  return best;
}
// A prefill GEMM on the phase's partition, the last wave of tiles cut along K.
hipError_t prefill_gemm(const Phase& ph, const PrefillGemm& gm, int epi, const bf16* A, int lda, const bf16* W, int ldw, void* C, int ldc, int m, int n, int k, ResidNorm* norm = nullptr, const QkvOut* qkv = nullptr) {
  const GemmTail tail{gemm_wgs_per_cu(gm.cfg) * ph.cus, ph.tail_ws, ph.tail_ws_bytes, norm};
  return gemm_bf16(ph.stream, gm.cfg, epi, A, lda, W, ldw, C, ldc, m, n, k, 1, 0, &tail, true, false, gm.row_tiles, qkv);
}
int plan_splits(double rate_256, double partial_bw, int cfg, int m, int n, int k, int cus) {
  const int tiles = ((m + gemm_tile_m(cfg) - 1) / gemm_tile_m(cfg)) * (n / gemm_tile_n(cfg));
  const int slots = gemm_wgs_per_cu(cfg) * std::max(cus, 8);
  const int s_max = std::min(8, std::max(1, k / 512));            // at least 8 K-steps per slice
  if (gemm_wgs_per_cu(cfg) == 1 && gemm_tile_m(cfg) >= 256) {
    // one workgroup owns a CU, so rounds of workgroups are strict: estimated time of s slices =
    // ceil(tiles * s / slots) rounds of a 1/s tile at the measured rate of that tile, plus the fp32
    // partial sums written and read back at the measured per-CU rate; the cheapest s wins
    const double tile_s = 2.0 * gemm_tile_m(cfg) * gemm_tile_n(cfg) * k / (rate_256 * 1e12);
    const double part_s = 8.0 * m * n / (std::max(cus, 8) * partial_bw);
    int best = 1; double best_t = 1e300;
    for (int s = 1; s <= s_max; s++) {
      const double t = (double)(((long long)tiles * s + slots - 1) / slots) * tile_s / s + s * part_s;
      if (t < best_t - 1e-9) { best_t = t; best = s; }
    }
    return best;
  }
  const int s = (slots + tiles - 1) / tiles;                        // fill the partition's workgroup slots
  return std::max(1, std::min(s, s_max));
}

// Tile shape and split-K of one decode GEMM. Above 64 rows: the prefill shapes (pick_cfg) with a split that
// fills the partition. Up to 64 rows the GEMM streams its weights once and runs at the pace at which the
// partition's CUs pull bytes, and everything a workgroup reads counts: its K range of the W columns and, beside
// them, the 64 activation rows of that range again for every workgroup. The candidates are the 64x128 tiles
// through LDS and the skinny tiles of 4 to 8 waves (256 to 512 columns, 64 per wave; the four-wave tiles run two
// workgroups per CU) whose width divides N, each with 1 .. 8 slices along K, and the estimate is
//   rounds of workgroups x (bytes of the workgroups a CU holds / per-CU streaming rate + a start-up time),
// not less than the weight bytes at the rate the memory system gives a whole GPU, plus -- when the output
// leaves as fp32 partial sums for a reduce kernel -- those partial sums written and read back. A wide tile reads
// the activations less often (a small partition is bound by what its CUs can pull); a narrow one, or a deeper
// split, makes more workgroups (a large partition needs them all busy) and fills the last round better: with
// 7 x 2^k columns (the MLP width of the Llama shapes) on 32 or 64 CUs only the 7-wave tile comes out in whole
// rounds.
// `partials`: the output goes through fp32 partial sums (a split needs that; the caller's next kernel reads them).
// Returns the estimated seconds.
struct StreamRates { double rate_128, rate_256, partial_bw, stream_bw_cu, stream_bw_gpu; };
double plan_decode_gemm(const StreamRates& r, int m, int n, int k, int cus, bool may_split, bool partials, int* cfg, int* splits);
StreamRates rates_of(const sts_ctx* ctx) { return StreamRates{ctx->rate_128, ctx->rate_256, ctx->partial_bw, ctx->stream_bw_cu, ctx->stream_bw_gpu}; }
double pick_decode_gemm(const sts_ctx* ctx, int m, int n, int k, int cus, bool may_split, bool partials, int* cfg, int* splits) {
  return plan_decode_gemm(rates_of(ctx), m, n, k, cus, may_split, partials, cfg, splits);
}
// r: measured on the part by the offline profiler -- rate_128 and rate_256 (TFLOP/s per busy CU of 128x128 and 256x256 tiles) and partial_bw (bytes/s
// per CU for partial sums) of the tile model; stream_bw_cu and stream_bw_gpu, what a plain read-only stream reaches per CU of a
// 32-CU partition and on the whole GPU. A GEMM's weight stream gets 0.93 and 0.85 of those (its loads share the CU with the
// operand reads and the matrix cores; the best decode GEMMs measured 55 of 58-59 GB/s per CU and 5.1 of 6 TB/s).
double plan_decode_gemm(const StreamRates& r, int m, int n, int k, int cus, bool may_split, bool partials, int* cfg, int* splits) {
  const int c = std::max(cus, 8);
  const double rate_256 = r.rate_256, partial_bw = r.partial_bw;
  const double cu_rate = 0.93 * r.stream_bw_cu;      // bytes/s one CU pulls from memory for a GEMM's streams
  const double mem_rate = 0.85 * r.stream_bw_gpu;    // bytes/s the memory system gives a full GPU of such streams
  constexpr double start_s = 2.5e-6;                 // a workgroup's first loads and its epilogue
  auto estimate = [&](int cand, int s) {
    const int bn = gemm_tile_n(cand), bm = gemm_tile_m(cand), per_cu = gemm_wgs_per_cu(cand);
    const long long wgs = (long long)((m + bm - 1) / bm) * (n / bn) * s, slots = (long long)c * per_cu;
    const long long rounds = (wgs + slots - 1) / slots, last = wgs - (rounds - 1) * slots;
    const double wg_bytes = 2.0 * (k / s) * (bn + bm);
    // one workgroup alone pulls what its loads in flight allow: on a busy memory system a wave of a skinny tile a
    // sixth of the CU's rate (10 GB/s), the four waves of a tile staged through LDS 0.6 of it (34 GB/s)
    const double wg_rate = cand >= GEMM_64x256S ? std::min(cu_rate, cu_rate / 5.5 * (bn / 64)) : 0.62 * cu_rate;
    auto cu_time = [&](long long held) { return std::max(held * wg_bytes / cu_rate, wg_bytes / wg_rate); };
    // complete rounds hold per_cu workgroups on every CU; the last round what is left, dealt over the CUs
    double t = (rounds - 1) * cu_time(per_cu) + cu_time((last + c - 1) / c);
    t = std::max(t, 2.0 * n * k / mem_rate) + rounds * start_s;
    if (partials) t += 8.0 * s * m * n / (c * partial_bw);
    return t;
  };
  if (m > 64 || n % 128 != 0) {
    *cfg = pick_cfg(m, n, k, cus);
    *splits = may_split ? plan_splits(rate_256, partial_bw, *cfg, m, n, k, cus) : 1;
    return estimate(*cfg, *splits);
  }
  const int s_max = may_split ? std::min(8, std::max(1, k / 512)) : 1;
  double best_t = 1e300;
  *cfg = GEMM_64x128; *splits = 1;
  const int cands[6] = {GEMM_64x256S, GEMM_64x320S, GEMM_64x384S, GEMM_64x448S, GEMM_64x512S, GEMM_64x128};
  for (int cand : cands) {
    if (n % gemm_tile_n(cand) != 0) continue;
    // a GEMM that keeps its output (no partial sums) may carry the SwiGLU epilogue, and the 64x128 tile's form of it
    // (wave tiles of 32 x 64) is slow when a CU holds one workgroup: taken only if no skinny width divides N
    if (!partials && cand == GEMM_64x128 && best_t < 1e300) continue;
    for (int s = 1; s <= s_max; s++) {
      const double t = estimate(cand, s);
      if (t < best_t - 1e-12) { best_t = t; *cfg = cand; *splits = s; }
    }
  }
  return best_t;
}

// Estimated seconds of a GEMM that finishes its own output (gemm_kslice.hip): the weights at the rate of a read-only
// stream, or what its workgroups make the busiest CU pull -- the weights of their 16 or 32 columns and, for each of them, the
// activations of the whole K, whose 16-byte pieces cost about twice their bytes. Measured against it: 28672 x 4096 at 1 / 16 rows
// 37 / 41 us on 256 CUs (38 / 38 estimated), 46 / 62 on 128 (42 / 65), 153 / 220 on 32 (140 / 260).
double kslice_time(const sts_ctx* ctx, int epi, int m, int n, int k, int cus) {
  if (!kslice_covers(n, k)) return HUGE_VAL;         // a vocabulary of 2^23 at hidden 256, 262144 at 8192: the tile forms take those
  const int c = std::max(cus, 8), cols = kslice_cols(epi, n, c), wgs = n / cols;
  const double per_cu = wgs <= c ? 1.0 : (double)wgs / c;
  return std::max(2.0 * n * k / (0.95 * ctx->stream_bw_gpu), per_cu * 2.0 * k * (cols + 2 * m) / (0.93 * ctx->stream_bw_cu)) + 2.5e-6;
}
constexpr double SMALL_KERNEL_S = 4.5e-6;     // one of the kernels that add up partial sums (4.6 to 5.4 us at 1 to 64 rows)

// The GEMMs of one decode layer. kslice: all four finish their own output and no reduce kernel runs; taken when the sum of the
// estimates, with the reduce kernels of the split form, is the smaller one. Otherwise tile and split of each, with SwiGLU in the
// gate/up GEMM unless cutting K is estimated faster. Both measured on 256 CUs, 8B shape: 1 row 73 us of GEMMs against 82 + 20 of
// reduce kernels; at 32 rows 112 us against 86 + 20, so the form ends at 16 rows (one row block of the matrix cores).
struct DecodeGemm { int cfg = 0, splits = 1, row_tiles = 0; bool cols = false; };
struct DecodePlan { bool kslice = false, gu_fused = false; DecodeGemm qkv, o, gu, down; };
// More than 64 rows: the tiles for the slices that pick_decode_gemm decided on -- 128x128, or 256 columns with the rows in any number of
// row tiles, whichever takes the least estimated time. The slices stay, and with them the order of the sums: every shape gives the same
// bits. Estimate: rounds of workgroups at the tile's rate; the first loads and the partial sums of a launch, 8 us, are much the same for all
// shapes and left out. Measured / estimated (with the 8 us) at 223 rows on 256 CUs: 6144 x 4096 in 6 slices 31 / 32 us as 128x128, 26 / 25 in one row tile, 29 / 30 in two; 4096 x 4096 in 8
// slices 21 / 20 in one, 16 / 16 in two; 4096 x 14336 48 / 51 and 39 / 36; 28672 x 4096 in 2 slices 58 / 57 in one row tile.
double pick_tall_tiles(const StreamRates& r, int m, int n, int k, int cus, DecodeGemm* g) {
  if (m <= 64) return HUGE_VAL;
  const int c = std::max(cus, 8), ksteps = k / 64, len = (ksteps + g->splits - 1) / g->splits * 64, blocks = (m + 31) / 32;
  double best = 1e300;
  auto consider = [&](int cfg, int row_tiles, long long wgs, int slots, double tile_s) {
    const double t = (double)((wgs + slots - 1) / slots) * tile_s;
    if (t < best) { best = t; g->cfg = cfg; g->row_tiles = row_tiles; }
  };
  consider(GEMM_128x128, 0, (long long)((m + 127) / 128) * (n / 128) * g->splits, 2 * c, 2.0 * 128 * 128 * len / (r.rate_128 * 1e12 / 2));
  const double tall_s = 2.0 * 256 * 256 * len / (r.rate_256 * 1e12);
  const int least = (blocks + 7) / 8;
  for (int t = least; n % 256 == 0 && t <= std::min(blocks, 2 * least + 2); t++)
    consider(GEMM_256x256, t, (long long)t * (n / 256) * g->splits, c, TILE_HEIGHT_COST[(blocks + t - 1) / t - 1] * tall_s);
  return best;
}

// gemm_cols in the place of tiles for the same slices (the same bits): it leaves partial sums as they do, or takes gate/up whole with
// SwiGLU. Estimate of a launch: the lines its workgroups make a CU pull, or the weights at the whole GPU's rate, and 9 us of first loads,
// output and launch. Measured / estimated on 256 CUs, 28672 x 4096 with SwiGLU: 64 rows 40 / 47 us, 128 rows 50 / 47, 192 rows 56 / 49, 256 rows
// 67 / 63; 57344 x 8192: 96 rows 161 / 161, 192 rows 194 / 188, 256 rows 229 / 224 (tiles and their reduce kernel 214: they stay).
double cols_time(const StreamRates& r, int m, int n, int k, int per_wg, int wgs, int cus) {
  const int held = (wgs + cus - 1) / cus, rows = (m + 31) / 32 * 32;
  return std::max(held * 2.0 * per_wg * (rows + 128) / r.stream_bw_cu, 2.0 * n * k / (0.95 * r.stream_bw_gpu)) + 9e-6;
}
// Partitions that it was measured on, from 128 CUs by 32 (the scheduler's step). On others the shader engines have unequal CUs and two workgroups
// meet on one: 16640 x 4096 with SwiGLU, 130 workgroups on 144 CUs, 96 rows in tiles 55.5 us, so 67.3 (on 160 CUs 55.7 / 43.5).
// Fewer than 128: there the wide tiles of up to 64 rows read the activations less often.
bool cols_covers(int m, int n, int cus) { return cus >= 128 && cus % 32 == 0 && m <= COLS_MAX_ROWS && n % 128 == 0; }
// Where partial sums are left, by 2 500 launches of twelve models on 128 to 256 CUs in both forms (cfg: the tile that it would replace; us in tiles / so).
// Up to 64 rows it replaces 64x128 tiles, which read the same operands, in slices that are long enough beside its start: with one workgroup a CU
// from 16 K tiles up to 32 rows and 24 up to 64 (4096 x 14336 of 17 rows 23.9 / 21.7, of 64 26.2 / 26.0; 22 tiles: 5120 x 8192 of 64 21.1 / 22.2), with two from 20 up
// to 32 rows (10240 x 8192 of 24 rows in 4 slices 39.0 / 36.5; 16 tiles: 6144 x 6144 of 32 on 160 CUs 16.8 / 20.7) and, up to 64, from 32 where some CUs hold one and
// some two (43.4 / 40.9; on all: 8192 x 8192 in 4 slices on 128 CUs 38.4 / 40.5). Skinny tiles of 256 columns and more stay: they pull the rows less often (5120 x 13824 of 32 rows on 128 CUs 34.6 / 40.3,
// 24576 x 16384 of 24 on 224 119 / 136), but for 512 columns in slices of 16 to 31 tiles up to 32 rows, which are short for them (10240 x 8192 of 24 rows in 6 slices on
// 128 CUs 67.7 / 42.7; 56 tiles: 8192 x 28672 of 24 93.6 / 97.9).
// Above 64 rows the launch has to deal evenly (288 workgroups on 256 CUs take as long as 512) and to be estimated faster than the tiles, these at nine tenths
// of the estimate that chose their shape, which rests on a slower tile's rate. With one workgroup on at least three quarters of the CUs (64 workgroups on
// 160, 2048 x 2048 of 256 rows: 13.9 / 17.1) from 16 K tiles (4096 x 14336 of 96 rows 32.9 / 29.0, of 256 43.9 / 41.1), or from 8 above 192 rows with one on every CU and 32 MB of weights (4096 x 4096
// of 223 rows 20.0 / 18.3, but 4608 x 3072 of 224 18.4 / 20.2). With two a CU, up to 192 rows (a CU has LDS for one workgroup of more), from 224 CUs, where HBM and not
// what a CU pulls decides: from 16 tiles up to 96 rows (8192 x 8192 of 80 on 256 32.3 / 30.4, on 192 32.5 / 35.1), from 48 above (8192 x 28672 of 160 112 / 98; 16384 x 8192 in 32 of 160 60.1 / 63.5).
// Three a CU above 64 rows were 0.8 to 0.95 of the tiles' time and are not taken yet.
bool cols_pays(const StreamRates& r, int m, int n, int k, int cfg, int splits, int cus, double t_tall) {
  if (!cols_covers(m, n, cus)) return false;
  const int wgs = n / 128 * splits, held = (wgs + cus - 1) / cus, len = (k / 64 + splits - 1) / splits;
  const bool even = held == 1 || 10 * wgs >= 9 * held * cus;
  if (m <= 64) {
    if (cfg == GEMM_64x512S) return m <= 32 && (held == 3 || held == 4) && len >= 16 && len < 32;
    if (cfg != GEMM_64x128 || held > 2) return false;
    if (held == 1) return len >= (m <= 32 ? 16 : 24);
    return m <= 32 ? len >= 20 : !even && len >= 32;
  }
  if (held == 1 ? 4 * wgs < 3 * cus || (len < 16 && (m <= 192 || wgs < cus || (long long)n * k < 1 << 24))
                : held > 2 || m > 192 || !even || cus < 224 || len < (m <= 96 ? 16 : 48)) return false;
  return cols_time(r, m, n, k, len * 64, wgs, cus) < std::max(0.9 * t_tall, 2.0 * n * k / (0.85 * r.stream_bw_gpu)) + 9e-6;
}

// A GEMM whose partial sums the layer's next kernel adds up, and gate/up, whose SwiGLU is its epilogue or (not fused) that kernel's. Both return
// the estimate that the choice between the layer's forms goes by, which is of the tiles.
double plan_partials(const StreamRates& r, int m, int n, int k, int cus, DecodeGemm* g) {
  const double t = plan_decode_gemm(r, m, n, k, cus, true, true, &g->cfg, &g->splits);
  const double t_tall = pick_tall_tiles(r, m, n, k, cus, g);
  g->cols = cols_pays(r, m, n, k, g->cfg, g->splits, cus, t_tall);
  return t;
}
double plan_gateup(const StreamRates& r, int m, int n, int k, int cus, DecodeGemm* g, bool* gu_fused) {
  DecodeGemm fused;
  const double t_split = plan_decode_gemm(r, m, n, k, cus, true, true, &g->cfg, &g->splits) + 4e-6;
  const double t_fused = plan_decode_gemm(r, m, n, k, cus, false, false, &fused.cfg, &fused.splits);
  const bool can_fuse = fused.cfg == GEMM_64x128 || (fused.cfg >= GEMM_64x256S && fused.cfg <= GEMM_64x512S);
  *gu_fused = can_fuse && (t_fused <= t_split || g->splits == 1);
  if (*gu_fused) { *g = fused; return t_fused; }
  const double t_tall = pick_tall_tiles(r, m, n, k, cus, g), w_bytes = 2.0 * n * k, part_bytes = 4.0 * g->splits * m * n;
  const double t_two = m <= 64 ? t_split : std::max(0.9 * t_tall, w_bytes / (0.85 * r.stream_bw_gpu)) + 9e-6 + SMALL_KERNEL_S + part_bytes / (0.9 * r.stream_bw_gpu);
  // Widths without 256-column tiles (odd multiples of 128) leave 128x128 tiles, which were slower than their estimate and than all rows in a workgroup in each
  // of 105 launches on 128 to 256 CUs: 28800 x 4224 of 96 rows 76.7 / 49.9 us and of 256 rows 109.3 / 73.4 on 256 CUs, 57472 x 8192 of 128 rows on 128 CUs 317 / 303,
  // 11392 x 2176 of 65 rows on 256 CUs 25.0 / 22.9.
  // Above 192 rows a CU has LDS for one workgroup, and launches of more than one a CU lose: 51200 x 5120 of 256 rows on 256 CUs 155.5 / 169.1.
  const bool no_tall = m > 64 && n % 256 != 0;
  g->cols = cols_covers(m, n, cus) && (m <= 192 || n / 128 <= cus || no_tall) && (no_tall || cols_time(r, m, n, k, k, n / 128, cus) < t_two);
  return t_split;
}

DecodePlan decode_layer_plan(const sts_ctx* ctx, int n, int cus) {
  const sts_model_desc& d = ctx->d;
  const StreamRates r = rates_of(ctx);
  DecodePlan p;
  double t = plan_partials(r, n, ctx->qkvn, d.hidden, cus, &p.qkv) + plan_partials(r, n, d.hidden, ctx->qd, cus, &p.o) + plan_partials(r, n, d.hidden, d.mlp, cus, &p.down);
  t += plan_gateup(r, n, 2 * d.mlp, d.hidden, cus, &p.gu, &p.gu_fused) + 3 * SMALL_KERNEL_S;
  if (n <= KSLICE_MAX_ROWS)
    p.kslice = kslice_time(ctx, KS_QKV, n, ctx->qkvn, d.hidden, cus) + kslice_time(ctx, KS_RESID, n, d.hidden, ctx->qd, cus) +
               kslice_time(ctx, KS_SWIGLU, n, 2 * d.mlp, d.hidden, cus) + kslice_time(ctx, KS_RESID, n, d.hidden, d.mlp, cus) < t;
  return p;
}

int64_t now_ns();

// Wait for a stream with a short busy poll before blocking: a layer slice or a decode step lasts
// around a millisecond, and the wake-up latency of a blocking wait would be a visible share of it.
hipError_t wait_stream(hipStream_t st) {
  const int64_t t0 = now_ns();
  for (;;) {
    const hipError_t e = hipStreamQuery(st);
    if (e != hipErrorNotReady) return e;                     // done, or a real error
    if (now_ns() - t0 > 20000000) return hipStreamSynchronize(st);
#if defined(__x86_64__)
    __builtin_ia32_pause();
#endif
  }
}

bool valid_seq(sts_ctx* c, int s) { return s >= 0 && s < (int)c->seqs.size() && c->seqs[s].used; }

// Make `seq` own enough pages for n_tokens; caller holds no lock.
// After a failure between the launches of a step: waits for those already queued, whose metadata the next call rewrites, and
// forgets their timing events and those of the step (a beginning without an end).
void drop_queued(Phase& ph) {
  if (ph.stream) (void)wait_stream(ph.stream);
  ph.kkind.clear(); ph.kused = 0; ph.ran = false;
}

int reserve_pages(sts_ctx* c, const std::vector<std::pair<int, int>>& wants) {   // (seq, tokens)
  std::lock_guard<std::mutex> g(c->alloc_mu);
  size_t need = 0;
  for (auto& w : wants) {
    const int np = (w.second + c->geo.page_tokens - 1) / c->geo.page_tokens;
    if (np > c->p.max_pages_per_seq) return STS_EINVAL;
    need += std::max(0, np - (int)c->seqs[w.first].pages.size());
  }
  if (need > c->free_pages.size()) return STS_ENOMEM;
  for (auto& w : wants) {
    const int np = (w.second + c->geo.page_tokens - 1) / c->geo.page_tokens;
    Seq& s = c->seqs[w.first];
    while ((int)s.pages.size() < np) {
      const int pg = c->free_pages.back(); c->free_pages.pop_back();
      c->page_used[pg] = 1; s.pages.push_back(pg);
    }
  }
  return STS_OK;
}

// Up to this many rows the embedding kernel reads its tokens and positions from pinned host memory (one bus read each) instead
// of waiting for a kernel that copies them. With 8B rows, both kernels / the one: 13.3 / 9.2 us at 64 rows, 17.4 / 12.8 at 512 on 256 CUs and
// 21.3 / 19.3 on 64; at 1024 rows 19.6 / 15.1 on 256 CUs but 29.5 / 31.3 on 64, whose few workgroups wait for the bus in turn
// (8192 rows: 50 / 56 and 114 / 188).
constexpr int META_FUSED_ROWS = 512;
// Logits up to these sizes are stored to host memory by the kernel that reads or writes them last (the head, or greedy sampling on the side), larger ones
// go by a runtime copy, which leaves the stream idle for about 15 us (a program that copied 2 to 4 MB on every step lost 200: 4 rows 590, stored 369). One layer of the 8B shape, vocabulary 128256, us a step by copy / stored.
// A phase alone, logits of a decode step on 256 CUs: 1 row 294 / 270, 16 rows 711 / 627, 64 rows (31 MiB) 1985 / 1896; of a prefill batch of 8 tokens each 311 / 285, 774 / 700,
// 2179 / 2095, on 32 CUs 1085 / 1065 and (64 rows) 3653 / 3102. With tokens: 1 row 298 / 284, 16 rows 721 / 705, 40 rows 1361 / 1342, 48 rows (23.5 MiB) 1591 / 1583, 64 rows 1979 / 1987.
// Both phases at once store at each other's expense on the bus (rows of each, with tokens): 256 / 256 CUs 8 rows 1301 / 907, 16 rows (7.8 MiB) 2457 / 2490, 24 rows 3147 / 3261, 64 rows 6452 / 6858;
// 128 / 128 16 rows 1311 / 1305, 32 rows 2075 / 2173; 224 / 32 16 rows 1557 / 1526, 20 rows 1778 / 1848, 32 rows 2104 / 2294.
constexpr size_t STORED_LOGITS_BYTES = 32 << 20, STORED_WITH_TOKENS_BYTES = 24 << 20, STORED_BESIDE_BYTES = 8 << 20;
size_t stored_logits_bytes(const Phase& ph, bool with_tokens) { return !ph.alone ? STORED_BESIDE_BYTES : with_tokens ? STORED_WITH_TOKENS_BYTES : STORED_LOGITS_BYTES; }

bf16* layer_pool(sts_ctx* c, int l) { return c->pool + (size_t)l * c->pool_layer_elems; }

// Final norm and LM head of n rows into out. x: the residual stream, whose rows (rows idx[i] if idx is given) are normalised
// into xn; null if xn holds them normalised already. With scale.ssq xn holds the rows scaled by the final gains, and a head that
// applies the row factor itself needs no norm. The head runs unsplit, or with K cut over workgroups and a kernel that adds up the partial sums (a small vocabulary has too few tiles:
// 1024 x 4096 took 33 us unsplit against 7 + 4), or as a GEMM that cuts K inside its workgroups.
int run_head(sts_ctx* c, Phase& ph, const float* x, const int* idx, bf16* xn, RowScale scale, int n, float* scratch, size_t scratch_floats, bool nt, float* out) {
  const int v = c->d.vocab, h = c->d.hidden;
  int cfg, one, split_cfg, splits;
  const double t_one = pick_decode_gemm(c, n, v, h, ph.cus, false, false, &cfg, &one);
  const double t_split = pick_decode_gemm(c, n, v, h, ph.cus, true, true, &split_cfg, &splits) + SMALL_KERNEL_S;
  const double t_norm = scale.ssq ? SMALL_KERNEL_S : 0.0;
  const bool split = splits > 1 && t_split < t_one && (size_t)splits * n * v <= scratch_floats;
  const bool kslice = n <= KSLICE_MAX_ROWS && kslice_time(c, KS_F32, n, v, h, ph.cus) < (split ? t_split : t_one) + t_norm;
  if (x && !(kslice && scale.ssq)) {
    KL(ph, STS_K_NORM, rmsnorm_rows(ph.stream, xn, x, c->gf, c->d.rms_eps, n, h, idx));
    scale = RowScale{nullptr, 0, 0.f};
  }
  if (kslice) {
    KL(ph, STS_K_HEAD, kslice_f32(ph.stream, KsliceIn{xn, h, scale, c->lm, n, v, h}, ph.cus, out, v));
  } else if (split) {
    const int ksteps = h / 64, per = (ksteps + splits - 1) / splits, used = (ksteps + per - 1) / per;   // slices the launch makes
    KL(ph, STS_K_HEAD, gemm_bf16(ph.stream, split_cfg, EPI_F32, xn, h, c->lm, h, scratch, v, n, v, h, splits, (long long)n * v, nullptr, true, nt));
    KL(ph, STS_K_REDUCE, reduce_f32(ph.stream, out, scratch, used, (long long)n * v, (size_t)n * v));
  } else {
    KL(ph, STS_K_HEAD, gemm_bf16(ph.stream, cfg, EPI_F32, xn, h, c->lm, h, out, v, n, v, h, 1, 0, nullptr, true, nt));
  }
  return STS_OK;
}

// The GEMMs of a layer's few rows and the kernels that finish them, around the attention: decode steps, and prefill batches of so few
// rows that their GEMMs wait for weights.
struct FewRows {
  sts_ctx* c = nullptr; Phase* ph = nullptr; int n = 0;
  DecodePlan plan;
  bool nt = false;
  RowScale by_rms{}, xn_scale{nullptr, 0, 0.f};

  FewRows() = default;
  FewRows(sts_ctx* c_, Phase& ph_, int n_, const DecodePlan& plan_) : c(c_), ph(&ph_), n(n_), plan(plan_) {
    // On a large partition the decode streams (K and V, the weights of the skinny tiles) are fetched with the non-temporal
    // hint: measured on a 6-layer model, the layer-step is 6 % shorter on 256 CUs (attention 72 -> 63 us), 3 % on 128,
    // and no different on 32, where the same hint cost a prefill slice running beside it 0.5 %.
    nt = ph->cus >= 128;
    // kslice layers: the residual GEMMs leave Xn scaled by the next gains and the rows' sums of squares in ssq
    by_rms = RowScale{ph->ssq, c->d.hidden / kslice_cols(KS_RESID, c->d.hidden, ph->cus), c->d.rms_eps};
  }
  int partials(int kind, const DecodeGemm& gm, const bf16* A, const bf16* W, int N, int K) {
    if (gm.cols) {
      KL((*ph), kind, gemm_cols(ph->stream, EPI_F32, A, K, W, ph->part, N, n, N, K, gm.splits, (long long)n * N));
    } else {
      KL((*ph), kind, gemm_bf16(ph->stream, gm.cfg, EPI_F32, A, K, W, K, ph->part, N, n, N, K, gm.splits, (long long)n * N, nullptr, true, nt, gm.row_tiles));
    }
    return STS_OK;
  }
  // Xn (normalised, or as xn_scale says) through the QKV projection: rotated queries to q_out, K and V to the rows' places
  int qkv(int l, bf16* q_out) {
    const sts_model_desc& d = c->d;
    const LayerW& w = c->layers[l];
    if (plan.kslice) {
      KL((*ph), STS_K_QKV, kslice_qkv(ph->stream, KsliceIn{ph->Xn, d.hidden, xn_scale, w.wqkv, n, c->qkvn, d.hidden}, ph->d_place, ph->rot, q_out, layer_pool(c, l), c->geo, d.n_q_heads));
      return STS_OK;
    }
    STSCK(partials(STS_K_QKV, plan.qkv, ph->Xn, w.wqkv, c->qkvn, d.hidden));
    KL((*ph), STS_K_ROPE, decode_qkv_finish(ph->stream, ph->part, plan.qkv.splits, (long long)n * c->qkvn, c->qkvn, ph->d_place, ph->rot, q_out, layer_pool(c, l), c->geo, n, d.n_q_heads));
    return STS_OK;
  }
  // The attention's output through the rest of the layer. Leaves X, and Xn for the next layer, whose gains next_gain are.
  int rest(int l, const float* next_gain) {
    const sts_model_desc& d = c->d;
    const LayerW& w = c->layers[l];
    const int h = d.hidden, norm_kind = ph->side == 0 ? STS_K_NORM : STS_K_REDUCE;
    hipStream_t st = ph->stream;
    if (plan.kslice) {
      KL((*ph), STS_K_O, kslice_resid(st, KsliceIn{ph->A, c->qd, RowScale{nullptr, 0, 0.f}, w.wo, n, h, c->qd}, ph->cus, ph->X, w.g2, ph->Xn, ph->ssq));
      KL((*ph), STS_K_GATEUP, kslice_swiglu(st, KsliceIn{ph->Xn, h, by_rms, w.wgu, n, 2 * d.mlp, h}, ph->H));
      KL((*ph), STS_K_DOWN, kslice_resid(st, KsliceIn{ph->H, d.mlp, RowScale{nullptr, 0, 0.f}, w.wd, n, h, d.mlp}, ph->cus, ph->X, next_gain, ph->Xn, ph->ssq));
      xn_scale = by_rms;
      return STS_OK;
    }
    STSCK(partials(STS_K_O, plan.o, ph->A, w.wo, h, c->qd));
    KL((*ph), norm_kind, reduce_resid_norm(st, ph->X, ph->part, plan.o.splits, (long long)n * h, ph->Xn, w.g2, d.rms_eps, n, h));
    if (plan.gu_fused) {
      KL((*ph), STS_K_GATEUP, gemm_bf16(st, plan.gu.cfg, EPI_SWIGLU_BF16, ph->Xn, h, w.wgu, h, ph->H, d.mlp, n, 2 * d.mlp, h, 1, 0, nullptr, true, nt));
    } else if (plan.gu.cols) {
      KL((*ph), STS_K_GATEUP, gemm_cols(st, EPI_SWIGLU_BF16, ph->Xn, h, w.wgu, ph->H, d.mlp, n, 2 * d.mlp, h, plan.gu.splits, 0));
    } else {
      STSCK(partials(STS_K_GATEUP, plan.gu, ph->Xn, w.wgu, 2 * d.mlp, h));
      KL((*ph), STS_K_SWIGLU, reduce_swiglu(st, ph->H, ph->part, plan.gu.splits, (long long)n * 2 * d.mlp, n, d.mlp));
    }
    STSCK(partials(STS_K_DOWN, plan.down, ph->H, w.wd, h, d.mlp));
    KL((*ph), norm_kind, reduce_resid_norm(st, ph->X, ph->part, plan.down.splits, (long long)n * h, ph->Xn, next_gain, d.rms_eps, n, h));
    return STS_OK;
  }
};

// ------------------------------------------------------------------------------------ prefill
// Checks of a prefill slice that touch no state: arguments, the order of layer slices, and the
// pages the batch will need (appended to `wants` for slice 0). Nothing is launched or reserved.
int prefill_validate(sts_ctx* c, int n_seqs, const int32_t* seqs, const int32_t* lens, const int32_t* tokens, int lb, int le,
                     std::vector<std::pair<int, int>>* wants) {
  Phase& ph = c->ph[0];
  const sts_model_desc& d = c->d;
  if (n_seqs < 1 || n_seqs > c->p.max_prefill_seqs || !seqs || !lens) return STS_EINVAL;
  if (lb < 0 || le <= lb || le > d.n_layers) return STS_EINVAL;
  if (ph.stream == nullptr) return STS_ESTATE;               // prefill suspended (0 CUs)
  int rows = 0;
  for (int i = 0; i < n_seqs; i++) {
    if (!valid_seq(c, seqs[i]) || lens[i] < 1) return STS_EINVAL;
    for (int j = 0; j < i; j++) if (seqs[j] == seqs[i]) return STS_EINVAL;
    rows += lens[i];
    if (rows > c->p.max_prefill_tokens) return STS_EINVAL;
  }
  std::lock_guard<std::mutex> g(c->state_mu);
  for (int i = 0; i < n_seqs; i++) for (int s : c->pend_dseqs) if (s == seqs[i]) return STS_EINVAL;   // a request is in one phase only
  if (lb == 0) {
    if (!tokens) return STS_EINVAL;
    for (int i = 0; i < rows; i++) if (tokens[i] < 0 || tokens[i] >= d.vocab) return STS_EINVAL;
    if (c->pf_active) return STS_ESTATE;
    for (int i = 0; i < n_seqs; i++) {
      const int total = c->seqs[seqs[i]].len + lens[i];
      if ((total + c->geo.page_tokens - 1) / c->geo.page_tokens > c->p.max_pages_per_seq) return STS_EINVAL;
      wants->push_back({seqs[i], total});
    }
  } else {
    if (!c->pf_active || lb != c->pf_next_layer || (int)c->pf_seqs.size() != n_seqs) return STS_ESTATE;
    for (int i = 0; i < n_seqs; i++) if (c->pf_seqs[i] != seqs[i] || c->pf_lens[i] != lens[i]) return STS_ESTATE;
  }
  return STS_OK;
}

// Queues a validated slice whose pages are reserved. A failure in here (a HIP error) leaves nothing of it in flight and drops the
// batch: the residual stream of its rows is neither that of this slice's beginning nor of its end.
struct DecodeRun;
int prefill_launch_checked(sts_ctx* c, int n_seqs, const int32_t* seqs, const int32_t* lens, const int32_t* tokens,
                           int lb, int le, bool want_logits, DecodeRun* beside = nullptr);

int prefill_enqueue(sts_ctx* c, int n_seqs, const int32_t* seqs, const int32_t* lens, const int32_t* tokens,
                    int lb, int le, bool want_logits) {
  std::vector<std::pair<int, int>> wants;
  STSCK(prefill_validate(c, n_seqs, seqs, lens, tokens, lb, le, &wants));
  STSCK(reserve_pages(c, wants));
  return prefill_launch_checked(c, n_seqs, seqs, lens, tokens, lb, le, want_logits);
}

int prefill_launch_body(sts_ctx* c, int n_seqs, const int32_t* seqs, const int32_t* lens, const int32_t* tokens,
                        int lb, int le, bool want_logits, DecodeRun* beside);

// beside: a decode step that is queued in turns with this slice, a layer each, on its own stream; the caller queues what is left of it.
int prefill_launch_checked(sts_ctx* c, int n_seqs, const int32_t* seqs, const int32_t* lens, const int32_t* tokens,
                           int lb, int le, bool want_logits, DecodeRun* beside) {
  if (lb == 0) {
    std::lock_guard<std::mutex> g(c->state_mu);
    c->pf_active = true; c->pf_next_layer = 0;
    c->pf_seqs.assign(seqs, seqs + n_seqs); c->pf_lens.assign(lens, lens + n_seqs);
  }
  const int rc = prefill_launch_body(c, n_seqs, seqs, lens, tokens, lb, le, want_logits, beside);
  if (rc != STS_OK) {
    drop_queued(c->ph[0]);
    (void)sts_prefill_abort(c);
  }
  return rc;
}

int prefill_finish(sts_ctx* c, int n_seqs, const int32_t* seqs, const int32_t* lens, int le, float* logits) {
  Phase& ph = c->ph[0];
  HIPCK(wait_stream(ph.stream));
  STSCK(k_collect(c, ph));
  c->pf_next_layer = le;
  if (le == c->d.n_layers) {
    for (int i = 0; i < n_seqs; i++) c->seqs[seqs[i]].len += lens[i];
    { std::lock_guard<std::mutex> g(c->state_mu); c->pf_active = false; }
    if (logits) std::memcpy(logits, ph.h_logits, (size_t)n_seqs * c->d.vocab * sizeof(float));
  }
  return STS_OK;
}

// ------------------------------------------------------------------------------------ decode
// Context chunks of at most chunk_pages pages: the largest of 64/32/16/8 that still yields about
// four workgroups per CU of the partition (8 pages keep the four waves of a workgroup busy with
// one two-page block each), never more than 128 chunks for the longest context. Also where every context would fit one chunk and need no merge: left whole, 1
// request of 150 tokens took 86.4 us a layer for 88.0, 32 of 700 115.1 for 122.1 (256 CUs, hidden 4096), but the logits were further from 64 bits, 0.008363 ->
// 0.008398 in the mean of 230 steps (paired difference 3.5e-5 +- 0.5e-5, with other weights 3.2e-5): the largest probability of a wave's part of a chunk is
// 1, which bf16 holds exactly, and fewer chunks have fewer of them.
void decode_chunk_plan(const int* n_pages, int n, int n_kv, int cus, int page_tokens, int* chunk_pages_out, int* max_chunks_out) {
  int max_pages = 1;
  for (int i = 0; i < n; i++) max_pages = std::max(max_pages, n_pages[i]);
  int chunk_pages = attn_decode_max_chunk_tokens() / page_tokens;
  const int floor_pages = std::max(8, (max_pages + 127) / 128);
  while (chunk_pages / 2 >= floor_pages) {
    long long wgs = 0;
    for (int i = 0; i < n; i++) wgs += (n_pages[i] + chunk_pages - 1) / chunk_pages;
    if (wgs * n_kv >= 4LL * cus) break;
    chunk_pages /= 2;
  }
  *chunk_pages_out = chunk_pages;
  *max_chunks_out = (max_pages + chunk_pages - 1) / chunk_pages;
}
// Chunks per context the merge workspace and the work list are allocated for: chunks hold at least
// 8 pages (fewer than one chunk per 4 pages), and never more than 128 per context.
int decode_max_chunks(int max_pages_per_seq) { return (int)std::min<size_t>(128, ((size_t)max_pages_per_seq + 3) / 4); }

// Checks of a decode step that touch no state; the page each request needs for its new token is
// appended to `wants`.
int decode_validate(sts_ctx* c, const int32_t* seqs, const int32_t* in_tokens, int n, std::vector<std::pair<int, int>>* wants) {
  Phase& ph = c->ph[1];
  const sts_model_desc& d = c->d;
  if (n < 1 || n > c->p.max_decode_batch || !seqs || !in_tokens) return STS_EINVAL;
  if (ph.stream == nullptr) return STS_ESTATE;               // decode suspended (0 CUs)
  std::vector<char> seen(c->seqs.size());
  for (int i = 0; i < n; i++) {
    if (!valid_seq(c, seqs[i]) || in_tokens[i] < 0 || in_tokens[i] >= d.vocab) return STS_EINVAL;
    if (seen[seqs[i]]++) return STS_EINVAL;
    if ((c->seqs[seqs[i]].len + 1 + c->geo.page_tokens - 1) / c->geo.page_tokens > c->p.max_pages_per_seq) return STS_EINVAL;
  }
  {
    std::lock_guard<std::mutex> g(c->state_mu);                                        // a request is in one phase only
    if (c->pf_active) for (int i = 0; i < n; i++) for (int s : c->pf_seqs) if (s == seqs[i]) return STS_EINVAL;
  }
  for (int i = 0; i < n; i++) wants->push_back({seqs[i], c->seqs[seqs[i]].len + 1});
  return STS_OK;
}

int decode_launch_checked(sts_ctx* c, const int32_t* seqs, const int32_t* in_tokens, int n, bool want_logits, bool want_next);

int decode_enqueue(sts_ctx* c, const int32_t* seqs, const int32_t* in_tokens, int n, bool want_logits, bool want_next) {
  std::vector<std::pair<int, int>> wants;
  STSCK(decode_validate(c, seqs, in_tokens, n, &wants));
  STSCK(reserve_pages(c, wants));
  return decode_launch_checked(c, seqs, in_tokens, n, want_logits, want_next);
}

// A validated decode step whose pages are reserved, queued in pieces: its metadata and embedding, the layers one by one, the head.
struct DecodeRun {
  sts_ctx* c; const int32_t* seqs; const int32_t* in_tokens; int n; bool want_logits, want_next;
  int rc = STS_OK, layer = -1;                               // first failure; next piece (-1: not begun)
  int n_items = 0, n_multi = 0, chunk_pages = 0, max_chunks = 0;
  DecodeMerge* d_multi = nullptr;
  RowRotation rot{};
  FewRows few;

  int begin();
  int one_layer(int l);
  int end();
  void turn() {                                              // the next piece; none once all layers are queued
    if (rc != STS_OK || layer >= c->d.n_layers) return;
    rc = layer < 0 ? begin() : one_layer(layer);
    layer++;
  }
  int finish_queue() {                                       // what is left
    while (rc == STS_OK && layer < c->d.n_layers) turn();
    if (rc == STS_OK) rc = end();
    if (rc != STS_OK) drop_queued(c->ph[1]);
    return rc;
  }
};

int decode_launch_checked(sts_ctx* c, const int32_t* seqs, const int32_t* in_tokens, int n, bool want_logits, bool want_next) {
  return DecodeRun{c, seqs, in_tokens, n, want_logits, want_next}.finish_queue();
}

int DecodeRun::begin() {
  Phase& ph = c->ph[1];
  const sts_model_desc& d = c->d;
  const int mp = c->p.max_pages_per_seq, pt = c->geo.page_tokens;
  ph.meta_used = 0;
  meta_take(ph, &ph.h_dseq, &ph.d_dseq, n);
  meta_take(ph, &ph.h_tokens, &ph.d_tokens, n);
  meta_take(ph, &ph.h_pos, &ph.d_pos, n);
  meta_take(ph, &ph.h_place, &ph.d_place, n);
  size_t bt_entries = 0;                                     // block tables are packed back to back
  for (int i = 0; i < n; i++) bt_entries += (c->seqs[seqs[i]].len + 1 + pt - 1) / pt;
  meta_take(ph, &ph.h_bt, &ph.d_bt, bt_entries);
  if (ph.meta_used > ph.meta_bytes) return STS_EINVAL;
  int max_pages = 1, bt_off = 0;
  for (int i = 0; i < n; i++) {
    const Seq& s = c->seqs[seqs[i]];
    const int np = (s.len + 1 + pt - 1) / pt;
    ph.h_dseq[i] = DecodeSeq{s.len, bt_off, np};
    std::memcpy(ph.h_bt + bt_off, s.pages.data(), np * sizeof(int));
    bt_off += np;
    max_pages = std::max(max_pages, np);
    ph.h_tokens[i] = in_tokens[i];
    ph.h_pos[i] = s.len;
    ph.h_place[i] = s.pages[s.len / pt] * pt + s.len % pt;
  }
  std::vector<int> np_list(n);
  for (int i = 0; i < n; i++) np_list[i] = ph.h_dseq[i].n_pages;
  decode_chunk_plan(np_list.data(), n, d.n_kv_heads, ph.cus, pt, &chunk_pages, &max_chunks);
  if (max_chunks > decode_max_chunks(mp)) return STS_EINVAL;   // cannot happen within sts_init's bound on max_pages_per_seq
  // One attention workgroup row per context chunk that exists, longest chunks first: the workgroups that finish the launch are then the
  // short ones. A context's chunks are equal (its pages / chunks), so a pass over the requests counts the items of each length and a second
  // one places them, in the requests' order.
  auto chunks_of = [&](int i) { return (np_list[i] + chunk_pages - 1) / chunk_pages; };
  std::vector<int> place(chunk_pages + 2, 0);                // place[chunk_pages - length]: where the next item of that length goes
  for (int i = 0; i < n; i++) {
    const int chunks = chunks_of(i);
    place[chunk_pages - (np_list[i] + chunks - 1) / chunks + 1] += chunks;
    n_items += chunks;
  }
  for (int b = 1; b <= chunk_pages; b++) place[b] += place[b - 1];
  meta_take(ph, &ph.h_ditems, &ph.d_ditems, n_items);
  if (ph.meta_used > ph.meta_bytes) return STS_EINVAL;
  for (int i = 0; i < n; i++) {
    const int chunks = chunks_of(i);
    int& at = place[chunk_pages - (np_list[i] + chunks - 1) / chunks];
    for (int ch = 0; ch < chunks; ch++) ph.h_ditems[at++] = DecodeItem{i, ch, ph.h_dseq[i].cl, ph.h_dseq[i].bt_off};
  }
  // requests whose context has more than one chunk: only they need the merge kernel
  DecodeMerge* h_multi = nullptr;
  meta_take(ph, &h_multi, &d_multi, (size_t)n);
  if (ph.meta_used > ph.meta_bytes) return STS_EINVAL;
  for (int i = 0; i < n; i++)
    if (ph.h_dseq[i].n_pages > chunk_pages) h_multi[n_multi++] = DecodeMerge{i, (ph.h_dseq[i].n_pages + chunk_pages - 1) / chunk_pages};
  hipStream_t st = ph.stream;
  HIPCK(hipEventRecord(ph.ev0, st));
  const int h = d.hidden;
  const MetaCopy meta{ph.h_meta, ph.d_meta, (int)ph.meta_used};
  const bool fused_meta = h <= 8192 && n <= META_FUSED_ROWS;
  rot = RowRotation{ph.rot, fused_meta ? ph.h_pos : ph.d_pos, c->inv_freq, d.head_dim};
  if (!fused_meta) KL(ph, STS_K_EMBED, copy_in(st, meta));
  if (h <= 8192) {
    KL(ph, STS_K_EMBED, embed_norm_rows(st, ph.X, ph.Xn, c->emb, fused_meta ? ph.h_tokens : ph.d_tokens, c->layers[0].g1, d.rms_eps, n, h, rot, fused_meta ? meta : MetaCopy{nullptr, nullptr, 0}));
  } else {
    KL(ph, STS_K_EMBED, embed_rows(st, ph.X, c->emb, ph.d_tokens, n, h));
    KL(ph, STS_K_NORM, rmsnorm_rows(st, ph.Xn, ph.X, c->layers[0].g1, d.rms_eps, n, h));
    KL(ph, STS_K_ROPE, row_rotation(st, rot, n));
  }
  few = FewRows(c, ph, n, decode_layer_plan(c, n, ph.cus));
  return STS_OK;
}

int DecodeRun::one_layer(int l) {
  Phase& ph = c->ph[1];
  const sts_model_desc& d = c->d;
  STSCK(few.qkv(l, ph.Q));
  KL(ph, STS_K_ATTN, attn_decode(ph.stream, ph.Q, ph.A, ph.d_dseq, ph.d_ditems, n_items, d_multi, n_multi, ph.d_bt, layer_pool(c, l), c->geo, n, d.n_q_heads, chunk_pages, max_chunks, ph.attn_ws, few.nt));
  return few.rest(l, (l + 1 < d.n_layers) ? c->layers[l + 1].g1 : c->gf);
}

int DecodeRun::end() {
  Phase& ph = c->ph[1];
  const sts_model_desc& d = c->d;
  hipStream_t st = ph.stream;
  if (want_logits || want_next) {
    // (the last reduce kernel of the split form has written Xn normalised)
    const size_t bytes = (size_t)n * d.vocab * sizeof(float);
    const bool stored = want_logits && bytes <= stored_logits_bytes(ph, want_next), direct = stored && !want_next;
    STSCK(run_head(c, ph, few.plan.kslice ? ph.X : nullptr, nullptr, ph.Xn, few.xn_scale, n, ph.part, ph.part_floats, few.nt, direct ? ph.h_logits : ph.logits));
    if (want_next) KL(ph, STS_K_SAMPLE, argmax_rows(st, ph.h_best, ph.logits, n, d.vocab, stored ? ph.h_logits : nullptr));
    if (want_logits && !stored) HIPCK(hipMemcpyAsync(ph.h_logits, ph.logits, bytes, hipMemcpyDeviceToHost, st));
  }
  HIPCK(hipEventRecord(ph.ev1, st));
  ph.ran = true; ph.rows = n;
  return STS_OK;
}

// A prefill batch of few rows waits for its weights, as a decode step does, and takes the same GEMMs (but not the form that leaves rows
// scaled: a row's norm is rounded as in a larger batch), where its partition is the whole GPU. On a part of it they are as fast, but take from
// the decode step beside them what they gain: 45 rows beside 71 requests on 128 / 128 CUs 418 -> 390 us for the slice, 499 -> 515 for the step; 100 rows beside 2 requests on 224 / 32
// 370 -> 311 and 660 -> 702. Where both phases have the whole GPU and a decode step does run beside, the whole step is the shorter one (four layers, us: 45 rows beside 16 requests
// 906 -> 734, 100 beside 71 1066 -> 983, 200 beside 2 999 -> 934; hidden 8192, two layers, 16 beside 16 1241 -> 1132, 100 beside 71 1468 -> 1422; 16 beside 71 934 -> 952 is the one of 24 that is
// not), though one phase of it may take longer (hidden 8192, 45 beside 2: the slice 1207 -> 1163, the decode step 898 -> 1062). So the partition alone decides, and a
// batch's numbers do not depend on what runs beside it.
// Distance of the logits from 64 bits, tiles / so: 0.009524 / 0.009526 in the mean of 300 batches of 1 to 256 rows (paired difference 2.5e-6 +- 4.5e-6).
// Up to 64 rows: its 64x128 tiles unsplit, with a cut last wave, pull less than split and skinny tiles. Device time of 2 layers, before / now: 1 row 264 / 187 us,
// 16 rows 266 / 189, 64 rows 291 / 210; hidden 8192 8 rows 678 / 563, 64 rows 708 / 604. Up to 16 rows not where the layer is launches (hidden 256: 8 rows 69 / 70). From 17 to 64 rows in a
// layer of any size (four layers, 17 and 64 rows: hidden 256 144 / 139 and 169 / 146, 512 176 / 168 and 183 / 177, 1024 201 / 169 and 214 / 182, 2048 273 / 209 and 298 / 233, 3072 407 / 304 and 433 / 352).
// Beyond, all four through gemm_cols in as many slices as give every CU a workgroup, where both sides' estimates say so: a tile launch and
// its fix-up or norm at three quarters of the estimate that chose its shape (which rests on a slower tile's rate) plus 12 us. 65 rows 298 / 226 us, 96 rows 305 / 251,
// 160 rows 358 / 294, 256 rows 389 / 360; hidden 8192 96 rows 740 / 657, 128 rows 776 / 711; 192 rows 888 for 820, which it leaves. Above 256 rows the tiles of
// two row tiles are level. Eleven more models (hidden 2048 to 16384, MLP 8192 to 28736, widths without 256-column tiles among them), 165 batches of 1 to 256 rows: 0.69 to 1.013 of the tiles'
// time, 0.87 in the mean.
constexpr int FEW_ROWS_MAX = 256;
bool prefill_few_rows(sts_ctx* c, Phase& ph, int rows, const PrefillGemm (&tiles)[4], FewRows* few) {
  if (rows > FEW_ROWS_MAX || ph.cus < c->n_cu) return false;
  const sts_model_desc& d = c->d;
  const double w_s = 2.0 * ((double)c->qkvn * d.hidden + (double)d.hidden * c->qd + 3.0 * d.mlp * d.hidden) / c->stream_bw_gpu;   // a layer's weights
  if ((rows <= 16 || rows > 64) && w_s < 20e-6) return false;
  DecodePlan p = decode_layer_plan(c, rows, ph.cus);
  p.kslice = false;
  if (rows > 64) {
    const int shape[4][2] = {{c->qkvn, d.hidden}, {d.hidden, c->qd}, {d.hidden, d.mlp}, {2 * d.mlp, d.hidden}};
    DecodeGemm* gm[4] = {&p.qkv, &p.o, &p.down, &p.gu};
    double t_tiles = 0.0, t_cols = 0.0;
    for (int i = 0; i < 4; i++) {
      const int n = shape[i][0], k = shape[i][1], cut = i == 3 ? 1 : std::max(1, std::min(std::min(8, k / 512), ph.cus / (n / 128)));
      const int len = (k / 64 + cut - 1) / cut, used = (k / 64 + len - 1) / len;
      *gm[i] = DecodeGemm{GEMM_128x128, used, 0, true};
      t_tiles += std::max(0.75 * tiles[i].est_s, 2.0 * n * k / (0.85 * c->stream_bw_gpu)) + 12e-6;
      t_cols += cols_time(rates_of(c), rows, n, k, len * 64, n / 128 * used, ph.cus) + (i == 3 ? 0.0 : SMALL_KERNEL_S + 4.0 * used * rows * n / 4e12);
    }
    if (t_tiles <= 1.03 * t_cols) return false;
    p.gu_fused = false;
  }
  auto fits = [&](const DecodeGemm& g, int n) { return (size_t)g.splits * rows * n <= ph.part_floats; };
  if (!(fits(p.qkv, c->qkvn) && fits(p.o, d.hidden) && fits(p.down, d.hidden) && (p.gu_fused || p.gu.cols || fits(p.gu, 2 * d.mlp)))) return false;
  *few = FewRows(c, ph, rows, p);
  return true;
}

int prefill_launch_body(sts_ctx* c, int n_seqs, const int32_t* seqs, const int32_t* lens, const int32_t* tokens,
                        int lb, int le, bool want_logits, DecodeRun* beside) {
  Phase& ph = c->ph[0];
  const sts_model_desc& d = c->d;
  int rows = 0;
  for (int i = 0; i < n_seqs; i++) rows += lens[i];
  std::vector<int> priors(n_seqs);
  for (int i = 0; i < n_seqs; i++) priors[i] = c->seqs[seqs[i]].len;
  const AttnPlan attn = attn_prefill_plan(n_seqs, lens, priors.data(), d.n_q_heads, 2 * ph.cus, ph.max_attn_extra,
                                          (long long)(ph.tail_ws_bytes / sizeof(float) / attn_prefill_part_floats(d.n_q_heads, d.head_dim)));
  const int n_items = (int)attn.items.size(), n_merges = (int)attn.merges.size(), attn_heads = attn_prefill_heads(attn.pairs, d.n_q_heads, d.n_kv_heads, d.head_dim);
  auto pick = [&](int n, int k) { return pick_prefill_gemm(c, rows, n, k, ph.cus, ph.tail_ws_bytes); };
  const int h = d.hidden;
  const PrefillGemm g_qkv = pick(c->qkvn, h), g_o = pick(h, c->qd), g_gu = pick(2 * d.mlp, h), g_down = pick(h, d.mlp);
  FewRows few;
  const bool few_rows = prefill_few_rows(c, ph, rows, {g_qkv, g_o, g_down, g_gu}, &few);
  const bool qkv_places = few_rows || g_qkv.cfg == GEMM_256x256;   // the QKV GEMM, or what finishes it, writes K and V to the rows' places
  // ---- stage metadata
  ph.meta_used = 0;
  meta_take(ph, &ph.h_pseq, &ph.d_pseq, n_seqs);
  meta_take(ph, &ph.h_rows, &ph.d_rows, n_seqs);
  meta_take(ph, &ph.h_items, &ph.d_items, n_items);
  AttnMerge *h_merges = nullptr, *d_merges = nullptr;
  meta_take(ph, &h_merges, &d_merges, n_merges);
  meta_take(ph, &ph.h_tokens, &ph.d_tokens, lb == 0 ? rows : 0);
  meta_take(ph, &ph.h_pos, &ph.d_pos, lb == 0 ? rows : 0);
  meta_take(ph, &ph.h_place, &ph.d_place, qkv_places ? rows : 0);
  size_t bt_entries = 0;                                     // block tables are packed back to back
  for (int i = 0; i < n_seqs; i++) bt_entries += c->seqs[seqs[i]].pages.size();
  meta_take(ph, &ph.h_bt, &ph.d_bt, bt_entries);
  if (ph.meta_used > ph.meta_bytes) return STS_EINVAL;
  int r0 = 0, bt_off = 0;
  for (int i = 0; i < n_seqs; i++) {
    const Seq& s = c->seqs[seqs[i]];
    ph.h_pseq[i] = PrefillSeq{r0, lens[i], s.len, bt_off, (int)s.pages.size()};
    std::memcpy(ph.h_bt + bt_off, s.pages.data(), s.pages.size() * sizeof(int));
    bt_off += (int)s.pages.size();
    ph.h_rows[i] = r0 + lens[i] - 1;
    for (int j = 0; lb == 0 && j < lens[i]; j++) ph.h_pos[r0 + j] = s.len + j;
    for (int j = 0, pt = c->geo.page_tokens; qkv_places && j < lens[i];) {   // a page's slots follow each other
      const int slot = (s.len + j) % pt, end = std::min(j + pt - slot, lens[i]);
      for (int place = s.pages[(s.len + j) / pt] * pt + slot; j < end; j++) ph.h_place[r0 + j] = place++;
    }
    r0 += lens[i];
  }
  std::memcpy(ph.h_items, attn.items.data(), n_items * sizeof(AttnItem));
  if (n_merges > 0) std::memcpy(h_merges, attn.merges.data(), n_merges * sizeof(AttnMerge));
  hipStream_t st = ph.stream;
  HIPCK(hipEventRecord(ph.ev0, st));
  if (lb == 0) std::memcpy(ph.h_tokens, tokens, rows * sizeof(int));
  const bool fused_embed = lb == 0 && h <= 8192;             // the embedding kernel also writes layer 0's normalised rows
  const MetaCopy meta{ph.h_meta, ph.d_meta, (int)ph.meta_used};
  // few rows: the embedding kernel reads tokens and positions from host memory itself and copies the metadata on the side
  const bool fused_meta = fused_embed && rows <= META_FUSED_ROWS;
  RowRotation rot{ph.rot, fused_meta ? ph.h_pos : ph.d_pos, c->inv_freq, d.head_dim};
  if (!fused_meta) KL(ph, STS_K_EMBED, copy_in(st, meta));
  if (fused_embed) {
    KL(ph, STS_K_EMBED, embed_norm_rows(st, ph.X, ph.Xn, c->emb, fused_meta ? ph.h_tokens : ph.d_tokens, c->layers[0].g1, d.rms_eps, rows, h, rot, fused_meta ? meta : MetaCopy{nullptr, nullptr, 0}));
  } else if (lb == 0) {
    KL(ph, STS_K_EMBED, embed_rows(st, ph.X, c->emb, ph.d_tokens, rows, h));
    KL(ph, STS_K_ROPE, row_rotation(st, rot, rows));
  }
  if (beside) beside->turn();
  bool normed = fused_embed;                                 // Xn holds this layer's input already
  for (int l = lb; l < le; l++) {
    const LayerW& w = c->layers[l];
    ResidNorm post{ph.Xn, w.g2, d.rms_eps, false}, next{ph.Xn, l + 1 < le ? c->layers[l + 1].g1 : nullptr, d.rms_eps, false};
    if (!normed) KL(ph, STS_K_NORM, rmsnorm_rows(st, ph.Xn, ph.X, w.g1, d.rms_eps, rows, h));
    if (few_rows) {
      STSCK(few.qkv(l, ph.QKV));
    } else if (qkv_places) {
      const QkvOut out{ph.rot, ph.d_place, layer_pool(c, l), c->geo, d.n_q_heads};
      KL(ph, STS_K_QKV, prefill_gemm(ph, g_qkv, EPI_QKV, ph.Xn, h, w.wqkv, h, ph.QKV, c->qkvn, rows, c->qkvn, h, nullptr, &out));
    } else {
      KL(ph, STS_K_QKV, prefill_gemm(ph, g_qkv, EPI_BF16, ph.Xn, h, w.wqkv, h, ph.QKV, c->qkvn, rows, c->qkvn, h));
      KL(ph, STS_K_ROPE, rope_kv_write_prefill(st, ph.QKV, c->qkvn, ph.d_pseq, n_seqs, ph.d_bt, ph.rot, layer_pool(c, l), c->geo, rows, d.n_q_heads));
    }
    KL(ph, STS_K_ATTN, attn_prefill(st, ph.QKV, few_rows ? c->qd : c->qkvn, ph.A, c->qd, ph.d_pseq, ph.d_items, n_items, attn_heads, d_merges, n_merges, ph.d_bt, layer_pool(c, l), c->geo, d.n_q_heads, ph.tail_ws));
    if (few_rows) {
      STSCK(few.rest(l, l + 1 < d.n_layers ? c->layers[l + 1].g1 : c->gf));
      normed = true;
      if (beside) beside->turn();
      continue;
    }
    KL(ph, STS_K_O, prefill_gemm(ph, g_o, EPI_RESID_F32, ph.A, c->qd, w.wo, c->qd, ph.X, h, rows, h, c->qd, &post));
    if (!post.done) KL(ph, STS_K_NORM, rmsnorm_rows(st, ph.Xn, ph.X, w.g2, d.rms_eps, rows, h));
    KL(ph, STS_K_GATEUP, prefill_gemm(ph, g_gu, EPI_SWIGLU_BF16, ph.Xn, h, w.wgu, h, ph.H, d.mlp, rows, 2 * d.mlp, h));
    KL(ph, STS_K_DOWN, prefill_gemm(ph, g_down, EPI_RESID_F32, ph.H, d.mlp, w.wd, d.mlp, ph.X, h, rows, h, d.mlp, l + 1 < le ? &next : nullptr));
    normed = next.done;
    if (beside) beside->turn();
  }
  if (le == d.n_layers && want_logits) {
    const size_t bytes = (size_t)n_seqs * d.vocab * sizeof(float);
    const bool direct = bytes <= stored_logits_bytes(ph, false);   // the head's last kernel stores to host memory
    STSCK(run_head(c, ph, ph.X, ph.d_rows, ph.Xlast_n, RowScale{nullptr, 0, 0.f}, n_seqs, ph.tail_ws, ph.tail_ws_bytes / sizeof(float), false, direct ? ph.h_logits : ph.logits));
    if (!direct) HIPCK(hipMemcpyAsync(ph.h_logits, ph.logits, bytes, hipMemcpyDeviceToHost, st));
  }
  HIPCK(hipEventRecord(ph.ev1, st));
  ph.ran = true; ph.rows = rows;
  return STS_OK;
}

int decode_finish(sts_ctx* c, const int32_t* seqs, int n, float* logits, int32_t* next) {
  Phase& ph = c->ph[1];
  HIPCK(wait_stream(ph.stream));
  STSCK(k_collect(c, ph));
  for (int i = 0; i < n; i++) c->seqs[seqs[i]].len += 1;
  if (logits) std::memcpy(logits, ph.h_logits, (size_t)n * c->d.vocab * sizeof(float));
  for (int i = 0, parts = argmax_parts(n, c->d.vocab); next && i < n; i++) {
    ArgBest best{-INFINITY, 0};                              // a row without any value above -inf: token 0
    for (const ArgBest* p = ph.h_best + (size_t)i * parts; p < ph.h_best + (size_t)(i + 1) * parts; p++)
      if (p->value > best.value) best = *p;
    next[i] = best.index;
  }
  return STS_OK;
}

int64_t now_ns() {
  return std::chrono::duration_cast<std::chrono::nanoseconds>(std::chrono::steady_clock::now().time_since_epoch()).count();
}

int alloc_phase(sts_ctx* c, int side) {
  Phase& ph = c->ph[side];
  ph.side = side;
  const sts_model_desc& d = c->d;
  const size_t rows = side == 0 ? c->p.max_prefill_tokens : c->p.max_decode_batch;
  const size_t nseq = side == 0 ? c->p.max_prefill_seqs : c->p.max_decode_batch;
  const size_t mp = c->p.max_pages_per_seq;
  HIPCK(hipEventCreate(&ph.ev0)); HIPCK(hipEventCreate(&ph.ev1));
  STSCK(dev_alloc(c, &ph.X, rows * d.hidden));
  STSCK(dev_alloc(c, &ph.Xn, rows * d.hidden));
  STSCK(dev_alloc(c, &ph.A, rows * c->qd));
  STSCK(dev_alloc(c, &ph.H, rows * d.mlp));
  STSCK(dev_alloc(c, &ph.Xlast_n, nseq * d.hidden));
  STSCK(dev_alloc(c, &ph.logits, nseq * d.vocab));
  STSCK(dev_alloc(c, &ph.rot, rows * d.head_dim));
  {
    // prefill attention: a query tile per 128 rows, and as many again for the parts of cut key ranges
    const size_t q_tiles = side == 0 ? rows / attn_prefill_tile_q() + nseq + 1 : 0;
    ph.max_attn_extra = (int)q_tiles + 256;
    const size_t items = 2 * q_tiles + 256;
    // decode attention items: a context has at most 128 chunks, and fewer than one per 4 pages (chunks hold >= 8)
    const size_t dec_items = side == 1 ? nseq * (size_t)decode_max_chunks((int)mp) : 0;
    ph.meta_bytes = nseq * (sizeof(PrefillSeq) + sizeof(DecodeSeq) + sizeof(DecodeMerge) + sizeof(int)) + items * (sizeof(AttnItem) + sizeof(AttnMerge)) + dec_items * sizeof(DecodeItem) +
                    3 * rows * sizeof(int) + nseq * mp * sizeof(int) + 9 * 256;
    STSCK(dev_alloc(c, &ph.d_meta, ph.meta_bytes + 16));      // copied in 16-byte pieces
    STSCK(host_alloc(&ph.h_meta, ph.meta_bytes + 16));
  }
  STSCK(host_alloc(&ph.h_logits, nseq * d.vocab));
  if (side == 0) {
    STSCK(dev_alloc(c, &ph.QKV, rows * c->qkvn));
    const size_t tail_floats = (size_t)c->n_cu * 256 * 256;   // one wave of partial tiles at the largest tile on every CU
    STSCK(dev_alloc(c, &ph.tail_ws, tail_floats));
    ph.tail_ws_bytes = tail_floats * sizeof(float);
    ph.part = ph.tail_ws; ph.part_floats = tail_floats;       // partial sums of few rows
  } else {
    const size_t widest = std::max<size_t>(std::max(c->qkvn, 2 * d.mlp), d.hidden);
    const size_t max_chunks = decode_max_chunks((int)mp);
    ph.part_floats = 8 * rows * widest;
    STSCK(dev_alloc(c, &ph.part, ph.part_floats));
    STSCK(dev_alloc(c, &ph.ssq, (size_t)KSLICE_MAX_ROWS * (d.hidden / 16)));
    STSCK(host_alloc(&ph.h_best, nseq * ARGMAX_MAX_PARTS));
    STSCK(dev_alloc(c, &ph.Q, rows * c->qd));
    STSCK(dev_alloc(c, &ph.attn_ws, attn_decode_ws_floats((int)rows, d.n_q_heads, d.head_dim, (int)max_chunks)));
  }
  return STS_OK;
}

// packed: the tensor is a GEMM weight kept in the packed block layout; the embedding table, read by rows, is row-major
struct TensorRef { bf16* w = nullptr; float* g = nullptr; int ld = 0, rows = 0, cols = 0, row_off = 0, ib = 0, phase = 0; uint64_t tid = 0; int packed = 1; };

int find_tensor(sts_ctx* c, int layer, const char* name, TensorRef* t) {
  const sts_model_desc& d = c->d;
  const std::string n(name ? name : "");
  if (n == "emb") { *t = TensorRef{c->emb, nullptr, d.hidden, d.vocab, d.hidden, 0, 0, 0, 0, 0}; return STS_OK; }
  if (n == "lm") { *t = TensorRef{c->lm, nullptr, d.hidden, d.vocab, d.hidden, 0, 0, 0, 1}; return STS_OK; }
  if (n == "gf") { *t = TensorRef{nullptr, c->gf, 0, 1, d.hidden}; return STS_OK; }
  if (layer < 0 || layer >= d.n_layers) return STS_EINVAL;
  LayerW& w = c->layers[layer];
  const uint64_t base = (uint64_t)(layer + 1) * 16;
  if (n == "g1") { *t = TensorRef{nullptr, w.g1, 0, 1, d.hidden}; return STS_OK; }
  if (n == "g2") { *t = TensorRef{nullptr, w.g2, 0, 1, d.hidden}; return STS_OK; }
  if (n == "wq") { *t = TensorRef{w.wqkv, nullptr, d.hidden, c->qd, d.hidden, 0, 0, 0, base + 0}; return STS_OK; }
  if (n == "wk") { *t = TensorRef{w.wqkv, nullptr, d.hidden, c->kvd, d.hidden, c->qd, 0, 0, base + 1}; return STS_OK; }
  if (n == "wv") { *t = TensorRef{w.wqkv, nullptr, d.hidden, c->kvd, d.hidden, c->qd + c->kvd, 0, 0, base + 2}; return STS_OK; }
  if (n == "wo") { *t = TensorRef{w.wo, nullptr, c->qd, d.hidden, c->qd, 0, 0, 0, base + 3}; return STS_OK; }
  if (n == "wg") { *t = TensorRef{w.wgu, nullptr, d.hidden, d.mlp, d.hidden, 0, 32, 0, base + 4}; return STS_OK; }
  if (n == "wu") { *t = TensorRef{w.wgu, nullptr, d.hidden, d.mlp, d.hidden, 0, 32, 1, base + 5}; return STS_OK; }
  if (n == "wd") { *t = TensorRef{w.wd, nullptr, d.mlp, d.hidden, d.mlp, 0, 0, 0, base + 6}; return STS_OK; }
  return STS_EINVAL;
}

}  // namespace

// ======================================================================================= C ABI
extern "C" int sts_init(const sts_model_desc* desc, const sts_init_params* params, sts_ctx** out) {
  if (!desc || !params || !out) return STS_EINVAL;
  const sts_model_desc& d = *desc;
  if (d.n_layers < 1 || d.hidden < 64 || d.hidden % 128 || d.mlp % 64 || (2 * d.mlp) % 128 || d.vocab % 128) return STS_EINVAL;
  if ((d.head_dim != 64 && d.head_dim != 128) || d.page_tokens != 16) return STS_EINVAL;
  if (d.n_kv_heads < 1 || d.n_q_heads % d.n_kv_heads) return STS_EINVAL;
  const int grp = d.n_q_heads / d.n_kv_heads;
  if (!(grp == 1 || grp == 4 || (grp == 8 && d.head_dim == 128))) return STS_EINVAL;
  if (((d.n_q_heads + 2 * d.n_kv_heads) * d.head_dim) % 128 || (d.n_q_heads * d.head_dim) % 64 || d.mlp % 32) return STS_EINVAL;
  if (params->kv_pool_pages < 1 || params->max_prefill_tokens < 1 || params->max_prefill_seqs < 1 ||
      params->max_decode_batch < 1 || params->max_seqs < 1 || params->max_pages_per_seq < 1) return STS_EINVAL;
  // decode attention cuts a context into at most 128 chunks (the merge workspace and the work list are sized for that)
  if (params->max_pages_per_seq > sts_max_pages_per_seq_limit(d.page_tokens)) return STS_EINVAL;
  if (g_streams_released.load()) return STS_ESTATE;
  int ndev = 0;
  HIPCK(hipGetDeviceCount(&ndev));
  if (ndev < 1) { g_hip_err = (int)hipErrorNoDevice; return STS_EHIP; }
  HIPCK(hipSetDevice(0));
  hipDeviceProp_t prop;
  HIPCK(hipGetDeviceProperties(&prop, 0));
  sts_ctx* c = new sts_ctx();
  g_live_ctx++;
  c->d = d; c->p = *params; c->n_cu = prop.multiProcessorCount;
  c->qd = d.n_q_heads * d.head_dim; c->kvd = d.n_kv_heads * d.head_dim; c->qkvn = c->qd + 2 * c->kvd;
  c->geo = KvGeom{d.n_kv_heads, d.head_dim, d.page_tokens};
  auto fail = [&](int rc) { sts_destroy(c); return rc; };
  int rc;
  // weights
  if ((rc = dev_alloc(c, &c->emb, (size_t)d.vocab * d.hidden)) || (rc = dev_alloc(c, &c->lm, (size_t)d.vocab * d.hidden)) ||
      (rc = dev_alloc(c, &c->gf, d.hidden))) return fail(rc);
  c->layers.resize(d.n_layers);
  for (auto& w : c->layers) {
    if ((rc = dev_alloc(c, &w.wqkv, (size_t)c->qkvn * d.hidden)) || (rc = dev_alloc(c, &w.wo, (size_t)d.hidden * c->qd)) ||
        (rc = dev_alloc(c, &w.wgu, (size_t)2 * d.mlp * d.hidden)) || (rc = dev_alloc(c, &w.wd, (size_t)d.hidden * d.mlp)) ||
        (rc = dev_alloc(c, &w.g1, d.hidden)) || (rc = dev_alloc(c, &w.g2, d.hidden))) return fail(rc);
  }
  // KV pool
  c->pool_layer_elems = (size_t)params->kv_pool_pages * c->geo.page_elems();
  if ((rc = dev_alloc(c, &c->pool, c->pool_layer_elems * d.n_layers))) return fail(rc);
  if (hipMemset(c->pool, 0, c->pool_layer_elems * d.n_layers * sizeof(bf16)) != hipSuccess) return fail(STS_EHIP);
  c->page_used.assign(params->kv_pool_pages, 0);
  for (int pg = params->kv_pool_pages - 1; pg >= 0; pg--) c->free_pages.push_back(pg);   // pop_back hands out page 0 first
  c->seqs.resize(params->max_seqs);
  // rotary frequencies theta^(-2i/d), in double
  {
    std::vector<double> f(d.head_dim / 2);
    for (int i = 0; i < d.head_dim / 2; i++) f[i] = std::pow((double)d.rope_theta, -2.0 * i / d.head_dim);
    if ((rc = dev_alloc(c, &c->inv_freq, f.size()))) return fail(rc);
    if (hipMemcpy(c->inv_freq, f.data(), f.size() * sizeof(double), hipMemcpyHostToDevice) != hipSuccess) return fail(STS_EHIP);
  }
  for (int side = 0; side < 2; side++) if ((rc = alloc_phase(c, side))) return fail(rc);
  // gains = 1, weights generated or zero
  auto ones = [&](float* g) { return fill_f32(nullptr, g, 1.0f, d.hidden) == hipSuccess ? STS_OK : STS_EHIP; };
  if ((rc = ones(c->gf))) return fail(rc);
  for (auto& w : c->layers) if ((rc = ones(w.g1)) || (rc = ones(w.g2))) return fail(rc);
  const char* mats[] = {"emb", "lm", "wq", "wk", "wv", "wo", "wg", "wu", "wd"};
  for (int l = 0; l < d.n_layers; l++) {
    for (const char* name : mats) {
      const bool global = !std::strcmp(name, "emb") || !std::strcmp(name, "lm");
      if (global && l > 0) continue;
      TensorRef t;
      if ((rc = find_tensor(c, l, name, &t))) return fail(rc);
      hipError_t e;
      if (params->init_weights) e = init_weight(nullptr, t.w, t.ld, params->weight_seed, t.tid, t.rows, t.cols, t.row_off, t.ib, t.phase, t.packed);
      else e = hipMemset(t.w + (size_t)(t.ib ? 0 : t.row_off) * t.ld, 0, (size_t)(t.ib ? 2 * t.rows : t.rows) * t.ld * sizeof(bf16));
      if (e != hipSuccess) { g_hip_err = (int)e; return fail(STS_EHIP); }
    }
  }
  if (hipDeviceSynchronize() != hipSuccess) return fail(STS_EHIP);
  // default partition: the whole GPU for both phases (time-multiplexed) until told otherwise
  c->part_cus[0] = c->part_cus[1] = c->n_cu;
  if ((rc = select_streams(c))) return fail(rc);
  *out = c;
  return STS_OK;
}

extern "C" int sts_max_pages_per_seq_limit(int32_t page_tokens) {
  return page_tokens > 0 ? 128 * (attn_decode_max_chunk_tokens() / page_tokens) : 0;
}
extern "C" int sts_decode_gemm_plan(int32_t m, int32_t n, int32_t k, int32_t cus, int32_t may_split, int32_t partials, int64_t gemm_rate_256,
                                    int64_t partial_bw_cu, int64_t stream_bw_cu, int64_t stream_bw_gpu, int32_t* tile_cfg, int32_t* split_k, int64_t* est_ns) {
  if (m < 1 || n < 128 || n % 128 != 0 || k < 64 || k % 64 != 0 || cus < 1 || gemm_rate_256 < 1 || partial_bw_cu < 1 || stream_bw_cu < 1 ||
      stream_bw_gpu < 1 || !tile_cfg || !split_k) return STS_EINVAL;
  int cfg = 0, splits = 1;
  const StreamRates r{0.757 * gemm_rate_256 * 1e-3, gemm_rate_256 * 1e-3, partial_bw_cu * 1e6, stream_bw_cu * 1e6, stream_bw_gpu * 1e6};
  const double t = plan_decode_gemm(r, m, n, k, cus, may_split != 0, partials != 0, &cfg, &splits);
  DecodeGemm g{cfg, splits, 0};
  if (partials) pick_tall_tiles(r, m, n, k, cus, &g);
  *tile_cfg = g.cfg; *split_k = splits;
  if (est_ns) *est_ns = (int64_t)(t * 1e9);
  return STS_OK;
}
extern "C" int sts_decode_layer_plan(sts_ctx* c, int32_t batch, int32_t cus, int32_t* tile_cfg, int32_t* split_k, int32_t* row_tiles) {
  if (!c || batch < 1 || batch > c->p.max_decode_batch || cus < 8 || cus > c->n_cu || cus % 8 != 0 || !tile_cfg || !split_k || !row_tiles) return STS_EINVAL;
  const DecodePlan p = decode_layer_plan(c, batch, cus);
  const DecodeGemm g[4] = {p.qkv, p.o, p.gu, p.down};
  for (int i = 0; i < 4; i++) { tile_cfg[i] = p.kslice ? -1 : g[i].cfg; split_k[i] = p.kslice ? 1 : g[i].splits; row_tiles[i] = p.kslice ? 0 : g[i].row_tiles; }
  return STS_OK;
}
extern "C" int sts_decode_layer_all_rows(sts_ctx* c, int32_t batch, int32_t cus, int32_t* all_rows) {
  if (!c || batch < 1 || batch > c->p.max_decode_batch || cus < 8 || cus > c->n_cu || cus % 8 != 0 || !all_rows) return STS_EINVAL;
  const DecodePlan p = decode_layer_plan(c, batch, cus);
  const DecodeGemm g[4] = {p.qkv, p.o, p.gu, p.down};
  for (int i = 0; i < 4; i++) all_rows[i] = !p.kslice && g[i].cols;
  return STS_OK;
}
extern "C" int sts_decode_gemm_all_rows(int32_t m, int32_t n, int32_t k, int32_t cus, int32_t swiglu, int64_t gemm_rate_128, int64_t gemm_rate_256, int64_t partial_bw_cu,
                                        int64_t stream_bw_cu, int64_t stream_bw_gpu, int32_t* all_rows) {
  if (m < 1 || n < 128 || n % 128 != 0 || k < 64 || k % 64 != 0 || cus < 1 || gemm_rate_128 < 1 || gemm_rate_256 < 1 || partial_bw_cu < 1 || stream_bw_cu < 1 ||
      stream_bw_gpu < 1 || !all_rows) return STS_EINVAL;
  const StreamRates r{gemm_rate_128 * 1e-3, gemm_rate_256 * 1e-3, partial_bw_cu * 1e6, stream_bw_cu * 1e6, stream_bw_gpu * 1e6};
  DecodeGemm g;
  bool fused;
  if (swiglu) plan_gateup(r, m, n, k, cus, &g, &fused);
  else plan_partials(r, m, n, k, cus, &g);
  *all_rows = g.cols;
  return STS_OK;
}
extern "C" int sts_attn_prefill_plan(int32_t n_seqs, const int32_t* lens, const int32_t* priors, int32_t n_q, int32_t n_kv, int32_t d, int32_t cus,
                                     int32_t* items, int32_t* parts, int32_t* heads) {
  if (n_seqs < 1 || !lens || !priors || n_q < 1 || n_kv < 1 || n_q % n_kv != 0 || (d != 64 && d != 128) || cus < 1 || !items || !parts || !heads) return STS_EINVAL;
  for (int i = 0; i < n_seqs; i++) if (lens[i] < 1 || priors[i] < 0 || lens[i] > (1 << 24) || priors[i] > (1 << 24)) return STS_EINVAL;
  const AttnPlan plan = attn_prefill_plan(n_seqs, lens, priors, n_q, 2 * cus, 1 << 20, 1 << 20);
  *items = (int)plan.items.size(); *parts = plan.parts; *heads = attn_prefill_heads(plan.pairs, n_q, n_kv, d);
  return STS_OK;
}
extern "C" int sts_decode_chunk_plan(const int32_t* n_pages, int32_t n, int32_t n_kv_heads, int32_t cus, int32_t page_tokens,
                                     int32_t max_pages_per_seq, int32_t* chunk_pages, int32_t* max_chunks, int32_t* allocated_chunks) {
  if (!n_pages || n < 1 || n_kv_heads < 1 || cus < 1 || page_tokens < 1 || page_tokens > attn_decode_max_chunk_tokens() || !chunk_pages || !max_chunks || !allocated_chunks) return STS_EINVAL;
  for (int i = 0; i < n; i++) if (n_pages[i] < 1 || n_pages[i] > max_pages_per_seq) return STS_EINVAL;
  decode_chunk_plan(n_pages, n, n_kv_heads, cus, page_tokens, chunk_pages, max_chunks);
  *allocated_chunks = decode_max_chunks(max_pages_per_seq);
  return STS_OK;
}

extern "C" int sts_destroy(sts_ctx* c) {
  if (!c) return STS_EINVAL;
  // Everything this ctx ever queued must have drained before its buffers go: the pooled streams of
  // every partition it selected (they outlive the ctx), and the null stream used by the weight
  // loaders and the KV test hooks.
  trace("destroy: sync every stream this ctx used");
  for (hipStream_t s : c->used_streams) (void)hipStreamSynchronize(s);
  (void)hipStreamSynchronize(nullptr);
  trace("destroy: events and pinned buffers");
  for (int side = 0; side < 2; side++) {
    Phase& ph = c->ph[side];
    if (ph.ev0) (void)hipEventDestroy(ph.ev0);
    if (ph.ev1) (void)hipEventDestroy(ph.ev1);
    for (hipEvent_t e : ph.kev) (void)hipEventDestroy(e);
    void* hosts[] = {ph.h_meta, ph.h_logits, ph.h_best};
    for (void* p : hosts) if (p) (void)hipHostFree(p);
  }
  trace("destroy: device memory");
  for (void* p : c->allocs) (void)hipFree(p);
  if (c->probe_src) (void)hipFree(c->probe_src);
  if (c->probe_dst) (void)hipFree(c->probe_dst);
  delete c;
  g_live_ctx--;
  trace("destroy: done");
  return STS_OK;
}

extern "C" int sts_release_streams(void) {
  std::lock_guard<std::mutex> g(g_stream_mu);
  if (g_live_ctx.load() != 0) return STS_ESTATE;
  g_streams_released.store(true);
  for (auto& kv : g_streams) (void)hipStreamSynchronize(kv.second);
  while (!g_streams.empty()) {
    hipStream_t s = g_streams.begin()->second;
    g_streams.erase(g_streams.begin());
    HIPCK(hipStreamDestroy(s));
  }
  return STS_OK;
}

extern "C" int sts_load_weights(sts_ctx* c, int32_t layer, const char* name, const float* host, size_t count) {
  if (!c || !host) return STS_EINVAL;
  TensorRef t;
  STSCK(find_tensor(c, layer, name, &t));
  if (count != (size_t)t.rows * t.cols) return STS_EINVAL;
  if (t.g) { HIPCK(hipMemcpy(t.g, host, count * sizeof(float), hipMemcpyHostToDevice)); return STS_OK; }
  float* tmp = nullptr;
  HIPCK(hipMalloc(&tmp, count * sizeof(float)));
  hipError_t e = hipMemcpy(tmp, host, count * sizeof(float), hipMemcpyHostToDevice);
  if (e == hipSuccess) e = convert_weight(nullptr, t.w, t.ld, tmp, t.rows, t.cols, t.row_off, t.ib, t.phase, t.packed);
  if (e == hipSuccess) e = hipDeviceSynchronize();
  (void)hipFree(tmp);
  HIPCK(e);
  return STS_OK;
}

extern "C" int sts_read_weights(sts_ctx* c, int32_t layer, const char* name, float* host, size_t count) {
  if (!c || !host) return STS_EINVAL;
  TensorRef t;
  STSCK(find_tensor(c, layer, name, &t));
  if (count != (size_t)t.rows * t.cols) return STS_EINVAL;
  if (t.g) { HIPCK(hipMemcpy(host, t.g, count * sizeof(float), hipMemcpyDeviceToHost)); return STS_OK; }
  float* tmp = nullptr;
  HIPCK(hipMalloc(&tmp, count * sizeof(float)));
  hipError_t e = export_weight(nullptr, tmp, t.w, t.ld, t.rows, t.cols, t.row_off, t.ib, t.phase, t.packed);
  if (e == hipSuccess) e = hipMemcpy(host, tmp, count * sizeof(float), hipMemcpyDeviceToHost);
  (void)hipFree(tmp);
  HIPCK(e);
  return STS_OK;
}

// ---- sequences
extern "C" int sts_seq_create(sts_ctx* c, int32_t* seq_out) {
  if (!c || !seq_out) return STS_EINVAL;
  std::lock_guard<std::mutex> g(c->alloc_mu);
  for (size_t i = 0; i < c->seqs.size(); i++)
    if (!c->seqs[i].used) { c->seqs[i] = Seq(); c->seqs[i].used = true; *seq_out = (int)i; return STS_OK; }
  return STS_ENOMEM;
}
extern "C" int sts_seq_free(sts_ctx* c, int32_t seq) {
  if (!c || !valid_seq(c, seq)) return STS_EINVAL;
  {
    // a sequence of the layer-sliced batch or of a launch still in flight keeps its pages: kernels
    // may be reading and writing them
    std::lock_guard<std::mutex> g(c->state_mu);
    if (c->pf_active) for (int s : c->pf_seqs) if (s == seq) return STS_ESTATE;
    for (int s : c->pend_pseqs) if (s == seq) return STS_ESTATE;
    for (int s : c->pend_dseqs) if (s == seq) return STS_ESTATE;
  }
  std::lock_guard<std::mutex> g(c->alloc_mu);
  for (int pg : c->seqs[seq].pages) { c->page_used[pg] = 0; c->free_pages.push_back(pg); }
  c->seqs[seq] = Seq();
  return STS_OK;
}
extern "C" int sts_seq_length(sts_ctx* c, int32_t seq, int32_t* len_out) {
  if (!c || !valid_seq(c, seq) || !len_out) return STS_EINVAL;
  *len_out = c->seqs[seq].len;
  return STS_OK;
}
extern "C" int sts_seq_truncate(sts_ctx* c, int32_t seq, int32_t new_len) {
  if (!c || !valid_seq(c, seq) || new_len < 0) return STS_EINVAL;
  {
    std::lock_guard<std::mutex> g(c->state_mu);      // not under kernels that append to it or read its length
    if (c->pf_active) for (int s : c->pf_seqs) if (s == seq) return STS_ESTATE;
    for (int s : c->pend_pseqs) if (s == seq) return STS_ESTATE;
    for (int s : c->pend_dseqs) if (s == seq) return STS_ESTATE;
  }
  std::lock_guard<std::mutex> g(c->alloc_mu);
  if (new_len > c->seqs[seq].len) return STS_EINVAL;
  c->seqs[seq].len = new_len;
  return STS_OK;
}
extern "C" int sts_seq_reserve(sts_ctx* c, int32_t seq, int32_t n_tokens) {
  if (!c || !valid_seq(c, seq) || n_tokens < 0) return STS_EINVAL;
  return reserve_pages(c, {{seq, n_tokens}});
}
extern "C" int sts_pages_free(sts_ctx* c, int32_t* n_out) {
  if (!c || !n_out) return STS_EINVAL;
  std::lock_guard<std::mutex> g(c->alloc_mu);
  *n_out = (int)c->free_pages.size();
  return STS_OK;
}
extern "C" int sts_seq_set_block_table(sts_ctx* c, int32_t seq, const int32_t* pages, int32_t n) {
  if (!c || !valid_seq(c, seq) || !pages || n < 0 || n > c->p.max_pages_per_seq) return STS_EINVAL;
  std::lock_guard<std::mutex> g(c->alloc_mu);
  Seq& s = c->seqs[seq];
  if (s.len != 0 || !s.pages.empty()) return STS_ESTATE;
  for (int i = 0; i < n; i++) {
    if (pages[i] < 0 || pages[i] >= c->p.kv_pool_pages || c->page_used[pages[i]]) return STS_EINVAL;
    for (int j = 0; j < i; j++) if (pages[j] == pages[i]) return STS_EINVAL;
  }
  for (int i = 0; i < n; i++) {
    c->page_used[pages[i]] = 1;
    c->free_pages.erase(std::find(c->free_pages.begin(), c->free_pages.end(), pages[i]));
    s.pages.push_back(pages[i]);
  }
  return STS_OK;
}
extern "C" int sts_seq_get_block_table(sts_ctx* c, int32_t seq, int32_t* pages, int32_t cap, int32_t* n_out) {
  if (!c || !valid_seq(c, seq) || !n_out) return STS_EINVAL;
  const Seq& s = c->seqs[seq];
  *n_out = (int)s.pages.size();
  for (int i = 0; i < std::min<int>(cap, (int)s.pages.size()); i++) pages[i] = s.pages[i];
  return STS_OK;
}

namespace {
int upload_bt(sts_ctx* c, const Seq& s, int** d_bt) {
  HIPCK(hipMalloc(d_bt, std::max<size_t>(1, s.pages.size()) * sizeof(int)));
  HIPCK(hipMemcpy(*d_bt, s.pages.data(), s.pages.size() * sizeof(int), hipMemcpyHostToDevice));
  return STS_OK;
}
}  // namespace

extern "C" int sts_kv_write(sts_ctx* c, int32_t layer, int32_t seq, int32_t pos0, int32_t n, const float* k, const float* v) {
  if (!c || !valid_seq(c, seq) || layer < 0 || layer >= c->d.n_layers || pos0 < 0 || n < 1 || !k || !v) return STS_EINVAL;
  STSCK(reserve_pages(c, {{seq, pos0 + n}}));
  Seq& s = c->seqs[seq];
  const size_t cnt = (size_t)n * c->kvd;
  int* d_bt = nullptr; float *dk = nullptr, *dv = nullptr;
  STSCK(upload_bt(c, s, &d_bt));
  HIPCK(hipMalloc(&dk, cnt * sizeof(float))); HIPCK(hipMalloc(&dv, cnt * sizeof(float)));
  HIPCK(hipMemcpy(dk, k, cnt * sizeof(float), hipMemcpyHostToDevice));
  HIPCK(hipMemcpy(dv, v, cnt * sizeof(float), hipMemcpyHostToDevice));
  HIPCK(kv_write_tokens(nullptr, layer_pool(c, layer), c->geo, d_bt, pos0, n, dk, dv));
  HIPCK(hipDeviceSynchronize());
  (void)hipFree(d_bt); (void)hipFree(dk); (void)hipFree(dv);
  s.len = std::max(s.len, pos0 + n);
  return STS_OK;
}
extern "C" int sts_kv_read(sts_ctx* c, int32_t layer, int32_t seq, int32_t pos0, int32_t n, float* k, float* v) {
  if (!c || !valid_seq(c, seq) || layer < 0 || layer >= c->d.n_layers || pos0 < 0 || n < 1 || !k || !v) return STS_EINVAL;
  Seq& s = c->seqs[seq];
  if ((size_t)(pos0 + n + c->geo.page_tokens - 1) / c->geo.page_tokens > s.pages.size()) return STS_EINVAL;
  const size_t cnt = (size_t)n * c->kvd;
  int* d_bt = nullptr; float *dk = nullptr, *dv = nullptr;
  STSCK(upload_bt(c, s, &d_bt));
  HIPCK(hipMalloc(&dk, cnt * sizeof(float))); HIPCK(hipMalloc(&dv, cnt * sizeof(float)));
  HIPCK(kv_read_tokens(nullptr, layer_pool(c, layer), c->geo, d_bt, pos0, n, dk, dv));
  HIPCK(hipMemcpy(k, dk, cnt * sizeof(float), hipMemcpyDeviceToHost));
  HIPCK(hipMemcpy(v, dv, cnt * sizeof(float), hipMemcpyDeviceToHost));
  (void)hipFree(d_bt); (void)hipFree(dk); (void)hipFree(dv);
  return STS_OK;
}
extern "C" int sts_kv_fill_random(sts_ctx* c, int32_t seq, int32_t n, uint64_t seed) {
  if (!c || !valid_seq(c, seq) || n < 1) return STS_EINVAL;
  STSCK(reserve_pages(c, {{seq, n}}));
  Seq& s = c->seqs[seq];
  int* d_bt = nullptr;
  STSCK(upload_bt(c, s, &d_bt));
  for (int l = 0; l < c->d.n_layers; l++) HIPCK(kv_fill_random(nullptr, layer_pool(c, l), c->geo, d_bt, 0, n, seed, l));
  HIPCK(hipDeviceSynchronize());
  (void)hipFree(d_bt);
  s.len = n;
  return STS_OK;
}

// ---- the step
static bool in_flight(sts_ctx* c, int side) {
  std::lock_guard<std::mutex> g(c->state_mu);
  return !(side == 0 ? c->pend_pseqs : c->pend_dseqs).empty();
}
extern "C" int sts_prefill_batch(sts_ctx* c, int32_t n_seqs, const int32_t* seqs, const int32_t* lens, const int32_t* tokens,
                                 int32_t lb, int32_t le, float* logits) {
  if (!c) return STS_EINVAL;
  if (c->pend_prefill) return STS_ESTATE;
  const int64_t t0 = now_ns();
  c->ph[0].alone = !in_flight(c, 1);
  STSCK(prefill_enqueue(c, n_seqs, seqs, lens, tokens, lb, le, logits != nullptr));
  STSCK(prefill_finish(c, n_seqs, seqs, lens, le, logits));
  c->last_wall_ns = now_ns() - t0;
  return STS_OK;
}
extern "C" int sts_prefill_append(sts_ctx* c, int32_t seq, const int32_t* tokens, int32_t n_tokens, int32_t lb, int32_t le, float* logits) {
  return sts_prefill_batch(c, 1, &seq, &n_tokens, tokens, lb, le, logits);
}
// ---- the same step, split into launch / poll / finish for serving loops that keep both phases in
// flight from one control thread
extern "C" int sts_prefill_launch(sts_ctx* c, int32_t n_seqs, const int32_t* seqs, const int32_t* lens, const int32_t* tokens,
                                  int32_t lb, int32_t le, int32_t want_logits) {
  if (!c) return STS_EINVAL;
  if (c->pend_prefill) return STS_ESTATE;
  c->ph[0].alone = false;                                    // a decode step may be launched beside it
  STSCK(prefill_enqueue(c, n_seqs, seqs, lens, tokens, lb, le, want_logits != 0));
  std::lock_guard<std::mutex> g(c->state_mu);
  c->pend_prefill = true; c->pend_le = le;
  c->pend_pseqs.assign(seqs, seqs + n_seqs); c->pend_plens.assign(lens, lens + n_seqs);
  return STS_OK;
}
extern "C" int sts_decode_launch(sts_ctx* c, const int32_t* seqs, const int32_t* in_tokens, int32_t n, int32_t want_logits, int32_t want_next) {
  if (!c) return STS_EINVAL;
  if (c->pend_decode) return STS_ESTATE;
  {
    // the batch is listed before anything is queued, so that from this moment neither a prefill of
    // one of its sequences nor sts_seq_free gets through
    std::lock_guard<std::mutex> g(c->state_mu);
    c->pend_dseqs.assign(seqs, seqs + std::max(n, 0));
  }
  c->ph[1].alone = false;                                    // a prefill may be launched beside it
  const int rc = decode_enqueue(c, seqs, in_tokens, n, want_logits != 0, want_next != 0);
  if (rc != STS_OK) { std::lock_guard<std::mutex> g(c->state_mu); c->pend_dseqs.clear(); return rc; }
  c->pend_decode = true;
  return STS_OK;
}
extern "C" int sts_phase_done(sts_ctx* c, int32_t phase, int32_t* done) {
  if (!c || phase < 0 || phase > 1 || !done) return STS_EINVAL;
  if (!(phase == 0 ? c->pend_prefill : c->pend_decode)) return STS_ESTATE;
  const hipError_t e = hipEventQuery(c->ph[phase].ev1);
  if (e == hipSuccess) *done = 1;
  else if (e == hipErrorNotReady) *done = 0;
  else { g_hip_err = (int)e; return STS_EHIP; }
  return STS_OK;
}
extern "C" int sts_prefill_finish(sts_ctx* c, float* logits) {
  if (!c) return STS_EINVAL;
  if (!c->pend_prefill) return STS_ESTATE;
  const std::vector<int> seqs = c->pend_pseqs, lens = c->pend_plens;
  const int rc = prefill_finish(c, (int)seqs.size(), seqs.data(), lens.data(), c->pend_le, logits);
  std::lock_guard<std::mutex> g(c->state_mu);
  c->pend_prefill = false; c->pend_pseqs.clear(); c->pend_plens.clear();
  return rc;
}
extern "C" int sts_decode_finish(sts_ctx* c, float* logits, int32_t* next) {
  if (!c) return STS_EINVAL;
  if (!c->pend_decode) return STS_ESTATE;
  const std::vector<int> seqs = c->pend_dseqs;
  const int rc = decode_finish(c, seqs.data(), (int)seqs.size(), logits, next);
  std::lock_guard<std::mutex> g(c->state_mu);
  c->pend_decode = false; c->pend_dseqs.clear();
  return rc;
}
extern "C" int sts_prefill_abort(sts_ctx* c) {
  if (!c) return STS_EINVAL;
  std::lock_guard<std::mutex> g(c->state_mu);
  c->pf_active = false; c->pf_next_layer = 0; c->pf_seqs.clear(); c->pf_lens.clear();
  return STS_OK;
}
extern "C" int sts_decode_step(sts_ctx* c, const int32_t* seqs, const int32_t* in_tokens, int32_t n, float* logits, int32_t* next) {
  if (!c) return STS_EINVAL;
  if (c->pend_decode) return STS_ESTATE;
  const int64_t t0 = now_ns();
  c->ph[1].alone = !in_flight(c, 0);
  STSCK(decode_enqueue(c, seqs, in_tokens, n, logits != nullptr, next != nullptr));
  STSCK(decode_finish(c, seqs, n, logits, next));
  c->last_wall_ns = now_ns() - t0;
  return STS_OK;
}
extern "C" int sts_step_concurrent(sts_ctx* c, int32_t n_pseqs, const int32_t* pseqs, const int32_t* plens, const int32_t* ptokens,
                                   int32_t lb, int32_t le, float* plogits, const int32_t* dseqs, const int32_t* dtokens,
                                   int32_t n_decode, float* dlogits, int32_t* dnext) {
  if (!c || n_pseqs < 0 || n_decode < 0 || (n_pseqs == 0 && n_decode == 0)) return STS_EINVAL;
  if (c->pend_prefill || c->pend_decode) return STS_ESTATE;
  for (int i = 0; i < n_pseqs; i++) for (int j = 0; j < n_decode; j++) if (pseqs && dseqs && pseqs[i] == dseqs[j]) return STS_EINVAL;
  const int64_t t0 = now_ns();
  c->ph[0].ran = c->ph[1].ran = false;
  c->ph[0].alone = n_decode == 0; c->ph[1].alone = n_pseqs == 0;
  // Both sides are checked and the pages of both are reserved in one step before anything is
  // queued: an invalid argument or an exhausted pool on either side leaves every sequence as it was.
  std::vector<std::pair<int, int>> wants;
  if (n_pseqs > 0) STSCK(prefill_validate(c, n_pseqs, pseqs, plens, ptokens, lb, le, &wants));
  if (n_decode > 0) STSCK(decode_validate(c, dseqs, dtokens, n_decode, &wants));
  STSCK(reserve_pages(c, wants));
  // Both phases are queued in turns, a layer each: queued one after the other, the second's stream stays idle for as long as the
  // first's launches take.
  DecodeRun run{c, dseqs, dtokens, n_decode, dlogits != nullptr, dnext != nullptr};
  int rc = STS_OK;
  if (n_pseqs > 0) rc = prefill_launch_checked(c, n_pseqs, pseqs, plens, ptokens, lb, le, plogits != nullptr, n_decode > 0 ? &run : nullptr);
  const bool prefill_failed = rc != STS_OK;
  if (rc == STS_OK && n_decode > 0) rc = run.finish_queue();
  const int64_t t1 = now_ns();
  if (rc != STS_OK) {
    // only a HIP failure can get here; the phase that failed has dropped its own part, what the other one has queued is dropped with it
    if (prefill_failed) { if (n_decode > 0) drop_queued(c->ph[1]); }
    else if (n_pseqs > 0) { drop_queued(c->ph[0]); (void)sts_prefill_abort(c); }
    return rc;
  }
  if (n_pseqs > 0) STSCK(prefill_finish(c, n_pseqs, pseqs, plens, le, plogits));
  const int64_t t2 = now_ns();
  if (n_decode > 0) STSCK(decode_finish(c, dseqs, n_decode, dlogits, dnext));
  c->last_wall_ns = now_ns() - t0;
  if (getenv("STS_PROF")) fprintf(stderr, "[sts prof] enqueue %lld prefill_wait %lld decode_finish %lld us\n",
                                  (long long)(t1 - t0) / 1000, (long long)(t2 - t1) / 1000, (long long)(now_ns() - t2) / 1000);
  return STS_OK;
}
extern "C" int sts_last_timing(sts_ctx* c, int64_t* prefill_ns, int64_t* decode_ns, int64_t* wall_ns) {
  if (!c) return STS_EINVAL;
  int64_t t[2] = {0, 0};
  for (int side = 0; side < 2; side++) {
    if (!c->ph[side].ran) continue;
    float ms = 0.f;
    const hipError_t e = hipEventElapsedTime(&ms, c->ph[side].ev0, c->ph[side].ev1);
    if (e == hipErrorNotReady) { (void)hipGetLastError(); continue; }   // that phase has a launch in flight: reported as 0
    HIPCK(e);
    t[side] = (int64_t)((double)ms * 1e6);
  }
  if (prefill_ns) *prefill_ns = t[0];
  if (decode_ns) *decode_ns = t[1];
  if (wall_ns) *wall_ns = c->last_wall_ns;
  return STS_OK;
}
extern "C" int sts_read_hidden(sts_ctx* c, int32_t phase, float* out, int32_t rows) {
  if (!c || phase < 0 || phase > 1 || !out || rows < 1 || rows > c->ph[phase].rows) return STS_EINVAL;
  HIPCK(hipMemcpy(out, c->ph[phase].X, (size_t)rows * c->d.hidden * sizeof(float), hipMemcpyDeviceToHost));
  return STS_OK;
}

// ---- partition
extern "C" int sts_set_partition(sts_ctx* c, int32_t prefill_cus, int32_t decode_cus) {
  if (!c) return STS_EINVAL;
  std::lock_guard<std::mutex> g(c->part_mu);
  const int old[2] = {c->part_cus[0], c->part_cus[1]};
  if (prefill_cus == -1) prefill_cus = old[0];
  if (decode_cus == -1) decode_cus = old[1];
  const int v[2] = {prefill_cus, decode_cus};
  for (int x : v) if (x != 0 && (x < 8 || x > c->n_cu || x % 8 != 0)) return STS_EINVAL;
  if ((prefill_cus != old[0] && c->pend_prefill) || (decode_cus != old[1] && c->pend_decode)) return STS_ESTATE;
  // only a side whose CU count changes is touched: the other side's control thread may be queuing
  // a step on its stream at this moment
  hipStream_t st[2] = {c->ph[0].stream, c->ph[1].stream};
  for (int side = 0; side < 2; side++) {
    if (v[side] == old[side]) continue;
    if (v[side] == 0) { st[side] = nullptr; continue; }
    const int rc = get_stream(c, side, v[side], &st[side]);
    if (rc != STS_OK) return rc;                  // nothing was changed yet
  }
  for (int side = 0; side < 2; side++) {
    if (v[side] == old[side]) continue;
    c->part_cus[side] = v[side]; c->ph[side].stream = st[side]; c->ph[side].cus = v[side];
    remember_stream(c, st[side]);
  }
  return STS_OK;
}
extern "C" int sts_get_partition(sts_ctx* c, int32_t* prefill_cus, int32_t* decode_cus, int32_t* total_cus) {
  if (!c) return STS_EINVAL;
  if (prefill_cus) *prefill_cus = c->part_cus[0];
  if (decode_cus) *decode_cus = c->part_cus[1];
  if (total_cus) *total_cus = c->n_cu;
  return STS_OK;
}

// ---- measurement hooks
extern "C" int sts_kernel_timing(sts_ctx* c, int32_t on) {
  if (!c) return STS_EINVAL;
  c->ktiming = on != 0;
  return STS_OK;
}
extern "C" int sts_fail_launch(sts_ctx* c, int32_t phase, int32_t after) {
  if (!c || phase < 0 || phase > 1 || after < -1) return STS_EINVAL;
  c->ph[phase].fail_after = after;
  return STS_OK;
}
extern "C" int sts_kernel_times(sts_ctx* c, int32_t phase, int64_t* ns, int64_t* launches, int32_t reset) {
  if (!c || phase < 0 || phase > 1) return STS_EINVAL;
  Phase& ph = c->ph[phase];
  for (int k = 0; k < STS_K_COUNT; k++) {
    if (ns) ns[k] = ph.kns[k];
    if (launches) launches[k] = ph.kcnt[k];
    if (reset) { ph.kns[k] = 0; ph.kcnt[k] = 0; }
  }
  return STS_OK;
}
extern "C" int sts_set_tile_model(sts_ctx* c, int64_t gemm_rate_128, int64_t gemm_rate_256, int64_t gemm_rate_128x256, int64_t gemm_fixed_128x256,
                                  int64_t partial_bw_cu) {
  if (!c || gemm_rate_128 < 1 || gemm_rate_256 < 1 || gemm_rate_128x256 < 1 || gemm_fixed_128x256 < 0 || partial_bw_cu < 1) return STS_EINVAL;
  if (c->pend_prefill || c->pend_decode) return STS_ESTATE;
  c->rate_128 = gemm_rate_128 * 1e-3; c->rate_256 = gemm_rate_256 * 1e-3; c->partial_bw = partial_bw_cu * 1e6;
  return STS_OK;
}
extern "C" int sts_set_stream_model(sts_ctx* c, int64_t stream_bw_cu, int64_t stream_bw_gpu) {
  if (!c || stream_bw_cu < 1 || stream_bw_gpu < stream_bw_cu) return STS_EINVAL;
  c->stream_bw_cu = stream_bw_cu * 1e6; c->stream_bw_gpu = stream_bw_gpu * 1e6;
  return STS_OK;
}
extern "C" int sts_probe_gemm(sts_ctx* c, int32_t cus, int32_t tile_cfg, int32_t product, int32_t m, int32_t n, int32_t iters, int64_t* ns_out) {
  if (!c || !ns_out || iters < 1 || tile_cfg < 0 || tile_cfg >= GEMM_NCFG || product < 0 || product > 2) return STS_EINVAL;
  const sts_model_desc& d = c->d;
  const int n_max = product == 0 ? 2 * d.mlp : d.hidden;
  if (m < 1 || m > c->p.max_prefill_tokens || n < 64 || n > n_max || n % 64 || n % gemm_tile_n(tile_cfg)) return STS_EINVAL;
  // gate/up runs with its SwiGLU epilogue, which needs gate/up block pairs in a wave tile
  if (product == 0 && (tile_cfg == GEMM_64x256 || tile_cfg == GEMM_128x256)) return STS_EINVAL;
  if (c->pend_prefill) return STS_ESTATE;
  hipStream_t st;
  STSCK(get_stream(c, 0, cus, &st));
  { std::lock_guard<std::mutex> g(c->part_mu); remember_stream(c, st); }
  Phase& ph = c->ph[0];
  struct Events {
    hipEvent_t e0 = nullptr, e1 = nullptr;
    ~Events() { if (e0) (void)hipEventDestroy(e0); if (e1) (void)hipEventDestroy(e1); }
  } ev;
  HIPCK(hipEventCreate(&ev.e0)); HIPCK(hipEventCreate(&ev.e1));
  const LayerW& w0 = c->layers[0];
  auto run = [&]() {
    if (product == 1) return gemm_bf16(st, tile_cfg, EPI_RESID_F32, ph.A, c->qd, w0.wo, c->qd, ph.X, d.hidden, m, n, c->qd, 1, 0);
    if (product == 2) return gemm_bf16(st, tile_cfg, EPI_RESID_F32, ph.H, d.mlp, w0.wd, d.mlp, ph.X, d.hidden, m, n, d.mlp, 1, 0);
    return gemm_bf16(st, tile_cfg, EPI_SWIGLU_BF16, ph.Xn, d.hidden, w0.wgu, d.hidden, ph.H, d.mlp, m, n, d.hidden, 1, 0);
  };
  for (int i = 0; i < 2; i++) HIPCK(run());                         // warm-up
  HIPCK(hipEventRecord(ev.e0, st));
  for (int i = 0; i < iters; i++) HIPCK(run());
  HIPCK(hipEventRecord(ev.e1, st));
  HIPCK(hipEventSynchronize(ev.e1));
  float ms = 0.f;
  HIPCK(hipEventElapsedTime(&ms, ev.e0, ev.e1));
  *ns_out = (int64_t)((double)ms * 1e6);
  return STS_OK;
}
static int probe_stream(sts_ctx* c, int32_t side, int32_t cus, size_t bytes, int32_t iters, int64_t* ns_out, bool read_only) {
  if (!c || side < 0 || side > 1 || bytes < 4096 || bytes % 16 || iters < 1 || !ns_out) return STS_EINVAL;
  hipStream_t st;
  STSCK(get_stream(c, side, cus, &st));
  { std::lock_guard<std::mutex> g(c->part_mu); remember_stream(c, st); }
  if (c->probe_bytes < bytes) {
    if (c->probe_src) { (void)hipFree(c->probe_src); (void)hipFree(c->probe_dst); c->probe_src = c->probe_dst = nullptr; c->probe_bytes = 0; }
    HIPCK(hipMalloc(&c->probe_src, bytes)); HIPCK(hipMalloc(&c->probe_dst, bytes));
    HIPCK(hipMemset(c->probe_src, 1, bytes)); HIPCK(hipMemset(c->probe_dst, 0, bytes));
    HIPCK(hipDeviceSynchronize());
    c->probe_bytes = bytes;
  }
  struct Events {                                                   // destroyed on every return path
    hipEvent_t e0 = nullptr, e1 = nullptr;
    ~Events() { if (e0) (void)hipEventDestroy(e0); if (e1) (void)hipEventDestroy(e1); }
  } ev;
  HIPCK(hipEventCreate(&ev.e0)); HIPCK(hipEventCreate(&ev.e1));
  // The copy runs 8 workgroups per CU. The read stream's rate depends on how many workgroups share a CU (on the whole GPU
  // two per CU read a fifth more than eight), and the probe reports what the memory system can give: the best of 2, 4 and 8.
  // Its sink is the first word of the copy's destination buffer.
  float best_ms = 0.f;
  for (int per_cu : {8, 4, 2}) {
    const int grid = cus * per_cu;
    auto launch = [&]() { return read_only ? read_probe(st, c->probe_src, bytes, reinterpret_cast<unsigned*>(c->probe_dst), grid)
                                           : copy_probe(st, c->probe_dst, c->probe_src, bytes, grid); };
    HIPCK(launch());   // warm-up
    HIPCK(hipEventRecord(ev.e0, st));
    for (int i = 0; i < iters; i++) HIPCK(launch());
    HIPCK(hipEventRecord(ev.e1, st));
    HIPCK(hipEventSynchronize(ev.e1));
    float ms = 0.f;
    HIPCK(hipEventElapsedTime(&ms, ev.e0, ev.e1));
    if (best_ms == 0.f || ms < best_ms) best_ms = ms;
    if (!read_only) break;
  }
  *ns_out = (int64_t)((double)best_ms * 1e6);
  return STS_OK;
}
extern "C" int sts_probe_copy(sts_ctx* c, int32_t side, int32_t cus, size_t bytes, int32_t iters, int64_t* ns_out) {
  return probe_stream(c, side, cus, bytes, iters, ns_out, false);
}
extern "C" int sts_probe_read(sts_ctx* c, int32_t side, int32_t cus, size_t bytes, int32_t iters, int64_t* ns_out) {
  return probe_stream(c, side, cus, bytes, iters, ns_out, true);
}
