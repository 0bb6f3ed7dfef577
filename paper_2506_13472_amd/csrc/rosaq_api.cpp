// C ABI of the library: argument validation, handle ownership, device upload and
// the per-call launch sequence.  No arithmetic of the method happens here.
#include <hip/hip_runtime_api.h>

#include <atomic>
#include <climits>
#include <cstdlib>
#include <cstring>
#include <exception>
#include <new>
#include <type_traits>

#include "rosaq_internal.h"

namespace rosaq {

static thread_local std::string g_error;
void set_error(const std::string& s) { g_error = s; }

static GemmTune g_tune;         // all zero = heuristics
static GemmTune g_tune_rot;     // same, for the dense-rotation launch
static int g_tune_stages = 3;  // bit 0: prologue kernels, bit 1: main GEMM (timing aid)

static int fail(int code, const std::string& msg) {
  set_error(msg);
  return code;
}

static size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }


// Workspace carve-up for one call with M rows.
// [xhat fragments | second copy for the dense rotation | tickets of the rotation GEMM and of the
// main GEMM | fp32 partial tiles of split launches].  `required` is what a call cannot do without;
// whatever the caller gives beyond it is room for partial tiles.
struct WsPlan {
  size_t xf_a = 0, xf_b = 0, tickets = 0, part = 0, required = 0, total = 0;
};
constexpr size_t kTicketBytes = 2 * static_cast<size_t>(kTicketsPerLaunch) * sizeof(uint32_t);

// partial tiles of one launch at the largest split: rows padded to whole tiles, fp32
static size_t part_room(int M, size_t channels) {
  if (M > 64) return 0;                                   // only launches of up to 64 rows are split
  const size_t rows = M > 32 ? 64 : (M > 16 ? 32 : 16);
  return static_cast<size_t>(kMaxSplits) * rows * align_up(channels, 96) * 4;
}

static WsPlan plan_workspace(const rosaq_packed& p, int M, size_t channels_total = 0) {
  WsPlan w;
  const Canonical& c = p.c;
  const size_t mblocks = (static_cast<size_t>(M) + kMBlock - 1) / kMBlock;
  const size_t xf_bytes = mblocks * (c.D / kKStep) * 4 * 64 * 16;
  size_t off = 0;
  w.xf_a = off; off += align_up(xf_bytes, 256);
  if (c.q_mode == ROSAQ_Q_FULL) {
    w.xf_b = off; off += align_up(xf_bytes, 256);
  }
  w.tickets = off; off += kTicketBytes;
  w.required = off;
  w.part = off;
  const size_t widest = std::max<size_t>(channels_total ? channels_total : c.N,
                                         c.q_mode == ROSAQ_Q_FULL ? c.D : 0);
  off += align_up(part_room(M, widest), 256);
  w.total = off;
  return w;
}

static int check_desc(const rosaq_pack_desc* d) {
  if (!d) return fail(ROSAQ_ERR_NULL, "desc is NULL");
  if (!d->W) return fail(ROSAQ_ERR_NULL, "desc.W is NULL");
  if (!d->eigenvalues) return fail(ROSAQ_ERR_NULL, "desc.eigenvalues is NULL");
  if (d->q_mode < ROSAQ_Q_NONE || d->q_mode > ROSAQ_Q_HEADWISE)
    return fail(ROSAQ_ERR_ARG, "q_mode is not one of ROSAQ_Q_*");
  if (d->q_mode != ROSAQ_Q_NONE && !d->Q) return fail(ROSAQ_ERR_NULL, "desc.Q is NULL");
  if (d->bits != 3 && d->bits != 4) return fail(ROSAQ_ERR_ARG, "bits must be 3 or 4");
  if (d->group != kGroup) return fail(ROSAQ_ERR_ARG, "group must be 128");
  if (d->q_mode == ROSAQ_Q_HEADWISE && d->head_dim != kHeadDim)
    return fail(ROSAQ_ERR_ARG, "head_dim must be 128");
  if (d->select_rule < ROSAQ_SELECT_TOP || d->select_rule > ROSAQ_SELECT_TOP_AND_BOTTOM)
    return fail(ROSAQ_ERR_ARG, "select_rule is not one of ROSAQ_SELECT_*");
  if (d->out_features < 1 || d->in_features < 1)
    return fail(ROSAQ_ERR_SHAPE, "out_features and in_features must be positive");
  if (d->in_features % 128 != 0) return fail(ROSAQ_ERR_SHAPE, "in_features must be a multiple of 128");
  if (d->K < 0 || d->K > d->in_features) return fail(ROSAQ_ERR_SHAPE, "K must be in [0, in_features]");
  if (d->K % kKStep != 0) return fail(ROSAQ_ERR_SHAPE, "K must be a multiple of 32");
  if ((d->in_features - d->K) % d->group != 0)
    return fail(ROSAQ_ERR_SHAPE, "in_features - K must be a multiple of group");
  if (d->ldw < d->in_features) return fail(ROSAQ_ERR_SHAPE, "ldw is smaller than in_features");
  if (d->select_rule == ROSAQ_SELECT_TOP_PER_HEAD && d->K % (d->in_features / kHeadDim) != 0)
    return fail(ROSAQ_ERR_SHAPE, "K must be a multiple of the number of 128-channel heads");
  if (d->select_rule == ROSAQ_SELECT_TOP_AND_BOTTOM && d->K % 2 != 0)
    return fail(ROSAQ_ERR_SHAPE, "K must be even for TOP_AND_BOTTOM");
  if (d->select_rule == ROSAQ_SELECT_CONSECUTIVE &&
      (d->select_arg < 0 || d->select_arg > d->in_features - d->K))
    return fail(ROSAQ_ERR_SHAPE, "select_arg must lie in [0, in_features - K]");
  return ROSAQ_OK;
}

#define ROSAQ_HIP(call)                                                         \
  do {                                                                          \
    hipError_t e_ = (call);                                                     \
    if (e_ != hipSuccess) {                                                     \
      set_error(std::string(#call) + ": " + hipGetErrorString(e_));            \
      return ROSAQ_ERR_HIP;                                                     \
    }                                                                           \
  } while (0)

// What one offline step on the GPU holds besides the handle's own buffer; given back on every way out.
struct PackScratch {
  char* mem = nullptr;
  hipStream_t work = nullptr;        // the caller's stream
  hipStream_t copies = nullptr;      // uploads and downloads: beside the kernels, or `work` itself for a single chunk
  std::vector<hipEvent_t> events;
  hipError_t event(hipEvent_t* e) {
    events.push_back(nullptr);
    const hipError_t r = hipEventCreateWithFlags(&events.back(), hipEventDisableTiming);
    *e = events.back();
    return r;
  }
  ~PackScratch() {
    if (copies != work) { (void)hipStreamSynchronize(copies); (void)hipStreamDestroy(copies); }
    if (mem) { (void)hipStreamSynchronize(work); (void)hipFree(mem); }
    for (hipEvent_t e : events) if (e) (void)hipEventDestroy(e);
  }
};

// The offline step with the layer on the GPU: upload Q and W, rotate in fp64 (Eq. 1), then one
// pass from the rotated fp16 weight to the fragment images the kernels read and to the canonical
// arrays (Sec. 3.2-3.3, Eq. 3), which come back to the host for rosaq_packed_export.  Only the
// ranking of D eigenvalues stays on the host.
// The rows go through in chunks: while the GPU works on one, the next is uploaded and finished ones are
// downloaded on a second stream, and the pages of the arrays they go to are touched by several threads
// (a download into untouched memory runs at 4 GB/s, into touched memory at 16).  Inf / NaN in W and Q and the rotation's
// fingerprint are found by kernels on the uploaded copies; a byte-wise hash of a 4096 x 4096 rotation on the host
// alone took 54 ms.  11008 x 4096 INT3 with a dense rotation, export included: 80 to 90 -> 12 to 17 ms from box to box.
static int pack_device(const rosaq_pack_desc& d, hipStream_t st, rosaq_packed* p) {
  std::string err;
  int rc = pack_validate_eigenvalues(d, &err);
  if (rc != ROSAQ_OK) return fail(rc, err);
  pack_select(d, &p->c);
  Canonical& c = p->c;
  const size_t N = c.N, D = c.D, K = c.K, C = D - K, G = c.G;
  const size_t ntiles = (N + 127) / 128 * 8, ks_s = K / kKStep;
  const bool rotate = d.q_mode != ROSAQ_Q_NONE, headwise = d.q_mode == ROSAQ_Q_HEADWISE;
  const bool keep_q = rotate && !d.rotation_absorbed;
  const size_t rec_dwords = (c.bits == 4 ? 256 : 192) + 16;
  const size_t wS_bytes = ntiles * ks_s * 64 * 16, wq_bytes = ntiles * G * rec_dwords * 4;
  const size_t qf_bytes = !keep_q ? 0 : (headwise ? (D / kHeadDim) * 8 * 4 * 64 * 16
                                                  : (D / kTileN) * (D / kKStep) * 64 * 16);
  const size_t q_words = !rotate ? 0 : (headwise ? D * kHeadDim : D * D);

  // the handle's device buffer: [wS | wq | qf | perm | pos]
  struct Part { size_t bytes; void** dst; };
  void *d_perm = nullptr, *d_pos = nullptr;
  Part parts[] = {{wS_bytes, &p->d_wS}, {wq_bytes, &p->d_wq}, {qf_bytes, &p->d_qf},
                  {D * 4, &d_perm}, {D * 4, &d_pos}};
  size_t total = 0;
  for (const Part& q : parts) total += align_up(std::max<size_t>(q.bytes, 16), 256);
  ROSAQ_HIP(hipGetDevice(&p->device));
  ROSAQ_HIP(hipMalloc(&p->d_blob, total));       // owned by the handle from here on (rosaq_free)
  p->blob_bytes = total;
  p->host_only = false;
  size_t off = 0;
  for (const Part& q : parts) {
    *q.dst = static_cast<char*>(p->d_blob) + off;
    off += align_up(std::max<size_t>(q.bytes, 16), 256);
  }
  p->d_perm = static_cast<int32_t*>(d_perm);
  p->d_pos = static_cast<int32_t*>(d_pos);

  // host arrays the canonical form comes back into
  c.W_S.resize(N * K); c.codes.resize(N * C); c.scales.resize(N * G); c.zeros.resize(N * G);
  // chunks: at most eight, at least 8 MiB of W each, of a number of rows whose 128 x 128 tiles of the rotation come to
  // two whole workgroups per compute unit
  const size_t round_rows = 128 * ((512 * 128 + D - 1) / D);
  const size_t chunk = align_up(std::max<size_t>((N + 7) / 8, (size_t{4} << 20) / D), rotate && !headwise ? round_rows : 128);
  const size_t chunks = (N + chunk - 1) / chunk;
  PackScratch t;
  t.work = t.copies = st;
  t.events.reserve(2 * chunks);
  // scratch of this call: [W | What | Q | W_S | codes | scales | zeros | flags and hash]
  const size_t sizes[] = {N * D * 2, rotate ? N * D * 2 : 0, q_words * 4, N * K * 2, N * C, N * G * 2, N * G * 2, 256};
  size_t offs[8], tmp_total = 0;
  for (int i = 0; i < 8; ++i) { offs[i] = tmp_total; tmp_total += align_up(std::max<size_t>(sizes[i], 16), 256); }
  ROSAQ_HIP(hipMalloc(reinterpret_cast<void**>(&t.mem), tmp_total));
  if (chunks > 1) {      // nothing to overlap within one chunk: creating a stream and its events takes longer than they save
    hipStream_t copies;
    ROSAQ_HIP(hipStreamCreateWithFlags(&copies, hipStreamNonBlocking));
    t.copies = copies;
  }
  const bool beside = t.copies != st;
  char* const w_dev = t.mem + offs[0];
  char* const what = rotate ? t.mem + offs[1] : w_dev;
  char* const q_dev = t.mem + offs[2];
  char* const flags = t.mem + offs[7];           // words: rotated weight, W, Q; then Q's hash in 64 bits
  ROSAQ_HIP(hipMemsetAsync(flags, 0, 256, st));
  ROSAQ_HIP(hipMemcpyAsync(d_perm, c.perm.data(), D * 4, hipMemcpyHostToDevice, t.copies));
  ROSAQ_HIP(hipMemcpyAsync(d_pos, c.pos.data(), D * 4, hipMemcpyHostToDevice, t.copies));
  if (rotate) ROSAQ_HIP(hipMemcpyAsync(q_dev, d.Q, q_words * 4, hipMemcpyHostToDevice, t.copies));
  std::vector<hipEvent_t> finished(chunks);
  for (size_t i = 0; i < chunks; ++i) {
    const size_t n0 = i * chunk, rows = std::min(chunk, N - n0), tile0 = n0 / kTileN;
    char* const w = w_dev + n0 * D * 2;
    if (static_cast<size_t>(d.ldw) == D)
      ROSAQ_HIP(hipMemcpyAsync(w, d.W + n0 * D, rows * D * 2, hipMemcpyHostToDevice, t.copies));
    else
      ROSAQ_HIP(hipMemcpy2DAsync(w, D * 2, d.W + n0 * static_cast<size_t>(d.ldw), static_cast<size_t>(d.ldw) * 2, D * 2,
                                 rows, hipMemcpyHostToDevice, t.copies));
    if (beside) {
      hipEvent_t uploaded;
      ROSAQ_HIP(t.event(&uploaded));
      ROSAQ_HIP(hipEventRecord(uploaded, t.copies));
      ROSAQ_HIP(hipStreamWaitEvent(st, uploaded, 0));
    }
    if (i == 0 && rotate && (rc = launch_check_rotation(q_dev, q_words, flags + 8, flags + 16, st)) != ROSAQ_OK) return rc;
    if (i == 0 && keep_q && (rc = launch_rotation_image(q_dev, c.D, headwise ? 1 : 0, p->d_perm, p->d_qf, st)) != ROSAQ_OK)
      return rc;
    if ((rc = launch_check_weight(w, rows * D, flags + 4, st)) != ROSAQ_OK) return rc;
    if (rotate && (rc = launch_rotate_weights_f64(w, q_dev, what + n0 * D * 2, static_cast<int>(rows), c.D,
                                                  headwise ? 1 : 0, st)) != ROSAQ_OK)
      return rc;
    QuantPackArgs a{};
    a.what16 = what + n0 * D * 2; a.N = static_cast<int>(rows); a.D = c.D; a.K = c.K; a.bits = c.bits; a.perm = p->d_perm;
    a.wS_image = static_cast<char*>(p->d_wS) + tile0 * ks_s * 64 * 16;
    a.wq_image = static_cast<char*>(p->d_wq) + tile0 * G * rec_dwords * 4;
    a.W_S = t.mem + offs[3] + n0 * K * 2; a.codes = t.mem + offs[4] + n0 * C;
    a.scales = t.mem + offs[5] + n0 * G * 2; a.zeros = t.mem + offs[6] + n0 * G * 2;
    a.flag = flags;
    if ((rc = launch_quantize_pack(a, st)) != ROSAQ_OK) return rc;
    if (beside) {
      ROSAQ_HIP(t.event(&finished[i]));
      ROSAQ_HIP(hipEventRecord(finished[i], st));
    }
  }
  struct Array { char* host; size_t dev, row_bytes; };
  const Array arrays[] = {{reinterpret_cast<char*>(c.codes.data()), offs[4], C}, {reinterpret_cast<char*>(c.W_S.data()), offs[3], K * 2},
                          {reinterpret_cast<char*>(c.scales.data()), offs[5], G * 2}, {reinterpret_cast<char*>(c.zeros.data()), offs[6], G * 2}};
  for (const Array& a : arrays) {
    constexpr size_t kPage = 4096;
    const size_t pages = N * a.row_bytes / kPage;
    parallel_rows(static_cast<int>(pages / 64), [&](int lo, int hi) {
      for (size_t pg = static_cast<size_t>(lo) * 64; pg < static_cast<size_t>(hi) * 64; ++pg) a.host[pg * kPage] = 0;
    });
  }
  for (size_t i = 0; i < chunks; ++i) {
    const size_t n0 = i * chunk, rows = std::min(chunk, N - n0);
    if (beside) ROSAQ_HIP(hipStreamWaitEvent(t.copies, finished[i], 0));
    for (const Array& a : arrays)
      if (a.row_bytes)
        ROSAQ_HIP(hipMemcpyAsync(a.host + n0 * a.row_bytes, t.mem + a.dev + n0 * a.row_bytes, rows * a.row_bytes,
                                 hipMemcpyDeviceToHost, t.copies));
  }
  uint32_t found[6];
  ROSAQ_HIP(hipMemcpyAsync(found, flags, sizeof(found), hipMemcpyDeviceToHost, t.copies));
  ROSAQ_HIP(hipStreamSynchronize(t.copies));
  ROSAQ_HIP(hipStreamSynchronize(st));
  if (found[1]) return fail(ROSAQ_ERR_NONFINITE, "W contains NaN/Inf");
  if (found[2]) return fail(ROSAQ_ERR_NONFINITE, "Q contains NaN/Inf");
  if (found[0]) return fail(ROSAQ_ERR_NONFINITE, "rotated weight overflows fp16");
  std::memcpy(&p->rot_fingerprint, &found[4], 8);
  return ROSAQ_OK;
}

// The same hash of the rotation for a layer that stays on the host.
static uint64_t rotation_hash_host(const float* Q, size_t words) {
  std::atomic<uint64_t> sum{0};
  constexpr size_t kSlice = 4096;
  parallel_rows(static_cast<int>((words + kSlice - 1) / kSlice), [&](int lo, int hi) {
    uint64_t h = 0;
    for (size_t i = static_cast<size_t>(lo) * kSlice; i < std::min(words, static_cast<size_t>(hi) * kSlice); ++i) {
      uint32_t w;
      std::memcpy(&w, Q + i, 4);
      h += rotation_hash_word(i, w);
    }
    sum.fetch_add(h, std::memory_order_relaxed);
  });
  return sum.load();
}

static int check_call(const rosaq_packed_t* p, const void* x, int32_t M, int64_t ldx, void* y,
                      int64_t ldy, void* ws, size_t ws_bytes, bool headwise, WsPlan* plan) {
  if (!p) return fail(ROSAQ_ERR_NULL, "handle is NULL");
  if (!x || !y) return fail(ROSAQ_ERR_NULL, "x or y is NULL");
  if ((p->c.q_mode == ROSAQ_Q_HEADWISE) != headwise)
    return fail(ROSAQ_ERR_MODE, headwise ? "rosaq_linear_headwise needs a HEADWISE handle"
                                         : "rosaq_linear does not serve a HEADWISE handle");
  if (M < 1) return fail(ROSAQ_ERR_SHAPE, "M must be at least 1");
  if (M > (1 << 20)) return fail(ROSAQ_ERR_SHAPE, "M above 2^20: split the call");
  // the prologue kernels index the fragment copy of x with 32-bit integers (16 bytes per index)
  if ((static_cast<int64_t>(M) + kMBlock - 1) / kMBlock * kMBlock * p->c.D / 8 > INT32_MAX)
    return fail(ROSAQ_ERR_SHAPE, "M x in_features above 2^34: split the call");
  if (ldx < p->c.D || ldy < p->c.N) return fail(ROSAQ_ERR_SHAPE, "leading dimension smaller than width");
  if (reinterpret_cast<uintptr_t>(x) % 16 || ldx % 8)
    return fail(ROSAQ_ERR_ALIGN, "x must be 16-byte aligned and ldx a multiple of 8");
  if (reinterpret_cast<uintptr_t>(y) % 2) return fail(ROSAQ_ERR_ALIGN, "y must be 2-byte aligned");
  *plan = plan_workspace(*p, M);
  if (!ws || ws_bytes < plan->required) return fail(ROSAQ_ERR_WORKSPACE, "workspace missing or too small");
  if (reinterpret_cast<uintptr_t>(ws) % 256) return fail(ROSAQ_ERR_ALIGN, "workspace must be 256-byte aligned");
  return ROSAQ_OK;
}

static int check_device(const rosaq_packed_t* const* ps, int count) {
  for (int i = 0; i < count; ++i)
    if (ps[i]->host_only) return fail(ROSAQ_ERR_HOSTONLY, "handle was packed with host_only");
  return ROSAQ_OK;
}

// Buffers of one main-GEMM launch.  `chain_*`: a gated pair that feeds a following layer writes its
// product as that layer's input fragments (rosaq_mlp_swiglu) and clears that layer's tickets.
struct GemmIO {
  const void* xf;            // xhat fragments the launch reads
  void* tickets;             // kTicketsPerLaunch words, zero before the launch
  void* part;                // room for partial tiles of a split launch
  size_t part_bytes;
  const int32_t* chain_pos = nullptr;   // device: channel -> storage position of the next layer
  int chain_ks = 0;                     // k-steps of the next layer's input
  void* zero_ptr = nullptr;
  int zero_count = 0;
};

static GemmIO plan_io(const rosaq_packed& p0, const WsPlan& w, char* ws, size_t ws_bytes) {
  GemmIO io{};
  io.xf = ws + (p0.c.q_mode == ROSAQ_Q_FULL ? w.xf_b : w.xf_a);
  io.tickets = ws + w.tickets + kTicketsPerLaunch * sizeof(uint32_t);
  io.part = ws + w.part;
  io.part_bytes = ws_bytes > w.part ? ws_bytes - w.part : 0;
  return io;
}

// y_i = xhat W_i^T for `count` layers that share the xhat fragments `io.xf`.
static GemmArgs main_gemm(const rosaq_packed_t* const* ps, int count, const GemmIO& io, int M,
                          void* const* ys, const int64_t* ldys, bool swiglu = false) {
  const Canonical& c = ps[0]->c;
  GemmArgs a{};
  a.xf = io.xf;
  a.nseg = count;
  for (int i = 0; i < count; ++i) {
    const rosaq_packed_t* p = ps[i];
    a.seg[i].wS = p->d_wS; a.seg[i].wq = p->d_wq;
    a.seg[i].out = ys[i]; a.seg[i].ldo = ldys[i]; a.seg[i].N = p->c.N;
  }
  a.M = M;
  a.ks_s = c.K / kKStep; a.G = c.G; a.KS = c.D / kKStep; a.KS_out = 0;
  a.bits = c.bits; a.out_frag = 0;
  if (io.chain_pos) { a.out_frag = 2; a.out_pos = io.chain_pos; a.KS_out = io.chain_ks; }
  a.part = io.part; a.part_bytes = io.part_bytes;
  a.tickets = io.tickets; a.ticket_count = kTicketsPerLaunch;
  a.zero_ptr = io.zero_ptr; a.zero_count = io.zero_count;
  a.swiglu = swiglu ? 1 : 0;
  return a;
}
// The words the first launch of a call clears: the tickets of the GEMM launch behind it, if that is split.  (Cleared
// always, they were 32 KiB of stores in launches that are bound by the way of their stores to memory.)
static int ticket_words(const GemmPlan& plan) { return plan.shape.splits > 1 ? 2 * kTicketsPerLaunch : 0; }

// Settings of the dense rotation's launch: "rot_splits" selects the slab launches, never a ticketed split (no room for
// partial tiles is offered).
static GemmTune rotation_tune() {
  GemmTune tune = g_tune_rot;
  tune.splits = 0;
  return tune;
}

// The head-wise rotation of many rows: a launch of one workgroup per head and 64 rows takes 6.0 to 6.4 us until it has more
// workgroups than compute units, one of a workgroup per column tile (eight times as many) less than that while it is small.  us, per head / per column tile: 4096 channels at
// 256 rows (128 heads x blocks) 6.0 / 5.3, at 384 (192) 6.2 / 6.9, at 512 6.4 / 8.7, at 2048 15.8 / 26.2; 5120 at 256 rows
// (160) 6.1 / 6.0, at 2048 18.8 / 32.8; 1024 at 1024 rows (128) 6.1 / 5.2, at 2048 (256) 6.6 / 8.8.
static bool rotates_whole_heads(int D, int M) {
  const int64_t head_blocks = static_cast<int64_t>(D / kHeadDim) * ((M + kMBlock - 1) / kMBlock);
  return g_tune_rot.wide == 2 ? M > kMBlock : (g_tune_rot.wide == 0 && M > kMBlock && head_blocks > 160);
}

// Whether the dense rotation reads row-major x itself, without a copy into fragments in front of it.  That saves a launch (1.5
// us in a graph, more where the host issues it), but its loads then take 64 bytes of each of 16 rows where those of fragments
// take 1 KiB in a row, which costs more the more of them there are.  The lines are where it is faster both with Q from memory and with Q in
// a cache, which leaves less time to hide those loads in.  us of a call with 512 channels behind the rotation, in a graph, copy / in place, Q from
// memory and (one layer) in a cache: 1408 channels at 17 rows 10.1 / 8.5 and 8.8 / 7.5, at 64 10.6 / 9.2 and 9.1 / 8.0; 2048 at 64 12.8 / 11.4 and 10.3 /
// 9.2; 2560 at 48 14.4 / 13.2 and 10.7 / 9.9, at 56 15.8 / 15.2 and 11.3 / 12.1; 3072 at 32 15.4 / 14.4 and 11.7 / 11.1, at 37 16.7 / 15.8 and 12.9 /
// 13.7; 4096 at 32 18.5 / 17.5 and 13.8 / 12.9, at 37 20.1 / 19.7 and 15.2 / 16.8, at 64 20.5 / 21.4 and 15.5 / 16.3.  Above, Q out of the last-level cache:
// 5120 at 17 26.3 / 24.6, at 24 24.4 / 24.9, at 32 24.6 / 27.5, at 37 25.6 / 23.6, at 48 26.3 / 25.7, at 64 26.5 / 28.6; 6144 at 17 30.6 / 28.6, at 32
// 29.6 / 32.5, at 37 29.8 / 29.4, at 64 30.4 / 32.8; 8192 at 17 38.5 / 36.8, at 32 39.2 / 44.0, at 37 58.0 / 53.6, at 64 58.4 / 57.9.
static bool rotates_in_place(int D, int M) { return M <= (D <= 2048 ? 64 : (D <= 2560 ? 48 : (D <= 4096 ? 32 : 16))); }

// x -> xhat fragments in the workspace (gather / head-wise blocks / dense rotation).
static int run_prologue(const rosaq_packed_t* p, const WsPlan& w, const void* x_dev, int M,
                        int64_t ldx, char* ws, size_t ws_bytes, int n_tickets, void* hip_stream) {
  const Canonical& c = p->c;
  void* tickets = ws + w.tickets;
  if (c.q_mode == ROSAQ_Q_HEADWISE && rotates_whole_heads(c.D, M))
    return launch_rotate_rows(x_dev, ldx, M, c.D, p->d_qf, p->d_perm, p->d_pos, ws + w.xf_a, tickets, n_tickets,
                              hip_stream);
  if (c.q_mode == ROSAQ_Q_HEADWISE)
    return launch_rotate_headwise(x_dev, ldx, M, c.D, p->d_qf, p->d_pos, ws + w.xf_a, tickets, n_tickets,
                                  hip_stream);
  if (c.q_mode == ROSAQ_Q_NONE)
    return launch_gather(x_dev, ldx, M, c.D, p->d_perm, ws + w.xf_a, tickets, n_tickets, hip_stream);
  // xhat = x fp16(Q), a dense fp16 contraction.
  // rosaq_tune("rot_splits", n >= 2), 17 to 64 rows: slabs of the contraction and a summing launch,
  // when the caller's workspace has room for the partial tiles.  Not the default: measured at
  // 4096^2 and 64 rows, a stream of single calls gains 6 % (17.3 against 18.5 us) but a whole decode
  // step, where other launches sit between the rotations, loses 0.2 % (3.125 against 3.118 ms).
  if (M > 16 && M <= kMBlock && g_tune_rot.splits >= 2) {
    const int slabs = pick_rotate_slabs(c.D, g_tune_rot.splits);
    if (slabs >= 1 && ws_bytes >= w.part + rotate_slab_part_bytes(c.D, slabs))
      return launch_rotate_slabs(x_dev, ldx, M, c.D, p->d_qf, slabs, ws + w.part, ws + w.xf_b, tickets,
                                 n_tickets, hip_stream);
  }
  // the default: one launch of the all-fp16 GEMM whose "weight" is Q^T with rows already in
  // storage order
  GemmArgs a{};
  a.xf = ws + w.xf_a;
  if (rotates_in_place(c.D, M)) {
    a.xrow = x_dev;
    a.ldx = ldx;
    // no launch in front of the rotation: it runs unsplit and clears the main GEMM's tickets itself
    a.zero_ptr = n_tickets ? tickets : nullptr;
    a.zero_count = n_tickets;
  } else {
    const int rc = launch_gather(x_dev, ldx, M, c.D, nullptr, ws + w.xf_a, tickets, n_tickets, hip_stream);
    if (rc != ROSAQ_OK) return rc;
  }
  a.nseg = 1;
  a.seg[0].wS = p->d_qf; a.seg[0].wq = nullptr;
  a.seg[0].out = ws + w.xf_b; a.seg[0].ldo = 0; a.seg[0].N = c.D;
  a.M = M;
  a.ks_s = c.D / kKStep; a.G = 0; a.KS = c.D / kKStep; a.KS_out = c.D / kKStep;
  a.bits = 4; a.out_frag = 1;
  return launch_gemm(a, plan_gemm(a, rotation_tune()), hip_stream);
}

// Whether an output of the call lies in the memory between x's first and last element.
static bool overlaps(const GemmArgs& a, const void* x_dev, int M, int64_t ldx) {
  const uintptr_t x0 = reinterpret_cast<uintptr_t>(x_dev), x1 = x0 + 2 * (static_cast<uint64_t>(M - 1) * ldx + static_cast<uint64_t>(a.KS) * kKStep);
  for (int i = 0; i < a.nseg; ++i) {
    const uintptr_t y0 = reinterpret_cast<uintptr_t>(a.seg[i].out), y1 = y0 + 2 * (static_cast<uint64_t>(M - 1) * a.seg[i].ldo + a.seg[i].N);
    if (x0 < y1 && y0 < x1) return true;
  }
  return false;
}

static int run_call(const rosaq_packed_t* const* ps, int count, const void* x_dev, int M,
                    int64_t ldx, void* const* ys, const int64_t* ldys, char* ws, size_t ws_bytes,
                    const WsPlan& w, void* hip_stream, bool swiglu = false) {
  const GemmArgs a = main_gemm(ps, count, plan_io(*ps[0], w, ws, ws_bytes), M, ys, ldys, swiglu);
  const GemmPlan plan = plan_gemm(a, g_tune);
  const rosaq_packed& p0 = *ps[0];
  // in one launch, x is read while outputs are stored: not where they share memory
  if (p0.c.q_mode == ROSAQ_Q_HEADWISE && g_tune_stages == 3 && g_tune_rot.wide == 0 && !overlaps(a, x_dev, M, ldx) &&
      fuses_rotation(a, plan, hip_stream))
    return launch_rotate_gemm(a, x_dev, ldx, p0.d_qf, p0.d_pos, hip_stream);
  const int n_tickets = ticket_words(plan);
  int rc = ROSAQ_OK;
  if (g_tune_stages & 1)
    rc = run_prologue(ps[0], w, x_dev, M, ldx, ws, ws_bytes, n_tickets, hip_stream);
  else if (n_tickets)    // what an earlier call left in the workspace are activations; its tickets it may not have used
    rc = launch_clear(ws + w.tickets, n_tickets, hip_stream);
  if (rc != ROSAQ_OK) return rc;
  if (!(g_tune_stages & 2)) return ROSAQ_OK;
  return launch_gemm(a, plan, hip_stream);
}

static uint64_t fnv1a(uint64_t h, const void* data, size_t n) {
  const unsigned char* b = static_cast<const unsigned char*>(data);
  for (size_t i = 0; i < n; ++i) { h ^= b[i]; h *= 1099511628211ull; }
  return h;
}

}  // namespace rosaq

using namespace rosaq;

extern "C" {

int rosaq_pack_weights(const rosaq_pack_desc* desc, void* hip_stream, rosaq_packed_t** out) {
  if (!out) return fail(ROSAQ_ERR_NULL, "out is NULL");
  *out = nullptr;
  int rc = check_desc(desc);
  if (rc != ROSAQ_OK) return rc;
  rosaq_packed* p = new (std::nothrow) rosaq_packed();
  if (!p) return fail(ROSAQ_ERR_NOMEM, "out of host memory");
  std::string err;
  try {
    if (desc->host_only) {
      rc = pack_host(*desc, &p->c, &err);
      if (rc != ROSAQ_OK) set_error(err);
      else if (desc->q_mode != ROSAQ_Q_NONE)
        p->rot_fingerprint = rotation_hash_host(desc->Q, static_cast<size_t>(desc->in_features) *
                                                             (desc->q_mode == ROSAQ_Q_FULL ? desc->in_features : kHeadDim));
    } else {
      try {
        rc = pack_device(*desc, static_cast<hipStream_t>(hip_stream), p);
      } catch (const std::exception&) { rc = fail(ROSAQ_ERR_NOMEM, "out of host memory"); }
      // Without a GPU that could look (no device, no memory), the host does: bad input is named as such either way.
      if ((rc == ROSAQ_ERR_HIP || rc == ROSAQ_ERR_NOMEM) && pack_validate(*desc, &err) != ROSAQ_OK)
        rc = fail(ROSAQ_ERR_NONFINITE, err);
    }
  } catch (const std::exception&) { rc = fail(ROSAQ_ERR_NOMEM, "out of host memory"); }
  if (rc != ROSAQ_OK) { rosaq_free(p); return rc; }
  // the storage order's bytes and the rotation's hash (left in the handle by the device path)
  uint64_t h = fnv1a(1469598103934665603ull, &desc->q_mode, sizeof(desc->q_mode));
  h = fnv1a(h, p->c.perm.data(), p->c.perm.size() * sizeof(int32_t));
  p->rot_fingerprint = fnv1a(h, &p->rot_fingerprint, sizeof(p->rot_fingerprint));
  if (desc->rotation_absorbed) p->c.q_mode = ROSAQ_Q_NONE;   // run time sees rotated activations
  *out = p;
  return ROSAQ_OK;
}

int rosaq_packed_clone(const rosaq_packed_t* src, void* hip_stream, rosaq_packed_t** out) {
  if (!out) return fail(ROSAQ_ERR_NULL, "out is NULL");
  *out = nullptr;
  if (!src) return fail(ROSAQ_ERR_NULL, "handle is NULL");
  rosaq_packed* p = nullptr;
  try {
    p = new rosaq_packed(*src);
  } catch (const std::bad_alloc&) { return fail(ROSAQ_ERR_NOMEM, "out of host memory"); }
  p->d_blob = nullptr;
  if (!src->host_only) {
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    hipError_t e = hipMalloc(&p->d_blob, src->blob_bytes);
    if (e == hipSuccess)
      e = hipMemcpyAsync(p->d_blob, src->d_blob, src->blob_bytes, hipMemcpyDeviceToDevice, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) {
      set_error(std::string("rosaq_packed_clone: ") + hipGetErrorString(e));
      if (p->d_blob) (void)hipFree(p->d_blob);
      delete p;
      return ROSAQ_ERR_HIP;
    }
    const ptrdiff_t shift = static_cast<char*>(p->d_blob) - static_cast<char*>(src->d_blob);
    auto move = [shift](auto*& q) { q = reinterpret_cast<std::remove_reference_t<decltype(q)>>(
                                        reinterpret_cast<char*>(q) + shift); };
    move(p->d_wS); move(p->d_wq); move(p->d_qf); move(p->d_perm); move(p->d_pos);
  }
  *out = p;
  return ROSAQ_OK;
}

size_t rosaq_workspace_bytes(const rosaq_packed_t* p, int32_t M) {
  if (!p || M < 1) return 0;
  return std::max<size_t>(plan_workspace(*p, M).total, 256);
}

size_t rosaq_workspace_bytes_min(const rosaq_packed_t* p, int32_t M) {
  if (!p || M < 1) return 0;
  return std::max<size_t>(plan_workspace(*p, M).required, 256);
}

size_t rosaq_workspace_bytes_batch(const rosaq_packed_t* const* layers, int32_t count, int32_t M) {
  if (!layers || count < 1 || count > kMaxBatch || M < 1) return 0;
  size_t channels = 0;
  for (int i = 0; i < count; ++i) {
    if (!layers[i]) return 0;
    channels += align_up(static_cast<size_t>(layers[i]->c.N), kTileN);
  }
  return std::max<size_t>(plan_workspace(*layers[0], M, channels).total, 256);
}

int rosaq_linear(const rosaq_packed_t* p, const void* x_dev, int32_t M, int64_t ldx, void* y_dev,
                 int64_t ldy, void* ws_dev, size_t ws_bytes, void* hip_stream) {
  WsPlan w;
  int rc = check_call(p, x_dev, M, ldx, y_dev, ldy, ws_dev, ws_bytes, false, &w);
  if (rc == ROSAQ_OK) rc = check_device(&p, 1);
  if (rc != ROSAQ_OK) return rc;
  return run_call(&p, 1, x_dev, M, ldx, &y_dev, &ldy, static_cast<char*>(ws_dev), ws_bytes, w, hip_stream);
}

int rosaq_linear_headwise(const rosaq_packed_t* p, const void* x_dev, int32_t M, int64_t ldx,
                          void* y_dev, int64_t ldy, void* ws_dev, size_t ws_bytes,
                          void* hip_stream) {
  WsPlan w;
  int rc = check_call(p, x_dev, M, ldx, y_dev, ldy, ws_dev, ws_bytes, true, &w);
  if (rc == ROSAQ_OK) rc = check_device(&p, 1);
  if (rc != ROSAQ_OK) return rc;
  return run_call(&p, 1, x_dev, M, ldx, &y_dev, &ldy, static_cast<char*>(ws_dev), ws_bytes, w, hip_stream);
}

int rosaq_linear_headwise_static(const rosaq_packed_t* p, const void* x_dev, int32_t M, int64_t ldx,
                                 void* y_dev, int64_t ldy, void* hip_stream) {
  if (!p) return fail(ROSAQ_ERR_NULL, "handle is NULL");
  if (M < 1) return fail(ROSAQ_ERR_SHAPE, "M must be at least 1");
  // the size test comes first: it needs no GPU
  const WsPlan need = plan_workspace(*p, M);
  if (need.required > kStaticScratchBytes)
    return fail(ROSAQ_ERR_WORKSPACE, "call needs more scratch than the library's static 8 MiB: use "
                                     "rosaq_linear_headwise with a workspace");
  // the address is only compared against NULL and alignment until the handle has passed its checks
  WsPlan w;
  void* probe = reinterpret_cast<void*>(uintptr_t{256});
  int rc = check_call(p, x_dev, M, ldx, y_dev, ldy, probe, kStaticScratchBytes, true, &w);
  if (rc == ROSAQ_OK) rc = check_device(&p, 1);
  if (rc != ROSAQ_OK) return rc;
  void* ws = nullptr;
  rc = static_scratch(&ws);
  if (rc != ROSAQ_OK) return rc;
  const size_t ws_bytes = std::min(w.total, kStaticScratchBytes);
  return run_call(&p, 1, x_dev, M, ldx, &y_dev, &ldy, static_cast<char*>(ws), ws_bytes, w, hip_stream);
}

int rosaq_linear_batch(const rosaq_packed_t* const* layers, int32_t count, const void* x_dev,
                       int32_t M, int64_t ldx, void* const* y_dev, const int64_t* ldy,
                       void* ws_dev, size_t ws_bytes, void* hip_stream) {
  if (!layers || !y_dev || !ldy) return fail(ROSAQ_ERR_NULL, "layers, y_dev or ldy is NULL");
  if (count < 1 || count > kMaxBatch) return fail(ROSAQ_ERR_ARG, "count must be between 1 and 4");
  for (int i = 0; i < count; ++i)
    if (!layers[i]) return fail(ROSAQ_ERR_NULL, "a layer handle is NULL");
  const rosaq_packed_t* p0 = layers[0];
  for (int i = 1; i < count; ++i) {
    const Canonical& a = layers[i]->c;
    if (a.D != p0->c.D || a.K != p0->c.K || a.bits != p0->c.bits || a.q_mode != p0->c.q_mode ||
        layers[i]->rot_fingerprint != p0->rot_fingerprint)
      return fail(ROSAQ_ERR_MODE, "layers of a batch must share D, K, bits and the rotation");
  }
  WsPlan w;
  for (int i = 0; i < count; ++i) {
    const int rc = check_call(layers[i], x_dev, M, ldx, y_dev[i], ldy[i], ws_dev, ws_bytes,
                              p0->c.q_mode == ROSAQ_Q_HEADWISE, &w);
    if (rc != ROSAQ_OK) return rc;
  }
  if (check_device(layers, count) != ROSAQ_OK) return ROSAQ_ERR_HOSTONLY;
  return run_call(layers, count, x_dev, M, ldx, y_dev, ldy, static_cast<char*>(ws_dev), ws_bytes, w, hip_stream);
}

int rosaq_linear_swiglu(const rosaq_packed_t* gate, const rosaq_packed_t* up, const void* x_dev, int32_t M,
                        int64_t ldx, void* y_dev, int64_t ldy, void* ws_dev, size_t ws_bytes,
                        void* hip_stream) {
  if (!gate || !up) return fail(ROSAQ_ERR_NULL, "a layer handle is NULL");
  const Canonical &a = gate->c, &b = up->c;
  if (a.N != b.N || a.D != b.D || a.K != b.K || a.bits != b.bits || a.q_mode != b.q_mode ||
      gate->rot_fingerprint != up->rot_fingerprint)
    return fail(ROSAQ_ERR_MODE, "gate and up must share N, D, K, bits and the rotation");
  WsPlan w;
  const bool headwise = a.q_mode == ROSAQ_Q_HEADWISE;
  int rc = check_call(gate, x_dev, M, ldx, y_dev, ldy, ws_dev, ws_bytes, headwise, &w);
  if (rc != ROSAQ_OK) return rc;
  const rosaq_packed_t* ps[2] = {gate, up};
  if (check_device(ps, 2) != ROSAQ_OK) return ROSAQ_ERR_HOSTONLY;
  void* ys[2] = {y_dev, y_dev};
  const int64_t ldys[2] = {ldy, ldy};
  return run_call(ps, 2, x_dev, M, ldx, ys, ldys, static_cast<char*>(ws_dev), ws_bytes, w, hip_stream, true);
}

// Workspace of rosaq_mlp_swiglu: [gate / up: what rosaq_linear_swiglu needs without room for partial
// tiles | down: xhat fragments, tickets | room for the down launch's partial tiles].
struct MlpPlan {
  WsPlan gate;
  size_t down_xf = 0, down_tickets = 0, required = 0, part = 0, total = 0;
};
static MlpPlan plan_mlp(const rosaq_packed& gate, const rosaq_packed& down, int M) {
  MlpPlan m;
  m.gate = plan_workspace(gate, M);
  const size_t mblocks = (static_cast<size_t>(M) + kMBlock - 1) / kMBlock;
  size_t off = m.gate.required;
  m.down_xf = off; off += align_up(mblocks * (down.c.D / kKStep) * 4 * 64 * 16, 256);
  m.down_tickets = off; off += kTicketBytes;
  m.required = off;
  m.part = off;
  off += align_up(part_room(M, down.c.N), 256);
  m.total = off;
  return m;
}

static int check_mlp(const rosaq_packed_t* gate, const rosaq_packed_t* up, const rosaq_packed_t* down) {
  if (!gate || !up || !down) return fail(ROSAQ_ERR_NULL, "a layer handle is NULL");
  const Canonical &a = gate->c, &b = up->c, &d = down->c;
  if (a.N != b.N || a.D != b.D || a.K != b.K || a.bits != b.bits || a.q_mode != b.q_mode ||
      gate->rot_fingerprint != up->rot_fingerprint)
    return fail(ROSAQ_ERR_MODE, "gate and up must share N, D, K, bits and the rotation");
  if (d.D != a.N) return fail(ROSAQ_ERR_SHAPE, "down must take gate's output channels as its input");
  if (d.q_mode != ROSAQ_Q_NONE)
    return fail(ROSAQ_ERR_MODE, "down must run without a run-time rotation (q_mode NONE or rotation_absorbed)");
  return ROSAQ_OK;
}

size_t rosaq_workspace_bytes_mlp(const rosaq_packed_t* gate, const rosaq_packed_t* up,
                                 const rosaq_packed_t* down, int32_t M) {
  if (check_mlp(gate, up, down) != ROSAQ_OK || M < 1) return 0;
  return plan_mlp(*gate, *down, M).total;
}

int rosaq_mlp_swiglu(const rosaq_packed_t* gate, const rosaq_packed_t* up, const rosaq_packed_t* down,
                     const void* x_dev, int32_t M, int64_t ldx, void* y_dev, int64_t ldy, void* ws_dev,
                     size_t ws_bytes, void* hip_stream) {
  int rc = check_mlp(gate, up, down);
  if (rc != ROSAQ_OK) return rc;
  // x against gate, y against down; the workspace is checked against this call's own plan below
  WsPlan unused;
  const bool headwise = gate->c.q_mode == ROSAQ_Q_HEADWISE;
  char* ws = static_cast<char*>(ws_dev);
  rc = check_call(gate, x_dev, M, ldx, y_dev, gate->c.N, ws_dev, ws_bytes, headwise, &unused);
  if (rc != ROSAQ_OK) return rc;
  if (!y_dev) return fail(ROSAQ_ERR_NULL, "y is NULL");
  if (ldy < down->c.N) return fail(ROSAQ_ERR_SHAPE, "leading dimension smaller than width");
  if ((static_cast<int64_t>(M) + kMBlock - 1) / kMBlock * kMBlock * down->c.D / 8 > INT32_MAX)
    return fail(ROSAQ_ERR_SHAPE, "M x in_features above 2^34: split the call");
  const MlpPlan m = plan_mlp(*gate, *down, M);
  if (ws_bytes < m.required) return fail(ROSAQ_ERR_WORKSPACE, "workspace missing or too small");
  const rosaq_packed_t* gu[2] = {gate, up};
  const rosaq_packed_t* all[3] = {gate, up, down};
  if (check_device(all, 3) != ROSAQ_OK) return ROSAQ_ERR_HOSTONLY;
  // 1. xhat of the input
  if (g_tune_stages & 1) {
    rc = run_prologue(gate, m.gate, x_dev, M, ldx, ws, m.gate.required, 0, hip_stream);   // a gated launch is never split
    if (rc != ROSAQ_OK) return rc;
  }
  if (!(g_tune_stages & 2)) return ROSAQ_OK;
  // 3. y = h What_down^T
  GemmIO dn{};
  dn.xf = ws + m.down_xf;
  dn.tickets = ws + m.down_tickets + kTicketsPerLaunch * sizeof(uint32_t);
  dn.part = ws + m.part;
  dn.part_bytes = ws_bytes > m.part ? ws_bytes - m.part : 0;
  const int64_t ldys[1] = {ldy};
  const GemmArgs third = main_gemm(&down, 1, dn, M, &y_dev, ldys);
  const GemmPlan third_plan = plan_gemm(third, g_tune);
  // 2. silu(gate) * up, written as down's input fragments at down's storage positions; clears that launch's tickets
  GemmIO io = plan_io(*gate, m.gate, ws, m.gate.required);
  io.part = nullptr; io.part_bytes = 0;
  io.chain_pos = down->d_pos; io.chain_ks = down->c.D / kKStep;
  io.zero_count = ticket_words(third_plan);
  io.zero_ptr = io.zero_count ? ws + m.down_tickets : nullptr;
  void* hs[2] = {ws + m.down_xf, ws + m.down_xf};
  const int64_t ldh[2] = {0, 0};
  const GemmArgs second = main_gemm(gu, 2, io, M, hs, ldh, true);
  rc = launch_gemm(second, plan_gemm(second, g_tune), hip_stream);
  return rc != ROSAQ_OK ? rc : launch_gemm(third, third_plan, hip_stream);
}

int rosaq_packed_info(const rosaq_packed_t* p, int32_t* N, int32_t* D, int32_t* K, int32_t* bits,
                      int32_t* group, int32_t* q_mode, size_t* device_bytes) {
  if (!p) return fail(ROSAQ_ERR_NULL, "handle is NULL");
  if (N) *N = p->c.N;
  if (D) *D = p->c.D;
  if (K) *K = p->c.K;
  if (bits) *bits = p->c.bits;
  if (group) *group = kGroup;
  if (q_mode) *q_mode = p->c.q_mode;
  if (device_bytes) *device_bytes = p->blob_bytes;
  return ROSAQ_OK;
}

int rosaq_packed_export(const rosaq_packed_t* p, int32_t* salient_idx, uint16_t* W_S, uint8_t* codes,
                        uint16_t* scales, uint16_t* zeros) {
  if (!p) return fail(ROSAQ_ERR_NULL, "handle is NULL");
  const Canonical& c = p->c;
  // by several threads: a caller's fresh 45 MB array costs one thread 10 ms in page faults
  auto copy = [](void* dst, const void* src, size_t bytes) {
    constexpr size_t kSlice = size_t{256} << 10;
    if (!dst) return;
    parallel_rows(static_cast<int>((bytes + kSlice - 1) / kSlice), [&](int lo, int hi) {
      const size_t from = lo * kSlice, to = std::min(bytes, hi * kSlice);
      if (from < to) std::memcpy(static_cast<char*>(dst) + from, static_cast<const char*>(src) + from, to - from);
    });
  };
  try {
    copy(salient_idx, c.salient_idx.data(), c.salient_idx.size() * 4);
    copy(W_S, c.W_S.data(), c.W_S.size() * 2);
    copy(codes, c.codes.data(), c.codes.size());
    copy(scales, c.scales.data(), c.scales.size() * 2);
    copy(zeros, c.zeros.data(), c.zeros.size() * 2);
  } catch (const std::exception&) { return fail(ROSAQ_ERR_NOMEM, "out of host memory"); }
  return ROSAQ_OK;
}

int rosaq_pca_headwise(const void* X_dev, int32_t n_cal, int32_t D, int64_t ldx, float* Q_host,
                       double* eigenvalues_host, void* hip_stream) {
  if (!X_dev || !Q_host || !eigenvalues_host) return fail(ROSAQ_ERR_NULL, "a pointer is NULL");
  if (n_cal < 1 || D < kHeadDim || D % kHeadDim != 0 || ldx < D)
    return fail(ROSAQ_ERR_SHAPE, "n_cal >= 1, D a positive multiple of 128, ldx >= D");
  if (reinterpret_cast<uintptr_t>(X_dev) % 2) return fail(ROSAQ_ERR_ALIGN, "X must be 2-byte aligned");
  try {   // the solver keeps host-side bookkeeping in vectors
    return pca_headwise_device(X_dev, n_cal, D, ldx, Q_host, eigenvalues_host, hip_stream);
  } catch (const std::exception&) { return fail(ROSAQ_ERR_NOMEM, "out of host memory"); }
}

int rosaq_pca_full(const void* X_dev, int32_t n_cal, int32_t D, int64_t ldx, float* Q_host,
                   double* eigenvalues_host, void* hip_stream) {
  if (!X_dev || !Q_host || !eigenvalues_host) return fail(ROSAQ_ERR_NULL, "a pointer is NULL");
  if (n_cal < 1 || D < kGroup || D % kGroup != 0 || D > 8192 || ldx < D)
    return fail(ROSAQ_ERR_SHAPE, "n_cal >= 1, D a multiple of 128 up to 8192, ldx >= D");
  if (reinterpret_cast<uintptr_t>(X_dev) % 2) return fail(ROSAQ_ERR_ALIGN, "X must be 2-byte aligned");
  try {
    return pca_full_device(X_dev, n_cal, D, ldx, Q_host, eigenvalues_host, hip_stream);
  } catch (const std::exception&) { return fail(ROSAQ_ERR_NOMEM, "out of host memory"); }
}

int rosaq_stream_probe(const void* src_dev, size_t src_bytes, const void* shared_dev,
                       size_t shared_bytes, size_t shared_bytes_per_workgroup, int32_t workgroups,
                       int32_t threads, void* sink_dev, size_t sink_bytes, void* hip_stream) {
  if (!src_dev || !sink_dev) return fail(ROSAQ_ERR_NULL, "src_dev or sink_dev is NULL");
  if (workgroups < 1 || threads < 64 || threads > 1024 || threads % 64)
    return fail(ROSAQ_ERR_ARG, "workgroups >= 1 and threads a multiple of 64 up to 1024");
  const size_t waves = static_cast<size_t>(workgroups) * (threads / 64);
  if (src_bytes == 0 || src_bytes % (waves * 1024))
    return fail(ROSAQ_ERR_SHAPE, "src_bytes must be a positive multiple of 1 KiB per wave");
  const size_t wpw = static_cast<size_t>(threads / 64) * 1024;
  if (shared_bytes_per_workgroup % wpw || shared_bytes % 1024)
    return fail(ROSAQ_ERR_SHAPE, "shared sizes must be multiples of 1 KiB (per wave)");
  if (shared_bytes_per_workgroup && (!shared_dev || shared_bytes < shared_bytes_per_workgroup / (threads / 64)))
    return fail(ROSAQ_ERR_SHAPE, "shared buffer missing or smaller than one wave's share");
  if (sink_bytes < waves * 1024) return fail(ROSAQ_ERR_WORKSPACE, "sink smaller than 16 bytes per thread");
  if (reinterpret_cast<uintptr_t>(src_dev) % 16 || reinterpret_cast<uintptr_t>(shared_dev) % 16 ||
      reinterpret_cast<uintptr_t>(sink_dev) % 16)
    return fail(ROSAQ_ERR_ALIGN, "probe buffers must be 16-byte aligned");
  return launch_stream_probe(src_dev, shared_dev, workgroups, threads,
                             static_cast<int>(src_bytes / (waves * 1024)),
                             static_cast<int>(shared_bytes_per_workgroup / wpw),
                             static_cast<int>(shared_bytes / 1024), sink_dev, hip_stream);
}

int rosaq_tune(const char* key, int32_t value) {
  if (!key) return fail(ROSAQ_ERR_NULL, "key is NULL");
  if (!std::strcmp(key, "wpb")) {
    if (value != 0 && value != 4 && value != 8 && value != 16)
      return fail(ROSAQ_ERR_ARG, "wpb must be 0, 4, 8 or 16");
    g_tune.wpb = value; return ROSAQ_OK;
  }
  if (!std::strncmp(key, "rot_", 4) && std::strcmp(key, "rot_splits")) {
    const char* k = key + 4;
    if (value < 0 || value > 4 || value == 3) {
      if (!((std::strcmp(k, "depth") == 0 || std::strcmp(k, "nt") == 0) && value == 3) && !(std::strcmp(k, "nt") == 0 && value == 5))
        return fail(ROSAQ_ERR_ARG, "bad rotation tuning value");
    }
    if (!std::strcmp(k, "mt")) { g_tune_rot.mt = value; return ROSAQ_OK; }
    if (!std::strcmp(k, "nt")) { g_tune_rot.nt = value; return ROSAQ_OK; }
    if (!std::strcmp(k, "depth")) { g_tune_rot.depth = value; return ROSAQ_OK; }
    return fail(ROSAQ_ERR_ARG, "unknown tuning key");
  }
  if (!std::strcmp(key, "wide")) {
    if (value < 0 || value > 2) return fail(ROSAQ_ERR_ARG, "wide must be 0, 1 or 2");
    g_tune.wide = g_tune_rot.wide = value; return ROSAQ_OK;
  }
  if (!std::strcmp(key, "depth")) {
    if (value < 0 || value > 4) return fail(ROSAQ_ERR_ARG, "depth must be 0 to 4");
    g_tune.depth = value; return ROSAQ_OK;
  }
  if (!std::strcmp(key, "splits") || !std::strcmp(key, "rot_splits")) {
    if (value < 0 || value > kMaxSplits) return fail(ROSAQ_ERR_ARG, "splits must be 0 to 16");
    (key[0] == 'r' ? g_tune_rot : g_tune).splits = value; return ROSAQ_OK;
  }
  if (!std::strcmp(key, "mt") || !std::strcmp(key, "nt")) {
    const bool wide = key[0] == 'n' && (value == 3 || value == 6);
    if (value != 0 && value != 1 && value != 2 && value != 4 && !wide)
      return fail(ROSAQ_ERR_ARG, "tile counts must be 0, 1, 2 or 4 (nt also 3 or 6)");
    (key[0] == 'm' ? g_tune.mt : g_tune.nt) = value; return ROSAQ_OK;
  }
  if (!std::strcmp(key, "pca_sweeps")) {
    if (value < 0 || value > 1) return fail(ROSAQ_ERR_ARG, "pca_sweeps must be 0 or 1");
    g_tune_pca_sweeps = value == 1; return ROSAQ_OK;
  }
  if (!std::strcmp(key, "stages")) {
    if (value < 1 || value > 3) return fail(ROSAQ_ERR_ARG, "stages must be 1, 2 or 3");
    g_tune_stages = value; return ROSAQ_OK;
  }
  return fail(ROSAQ_ERR_ARG, "unknown tuning key");
}

int rosaq_launch_shape(int32_t M, int32_t channels, int32_t in_features, int32_t bits, int32_t* shape_out) {
  if (!shape_out) return fail(ROSAQ_ERR_NULL, "shape_out is NULL");
  if (M < 1 || channels < 1 || channels % kTileN || in_features < kGroup || in_features % kGroup)
    return fail(ROSAQ_ERR_SHAPE, "M >= 1, channels a positive multiple of 16, in_features a positive multiple of 128");
  if (bits != 3 && bits != 4 && bits != 16) return fail(ROSAQ_ERR_ARG, "bits must be 3, 4 or 16");
  const GemmShape s = pick_gemm_shape(M, channels / kTileN, in_features, bits, g_tune,
                                      part_room(M, channels), kTicketsPerLaunch);
  shape_out[0] = s.mt; shape_out[1] = s.nt; shape_out[2] = s.wpb; shape_out[3] = s.depth;
  shape_out[4] = s.splits;
  return ROSAQ_OK;
}

int rosaq_launch_many_rows(int32_t M, int32_t channels, int32_t in_features, int32_t K, int32_t bits, int32_t q_mode,
                           int32_t* uses_out) {
  if (!uses_out) return fail(ROSAQ_ERR_NULL, "uses_out is NULL");
  if (M < 1 || channels < 1 || channels % kTileN || in_features < kGroup || in_features % kGroup || K < 0 ||
      K > in_features || K % kGroup)
    return fail(ROSAQ_ERR_SHAPE, "M >= 1, channels a positive multiple of 16, in_features a positive multiple of 128, "
                                 "K a multiple of 128 up to in_features");
  if (bits != 3 && bits != 4) return fail(ROSAQ_ERR_ARG, "bits must be 3 or 4");
  if (q_mode < ROSAQ_Q_NONE || q_mode > ROSAQ_Q_HEADWISE) return fail(ROSAQ_ERR_ARG, "unknown q_mode");
  const int D = in_features;
  int uses = prefers_wide(M, channels / kTileN, D, K, K == D ? 16 : bits, g_tune) ? 1 : 0;
  if (q_mode == ROSAQ_Q_HEADWISE && rotates_whole_heads(D, M)) uses |= 2;
  if (q_mode == ROSAQ_Q_FULL && prefers_wide(M, D / kTileN, D, D, 16, rotation_tune())) uses |= 2;
  *uses_out = uses;
  return ROSAQ_OK;
}

int rosaq_packed_image(const rosaq_packed_t* p, int32_t which, void* out_host, size_t* bytes) {
  if (!p || !bytes) return fail(ROSAQ_ERR_NULL, "handle or bytes is NULL");
  if (which < 0 || which > 3)
    return fail(ROSAQ_ERR_ARG, "which must be 0 / 1 (fp16 fragments / low-bit records rebuilt on the host) or 2 / 3 "
                               "(the same two read back from the device)");
  if (which >= 2) {
    if (p->host_only) return fail(ROSAQ_ERR_HOSTONLY, "handle was packed with host_only");
    const size_t tiles = (static_cast<size_t>(p->c.N) + 127) / 128 * 8;
    const size_t need = which == 2 ? tiles * (p->c.K / kKStep) * 64 * 16
                                   : tiles * p->c.G * ((p->c.bits == 4 ? 256 : 192) + 16) * 4;
    if (out_host) {
      if (*bytes < need) { *bytes = need; return fail(ROSAQ_ERR_WORKSPACE, "image buffer too small"); }
      if (need) ROSAQ_HIP(hipMemcpy(out_host, which == 2 ? p->d_wS : p->d_wq, need, hipMemcpyDeviceToHost));
    }
    *bytes = need;
    return ROSAQ_OK;
  }
  DeviceImage img;
  try {
    build_device_image(p->c, nullptr, &img);
  } catch (const std::exception&) { return fail(ROSAQ_ERR_NOMEM, "out of host memory"); }
  const std::vector<uint32_t>& v = which == 0 ? img.wS : img.wq;
  const size_t need = v.size() * sizeof(uint32_t);
  if (out_host) {
    if (*bytes < need) { *bytes = need; return fail(ROSAQ_ERR_WORKSPACE, "image buffer too small"); }
    if (need) std::memcpy(out_host, v.data(), need);
  }
  *bytes = need;
  return ROSAQ_OK;
}

int rosaq_block_map(int32_t workgroup, int32_t chunks, int32_t row_groups, int32_t* chunk_out, int32_t* row_group_out) {
  if (chunks < 1 || row_groups < 1) return fail(ROSAQ_ERR_SHAPE, "chunks and row_groups must be positive");
  if (workgroup >= 0 && (!chunk_out || !row_group_out)) return fail(ROSAQ_ERR_NULL, "output pointer is NULL");
  int c = -1, m = -1;
  const int r = block_map_host(workgroup, chunks, row_groups, &c, &m);
  if (workgroup < 0) return r;
  *chunk_out = r ? c : -1;
  *row_group_out = r ? m : -1;
  return r;
}

void rosaq_free(rosaq_packed_t* p) {
  if (!p) return;
  if (p->d_blob) (void)hipFree(p->d_blob);
  delete p;
}

const char* rosaq_last_error(void) { return g_error.c_str(); }

}  // extern "C"
