// C ABI of the LQ-SGD compressor: context, device state, phase sequencing,
// taps and timing.  All arithmetic of the method runs in the kernels; this
// file only moves bytes and launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "lqsgd.h"
#include "lqsgd_kernels.h"
#include "lqsgd_plan.h"

using namespace lqsgd;

namespace {

thread_local std::string g_create_error;

enum State { kIdle = 0, kPCompressed = 1, kPDone = 2, kQCompressed = 3 };

struct EventPair {
  hipEvent_t a, b;
  int kernel;
};

}  // namespace

struct lqsgd_ctx {
  Plan plan;
  hipStream_t stream = nullptr;
  int device = 0;
  State state = kIdle;
  int sweep_dir = 0;        // direction of the next streaming sweep (alternates)
  bool flip = true;
  bool eager = false;       // LQSGD_FLAG_EAGER_RESIDUAL
  bool pending = false;     // E buffer holds M; E = M - P-bar Q-bar^T not applied yet
  CoopState coop;           // one-launch Gram-Schmidt: launch count, device capacity, wait bound
  int* status = nullptr;    // pinned, device-visible: non-zero once a bounded device-side wait has expired
  char* bounce = nullptr;   // kBounceBytes of pinned memory behind it (fetch)
  std::string err;
  std::vector<void*> allocs;
  // When set, device memory is carved out of this caller-provided block instead of being allocated
  // (the context then owns no device memory at all).
  unsigned char* arena = nullptr;
  size_t arena_cap = 0, arena_used = 0;
  unsigned char* operands = nullptr;   // ... and another for padded operand copies and items that it has no room for
  size_t operands_cap = 0, operands_used = 0;
  float* grams = nullptr;              // ... and one for second-pass Gram matrices, as large as the first block
  DevArgs args{};
  // device copies of the work lists
  Tile* d_tilesA = nullptr; Tile* d_tilesB = nullptr; Tile* d_tilesG = nullptr; Tile* d_tilesBM = nullptr; Tile* d_tilesAG = nullptr; Tile* d_tilesR = nullptr;
  XTile* d_tilesXP = nullptr; XTile* d_tilesXQ = nullptr;
  RTile* d_tilesRQ = nullptr; RTile* d_tilesRP = nullptr; VTile* d_tilesV = nullptr;
  // pointer tables
  const float** d_grads = nullptr; float** d_ghat = nullptr;
  std::vector<const float*> h_grads; std::vector<float*> h_ghat;
  bool grads_valid = false, ghat_valid = false;
  bool stale[2] = {false, false};   // the padded copies of P-bar / Q-bar lag behind a factor that the host has set
  bool alias_checked = false;   // the bound gradient and output tables have been checked against each other
  // timing
  std::string launched[LQSGD_KERNEL_COUNT];   // device function last launched for each timing slot
  bool timing = false;
  std::vector<EventPair> events;
  size_t events_used = 0;
};

namespace {

int fail(lqsgd_ctx* c, int code, const std::string& msg) {
  if (c) c->err = msg; else g_create_error = msg;
  return code;
}

int fail_hip(lqsgd_ctx* c, hipError_t e, const char* what) {
  // Clear the sticky error so that a later call does not report it again.
  (void)hipGetLastError();
  return fail(c, LQSGD_EHIP, std::string(what) + ": " + hipGetErrorString(e));
}

#define HIP_TRY(ctx, expr)                                   \
  do {                                                       \
    hipError_t e_ = (expr);                                  \
    if (e_ != hipSuccess) return fail_hip(ctx, e_, #expr);   \
  } while (0)

template <typename T>
int dev_alloc(lqsgd_ctx* c, T** out, size_t count, bool zero) {
  *out = nullptr;
  if (count == 0) count = 1;
  if (c->arena) {     // bump allocation, 256-byte granules; the block is cleared as a whole by whoever set it up
    const size_t bytes = (count * sizeof(T) + 255) & ~(size_t)255;
    if (bytes > c->arena_cap - c->arena_used) {
      char buf[200];
      std::snprintf(buf, sizeof buf, "this configuration needs more scratch memory than the static buffer holds (%zu bytes)",
                    c->arena_cap);
      return fail(c, LQSGD_EUNSUPPORTED, buf);
    }
    *out = reinterpret_cast<T*>(c->arena + c->arena_used);
    c->arena_used += bytes;
    return LQSGD_OK;
  }
  void* p = nullptr;
  hipError_t e = hipMalloc(&p, count * sizeof(T));
  if (e != hipSuccess) {
    (void)hipGetLastError();
    char buf[160];
    std::snprintf(buf, sizeof buf, "hipMalloc of %zu bytes failed: %s", count * sizeof(T), hipGetErrorString(e));
    return fail(c, LQSGD_ENOMEM, buf);
  }
  c->allocs.push_back(p);
  if (zero) HIP_TRY(c, hipMemsetAsync(p, 0, count * sizeof(T), c->stream));
  *out = static_cast<T*>(p);
  return LQSGD_OK;
}

template <typename T>
int dev_upload(lqsgd_ctx* c, T** out, const std::vector<T>& v) {
  int rc = dev_alloc(c, out, v.size(), false);
  if (rc) return rc;
  if (!v.empty()) HIP_TRY(c, hipMemcpy(*out, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice));
  return LQSGD_OK;
}

struct Timed {
  lqsgd_ctx* c;
  int kernel;
  EventPair* ep = nullptr;
  Timed(lqsgd_ctx* ctx, int k) : c(ctx), kernel(k) {
    if (!c->timing) return;
    if (c->events_used == c->events.size()) {
      EventPair p{};
      if (hipEventCreate(&p.a) != hipSuccess || hipEventCreate(&p.b) != hipSuccess) { (void)hipGetLastError(); return; }
      c->events.push_back(p);
    }
    ep = &c->events[c->events_used++];
    ep->kernel = kernel;
    (void)hipEventRecord(ep->a, c->stream);
  }
  ~Timed() {
    if (ep) (void)hipEventRecord(ep->b, c->stream);
    c->launched[kernel] = last_launched_kernel();
  }
};

// Waits for the context's stream and reports a device-side wait that expired.
int sync_stream(lqsgd_ctx* c) {
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  if (c->status && *static_cast<volatile int*>(c->status) != 0)
    return fail(c, LQSGD_EHIP, "a device-side barrier wait expired; results of this context are invalid");
  return LQSGD_OK;
}

// Device values for the host, once the stream is done.  Up to 64 KiB they are copied behind the work on the stream into pinned
// memory and from there, with one wait for both (us, on an idle stream: 16 KiB 17 -> 12, just under 64 KiB 35 -> 11, 64 KiB 11 -> 11; a step
// of 1024 x 64, r = 16 and its 64 KiB P-bar 69.7 -> 66.6).  From 64 KiB on the runtime's own staging is as fast, and memory for more would
// make contexts slower to create (256 KiB 60 to 150 us).
constexpr size_t kBounceBytes = 64 << 10;
int fetch(lqsgd_ctx* c, void* host, const void* src, size_t bytes) {
  const bool bounce = c->bounce && bytes <= kBounceBytes;
  if (bounce) HIP_TRY(c, hipMemcpyAsync(c->bounce, src, bytes, hipMemcpyDeviceToHost, c->stream));
  if (int rcs = sync_stream(c)) return rcs;
  if (bounce) std::memcpy(host, c->bounce, bytes);
  else HIP_TRY(c, hipMemcpy(host, src, bytes, hipMemcpyDeviceToHost));
  return LQSGD_OK;
}

int check_matrix_layer(lqsgd_ctx* c, int32_t layer, const LayerDesc** out) {
  if (layer < 0 || layer >= c->plan.n_all) return fail(c, LQSGD_ESHAPE, "layer index out of range");
  const int k = c->plan.kind_of[layer];
  if (k < 0) return fail(c, LQSGD_ESHAPE, "layer is a VECTOR layer");
  *out = &c->plan.layers[k];
  return LQSGD_OK;
}

int check_worker(lqsgd_ctx* c, int32_t worker) {
  if (worker < 0 || worker >= c->plan.W) return fail(c, LQSGD_ESHAPE, "worker index out of range");
  return LQSGD_OK;
}

// Copies a pointer list to its device table, which launches already enqueued may still be reading.  Short lists go
// there in stream order (ResNet-18 set, W = 8, other buffers every step: the wait and the two copies cost 60 us a step),
// long ones after a wait.  A list cannot change while the stream is being captured: a captured copy would bring this
// call's pointers back at every replay, and a wait would end the capture.  Such a call is refused before it touches
// the stream, and the list that is bound stays bound.  *valid: whether the table holds the host's copy of the list.
int upload_pointers(lqsgd_ctx* c, const void** dst, const void* const* src, size_t n, bool* valid) {
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  const bool known = hipStreamIsCapturing(c->stream, &cap) == hipSuccess;
  if (!known) (void)hipGetLastError();
  if (known && cap != hipStreamCaptureStatusNone)
    return fail(c, LQSGD_EHIP, "the pointer lists of a call that is being captured must have been used in an ordinary call before");
  *valid = false;
  if (known && n <= 4 * (size_t)kPointerBatch) {
    HIP_TRY(c, launch_write_pointers(dst, src, n, c->stream));
    return LQSGD_OK;
  }
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  HIP_TRY(c, hipMemcpy(dst, src, n * sizeof(void*), hipMemcpyHostToDevice));
  return LQSGD_OK;
}

// Copies the caller's pointer list to the device table when it changed.
int bind_grads(lqsgd_ctx* c, const float* const* grads) {
  const size_t n = (size_t)c->plan.W * c->plan.n_all;
  for (size_t i = 0; i < n; ++i) {
    if (!grads[i]) return fail(c, LQSGD_EINVAL, "NULL gradient pointer");
    if (reinterpret_cast<uintptr_t>(grads[i]) & 15u) return fail(c, LQSGD_EINVAL, "gradient pointer not 16-byte aligned");
  }
  if (c->grads_valid && std::memcmp(c->h_grads.data(), grads, n * sizeof(float*)) == 0) return LQSGD_OK;
  if (int rc = upload_pointers(c, reinterpret_cast<const void**>(c->d_grads), reinterpret_cast<const void* const*>(grads), n, &c->grads_valid)) return rc;
  c->h_grads.assign(grads, grads + n);
  c->grads_valid = true;
  c->alias_checked = false;
  return LQSGD_OK;
}

int bind_ghat(lqsgd_ctx* c, float* const* ghat) {
  if (!ghat) { c->args.ghat = nullptr; return LQSGD_OK; }
  const size_t n = (size_t)c->plan.n_all;
  for (size_t i = 0; i < n; ++i)
    if (ghat[i] && (reinterpret_cast<uintptr_t>(ghat[i]) & 15u))
      return fail(c, LQSGD_EINVAL, "G-hat pointer not 16-byte aligned");
  if (!(c->ghat_valid && std::memcmp(c->h_ghat.data(), ghat, n * sizeof(float*)) == 0)) {
    if (int rc = upload_pointers(c, const_cast<const void**>(reinterpret_cast<void**>(c->d_ghat)), reinterpret_cast<const void* const*>(ghat), n, &c->ghat_valid)) return rc;
    c->h_ghat.assign(ghat, ghat + n);
    c->ghat_valid = true;
    c->alias_checked = false;
  }
  c->args.ghat = c->d_ghat;
  return LQSGD_OK;
}

// ---- the phases -------------------------------------------------------------
int next_dir(lqsgd_ctx* c) {
  const int d = c->sweep_dir;
  if (c->flip) c->sweep_dir ^= 1;
  return d;
}

// The sweeps read P-bar and Q-bar from copies with padded rows when some layer has fewer ranks than the register
// pad.  The exchange and the Gram-Schmidt of an aggregate by one workgroup write factor and copy together; other kernels
// that write a factor are followed by this.
int refresh_padded(lqsgd_ctx* c, int which) {
  if (c->plan.padded) HIP_TRY(c, launch_pad_factor(c->plan.RP, which, c->args, c->stream));
  return LQSGD_OK;
}
// A factor that the host has set is copied by the next sweep that reads copies: one launch for all layers set by then.
// While the stream is being captured the launch only becomes part of the graph, and the factor stays to be copied.
int refresh_stale(lqsgd_ctx* c) {
  for (int which = 0; which < 2; ++which) {
    if (!c->stale[which]) continue;
    if (int rc = refresh_padded(c, which)) return rc;
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(c->stream, &cap) != hipSuccess) { (void)hipGetLastError(); cap = hipStreamCaptureStatusNone; }
    c->stale[which] = cap != hipStreamCaptureStatusNone;
  }
  return LQSGD_OK;
}

// The one-launch Gram-Schmidt's state, or null where the context must not launch cooperatively.
CoopState* coop_state(lqsgd_ctx* c) {
  return (c->plan.cfg.flags & LQSGD_FLAG_NO_COOPERATIVE_LAUNCH) ? nullptr : &c->coop;
}

int run_sweep0(lqsgd_ctx* c) {
  if (int rc = refresh_stale(c)) return rc;
  int dir = next_dir(c);
  // A list that starts with the widest items (Plan::build) is not taken from its end, as a residual pass in between (get_state of E)
  // would have it from then on: a step after one, ResNet-18 set, W = 8, r = 50 605 us, in the list's order 595, r = 32 398 and 389,
  // ragged set, r = 20, W = 4 137 and 133.  The eager schedule's three sweeps do alternate (r = 50 810 and 819, r = 32 527 and 541).
  if (c->plan.mfma && c->pending) {
    dir = 0;
    if (c->flip) c->sweep_dir = 1;
  }
  { Timed t(c, LQSGD_KERNEL_ADD_PROJECT);
    if (c->plan.mfma_a)
      HIP_TRY(c, launch_mfma_sweep(c->plan.RP, c->pending ? 1 : 0, c->args, c->d_tilesA, (int)c->plan.tilesA.size(),
                                   c->plan.twoA, dir, c->stream));
    else
      HIP_TRY(c, launch_add_project(c->plan.RP, c->args, c->d_tilesA, (int)c->plan.tilesA.size(), c->pending ? 1 : 0,
                                    c->plan.narrow_rows ? 1 : 0, dir, c->stream)); }
  c->pending = false;
  if (c->plan.agg_first) {   // the exchange comes first: only add up the partial planes (and take the absmax)
    Timed t(c, LQSGD_KERNEL_REDUCE_P);
    HIP_TRY(c, launch_reduce_q(0, c->args, c->d_tilesRP, (int)c->plan.tilesRP.size(), c->stream));
  } else {
    Timed t(c, LQSGD_KERNEL_ORTH);
    bool copied = false;
    HIP_TRY(c, launch_orth(c->plan.RP, c->plan.max_rows, c->plan.max_rank, c->plan.plane_rows, c->args, coop_state(c), &copied, c->stream));
  }
  return LQSGD_OK;
}
// Aggregate-first order: Gram-Schmidt once per layer, in place on the aggregated P; the aggregate
// as it was before goes to worker 0's slot of the (otherwise unused) per-worker Gram-Schmidt output.
int run_orth_shared(lqsgd_ctx* c) {
  Timed t(c, LQSGD_KERNEL_ORTH);
  DevArgs a = c->args;
  a.W = 1;
  a.orth_shared = 1;
  a.Ppart = c->args.Pbar; a.ppart_stride = 0;
  a.Ppre = c->args.Porth;
  a.Porth = c->args.Pbar;
  bool copied = false;
  HIP_TRY(c, launch_orth(c->plan.RP, c->plan.max_rows, c->plan.max_rank, c->plan.max_rows, a, coop_state(c), &copied, c->stream));
  return copied ? LQSGD_OK : refresh_padded(c, 0);
}
int run_exchange(lqsgd_ctx* c, int mode, int phase) {
  { Timed t(c, phase ? LQSGD_KERNEL_EXCHANGE_Q : LQSGD_KERNEL_EXCHANGE_P);
    const auto& tl = phase ? c->plan.tilesXQ : c->plan.tilesXP;
    DevArgs a = c->args;
    if (c->plan.agg_first && phase == 0) {
      a.Porth = c->args.Ppre;                    // the raw factors are what gets quantised
      a.padded = 0;                              // Gram-Schmidt is still to come
    }
    HIP_TRY(c, launch_exchange(mode, phase, a, phase ? c->d_tilesXQ : c->d_tilesXP, (int)tl.size(), c->stream)); }
  if (c->plan.agg_first && phase == 0 && mode != kQuantOnly) return run_orth_shared(c);
  return LQSGD_OK;
}
int run_sweep1(lqsgd_ctx* c, bool with_vectors) {
  if (int rc = refresh_stale(c)) return rc;
  { Timed t(c, LQSGD_KERNEL_BACK_PROJECT);
    const int nv = with_vectors ? (int)c->plan.tilesV.size() : 0;
    if (c->plan.mfma)
      HIP_TRY(c, launch_back_project_mfma(c->plan.RP, c->args, c->d_tilesBM, (int)c->plan.tilesBM.size(), c->d_tilesV, nv,
                                          next_dir(c), c->stream));
    else
      HIP_TRY(c, launch_back_project(c->plan.RP, c->args, c->d_tilesB, (int)c->plan.tilesB.size(), c->d_tilesV, nv,
                                     next_dir(c), c->stream)); }
  if (!c->plan.tilesRQ.empty()) {      // layers whose sweep-1 items each cover all rows have stored Q_w themselves
    Timed t(c, LQSGD_KERNEL_REDUCE_Q);
    HIP_TRY(c, launch_reduce_q(1, c->args, c->d_tilesRQ, (int)c->plan.tilesRQ.size(), c->stream)); }
  return LQSGD_OK;
}
// End of an iteration: either apply E = M - P-bar Q-bar^T now (eager), or leave M
// in place and let the next iteration's first sweep apply it on the fly; G-hat,
// when asked for, is then written by a pass of its own over the layers.
int run_sweep2(lqsgd_ctx* c, bool write_ghat) {
  const Plan& p = c->plan;
  if (int rc = refresh_stale(c)) return rc;
  Timed t(c, LQSGD_KERNEL_RESIDUAL);
  if (c->eager) {
    if (p.mfma_a)
      HIP_TRY(c, launch_mfma_sweep(p.RP, write_ghat ? 3 : 2, c->args, c->d_tilesA, (int)p.tilesA.size(), p.twoA, next_dir(c), c->stream));
    else
      HIP_TRY(c, launch_residual(p.RP, write_ghat ? 1 : 0, c->args, c->d_tilesR, (int)p.tilesR.size(), p.narrow_rows ? 1 : 0, next_dir(c), c->stream));
  } else {
    if (write_ghat) {
      if (p.mfma_a)
        HIP_TRY(c, launch_mfma_sweep(p.RP, 4, c->args, c->d_tilesAG, (int)p.tilesAG.size(), 0, 0, c->stream));
      else
        HIP_TRY(c, launch_residual(p.RP, 2, c->args, c->d_tilesG, (int)p.tilesG.size(), 0, 0, c->stream));
    }
    c->pending = true;
  }
  return LQSGD_OK;
}
// Applies a deferred residual update, so that the buffer holds E again.
int materialise(lqsgd_ctx* c) {
  if (!c->pending) return LQSGD_OK;
  const Plan& p = c->plan;
  if (int rc = refresh_stale(c)) return rc;
  Timed t(c, LQSGD_KERNEL_RESIDUAL);
  if (p.mfma_a)
    HIP_TRY(c, launch_mfma_sweep(p.RP, 2, c->args, c->d_tilesA, (int)p.tilesA.size(), p.twoA, next_dir(c), c->stream));
  else
    HIP_TRY(c, launch_residual(p.RP, 0, c->args, c->d_tilesR, (int)p.tilesR.size(), p.narrow_rows ? 1 : 0, next_dir(c), c->stream));
  c->pending = false;
  return LQSGD_OK;
}

struct PacketLoc {
  uint8_t* mag; uint8_t* sgn; float* scale;
  int64_t n_el, groups, mag_len, sign_len;
  int bits;
};

int locate_packet(lqsgd_ctx* c, int32_t phase, int32_t layer, int32_t worker, PacketLoc* out) {
  if (phase != LQSGD_PHASE_P && phase != LQSGD_PHASE_Q) return fail(c, LQSGD_EINVAL, "phase must be LQSGD_PHASE_P or LQSGD_PHASE_Q");
  const LayerDesc* ld = nullptr;
  int rc = check_matrix_layer(c, layer, &ld);
  if (rc) return rc;
  if ((rc = check_worker(c, worker))) return rc;
  const int li = c->plan.kind_of[layer];
  const DevArgs& a = c->args;
  out->bits = phase ? a.bits_q : a.bits_p;
  if (out->bits == 0) return fail(c, LQSGD_EUNSUPPORTED, "quantisation is off for this phase: the packet is the fp32 factor");
  out->n_el = phase ? ld->nq_el : ld->np_el;
  out->groups = (out->n_el + kXGroup - 1) / kXGroup;
  out->mag_len = out->groups * out->bits;
  out->sign_len = out->groups;
  if (phase) {
    out->mag = a.magQ + (size_t)worker * a.magq_stride + ld->magq_off;
    out->sgn = a.sgnQ + (size_t)worker * a.sgnq_stride + ld->sgnq_off;
    out->scale = a.scaleQ + (size_t)worker * a.L + li;
  } else {
    out->mag = a.magP + (size_t)worker * a.magp_stride + ld->magp_off;
    out->sgn = a.sgnP + (size_t)worker * a.sgnp_stride + ld->sgnp_off;
    out->scale = a.scaleP + (size_t)worker * a.L + li;
  }
  return LQSGD_OK;
}

}  // namespace

// =============================================================================
extern "C" {

int lqsgd_plan_query(const lqsgd_config* cfg, const lqsgd_layer* layers, int32_t n_layers, lqsgd_plan_info* out) {
  if (!out) return fail(nullptr, LQSGD_EINVAL, "NULL output");
  Plan p;
  const int rc = p.build(cfg, layers, n_layers);
  if (rc) return fail(nullptr, rc, p.err);
  out->device_bytes = p.device_bytes;
  out->wire_bytes = p.wire_bytes;
  out->matrix_elements = p.matrix_elements;
  out->n_matrix = p.L;
  out->n_vector = p.V;
  out->rank_pad = p.RP;
  out->tiles[0] = (int32_t)p.tilesA.size();
  out->tiles[1] = (int32_t)(p.mfma ? p.tilesBM.size() : p.tilesB.size());
  out->tiles[2] = (int32_t)(p.mfma_a ? p.tilesA.size() : p.tilesR.size());
  out->residual_stride = p.m_stride;
  out->warm_q_floats = p.q_stride + kFactorSlack;
  return LQSGD_OK;
}

int64_t lqsgd_plan_tiles(const lqsgd_config* cfg, const lqsgd_layer* layers, int32_t n_layers, int32_t sweep,
                         int32_t* out, int64_t cap) {
  if (sweep < 0 || sweep > 3) return fail(nullptr, LQSGD_EINVAL, "sweep must be 0, 1, 2 or 3");
  Plan p;
  const int rc = p.build(cfg, layers, n_layers);
  if (rc) return fail(nullptr, rc, p.err);
  const bool bm = sweep == 1 && p.mfma;
  const bool as0 = sweep == 0 || (sweep >= 2 && p.mfma_a);     // items of sweep 0's kind
  const std::vector<Tile>& tl = sweep == 3 ? (p.mfma_a ? p.tilesAG : p.tilesG)
                                           : as0 ? p.tilesA : (bm ? p.tilesBM : sweep == 2 ? p.tilesR : p.tilesB);
  if (out) {
    const int64_t n = std::min<int64_t>(cap, (int64_t)tl.size());
    for (int64_t i = 0; i < n; ++i) {
      const Tile& t = tl[i];
      const int li = t.lw / p.W;
      const LayerDesc& d = p.layers[li];
      int32_t* o = out + 6 * i;
      o[0] = d.gidx;
      o[1] = t.lw - li * p.W;
      o[2] = t.row0;
      o[3] = t.nrows;
      if (as0) {
        const int w = sweep == 3 ? kGhatCols : d.segw;
        o[4] = t.aux * w;
        o[5] = std::min(d.cols, o[4] + w) - o[4];
      } else {
        const int cw = bm ? kMfmaCols : sweep == 1 ? d.bcw : kWave * 4;
        o[4] = t.aux * cw;
        o[5] = std::min(d.cols, o[4] + cw) - o[4];
      }
    }
  }
  return (int64_t)tl.size();
}

namespace {
// Fills c->args and uploads the tables of c->plan.  Device memory comes from hipMalloc or, when
// c->arena is set, from that block: then the residual slabs and the warm-start Q are not allocated
// (the caller's buffers are bound per call), and the one-launch Gram-Schmidt of tall factors, which
// needs a pinned status word and a table that starts from zero, is off (its forms of several launches run).
// On failure the caller releases c->allocs / c->status.
int setup_device(lqsgd_ctx* c, uint32_t flags) {
  int rc;
  const bool ext = c->arena != nullptr;
  c->eager = ext || (flags & LQSGD_FLAG_EAGER_RESIDUAL) != 0;
  HIP_TRY(c, hipGetDevice(&c->device));
  const Plan& p = c->plan;
  DevArgs& a = c->args;
  a.W = p.W; a.L = p.L; a.n_all = p.n_all; a.rank_pad = p.RP; a.slices = p.slices; a.bits_p = p.cfg.bits_p; a.bits_q = p.cfg.bits_q;
  a.alpha = p.cfg.alpha;
  a.agg_first = p.agg_first ? 1 : 0; a.orth_shared = 0; a.update = 0; a.eta = 0.0f;
  a.g_bf16 = (flags & LQSGD_FLAG_BF16_GRADIENTS) ? 1 : 0;
  // The residual / M slabs are read and written once per sweep.  While they are about the size of
  // the memory-side cache (256 MB), plain loads and stores in sweep 0 are faster (ResNet-18 set,
  // 357 MB: a step takes 276 us; 284 us with non-temporal loads of E, 295 us with non-temporal
  // stores as well).  Far beyond it, the dirty lines that plain stores leave in that cache are
  // written back underneath the following reads, and streaming both ways wins (8192^2 x 16,
  // 4.3 GB: sweep 0 2.27 -> 2.04 - 2.14 ms).  Measured crossover: 0.55 - 0.7 GB.
  {
    // Non-temporal stores do not wait for the rest of a line of 128 bytes: rows that start anywhere in a line leave two
    // partial ones per KiB, written apart.  So not where most elements are in rows that are no multiple of 64 bytes (W = 8,
    // a step with and without, us: 4 x (3000 x 5000) r = 4 1662 / 1592, r = 16 2084 / 1814, r = 50 2648 / 2527; 4 x (3001 x 5001)
    // r = 4 1759 / 1620, r = 20 2042 / 1954; rows of 64 bytes, 3000 x 5008, r = 4 1539 / 1549; of 128, 3000 x 4992 1440 / 1476).
    int64_t askew = 0;
    for (const LayerDesc& d : p.layers)
      if (d.cols % 16) askew += (int64_t)d.rows * d.cols;
    const int64_t slab_bytes = 4 * (int64_t)p.W * p.m_stride;
    const bool rows_whole = 2 * askew <= p.matrix_elements;
    a.nt_store = slab_bytes >= ((int64_t)640 << 20) && rows_whole ? 1 : 0;
    // Sweep 0 by rounds (rank pads 16 and 32) with the deferred residual and float32 gradients stores whole KiBs of rows and gains
    // from 310 MB on (a step plain / non-temporal, us, W = 8, r = 16 and r = 32: 8 x (512 x 2048), 268 MB 287 / 291 and 319 / 323;
    // 8 x (512 x 2304), 302 MB 302 / 304 and 347 / 343; 5 x (512 x 4096), 336 MB 326 / 318 and 366 / 358; ResNet-18 set, 357 MB
    // 332 / 326 and 402 / 389; 8 x (512 x 4096), 537 MB 465 / 426 and 587 / 576; 8 x (512 x 4608), 604 MB 523 / 501 and
    // 604 / 579).  First iterations and bfloat16 gradients do not: ResNet-18 set, first sweep 0 179 / 200, a step with bfloat16
    // gradients 282 / 296.
    a.nt_fused = a.nt_store || (p.mfma_a && p.RP <= 32 && !a.g_bf16 && rows_whole && slab_bytes >= ((int64_t)320 << 20)) ? 1 : 0;
    // Rank pad 16, deferred residual, float32 gradients, plain stores: whole 64-column blocks per wavefront instead of rounds where
    // rounds would be left half empty, or where the slabs are about the size of the memory-side cache, in which they leave sweep 1 less
    // of M (a step by rounds / by blocks, us, W = 8, r = 16: 16 x (512 x 320), 84 MB 147 / 140; 24 x (512 x 384), 151 MB 209 / 196;
    // 8 x (512 x 448), 59 MB 103 / 101; 64 x (512 x 64) 215 / 213; 16 x (512 x 576), 151 MB 198 / 190, but 8 of them 121 / 121;
    // 16 x (512 x 832), 218 MB 265 / 251, but 8 of them 152 / 153; 64 x (512 x 256), 268 MB 318 / 305; 16 x (512 x 384) beside 8 and
    // 12 x (512 x 1024) 280 / 266 and 320 / 315, 8 x (512 x 576) beside 14 of them 318 / 321).  Blocks that are cut off are the
    // rounds' (6 x (512 x 340) 90 / 95, 10 x (512 x 412) 122 / 129), and so are bfloat16 gradients (ResNet-18 set, r = 12 276 / 336).
    int64_t blocks = 0;
    for (const LayerDesc& d : p.layers) {
      const bool few = d.cols == 64 || (d.cols > 256 && d.cols <= 448), some = d.cols == 256 || (d.cols > 256 && d.cols % 256 != 0);
      if (d.cols % 64 == 0 && d.cols <= 1024 && (few || (some && slab_bytes >= ((int64_t)112 << 20)))) blocks += (int64_t)d.rows * d.cols;
    }
    a.by_blocks = p.RP == 16 && !a.g_bf16 && !a.nt_fused && 4 * blocks >= p.matrix_elements ? 1 : 0;
    // Lists that have a CU an item take as long as their longest item (figures also at mfma_sweep32_kernel; a step and a first
    // iteration's sweep 0, W = 4, by rounds / by blocks).
    if (p.tilesA.size() <= 256 && p.RP <= 32 && !a.nt_fused) {
      bool half = false, whole = false, low = false, wide = false, segments = false;
      for (const LayerDesc& d : p.layers) {
        const int last = d.cols > 256 ? d.cols % 256 : 0;
        half = half || (last > 0 && last <= 128);
        whole = whole || (last > 0 && last <= 128 && last % 64 == 0);
        low = low || (d.cols > 768 && d.rows % 32 != 0);
        wide = wide || d.cols > 192;
        segments = segments || d.cols >= 1024;
      }
      // Rank pad 32, 32 x 32 blocks per wavefront: always without a deferred residual (1).  With it, too (2), where rounds would
      // be cut short: items of fewer than 32 rows and many columns, last rounds at most half full unless some layer has longer
      // rows than that (4 x (256 x 1088) 87.5 / 88.9, 4 x (256 x 320) beside 2 x (256 x 1024) 86.5 / 89.3), one narrow round.  (More
      // items, r = 32, W = 8, sweep 0: 512, 8 x (256 x 1024) 43 / 51, in a first iteration 43 / 43; 384, 24 x (40 x 1024) 37 / 44 and
      // 35 / 35.)
      if (p.RP == 32) a.by_blocks = low || !wide || (half && !segments) ? 2 : 1;
      // Rank pad 16, 64-column blocks: also without a deferred residual (2) where last rounds are at most half full (4 x (256 x 576)
      // 64.7 / 63.1 and 15.9 / 14.7, 4 x (128 x 576) 54.3 / 52.5 and 14.9 / 13.3, 4 x (256 x 640) 63.4 / 62.6 and 16.4 / 15.1; longer rows
      // 4 x (256 x 1088) 63.9 / 66.6, 4 x (256 x 1920) 72.9 / 74.9).
      if (p.RP == 16 && !a.g_bf16 && whole && !segments) a.by_blocks = 2;
    }
    // Rank pad 32, lists of any length, first iterations only: rows of a whole round and at most a quarter more that start on lines
    // of 128 bytes (sweep 0, W = 8, 16 x (512 x 288) 66 / 60, 24 x (512 x 320) 96 / 92; but 16 x (512 x 304) 68 / 74, 16 x (512 x 384)
    // 71 / 72, 8 x (512 x 576) 52 / 53).
    if (p.RP == 32 && !a.g_bf16 && !a.nt_store && !a.by_blocks) {
      int64_t quarter = 0;
      for (const LayerDesc& d : p.layers)
        if (d.cols > 256 && d.cols <= 320 && d.cols % 32 == 0) quarter += (int64_t)d.rows * d.cols;
      if (2 * quarter >= p.matrix_elements) a.by_blocks = 1;
    }
#ifdef LQSGD_TUNING     // a tuning build can force the choice and switch the alternating sweep direction off
    if (const char* f = std::getenv("LQSGD_BY_BLOCKS"))
      a.by_blocks = (p.RP == 16 && !a.g_bf16) || p.RP == 32 ? (a.nt_store ? 0 : f[0] - '0') : 0;
    if (const char* f = std::getenv("LQSGD_NT_STORE")) {
      if (f[0] == '1') a.nt_store = a.nt_fused = 1;
      if (f[0] == '2') a.nt_store = a.nt_fused = 0;
    }
    if (const char* f = std::getenv("LQSGD_FLIP")) c->flip = (f[0] != '0');
#endif
  }
  // The estimate of a code is off by the rounding of 1 + alpha u and of log2 (about 2e-7 together, near 1) times qscale:
  // below 0.01 levels from alpha = 1/16 up.  Up to 2^40 the first threshold lies above 2^-47, far from where the
  // quotient's remainder could underflow.  Outside, the quantiser divides and walks.
  a.quant_fast = p.cfg.alpha >= 0.0625f && p.cfg.alpha <= 0x1p40f ? 1 : 0;
  a.qscale_p = (float)(((1 << p.cfg.bits_p) - 1) / std::log2(1.0 + (double)p.cfg.alpha));
  a.qscale_q = (float)(((1 << p.cfg.bits_q) - 1) / std::log2(1.0 + (double)p.cfg.alpha));
  a.m_stride = p.m_stride; a.p_stride = p.p_stride; a.q_stride = p.q_stride;
  a.ppart_stride = p.ppart_stride; a.qpart_stride = p.qpart_stride;
  a.magp_stride = p.magp_stride; a.sgnp_stride = p.sgnp_stride;
  a.magq_stride = p.magq_stride; a.sgnq_stride = p.sgnq_stride;
  const size_t W = (size_t)p.W;
  LayerDesc* d_layers = nullptr; VecDesc* d_vecs = nullptr;
  float *thrP = nullptr, *levP = nullptr, *thrQ = nullptr, *levQ = nullptr;
  std::vector<float> tP, lP, tQ, lQ;
  quantiser_tables(p.cfg.bits_p, (double)p.cfg.alpha, tP, lP);
  quantiser_tables(p.cfg.bits_q, (double)p.cfg.alpha, tQ, lQ);
#define TRY_(x) do { if ((rc = (x))) return rc; } while (0)
  // Loaders fetch whole padded rows, and four of them at a time, and may run up to 63 floats past the last
  // row of a factor: every factor buffer ends with this much readable slack.
  constexpr size_t kSlack = kFactorSlack;
  const size_t orth_cells = 2 * W * (size_t)std::max(p.L, 1) * ((p.max_rows + 255) / 256) * p.RP;
  a.E = nullptr; a.Qbar = nullptr; a.orth_table = nullptr; a.status = nullptr;
  a.chol_table = nullptr; a.chol_part = nullptr; a.chol_part2 = nullptr; a.chol_redo = nullptr;
  if (!ext) TRY_(dev_alloc(c, &a.E, W * p.m_stride, true));
  TRY_(dev_alloc(c, &a.Ppart, W * p.ppart_stride + kSlack, true));
  TRY_(dev_alloc(c, &a.Ppre, W * p.p_stride + kSlack, true));
  TRY_(dev_alloc(c, &a.Porth, W * p.p_stride + kSlack, true));
  TRY_(dev_alloc(c, &a.orth_part, orth_cells, true));
  // Tall factors at rank pads >= 8 exchange whole Gram matrices instead of single columns (launch_orth decides per call).
  // A caller-provided block and factors of more than 64 slices get the buffers of the form of three launches only, which
  // gives the same bits.
  const size_t nslice = (size_t)(p.max_rows + 255) / 256, pairs = W * (size_t)std::max(p.L, 1);
  const size_t ne = (size_t)chol_entries(p.RP);
  // (table and first-pass matrices; a limit on the second-pass ones as well would give sets near it another method)
  const bool chol_size = ne && pairs * (nslice + 1) * ne * 12 <= ((size_t)1 << 30);
  if (chol_size && nslice >= 8) {
    TRY_(dev_alloc(c, &a.chol_part, pairs * nslice * ne, true));
    TRY_(dev_alloc(c, &a.chol_redo, pairs, true));
  }
  if (!ext) {
    TRY_(dev_alloc(c, &a.orth_table, orth_cells, true));
    void* hp = nullptr;
    hipError_t e = hipHostMalloc(&hp, 256 + kBounceBytes, hipHostMallocDefault);      // status word, memory for fetch()
    if (e != hipSuccess) { fail_hip(c, e, "hipHostMalloc"); return LQSGD_ENOMEM; }
    c->status = static_cast<int*>(hp);
    c->bounce = static_cast<char*>(hp) + 256;
    *c->status = 0;
    a.status = c->status;
  }
  TRY_(dev_alloc(c, &a.Pbar, (size_t)p.p_stride + kSlack, true));
  TRY_(dev_alloc(c, &a.Qpart, W * p.qpart_stride + kSlack, true));
  // Rank pad 64 leaves the one-workgroup form at 1024 rows already.  From there to 8 slices the Gram matrices lie where
  // sweep 1 will put its partial planes, which are dead while Gram-Schmidt runs, or, in a set whose planes are too small
  // for them, the columns are exchanged one by one: the same choice with and without a caller-provided block, whose sizes
  // this leaves alone (it is another method with other rounding: 2 x (1700 x 640), W = 4, 160 us against 8.6 ms in memory).
  if (chol_size && p.RP == 64 && p.max_rows > 1024 && nslice < 8 && pairs * (nslice * ne + 1) <= W * (size_t)p.qpart_stride) {
    a.chol_part = a.Qpart;
    a.chol_redo = reinterpret_cast<int*>(a.Qpart + pairs * nslice * ne);
  }
  if (a.chol_part && ext) a.chol_part2 = c->grams;
  if (a.chol_part && !ext) TRY_(dev_alloc(c, &a.chol_part2, pairs * nslice * ne, true));
  if (!ext && a.chol_part && nslice <= 64) TRY_(dev_alloc(c, &a.chol_table, pairs * (nslice + 1) * ne, true));   // the one-launch form's limit
  TRY_(dev_alloc(c, &a.Qw, W * p.q_stride + kSlack, true));
  if (!ext) TRY_(dev_alloc(c, &a.Qbar, (size_t)p.q_stride + kSlack, true));
  a.padded = p.padded ? 1 : 0;
  a.Pop = a.Pbar; a.Qop = a.Qbar;
  if (p.padded && !ext) {
    TRY_(dev_alloc(c, &a.Pop, (size_t)p.ppad_total + kSlack, true));
    TRY_(dev_alloc(c, &a.Qop, (size_t)p.qpad_total + kSlack, true));
  }
  TRY_(dev_alloc(c, &a.magP, W * p.magp_stride, true));
  TRY_(dev_alloc(c, &a.sgnP, W * p.sgnp_stride, true));
  TRY_(dev_alloc(c, &a.scaleP, W * (size_t)std::max(p.L, 1), true));
  TRY_(dev_alloc(c, &a.magQ, W * p.magq_stride, true));
  TRY_(dev_alloc(c, &a.sgnQ, W * p.sgnq_stride, true));
  TRY_(dev_alloc(c, &a.scaleQ, W * (size_t)std::max(p.L, 1), true));
  TRY_(dev_alloc(c, &a.vmean, (size_t)p.v_total, true));
  TRY_(dev_alloc(c, &c->d_grads, W * p.n_all, true));
  TRY_(dev_alloc(c, &c->d_ghat, (size_t)p.n_all, true));
  // In a caller-provided block everything above is cleared here, by a kernel, before the tables
  // below are copied in (the block keeps whatever its last user left).
  if (ext) HIP_TRY(c, launch_fill_zero(c->arena, c->arena_used, c->stream));
  if (ext) HIP_TRY(c, hipStreamSynchronize(c->stream));
  TRY_(dev_upload(c, &d_layers, p.layers));
  TRY_(dev_upload(c, &d_vecs, p.vecs));
  TRY_(dev_upload(c, &thrP, tP)); TRY_(dev_upload(c, &levP, lP));
  TRY_(dev_upload(c, &thrQ, tQ)); TRY_(dev_upload(c, &levQ, lQ));
  TRY_(dev_upload(c, &c->d_tilesA, p.tilesA));
  TRY_(dev_upload(c, &c->d_tilesB, p.tilesB));
  TRY_(dev_upload(c, &c->d_tilesBM, p.tilesBM));
  if (!ext) {                                    // (G-hat passes of deferred residuals)
    TRY_(dev_upload(c, &c->d_tilesG, p.tilesG));
    TRY_(dev_upload(c, &c->d_tilesAG, p.tilesAG));
  }
  TRY_(dev_upload(c, &c->d_tilesXP, p.tilesXP));
  TRY_(dev_upload(c, &c->d_tilesXQ, p.tilesXQ));
  TRY_(dev_upload(c, &c->d_tilesRQ, p.tilesRQ));
  TRY_(dev_upload(c, &c->d_tilesRP, p.tilesRP));
  TRY_(dev_upload(c, &c->d_tilesV, p.tilesV));
  // The padded copies of a caller-held state and the residual sweep's own items, which came after the block's size, go to the
  // second block where the first has no room left.
  auto late = [&](void** out, size_t bytes) {
    bytes = (size_t)round_up((int64_t)bytes, 256);
    if (bytes <= c->arena_cap - c->arena_used) {
      *out = c->arena + c->arena_used;
      c->arena_used += bytes;
    } else if (bytes <= c->operands_cap - c->operands_used) {
      *out = c->operands + c->operands_used;
      c->operands_used += bytes;
    } else {
      char buf[200];
      std::snprintf(buf, sizeof buf, "this configuration needs more scratch memory than the static buffers hold (%zu bytes of operand copies or items)", bytes);
      return fail(c, LQSGD_EUNSUPPORTED, buf);
    }
    return (int)LQSGD_OK;
  };
  if (p.padded && ext) {
    const size_t pb = (size_t)round_up(4 * (p.ppad_total + kFactorSlack), 256), qb = (size_t)round_up(4 * (p.qpad_total + kFactorSlack), 256);
    void* at = nullptr;
    TRY_(late(&at, pb + qb));
    a.Pop = static_cast<float*>(at);
    a.Qop = a.Pop + pb / 4;
    HIP_TRY(c, launch_fill_zero(at, pb + qb, c->stream));
  }
  if (!p.mfma_a && !ext) TRY_(dev_upload(c, &c->d_tilesR, p.tilesR));
  if (!p.mfma_a && ext && !p.tilesR.empty()) {
    void* at = nullptr;
    TRY_(late(&at, p.tilesR.size() * sizeof(Tile)));
    c->d_tilesR = static_cast<Tile*>(at);
    HIP_TRY(c, hipMemcpy(at, p.tilesR.data(), p.tilesR.size() * sizeof(Tile), hipMemcpyHostToDevice));
  }
#undef TRY_
  a.layers = d_layers; a.vecs = d_vecs;
  a.thrP = thrP; a.levP = levP; a.thrQ = thrQ; a.levQ = levQ;
  a.grads = c->d_grads; a.ghat = nullptr;
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  return LQSGD_OK;
}
}  // namespace

int lqsgd_create(const lqsgd_config* cfg, const lqsgd_layer* layers, int32_t n_layers, void* hip_stream,
                 lqsgd_ctx** out) {
  if (!out) return fail(nullptr, LQSGD_EINVAL, "NULL output pointer");
  *out = nullptr;
  lqsgd_ctx* c = new (std::nothrow) lqsgd_ctx();
  if (!c) return fail(nullptr, LQSGD_ENOMEM, "out of host memory");
  int rc = c->plan.build(cfg, layers, n_layers);
  if (rc) {
    g_create_error = c->plan.err;
    delete c;
    return rc;
  }
  c->stream = static_cast<hipStream_t>(hip_stream);
  // The bound of the device-side waits of the one-launch Gram-Schmidt can be shortened for a test
  // of the expiry path (read once, here; nothing else in the library reads the environment).  Tall factors at rank
  // pads 1 to 4 then take the form that waits, with the same bits (launch_orth).
  if (const char* e = std::getenv("LQSGD_TABLE_POLLS")) {
    const long v = std::strtol(e, nullptr, 10);
    if (v >= 1) c->coop.max_polls = (unsigned)v;
  }
  if ((rc = setup_device(c, cfg->flags))) {
    g_create_error = c->err;
    for (void* p : c->allocs) (void)hipFree(p);
    if (c->status) (void)hipHostFree(c->status);
    delete c;
    return rc;
  }
  *out = c;
  return LQSGD_OK;
}

int lqsgd_destroy(lqsgd_ctx* c) {
  if (!c) return LQSGD_OK;
  (void)hipStreamSynchronize(c->stream);
  for (EventPair& e : c->events) { (void)hipEventDestroy(e.a); (void)hipEventDestroy(e.b); }
  for (void* p : c->allocs) (void)hipFree(p);
  if (c->status) (void)hipHostFree(c->status);
  (void)hipGetLastError();
  delete c;
  return LQSGD_OK;
}

int lqsgd_synchronize(lqsgd_ctx* c) {
  if (!c) return fail(nullptr, LQSGD_EINVAL, "NULL context");
  if (int rcs = sync_stream(c)) return rcs;
  return LQSGD_OK;
}

const char* lqsgd_last_error(const lqsgd_ctx* c) { return c ? c->err.c_str() : g_create_error.c_str(); }

int lqsgd_set_q(lqsgd_ctx* c, int32_t layer, const float* host_q) {
  if (!c) return fail(nullptr, LQSGD_EINVAL, "NULL context");
  if (!host_q) return fail(c, LQSGD_EINVAL, "NULL host_q");
  return lqsgd_set_state(c, layer, 0, nullptr, host_q);
}

int lqsgd_get_state(lqsgd_ctx* c, int32_t layer, int32_t worker, float* host_e, float* host_q) {
  if (!c) return fail(nullptr, LQSGD_EINVAL, "NULL context");
  const LayerDesc* ld = nullptr;
  int rc = check_matrix_layer(c, layer, &ld);
  if (rc) return rc;
  if ((rc = check_worker(c, worker))) return rc;
  if (host_e && (rc = materialise(c))) return rc;
  if (int rcs = sync_stream(c)) return rcs;
  if (host_e)
    HIP_TRY(c, hipMemcpy(host_e, c->args.E + (size_t)worker * c->args.m_stride + ld->m_off,
                         (size_t)ld->rows * ld->cols * sizeof(float), hipMemcpyDeviceToHost));
  if (host_q)
    HIP_TRY(c, hipMemcpy(host_q, c->args.Qbar + ld->q_off, (size_t)ld->nq_el * sizeof(float), hipMemcpyDeviceToHost));
  return LQSGD_OK;
}

int lqsgd_set_state(lqsgd_ctx* c, int32_t layer, int32_t worker, const float* host_e, const float* host_q) {
  if (!c) return fail(nullptr, LQSGD_EINVAL, "NULL context");
  const LayerDesc* ld = nullptr;
  int rc = check_matrix_layer(c, layer, &ld);
  if (rc) return rc;
  if ((rc = check_worker(c, worker))) return rc;
  if ((rc = materialise(c))) return rc;      // a deferred update depends on the old E buffer and the old Q
  if (int rcs = sync_stream(c)) return rcs;
  if (host_e)
    HIP_TRY(c, hipMemcpy(c->args.E + (size_t)worker * c->args.m_stride + ld->m_off, host_e,
                         (size_t)ld->rows * ld->cols * sizeof(float), hipMemcpyHostToDevice));
  if (host_q) {
    HIP_TRY(c, hipMemcpy(c->args.Qbar + ld->q_off, host_q, (size_t)ld->nq_el * sizeof(float), hipMemcpyHostToDevice));
    c->stale[1] = c->plan.padded;
  }
  return LQSGD_OK;
}

int lqsgd_compress(lqsgd_ctx* c, int32_t phase, const float* const* grads) {
  if (!c) return fail(nullptr, LQSGD_EINVAL, "NULL context");
  int rc;
  if (phase == LQSGD_PHASE_P) {
    if (c->state != kIdle) return fail(c, LQSGD_ESTATE, "compress(P) must start an iteration");
    if (!grads) return fail(c, LQSGD_EINVAL, "NULL gradient list");
    if ((rc = bind_grads(c, grads))) return rc;
    if ((rc = run_sweep0(c))) return rc;
    if ((rc = run_exchange(c, kQuantOnly, 0))) return rc;
    c->state = kPCompressed;
    return LQSGD_OK;
  }
  if (phase == LQSGD_PHASE_Q) {
    if (c->state != kPDone) return fail(c, LQSGD_ESTATE, "compress(Q) must follow decompress(P)");
    if ((rc = run_sweep1(c, false))) return rc;
    if ((rc = run_exchange(c, kQuantOnly, 1))) return rc;
    c->state = kQCompressed;
    return LQSGD_OK;
  }
  return fail(c, LQSGD_EINVAL, "phase must be LQSGD_PHASE_P or LQSGD_PHASE_Q");
}

int lqsgd_decompress(lqsgd_ctx* c, int32_t phase) {
  if (!c) return fail(nullptr, LQSGD_EINVAL, "NULL context");
  int rc;
  if (phase == LQSGD_PHASE_P) {
    if (c->state != kPCompressed) return fail(c, LQSGD_ESTATE, "decompress(P) must follow compress(P)");
    if ((rc = run_exchange(c, kMeanOnly, 0))) return rc;
    c->state = kPDone;
    return LQSGD_OK;
  }
  if (phase == LQSGD_PHASE_Q) {
    if (c->state != kQCompressed) return fail(c, LQSGD_ESTATE, "decompress(Q) must follow compress(Q)");
    if ((rc = run_exchange(c, kMeanOnly, 1))) return rc;
    c->args.ghat = nullptr;
    if ((rc = run_sweep2(c, false))) return rc;
    c->state = kIdle;
    return LQSGD_OK;
  }
  return fail(c, LQSGD_EINVAL, "phase must be LQSGD_PHASE_P or LQSGD_PHASE_Q");
}

namespace {
int step_impl(lqsgd_ctx* c, const float* const* grads, float* const* ghat);
}

int lqsgd_step(lqsgd_ctx* c, const float* const* grads, float* const* ghat) {
  if (!c) return fail(nullptr, LQSGD_EINVAL, "NULL context");
  return step_impl(c, grads, ghat);
}

int lqsgd_step_update(lqsgd_ctx* c, const float* const* grads, float* const* params, float eta) {
  if (!c) return fail(nullptr, LQSGD_EINVAL, "NULL context");
  if (!params) return fail(c, LQSGD_EINVAL, "NULL parameter list");
  if (!std::isfinite(eta)) return fail(c, LQSGD_EINVAL, "eta must be finite");
  c->args.update = 1;
  c->args.eta = eta;
  const int rc = step_impl(c, grads, params);
  c->args.update = 0;
  c->args.eta = 0.0f;
  return rc;
}

namespace {
int step_impl(lqsgd_ctx* c, const float* const* grads, float* const* ghat) {
  if (c->state != kIdle) return fail(c, LQSGD_ESTATE, "a staged iteration is in progress");
  if (!grads) return fail(c, LQSGD_EINVAL, "NULL gradient list");
  int rc;
  if ((rc = bind_grads(c, grads))) return rc;
  if ((rc = bind_ghat(c, ghat))) return rc;
  if (ghat && !c->alias_checked) {   // both tables are the host copies just compared equal or re-bound
    const size_t n = (size_t)c->plan.W * c->plan.n_all;
    for (int i = 0; i < c->plan.n_all; ++i)
      if (ghat[i])
        for (size_t j = 0; j < n; ++j)
          if (grads[j] == ghat[i]) return fail(c, LQSGD_EINVAL, "an output pointer aliases a gradient");
    c->alias_checked = true;
  }
  if ((rc = run_sweep0(c))) return rc;
  if ((rc = run_exchange(c, kFused, 0))) return rc;
  if ((rc = run_sweep1(c, true))) return rc;
  if ((rc = run_exchange(c, kFused, 1))) return rc;
  if ((rc = run_sweep2(c, ghat != nullptr))) return rc;
  return LQSGD_OK;
}
}  // namespace

int lqsgd_get_packet_raw(lqsgd_ctx* c, int32_t phase, int32_t layer, int32_t worker, uint8_t* mag_plane,
                         int64_t* mag_len, uint8_t* sign_plane, int64_t* sign_len) {
  if (!c) return fail(nullptr, LQSGD_EINVAL, "NULL context");
  PacketLoc loc{};
  int rc = locate_packet(c, phase, layer, worker, &loc);
  if (rc) return rc;
  if (mag_len) *mag_len = loc.mag_len;
  if (sign_len) *sign_len = loc.sign_len;
  if (!mag_plane && !sign_plane) return LQSGD_OK;
  if (int rcs = sync_stream(c)) return rcs;
  if (mag_plane) HIP_TRY(c, hipMemcpy(mag_plane, loc.mag, (size_t)loc.mag_len, hipMemcpyDeviceToHost));
  if (sign_plane) HIP_TRY(c, hipMemcpy(sign_plane, loc.sgn, (size_t)loc.sign_len, hipMemcpyDeviceToHost));
  return LQSGD_OK;
}

int lqsgd_packet_device(lqsgd_ctx* c, int32_t phase, int32_t layer, int32_t worker, uint8_t** mag_plane,
                        int64_t* mag_len, uint8_t** sign_plane, int64_t* sign_len, float** scale) {
  if (!c) return fail(nullptr, LQSGD_EINVAL, "NULL context");
  PacketLoc loc{};
  int rc = locate_packet(c, phase, layer, worker, &loc);
  if (rc) return rc;
  if (mag_plane) *mag_plane = loc.mag;
  if (mag_len) *mag_len = loc.mag_len;
  if (sign_plane) *sign_plane = loc.sgn;
  if (sign_len) *sign_len = loc.sign_len;
  if (scale) *scale = loc.scale;
  return LQSGD_OK;
}

int lqsgd_get_packet(lqsgd_ctx* c, int32_t phase, int32_t layer, int32_t worker, uint8_t* mag_codes,
                     uint8_t* sign_bits, float* scale) {
  if (!c) return fail(nullptr, LQSGD_EINVAL, "NULL context");
  PacketLoc loc{};
  int rc = locate_packet(c, phase, layer, worker, &loc);
  if (rc) return rc;
  if (int rcs = sync_stream(c)) return rcs;
  if (scale) HIP_TRY(c, hipMemcpy(scale, loc.scale, sizeof(float), hipMemcpyDeviceToHost));
  if (mag_codes) {
    std::vector<uint8_t> raw((size_t)loc.mag_len);
    HIP_TRY(c, hipMemcpy(raw.data(), loc.mag, raw.size(), hipMemcpyDeviceToHost));
    const unsigned mask = (1u << loc.bits) - 1u;
    for (int64_t e = 0; e < loc.n_el; ++e) {
      const int64_t bit = e * loc.bits;
      unsigned v = raw[(size_t)(bit >> 3)] >> (bit & 7);
      if ((bit & 7) + loc.bits > 8) v |= (unsigned)raw[(size_t)(bit >> 3) + 1] << (8 - (bit & 7));
      mag_codes[e] = (uint8_t)(v & mask);
    }
  }
  if (sign_bits) {
    std::vector<uint8_t> raw((size_t)loc.sign_len);
    HIP_TRY(c, hipMemcpy(raw.data(), loc.sgn, raw.size(), hipMemcpyDeviceToHost));
    for (int64_t e = 0; e < loc.n_el; ++e) sign_bits[e] = (raw[(size_t)(e >> 3)] >> (e & 7)) & 1u;
  }
  return LQSGD_OK;
}

int lqsgd_set_packet(lqsgd_ctx* c, int32_t phase, int32_t layer, int32_t worker, const uint8_t* mag_codes,
                     const uint8_t* sign_bits, float scale) {
  if (!c) return fail(nullptr, LQSGD_EINVAL, "NULL context");
  if (!mag_codes || !sign_bits) return fail(c, LQSGD_EINVAL, "NULL code array");
  PacketLoc loc{};
  int rc = locate_packet(c, phase, layer, worker, &loc);
  if (rc) return rc;
  const unsigned mask = (1u << loc.bits) - 1u;
  std::vector<uint8_t> mag((size_t)loc.mag_len, 0), sgn((size_t)loc.sign_len, 0);
  for (int64_t e = 0; e < loc.n_el; ++e) {
    if (mag_codes[e] > mask) return fail(c, LQSGD_EINVAL, "magnitude code exceeds 2^b - 1");
    const int64_t bit = e * loc.bits;
    const unsigned v = (unsigned)mag_codes[e] << (bit & 7);
    mag[(size_t)(bit >> 3)] |= (uint8_t)v;
    if ((bit & 7) + loc.bits > 8) mag[(size_t)(bit >> 3) + 1] |= (uint8_t)(v >> 8);
    if (sign_bits[e] & 1u) sgn[(size_t)(e >> 3)] |= (uint8_t)(1u << (e & 7));
  }
  if (int rcs = sync_stream(c)) return rcs;
  HIP_TRY(c, hipMemcpy(loc.mag, mag.data(), mag.size(), hipMemcpyHostToDevice));
  HIP_TRY(c, hipMemcpy(loc.sgn, sgn.data(), sgn.size(), hipMemcpyHostToDevice));
  HIP_TRY(c, hipMemcpy(loc.scale, &scale, sizeof(float), hipMemcpyHostToDevice));
  return LQSGD_OK;
}

int lqsgd_get_factor(lqsgd_ctx* c, int32_t which, int32_t layer, int32_t worker, float* host) {
  if (!c) return fail(nullptr, LQSGD_EINVAL, "NULL context");
  if (!host) return fail(c, LQSGD_EINVAL, "NULL host buffer");
  const DevArgs& a = c->args;
  if (which == LQSGD_FACTOR_VMEAN) {
    if (layer < 0 || layer >= c->plan.n_all) return fail(c, LQSGD_ESHAPE, "layer index out of range");
    const int k = c->plan.kind_of[layer];
    if (k >= 0) return fail(c, LQSGD_ESHAPE, "layer is not a VECTOR layer");
    const VecDesc& vd = c->plan.vecs[-k - 1];
    return fetch(c, host, a.vmean + vd.off, (size_t)vd.len * sizeof(float));
  }
  const LayerDesc* ld = nullptr;
  int rc = check_matrix_layer(c, layer, &ld);
  if (rc) return rc;
  const float* src = nullptr;
  size_t n = 0;
  const bool per_worker = which == LQSGD_FACTOR_P_PRE || which == LQSGD_FACTOR_P_ORTH || which == LQSGD_FACTOR_Q_W;
  if (per_worker && (rc = check_worker(c, worker))) return rc;
  if (which == LQSGD_FACTOR_P_ORTH && c->plan.agg_first)
    return fail(c, LQSGD_EINVAL, "no per-worker Gram-Schmidt output in the aggregate-first order");
  if (which == LQSGD_FACTOR_P_MEAN && !c->plan.agg_first)
    return fail(c, LQSGD_EINVAL, "LQSGD_FACTOR_P_MEAN exists in the aggregate-first order only");
  switch (which) {
    case LQSGD_FACTOR_P_MEAN: src = a.Porth + ld->p_off; n = ld->np_el; break;
    case LQSGD_FACTOR_P_PRE: src = a.Ppre + (size_t)worker * a.p_stride + ld->p_off; n = ld->np_el; break;
    case LQSGD_FACTOR_P_ORTH: src = a.Porth + (size_t)worker * a.p_stride + ld->p_off; n = ld->np_el; break;
    case LQSGD_FACTOR_P_BAR: src = a.Pbar + ld->p_off; n = ld->np_el; break;
    case LQSGD_FACTOR_Q_W: src = a.Qw + (size_t)worker * a.q_stride + ld->q_off; n = ld->nq_el; break;
    case LQSGD_FACTOR_Q_BAR: src = a.Qbar + ld->q_off; n = ld->nq_el; break;
    default: return fail(c, LQSGD_EINVAL, "unknown factor id");
  }
  return fetch(c, host, src, n * sizeof(float));
}

int lqsgd_set_factor(lqsgd_ctx* c, int32_t which, int32_t layer, const float* host) {
  if (!c) return fail(nullptr, LQSGD_EINVAL, "NULL context");
  if (!host) return fail(c, LQSGD_EINVAL, "NULL host buffer");
  const LayerDesc* ld = nullptr;
  int rc = check_matrix_layer(c, layer, &ld);
  if (rc) return rc;
  float* dst = nullptr;
  size_t n = 0;
  if (which == LQSGD_FACTOR_P_BAR) { dst = c->args.Pbar + ld->p_off; n = ld->np_el; }
  else if (which == LQSGD_FACTOR_Q_BAR) { dst = c->args.Qbar + ld->q_off; n = ld->nq_el; }
  else return fail(c, LQSGD_EINVAL, "only P-bar and Q-bar can be set");
  if ((rc = materialise(c))) return rc;      // a deferred update is defined by the old factors
  if (int rcs = sync_stream(c)) return rcs;
  HIP_TRY(c, hipMemcpy(dst, host, n * sizeof(float), hipMemcpyHostToDevice));
  c->stale[which == LQSGD_FACTOR_P_BAR ? 0 : 1] = c->plan.padded;
  return LQSGD_OK;
}

int64_t lqsgd_wire_bytes(const lqsgd_ctx* c) { return c ? c->plan.wire_bytes : (int64_t)LQSGD_EINVAL; }

int lqsgd_timing_enable(lqsgd_ctx* c, int32_t on) {
  if (!c) return fail(nullptr, LQSGD_EINVAL, "NULL context");
  if (int rcs = sync_stream(c)) return rcs;
  c->timing = on != 0;
  c->events_used = 0;
  return LQSGD_OK;
}

int lqsgd_timing_read(lqsgd_ctx* c, double* total_ms, int64_t* launches) {
  if (!c) return fail(nullptr, LQSGD_EINVAL, "NULL context");
  if (!total_ms || !launches) return fail(c, LQSGD_EINVAL, "NULL output array");
  if (int rcs = sync_stream(c)) return rcs;
  for (int k = 0; k < LQSGD_KERNEL_COUNT; ++k) { total_ms[k] = 0.0; launches[k] = 0; }
  for (size_t i = 0; i < c->events_used; ++i) {
    float ms = 0.0f;
    HIP_TRY(c, hipEventElapsedTime(&ms, c->events[i].a, c->events[i].b));
    total_ms[c->events[i].kernel] += ms;
    launches[c->events[i].kernel] += 1;
  }
  return LQSGD_OK;
}

const char* lqsgd_launched_kernel(const lqsgd_ctx* c, int32_t kernel) {
  if (!c || kernel < 0 || kernel >= LQSGD_KERNEL_COUNT) return "";
  return c->launched[kernel].c_str();
}

const char* lqsgd_kernel_name(int32_t kernel) {
  switch (kernel) {
    case LQSGD_KERNEL_ADD_PROJECT: return "sweep0_add_project";
    case LQSGD_KERNEL_ORTH: return "gram_schmidt";
    case LQSGD_KERNEL_EXCHANGE_P: return "exchange_p";
    case LQSGD_KERNEL_BACK_PROJECT: return "sweep1_back_project";
    case LQSGD_KERNEL_REDUCE_Q: return "reduce_q";
    case LQSGD_KERNEL_EXCHANGE_Q: return "exchange_q";
    case LQSGD_KERNEL_RESIDUAL: return "sweep2_residual_ghat";
    case LQSGD_KERNEL_REDUCE_P: return "reduce_p";
    default: return "";
  }
}

// ---- the entry point that allocates nothing ----------------------------------------------------
namespace {
// One slot per device: the host-side plan of the last configuration run there, whose device tables
// still lie in that device's static scratch block.
struct StaticSlot {
  lqsgd_ctx* ctx = nullptr;
  lqsgd_config cfg{};
  std::vector<lqsgd_layer> layers;
};
constexpr int kMaxDevices = 64;
StaticSlot g_static[kMaxDevices];
std::mutex g_static_mu;

bool same_config(const StaticSlot& s, const lqsgd_config* cfg, const lqsgd_layer* layers, int32_t n, hipStream_t stream) {
  if (!s.ctx || s.ctx->stream != stream || (int32_t)s.layers.size() != n) return false;
  if (s.cfg.rank != cfg->rank || s.cfg.bits_p != cfg->bits_p || s.cfg.bits_q != cfg->bits_q ||
      s.cfg.workers != cfg->workers || s.cfg.alpha != cfg->alpha || s.cfg.flags != cfg->flags)
    return false;
  for (int32_t i = 0; i < n; ++i)
    if (s.layers[i].rows != layers[i].rows || s.layers[i].cols != layers[i].cols || s.layers[i].flags != layers[i].flags)
      return false;
  return true;
}
}  // namespace

int lqsgd_step_static(const lqsgd_config* cfg, const lqsgd_layer* layers, int32_t n_layers, void* hip_stream,
                      const float* const* grads, float* residual, float* warm_q, float* const* ghat) {
  if (!cfg || !layers) return fail(nullptr, LQSGD_EINVAL, "NULL config or layer list");
  if (!grads) return fail(nullptr, LQSGD_EINVAL, "NULL gradient list");
  std::lock_guard<std::mutex> lock(g_static_mu);
  int dev = 0;
  {
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail_hip(nullptr, e, "hipGetDevice");
  }
  if (dev < 0 || dev >= kMaxDevices) return fail(nullptr, LQSGD_EUNSUPPORTED, "device index beyond the table of static scratch blocks");
  void *block = nullptr, *operands = nullptr, *grams = nullptr;
  {
    hipError_t e = static_scratch(dev, &block, &operands, &grams);
    if (e != hipSuccess) return fail_hip(nullptr, e, "hipGetSymbolAddress(scratch)");
  }
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  StaticSlot& slot = g_static[dev];
  if (!same_config(slot, cfg, layers, n_layers, stream)) {
    // A new configuration lays the block out anew: whatever the last one enqueued must have finished.
    if (slot.ctx) {
      (void)hipStreamSynchronize(slot.ctx->stream);
      (void)hipGetLastError();
      delete slot.ctx;
      slot.ctx = nullptr;
    }
    lqsgd_ctx* c = new (std::nothrow) lqsgd_ctx();
    if (!c) return fail(nullptr, LQSGD_ENOMEM, "out of host memory");
    int rc = c->plan.build(cfg, layers, n_layers);
    if (rc) {
      g_create_error = c->plan.err;
      delete c;
      return rc;
    }
    c->stream = stream;
    c->arena = static_cast<unsigned char*>(block);
    c->arena_cap = LQSGD_STATIC_SCRATCH_BYTES;
    c->operands = static_cast<unsigned char*>(operands);
    c->operands_cap = LQSGD_STATIC_OPERAND_BYTES;
    c->grams = static_cast<float*>(grams);
    if ((rc = setup_device(c, cfg->flags))) {
      g_create_error = c->err;
      delete c;
      return rc;
    }
    slot.ctx = c;
    slot.cfg = *cfg;
    slot.layers.assign(layers, layers + n_layers);
  }
  lqsgd_ctx* c = slot.ctx;
  const bool has_matrix = c->plan.L > 0;
  if (has_matrix && (!residual || !warm_q)) { g_create_error = "NULL residual or warm-start buffer"; return LQSGD_EINVAL; }
  if ((reinterpret_cast<uintptr_t>(residual) | reinterpret_cast<uintptr_t>(warm_q)) & 15u) {
    g_create_error = "residual / warm-start buffer not 16-byte aligned";
    return LQSGD_EINVAL;
  }
  c->args.E = residual;
  c->args.Qbar = warm_q;
  if (!c->plan.padded) c->args.Qop = warm_q;
  c->pending = false;                        // the caller's buffer holds E, and holds E again on return
  c->state = kIdle;
  int rc = refresh_padded(c, 1);             // the warm-start Q is the caller's
  if (!rc) rc = step_impl(c, grads, ghat);
  if (rc) g_create_error = c->err;
  return rc;
}

}  // extern "C"
