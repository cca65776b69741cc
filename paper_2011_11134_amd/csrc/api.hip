// api.hip -- the C ABI declared in include/dgal.h: argument validation on the
// host, then kernel dispatch on the caller's stream.  No allocation per call.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <new>
#include <string>
#include <vector>

#include "internal.hpp"

// A kind of call the autotuner tells apart: the entry point, register
// capacity K, fixed size, 3D, segmented (or saving, for the pair forward) and
// a size bucket (bit lengths of the counts).  Its text form, prefixed with
// the GPU architecture, keys the process-wide store and the cache file.  The
// number after a kind is raised whenever its kernels, or what a shape means to
// them, change: a choice measured on others is then not found again.
struct TuneKey {
  int kind, K, fixed, z3, seg;
  std::string bucket;
  std::string text(const std::string& arch) const {
    static const char* names[] = {"pairs_fwd.2", "pairs_bwd.2", "matrix_fwd.2",
                                  "matrix_bwd.2"};
    char b[160];
    snprintf(b, sizeof(b), "%s/%s/K%d/fixed%d/z%d/seg%d/b%s", arch.c_str(), names[kind], K, fixed,
             z3, seg, bucket.c_str());
    return b;
  }
};
enum { kTunePairsFwd, kTunePairsBwd, kTuneMatrixFwd, kTuneMatrixBwd };

struct dgal_ctx {
  dgal::CtxView v;
  dgal::Profiler prof;           // per-kernel timing (v.prof points here while on)
  bool tune = false;
  bool validate = false;         // check every input polygon before each call
  int64_t* n_bad = nullptr;      // device counter of the input check
  volatile int* err_host = nullptr;  // the device errors (v.err) as the host reads them
  unsigned long long* stats_dev = nullptr;  // path statistics (3 counters)
  std::string arch;              // e.g. "gfx950"
  std::map<std::string, dgal::LaunchShape> tuned;  // by TuneKey::text
};

namespace {

using dgal::aligned;
using dgal::DeviceGuard;
using dgal::poly_args;
using dgal::reg_k;
using dgal::valid_polys;

int status_of(hipError_t e) { return e == hipSuccess ? DGAL_OK : DGAL_EHIP; }

int bits_of(int64_t v) {
  int b = 0;
  while (v > 0) {
    ++b;
    v >>= 1;
  }
  return b;
}

std::string bucket_of(int64_t x, int64_t y = -1) {
  return y < 0 ? std::to_string(bits_of(x)) : std::to_string(bits_of(x)) + "." + std::to_string(bits_of(y));
}

// Sticky device errors: read (after the stream's work) and cleared; bit k of
// *out is word k.  Reading pinned host memory after one synchronisation takes
// 4 us where a copy of a device word took 22.
int read_err(dgal_ctx* ctx, hipStream_t stream, int* out) {
  if (hipStreamSynchronize(stream) != hipSuccess) return DGAL_EHIP;
  *out = 0;
  for (int k = 0; k < dgal::kErrWords; ++k) {
    if (ctx->err_host[k] == 0) continue;
    *out |= 1 << k;
    ctx->err_host[k] = 0;
  }
  return DGAL_OK;
}

// Whether no call of this context can have a tuned shape: then a call needs
// neither its key nor its candidates (1.5 us of the host's time).
bool untuned(const dgal_ctx* ctx) {
  return !ctx->tune && ctx->tuned.empty() && dgal::tune_store_empty();
}

// Runs launch(shape) with the shape tuned for `key`: the context's choice,
// else the process-wide store's (loaded from the cache file, or tuned by
// another context), else, while tuning is enabled, the fastest candidate.
// Every candidate is timed in two interleaved passes (each: one warm-up run,
// then three runs between HIP events on the caller's stream), keeping its
// faster pass; a candidate that raises the device error word (a table too
// small for its tile shape, say) is dropped and the word cleared.  The first
// candidate is the built-in shape; the fastest other one is timed against it
// three more times, alternately, and must beat it there by more than 5% to be
// chosen (run-to-run noise is about 2%, and a forward timed alone can favour
// a shape that is slower inside a forward + backward step).  The choice is kept in
// the context and the store (and written to the cache file, if one is set),
// and the call's outputs come from one more run of it.  Tuning is skipped
// while the error word already holds an error.  `fix` (optional) overrides
// fields of every shape the call launches.
template <class K, class C, class F, class G>
int run_tuned(dgal_ctx* ctx, K key, C candidates, hipStream_t stream, F launch, G fix) {
  auto go = [&](dgal::LaunchShape sh) { return launch(fix(sh)); };
  if (untuned(ctx)) return go(dgal::LaunchShape());
  const std::string text = key().text(ctx->arch);
  auto it = ctx->tuned.find(text);
  if (it != ctx->tuned.end()) return go(it->second);
  dgal::LaunchShape stored;
  if (dgal::tune_store_get(text, &stored) && dgal::shape_valid(stored)) {
    ctx->tuned[text] = stored;
    return go(stored);
  }
  if (!ctx->tune) return go(dgal::LaunchShape());
  int pending = 0;
  if (int st = read_err(ctx, stream, &pending)) return st;
  if (pending != 0) {  // an earlier call's error: put it back, tune another time
    for (int k = 0; k < dgal::kErrWords; ++k)
      if (pending >> k & 1) ctx->err_host[k] = 1;
    return go(dgal::LaunchShape());
  }
  const std::vector<dgal::LaunchShape> cands = candidates();
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
    if (e0) (void)hipEventDestroy(e0);
    return DGAL_EHIP;
  }
  int st = DGAL_OK;
  std::vector<float> best_of(cands.size(), -1.f);  // < 0: failed or not timed
  std::vector<char> failed(cands.size(), 0);
  for (int pass = 0; pass < 2 && st == DGAL_OK; ++pass) {
    for (size_t c = 0; c < cands.size() && st == DGAL_OK; ++c) {
      if (failed[c]) continue;
      st = go(cands[c]);
      if (st != DGAL_OK) break;
      if (hipEventRecord(e0, stream) != hipSuccess) st = DGAL_EHIP;
      for (int r = 0; r < 3 && st == DGAL_OK; ++r) st = go(cands[c]);
      float ms = 0.f;
      if (st == DGAL_OK && (hipEventRecord(e1, stream) != hipSuccess ||
                            hipEventSynchronize(e1) != hipSuccess ||
                            hipEventElapsedTime(&ms, e0, e1) != hipSuccess))
        st = DGAL_EHIP;
      int err = 0;
      if (st == DGAL_OK) st = read_err(ctx, stream, &err);
      if (st != DGAL_OK) break;
      if (err != 0) {
        failed[c] = 1;
        best_of[c] = -1.f;
      } else if (best_of[c] < 0.f || ms < best_of[c]) {
        best_of[c] = ms;
      }
    }
  }
  int best = -1;
  if (st == DGAL_OK)
    for (size_t c = 0; c < cands.size(); ++c)
      if (best_of[c] >= 0.f && (best < 0 || best_of[c] < best_of[best])) best = (int)c;
  // The minimum over many noisy timings favours a lucky draw: a challenger
  // is timed again against the built-in shape, alternately, and the verdict
  // rests on these fresh timings alone.
  if (st == DGAL_OK && best > 0 && best_of[0] >= 0.f) {
    float again[2] = {-1.f, -1.f};
    for (int round = 0; round < 3 && st == DGAL_OK; ++round)
      for (int k = 0; k < 2 && st == DGAL_OK; ++k) {
        const size_t c = k == 0 ? 0 : (size_t)best;
        if (hipEventRecord(e0, stream) != hipSuccess) st = DGAL_EHIP;
        for (int r = 0; r < 3 && st == DGAL_OK; ++r) st = go(cands[c]);
        float ms = 0.f;
        if (st == DGAL_OK && (hipEventRecord(e1, stream) != hipSuccess ||
                              hipEventSynchronize(e1) != hipSuccess ||
                              hipEventElapsedTime(&ms, e0, e1) != hipSuccess))
          st = DGAL_EHIP;
        if (st == DGAL_OK && (again[k] < 0.f || ms < again[k])) again[k] = ms;
      }
    if (st == DGAL_OK) {
      best_of[0] = again[0];
      best_of[best] = again[1];
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (st != DGAL_OK) return st;
  if (best < 0) return go(dgal::LaunchShape());  // every candidate failed: its error stands
  if (best != 0 && best_of[0] >= 0.f && best_of[best] > 0.95f * best_of[0]) best = 0;
  const float best_ms = best_of[best];
  const dgal::LaunchShape chosen = fix(cands[best]);
  ctx->tuned[text] = chosen;
  dgal::tune_store_put(text, chosen, best_ms / 3.0);
  if (const char* path = dgal::tune_cache_path()) (void)dgal::tune_store_save(path);
  return go(chosen);
}

template <class K, class C, class F>
int run_tuned(dgal_ctx* ctx, K key, C candidates, hipStream_t stream, F launch) {
  return run_tuned(ctx, key, candidates, stream, launch, [](dgal::LaunchShape sh) { return sh; });
}

std::vector<dgal::LaunchShape> pair_grids(int cus) {
  std::vector<dgal::LaunchShape> v;
  for (int64_t m : {0, 2, 4, 8, 16}) {
    dgal::LaunchShape s;
    s.grid = (int64_t)cus * m;
    v.push_back(s);
  }
  return v;
}

// The 8-slot pair backward's grid is what is resident unless a shape says
// otherwise (the LDS allows 4 workgroups a CU), also for the rows that are not
// loaded ahead: 262,144 pairs of 5-gons take 27.6 us with a workgroup for every
// block of pairs and 25.8 so, 3..7-gons 37.8 and 33.8, unaligned rows 38.1 and
// 34.8.
int64_t pairs_bwd_grid(int K, int cus, int64_t grid) {
  return K == 8 && grid == 0 ? (int64_t)cus * 4 : grid;
}

// Its candidates: those grids, with a workgroup for every block of pairs (the
// largest grid: the launch needs no more) where the default is the resident one.
std::vector<dgal::LaunchShape> pair_bwd_grids(int K, int cus) {
  std::vector<dgal::LaunchShape> v = pair_grids(cus);
  if (K == 8)
    for (dgal::LaunchShape& s : v)
      if (s.grid == (int64_t)cus * 4) s.grid = dgal::kMaxGrid;
  return v;
}

// Tile rows (unless the caller fixed them) x persistent grids of the cull
// and exact passes.  16-row tiles are tried only when the caller fixed them:
// the backward's 8-row groups scan each 16-row tile row's entries twice (c5
// backward 71 -> 85 us), a cost the forward's timing cannot see.
std::vector<dgal::LaunchShape> matrix_fwd_shapes(int fixed_rows) {
  std::vector<dgal::LaunchShape> v;
  for (int r : {8, 4, 16}) {  // the built-in shape (8, 8, 8) first
    if (fixed_rows != 0 ? r != fixed_rows : r == 16) continue;
    for (int c : {8, 4, 16})
      for (int e : {8, 4, 16}) {
        dgal::LaunchShape s;
        s.tile_rows = r;
        s.cull_mult = c;
        s.exact_mult = e;
        v.push_back(s);
      }
  }
  return v;
}

std::vector<dgal::LaunchShape> matrix_bwd_shapes() {
  std::vector<dgal::LaunchShape> v;
  for (int b : {8, 4, 16}) {  // the built-in multiplier first
    dgal::LaunchShape s;
    s.bwd_mult = b;
    v.push_back(s);
  }
  return v;
}

TuneKey matrix_key(int kind, const dgal_polys& a, const dgal_polys& b, const int64_t* a_off,
                   int nseg) {
  TuneKey k;
  k.kind = kind;
  k.K = reg_k(a.kmax, b.kmax);
  k.fixed = a.nv == nullptr && b.nv == nullptr;
  k.z3 = a.zlo != nullptr;
  k.seg = a_off != nullptr;
  k.bucket = bucket_of(a.count, a_off != nullptr ? (int64_t)nseg : b.count);
  return k;
}

// With input checking on (dgal_set_validate, or DGAL_DEBUG_VALIDATE=1 in the
// environment when the context was created), every polygon of the call's
// sets is checked on the device against the contract of Sec. III, and the
// call waits for the count: DGAL_EINVAL if any polygon breaks it.
int debug_validate(dgal_ctx* ctx, hipStream_t s, const dgal_polys& a, const dgal_polys* b,
                   bool simple = false) {
  if (!ctx->validate) return DGAL_OK;
  if (!valid_polys(a) || (b && !valid_polys(*b))) return DGAL_EINVAL;
  DeviceGuard g(ctx->v.device);
  if (!g.ok) return DGAL_EHIP;
  const dgal_polys* sets[2] = {&a, b};
  for (const dgal_polys* p : sets) {
    if (p == nullptr || p->count == 0) continue;
    const dgal::PolyArgs pa = poly_args(*p, 8);
    if (dgal::launch_validate(pa, nullptr, ctx->n_bad, simple, s) != hipSuccess) return DGAL_EHIP;
    int64_t host = 0;
    if (hipMemcpyAsync(&host, ctx->n_bad, sizeof(host), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
      return DGAL_EHIP;
    if (host != 0) return DGAL_EINVAL;
  }
  return DGAL_OK;
}

}  // namespace

extern "C" {

int dgal_create(dgal_ctx** out, int hip_device) {
  if (out == nullptr) return DGAL_EINVAL;
  *out = nullptr;
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess) return DGAL_EHIP;
  if (hip_device < 0 || hip_device >= ndev) return DGAL_EINVAL;
  DeviceGuard g(hip_device);
  if (!g.ok) return DGAL_EHIP;
  dgal_ctx* c = new (std::nothrow) dgal_ctx;
  if (c == nullptr) return DGAL_EHIP;
  c->v.device = hip_device;
  c->v.err = nullptr;
  c->v.prefix = nullptr;
  c->v.scan = nullptr;
  c->v.prof = nullptr;
  c->v.stats = nullptr;
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, hip_device) != hipSuccess ||
      cus <= 0)
    cus = 256;
  c->v.cus = cus;
  void* err_host = nullptr;
  if (hipHostMalloc(&err_host, dgal::kErrWords * sizeof(int),
                    hipHostMallocMapped | hipHostMallocCoherent) == hipSuccess) {
    c->err_host = static_cast<int*>(err_host);
    for (int k = 0; k < dgal::kErrWords; ++k) c->err_host[k] = 0;
  }
  if (err_host == nullptr ||
      hipHostGetDevicePointer(reinterpret_cast<void**>(&c->v.err), err_host, 0) != hipSuccess ||
      hipMalloc(reinterpret_cast<void**>(&c->v.prefix), sizeof(int64_t) * 2 * (DGAL_MAX_SEGMENTS + 1)) !=
          hipSuccess ||
      hipMalloc(reinterpret_cast<void**>(&c->v.scan), sizeof(int64_t) * dgal::kScanTotals) !=
          hipSuccess ||
      hipMalloc(reinterpret_cast<void**>(&c->n_bad), sizeof(int64_t)) != hipSuccess ||
      hipMalloc(reinterpret_cast<void**>(&c->stats_dev), 3 * sizeof(unsigned long long)) !=
          hipSuccess ||
      hipMemset(c->stats_dev, 0, 3 * sizeof(unsigned long long)) != hipSuccess ||
      hipDeviceSynchronize() != hipSuccess) {
    if (c->stats_dev) (void)hipFree(c->stats_dev);
    if (err_host) (void)hipHostFree(err_host);
    if (c->v.prefix) (void)hipFree(c->v.prefix);
    if (c->v.scan) (void)hipFree(c->v.scan);
    if (c->n_bad) (void)hipFree(c->n_bad);
    delete c;
    return DGAL_EHIP;
  }
  // the allocation-free matrix forward's static scratch: its address on this
  // device, taken once per device (here, with the device current)
  if (dgal::matrix_scratch_init(hip_device) != DGAL_OK) {
    (void)hipHostFree(err_host);
    (void)hipFree(c->v.prefix);
    (void)hipFree(c->v.scan);
    (void)hipFree(c->n_bad);
    (void)hipFree(c->stats_dev);
    delete c;
    return DGAL_EHIP;
  }
  const char* dbg = getenv("DGAL_DEBUG_VALIDATE");
  c->validate = dbg != nullptr && strcmp(dbg, "1") == 0;
  hipDeviceProp_t prop;
  if (hipGetDeviceProperties(&prop, hip_device) == hipSuccess) {
    c->arch.assign(prop.gcnArchName, strnlen(prop.gcnArchName, sizeof(prop.gcnArchName)));
    const size_t colon = c->arch.find(':');  // "gfx950:sramecc+:xnack-" -> "gfx950"
    if (colon != std::string::npos) c->arch.resize(colon);
  }
  if (c->arch.empty()) c->arch = "unknown";
  (void)dgal::tune_cache_path();  // DGAL_TUNE_CACHE: loaded once per process
  *out = c;
  return DGAL_OK;
}

void dgal_destroy(dgal_ctx* ctx) {
  if (ctx == nullptr) return;
  DeviceGuard g(ctx->v.device);
  if (ctx->prof.e0) (void)hipEventDestroy(ctx->prof.e0);
  if (ctx->prof.e1) (void)hipEventDestroy(ctx->prof.e1);
  if (ctx->err_host) (void)hipHostFree(const_cast<int*>(ctx->err_host));
  if (ctx->v.prefix) (void)hipFree(ctx->v.prefix);
  if (ctx->v.scan) (void)hipFree(ctx->v.scan);
  if (ctx->n_bad) (void)hipFree(ctx->n_bad);
  if (ctx->stats_dev) (void)hipFree(ctx->stats_dev);
  delete ctx;
}

const char* dgal_status_string(int status) {
  switch (status) {
    case DGAL_OK: return "DGAL_OK";
    case DGAL_EINVAL: return "DGAL_EINVAL: invalid argument";
    case DGAL_ECAPACITY: return "DGAL_ECAPACITY: capacity exceeded";
    case DGAL_EHIP: return "DGAL_EHIP: HIP runtime error";
    case DGAL_EIO: return "DGAL_EIO: file could not be read or written";
    default: return "unknown dgal status";
  }
}

int dgal_check(dgal_ctx* ctx, void* stream) {
  if (ctx == nullptr) return DGAL_EINVAL;
  DeviceGuard g(ctx->v.device);
  if (!g.ok) return DGAL_EHIP;
  int errs = 0;
  if (int st = read_err(ctx, static_cast<hipStream_t>(stream), &errs)) return st;
  if (errs >> dgal::kErrCapacity & 1) return DGAL_ECAPACITY;
  return errs != 0 ? DGAL_EINVAL : DGAL_OK;
}

int dgal_iou_pairs(dgal_ctx* ctx, dgal_polys a, dgal_polys b, float* iou, uint8_t* nx,
                   uint8_t* xflags, void* stream) {
  if (ctx == nullptr || !valid_polys(a) || !valid_polys(b)) return DGAL_EINVAL;
  if (a.count != b.count) return DGAL_EINVAL;
  if ((nx == nullptr) != (xflags == nullptr)) return DGAL_EINVAL;
  if ((a.zlo == nullptr) != (b.zlo == nullptr)) return DGAL_EINVAL;
  if (a.count > 0 && iou == nullptr) return DGAL_EINVAL;
  if (a.count == 0) return DGAL_OK;
  if (int st = debug_validate(ctx, static_cast<hipStream_t>(stream), a, &b)) return st;
  DeviceGuard g(ctx->v.device);
  if (!g.ok) return DGAL_EHIP;
  const int K = reg_k(a.kmax, b.kmax);
  dgal::PairsFwdArgs args;
  args.a = poly_args(a, K);
  args.b = poly_args(b, K);
  args.iou = iou;
  args.nx = nx;
  args.xflags = xflags;
  args.cap = a.kmax + b.kmax;
  args.flags_vec = args.cap == 2 * K && aligned(xflags, (uintptr_t)(2 * K));
  args.err = ctx->v.err;
  args.stats = ctx->v.stats;
  // the fixed-size kernels also assume vector-aligned rows of coordinates and codes
  const bool fixed = a.nv == nullptr && b.nv == nullptr && a.kmax == K && b.kmax == K &&
                     args.a.vec4 && args.b.vec4 && (nx == nullptr || args.flags_vec);
  const bool z3 = a.zlo != nullptr, save = nx != nullptr;
  hipStream_t s = static_cast<hipStream_t>(stream);
  auto key = [&] { return TuneKey{kTunePairsFwd, K, fixed, z3, save, bucket_of(a.count)}; };
  return run_tuned(ctx, key, [&] { return pair_grids(ctx->v.cus); }, s,
                   [&](const dgal::LaunchShape& sh) {
                     dgal::prof_begin(ctx->v.prof, s);
                     const hipError_t e = dgal::launch_pairs_fwd(args, K, fixed, z3, save, s, sh);
                     dgal::prof_end(ctx->v.prof, "k_pairs_fwd", s);
                     return status_of(e);
                   });
}

int dgal_iou_backward(dgal_ctx* ctx, int32_t mode, dgal_polys a, dgal_polys b,
                      const int64_t* a_off, const int64_t* b_off, const int64_t* out_off,
                      int32_t nseg, int32_t self_pairs, const float* grad_iou, int64_t out_size,
                      const uint8_t* nx, const uint8_t* xflags, const dgal_saved* saved,
                      float* grad_a_xy, float* grad_b_xy, float* grad_a_z, float* grad_b_z,
                      void* stream) {
  if (ctx == nullptr || !valid_polys(a) || !valid_polys(b)) return DGAL_EINVAL;
  const bool z3 = a.zlo != nullptr;
  if ((a.zlo == nullptr) != (b.zlo == nullptr)) return DGAL_EINVAL;
  if (int st = debug_validate(ctx, static_cast<hipStream_t>(stream), a, &b)) return st;
  if (mode == DGAL_PAIRS) {
    (void)a_off;
    (void)b_off;
    (void)out_off;
    (void)nseg;
    (void)self_pairs;
    (void)saved;
    (void)out_size;
    if (a.count != b.count) return DGAL_EINVAL;
    if (a.count == 0) return DGAL_OK;
    if (grad_iou == nullptr || nx == nullptr || xflags == nullptr || grad_a_xy == nullptr ||
        grad_b_xy == nullptr)
      return DGAL_EINVAL;
    if (z3 != (grad_a_z != nullptr) || z3 != (grad_b_z != nullptr)) return DGAL_EINVAL;
    if (!aligned(grad_a_xy, 8) || !aligned(grad_b_xy, 8)) return DGAL_EINVAL;
    if (z3 && (!aligned(grad_a_z, 8) || !aligned(grad_b_z, 8))) return DGAL_EINVAL;
    DeviceGuard g(ctx->v.device);
    if (!g.ok) return DGAL_EHIP;
    const int K = reg_k(a.kmax, b.kmax);
    dgal::PairsBwdArgs args;
    args.a = poly_args(a, K);
    args.b = poly_args(b, K);
    // the gradient rows are written with the same vector width as the inputs
    args.a.vec4 = args.a.vec4 && aligned(grad_a_xy, 16);
    args.b.vec4 = args.b.vec4 && aligned(grad_b_xy, 16);
    args.grad = grad_iou;
    args.nx = nx;
    args.xflags = xflags;
    args.cap = a.kmax + b.kmax;
    args.flags_vec = args.cap == 2 * K && aligned(xflags, (uintptr_t)(2 * K));
    args.ga_xy = grad_a_xy;
    args.gb_xy = grad_b_xy;
    args.ga_z = grad_a_z;
    args.gb_z = grad_b_z;
    const bool fixed = a.nv == nullptr && b.nv == nullptr && a.kmax == K && b.kmax == K &&
                       args.a.vec4 && args.b.vec4 && args.flags_vec;
    hipStream_t s = static_cast<hipStream_t>(stream);
    auto key = [&] { return TuneKey{kTunePairsBwd, K, fixed, z3, 0, bucket_of(a.count)}; };
    return run_tuned(ctx, key, [&] { return pair_bwd_grids(K, ctx->v.cus); }, s,
                     [&](dgal::LaunchShape sh) {
                       sh.grid = pairs_bwd_grid(K, ctx->v.cus, sh.grid);
                       dgal::prof_begin(ctx->v.prof, s);
                       const hipError_t e = dgal::launch_pairs_bwd(args, K, fixed, z3, s, sh);
                       dgal::prof_end(ctx->v.prof, "k_pairs_bwd", s);
                       return status_of(e);
                     });
  }
  if (mode == DGAL_MATRIX) {
    hipStream_t s = static_cast<hipStream_t>(stream);
    auto launch = [&](const dgal::LaunchShape& sh) {
      return dgal::matrix_backward(ctx->v, a, b, a_off, b_off, out_off, nseg, self_pairs,
                                   grad_iou, out_size, saved, grad_a_xy, grad_b_xy, grad_a_z,
                                   grad_b_z, s, sh);
    };
    // a block whose grid is its row groups has one shape: nothing to choose
    if (dgal::matrix_bwd_split(ctx->v, a_off != nullptr, reg_k(a.kmax, b.kmax), a.count, b.count))
      return launch(dgal::LaunchShape());
    auto key = [&] { return matrix_key(kTuneMatrixBwd, a, b, a_off, nseg); };
    return run_tuned(ctx, key, matrix_bwd_shapes, s, launch);
  }
  return DGAL_EINVAL;
}

int dgal_iou_matrix(dgal_ctx* ctx, dgal_polys a, dgal_polys b, const int64_t* a_off,
                    const int64_t* b_off, const int64_t* out_off, int32_t nseg,
                    int32_t self_pairs, float* iou, int64_t out_size, dgal_saved* saved,
                    void* stream) {
  if (ctx == nullptr || saved == nullptr) return DGAL_EINVAL;
  // the caller's tile rows, if fixed, hold for every shape the call launches
  const int rows = saved->tile_rows;
  if (rows != 0 && rows != 4 && rows != 8 && rows != 16) return DGAL_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (int st = debug_validate(ctx, s, a, dgal::same_polys(a, b) ? nullptr : &b)) return st;
  auto key = [&] { return matrix_key(kTuneMatrixFwd, a, b, a_off, nseg); };
  return run_tuned(
      ctx, key, [&] { return matrix_fwd_shapes(rows); }, s,
      [&](const dgal::LaunchShape& sh) {
        return dgal::matrix_forward(ctx->v, a, b, a_off, b_off, out_off, nseg, self_pairs, iou,
                                    out_size, saved, s, sh);
      },
      [&](dgal::LaunchShape sh) {
        sh.tile_rows = rows != 0 ? rows : (sh.tile_rows != 0 ? sh.tile_rows : DGAL_TILE_ROWS_DEFAULT);
        return sh;
      });
}

int dgal_iou_matrix_noalloc(dgal_ctx* ctx, dgal_polys a, dgal_polys b, const int64_t* a_off,
                            const int64_t* b_off, const int64_t* out_off, int32_t nseg,
                            int32_t self_pairs, float* iou, int64_t out_size, void* stream) {
  if (ctx == nullptr) return DGAL_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (int st = debug_validate(ctx, s, a, dgal::same_polys(a, b) ? nullptr : &b)) return st;
  // a shape the autotuner already chose for dgal_iou_matrix (in this context,
  // or in the process-wide store) is reused; nothing is tuned here (tuning
  // allocates events and records its choice)
  dgal::LaunchShape shape;
  if (!untuned(ctx)) {
    const std::string key = matrix_key(kTuneMatrixFwd, a, b, a_off, nseg).text(ctx->arch);
    const auto it = ctx->tuned.find(key);
    if (it != ctx->tuned.end()) shape = it->second;
    else if (!dgal::tune_store_get(key, &shape) || !dgal::shape_valid(shape)) shape = dgal::LaunchShape();
  }
  return dgal::matrix_forward_noalloc(ctx->v, a, b, a_off, b_off, out_off, nseg, self_pairs, iou,
                                      out_size, s, shape);
}

int dgal_intersect(dgal_ctx* ctx, dgal_polys a, dgal_polys b, float* out_xy, uint8_t* nx,
                   uint8_t* xflags, void* stream) {
  if (ctx == nullptr || !valid_polys(a) || !valid_polys(b)) return DGAL_EINVAL;
  if (a.count != b.count) return DGAL_EINVAL;
  if (a.count == 0) return DGAL_OK;
  if (out_xy == nullptr || nx == nullptr || xflags == nullptr || !aligned(out_xy, 8))
    return DGAL_EINVAL;
  if (int st = debug_validate(ctx, static_cast<hipStream_t>(stream), a, &b)) return st;
  DeviceGuard g(ctx->v.device);
  if (!g.ok) return DGAL_EHIP;
  const int K = reg_k(a.kmax, b.kmax);
  dgal::IntersectArgs args;
  args.a = poly_args(a, K);
  args.b = poly_args(b, K);
  args.out_xy = out_xy;
  args.nx = nx;
  args.xflags = xflags;
  args.cap = a.kmax + b.kmax;
  args.rows_vec = args.cap == 2 * K && aligned(out_xy, 16) && aligned(xflags, (uintptr_t)(2 * K));
  args.err = ctx->v.err;
  args.stats = ctx->v.stats;
  const bool fixed = a.nv == nullptr && b.nv == nullptr && a.kmax == K && b.kmax == K &&
                     args.a.vec4 && args.b.vec4 && args.rows_vec;
  const hipError_t e_ = [&] {
    dgal::prof_begin(ctx->v.prof, static_cast<hipStream_t>(stream));
    const hipError_t r_ = dgal::launch_intersect_fwd(args, K, fixed, static_cast<hipStream_t>(stream));
    dgal::prof_end(ctx->v.prof, "k_intersect_fwd", static_cast<hipStream_t>(stream));
    return r_;
  }();
  return status_of(e_);
}

int dgal_intersect_backward(dgal_ctx* ctx, dgal_polys a, dgal_polys b, const float* grad_xy,
                            const uint8_t* nx, const uint8_t* xflags, float* grad_a_xy,
                            float* grad_b_xy, void* stream) {
  if (ctx == nullptr || !valid_polys(a) || !valid_polys(b)) return DGAL_EINVAL;
  if (a.count != b.count) return DGAL_EINVAL;
  if (a.count == 0) return DGAL_OK;
  if (grad_xy == nullptr || nx == nullptr || xflags == nullptr || grad_a_xy == nullptr ||
      grad_b_xy == nullptr)
    return DGAL_EINVAL;
  if (!aligned(grad_xy, 8) || !aligned(grad_a_xy, 8) || !aligned(grad_b_xy, 8)) return DGAL_EINVAL;
  if (int st = debug_validate(ctx, static_cast<hipStream_t>(stream), a, &b)) return st;
  DeviceGuard g(ctx->v.device);
  if (!g.ok) return DGAL_EHIP;
  const int K = reg_k(a.kmax, b.kmax);
  dgal::IntersectBwdArgs args;
  args.a = poly_args(a, K);
  args.b = poly_args(b, K);
  args.grad_xy = grad_xy;
  args.nx = nx;
  args.xflags = xflags;
  args.cap = a.kmax + b.kmax;
  args.ga_xy = grad_a_xy;
  args.gb_xy = grad_b_xy;
  args.rows_vec = args.cap == 2 * K && aligned(grad_xy, 16) && aligned(xflags, (uintptr_t)(2 * K)) &&
                  aligned(grad_a_xy, 16) && aligned(grad_b_xy, 16);
  const bool fixed = a.nv == nullptr && b.nv == nullptr && a.kmax == K && b.kmax == K &&
                     args.a.vec4 && args.b.vec4 && args.rows_vec;
  const hipError_t e_ = [&] {
    dgal::prof_begin(ctx->v.prof, static_cast<hipStream_t>(stream));
    const hipError_t r_ = dgal::launch_intersect_bwd(args, K, fixed, static_cast<hipStream_t>(stream));
    dgal::prof_end(ctx->v.prof, "k_intersect_bwd", static_cast<hipStream_t>(stream));
    return r_;
  }();
  return status_of(e_);
}

int dgal_area(dgal_ctx* ctx, dgal_polys p, float* area, void* stream) {
  if (ctx == nullptr || !valid_polys(p)) return DGAL_EINVAL;
  if (p.count == 0) return DGAL_OK;
  if (area == nullptr) return DGAL_EINVAL;
  DeviceGuard g(ctx->v.device);
  if (!g.ok) return DGAL_EHIP;
  const int K = p.kmax <= 4 ? 4 : 8;
  const dgal::PolyArgs pa = poly_args(p, K);
  const bool fixed = p.nv == nullptr && p.kmax == K && pa.vec4;
  const hipError_t e_ = [&] {
    dgal::prof_begin(ctx->v.prof, static_cast<hipStream_t>(stream));
    const hipError_t r_ =
        dgal::launch_area(pa, nullptr, area, K, fixed, false, static_cast<hipStream_t>(stream));
    dgal::prof_end(ctx->v.prof, "k_area", static_cast<hipStream_t>(stream));
    return r_;
  }();
  return status_of(e_);
}

int dgal_area_backward(dgal_ctx* ctx, dgal_polys p, const float* grad_area, float* grad_xy,
                       void* stream) {
  if (ctx == nullptr || !valid_polys(p)) return DGAL_EINVAL;
  if (p.count == 0) return DGAL_OK;
  if (grad_area == nullptr || grad_xy == nullptr || !aligned(grad_xy, 8)) return DGAL_EINVAL;
  DeviceGuard g(ctx->v.device);
  if (!g.ok) return DGAL_EHIP;
  const int K = p.kmax <= 4 ? 4 : 8;
  const dgal::PolyArgs pa = poly_args(p, K);
  const bool fixed = p.nv == nullptr && p.kmax == K && pa.vec4;
  const hipError_t e_ = [&] {
    dgal::prof_begin(ctx->v.prof, static_cast<hipStream_t>(stream));
    const hipError_t r_ = dgal::launch_area(pa, grad_area, grad_xy, K, fixed, true,
                                     static_cast<hipStream_t>(stream));
    dgal::prof_end(ctx->v.prof, "k_area_bwd", static_cast<hipStream_t>(stream));
    return r_;
  }();
  return status_of(e_);
}

}  // extern "C"

namespace {

bool valid_boxes(const dgal_boxes& a, const dgal_boxes& b) {
  if (a.count < 0 || a.count != b.count || a.dim != b.dim || (a.dim != 5 && a.dim != 7))
    return false;
  if (a.count > 0 && (a.p == nullptr || b.p == nullptr || !aligned(a.p, 4) || !aligned(b.p, 4)))
    return false;
  return true;
}

}  // namespace

extern "C" {

int dgal_iou_simple_pairs(dgal_ctx* ctx, dgal_polys a, dgal_polys b, float* iou, uint64_t* xmask,
                          uint64_t* smask, uint8_t* inside, void* stream) {
  if (ctx == nullptr || !valid_polys(a) || !valid_polys(b)) return DGAL_EINVAL;
  if (a.count != b.count || a.zlo != nullptr || b.zlo != nullptr) return DGAL_EINVAL;
  const bool save = xmask != nullptr;
  if ((smask != nullptr) != save || (inside != nullptr) != save) return DGAL_EINVAL;
  if (save && (!aligned(xmask, 8) || !aligned(smask, 8))) return DGAL_EINVAL;
  if (a.count == 0) return DGAL_OK;
  if (iou == nullptr) return DGAL_EINVAL;
  if (int st = debug_validate(ctx, static_cast<hipStream_t>(stream), a, &b, true)) return st;
  DeviceGuard g(ctx->v.device);
  if (!g.ok) return DGAL_EHIP;
  const int K = reg_k(a.kmax, b.kmax);
  dgal::SimpleFwdArgs args;
  args.a = poly_args(a, K);
  args.b = poly_args(b, K);
  args.iou = iou;
  args.xmask = xmask;
  args.smask = smask;
  args.inside = inside;
  const hipError_t e_ = [&] {
    dgal::prof_begin(ctx->v.prof, static_cast<hipStream_t>(stream));
    const hipError_t r_ = dgal::launch_simple_fwd(args, K, static_cast<hipStream_t>(stream));
    dgal::prof_end(ctx->v.prof, "k_simple_fwd", static_cast<hipStream_t>(stream));
    return r_;
  }();
  return status_of(e_);
}

int dgal_iou_simple_backward(dgal_ctx* ctx, dgal_polys a, dgal_polys b, const float* grad_iou,
                             const uint64_t* xmask, const uint64_t* smask, const uint8_t* inside,
                             float* grad_a_xy, float* grad_b_xy, void* stream) {
  if (ctx == nullptr || !valid_polys(a) || !valid_polys(b)) return DGAL_EINVAL;
  if (a.count != b.count || a.zlo != nullptr || b.zlo != nullptr) return DGAL_EINVAL;
  if (a.count == 0) return DGAL_OK;
  if (grad_iou == nullptr || xmask == nullptr || smask == nullptr || inside == nullptr ||
      grad_a_xy == nullptr || grad_b_xy == nullptr)
    return DGAL_EINVAL;
  if (!aligned(xmask, 8) || !aligned(smask, 8) || !aligned(grad_a_xy, 8) || !aligned(grad_b_xy, 8))
    return DGAL_EINVAL;
  if (int st = debug_validate(ctx, static_cast<hipStream_t>(stream), a, &b, true)) return st;
  DeviceGuard g(ctx->v.device);
  if (!g.ok) return DGAL_EHIP;
  const int K = reg_k(a.kmax, b.kmax);
  dgal::SimpleBwdArgs args;
  args.a = poly_args(a, K);
  args.b = poly_args(b, K);
  args.grad = grad_iou;
  args.xmask = xmask;
  args.smask = smask;
  args.inside = inside;
  // the gradient rows are written with the same vector width as the inputs
  args.a.vec4 = args.a.vec4 && aligned(grad_a_xy, 16);
  args.b.vec4 = args.b.vec4 && aligned(grad_b_xy, 16);
  args.ga_xy = grad_a_xy;
  args.gb_xy = grad_b_xy;
  const hipError_t e_ = [&] {
    dgal::prof_begin(ctx->v.prof, static_cast<hipStream_t>(stream));
    const hipError_t r_ = dgal::launch_simple_bwd(args, K, static_cast<hipStream_t>(stream));
    dgal::prof_end(ctx->v.prof, "k_simple_bwd", static_cast<hipStream_t>(stream));
    return r_;
  }();
  return status_of(e_);
}

int dgal_validate(dgal_ctx* ctx, dgal_polys p, uint8_t* status, int64_t* n_bad, void* stream) {
  if (ctx == nullptr || !valid_polys(p)) return DGAL_EINVAL;
  if (status == nullptr && n_bad == nullptr) return DGAL_EINVAL;
  if (n_bad != nullptr && !aligned(n_bad, 8)) return DGAL_EINVAL;
  if (p.count > 0 && p.xy == nullptr) return DGAL_EINVAL;
  DeviceGuard g(ctx->v.device);
  if (!g.ok) return DGAL_EHIP;
  return status_of(dgal::launch_validate(poly_args(p, 8), status, n_bad, false,
                                         static_cast<hipStream_t>(stream)));
}

int dgal_validate_simple(dgal_ctx* ctx, dgal_polys p, uint8_t* status, int64_t* n_bad,
                         void* stream) {
  if (ctx == nullptr || !valid_polys(p)) return DGAL_EINVAL;
  if (status == nullptr && n_bad == nullptr) return DGAL_EINVAL;
  if (n_bad != nullptr && !aligned(n_bad, 8)) return DGAL_EINVAL;
  if (p.count > 0 && p.xy == nullptr) return DGAL_EINVAL;
  DeviceGuard g(ctx->v.device);
  if (!g.ok) return DGAL_EHIP;
  return status_of(dgal::launch_validate(poly_args(p, 8), status, n_bad, true,
                                         static_cast<hipStream_t>(stream)));
}

int dgal_set_validate(dgal_ctx* ctx, int32_t enable) {
  if (ctx == nullptr) return DGAL_EINVAL;
  ctx->validate = enable != 0;
  return DGAL_OK;
}

int dgal_set_autotune(dgal_ctx* ctx, int32_t enable) {
  if (ctx == nullptr) return DGAL_EINVAL;
  ctx->tune = enable != 0;
  return DGAL_OK;
}

int dgal_set_profiling(dgal_ctx* ctx, int32_t enable) {
  if (ctx == nullptr) return DGAL_EINVAL;
  DeviceGuard g(ctx->v.device);
  if (!g.ok) return DGAL_EHIP;
  if (enable) {
    if (ctx->prof.e0 == nullptr && hipEventCreate(&ctx->prof.e0) != hipSuccess) return DGAL_EHIP;
    if (ctx->prof.e1 == nullptr && hipEventCreate(&ctx->prof.e1) != hipSuccess) return DGAL_EHIP;
    ctx->prof.n = 0;
    ctx->prof.err = hipSuccess;
    ctx->v.prof = &ctx->prof;
  } else {
    ctx->v.prof = nullptr;
  }
  return DGAL_OK;
}

int dgal_set_path_stats(dgal_ctx* ctx, int32_t enable) {
  if (ctx == nullptr) return DGAL_EINVAL;
  ctx->v.stats = enable ? ctx->stats_dev : nullptr;
  return DGAL_OK;
}

int dgal_path_stats(dgal_ctx* ctx, int64_t* pairs, int64_t* fp64_pairs, int64_t* thin_pairs,
                    void* stream) {
  if (ctx == nullptr || pairs == nullptr || fp64_pairs == nullptr || thin_pairs == nullptr)
    return DGAL_EINVAL;
  DeviceGuard g(ctx->v.device);
  if (!g.ok) return DGAL_EHIP;
  unsigned long long host[3] = {0ull, 0ull, 0ull};
  const unsigned long long zeros[3] = {0ull, 0ull, 0ull};
  if (hipStreamSynchronize(static_cast<hipStream_t>(stream)) != hipSuccess ||
      hipMemcpy(host, ctx->stats_dev, sizeof(host), hipMemcpyDeviceToHost) != hipSuccess ||
      hipMemcpy(ctx->stats_dev, zeros, sizeof(zeros), hipMemcpyHostToDevice) != hipSuccess)
    return DGAL_EHIP;
  *pairs = (int64_t)host[0];
  *fp64_pairs = (int64_t)host[1];
  *thin_pairs = (int64_t)host[2];
  return DGAL_OK;
}

int dgal_profile_report(dgal_ctx* ctx, char* buf, int64_t size) {
  if (ctx == nullptr || (buf == nullptr && size > 0) || size < 0) return DGAL_EINVAL;
  if (ctx->prof.err != hipSuccess) return DGAL_EHIP;
  int64_t used = 0;
  if (size > 0) buf[0] = '\0';
  for (int k = 0; k < ctx->prof.n; ++k) {
    char line[160];
    const int n = snprintf(line, sizeof(line), "%s %lld %.6f\n", ctx->prof.name[k],
                           (long long)ctx->prof.launches[k], ctx->prof.ms[k]);
    if (n > 0 && used + n < size) {
      memcpy(buf + used, line, (size_t)n + 1);
      used += n;
    }
  }
  return ctx->prof.n;
}

int dgal_autotune_report(dgal_ctx* ctx, char* buf, int64_t size) {
  if (ctx == nullptr || (buf == nullptr && size > 0) || size < 0) return DGAL_EINVAL;
  int64_t used = 0;
  if (size > 0) buf[0] = '\0';
  for (const auto& kv : ctx->tuned) {
    const dgal::LaunchShape& sh = kv.second;
    char line[320];
    const int n = snprintf(line, sizeof(line), "%s: grid=%lld cull=%d exact=%d bwd=%d rows=%d\n",
                           kv.first.c_str(), (long long)sh.grid, sh.cull_mult, sh.exact_mult,
                           sh.bwd_mult, sh.tile_rows);
    if (n > 0 && used + n < size) {
      memcpy(buf + used, line, (size_t)n + 1);
      used += n;
    }
  }
  return (int)ctx->tuned.size();
}

int dgal_tune_cache_load(const char* path) {
  if (path == nullptr || path[0] == '\0') return DGAL_EINVAL;
  return dgal::tune_store_load(path);
}

int dgal_tune_cache_save(const char* path) {
  if (path == nullptr || path[0] == '\0') return DGAL_EINVAL;
  return dgal::tune_store_save(path);
}

int dgal_tune_cache_report(char* buf, int64_t size) {
  if ((buf == nullptr && size > 0) || size < 0) return DGAL_EINVAL;
  return dgal::tune_store_report(buf, size);
}

int dgal_tune_cache_clear(void) {
  dgal::tune_store_clear();
  return DGAL_OK;
}

int dgal_iou_boxes(dgal_ctx* ctx, dgal_boxes a, dgal_boxes b, float* iou, uint8_t* nx,
                   uint8_t* xflags, void* stream) {
  if (ctx == nullptr || !valid_boxes(a, b)) return DGAL_EINVAL;
  if ((nx == nullptr) != (xflags == nullptr)) return DGAL_EINVAL;
  if (a.count == 0) return DGAL_OK;
  if (iou == nullptr || (xflags != nullptr && !aligned(xflags, 8))) return DGAL_EINVAL;
  DeviceGuard g(ctx->v.device);
  if (!g.ok) return DGAL_EHIP;
  dgal::BoxesFwdArgs args;
  args.a = a.p;
  args.b = b.p;
  args.count = a.count;
  args.iou = iou;
  args.nx = nx;
  args.xflags = xflags;
  args.err = ctx->v.err;
  args.stats = ctx->v.stats;
  const hipError_t e_ = [&] {
    dgal::prof_begin(ctx->v.prof, static_cast<hipStream_t>(stream));
    const hipError_t r_ = dgal::launch_boxes_fwd(args, a.dim == 7, nx != nullptr,
                                          static_cast<hipStream_t>(stream));
    dgal::prof_end(ctx->v.prof, "k_boxes_fwd", static_cast<hipStream_t>(stream));
    return r_;
  }();
  return status_of(e_);
}

int dgal_iou_boxes_backward(dgal_ctx* ctx, dgal_boxes a, dgal_boxes b, const float* grad_iou,
                            const uint8_t* nx, const uint8_t* xflags, float* grad_a,
                            float* grad_b, void* stream) {
  if (ctx == nullptr || !valid_boxes(a, b)) return DGAL_EINVAL;
  if (a.count == 0) return DGAL_OK;
  if (grad_iou == nullptr || nx == nullptr || xflags == nullptr || grad_a == nullptr ||
      grad_b == nullptr || !aligned(xflags, 8) || !aligned(grad_a, 4) || !aligned(grad_b, 4))
    return DGAL_EINVAL;
  DeviceGuard g(ctx->v.device);
  if (!g.ok) return DGAL_EHIP;
  dgal::BoxesBwdArgs args;
  args.a = a.p;
  args.b = b.p;
  args.count = a.count;
  args.grad = grad_iou;
  args.nx = nx;
  args.xflags = xflags;
  args.ga = grad_a;
  args.gb = grad_b;
  const hipError_t e_ = [&] {
    dgal::prof_begin(ctx->v.prof, static_cast<hipStream_t>(stream));
    const hipError_t r_ = dgal::launch_boxes_bwd(args, a.dim == 7, static_cast<hipStream_t>(stream));
    dgal::prof_end(ctx->v.prof, "k_boxes_bwd", static_cast<hipStream_t>(stream));
    return r_;
  }();
  return status_of(e_);
}

}  // extern "C"
