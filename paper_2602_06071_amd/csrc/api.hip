// C ABI of the library: argument checks, seed -> wiring derivation, variant
// dispatch and workspace management.  No arithmetic of the sketch apply itself
// lives here; it is all in the k_*.hip kernels.
#include <math.h>
#include <stdio.h>
#include <string.h>
#include <new>

#include "handle.h"
#include "mfma_plan.h"
#include "spec.h"

fs_status fs::hip_fail(fs_sketch_t h, hipError_t e) {
  if (h) h->last_hip_error = (int)e;
  (void)hipGetLastError();  // clear the sticky launch error
  return FS_ERR_HIP;
}

namespace {

using fs::hip_fail;

uint32_t radical(uint32_t m) {
  uint32_t r = 1;
  for (uint32_t p = 2; (uint64_t)p * p <= m; ++p) {
    if (m % p == 0) {
      r *= p;
      while (m % p == 0) m /= p;
    }
  }
  if (m > 1) r *= m;
  return r;
}

uint32_t lcm_u32(uint32_t x, uint32_t y) { return x / fs::gcd_u32(x, y) * y; }

// inverse of a modulo M by the extended Euclidean algorithm (gcd(a, M) = 1)
uint32_t mod_inverse(uint32_t a, uint32_t M) {
  int64_t t = 0, nt = 1, r = M, nr = a % M;
  while (nr != 0) {
    int64_t q = r / nr;
    int64_t tmp = t - q * nt; t = nt; nt = tmp;
    tmp = r - q * nr; r = nr; nr = tmp;
  }
  if (t < 0) t += M;
  return (uint32_t)t;
}

// Appendix E, "Full-cycle affine construction": b coprime to M, a - 1 divisible by
// every prime of M and by 4 when 4 | M.  (a, b) are drawn from the seed keys.
void derive_wiring(uint32_t M, uint32_t key1, uint32_t* a, uint32_t* b, uint32_t* a_inv) {
  if (M == 1) { *a = 0; *b = 0; *a_inv = 0; return; }
  const uint32_t L = lcm_u32(radical(M), (M % 4 == 0) ? 4u : 1u);
  const uint32_t ha = fs::mix32(key1 ^ 1u), hb = fs::mix32(key1 ^ 2u);
  *a = (uint32_t)((1u + (uint64_t)L * (ha % (M / L))) % M);
  uint32_t bb = hb % M;
  while (fs::gcd_u32(bb, M) != 1u) bb = (bb + 1u) % M;
  *b = bb;
  *a_inv = mod_inverse(*a, M);
}

bool is_pow2(uint32_t x) { return x && !(x & (x - 1)); }

bool valid_dtype(fs_dtype dt) { return dt == FS_F32 || dt == FS_BF16 || dt == FS_F16; }

// Whether a call of a kind other than BLOCKPERM runs, and its workspace.
fs_status other_kind(fs_sketch_t h, const void* A, int64_t lda, int64_t n, fs_dtype dt, fs::Workspace* need) {
  *need = {};
  if (h->kind == FS_KIND_SJLT_SCATTER) need->floor = need->want = fs::scatter_workspace_bytes(h->p, n, dt);
  if (h->kind == FS_KIND_GAUSS_DENSE && !fs::gauss_supported(h->p.k, h->p.d, A, lda, n, dt)) return FS_ERR_UNSUPPORTED;
  return FS_OK;
}

size_t rows_want(const fs::mm::RowsPlan& pl) { return !pl.ok ? 0 : pl.ws > pl.ws_floor ? pl.ws : pl.ws_floor; }

// Whether `st` is being captured into a graph (the NULL stream cannot be).
bool capturing(hipStream_t st) {
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (!st) return false;
  if (hipStreamIsCapturing(st, &cap) != hipSuccess) { (void)hipGetLastError(); return false; }
  return cap != hipStreamCaptureStatusNone;
}

// Gives up the handle's own workspace: frees it (which waits for work that may still use it) or, if a
// graph may still use it, sets it aside until the handle is destroyed.
fs_status drop_workspace(fs_sketch_t h) {
  if (!h->ws || !h->ws_owned) return FS_OK;
  void* p = h->ws;
  const bool keep = h->ws_captured;
  h->ws = nullptr; h->ws_bytes = 0; h->ws_captured = false;
  if (keep) {
    h->ws_retired.push_back(p);  // (room was reserved when it was marked)
    return FS_OK;
  }
  const hipError_t e = hipFree(p);
  return e == hipSuccess ? FS_OK : hip_fail(h, e);
}

fs_status ensure_workspace(fs_sketch_t h, size_t need) {
  if (need <= h->ws_bytes) return FS_OK;
  if (h->ws && !h->ws_owned) return FS_ERR_ALLOC;  // caller-owned and too small
  const fs_status rc = drop_workspace(h);
  if (rc != FS_OK) return rc;
  void* p = nullptr;
  hipError_t e = hipMalloc(&p, need);
  if (e != hipSuccess) { hip_fail(h, e); return FS_ERR_ALLOC; }
  h->ws = p; h->ws_bytes = need; h->ws_owned = true;
  return FS_OK;
}

// Workspace for a call that runs with `w.floor` bytes and is fastest with `w.want`.  An attached
// workspace is taken as it is if it holds the floor.  The handle's own is allocated by the first call
// that wants one, with kSplitScratch at least; `want` exceeds the floor only up to that size, so that
// later calls free and replace it only for a larger floor, not because a smaller problem is split into
// more pieces.  A call that the present size can serve is served by it where it may not or could not
// be larger: while `st` is being captured into a graph (nothing may be allocated there) and after the
// device was too full for kSplitScratch (nothing is freed that a call can run with, and a refused
// allocation is not tried again for speed alone).
fs_status ensure_workspace(fs_sketch_t h, const fs::Workspace& w, hipStream_t st) {
  const bool needs_none = w.want == 0 || (h->ws && !h->ws_owned);
  if (w.floor > h->ws_bytes || (w.want > h->ws_bytes && !h->ws && !h->ws_refused && !capturing(st))) {
    const size_t ask = w.want > fs::kSplitScratch ? w.want : fs::kSplitScratch;
    fs_status rc = ensure_workspace(h, ask);
    if (rc == FS_ERR_ALLOC && !h->ws) {
      h->ws_refused = true;  // short of memory: what the call must have
      if (w.floor < ask) rc = ensure_workspace(h, w.floor);
    }
    if (rc != FS_OK) return rc;
  }
  if (needs_none || !h->ws || h->ws_captured || !capturing(st)) return FS_OK;
  try {
    h->ws_retired.reserve(h->ws_retired.size() + 1);
  } catch (const std::bad_alloc&) {
    return FS_ERR_ALLOC;
  }
  h->ws_captured = true;
  return FS_OK;
}

// pos2blk[q] = f^q(0), blk2pos = its inverse: allocated once per handle and filled by a small
// kernel enqueued on `st` (no copy, no synchronisation).
fs_status ensure_orbit(fs_sketch_t h, hipStream_t st) {
  if (h->orbit || !fs::mfma_wants_orbit(h->p)) return FS_OK;
  void* dev = nullptr;
  hipError_t e = hipMalloc(&dev, 2 * (size_t)h->p.M * sizeof(uint32_t));
  if (e != hipSuccess) { hip_fail(h, e); return FS_ERR_ALLOC; }
  e = fs::launch_orbit(h->p, (uint32_t*)dev, st);
  if (e != hipSuccess) { (void)hipFree(dev); return hip_fail(h, e); }
  h->orbit = (uint32_t*)dev;
  return FS_OK;
}

// The next unused set of profiling events (all null when not profiling).  `begin` is recorded
// here, before anything the apply enqueues; the caller records `end` after its last launch.
struct ProfSet {
  fs::EventPair kernel;
  hipEvent_t end = nullptr;
};
ProfSet next_events(fs_sketch_t h, hipStream_t st) {
  ProfSet ps;
  if (h->profiling && h->prof_used < (int)h->prof_begin.size()) {
    const int i = h->prof_used++;
    if (h->prof_scope & FS_PROFILE_KERNEL) {
      ps.kernel.start = h->prof_start[i];
      ps.kernel.stop = h->prof_stop[i];
    }
    if (h->prof_scope & FS_PROFILE_APPLY) {
      ps.end = h->prof_end[i];
      (void)hipEventRecord(h->prof_begin[i], st);
    }
  }
  return ps;
}

}  // namespace

extern "C" {

const char* fs_status_string(fs_status st) {
  switch (st) {
    case FS_OK: return "ok";
    case FS_ERR_INVALID_ARG: return "invalid argument";
    case FS_ERR_UNSUPPORTED: return "unsupported shape or variant";
    case FS_ERR_ALLOC: return "allocation failed or workspace too small";
    case FS_ERR_HIP: return "HIP runtime error";
  }
  return "unknown status";
}

fs_status fs_sketch_create_kind(fs_sketch_t* out, fs_kind kind, int64_t d, int64_t k, int32_t Bc,
                                int32_t Br, int32_t kappa, int32_t s, uint64_t seed) {
  if (!out) return FS_ERR_INVALID_ARG;
  *out = nullptr;
  if (kind != FS_KIND_BLOCKPERM && kind != FS_KIND_SJLT_SCATTER && kind != FS_KIND_GAUSS_DENSE &&
      kind != FS_KIND_BLOCKROW)
    return FS_ERR_INVALID_ARG;
  if (d < 1 || k < 1 || d > ((int64_t)1 << 40) || k > ((int64_t)1 << 31)) return FS_ERR_INVALID_ARG;
  if (kind == FS_KIND_GAUSS_DENSE) { Bc = (int32_t)(d > 0x7fffffff ? 0x7fffffff : d); Br = 1; kappa = 1; s = 1; }
  if (kind != FS_KIND_GAUSS_DENSE) {
    if (Bc < 1 || Br < 1 || kappa < 1 || s < 1) return FS_ERR_INVALID_ARG;
    // the block grid is square: M = k/Br = ceil(d/Bc); a last input block that is only partly
    // filled is treated as zero-padded (Section 4, "general cases ... by padding")
    if (k % Br || (d + Bc - 1) / Bc != k / Br) return FS_ERR_INVALID_ARG;
    const int64_t M = k / Br;
    if (M > (1 << 24) || kappa > M) return FS_ERR_INVALID_ARG;
    if (s > Br || s > 32 || Br > 65536) return FS_ERR_INVALID_ARG;
    // (the scatter kernel walks exactly Bc rows of A: a padded block, Bc > d, is not accepted)
    if (kind == FS_KIND_SJLT_SCATTER && (M != 1 || kappa != 1 || Bc != d)) return FS_ERR_INVALID_ARG;
  }
  fs_sketch_s* h = new (std::nothrow) fs_sketch_s();
  if (!h) return FS_ERR_ALLOC;
  SketchParams& p = h->p;
  p.d = d; p.k = k;
  p.Bc = (uint32_t)Bc; p.Br = (uint32_t)Br; p.kappa = (uint32_t)kappa; p.s = (uint32_t)s;
  p.M = kind == FS_KIND_GAUSS_DENSE ? 1u : (uint32_t)(k / Br);
  h->key0 = fs::mix32((uint32_t)(seed & 0xFFFFFFFFu) ^ fs::kC1);
  p.key1 = fs::mix32((uint32_t)(seed >> 32) ^ h->key0 ^ fs::kC2);
  derive_wiring(p.M, p.key1, &p.a, &p.b, &p.a_inv);
  p.br_pow2 = is_pow2(p.Br) ? 1u : 0u;
  p.scale = kind == FS_KIND_GAUSS_DENSE ? (float)(1.0 / sqrt((double)k))
            : kind == FS_KIND_BLOCKROW  ? (float)(sqrt((double)d / (double)k) / sqrt((double)kappa * (double)s))
                                        : (float)(1.0 / sqrt((double)kappa * (double)s));
  h->kind = (int)kind;
  h->variant = FS_VARIANT_AUTO;
  h->last_variant = 0;
  h->last_mode = 0;
  h->last_hip_error = 0;
  h->last_kernel[0] = 0;
  h->device = -1;
  h->ws = nullptr; h->ws_bytes = 0; h->ws_owned = true; h->ws_refused = false; h->ws_captured = false;
  h->dense = nullptr; h->dense_scratch = 0; h->dense_half = false;
  h->profiling = false; h->prof_used = 0; h->prof_scope = 0;
  h->orbit = nullptr;

  if (kind == FS_KIND_GAUSS_DENSE) {
    if ((double)k * (double)d > 2.0e9) { delete h; return FS_ERR_UNSUPPORTED; }
    hipError_t e = hipErrorOutOfMemory;
    // what the device has room for: all of it, no half pieces, or the matrix alone (applies then do not split d)
    for (int have = 2; have >= 0 && e == hipErrorOutOfMemory; --have) {
      if (have < 2) (void)hipGetLastError();  // of the attempt before; what the caller left stays to be seen
      h->dense_half = have == 2;
      h->dense_scratch = have ? fs::kGaussScratch : 0;
      e = hipMalloc(&h->dense, fs::gauss_bytes(k, d) + (h->dense_half ? fs::gauss_half_bytes(k, d) : 0) + h->dense_scratch);
    }
    if (e == hipSuccess) e = fs::gauss_fill(h->dense, h->dense_half, k, d, p.key1, nullptr);
    if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
    if (e != hipSuccess) {
      (void)hipGetLastError();
      if (h->dense) (void)hipFree(h->dense);
      const bool oom = (e == hipErrorOutOfMemory);
      delete h;
      return oom ? FS_ERR_ALLOC : FS_ERR_HIP;
    }
  }
  *out = h;
  return FS_OK;
}

fs_status fs_sketch_create(fs_sketch_t* out, int64_t d, int64_t k, int32_t Bc, int32_t Br,
                           int32_t kappa, int32_t s, uint64_t seed) {
  return fs_sketch_create_kind(out, FS_KIND_BLOCKPERM, d, k, Bc, Br, kappa, s, seed);
}

static void release_events(fs_sketch_t h) {
  for (auto* v : {&h->prof_begin, &h->prof_start, &h->prof_stop, &h->prof_end}) {
    for (hipEvent_t e : *v) (void)hipEventDestroy(e);
    v->clear();
  }
  h->profiling = false; h->prof_used = 0;
}

fs_status fs_sketch_profile_begin(fs_sketch_t h, int32_t max_launches, int32_t scope) {
  if (!h || max_launches < 1 || max_launches > (1 << 20) || h->profiling) return FS_ERR_INVALID_ARG;
  if (scope < 1 || scope > (FS_PROFILE_KERNEL | FS_PROFILE_APPLY)) return FS_ERR_INVALID_ARG;
  h->prof_scope = scope;
  for (int i = 0; i < max_launches; ++i) {
    for (auto* v : {&h->prof_begin, &h->prof_start, &h->prof_stop, &h->prof_end}) {
      hipEvent_t ev = nullptr;
      const hipError_t e = hipEventCreate(&ev);
      if (e != hipSuccess) {
        release_events(h);
        return hip_fail(h, e);
      }
      v->push_back(ev);
    }
  }
  h->profiling = true; h->prof_used = 0;
  return FS_OK;
}

fs_status fs_sketch_profile_end(fs_sketch_t h, float* ms, float* ms_apply, int32_t* count) {
  if (!h || !ms || !count || !h->profiling) return FS_ERR_INVALID_ARG;
  fs_status rc = FS_OK;
  *count = h->prof_used;
  const bool k = h->prof_scope & FS_PROFILE_KERNEL, a = h->prof_scope & FS_PROFILE_APPLY;
  for (int i = 0; i < h->prof_used; ++i) {
    hipError_t e = hipEventSynchronize(a ? h->prof_end[i] : h->prof_stop[i]);
    ms[i] = 0.f;
    if (ms_apply) ms_apply[i] = 0.f;
    if (e == hipSuccess && k) e = hipEventElapsedTime(&ms[i], h->prof_start[i], h->prof_stop[i]);
    if (e == hipSuccess && a && ms_apply) e = hipEventElapsedTime(&ms_apply[i], h->prof_begin[i], h->prof_end[i]);
    if (e != hipSuccess) { rc = hip_fail(h, e); *count = i; break; }
  }
  release_events(h);
  return rc;
}

fs_status fs_sketch_destroy(fs_sketch_t h) {
  if (!h) return FS_ERR_INVALID_ARG;
  fs_status st = FS_OK;
  release_events(h);
  if (h->ws && h->ws_owned && hipFree(h->ws) != hipSuccess) st = FS_ERR_HIP;
  for (void* p : h->ws_retired)
    if (hipFree(p) != hipSuccess) st = FS_ERR_HIP;
  if (h->orbit && hipFree(h->orbit) != hipSuccess) st = FS_ERR_HIP;
  if (h->dense && hipFree(h->dense) != hipSuccess) st = FS_ERR_HIP;
  if (st != FS_OK) (void)hipGetLastError();
  delete h;
  return st;
}

fs_status fs_sketch_info(fs_sketch_t h, fs_info* o) {
  if (!h || !o) return FS_ERR_INVALID_ARG;
  const SketchParams& p = h->p;
  o->d = p.d; o->k = p.k;
  o->Bc = (int32_t)p.Bc; o->Br = (int32_t)p.Br; o->kappa = (int32_t)p.kappa; o->s = (int32_t)p.s;
  o->M = (int32_t)p.M; o->a = (int32_t)p.a; o->b = (int32_t)p.b; o->a_inv = (int32_t)p.a_inv;
  o->key0 = h->key0; o->key1 = p.key1;
  o->scale = p.scale;
  o->kind = h->kind; o->variant = h->variant; o->last_variant = h->last_variant; o->last_mode = h->last_mode;
  o->last_hip_error = h->last_hip_error;
  o->workspace_bytes = h->ws_bytes;
  memcpy(o->last_kernel, h->last_kernel, sizeof(o->last_kernel));
  return FS_OK;
}

fs_status fs_sketch_set_variant(fs_sketch_t h, fs_variant v) {
  if (!h) return FS_ERR_INVALID_ARG;
  if (v != FS_VARIANT_AUTO && v != FS_VARIANT_GENERIC && v != FS_VARIANT_MFMA)
    return FS_ERR_INVALID_ARG;
  h->variant = (int)v;
  return FS_OK;
}

fs_status fs_sketch_workspace_bytes(fs_sketch_t h, int64_t n, fs_dtype dt, size_t* bytes) {
  if (!h || !bytes || n < 0 || !valid_dtype(dt)) return FS_ERR_INVALID_ARG;
  *bytes = 0;
  if (n == 0) return FS_OK;
  if (h->kind == FS_KIND_SJLT_SCATTER) *bytes = fs::scatter_workspace_bytes(h->p, n, dt);
  // (a bound over alignments; shapes the matrix-core kernels do not take need none)
  if (h->kind == FS_KIND_BLOCKPERM && h->variant != FS_VARIANT_GENERIC) *bytes = fs::mfma_workspace_bytes(h->p, n, dt);
  return FS_OK;
}

fs_status fs_sketch_set_workspace(fs_sketch_t h, void* dev_ptr, size_t bytes) {
  if (!h) return FS_ERR_INVALID_ARG;
  if ((dev_ptr == nullptr) != (bytes == 0)) return FS_ERR_INVALID_ARG;
  if ((uintptr_t)dev_ptr % 256) return FS_ERR_INVALID_ARG;
  const fs_status rc = drop_workspace(h);
  if (rc != FS_OK) return rc;
  h->ws = dev_ptr; h->ws_bytes = bytes; h->ws_owned = (dev_ptr == nullptr);
  return FS_OK;
}

}  // extern "C"

// The apply of the column layout (declared in handle.h).
fs_status fs::apply_cols(fs_sketch_t h, const void* A, int64_t lda, int64_t n, void* out, int64_t ldo,
                         fs_dtype dt, void* stream, const fs::ScratchSource& src) {
  if (!h || n < 0 || !valid_dtype(dt)) return FS_ERR_INVALID_ARG;
  if (n == 0) return FS_OK;
  if (!A || !out || lda < n || ldo < n) return FS_ERR_INVALID_ARG;
  if (n > 0x7fffffff || lda > ((int64_t)1 << 40) || ldo > ((int64_t)1 << 40)) return FS_ERR_INVALID_ARG;
  const size_t esz = dt == FS_F32 ? 4 : 2;
  if ((uintptr_t)A % esz || (uintptr_t)out % esz) return FS_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;

  // whether the kernels will get the orbit table of the wiring (it shapes their plan)
  const bool with_orbit = h->kind == FS_KIND_BLOCKPERM && fs::mfma_wants_orbit(h->p) &&
                          (!src.external || 2 * (size_t)h->p.M * sizeof(uint32_t) <= src.orbit_bytes);
  int variant = FS_VARIANT_GENERIC;
  fs::Workspace need;
  fs::mm::Plan plan;
  fs_status rc = FS_OK;
  if (h->kind != FS_KIND_BLOCKPERM) {
    rc = other_kind(h, A, lda, n, dt, &need);
    if (rc != FS_OK) return rc;
  } else if (h->variant != FS_VARIANT_GENERIC) {
    plan = fs::plan_mfma(h->p, A, lda, n, dt, with_orbit, SIZE_MAX, h->variant == FS_VARIANT_AUTO);
    if (h->variant == FS_VARIANT_MFMA && !plan.ok) return FS_ERR_UNSUPPORTED;
    if (plan.ok) {
      variant = FS_VARIANT_MFMA;
      need = fs::mfma_workspace(h->p, plan);
    }
  }
  void* ws = nullptr;
  size_t ws_bytes = src.plane_bytes;
  const uint32_t* orbit = nullptr;
  if (src.external && need.floor > src.plane_bytes) return FS_ERR_ALLOC;  // beyond the supplied memory: nothing is launched
  if (!src.external) {
    rc = ensure_workspace(h, need, st);
    if (rc != FS_OK) return rc;
    ws_bytes = h->ws_bytes;
  }
  if (variant == FS_VARIANT_MFMA && need.want > ws_bytes)  // less than it would like: a split that fits
    plan = fs::plan_mfma(h->p, A, lda, n, dt, with_orbit, ws_bytes, h->variant == FS_VARIANT_AUTO);
  const ProfSet prof = next_events(h, st);
  const fs::EventPair ev = prof.kernel;
  if (src.external) {
    ws = src.planes;
    // such memory is shared between handles: the table of this handle's wiring is rebuilt on every
    // call (a wiring too long for the table's room runs without one: the kernels then skip the
    // orbit-ordered modes)
    if (variant == FS_VARIANT_MFMA && with_orbit) {
      const hipError_t e = fs::launch_orbit(h->p, src.orbit, st);
      if (e != hipSuccess) return hip_fail(h, e);
      orbit = src.orbit;
    }
  } else {
    if (variant == FS_VARIANT_MFMA) {
      rc = ensure_orbit(h, st);
      if (rc != FS_OK) return rc;
    }
    ws = h->ws;
    orbit = h->orbit;
  }

  hipError_t e;
  int mode = 0;
  const char* what = "";
  if (h->kind == FS_KIND_SJLT_SCATTER) {
    e = fs::launch_scatter(h->p, A, lda, n, out, ldo, dt, ws, st, ev);
    what = "scatter_kernel";
  } else if (h->kind == FS_KIND_GAUSS_DENSE) {
    e = fs::launch_gauss(h->dense, h->dense_half, h->dense_scratch, h->p.k, h->p.d, A, lda, n, out, ldo, dt, st, ev, h->last_kernel,
                         sizeof(h->last_kernel));
  } else if (h->kind == FS_KIND_BLOCKROW) {
    e = fs::launch_blockrow(h->p, A, lda, n, out, ldo, dt, st, ev);
    what = "blockrow_kernel";
  } else if (variant == FS_VARIANT_MFMA) {
    mode = fs::mfma_mode(plan);
    e = fs::launch_mfma(plan, h->p, A, lda, n, out, ldo, dt, ws, ws_bytes, orbit, st, ev, h->last_kernel,
                        sizeof(h->last_kernel));
  } else {
    e = fs::launch_generic(h->p, A, lda, n, out, ldo, dt, st, ev);
    what = "generic_kernel";
  }
  if (what[0]) snprintf(h->last_kernel, sizeof(h->last_kernel), "%s", what);
  if (prof.end) (void)hipEventRecord(prof.end, st);
  h->last_variant = variant;
  h->last_mode = mode;
  if (e != hipSuccess) return hip_fail(h, e);
  return FS_OK;
}

extern "C" {

fs_status fs_sketch_apply_ld(fs_sketch_t h, const void* A, int64_t lda, int64_t n, void* out,
                             int64_t ldo, fs_dtype dt, void* stream) {
  return fs::apply_cols(h, A, lda, n, out, ldo, dt, stream, fs::ScratchSource{});
}

fs_status fs_sketch_prepare(fs_sketch_t h, void* stream) {
  if (!h) return FS_ERR_INVALID_ARG;
  if (h->kind != FS_KIND_BLOCKPERM) return FS_OK;
  return ensure_orbit(h, (hipStream_t)stream);
}

fs_status fs_sketch_apply_rows(fs_sketch_t h, const void* G, int64_t ldg, int64_t n, void* out,
                               int64_t ldo, fs_dtype dt, void* stream) {
  if (!h || n < 0 || !valid_dtype(dt)) return FS_ERR_INVALID_ARG;
  if (n == 0) return FS_OK;
  if (!G || !out || ldg < h->p.d || ldo < h->p.k) return FS_ERR_INVALID_ARG;
  if (n > 0x7fffffff || ldg > ((int64_t)1 << 40) || ldo > ((int64_t)1 << 40)) return FS_ERR_INVALID_ARG;
  const size_t esz = dt == FS_F32 ? 4 : 2;
  if ((uintptr_t)G % esz || (uintptr_t)out % esz) return FS_ERR_INVALID_ARG;
  if (h->kind != FS_KIND_BLOCKPERM) return FS_ERR_UNSUPPORTED;
  fs::mm::RowsPlan plan;
  if (h->variant != FS_VARIANT_GENERIC) plan = fs::plan_rows(h->p, G, ldg, n, dt, SIZE_MAX, h->variant == FS_VARIANT_AUTO);
  if (h->variant == FS_VARIANT_MFMA && !plan.ok) return FS_ERR_UNSUPPORTED;
  const bool use_mfma = plan.ok;
  hipStream_t st = (hipStream_t)stream;
  fs_status rc = FS_OK;
  if (use_mfma) {
    rc = ensure_workspace(h, fs::Workspace{plan.ws_floor, rows_want(plan)}, st);
    if (rc != FS_OK) return rc;
    if (plan.ws > h->ws_bytes) plan = fs::plan_rows(h->p, G, ldg, n, dt, h->ws_bytes, h->variant == FS_VARIANT_AUTO);  // a split that fits
  }
  const ProfSet prof = next_events(h, st);
  const fs::EventPair ev = prof.kernel;
  if (!use_mfma) {
    const hipError_t e = fs::launch_generic_rows(h->p, G, ldg, n, out, ldo, dt, st, ev);
    if (prof.end) (void)hipEventRecord(prof.end, st);
    snprintf(h->last_kernel, sizeof(h->last_kernel), "generic_rows_kernel");
    h->last_variant = FS_VARIANT_GENERIC;
    h->last_mode = 0;
    if (e != hipSuccess) return hip_fail(h, e);
    return FS_OK;
  }
  rc = ensure_orbit(h, st);  // the gather-reduction walks the wiring through this table
  if (rc != FS_OK) return rc;
  const hipError_t e = fs::launch_rows(plan, h->p, G, ldg, n, out, ldo, dt, h->ws, h->ws_bytes, h->orbit, st, ev);
  if (prof.end) (void)hipEventRecord(prof.end, st);
  snprintf(h->last_kernel, sizeof(h->last_kernel), "%s", plan.few.ok ? "vector_kernel" : "rows_kernel");
  h->last_variant = FS_VARIANT_MFMA;
  h->last_mode = plan.out_stat ? 1 : 2;
  if (e != hipSuccess) return hip_fail(h, e);
  return FS_OK;
}

fs_status fs_sketch_rows_workspace_bytes(fs_sketch_t h, int64_t n, fs_dtype dt, size_t* bytes) {
  if (!h || !bytes || n < 0 || !valid_dtype(dt)) return FS_ERR_INVALID_ARG;
  *bytes = 0;
  if (n == 0 || h->kind != FS_KIND_BLOCKPERM) return FS_OK;
  const size_t esz = dt == FS_F32 ? 4 : 2;
  const int64_t ld = (h->p.d + 7) & ~(int64_t)7;  // a well-aligned call: packed rows rounded to 16 bytes
  if (34 * ld * (int64_t)esz >= ((int64_t)1 << 31)) return FS_OK;
  for (const bool vector : {false, true}) {
    const size_t want = rows_want(fs::plan_rows(h->p, (const void*)(uintptr_t)256, ld, n, dt, SIZE_MAX, vector));
    if (want > *bytes) *bytes = want;
  }
  return FS_OK;
}

fs_status fs_sketch_plan(fs_sketch_t h, const void* A, int64_t ld, int64_t n, fs_dtype dt, int32_t rows,
                         int32_t* variant, int32_t* mode, int32_t* flags, size_t* workspace_bytes) {
  if (!h || n < 0 || !valid_dtype(dt) || (rows != 0 && rows != 1)) return FS_ERR_INVALID_ARG;
  const size_t esz = dt == FS_F32 ? 4 : 2;
  if (!A || (uintptr_t)A % esz || ld < (rows ? h->p.d : n) || n > 0x7fffffff || ld > ((int64_t)1 << 40))
    return FS_ERR_INVALID_ARG;
  if (rows && h->kind != FS_KIND_BLOCKPERM) return FS_ERR_UNSUPPORTED;
  int v = FS_VARIANT_GENERIC, m = 0, f = 0;
  size_t ws = 0;
  if (n > 0 && h->kind == FS_KIND_BLOCKPERM) {
    if (rows) {
      const fs::mm::RowsPlan pl = fs::plan_rows(h->p, A, ld, n, dt, SIZE_MAX, h->variant == FS_VARIANT_AUTO);
      if (h->variant == FS_VARIANT_MFMA && !pl.ok) return FS_ERR_UNSUPPORTED;
      if (pl.ok && h->variant != FS_VARIANT_GENERIC) {
        v = FS_VARIANT_MFMA;
        m = pl.out_stat ? 1 : 2;
        f = (pl.vec ? 0 : FS_PLAN_ELEMENT_LOADS) | (pl.nsub > 1 ? FS_PLAN_ROW_SLICES : 0) |
            (pl.groups > 1 ? FS_PLAN_SLOT_GROUPS : 0) | (pl.zsplit > 1 || pl.nw > 1 ? FS_PLAN_SPLIT : 0);
        ws = rows_want(pl);
      }
    } else {
      const fs::mm::Plan pl = fs::plan_mfma(h->p, A, ld, n, dt, fs::mfma_wants_orbit(h->p), SIZE_MAX, h->variant == FS_VARIANT_AUTO);
      if (h->variant == FS_VARIANT_MFMA && !pl.ok) return FS_ERR_UNSUPPORTED;
      if (pl.ok && h->variant != FS_VARIANT_GENERIC) {
        v = FS_VARIANT_MFMA;
        m = fs::mfma_mode(pl);
        f = fs::mfma_flags(pl);
        ws = fs::mfma_workspace(h->p, pl).want;
      }
    }
  } else if (n > 0) {
    fs::Workspace need;
    const fs_status rc = other_kind(h, A, ld, n, dt, &need);
    if (rc != FS_OK) return rc;
    ws = need.want;
  }
  if (variant) *variant = v;
  if (mode) *mode = m;
  if (flags) *flags = f;
  if (workspace_bytes) *workspace_bytes = ws;
  return FS_OK;
}

fs_status fs_sketch_apply(fs_sketch_t h, const void* A, int64_t lda, int64_t n, void* out,
                          fs_dtype dt, void* stream) {
  return fs_sketch_apply_ld(h, A, lda, n, out, n, dt, stream);
}

fs_status fs_sketch_export(fs_sketch_t h, int32_t* rows, int8_t* signs, void* stream) {
  if (!h || !rows || !signs) return FS_ERR_INVALID_ARG;
  if (h->kind == FS_KIND_GAUSS_DENSE) return FS_ERR_UNSUPPORTED;
  hipError_t e = h->kind == FS_KIND_BLOCKROW
                     ? fs::launch_blockrow_export(h->p, rows, signs, (hipStream_t)stream)
                     : fs::launch_export(h->p, rows, signs, (hipStream_t)stream);
  if (e != hipSuccess) return hip_fail(h, e);
  return FS_OK;
}

fs_status fs_sketch_export_dense(fs_sketch_t h, float* S_dense, void* stream) {
  if (!h || !S_dense) return FS_ERR_INVALID_ARG;
  if (h->kind != FS_KIND_GAUSS_DENSE) return FS_ERR_UNSUPPORTED;
  hipError_t e = hipMemcpyAsync(S_dense, h->dense, (size_t)h->p.k * h->p.d * sizeof(float),
                                hipMemcpyDeviceToDevice, (hipStream_t)stream);
  if (e != hipSuccess) return hip_fail(h, e);
  return FS_OK;
}

}  // extern "C"
