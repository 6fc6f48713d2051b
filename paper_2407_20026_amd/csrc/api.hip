// C ABI and host runtime of libhipsso: problem lifecycle, device buffers, launch sequencing on
// the problem's stream, error mapping and per-stage timing.
#include <new>
#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <mutex>
#include <system_error>
#include <thread>
#include <vector>

#include "sso_internal.h"

using namespace sso;

// The static scratch of sso_size_objective_noalloc: one copy per device, for the life of the
// process.  In host code `scratch` names a host-side stand-in, not device memory; its device
// address on each GPU comes from hipGetSymbolAddress (taken once per device, with that device
// current) and only that address is ever handed to kernels.
static __device__ __align__(256) double scratch[SSO_NOALLOC_SCRATCH_BYTES / sizeof(double)];
static_assert(SSO_NOALLOC_MAX_QUADS * 15 + 2 * 1024 <=
                  (int64_t)(SSO_NOALLOC_SCRATCH_BYTES / sizeof(double)),
              "the no-allocation scratch holds the partials and 15 values per quad");

// A block pattern shared by the problems of one topology (sso_problem_create_like); the last
// problem to be destroyed frees it.
struct SharedPattern {
  Pattern pat;
  std::atomic<int> refs{1};
  // The direct solver's plan: built by a thread of its own while the creating call and the ones
  // after it go on (or by the first solve that may use it), uploaded by that solve.  Under the
  // mutex until READY or REFUSED, read-only afterwards; the host tables stay until the pattern
  // ends, so the upload is not waited for.
  std::mutex direct_mutex;
  enum { DIRECT_UNKNOWN, DIRECT_BUILT, DIRECT_READY, DIRECT_REFUSED };
  std::atomic<int> direct_state{DIRECT_UNKNOWN};
  std::vector<int32_t> brow, bcol;       // the pattern on the host, until the plan is built
  std::thread builder;
  bool builder_started = false;          // set by the creating call
  std::atomic<bool> builder_done{false};
  std::atomic<bool> unwanted{false};     // the last problem has ended: the builder may stop
  bool built = false;                    // the builder's result, read after joining it
  DirectPlan plan;
  DirectArgs tables{};                   // device tables, in the pattern's arena
  hipEvent_t uploaded = nullptr;         // orders other streams after the upload
  ~SharedPattern() {
    unwanted = true;
    if (builder.joinable()) builder.join();
    if (uploaded) (void)hipEventDestroy(uploaded);
  }
};

struct sso_problem {
  hipStream_t s = nullptr;
  Mesh m;
  Pattern pat;                  // the pattern's arrays (owned through `shared`)
  SharedPattern* shared = nullptr;
  Arena mem;                    // chunks holding the problem's own device buffers
  sso_options opt;
  int64_t n_coo = 0;
  double* coo = nullptr;
  double* qarea = nullptr;
  double* K = nullptr;
  double* Dinv = nullptr;
  double* B = nullptr;          // K times the block-Jacobi inverse (single-reduction PCG)
  float* B32 = nullptr;
  float* K32 = nullptr;         // mixed precision copies (allocated on first mixed solve)
  float* Dinv32 = nullptr;
  double* f = nullptr;          // right-hand side of the masked system (lifted when prescribed)
  double* fm = nullptr;         // applied load on the free DOFs, when displacements are prescribed
  double* u = nullptr;
  double* lam = nullptr;
  double* rhs = nullptr;
  double* gbeam = nullptr;
  double* gquad = nullptr;
  double* gw = nullptr;         // size objective: volume terms [14 n_quads], shares [n_quads],
  double* wv = nullptr;         //   partials (allocated on first use)
  double* xpart = nullptr;
  double* d_scal = nullptr;     // small device scalars (dot products, residual norms)
  double* h_scal = nullptr;     // pinned slot, what the stream leaves for the host: ||r||^2,
                                // ||b||^2 (or a dot product), the direct solver's flag and the
                                // elements' errors; [4, 6) the size objective's sums
  unsigned* d_err = nullptr;
  unsigned* h_err = nullptr;    // host mirror of d_err, in the same slot
  PcgWork w;
  int32_t* row_ptr = nullptr;   // scalar CSR view (built on demand)
  int32_t* col = nullptr;
  int32_t* perm = nullptr;
  int32_t* seg = nullptr;
  bool scalar_view = false;     // built
  bool direct = false;          // the last solve chose the direct solver
  bool factored = false;        // its factor is that of the current K
  bool unchecked = false;       // the elements' errors are still to be looked at
  DirectArgs da{};              // its arrays (allocated on first use)
  int direct_steps = 0;         // substitutions of the last solve
  double direct_rr = -1.0, direct_bb = 0.0;   // its last true residual and load, squared norms
  bool direct_done = false;     // begun solve: nothing left to iterate
  bool solved = false;
  bool in_batch = false;        // started with sso_solve_begin, not yet finished
  bool batch_pending = false;   // listed in a multi-problem launch not yet waited for
  hipEvent_t ev_move = nullptr; // orders a new stream after the old one (sso_problem_set_stream)
  int solver_used = SSO_SOLVER_STANDARD;   // recurrences of the last solve
  PcgDesc<double> desc{};       // its descriptor in multi-problem launches (standard / fused)
  FusedDesc<double> fdesc{};
  MixedState ms;                // mixed precision begun with sso_solve_begin
  hipEvent_t ev[6] = {};
  int device = 0;               // the device current at creation (holds the problem's memory)
  int64_t bytes = 0;            // device memory allocated for the problem (sso_problem_bytes)
};

struct sso_batch {
  hipStream_t s = nullptr;
  BatchWork bw;
  bool pending = false;                  // a launch not yet waited for
  std::vector<sso_problem*> listed;      // its problem list, in the caller's order
  std::vector<int> idx[5];               // positions in that list by launch kind
  DirectBatch db;                        // the direct solver's part of a launch
  std::vector<int> direct;               // its positions in the list
  int n_iter = 0;                        // iterations asked for
  std::vector<int> steps;                // of them the direct solver's, by position
  // sso_batch_profile: timing samples of the FP64 standard iterations
  int prof_every = 0, prof_span = 0;
  int64_t prof_calls = 0;                // launches that could be sampled so far
  int armed = 0;                         // iterations timed in the pending launch (0: none)
  std::vector<int> jn0;                  // its FP64 standard problems' next iteration index
  double prof_us = 0.0, prof_bytes = 0.0, prof_bytes_read = 0.0;
  int64_t prof_iters = 0;
};

namespace {

constexpr int MAX_DEVICES = 64;

// Most device memory that the direct solver's numeric arrays may take: what the fill of an open
// surface structure (grid-shell or shell of any outline) or of a chain needs, which grows as n log
// n.  Members joined in space fill more (a solid lattice of 20 x 20 x 20 nodes three times this) and
// also cost more operations than PCG's few hundred iterations there; PCG keeps them.  It is a bound
// on memory, not on time: closed surfaces lie close to it on either side (a tube of 20 x 20 quads
// takes 9.6 MB against 9.5 and a torus of 40 x 40 42.9 against 41.3, tubes of 40 and 100 a side are
// taken).  The serving loops' admission bounds a request's memory by the same formula.
double direct_max_bytes(const Mesh& m) {
  const double n = m.n_nodes;
  return 288.0 * (std::log2(n + 1.0) + 1.0) * (1.2 * n + 2.3 * m.n_beams + 6.3 * m.n_quads) +
         1048576.0;
}

sso_options default_options() {
  sso_options o;
  o.precision = SSO_PREC_FP64;
  o.rtol = 1e-8;
  o.max_it = 200000;
  o.refine_steps = 20;
  o.profile_every = 0;
  o.inner_rtol = 0.0;
  o.solver = SSO_SOLVER_AUTO;
  o.inner_max_it = 0;
  return o;
}

bool options_ok(const sso_options& o) {
  return (o.precision == SSO_PREC_FP64 || o.precision == SSO_PREC_MIXED ||
          o.precision == SSO_PREC_AUTO) && o.rtol >= 0.0 &&
         o.max_it > 0 && o.refine_steps >= 0 && o.profile_every >= 0 && o.inner_rtol >= 0.0 &&
         o.inner_rtol < 1.0 && o.solver >= SSO_SOLVER_AUTO && o.solver <= SSO_SOLVER_WG &&
         o.inner_max_it >= 0 && !(o.solver == SSO_SOLVER_WG && o.precision == SSO_PREC_MIXED);
}

// The precision a problem runs in: AUTO resolves by the size of its FP64 K.
bool mixed_for(const sso_options& o, int64_t n_blocks) {
  if (o.solver == SSO_SOLVER_WG) return false;   // the one-workgroup solver runs in FP64
  if (o.precision == SSO_PREC_AUTO) {
    const double k_bytes = 288.0 * (double)n_blocks;
    return k_bytes >= (o.rtol <= SSO_AUTO_TIGHT_RTOL ? SSO_AUTO_MIXED_TIGHT_K_BYTES
                                                    : SSO_AUTO_MIXED_K_BYTES);
  }
  return o.precision == SSO_PREC_MIXED;
}

__global__ void k_fill(int64_t n, double v, double* out) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) out[i] = v;
}


int map_hip(hipError_t e) {
  if (e == hipSuccess) return SSO_OK;
  if (e == hipErrorOutOfMemory) return SSO_ENOMEM;
  return SSO_EHIP;
}

#define TRY_HIP(x)                     \
  do {                                 \
    hipError_t e_ = (x);               \
    if (e_ != hipSuccess) return map_hip(e_); \
  } while (0)

float elapsed_us(hipEvent_t a, hipEvent_t b) {
  float ms = 0.f;
  if (hipEventElapsedTime(&ms, a, b) != hipSuccess) return 0.f;
  return 1000.f * ms;
}

// Pinned host memory that kernels write a problem's scalars into, so that the host reads them after
// a synchronisation without a copy: slots of 128 bytes from one block for the life of the process
// (pinning and unpinning cost up to a millisecond each), more from blocks of their own.
constexpr int PIN_SLOTS = 4096;
constexpr size_t PIN_DOUBLES = 16;
struct PinnedSlots {
  std::mutex mu;
  double* block = nullptr;
  std::vector<int> idle;
};
PinnedSlots pinned_slots;

hipError_t pinned_take(double** out) {
  *out = nullptr;
  {
    std::lock_guard<std::mutex> lock(pinned_slots.mu);
    if (!pinned_slots.block) {
      try {
        pinned_slots.idle.reserve(PIN_SLOTS);
      } catch (...) {
        return hipErrorOutOfMemory;
      }
      const hipError_t e =
          hipHostMalloc(reinterpret_cast<void**>(&pinned_slots.block),
                        sizeof(double) * PIN_DOUBLES * PIN_SLOTS, hipHostMallocPortable);
      if (e != hipSuccess) return e;
      for (int i = PIN_SLOTS - 1; i >= 0; --i) pinned_slots.idle.push_back(i);
    }
    if (!pinned_slots.idle.empty()) {
      *out = pinned_slots.block + PIN_DOUBLES * (size_t)pinned_slots.idle.back();
      pinned_slots.idle.pop_back();
    }
  }
  if (!*out) {
    const hipError_t e = hipHostMalloc(reinterpret_cast<void**>(out),
                                       sizeof(double) * PIN_DOUBLES, hipHostMallocPortable);
    if (e != hipSuccess) return e;
  }
  std::memset(*out, 0, sizeof(double) * PIN_DOUBLES);
  return hipSuccess;
}

void pinned_give(double* p) {
  if (!p) return;
  std::lock_guard<std::mutex> lock(pinned_slots.mu);
  if (p >= pinned_slots.block && p < pinned_slots.block + PIN_DOUBLES * PIN_SLOTS)
    pinned_slots.idle.push_back((int)((p - pinned_slots.block) / (ptrdiff_t)PIN_DOUBLES));
  else
    (void)hipHostFree(p);
}

// Makes a device current for as long as it lives.
struct OnDevice {
  int back = -1;
  explicit OnDevice(int device) {
    int cur = 0;
    if (hipGetDevice(&cur) == hipSuccess && cur != device && hipSetDevice(device) == hipSuccess)
      back = cur;
  }
  ~OnDevice() {
    if (back >= 0) (void)hipSetDevice(back);
  }
  OnDevice(const OnDevice&) = delete;
  OnDevice& operator=(const OnDevice&) = delete;
};

void free_problem(sso_problem* p) {
  if (!p) return;
  // the null stream is the current device's, and this may run while any is (a garbage collector)
  const OnDevice here(p->device);
  hipStream_t s = p->s;
  Mesh& m = p->m;
  for (void* q : {(void*)m.xyz, (void*)m.fixed, (void*)m.f_nodal, (void*)m.beam_nodes,
                  (void*)m.beam_prop, (void*)m.quad_nodes, (void*)m.quad_prop,
                  (void*)m.quad_scale, (void*)p->coo, (void*)p->qarea, (void*)p->K,
                  (void*)p->Dinv, (void*)p->f, (void*)p->K32, (void*)p->Dinv32, (void*)p->B, (void*)p->B32, (void*)p->u,
                  (void*)p->lam, (void*)p->rhs, (void*)p->gbeam, (void*)p->gquad,
                  (void*)p->d_scal, (void*)p->d_err, (void*)p->row_ptr, (void*)p->col,
                  (void*)p->perm, (void*)p->seg, (void*)m.u_presc, (void*)p->fm,
                  (void*)p->gw, (void*)p->wv, (void*)p->xpart})
    dev_release(q, &p->mem, s);
  pcg_free(p->w, &p->mem, s);
  for (auto& e : p->ev)
    if (e) (void)hipEventDestroy(e);
  if (p->ev_move) (void)hipEventDestroy(p->ev_move);
  // the chunks are idle once the stream is: for the next problem, unless the device has failed
  const bool idle = hipStreamSynchronize(s) == hipSuccess;
  if (p->shared) {
    if (p->shared->refs.fetch_sub(1) == 1) {   // the last problem of this topology
      p->shared->unwanted = true;
      if (p->shared->builder.joinable()) p->shared->builder.join();
      free_pattern(p->shared->pat, s, idle);
      delete p->shared;
    }
  } else {
    free_pattern(p->pat, s, idle);
  }
  if (idle)
    arena_recycle(p->mem, s);
  else
    arena_free(p->mem, s);
  if (idle) pinned_give(p->h_scal);   // else a kernel could still write it
  delete p;
}

// Debug mode (HIPSSO_DEBUG set, and not "0", when a problem is created): the block pattern, the
// sort permutation and the padded rows built on the GPU are copied to the host and checked
// invariant by invariant (check_pattern); a failure is reported on stderr and as SSO_EINVAL.
bool debug_mode() {
  const char* v = std::getenv("HIPSSO_DEBUG");
  return v && *v && !(v[0] == '0' && v[1] == '\0');
}

int debug_check_pattern(sso_problem* p) {
  const Mesh& m = p->m;
  const Pattern& pat = p->pat;
  hipStream_t s = p->s;
  const int n = m.n_nodes;
  const int64_t nb = pat.n_blocks, nc = pat.n_bcoo;
  std::vector<int32_t> brow(n + 1), bcol(nb), bseg(nb + 1), bperm(nc), bslot(nc), bdiag(n),
      bsrow(nb), bsym(2 * nb), est(n + 1), ell((int64_t)n * pat.ell_w), bn(2 * (int64_t)m.n_beams),
      qn(4 * (int64_t)m.n_quads);
  auto get = [&](std::vector<int32_t>& v, const int32_t* src) {
    return v.empty() ? hipSuccess
                     : hipMemcpyAsync(v.data(), src, sizeof(int32_t) * v.size(),
                                      hipMemcpyDeviceToHost, s);
  };
  TRY_HIP(get(brow, pat.brow_ptr));
  TRY_HIP(get(bcol, pat.bcol));
  TRY_HIP(get(bseg, pat.bseg));
  TRY_HIP(get(bperm, pat.bperm));
  TRY_HIP(get(bslot, pat.bslot));
  TRY_HIP(get(bdiag, pat.bdiag));
  TRY_HIP(get(bsrow, pat.bsrow));
  TRY_HIP(get(bsym, pat.bsym));
  TRY_HIP(get(est, pat.estart));
  TRY_HIP(get(ell, pat.bcol_ell));
  TRY_HIP(get(bn, m.beam_nodes));
  TRY_HIP(get(qn, m.quad_nodes));
  TRY_HIP(hipStreamSynchronize(s));
  HostPattern h;
  h.n_nodes = n;
  h.n_beams = m.n_beams;
  h.n_quads = m.n_quads;
  h.ell_w = pat.ell_w;
  h.n_blocks = nb;
  h.n_bcoo = nc;
  h.brow_ptr = brow.data();
  h.bcol = bcol.data();
  h.bseg = bseg.data();
  h.bperm = bperm.data();
  h.bslot = bslot.data();
  h.bdiag = bdiag.data();
  h.bsrow = bsrow.data();
  h.bsym = bsym.data();
  h.estart = est.data();
  h.bcol_ell = ell.data();
  h.beam_nodes = bn.data();
  h.quad_nodes = qn.data();
  char msg[256];
  if (check_pattern(h, msg, sizeof msg) != 0) {
    std::fprintf(stderr, "hipsso debug: %s\n", msg);
    return SSO_EINVAL;
  }
  return SSO_OK;
}

// 1 in *err where two connectivity arrays of n entries differ.
__global__ void k_same_topology(int64_t n, const int32_t* a, const int32_t* b, unsigned* err) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n && a[i] != b[i]) atomicOr(err, ERR_TOPO);
}

// Builds the direct solver's plan from the pattern's host copy; never throws.
void make_plan(SharedPattern* sh, double max_bytes) {
  try {
    sh->built = build_direct_plan((int)sh->brow.size() - 1, sh->brow.data(), sh->bcol.data(),
                                  max_bytes, sh->plan, &sh->unwanted);
  } catch (...) {   // out of host memory: PCG needs none of this
    sh->built = false;
  }
}

void start_plan(SharedPattern* sh, const Mesh& m) {
  const double max_bytes = direct_max_bytes(m);
  try {
    sh->builder = std::thread([sh, max_bytes] {
      make_plan(sh, max_bytes);
      sh->builder_done = true;
    });
    sh->builder_started = true;
  } catch (...) {   // no thread to be had: the first solve builds it
  }
}

// Enqueues the copy of the pattern to the host for a plan; left empty where host memory is short.
int fetch_pattern(sso_problem* p) {
  SharedPattern* sh = p->shared;
  try {
    sh->brow.resize(p->m.n_nodes + 1);
    sh->bcol.resize(p->pat.n_blocks);
  } catch (...) {
    sh->brow = {};
    sh->bcol = {};
    return SSO_OK;
  }
  TRY_HIP(hipMemcpyAsync(sh->brow.data(), p->pat.brow_ptr, sizeof(int32_t) * sh->brow.size(),
                         hipMemcpyDeviceToHost, p->s));
  TRY_HIP(hipMemcpyAsync(sh->bcol.data(), p->pat.bcol, sizeof(int32_t) * sh->bcol.size(),
                         hipMemcpyDeviceToHost, p->s));
  return SSO_OK;
}

// scratch: buffers that only the creation uses, idle once it has synchronised the stream.
int create_impl(const sso_mesh* mesh, const sso_options* opts, hipStream_t stream,
                sso_problem* p, const sso_problem* like, Arena& scratch) {
  p->s = stream;
  TRY_HIP(hipGetDevice(&p->device));
  p->opt = opts ? *opts : default_options();
  Mesh& m = p->m;
  m.n_nodes = mesh->n_nodes;
  m.n_beams = mesh->n_beams;
  m.n_quads = mesh->n_quads;
  m.unit_weight = mesh->unit_weight;
  m.surface_load = mesh->surface_load;
  const int64_t nn = m.n_nodes, nb = m.n_beams, nq = m.n_quads;
  hipStream_t s = p->s;
  TRY_HIP(dev_alloc(&m.xyz, 3 * nn, s));
  TRY_HIP(dev_alloc(&m.fixed, 6 * nn, s));
  TRY_HIP(dev_alloc(&m.f_nodal, 6 * nn, s));
  TRY_HIP(dev_alloc(&m.beam_nodes, 2 * nb, s));
  TRY_HIP(dev_alloc(&m.beam_prop, 6 * nb, s));
  TRY_HIP(dev_alloc(&m.quad_nodes, 4 * nq, s));
  TRY_HIP(dev_alloc(&m.quad_prop, 5 * nq, s));
  TRY_HIP(dev_alloc(&m.quad_scale, nq, s));
  if (mesh->u_prescribed) {
    TRY_HIP(dev_alloc(&m.u_presc, 6 * nn, s));
    TRY_HIP(hipMemcpyAsync(m.u_presc, mesh->u_prescribed, sizeof(double) * 6 * nn,
                           hipMemcpyDeviceToDevice, s));
    TRY_HIP(dev_alloc(&p->fm, 6 * nn, s));
  }
  TRY_HIP(hipMemcpyAsync(m.xyz, mesh->xyz, sizeof(double) * 3 * nn, hipMemcpyDeviceToDevice, s));
  TRY_HIP(hipMemcpyAsync(m.fixed, mesh->fixed, 6 * nn, hipMemcpyDeviceToDevice, s));
  TRY_HIP(hipMemcpyAsync(m.f_nodal, mesh->f_nodal, sizeof(double) * 6 * nn,
                         hipMemcpyDeviceToDevice, s));
  if (nb) {
    TRY_HIP(hipMemcpyAsync(m.beam_nodes, mesh->beam_nodes, sizeof(int32_t) * 2 * nb,
                           hipMemcpyDeviceToDevice, s));
    TRY_HIP(hipMemcpyAsync(m.beam_prop, mesh->beam_prop, sizeof(double) * 6 * nb,
                           hipMemcpyDeviceToDevice, s));
  }
  if (nq) {
    TRY_HIP(hipMemcpyAsync(m.quad_nodes, mesh->quad_nodes, sizeof(int32_t) * 4 * nq,
                           hipMemcpyDeviceToDevice, s));
    TRY_HIP(hipMemcpyAsync(m.quad_prop, mesh->quad_prop, sizeof(double) * 5 * nq,
                           hipMemcpyDeviceToDevice, s));
    if (mesh->quad_scale) {
      TRY_HIP(hipMemcpyAsync(m.quad_scale, mesh->quad_scale, sizeof(double) * nq,
                             hipMemcpyDeviceToDevice, s));
    } else {
      hipLaunchKernelGGL(k_fill, dim3((unsigned)((nq + 255) / 256)), dim3(256), 0, s, nq, 1.0,
                         m.quad_scale);
      TRY_HIP(hipGetLastError());
    }
  }
  TRY_HIP(dev_alloc(&p->d_err, 1, s));
  TRY_HIP(dev_alloc(&p->d_scal, 8, s));
  TRY_HIP(pinned_take(&p->h_scal));
  p->h_err = reinterpret_cast<unsigned*>(p->h_scal + 8);
  TRY_HIP(hipMemsetAsync(p->d_err, 0, sizeof(unsigned), s));
  *p->h_err = 0;
  if (like) {
    // the pattern of `like`, once its connectivity is shown to be this mesh's (checked with the
    // other errors at the end of creation)
    p->pat = like->pat;
    p->shared = like->shared;
    p->shared->refs.fetch_add(1);
    const int64_t nbn = 2 * (int64_t)nb, nqn = 4 * (int64_t)nq;
    if (nbn)
      hipLaunchKernelGGL(k_same_topology, dim3((unsigned)((nbn + 255) / 256)), dim3(256), 0, s,
                         nbn, m.beam_nodes, like->m.beam_nodes, p->d_err);
    if (nqn)
      hipLaunchKernelGGL(k_same_topology, dim3((unsigned)((nqn + 255) / 256)), dim3(256), 0, s,
                         nqn, m.quad_nodes, like->m.quad_nodes, p->d_err);
    TRY_HIP(hipGetLastError());
  } else {
    {
      AllocScope ps(&p->bytes, &p->pat.mem);   // the pattern outlives this problem if shared
      TRY_HIP(build_pattern(m, p->pat, p->d_err, s, p->h_err, scratch));
    }
    if (*p->h_err) return SSO_EINVAL;
    p->shared = new (std::nothrow) SharedPattern();
    if (!p->shared) return SSO_ENOMEM;
    p->shared->pat = p->pat;
    if (p->opt.solver == SSO_SOLVER_AUTO) {
      // the pattern for the direct solver's plan (its build starts after the synchronisation below)
      const int st = fetch_pattern(p);
      if (st != SSO_OK) return st;
    }
    if (debug_mode()) {
      const int st = debug_check_pattern(p);
      if (st != SSO_OK) return st;
    }
  }
  p->n_coo = 144 * nb + 576 * nq;
  TRY_HIP(dev_alloc(&p->coo, p->n_coo, s));
  TRY_HIP(dev_alloc(&p->qarea, nq, s));
  TRY_HIP(dev_alloc(&p->K, 36 * p->pat.n_blocks, s));
  TRY_HIP(dev_alloc(&p->Dinv, dinv_packed_len(nn), s));
  TRY_HIP(dev_alloc(&p->f, 6 * nn, s));
  TRY_HIP(dev_alloc(&p->u, 6 * nn, s));
  TRY_HIP(dev_alloc(&p->lam, 6 * nn, s));
  TRY_HIP(dev_alloc(&p->rhs, 6 * nn, s));
  TRY_HIP(dev_alloc(&p->gbeam, 6 * nb, s));
  TRY_HIP(dev_alloc(&p->gquad, 14 * nq, s));
  TRY_HIP(pcg_alloc(p->w, nn, mixed_for(p->opt, p->pat.n_blocks), s));
  for (auto& e : p->ev) TRY_HIP(hipEventCreate(&e));
  if (like) TRY_HIP(hipMemcpyAsync(p->h_err, p->d_err, sizeof(unsigned), hipMemcpyDeviceToHost, s));
  TRY_HIP(hipStreamSynchronize(s));
  if (like && *p->h_err) return SSO_EINVAL;
  if (!like && !p->shared->brow.empty()) start_plan(p->shared, m);
  return SSO_OK;
}

int read_errors(sso_problem* p) {
  TRY_HIP(hipMemcpyAsync(p->h_err, p->d_err, sizeof(unsigned), hipMemcpyDeviceToHost, p->s));
  TRY_HIP(hipStreamSynchronize(p->s));
  return *p->h_err ? SSO_EINVAL : SSO_OK;
}

}  // namespace

extern "C" {

int sso_problem_create(const sso_mesh* mesh, const sso_options* opts, hipStream_t stream,
                       sso_problem** out) {
  if (!mesh || !out) return SSO_EINVAL;
  *out = nullptr;
  if (mesh->n_nodes <= 0 || mesh->n_beams < 0 || mesh->n_quads < 0) return SSO_EINVAL;
  if (!mesh->xyz || !mesh->fixed || !mesh->f_nodal) return SSO_EINVAL;
  if (mesh->n_beams > 0 && (!mesh->beam_nodes || !mesh->beam_prop)) return SSO_EINVAL;
  if (mesh->n_quads > 0 && (!mesh->quad_nodes || !mesh->quad_prop)) return SSO_EINVAL;
  if (16 * (int64_t)mesh->n_quads + 4 * (int64_t)mesh->n_beams >= (int64_t)1 << 31)
    return SSO_EINVAL;
  if (opts && !options_ok(*opts)) return SSO_EINVAL;
  sso_problem* p = new (std::nothrow) sso_problem();
  if (!p) return SSO_ENOMEM;
  AllocScope ac(&p->bytes, &p->mem);
  Arena scratch;
  int st = create_impl(mesh, opts, stream, p, nullptr, scratch);
  if (st != SSO_OK) {
    arena_free(scratch, stream);
    free_problem(p);
    return st;
  }
  arena_recycle(scratch, stream);
  *out = p;
  return SSO_OK;
}

int sso_problem_create_like(const sso_problem* like, const sso_mesh* mesh,
                            const sso_options* opts, hipStream_t stream, sso_problem** out) {
  if (!like || !mesh || !out) return SSO_EINVAL;
  *out = nullptr;
  if (mesh->n_nodes != like->m.n_nodes || mesh->n_beams != like->m.n_beams ||
      mesh->n_quads != like->m.n_quads)
    return SSO_EINVAL;
  if (!mesh->xyz || !mesh->fixed || !mesh->f_nodal) return SSO_EINVAL;
  if (mesh->n_beams > 0 && (!mesh->beam_nodes || !mesh->beam_prop)) return SSO_EINVAL;
  if (mesh->n_quads > 0 && (!mesh->quad_nodes || !mesh->quad_prop)) return SSO_EINVAL;
  if (opts && !options_ok(*opts)) return SSO_EINVAL;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev != like->device) return SSO_EINVAL;
  sso_problem* p = new (std::nothrow) sso_problem();
  if (!p) return SSO_ENOMEM;
  AllocScope ac(&p->bytes, &p->mem);
  Arena scratch;
  int st = create_impl(mesh, opts, stream, p, like, scratch);
  if (st != SSO_OK) {
    arena_free(scratch, stream);
    free_problem(p);
    return st;
  }
  arena_recycle(scratch, stream);
  *out = p;
  return SSO_OK;
}

int sso_problem_update(sso_problem* p, const double* xyz, const double* quad_t,
                       const double* quad_scale) {
  if (!p) return SSO_EINVAL;
  Mesh& m = p->m;
  if (xyz)
    TRY_HIP(hipMemcpyAsync(m.xyz, xyz, sizeof(double) * 3 * (size_t)m.n_nodes,
                           hipMemcpyDeviceToDevice, p->s));
  if (quad_t && m.n_quads)
    TRY_HIP(hipMemcpy2DAsync(m.quad_prop, 5 * sizeof(double), quad_t, sizeof(double),
                             sizeof(double), (size_t)m.n_quads, hipMemcpyDeviceToDevice, p->s));
  if (quad_scale && m.n_quads)
    TRY_HIP(hipMemcpyAsync(m.quad_scale, quad_scale, sizeof(double) * (size_t)m.n_quads,
                           hipMemcpyDeviceToDevice, p->s));
  p->solved = false;
  return SSO_OK;
}

int sso_set_options(sso_problem* p, const sso_options* opts) {
  if (!p || !opts || !options_ok(*opts) || p->in_batch) return SSO_EINVAL;
  // K32 / B / B32 are built by sso_solve for the precision and recurrences it runs with
  if (opts->precision != p->opt.precision || opts->solver != p->opt.solver) p->solved = false;
  p->opt = *opts;
  return SSO_OK;
}

}  // extern "C"

namespace {

bool mixed(const sso_problem* p) { return mixed_for(p->opt, p->pat.n_blocks); }
bool fused(const sso_problem* p) { return p->solver_used == SSO_SOLVER_FUSED; }
bool one_wg(const sso_problem* p) { return p->solver_used == SSO_SOLVER_WG; }
// iteration of a begun problem has stopped (mixed precision: the refinement loop has)
bool stopped(const sso_problem* p) {
  return p->direct ? p->direct_done : mixed(p) ? p->ms.done : p->w.h_st->done != 0;
}

MixedParams mixed_params(const sso_problem* p) {
  MixedParams mp;
  mp.rtol = p->opt.rtol;
  mp.inner_rtol = p->opt.inner_rtol > 0.0 ? p->opt.inner_rtol : 1e-5;
  mp.max_it = p->opt.max_it;
  mp.refine_steps = p->opt.refine_steps;
  mp.inner_max_it = p->opt.inner_max_it;
  if (p->opt.precision == SSO_PREC_AUTO) {   // AUTO's mixed precision: capped inner solves
    constexpr int AUTO_INNER_CAP = 30;
    if (mp.inner_max_it == 0) mp.inner_max_it = AUTO_INNER_CAP;
    const int outer = p->opt.max_it / mp.inner_max_it + 1;
    if (mp.refine_steps < outer) mp.refine_steps = outer;
  }
  return mp;
}

// The direct solver's plan and tables for the problem's topology, on the device by the time the
// problem's stream gets there; *ready false: the direct solver is not for this structure.
int direct_tables(sso_problem* p, bool* ready) {
  SharedPattern* sh = p->shared;
  hipStream_t s = p->s;
  *ready = false;
  std::lock_guard<std::mutex> lock(sh->direct_mutex);
  if (sh->direct_state == SharedPattern::DIRECT_UNKNOWN) {
    if (sh->builder.joinable()) {
      sh->builder.join();
    } else {
      const int st = fetch_pattern(p);
      if (st != SSO_OK) return st;
      TRY_HIP(hipStreamSynchronize(s));
      if (!sh->brow.empty()) make_plan(sh, direct_max_bytes(p->m));
    }
    if (sh->built && debug_mode()) {
      char msg[256];
      if (check_direct_plan(p->m.n_nodes, sh->brow.data(), sh->bcol.data(), sh->plan, msg,
                            sizeof msg) != 0) {
        std::fprintf(stderr, "hipsso debug: %s\n", msg);
        return SSO_EINVAL;
      }
    }
    sh->brow = {};
    sh->bcol = {};
    sh->direct_state = sh->built ? SharedPattern::DIRECT_BUILT : SharedPattern::DIRECT_REFUSED;
  }
  if (sh->direct_state == SharedPattern::DIRECT_BUILT) {
    AllocScope ts(&p->bytes, &sh->pat.mem);
    DirectPlan& pl = sh->plan;
    DirectArgs t{};
    auto put = [&](auto** dst, const auto& v) {
      using V = typename std::decay_t<decltype(v)>::value_type;
      V* d = nullptr;
      hipError_t e = dev_alloc(&d, (int64_t)v.size(), s);
      if (e == hipSuccess && !v.empty())
        e = hipMemcpyAsync(d, v.data(), sizeof(V) * v.size(), hipMemcpyHostToDevice, s);
      *dst = d;
      return e;
    };
    hipError_t e = put(&t.fronts, pl.fronts);
    if (e == hipSuccess) e = put(&t.nodes, pl.nodes);
    if (e == hipSuccess) e = put(&t.maps, pl.maps);
    if (e == hipSuccess) e = put(&t.entries, pl.entries);
    if (e == hipSuccess) e = put(&t.tile_end, pl.tile_end);
    if (e == hipSuccess) e = put(&t.items, pl.items);
    if (e == hipSuccess) e = put(&t.steps, pl.steps);
    if (e == hipSuccess) e = put(&t.level_off, pl.level_off);
    if (e == hipSuccess) e = put(&t.level_np, pl.level_np);
    if (e == hipErrorOutOfMemory) {
      (void)hipGetLastError();
      sh->direct_state = SharedPattern::DIRECT_REFUSED;   // PCG needs less
      return SSO_OK;
    }
    TRY_HIP(e);
    if (!sh->uploaded)
      TRY_HIP(hipEventCreateWithFlags(&sh->uploaded, hipEventDisableTiming));
    TRY_HIP(hipEventRecord(sh->uploaded, s));
    t.n_levels = pl.levels();
    t.bdiag = p->pat.bdiag;
    sh->tables = t;
    sh->direct_state = SharedPattern::DIRECT_READY;
  }
  *ready = sh->direct_state == SharedPattern::DIRECT_READY;
  return SSO_OK;
}

// Whether the direct solver takes the coming solve: decided when the solve starts for a single
// one (with the solver's arrays in place), at the first launch for a begun one (direct_attach).
bool may_be_direct(const sso_problem* p) {
  return p->opt.solver == SSO_SOLVER_AUTO && p->shared->direct_state != SharedPattern::DIRECT_REFUSED;
}

// Whether the plan is still in the making.
bool plan_pending(const sso_problem* p) {
  const SharedPattern* sh = p->shared;
  return sh->direct_state == SharedPattern::DIRECT_UNKNOWN && sh->builder_started &&
         !sh->builder_done;
}

// The solver's arrays; p->direct becomes false where it does not apply.
int direct_attach(sso_problem* p) {
  p->direct = false;
  bool ready = false;
  const int st = direct_tables(p, &ready);
  if (st != SSO_OK || !ready) return st;
  if (!p->da.fact) {
    const DirectPlan& pl = p->shared->plan;
    const int64_t n = 6 * (int64_t)p->m.n_nodes;
    DirectArgs a = p->shared->tables;
    TRY_HIP(hipStreamWaitEvent(p->s, p->shared->uploaded, 0));
    // An eighth of the device's memory stays for what comes later (a problem holds three to five times
    // as much with these arrays as without: 112 and 36 MB for a 60 x 60 shell); one that would take of
    // it runs PCG.  Looking costs 4 us.
    size_t left = 0, total = 0;
    const OnDevice here(p->device);
    TRY_HIP(memory_left(p->device, &left, &total));
    if (8.0 * (double)pl.values() + (double)(total / 8) > (double)left) return SSO_OK;
    double* d = nullptr;
    const hipError_t e = dev_alloc(&d, pl.values() + 2, p->s);   // one buffer, cut below
    if (e == hipErrorOutOfMemory) {
      (void)hipGetLastError();
      return SSO_OK;               // PCG needs less
    }
    TRY_HIP(e);
    auto cut = [&](int64_t len) {
      double* q = d;
      d += len;
      return q;
    };
    a.f0 = cut(pl.work_len);       // the panels first: their lengths are even (16-byte loads)
    a.x1 = cut(pl.again_len);
    a.w = cut(pl.w_len);
    a.u = cut(pl.u_len);
    a.fact = cut(pl.fact_len);
    a.b = cut(n);
    a.sol = cut(n);
    a.v = cut(pl.v_len);
    a.flag = reinterpret_cast<unsigned*>(cut(1));
    a.K = p->K;
    p->da = a;
  }
  p->direct = true;
  return SSO_OK;
}

// What follows from the squared norms rr of the true residual and bb of the load after a
// substitution: the target is met, another substitution on the residual is worth it, refinement
// has done what it can (the rest is for PCG's corrections), or the factor is no good.
enum DirectNext { DIRECT_MET, DIRECT_AGAIN, DIRECT_STUCK, DIRECT_FAILED };
DirectNext direct_next(sso_problem* p, double rr, double bb, unsigned flag) {
  constexpr int MAX_STEPS = 7;
  const double rn = std::sqrt(rr), bn = std::sqrt(bb);
  const double prev = p->direct_rr < 0.0 ? -1.0 : std::sqrt(p->direct_rr);
  p->direct_rr = rr;
  p->direct_bb = bb;
  const int step = ++p->direct_steps;
  if (flag || !std::isfinite(rn)) return DIRECT_FAILED;
  p->factored = true;
  // A first solution that meets the target by less than FIRST takes one more step, after which u is
  // accurate to the last bits.  Its residual lies in smooth modes, where an iteration's is in rough
  // ones, and with a first residual between 0.3 and a half of the target u was up to 36 times as far
  // off as PCG's at the same target (an 11 x 11 grid-shell).  With the quarter, over 300 structures,
  // u and the gradient are closer than PCG's on shells and arches (0.03 to 0.9 times) and about as
  // close on grid-shells (up to 1.6 times in u, 1.8 in a linear objective's gradient, 3.5 once).
  // 0.03 would bring all below 0.25 and take 15 to 35 % longer on arches and small shells, which do
  // not need it (arch 444 -> 607 us, 16 x 16 shell 445 -> 565).
  constexpr double FIRST = 0.25;
  if (rn <= (step == 1 ? FIRST : 1.0) * p->opt.rtol * bn) return DIRECT_MET;
  if (step == MAX_STEPS || (prev >= 0.0 && rn > 0.5 * prev)) return DIRECT_STUCK;
  return DIRECT_AGAIN;
}

// Work that follows a solution on the stream, whatever the residual turns out to be: enqueued
// behind each substitution, so that the host's look at the residual does not hold it up.
using Tail = std::function<hipError_t()>;

// K x = b with the direct solver: factor K if the current one is not yet factored, substitute,
// and refine on the true residual (row sums in double-double) until it meets rtol, as long as a
// step gains a factor of two.  *done: met, and the stream idle; otherwise x is the best so far.  A
// K that is not positive definite to working precision leaves p->direct false and x = 0.
int run_direct(sso_problem* p, const double* b, double* x, bool* done, const Tail& tail) {
  hipStream_t s = p->s;
  const DirectPlan& pl = p->shared->plan;
  const DirectArgs& a = p->da;
  const int64_t n = 6 * (int64_t)p->m.n_nodes;
  *done = false;
  if (!a.fact) return SSO_EHIP;   // not attached: no launch may see these arguments
  if (!p->factored) {
    TRY_HIP(launch_direct_clear(a, s));
    TRY_HIP(launch_direct_factor(pl, a, s));
  }
  DirectArgs q = a;
  q.rhs = b;
  q.sol = x;
  TRY_HIP(launch_direct_solve(pl, q, s));
  p->direct_rr = -1.0;
  p->direct_steps = 0;
  for (;;) {
    TRY_HIP(launch_true_residual(p->m, p->pat, p->K, x, b, p->w.r, p->w, p->h_scal, s, a.flag,
                                 p->d_err));
    if (tail) TRY_HIP(tail());
    TRY_HIP(hipStreamSynchronize(s));
    if (p->unchecked) {
      p->unchecked = false;
      if (p->h_scal[3] != 0.0) return SSO_EINVAL;
    }
    const bool was = p->factored;
    const DirectNext next = direct_next(p, p->h_scal[0], p->h_scal[1],
                                        !was && p->h_scal[2] != 0.0);
    if (next == DIRECT_FAILED && was) {   // a good factor: the right-hand side is not finite
      *done = true;
      return SSO_EBREAKDOWN;
    }
    if (next == DIRECT_FAILED) {
      TRY_HIP(hipMemsetAsync(x, 0, sizeof(double) * n, s));
      p->direct = false;
      return SSO_OK;
    }
    if (next != DIRECT_AGAIN) {
      *done = next == DIRECT_MET;
      return SSO_OK;
    }
    q.rhs = p->w.r;
    q.sol = a.sol;
    TRY_HIP(launch_direct_solve(pl, q, s));
    TRY_HIP(launch_axpy(1.0, a.sol, x, n, s));
  }
}

// The FP32 copies that mixed precision's standard inner solves need, where the direct solver was
// to do without them.
int mixed_operands(sso_problem* p) {
  hipStream_t s = p->s;
  const int64_t nk = 36 * p->pat.n_blocks;
  if (!p->Dinv32) TRY_HIP(dev_alloc(&p->Dinv32, dinv_packed_len(p->m.n_nodes), s));
  if (!p->K32) TRY_HIP(dev_alloc(&p->K32, nk, s));
  TRY_HIP(pcg_alloc_mixed(p->w, s));
  TRY_HIP(launch_block_jacobi(p->m, p->pat, p->K, p->Dinv, p->Dinv32, p->d_err, s));
  TRY_HIP(launch_convert_f32(p->K, p->K32, nk, s));
  return SSO_OK;
}

// Solve K x = b (b masked) in the problem's precision mode.  *tailed (may be null): the tail has
// run behind the solution and the stream is idle.
int run_solver(sso_problem* p, const double* b, double* x, int* iters, int* outer,
               const Tail& tail = nullptr, bool* tailed = nullptr) {
  int status = SSO_OK;
  *outer = 0;
  if (tailed) *tailed = false;
  if (p->direct) {
    bool done = false;
    const int st = run_direct(p, b, x, &done, tail);
    if (mixed(p)) *outer = p->direct_steps;
    if (st == SSO_OK && done && tailed) *tailed = true;
    if (st != SSO_OK || done) return st;
    if (p->direct) {   // the target lies below what refinement reaches: corrections by PCG
      TRY_HIP(pcg_correct(p->m, p->pat, p->K, p->Dinv, b, x, p->opt.rtol, p->opt.max_it, p->w,
                          p->s, iters, &status));
      return status;
    }
    if (mixed(p)) {
      const int sm = mixed_operands(p);
      if (sm != SSO_OK) return sm;
    }
  }
  if (one_wg(p)) {
    TRY_HIP(pcg_solve_wg(p->m, p->pat, p->K, p->Dinv, b, x, p->opt.rtol, p->opt.max_it, p->w,
                         p->s, iters, &status, p->opt.profile_every));
  } else if (!mixed(p)) {
    TRY_HIP(pcg_solve(p->m, p->pat, p->K, p->Dinv, fused(p) ? p->B : nullptr, b, x, p->opt.rtol,
                      p->opt.max_it, p->w, p->s, iters, &status, p->opt.profile_every));
  } else {
    TRY_HIP(pcg_solve_mixed(p->m, p->pat, p->K, p->K32, p->Dinv32, fused(p) ? p->B32 : nullptr,
                            b, x, mixed_params(p), p->w, p->s, iters, &status, outer,
                            p->opt.profile_every));
  }
  return status;
}

// Elements, loads, assembly, masking, block-Jacobi and the operators the chosen PCG needs
// (B = K M for the single-reduction recurrences; FP32 copies for mixed precision).  Events 0-2
// bracket the stages.
int prepare(sso_problem* p, bool batch) {
  hipStream_t s = p->s;
  p->solver_used = pcg_pick_solver(p->opt.solver, p->m.n_nodes, p->pat.n_blocks,
                                   mixed_for(p->opt, p->pat.n_blocks));
  // multi-problem launches: many problems in flight make the iteration bandwidth-bound, where
  // the standard pair streams faster than the fused kernel (16 60 x 60 shells: 123 vs 93
  // solves/s; 256 80 x 80 shells: 13.2 vs 19.2 s).  A problem resident in one workgroup's LDS
  // keeps that solver in its kernel beside the launches (served stream: the small requests'
  // median latency 14.5 -> 5.1 ms at the same capacity).
  if (batch && p->opt.solver == SSO_SOLVER_AUTO && p->solver_used != SSO_SOLVER_WG)
    p->solver_used = SSO_SOLVER_STANDARD;
  p->direct = p->factored = p->direct_done = false;
  p->direct_rr = -1.0;
  p->direct_steps = 0;
  p->w.prof_us = 0.0;
  p->w.prof_n = 0;
  if (may_be_direct(p)) {
    if (batch) {
      p->direct = true;     // attached by the first launch: its plan may still be in the making
    } else {
      const int st = direct_attach(p);
      if (st != SSO_OK) return st;
    }
    // should it go back to PCG: the standard recurrences, which need the least beside K
    if (p->direct && p->solver_used != SSO_SOLVER_WG) p->solver_used = SSO_SOLVER_STANDARD;
  }
  const bool mx = mixed(p) && !p->direct, fu = fused(p);
  const int64_t nk = 36 * p->pat.n_blocks;
  const int64_t nb = 36 * right_precondition_blocks(p->pat, p->m.n_nodes);
  if (mx && !p->Dinv32) TRY_HIP(dev_alloc(&p->Dinv32, dinv_packed_len(p->m.n_nodes), s));
  if (mx && !fu && !p->K32) TRY_HIP(dev_alloc(&p->K32, nk, s));
  if (fu && !mx && !p->B) TRY_HIP(dev_alloc(&p->B, nb, s));
  if (fu && mx && !p->B32) TRY_HIP(dev_alloc(&p->B32, nb, s));
  TRY_HIP(hipMemsetAsync(p->d_err, 0, sizeof(unsigned), s));
  TRY_HIP(hipEventRecord(p->ev[0], s));
  TRY_HIP(launch_element_stiffness(p->m, p->coo, p->qarea, p->d_err, s));
  if (p->fm) {
    TRY_HIP(launch_loads(p->m, p->pat, p->qarea, p->fm, s));
    TRY_HIP(launch_lift(p->m, p->pat, p->coo, p->fm, p->f, s));
  } else {
    TRY_HIP(launch_loads(p->m, p->pat, p->qarea, p->f, s));
  }
  TRY_HIP(hipEventRecord(p->ev[1], s));
  TRY_HIP(launch_assemble(p->m, p->pat, p->coo, p->K, s));
  TRY_HIP(launch_block_jacobi(p->m, p->pat, p->K, p->Dinv, mx ? p->Dinv32 : nullptr, p->d_err,
                              s));
  if (mx && !fu) TRY_HIP(launch_convert_f32(p->K, p->K32, nk, s));
  if (fu)
    TRY_HIP(launch_right_precondition(p->m, p->pat, p->K, p->Dinv, mx ? nullptr : p->B,
                                      mx ? p->B32 : nullptr, s));
  TRY_HIP(hipEventRecord(p->ev[2], s));
  p->unchecked = p->direct && !batch;
  // a direct solve looks at the elements' errors together with its residual: what runs between is
  // bounded by the plan whatever the values
  return p->unchecked ? SSO_OK : read_errors(p);
}

// The start of a begun solve's PCG iteration (x = 0).
int begin_pcg(sso_problem* p) {
  hipStream_t s = p->s;
  if (mixed(p))
    TRY_HIP(mixed_begin(p->m, p->pat, p->K, p->K32, p->Dinv32, fused(p) ? p->B32 : nullptr, p->f,
                        p->u, mixed_params(p), p->w, s, p->ms));
  else if (fused(p))
    TRY_HIP(fused_begin(p->m, p->pat, p->B, p->Dinv, p->f, p->u, p->opt.rtol, p->opt.max_it,
                        p->w, s, &p->fdesc));
  else
    TRY_HIP(pcg_begin(p->m, p->pat, p->K, p->Dinv, p->f, p->u, p->opt.rtol, p->opt.max_it,
                      p->w, s, &p->desc));
  return SSO_OK;
}

// A begun solve that the direct solver does not take, or could not finish.  Where that fails, the
// problem is as no launch had taken it: it has no iteration that could go on.
int back_to_pcg(sso_problem* p) {
  p->direct = false;
  int st = mixed(p) ? mixed_operands(p) : SSO_OK;
  if (st == SSO_OK) st = begin_pcg(p);
  if (st != SSO_OK) {
    p->direct = true;
    p->factored = p->direct_done = false;
    p->direct_steps = 0;
    p->direct_rr = -1.0;
  }
  return st;
}

// ---- the two solvers' parts of a multi-problem launch ----------------------------------------

// The next step of the listed problems that the direct solver has and that have iterations left:
// jobs, factorisations first, their positions in b->direct.  A problem whose plan is still in the
// making is left out, or waited for; one that turns out not to be for the direct solver starts its
// PCG iteration and joins `turned`.
int direct_jobs(sso_batch* b, bool wait, std::vector<DirectJob>& jobs, std::vector<int>& turned) {
  std::vector<DirectJob> more;
  std::vector<int> at_more;
  jobs.clear();
  b->direct.clear();
  for (int i = 0; i < (int)b->listed.size(); ++i) {
    sso_problem* p = b->listed[i];
    if (!p->direct || p->direct_done || b->steps[i] >= b->n_iter) continue;
    AllocScope ac(&p->bytes, &p->mem);
    const bool factor = p->direct_steps == 0;
    if (factor) {
      if (!wait && plan_pending(p)) continue;
      const int st = direct_attach(p);
      if (st != SSO_OK) {
        p->direct = true;              // still to be taken
        return st;
      }
      if (!p->direct) {                // not for this structure
        const int sb = back_to_pcg(p);
        if (sb != SSO_OK) return sb;
        turned.push_back(i);
        continue;
      }
    }
    DirectJob j{&p->shared->plan, p->da,
                residual_job(p->m, p->pat, p->K, p->u, p->f, factor ? nullptr : p->da.sol, p->w,
                             p->da.flag),
                factor};
    j.a.rhs = factor ? p->f : p->w.r;
    j.a.sol = factor ? p->u : p->da.sol;
    (factor ? jobs : more).push_back(j);
    (factor ? b->direct : at_more).push_back(i);
  }
  jobs.insert(jobs.end(), more.begin(), more.end());
  b->direct.insert(b->direct.end(), at_more.begin(), at_more.end());
  return SSO_OK;
}

// What the launched jobs came to.
int direct_collect(sso_batch* b, std::vector<int>& turned) {
  if (b->direct.empty()) return SSO_OK;
  TRY_HIP(direct_batch_wait(b->db, b->s));
  const std::vector<int> at = std::move(b->direct);
  b->direct.clear();
  for (size_t k = 0; k < at.size(); ++k) {
    sso_problem* p = b->listed[at[k]];
    const double* r = b->db.out.data() + 3 * k;
    const DirectNext next = direct_next(p, r[0], r[1], r[2] != 0.0);
    ++b->steps[at[k]];
    p->direct_done = next == DIRECT_MET || next == DIRECT_STUCK;
    if (next == DIRECT_FAILED) {
      AllocScope ac(&p->bytes, &p->mem);
      const int st = back_to_pcg(p);
      if (st != SSO_OK) return st;
      turned.push_back(at[k]);
    }
  }
  return SSO_OK;
}

// Of the problems at these positions those that iterate, by launch kind (positions in b->idx).
BatchLists pcg_lists(sso_batch* b, const std::vector<int>& positions) {
  BatchLists lists;
  for (auto& v : b->idx) v.clear();
  for (int i : positions) {
    sso_problem* p = b->listed[i];
    if (p->direct || stopped(p)) continue;   // the direct solver's, or finished at an earlier poll
    if (mixed(p) && fused(p)) {
      lists.fused32.push_back(p->ms.fdesc);
      b->idx[3].push_back(i);
    } else if (mixed(p)) {
      lists.standard32.push_back(p->ms.sdesc);
      b->idx[2].push_back(i);
    } else if (fused(p)) {
      lists.fused.push_back(p->fdesc);
      b->idx[1].push_back(i);
    } else if (one_wg(p)) {
      PcgDesc<double> d = p->desc;
      d.n_wg = 1;
      lists.wg.push_back(d);
      b->idx[4].push_back(i);
    } else {
      lists.standard.push_back(p->desc);
      b->idx[0].push_back(i);
    }
  }
  return lists;
}

// Waits for the launched iterations and takes their states; a timing sample, and in mixed precision
// the outer step that follows a stopped inner solve.
int pcg_collect(sso_batch* b) {
  sso_problem* const* ps = b->listed.data();
  TRY_HIP(pcg_batch_wait(b->bw));
  size_t k0 = 0;
  for (const auto& v : b->idx)
    for (int i : v) *ps[i]->w.h_st = b->bw.h_states[k0++];
  if (b->armed > 0) {
    // each problem's iterations inside the timed span: how far its next iteration index moved
    // (an iteration that finds the problem stopped does no work and does not move it), at most
    // the span; bytes per iteration with all of K counted, and as the launch's product read K
    const int span = b->armed;
    b->armed = 0;
    float ms = 0.0f;
    TRY_HIP(hipEventElapsedTime(&ms, b->bw.ev_t0, b->bw.ev_t1));
    b->prof_us += 1000.0 * (double)ms;
    b->prof_iters += span;
    const bool sym = b->bw.standard.sym;
    for (size_t k = 0; k < b->idx[0].size(); ++k) {
      const sso_problem* p = ps[b->idx[0][k]];
      int d = p->w.h_st->jn - b->jn0[k];
      d = d < 0 ? 0 : (d > span ? span : d);
      b->prof_bytes += d * pcg_bytes_per_iteration(p->m.n_nodes, p->pat.n_blocks, false, false);
      b->prof_bytes_read += d * pcg_bytes_per_iteration(p->m.n_nodes, p->pat.n_blocks, false, sym);
    }
  }
  // mixed precision: a stopped inner solve is refined in FP64 and the next one started
  for (const std::vector<int>* v : {&b->idx[2], &b->idx[3]})
    for (int i : *v) {
      sso_problem* p = ps[i];
      TRY_HIP(mixed_step(p->m, p->pat, p->K, p->K32, p->Dinv32, fused(p) ? p->B32 : nullptr, p->f,
                         p->u, mixed_params(p), p->w, p->s, p->ms));
    }
  return SSO_OK;
}

// After a launch, or what follows one, that failed: nothing of it is left running, so that the
// problems can go on or end.  Iterations go on from the states on the device; a direct solve starts
// anew, since a correction that was added must not be added again.
int abandon(sso_batch* b, int status) {
  (void)hipStreamSynchronize(b->s);
  if (b->bw.s_wg) (void)hipStreamSynchronize(b->bw.s_wg);
  b->bw.pending_nt = -1;
  b->armed = 0;
  for (int i : b->direct) {
    sso_problem* p = b->listed[i];
    p->direct_steps = 0;
    p->factored = false;
    p->direct_rr = -1.0;
  }
  b->direct.clear();
  return status;
}

bool fused_used(const sso_problem* p) { return p->solver_used == SSO_SOLVER_FUSED; }

// single: a solve of its own (sso_solve, the adjoint), whose standard FP64 products read only
// K's upper triangle above the size pcg_sym_products names; multi-problem launches read all of K
bool sym_used(const sso_problem* p, bool single) {
  return single && p->solver_used == SSO_SOLVER_STANDARD && pcg_sym_products(p->pat.n_blocks, mixed(p));
}

double solve_bytes(const sso_problem* p, int iters, int outer, bool single) {
  const int64_t nn = p->m.n_nodes, nb = p->pat.n_blocks;
  if (fused_used(p) && !mixed(p)) return iters * fused_bytes_per_iteration(nn, nb, false);
  if (!mixed(p)) return iters * pcg_bytes_per_iteration(nn, nb, false, sym_used(p, single));
  // inner FP32 iterations + one FP64 residual SpMV (K, x, b read; r written) per outer step
  double resid = 292.0 * nb + 4.0 * (nn + 1) + 3.0 * 8.0 * 6.0 * nn;
  return iters * pcg_bytes_per_iteration(nn, nb, true, false) + (outer + 1) * resid;
}

// ---- penalised volume objective (Sec. 3.3): shared by the allocating and static-scratch forms

constexpr int SIZE_XWG = 1024;   // workgroups (partials) of the size-objective reduction

bool size_args_ok(const sso_problem* p, double eps1, double u_max, double t_min,
                  const double* out_host, const double* dg_dxyz) {
  return p && p->solved && out_host && dg_dxyz && eps1 >= 0.0 && std::isfinite(eps1) &&
         u_max > 0.0 && std::isfinite(u_max) && t_min > 0.0 && std::isfinite(t_min);
}

// g = (1 + eps1 c) W and its gradient with the scratch arrays xpart [2 SIZE_XWG], gw
// [14 n_quads] and wv [n_quads] given.
int size_objective_impl(sso_problem* p, double eps1, double u_max, double t_min,
                        double* out_host, double* dg_dxyz, double* dg_dt, sso_stats* stats,
                        double* xpart, double* gw, double* wv) {
  hipStream_t s = p->s;
  const Mesh& m = p->m;
  TRY_HIP(hipEventRecord(p->ev[4], s));
  // volume terms, then dc/du (masked) with the sums c and W in d_scal[2..3]
  TRY_HIP(launch_volume_terms(m, t_min, gw, wv, s));
  TRY_HIP(launch_size_terms(m, p->u, u_max, wv, p->rhs, xpart, SIZE_XWG, p->d_scal + 2, s));
  auto terms = [&] {
    hipError_t e =
        launch_adjoint_terms(m, p->pat, p->u, p->lam, 1.0, 0.0, p->gbeam, p->gquad, s);
    if (e == hipSuccess) e = launch_size_combine(m, eps1, p->d_scal + 2, gw, p->gbeam, p->gquad, s);
    if (e == hipSuccess)
      e = launch_gather(m, p->pat, p->gbeam, p->gquad, dg_dxyz, dg_dt, nullptr, s);
    if (e == hipSuccess) e = hipEventRecord(p->ev[5], s);
    return e != hipSuccess ? e
                           : hipMemcpyAsync(p->h_scal + 4, p->d_scal + 2, 2 * sizeof(double),
                                            hipMemcpyDeviceToHost, s);
  };
  int iters = 0, outer = 0;
  bool tailed = false;
  const int status =
      run_solver(p, p->rhs, p->lam, &iters, &outer, std::ref(terms), &tailed);
  if (status != SSO_OK && status != SSO_ENOTCONV) return status;
  if (!tailed) {
    TRY_HIP(terms());
    TRY_HIP(hipStreamSynchronize(s));
  }
  const double c = p->h_scal[4], W = p->h_scal[5];
  out_host[0] = (1.0 + eps1 * c) * W;
  out_host[1] = c;
  out_host[2] = W;
  if (stats) {
    std::memset(stats, 0, sizeof(*stats));
    stats->iters = iters;
    stats->t_adj_us = elapsed_us(p->ev[4], p->ev[5]);
  }
  return status;
}

std::mutex scratch_mutex;
double* scratch_ptr[MAX_DEVICES] = {};

int scratch_address(int device, double** out) {
  if (device < 0 || device >= MAX_DEVICES) return SSO_EINVAL;
  std::lock_guard<std::mutex> lock(scratch_mutex);
  if (!scratch_ptr[device]) {
    int cur = 0;
    TRY_HIP(hipGetDevice(&cur));
    if (cur != device) TRY_HIP(hipSetDevice(device));
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (cur != device) (void)hipSetDevice(cur);
    if (e != hipSuccess) return map_hip(e);
    if (!ptr) return SSO_EHIP;
    scratch_ptr[device] = static_cast<double*>(ptr);
  }
  *out = scratch_ptr[device];
  return SSO_OK;
}


std::mutex pool_mutex;
hipMemPool_t pools[MAX_DEVICES] = {};

// The device's pool, created on first use with an unlimited release threshold.
hipError_t device_pool(int device, hipMemPool_t* out) {
  std::lock_guard<std::mutex> lock(pool_mutex);
  if (!pools[device]) {
    hipMemPoolProps props = {};
    props.allocType = hipMemAllocationTypePinned;
    props.handleTypes = hipMemHandleTypeNone;
    props.location.type = hipMemLocationTypeDevice;
    props.location.id = device;
    hipMemPool_t pool = nullptr;
    hipError_t e = hipMemPoolCreate(&pool, &props);
    if (e != hipSuccess) return e;
    uint64_t keep = UINT64_MAX;
    e = hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &keep);
    if (e != hipSuccess) {
      (void)hipMemPoolDestroy(pool);
      return e;
    }
    pools[device] = pool;
  }
  *out = pools[device];
  return hipSuccess;
}

}  // namespace

namespace sso {

// Every device buffer of the library comes from a pool of its own per device that keeps freed
// memory for the next allocation.  The default pool's release threshold of zero hands freed
// memory back to the driver at each synchronisation and the next allocation maps it afresh,
// which cost about 0.85 ms per destroyed problem and 1 ms per created one on the served sizes.
hipError_t pool_alloc(void** p, size_t bytes, hipStream_t s) {
  int device = 0;
  hipError_t e = hipStreamGetDevice(s, &device);
  if (e != hipSuccess) return e;
  if (device < 0 || device >= MAX_DEVICES) return hipErrorInvalidDevice;
  hipMemPool_t pool = nullptr;
  e = device_pool(device, &pool);
  if (e != hipSuccess) return e;
  return hipMallocFromPoolAsync(p, bytes, pool, s);
}

// Chunks of ended problems, idle and still allocated, for the next problem on the device.  A
// stream-ordered free costs the host 20 to 150 us and an allocation up to 30, ten of each a served
// request: 1.6 ms to finish one and 0.95 to admit it, against 0.5 and 0.7 from here.  At most
// CACHE_BYTES are kept, sso_pool_trim gives all of it back, and so does an allocation that fails.
constexpr size_t CACHE_BYTES = (size_t)8 << 30;
struct ChunkCache {
  std::mutex mu;
  std::map<size_t, std::vector<char*>> idle;   // by size
  size_t bytes = 0;
};
static ChunkCache chunk_caches[MAX_DEVICES];

static ChunkCache* cache_of(hipStream_t s) {
  int device = 0;
  if (hipStreamGetDevice(s, &device) != hipSuccess || device < 0 || device >= MAX_DEVICES)
    return nullptr;
  return &chunk_caches[device];
}

hipError_t memory_left(int device, size_t* left, size_t* total) {
  hipError_t e = hipMemGetInfo(left, total);
  if (e != hipSuccess || device < 0 || device >= MAX_DEVICES) return e;
  hipMemPool_t pool = nullptr;
  {
    std::lock_guard<std::mutex> lock(pool_mutex);
    pool = pools[device];
  }
  if (pool) {
    uint64_t reserved = 0, used = 0;
    e = hipMemPoolGetAttribute(pool, hipMemPoolAttrReservedMemCurrent, &reserved);
    if (e == hipSuccess) e = hipMemPoolGetAttribute(pool, hipMemPoolAttrUsedMemCurrent, &used);
    if (e != hipSuccess) return e;
    if (reserved > used) *left += reserved - used;
  }
  ChunkCache& c = chunk_caches[device];
  std::lock_guard<std::mutex> lock(c.mu);
  *left += c.bytes;
  return hipSuccess;
}

static void cache_flush(ChunkCache& c, hipStream_t s) {
  std::map<size_t, std::vector<char*>> idle;
  {
    std::lock_guard<std::mutex> lock(c.mu);
    idle.swap(c.idle);
    c.bytes = 0;
  }
  for (const auto& k : idle)
    for (char* p : k.second) (void)hipFreeAsync(p, s);
}

// A chunk of exactly `bytes` (a chunk_size, or ARENA_CHUNK).
static hipError_t chunk_take(size_t bytes, hipStream_t s, void** out) {
  ChunkCache* c = cache_of(s);
  if (c) {
    std::lock_guard<std::mutex> lock(c->mu);
    auto it = c->idle.find(bytes);
    if (it != c->idle.end() && !it->second.empty()) {
      *out = it->second.back();
      it->second.pop_back();
      c->bytes -= bytes;
      return hipSuccess;
    }
  }
  hipError_t e = pool_alloc(out, bytes, s);
  if (e == hipErrorOutOfMemory && c) {
    (void)hipGetLastError();
    cache_flush(*c, s);
    e = hipStreamSynchronize(s);
    if (e == hipSuccess) e = pool_alloc(out, bytes, s);
  }
  return e;
}

hipError_t arena_alloc(Arena& a, size_t bytes, hipStream_t s, void** out, int64_t* held) {
  bytes = (bytes + ARENA_ALIGN - 1) / ARENA_ALIGN * ARENA_ALIGN;
  *held = 0;
  if (bytes > ARENA_CHUNK / 4) {   // a chunk of its own
    bytes = chunk_size(bytes);
    void* q = nullptr;
    const hipError_t e = chunk_take(bytes, s, &q);
    if (e != hipSuccess) return e;
    a.chunks.emplace_back(static_cast<char*>(q), bytes);
    *held = (int64_t)bytes;
    *out = q;
    return hipSuccess;
  }
  if (bytes > a.left) {
    void* q = nullptr;
    const hipError_t e = chunk_take(ARENA_CHUNK, s, &q);
    if (e != hipSuccess) return e;
    a.chunks.emplace_back(static_cast<char*>(q), ARENA_CHUNK);
    a.cur = static_cast<char*>(q);
    a.left = ARENA_CHUNK;
    *held = (int64_t)ARENA_CHUNK;
  }
  *out = a.cur;
  a.cur += bytes;
  a.left -= bytes;
  return hipSuccess;
}

void arena_recycle(Arena& a, hipStream_t s) {
  ChunkCache* c = cache_of(s);
  for (const auto& k : a.chunks) {
    bool kept = false;
    if (c) {
      std::lock_guard<std::mutex> lock(c->mu);
      if (c->bytes + k.second <= CACHE_BYTES) {
        try {
          c->idle[k.second].push_back(k.first);
          c->bytes += k.second;
          kept = true;
        } catch (...) {   // no host memory for the entry
        }
      }
    }
    if (!kept) (void)hipFreeAsync(k.first, s);
  }
  a = Arena();
}

bool arena_owns(const Arena& a, const void* p) {
  const char* c = static_cast<const char*>(p);
  for (const auto& k : a.chunks)
    if (c >= k.first && c < k.first + k.second) return true;
  return false;
}

void arena_free(Arena& a, hipStream_t s) {
  for (const auto& k : a.chunks) (void)hipFreeAsync(k.first, s);
  a = Arena();
}

}  // namespace sso

extern "C" {

int sso_solve(sso_problem* p, double* u_out, sso_stats* stats) {
  if (!p) return SSO_EINVAL;
  AllocScope ac(&p->bytes, &p->mem);
  hipStream_t s = p->s;
  p->solved = false;
  p->in_batch = false;
  int st = prepare(p, false);
  if (st != SSO_OK) return st;
  int iters = 0, outer = 0;
  const size_t u_bytes = sizeof(double) * 6 * (size_t)p->m.n_nodes;
  bool tailed = false;
  // prescribed displacements are written into u last, and refinement must not see them
  auto copy_out = [&] {
    hipError_t e = hipEventRecord(p->ev[3], s);
    if (e == hipSuccess && u_out && !p->m.u_presc)
      e = hipMemcpyAsync(u_out, p->u, u_bytes, hipMemcpyDeviceToDevice, s);
    return e;
  };
  int status = run_solver(p, p->f, p->u, &iters, &outer, std::ref(copy_out), &tailed);
  if (status == SSO_EHIP || status == SSO_ENOMEM || status == SSO_EINVAL) return status;
  if (!tailed) {
    TRY_HIP(hipEventRecord(p->ev[3], s));
    TRY_HIP(launch_true_residual(p->m, p->pat, p->K, p->u, p->f, nullptr, p->w, p->h_scal, s));
  }
  if (!tailed || p->m.u_presc) {
    if (p->m.u_presc) TRY_HIP(launch_apply_prescribed(p->m, p->u, s));
    if (u_out) TRY_HIP(hipMemcpyAsync(u_out, p->u, u_bytes, hipMemcpyDeviceToDevice, s));
    TRY_HIP(hipStreamSynchronize(s));
  }
  if (stats) {
    std::memset(stats, 0, sizeof(*stats));
    stats->iters = iters;
    stats->refine_steps = outer;
    stats->rel_residual = p->h_scal[1] > 0 ? sqrt(p->h_scal[0] / p->h_scal[1]) : 0.0;
    stats->t_elem_us = elapsed_us(p->ev[0], p->ev[1]);
    stats->t_asm_us = elapsed_us(p->ev[1], p->ev[2]);
    stats->t_solve_us = elapsed_us(p->ev[2], p->ev[3]);
    stats->bytes_moved = solve_bytes(p, iters, outer, true);
    stats->spmv_samples = p->w.prof_n;
    stats->spmv_us = p->w.prof_n ? p->w.prof_us / p->w.prof_n : 0.0;
    stats->spmv_bytes =
        fused_used(p) ? fused_bytes_per_iteration(p->m.n_nodes, p->pat.n_blocks, mixed(p))
                      : pcg_bytes_per_iteration(p->m.n_nodes, p->pat.n_blocks, mixed(p),
                                                sym_used(p, true));
    stats->solver = p->direct ? SSO_SOLVER_AUTO : p->solver_used;
    stats->sym_products = !p->direct && sym_used(p, true) ? 1 : 0;
  }
  // after SSO_ENOTCONV u holds the last iterate; objective and adjoint stay available
  p->solved = (status == SSO_OK || status == SSO_ENOTCONV);
  return status;
}

int sso_solve_begin(sso_problem* p) {
  if (!p) return SSO_EINVAL;
  AllocScope ac(&p->bytes, &p->mem);
  // multi-problem launches run FP64 iterations of either kind and FP32 single-reduction ones
  p->solved = false;
  p->in_batch = false;
  int st = prepare(p, true);
  if (st != SSO_OK) return st;
  if (!p->direct) {
    st = begin_pcg(p);
    if (st != SSO_OK) return st;
  }
  p->in_batch = true;
  return SSO_OK;
}

int sso_solve_end(sso_problem* p, double* u_out, sso_stats* stats) {
  if (!p || !p->in_batch || p->batch_pending) return SSO_EINVAL;
  AllocScope ac(&p->bytes, &p->mem);
  hipStream_t s = p->s;
  int status = SSO_OK, iters = 0, outer = 0;
  auto residual = [&] {   // into h_scal, once the stream gets there
    return launch_true_residual(p->m, p->pat, p->K, p->u, p->f, nullptr, p->w, p->h_scal, s);
  };
  const bool untaken = p->direct && p->direct_steps == 0;
  if (untaken) {
    // ended before a launch took it: u = 0, no factor, and perhaps no arrays to hold one; an
    // adjoint is solved by PCG, with its operands made here (some of those calls allocate nothing)
    if (mixed(p)) {
      const int st = mixed_operands(p);
      if (st != SSO_OK) return st;
    }
    TRY_HIP(hipMemsetAsync(p->u, 0, sizeof(double) * 6 * (size_t)p->m.n_nodes, s));
    status = SSO_ENOTCONV;
    TRY_HIP(residual());
  } else if (p->direct) {
    if (mixed(p)) outer = p->direct_steps;
    if (!p->direct_done) {
      status = SSO_ENOTCONV;
      TRY_HIP(residual());
    } else if (!(std::sqrt(p->direct_rr) <= p->opt.rtol * std::sqrt(p->direct_bb))) {
      TRY_HIP(pcg_correct(p->m, p->pat, p->K, p->Dinv, p->f, p->u, p->opt.rtol, p->opt.max_it,
                          p->w, s, &iters, &status));
      TRY_HIP(residual());
    } else {
      p->h_scal[0] = p->direct_rr;
      p->h_scal[1] = p->direct_bb;
    }
  } else {
    TRY_HIP(hipMemcpyAsync(p->w.h_st, p->w.st, sizeof(PcgState), hipMemcpyDeviceToHost, s));
    TRY_HIP(residual());
    TRY_HIP(hipStreamSynchronize(s));
    status = p->w.h_st->done ? p->w.h_st->status : SSO_ENOTCONV;
    iters = p->w.h_st->it;
    if (mixed(p)) {   // the refinement loop already ended on the FP64 true residual
      status = p->ms.done ? p->ms.status : SSO_ENOTCONV;
      iters = p->ms.iters;
      outer = p->ms.outer;
    } else if (status == SSO_OK) {
      TRY_HIP(pcg_correct(p->m, p->pat, p->K, p->Dinv, p->f, p->u, p->opt.rtol, p->opt.max_it,
                          p->w, s, &iters, &status));
      TRY_HIP(residual());
    }
  }
  if (p->m.u_presc) TRY_HIP(launch_apply_prescribed(p->m, p->u, s));
  if (u_out)
    TRY_HIP(hipMemcpyAsync(u_out, p->u, sizeof(double) * 6 * (size_t)p->m.n_nodes,
                           hipMemcpyDeviceToDevice, s));
  TRY_HIP(hipStreamSynchronize(s));
  if (untaken) p->direct = false;
  if (stats) {
    std::memset(stats, 0, sizeof(*stats));
    stats->iters = iters;
    stats->rel_residual = p->h_scal[1] > 0 ? sqrt(p->h_scal[0] / p->h_scal[1]) : 0.0;
    stats->refine_steps = outer;
    stats->bytes_moved = solve_bytes(p, iters, outer, false);
    stats->spmv_bytes =
        fused(p) ? fused_bytes_per_iteration(p->m.n_nodes, p->pat.n_blocks, mixed(p))
                 : pcg_bytes_per_iteration(p->m.n_nodes, p->pat.n_blocks, mixed(p), false);
    stats->solver = p->direct ? SSO_SOLVER_AUTO : p->solver_used;
  }
  p->in_batch = false;
  p->solved = (status == SSO_OK || status == SSO_ENOTCONV);
  return status;
}

int sso_batch_create(hipStream_t stream, sso_batch** out) {
  if (!out) return SSO_EINVAL;
  sso_batch* b = new (std::nothrow) sso_batch();
  if (!b) return SSO_ENOMEM;
  b->s = stream;
  *out = b;
  return SSO_OK;
}

int sso_solve_ready(const sso_problem* p, int32_t* ready) {
  if (!p || !ready || !p->in_batch) return SSO_EINVAL;
  *ready = p->direct && p->direct_steps == 0 && plan_pending(p) ? 0 : 1;
  return SSO_OK;
}

int sso_batch_launch(sso_batch* b, sso_problem* const* ps, int n, int n_iter) try {
  if (!b || (n > 0 && !ps) || n < 0 || n_iter < 0 || b->pending) return SSO_EINVAL;
  for (int i = 0; i < n; ++i) {
    sso_problem* p = ps[i];
    if (!p || !p->in_batch || p->s != b->s || p->batch_pending) return SSO_EINVAL;
    for (int k = 0; k < i; ++k)
      if (ps[k] == p) return SSO_EINVAL;   // a problem listed twice would advance twice
  }
  b->listed.assign(ps, ps + n);
  b->n_iter = n_iter;
  b->steps.assign(n, 0);
  std::vector<DirectJob> jobs;
  std::vector<int> all, turned;
  const int st = direct_jobs(b, false, jobs, turned);
  if (st != SSO_OK) {
    b->direct.clear();       // none of the jobs was launched
    return abandon(b, st);
  }
  for (int i = 0; i < n; ++i) all.push_back(i);
  BatchLists lists = pcg_lists(b, all);
  // a timing sample: every prof_every-th launch that holds FP64 standard problems and no other
  // kind on the batch stream (one-workgroup problems run on their own stream beside them)
  b->armed = 0;
  if (b->prof_every > 0 && n_iter > 0 && !lists.standard.empty() && lists.fused.empty() &&
      lists.standard32.empty() && lists.fused32.empty() &&
      b->prof_calls++ % b->prof_every == 0) {
    b->armed = b->prof_span < n_iter ? b->prof_span : n_iter;
    b->jn0.clear();
    for (int i : b->idx[0]) b->jn0.push_back(ps[i]->w.h_st->jn);
  }
  b->bw.time_span = b->armed;
  // what the second part needs is there before the first is enqueued
  hipError_t e = jobs.empty() ? hipSuccess : direct_batch_reserve((int)jobs.size(), b->db, b->s);
  if (e == hipSuccess) e = pcg_batch_launch(lists, n_iter, b->bw, b->s);
  if (e == hipSuccess && !jobs.empty()) e = direct_batch_launch(jobs, b->db, b->s);
  if (e != hipSuccess) return abandon(b, map_hip(e));
  for (int i = 0; i < n; ++i) ps[i]->batch_pending = true;
  b->pending = true;
  return SSO_OK;
} catch (...) {   // out of host memory for the lists
  return abandon(b, SSO_ENOMEM);
}

int sso_batch_wait(sso_batch* b, sso_problem* const* ps, int n, int32_t* done) try {
  if (!b || !b->pending || n != (int)b->listed.size() || (n > 0 && !ps)) return SSO_EINVAL;
  for (int i = 0; i < n; ++i)
    if (ps[i] != b->listed[i]) return SSO_EINVAL;
  b->pending = false;
  for (int i = 0; i < n; ++i) ps[i]->batch_pending = false;
  int st = pcg_collect(b);
  if (st != SSO_OK) return abandon(b, st);
  // the direct solver's further steps, each of which hangs on the residual of the one before, up to
  // the iterations asked for; a plan still in the making is waited for once nothing else is left
  std::vector<int> turned;                 // to PCG: their iterations are still to be run
  std::vector<DirectJob> jobs;
  for (;;) {
    st = direct_collect(b, turned);
    if (st == SSO_OK) st = direct_jobs(b, false, jobs, turned);
    if (st == SSO_OK && jobs.empty()) st = direct_jobs(b, true, jobs, turned);
    if (st != SSO_OK) return abandon(b, st);
    if (jobs.empty()) break;
    const hipError_t e = direct_batch_launch(jobs, b->db, b->s);
    if (e != hipSuccess) return abandon(b, map_hip(e));
  }
  if (!turned.empty()) {
    const BatchLists lists = pcg_lists(b, turned);
    b->bw.time_span = 0;
    const hipError_t e = pcg_batch_launch(lists, b->n_iter, b->bw, b->s);
    st = e == hipSuccess ? pcg_collect(b) : map_hip(e);
    if (st != SSO_OK) return abandon(b, st);
  }
  if (done)
    for (int i = 0; i < n; ++i) done[i] = stopped(ps[i]) ? 1 : 0;
  return SSO_OK;
} catch (...) {
  return abandon(b, SSO_ENOMEM);
}

int sso_batch_iterate(sso_batch* b, sso_problem* const* ps, int n, int n_iter, int32_t* done) {
  const int st = sso_batch_launch(b, ps, n, n_iter);
  if (st != SSO_OK) return st;
  return sso_batch_wait(b, ps, n, done);
}

int sso_problem_set_stream(sso_problem* p, hipStream_t stream) {
  if (!p || p->batch_pending) return SSO_EINVAL;
  if (stream == p->s) return SSO_OK;
  if (!p->ev_move) TRY_HIP(hipEventCreateWithFlags(&p->ev_move, hipEventDisableTiming));
  TRY_HIP(hipEventRecord(p->ev_move, p->s));
  TRY_HIP(hipStreamWaitEvent(stream, p->ev_move, 0));
  p->s = stream;
  return SSO_OK;
}

int sso_batch_profile(sso_batch* b, int every, int span) {
  if (!b || every < 0 || span < 0 || (every > 0 && span == 0) || b->pending) return SSO_EINVAL;
  if (every > 0 && !b->bw.ev_t0) {
    int dev = 0, cur = 0;
    TRY_HIP(hipStreamGetDevice(b->s, &dev));
    TRY_HIP(hipGetDevice(&cur));
    if (cur != dev) TRY_HIP(hipSetDevice(dev));
    hipError_t e = hipEventCreate(&b->bw.ev_t0);
    if (e == hipSuccess) e = hipEventCreate(&b->bw.ev_t1);
    if (cur != dev) (void)hipSetDevice(cur);
    TRY_HIP(e);
  }
  b->prof_every = every;
  b->prof_span = span;
  b->prof_calls = 0;
  b->prof_us = b->prof_bytes = b->prof_bytes_read = 0.0;
  b->prof_iters = 0;
  return SSO_OK;
}

int sso_batch_timing(const sso_batch* b, double* us, int64_t* iters, double* bytes,
                     double* bytes_read) {
  if (!b) return SSO_EINVAL;
  if (us) *us = b->prof_us;
  if (iters) *iters = b->prof_iters;
  if (bytes) *bytes = b->prof_bytes;
  if (bytes_read) *bytes_read = b->prof_bytes_read;
  return SSO_OK;
}

void sso_batch_destroy(sso_batch* b) {
  if (!b) return;
  for (sso_problem* p : b->listed)   // a launch never waited for: its problems are free again
    if (b->pending && p) p->batch_pending = false;
  batch_free(b->bw, b->s);
  direct_batch_free(b->db, b->s);
  (void)hipStreamSynchronize(b->s);
  delete b;
}

int sso_objective(sso_problem* p, int kind, const double* a, double* g_host) {
  if (!p || !g_host || !p->solved) return SSO_EINVAL;
  const double* lhs;
  double scale = 1.0;
  const double* load = p->fm ? p->fm : p->f;
  if (kind == SSO_OBJ_COMPLIANCE) {
    lhs = load;
  } else if (kind == SSO_OBJ_STRAIN_ENERGY) {
    lhs = load;
    scale = 0.5;
  } else if (kind == SSO_OBJ_LINEAR && a) {
    lhs = a;
  } else {
    return SSO_EINVAL;
  }
  const int64_t n = 6 * (int64_t)p->m.n_nodes;
  TRY_HIP(launch_dot(lhs, p->u, n, p->w, p->h_scal, p->s));
  TRY_HIP(hipStreamSynchronize(p->s));
  *g_host = scale * p->h_scal[0];
  return SSO_OK;
}

int sso_adjoint(sso_problem* p, int kind, const double* dg_du, double* dg_dxyz, double* dg_dt,
                double* dg_dscale, sso_stats* stats) {
  if (!p || !p->solved || !dg_dxyz) return SSO_EINVAL;
  AllocScope ac(&p->bytes, &p->mem);
  hipStream_t s = p->s;
  double c_lam = 1.0, c_u = 1.0;
  const double* lam = p->u;
  int iters = 0, status = SSO_OK;
  bool tailed = false;
  auto terms = [&] {
    hipError_t e = launch_adjoint_terms(p->m, p->pat, p->u, lam, c_lam, c_u, p->gbeam, p->gquad, s);
    if (e == hipSuccess)
      e = launch_gather(p->m, p->pat, p->gbeam, p->gquad, dg_dxyz, dg_dt, dg_dscale, s);
    return e == hipSuccess ? hipEventRecord(p->ev[5], s) : e;
  };
  TRY_HIP(hipEventRecord(p->ev[4], s));
  if (kind == SSO_OBJ_COMPLIANCE || kind == SSO_OBJ_STRAIN_ENERGY) {
    if (kind == SSO_OBJ_STRAIN_ENERGY) c_lam = c_u = 0.5;
    if (p->fm) {
      // prescribed displacements: u solves the lifted system, so K lambda = f needs a solve
      int outer = 0;
      lam = p->lam;
      status = run_solver(p, p->fm, p->lam, &iters, &outer, std::ref(terms), &tailed);
      if (status != SSO_OK && status != SSO_ENOTCONV) return status;
    }
  } else if (kind == SSO_OBJ_LINEAR || kind == SSO_OBJ_USER) {
    if (!dg_du) return SSO_EINVAL;
    c_u = 0.0;
    TRY_HIP(launch_mask_vector(p->m, dg_du, p->rhs, s));
    int outer = 0;
    lam = p->lam;
    status = run_solver(p, p->rhs, p->lam, &iters, &outer, std::ref(terms), &tailed);
    if (status != SSO_OK && status != SSO_ENOTCONV) return status;
  } else {
    return SSO_EINVAL;
  }
  if (!tailed) {
    TRY_HIP(terms());
    TRY_HIP(hipStreamSynchronize(s));
  }
  if (stats) {
    std::memset(stats, 0, sizeof(*stats));
    stats->iters = iters;
    stats->t_adj_us = elapsed_us(p->ev[4], p->ev[5]);
    stats->bytes_moved = solve_bytes(p, iters, 0, true);
  }
  return status;
}

int sso_size_objective(sso_problem* p, double eps1, double u_max, double t_min,
                       double* out_host, double* dg_dxyz, double* dg_dt, sso_stats* stats) {
  if (!size_args_ok(p, eps1, u_max, t_min, out_host, dg_dxyz)) return SSO_EINVAL;
  AllocScope ac(&p->bytes, &p->mem);
  if (!p->xpart) TRY_HIP(dev_alloc(&p->xpart, 2 * SIZE_XWG, p->s));
  if (!p->gw) TRY_HIP(dev_alloc(&p->gw, 14 * (int64_t)p->m.n_quads, p->s));
  if (!p->wv) TRY_HIP(dev_alloc(&p->wv, p->m.n_quads, p->s));
  return size_objective_impl(p, eps1, u_max, t_min, out_host, dg_dxyz, dg_dt, stats,
                             p->xpart, p->gw, p->wv);
}

int sso_size_penalty_update(double eps1, int violated, double kappa, double* eps1_next) {
  if (!eps1_next || !(eps1 >= 0.0) || !std::isfinite(eps1) || !(kappa > 0.0) ||
      !std::isfinite(kappa))
    return SSO_EINVAL;
  *eps1_next = violated ? eps1 * kappa : eps1 / kappa;
  return SSO_OK;
}

int sso_size_objective_noalloc(sso_problem* p, double eps1, double u_max, double t_min,
                               double* out_host, double* dg_dxyz, double* dg_dt,
                               sso_stats* stats) {
  if (p && p->m.n_quads > SSO_NOALLOC_MAX_QUADS) return SSO_ESIZE;
  if (!size_args_ok(p, eps1, u_max, t_min, out_host, dg_dxyz)) return SSO_EINVAL;
  double* base = nullptr;
  const int st = scratch_address(p->device, &base);
  if (st != SSO_OK) return st;
  // partials, then the per-quad volume terms and shares; every entry is written before it is
  // read, so nothing needs clearing between calls
  double* xpart = base;
  double* gw = xpart + 2 * SIZE_XWG;
  double* wv = gw + 14 * (int64_t)p->m.n_quads;
  return size_objective_impl(p, eps1, u_max, t_min, out_host, dg_dxyz, dg_dt, stats, xpart, gw,
                             wv);
}

int sso_hat_filter(sso_problem* p, int32_t n, const int32_t* nodes, const double* g,
                   double radius, double* out) {
  if (!p || n < 0 || (n > 0 && (!g || !out)) || !(radius > 0.0) || !std::isfinite(radius))
    return SSO_EINVAL;
  if (!nodes && n > p->m.n_nodes) return SSO_EINVAL;
  hipStream_t s = p->s;
  TRY_HIP(hipMemsetAsync(p->d_err, 0, sizeof(unsigned), s));
  TRY_HIP(launch_hat_filter(n, nodes, p->m, g, radius, out, p->d_err, s));
  return read_errors(p);
}

int sso_pattern(sso_problem* p, const int32_t** row_ptr, const int32_t** col,
                const int32_t** perm, const int32_t** seg, int64_t* nnz, int64_t* n_coo) {
  if (!p) return SSO_EINVAL;
  if (p->n_coo >= ((int64_t)1 << 31) || 36 * p->pat.n_blocks >= ((int64_t)1 << 31))
    return SSO_EINVAL;
  AllocScope ac(&p->bytes, &p->mem);
  const int64_t nz = 36 * p->pat.n_blocks;
  hipStream_t s = p->s;
  if (!p->scalar_view) {
    if (!p->row_ptr) TRY_HIP(dev_alloc(&p->row_ptr, 6 * (int64_t)p->m.n_nodes + 1, s));
    if (!p->col) TRY_HIP(dev_alloc(&p->col, nz, s));
    if (!p->perm) TRY_HIP(dev_alloc(&p->perm, p->n_coo, s));
    if (!p->seg) TRY_HIP(dev_alloc(&p->seg, nz + 1, s));
    TRY_HIP(build_scalar_view(p->m, p->pat, p->row_ptr, p->col, p->perm, p->seg, p->s));
    TRY_HIP(hipStreamSynchronize(p->s));
    p->scalar_view = true;
  }
  if (row_ptr) *row_ptr = p->row_ptr;
  if (col) *col = p->col;
  if (perm) *perm = p->perm;
  if (seg) *seg = p->seg;
  if (nnz) *nnz = nz;
  if (n_coo) *n_coo = p->n_coo;
  return SSO_OK;
}

int sso_matrix(sso_problem* p, double* vals, double* f) {
  if (!p || !vals) return SSO_EINVAL;
  TRY_HIP(launch_scalar_values(p->m, p->pat, p->K, vals, p->s));
  if (f)
    TRY_HIP(hipMemcpyAsync(f, p->f, sizeof(double) * 6 * (size_t)p->m.n_nodes,
                           hipMemcpyDeviceToDevice, p->s));
  TRY_HIP(hipStreamSynchronize(p->s));
  return SSO_OK;
}

int sso_problem_bytes(const sso_problem* p, int64_t* bytes) {
  if (!p || !bytes) return SSO_EINVAL;
  *bytes = p->bytes;
  return SSO_OK;
}

int sso_sizes(const sso_problem* p, int64_t* n_dof, int64_t* n_blocks, int64_t* nnz) {
  if (!p) return SSO_EINVAL;
  if (n_dof) *n_dof = 6 * (int64_t)p->m.n_nodes;
  if (n_blocks) *n_blocks = p->pat.n_blocks;
  if (nnz) *nnz = 36 * p->pat.n_blocks;
  return SSO_OK;
}

const char* sso_strerror(int status) {
  switch (status) {
    case SSO_OK: return "ok";
    case SSO_EINVAL: return "invalid argument or degenerate element";
    case SSO_ENOMEM: return "device memory allocation failed";
    case SSO_EHIP: return "HIP runtime error";
    case SSO_ENOTCONV: return "PCG did not reach the residual target within max_it";
    case SSO_EBREAKDOWN: return "PCG breakdown: stiffness not positive definite";
    case SSO_ESIZE: return "problem larger than the static scratch of the no-allocation entry point";
    default: return "unknown status";
  }
}

void sso_problem_destroy(sso_problem* p) { free_problem(p); }

int sso_pool_trim(int device, uint64_t keep_bytes) {
  if (device < 0 || device >= MAX_DEVICES) return SSO_EINVAL;
  hipMemPool_t pool = nullptr;
  {
    std::lock_guard<std::mutex> lock(pool_mutex);
    pool = pools[device];
  }
  if (!pool) return SSO_OK;
  {
    int cur = 0;
    TRY_HIP(hipGetDevice(&cur));
    if (cur != device) TRY_HIP(hipSetDevice(device));
    cache_flush(chunk_caches[device], nullptr);
    const hipError_t e = hipStreamSynchronize(nullptr);
    if (cur != device) (void)hipSetDevice(cur);
    TRY_HIP(e);
  }
  TRY_HIP(hipMemPoolTrimTo(pool, (size_t)keep_bytes));
  return SSO_OK;
}

}  // extern "C"
