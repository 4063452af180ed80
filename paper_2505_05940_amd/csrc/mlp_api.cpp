// Host side of the proposal network: layer bookkeeping and the phases of
// forward, backward and Adam that the kernel of mlp_kernels.hip runs.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/mlp.h"
#include "../../include/modal.h"
#include "mlp_kernels.h"

using namespace modal;

namespace {
thread_local std::string g_mlp_err;
int mfail(int code, const std::string& m) {
  g_mlp_err = m;
  if (code == MODAL_EHIP || code == MODAL_ENOMEM) (void)hipGetLastError();  // the launches read the last error
  return code;
}
#define MHIP(expr)                                                                     \
  do {                                                                                 \
    hipError_t e_ = (expr);                                                            \
    if (e_ != hipSuccess)                                                              \
      return mfail(MODAL_EHIP, std::string(#expr) + ": " + hipGetErrorString(e_));     \
  } while (0)
typedef unsigned short u16;
// whole fragments along a product's sum index, whole row blocks along the rows
// (of a matrix that is also stored along its columns: along both)
long long up16(long long n) { return (n + 15) / 16 * 16; }
long long up32(long long n) { return (n + 31) / 32 * 32; }
bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }
}  // namespace

struct mlp_ctx {
  int L = 0, max_batch = 0, last_batch = 0;
  std::vector<int> dims;
  std::vector<long long> w_off, b_off;
  long long n_params = 0;
  float *p = nullptr, *g = nullptr, *m = nullptr, *v = nullptr;
  // BF16 operands of the products, all in one allocation: of layer l the
  // weights along the inputs (wf) and along the outputs (wt) and its input
  // along the features (a1) and along the batch (a2), the network's input
  // twice (x1, x2: an epoch converts the next batch while one is in use);
  // gradients along the features (g1, those of two neighbouring layers) and
  // along the batch (g2) with their row blocks' column sums (cs), which wait
  // one phase longer
  u16* ops = nullptr;
  std::vector<u16*> wf, wt, a1, a2;
  u16 *x1[2] = {}, *x2[2] = {}, *g1[2] = {}, *g2[3] = {};
  float *fl = nullptr, *cs[3] = {}, *lpart = nullptr;
  int n_lpart = 0;
  // mlp_train_epoch: Adam's step count so far and the recorded epochs, each
  // with the device table its Adam steps read (learning rate, then the bias
  // corrections 1 - beta1^t, 1 - beta2^t of each step) and the host copy it
  // was last filled from
  int t = 0;
  hipStream_t cap = nullptr;
  struct Epoch {
    const float *X, *Z;
    const int64_t* order;
    int n_steps, B;
    float b1, b2, eps;
    float* loss;
    hipGraphExec_t exec;
    float* sched;
    std::vector<float> host;
    hipEvent_t copied;  // the last copy from `host` has been made
  };
  std::vector<Epoch> epochs;
};

namespace {

void cut(MlpJob& j, int width) {
  j.width = width;
  j.mt = (int)(up32(j.M) / 32);
  j.inv_mt = 0xffffffffu / (unsigned)j.mt;
  j.blocks = (int)((long long)j.mt * ((j.N + width - 1) / width));
}

MlpJob tiles(int M, int N) {
  MlpJob j = {};
  j.M = M;
  j.N = N;
  cut(j, 64);
  return j;
}

// The product's sum over K: slices of whole 64s, as many as give about 1024
// of them over all tiles (results depend on the sizes alone).  Tiles half as wide
// where the wide ones leave CUs idle: an epoch of 32 batches of 128 / 1024
// rows takes 2.16 / 2.63 ms with wide tiles only, 2.06 / 2.52 ms with this.
void sum_over(MlpJob& j, int K) {
  const int by64 = (K + 63) / 64;
  const long long n = j.blocks;
  const int want = (int)std::max(1LL, std::min({(long long)kMlpSlices, (long long)by64, (1024 + n - 1) / n}));
  j.nk = (int)(up16(K) / 16);
  j.ks = (by64 + want - 1) / want * 4;
  j.slices = (j.nk + j.ks - 1) / j.ks;
  if (n < 256) cut(j, 32);
}

// Adam's coefficients: the host's, or the schedule's of an epoch's step
struct Adam {
  float lr, b1, b2, eps;
  int t;
  const float* sched;
  int k;
};
void set_adam(MlpPhase& P, const Adam& a) {
  P.lr = a.lr;
  P.b1 = a.b1;
  P.b2 = a.b2;
  P.eps = a.eps;
  P.c1 = 1.f - powf(a.b1, (float)a.t);
  P.c2 = 1.f - powf(a.b2, (float)a.t);
  P.sched = a.sched;
  P.k = a.k;
}

// layer l's weights as operands, from the tile that holds them
void weight_operands(const mlp_ctx* c, int l, MlpJob& j) {
  j.o1 = c->wf[l];
  j.o1kt = (int)(up16(c->dims[l]) / 16);
  j.o2 = c->wt[l];
  j.o2kt = (int)(up32(c->dims[l + 1]) / 16);
}

void adam_weights(const mlp_ctx* c, int l, MlpJob& j) {
  j.p = c->p + c->w_off[l];
  j.m = c->m + c->w_off[l];
  j.v = c->v + c->w_off[l];
  j.bp = c->p + c->b_off[l];
  j.bm = c->m + c->b_off[l];
  j.bv = c->v + c->b_off[l];
  weight_operands(c, l, j);
}

// rows of the parameter arrays are whole aligned groups of four floats
int param_vec(const mlp_ctx* c, int l) { return c->dims[l] % 4 == 0 && c->w_off[l] % 4 == 0; }

// Every layer's operands from the parameters (a null), or an Adam step on the
// stored gradients first.
int weight_jobs(mlp_ctx* c, const Adam* a, hipStream_t s) {
  for (int l = 0; l < c->L;) {
    MlpPhase P = {};
    if (a) set_adam(P, *a);
    for (int k = 0; k < kMlpJobs && l < c->L; ++k, ++l) {
      MlpJob& j = P.job[k] = tiles(c->dims[l + 1], c->dims[l]);
      j.vec = param_vec(c, l);
      j.src = (a ? c->g : c->p) + c->w_off[l];
      weight_operands(c, l, j);
      if (a) {
        adam_weights(c, l, j);
        j.bg = c->g + c->b_off[l];
        j.bsum = j.bg;
        j.n_bsum = 1;
      }
    }
    MHIP(launch_mlp_phase(P, s));
  }
  return MODAL_OK;
}

// rows of x (idx or consecutive) as the network's input, buffer i
MlpJob input_job(const mlp_ctx* c, const float* x, const int64_t* idx, int B, int i) {
  MlpJob j = tiles(B, c->dims[0]);
  j.vec = c->dims[0] % 4 == 0 && aligned16(x);
  j.src = x;
  j.idx = reinterpret_cast<const long long*>(idx);
  j.o1 = c->x1[i];
  j.o1kt = (int)(up16(c->dims[0]) / 16);
  j.o2 = c->x2[i];
  j.o2kt = (int)(up32(c->max_batch) / 16);
  return j;
}

// the gradient at layer l's output, as operands and column sums
void output_gradient(const mlp_ctx* c, int l, MlpJob& j) {
  j.o1 = c->g1[l & 1];
  j.o1kt = (int)(up16(c->dims[l + 1]) / 16);
  j.o2 = c->g2[l % 3];
  j.o2kt = (int)(up32(c->max_batch) / 16);
  j.csum = c->cs[l % 3];
}

// The layers on input buffer i.  The last one stores y, or (Z) turns the
// output into the gradient of the mean squared error.
int forward_layers(mlp_ctx* c, int B, int i, float* y, const float* Z, const int64_t* idx, hipStream_t s) {
  c->a1[0] = c->x1[i];
  c->a2[0] = c->x2[i];
  for (int l = 0; l < c->L; ++l) {
    const int in = c->dims[l], out = c->dims[l + 1];
    MlpPhase P = {};
    MlpJob& j = P.job[0] = tiles(B, out);
    j.A = c->a1[l];
    j.B = c->wf[l];
    j.akt = j.bkt = (int)(up16(in) / 16);
    sum_over(j, in);
    j.bias = c->p + c->b_off[l];
    if (l + 1 < c->L) {
      j.relu = 1;
      j.o1 = c->a1[l + 1];
      j.o1kt = (int)(up16(out) / 16);
      j.o2 = c->a2[l + 1];
      j.o2kt = (int)(up32(c->max_batch) / 16);
    } else if (Z) {
      j.Z = Z;
      j.zidx = reinterpret_cast<const long long*>(idx);
      P.inv = 1.f / ((float)B * (float)out);
      P.lpart = c->lpart;
      c->n_lpart = j.blocks;
      output_gradient(c, l, j);
    } else {
      j.C = y;
      j.vec = out % 4 == 0 && aligned16(y);
    }
    MHIP(launch_mlp_phase(P, s));
  }
  c->last_batch = B;
  return MODAL_OK;
}

// The gradients for the last layer's output gradient.  A phase takes the
// gradient back through layer l and forms the weight gradient of layer l + 1
// (with a, its Adam step too: nothing reads those weights any more); the last
// phase forms those of the first two layers.  The first phase adds the loss
// and converts the next batch (`next`), if asked.
int backward_layers(mlp_ctx* c, const Adam* a, float* loss, const MlpJob* next, hipStream_t s) {
  const int B = c->last_batch, bkt = (int)(up32(c->max_batch) / 16);
  for (int l = c->L - 1; l >= 0; --l) {
    MlpPhase P = {};
    if (a) set_adam(P, *a);
    int n = 0;
    if (l > 0) {
      const int in = c->dims[l], out = c->dims[l + 1];
      MlpJob& j = P.job[n++] = tiles(B, in);
      j.A = c->g1[l & 1];
      j.akt = (int)(up16(out) / 16);
      sum_over(j, out);
      j.B = c->wt[l];
      j.bkt = (int)(up32(out) / 16);
      j.mask = c->a1[l];
      j.mkt = (int)(up16(in) / 16);
      output_gradient(c, l - 1, j);
    }
    for (int w : {l + 1, 0}) {
      if (w >= c->L || (w == 0 && l > 0)) continue;
      const int in = c->dims[w], out = c->dims[w + 1];
      MlpJob& j = P.job[n++] = tiles(out, in);
      j.A = c->g2[w % 3];
      j.B = c->a2[w];
      j.akt = j.bkt = bkt;
      sum_over(j, B);
      j.vec = param_vec(c, w);
      j.C = c->g + c->w_off[w];
      j.bg = c->g + c->b_off[w];
      j.bsum = c->cs[w % 3];
      j.n_bsum = (int)(up32(B) / 32);
      if (a) adam_weights(c, w, j);
    }
    if (l == c->L - 1) {
      if (loss) {
        P.loss = loss;
        P.inv = 1.f / ((float)B * (float)c->dims[c->L]);
        P.lpart = c->lpart;
        P.n_lpart = c->n_lpart;
      }
      if (next) P.job[n++] = *next;
    }
    MHIP(launch_mlp_phase(P, s));
  }
  return MODAL_OK;
}

}  // namespace

extern "C" {

const char* mlp_last_error(void) { return g_mlp_err.c_str(); }

void mlp_destroy(mlp_ctx* c) {
  if (!c) return;
  for (void* q : {(void*)c->p, (void*)c->g, (void*)c->m, (void*)c->v, (void*)c->ops, (void*)c->fl})
    if (q) (void)hipFree(q);
  for (auto& e : c->epochs) {
    (void)hipGraphExecDestroy(e.exec);
    (void)hipFree(e.sched);
    if (e.copied) (void)hipEventDestroy(e.copied);
  }
  if (c->cap) (void)hipStreamDestroy(c->cap);
  delete c;
}

int mlp_init(mlp_ctx** out, int32_t n_layers, const int32_t* dims, int32_t max_batch, void* stream) {
  if (!out || n_layers < 1 || !dims || max_batch < 1) return mfail(MODAL_EINVAL, "bad arguments");
  *out = nullptr;
  for (int l = 0; l <= n_layers; ++l)
    if (dims[l] < 1 || dims[l] > (1 << 16)) return mfail(MODAL_EINVAL, "layer width out of range");
  mlp_ctx* c = new mlp_ctx();
  c->L = n_layers;
  c->max_batch = max_batch;
  c->dims.assign(dims, dims + n_layers + 1);
  for (int l = 0; l < n_layers; ++l) {
    c->w_off.push_back(c->n_params);
    c->n_params += (long long)dims[l] * dims[l + 1];
    c->b_off.push_back(c->n_params);
    c->n_params += dims[l + 1];
  }
  hipStream_t s = (hipStream_t)stream;
  const size_t pb = sizeof(float) * (size_t)c->n_params;
  float** bufs[] = {&c->p, &c->g, &c->m, &c->v};
  for (float** b : bufs) {
    if (hipMalloc((void**)b, pb) != hipSuccess) {
      mlp_destroy(c);
      return mfail(MODAL_ENOMEM, "hipMalloc params");
    }
    if (hipMemsetAsync(*b, 0, pb, s) != hipSuccess) {
      mlp_destroy(c);
      return mfail(MODAL_EHIP, "memset");
    }
  }
  // two passes over the same list: sizes, then addresses
  const long long nb = up32(max_batch);
  int max_out = 1;
  for (int l = 1; l <= n_layers; ++l) max_out = std::max(max_out, dims[l]);
  c->wf.resize(n_layers), c->wt.resize(n_layers), c->a1.resize(n_layers), c->a2.resize(n_layers);
  const size_t blocks = (size_t)nb / 32;
  size_t n_ops = 0;
  for (int pass = 0; pass < 2; ++pass) {
    size_t at = 0;
    auto take = [&](u16*& q, long long rows, long long k) {
      q = c->ops + at;  // whole fragments of 512 elements
      at += (size_t)rows * (size_t)k;
    };
    for (int l = 0; l < n_layers; ++l) {
      take(c->wf[l], up32(dims[l + 1]), up16(dims[l]));
      take(c->wt[l], up32(dims[l]), up32(dims[l + 1]));
      if (l) take(c->a1[l], nb, up16(dims[l])), take(c->a2[l], up32(dims[l]), nb);
    }
    for (u16*& q : c->x1) take(q, nb, up16(dims[0]));
    for (u16*& q : c->x2) take(q, up32(dims[0]), nb);
    for (u16*& q : c->g1) take(q, nb, up16(max_out));
    for (u16*& q : c->g2) take(q, up32(max_out), nb);
    n_ops = at;
    if (!pass && hipMalloc((void**)&c->ops, sizeof(u16) * n_ops) != hipSuccess) {
      mlp_destroy(c);
      return mfail(MODAL_ENOMEM, "hipMalloc operands");
    }
  }
  c->a1[0] = c->x1[0], c->a2[0] = c->x2[0];
  const size_t n_cs = blocks * (size_t)max_out, n_lp = blocks * (size_t)(up32(dims[n_layers]) / 32);
  if (hipMalloc((void**)&c->fl, sizeof(float) * (3 * n_cs + n_lp)) != hipSuccess) {
    mlp_destroy(c);
    return mfail(MODAL_ENOMEM, "hipMalloc sums");
  }
  for (int i = 0; i < 3; ++i) c->cs[i] = c->fl + i * n_cs;
  c->lpart = c->fl + 3 * n_cs;
  // zero weights; what the operands hold past their rows and columns stays zero
  if (hipMemsetAsync(c->ops, 0, sizeof(u16) * n_ops, s) != hipSuccess) {
    mlp_destroy(c);
    return mfail(MODAL_EHIP, "memset");
  }
  *out = c;
  return MODAL_OK;
}

int mlp_n_params(const mlp_ctx* c, int64_t* n) {
  if (!c || !n) return mfail(MODAL_EINVAL, "NULL");
  *n = c->n_params;
  return MODAL_OK;
}

int mlp_set_params(mlp_ctx* c, const float* host, void* stream) {
  if (!c || !host) return mfail(MODAL_EINVAL, "NULL");
  hipStream_t s = (hipStream_t)stream;
  MHIP(hipMemcpyAsync(c->p, host, sizeof(float) * (size_t)c->n_params, hipMemcpyHostToDevice, s));
  MHIP(hipMemsetAsync(c->m, 0, sizeof(float) * (size_t)c->n_params, s));
  MHIP(hipMemsetAsync(c->v, 0, sizeof(float) * (size_t)c->n_params, s));
  int r = weight_jobs(c, nullptr, s);
  if (r) return r;
  MHIP(hipStreamSynchronize(s));
  c->t = 0;
  return MODAL_OK;
}

int mlp_get(mlp_ctx* c, int32_t which, float* host, void* stream) {
  if (!c || !host || which < 0 || which > 1) return mfail(MODAL_EINVAL, "bad arguments");
  hipStream_t s = (hipStream_t)stream;
  MHIP(hipMemcpyAsync(host, which == 0 ? c->p : c->g, sizeof(float) * (size_t)c->n_params,
                      hipMemcpyDeviceToHost, s));
  MHIP(hipStreamSynchronize(s));
  return MODAL_OK;
}

int mlp_forward(mlp_ctx* c, const float* x, int32_t B, float* y, void* stream) {
  if (!c || !x || !y || B < 1 || B > c->max_batch) return mfail(MODAL_EINVAL, "bad arguments");
  hipStream_t s = (hipStream_t)stream;
  MlpPhase P = {};
  P.job[0] = input_job(c, x, nullptr, B, 0);
  MHIP(launch_mlp_phase(P, s));
  return forward_layers(c, B, 0, y, nullptr, nullptr, s);
}

int mlp_backward(mlp_ctx* c, const float* dy, void* stream) {
  if (!c || !dy || c->last_batch < 1) return mfail(MODAL_ESTATE, "backward needs a forward first");
  hipStream_t s = (hipStream_t)stream;
  const int d = c->dims[c->L];
  MlpPhase P = {};
  MlpJob& j = P.job[0] = tiles(c->last_batch, d);
  j.vec = d % 4 == 0 && aligned16(dy);
  j.src = dy;
  output_gradient(c, c->L - 1, j);
  MHIP(launch_mlp_phase(P, s));
  return backward_layers(c, nullptr, nullptr, nullptr, s);
}

int mlp_train_step(mlp_ctx* c, const float* X, const float* Z, const int64_t* idx, int32_t B, float lr,
                   float beta1, float beta2, float eps, int32_t t, float* loss_acc, void* stream) {
  if (!c || !X || !Z || !idx || B < 1 || B > c->max_batch || t < 1) return mfail(MODAL_EINVAL, "bad arguments");
  hipStream_t s = (hipStream_t)stream;
  MlpPhase P = {};
  P.job[0] = input_job(c, X, idx, B, 0);
  MHIP(launch_mlp_phase(P, s));
  int r = forward_layers(c, B, 0, nullptr, Z, idx, s);
  if (r) return r;
  const Adam a = {lr, beta1, beta2, eps, t, nullptr, 0};
  return backward_layers(c, &a, loss_acc, nullptr, s);
}

int mlp_train_epoch(mlp_ctx* c, const float* X, const float* Z, const int64_t* order, int32_t n_steps,
                    int32_t B, float lr, float beta1, float beta2, float eps, float* loss_acc, void* stream) {
  if (!c || !X || !Z || !order || n_steps < 1 || B < 1 || B > c->max_batch)
    return mfail(MODAL_EINVAL, "bad arguments");
  hipStream_t s = (hipStream_t)stream;
  mlp_ctx::Epoch* ep = nullptr;
  for (auto& e : c->epochs)
    if (e.X == X && e.Z == Z && e.order == order && e.n_steps == n_steps && e.B == B && e.b1 == beta1 &&
        e.b2 == beta2 && e.eps == eps && e.loss == loss_acc)
      ep = &e;
  if (!ep) {
    float* sched = nullptr;
    MHIP(hipMalloc((void**)&sched, sizeof(float) * (1 + 2 * (size_t)n_steps)));
    hipGraphExec_t exec = nullptr;
    // record the epoch once on a private stream (the caller's may be the
    // legacy default stream, which cannot be captured)
    if (!c->cap) MHIP(hipStreamCreateWithFlags(&c->cap, hipStreamNonBlocking));
    hipGraph_t graph;
    MHIP(hipStreamBeginCapture(c->cap, hipStreamCaptureModeThreadLocal));
    int r = MODAL_OK;
    // each step's first backward phase converts the next step's batch
    MlpPhase first = {};
    first.job[0] = input_job(c, X, order, B, 0);
    hipError_t le = launch_mlp_phase(first, c->cap);
    if (le != hipSuccess) r = mfail(MODAL_EHIP, std::string("recording an epoch: ") + hipGetErrorString(le));
    for (int st = 0; st < n_steps && !r; ++st) {
      const int64_t* ix = order + (long long)st * B;
      r = forward_layers(c, B, st & 1, nullptr, Z, ix, c->cap);
      if (r) break;
      const Adam a = {0.f, beta1, beta2, eps, 1, sched, st};
      const MlpJob next = st + 1 < n_steps ? input_job(c, X, ix + B, B, (st + 1) & 1) : MlpJob();
      r = backward_layers(c, &a, loss_acc, st + 1 < n_steps ? &next : nullptr, c->cap);
    }
    hipError_t e = hipStreamEndCapture(c->cap, &graph);
    if (!r && e != hipSuccess) r = mfail(MODAL_EHIP, std::string("hipStreamEndCapture: ") + hipGetErrorString(e));
    if (!r) {
      e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
      (void)hipGraphDestroy(graph);
      if (e != hipSuccess) r = mfail(MODAL_EHIP, std::string("hipGraphInstantiate: ") + hipGetErrorString(e));
    }
    if (r) {
      (void)hipFree(sched);
      return r;
    }
    hipEvent_t ev = nullptr;
    e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
    if (e != hipSuccess) {
      (void)hipGraphExecDestroy(exec);
      (void)hipFree(sched);
      return mfail(MODAL_EHIP, std::string("hipEventCreate: ") + hipGetErrorString(e));
    }
    c->epochs.push_back({X, Z, order, n_steps, B, beta1, beta2, eps, loss_acc, exec, sched, {}, ev});
    ep = &c->epochs.back();
  } else {
    MHIP(hipEventSynchronize(ep->copied));  // before its host table is rewritten
  }
  // this epoch's schedule, the corrections formed on the host as
  // mlp_adam_step forms them
  std::vector<float>& h = ep->host;
  h.assign(1 + 2 * (size_t)n_steps, 0.f);
  h[0] = lr;
  for (int k = 0; k < n_steps; ++k) {
    const float t = (float)(c->t + k + 1);
    h[1 + 2 * k] = 1.f - powf(beta1, t);
    h[2 + 2 * k] = 1.f - powf(beta2, t);
  }
  MHIP(hipMemcpyAsync(ep->sched, h.data(), sizeof(float) * h.size(), hipMemcpyHostToDevice, s));
  MHIP(hipEventRecord(ep->copied, s));
  MHIP(hipGraphLaunch(ep->exec, s));
  c->t += n_steps;
  c->last_batch = B;
  // the last batch, as the recording left it
  c->a1[0] = c->x1[(n_steps - 1) & 1];
  c->a2[0] = c->x2[(n_steps - 1) & 1];
  return MODAL_OK;
}

int mlp_adam_step(mlp_ctx* c, float lr, float b1, float b2, float eps, int32_t t, void* stream) {
  if (!c || t < 1) return mfail(MODAL_EINVAL, "bad arguments");
  const Adam a = {lr, b1, b2, eps, t, nullptr, 0};
  return weight_jobs(c, &a, (hipStream_t)stream);
}

}  // extern "C"
