// Host side of libppo_learner.so: context, argument validation, parameter layout, and the
// launch sequences of ppo_buffer_write / ppo_gae / ppo_update / distill_update.
// Every step of the learner's path runs in the HIP kernels of gemm.hip.h and mem_kernels.hip.h.
#include "../../include/ppo_learner.h"
#include "../../include/ppo_learner_diag.h"

#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <condition_variable>
#include <map>
#include <mutex>
#include <string>
#include <thread>
#include <utility>
#include <vector>

#include "gemm.hip.h"
#include "gemm_dma.hip.h"
#include "mem_kernels.hip.h"
#include "fused.hip.h"
#include "conv_tile.hip.h"
#include "conv_dgrad_tile.hip.h"
#include "conv_dgrad_wgrad0_tile.hip.h"
#include "conv_dgrad_k2_tile.hip.h"
#include "conv16_tile.hip.h"
#include "conv0_tile.hip.h"
#include "conv0_wgrad_tile.hip.h"
#include "conv_small.hip.h"
#include "small_net.hip.h"
#include "head_loss.hip.h"
#include "wgrad_rs.hip.h"
#include "peaks.hip.h"
#include "recurrent.hip.h"
#include "ln0_tile.hip.h"

static_assert(sizeof(DevStats) == sizeof(ppo_mb_stats), "device and host statistics records must match");

// Scratch of ppo_permutation_static: bucket histogram + cursors [2*nb], bucket starts [nb], bucket-ordered
// indices [S], for up to STATIC_PERM_MAX_S samples (nb <= STATIC_PERM_MAX_NB buckets of about 32 keys).  Every GPU
// the library runs on holds its own copy of this array until the process ends (4.4 MiB).
constexpr int64_t STATIC_PERM_MAX_S = 1 << 20;
constexpr int STATIC_PERM_MAX_NB = 1 << 15;
constexpr int STATIC_MAX_DEVICES = 64;
static __device__ __align__(256) int32_t scratch[3 * STATIC_PERM_MAX_NB + STATIC_PERM_MAX_S];

namespace {

thread_local std::string g_create_error;

// Device address of `scratch` on the current device.  In host code the array's name is only a stand-in for the
// symbol, not an address a kernel can use: the address is asked for once per device (with that device current)
// and kept; host code passes this pointer, never the name, to kernels.
std::mutex g_scratch_mutex;
int32_t* g_scratch_ptr[STATIC_MAX_DEVICES] = {};
hipError_t static_scratch(int32_t** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= STATIC_MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = (int32_t*)p;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

struct Ctx {
  ppo_net_desc d;
  hipStream_t stream = nullptr;
  int dev = 0;  // the HIP device the context lives on (kernel attributes are set once per device)
  std::string err;
  // geometry
  int N = 0, T = 0, S = 0, V = 1, A = 0, P = 0, NH = 0, nconv = 0, nfc = 0;
  int cC[PPO_MAX_LAYERS + 1], cH[PPO_MAX_LAYERS + 1], cW[PPO_MAX_LAYERS + 1];
  int fin[PPO_MAX_LAYERS], fout[PPO_MAX_LAYERS];
  int flat = 0, feat_ld = 0, hid = 0;
  int64_t img_elems = 0;  // stored elements per view (padded rows)
  // internal parameter layout (fp32 master, bf16 shadow share the offsets)
  int64_t convW[PPO_MAX_LAYERS], convB[PPO_MAX_LAYERS], fcW[PPO_MAX_LAYERS], fcB[PPO_MAX_LAYERS];
  int64_t headW = 0, headB = 0, logstd = -1, total = 0;
  // optional parts of the network
  int XH = 0, X = 0, A_main = 0;            // auxiliary MLP head: hidden width, outputs; rows of the linear mean head
  int64_t aux1W = -1, aux1B = -1, aux2W = -1, aux2B = -1;
  bool ln = false;                          // layer normalisation after every convolution
  int64_t lnG[PPO_MAX_LAYERS], lnB[PPO_MAX_LAYERS];
  int E = 0, enc = 0;                       // embedding width (0: none); encoder output width per view
  int64_t embW = -1, embB = -1;
  int nl = 0, H = 0, lin[4] = {0, 0, 0, 0};  // LSTM layers, units, input width per layer
  int64_t lstmW[4], lstmB[4];               // per layer [4H][lin + H] (input and recurrent weights side by side), bias [4H]
  int feat_cols = 0;                        // V*enc + P: the feature columns of a row of the feature matrix
  // workspaces of the generic encoder (layer norm and / or embedding) and of the recurrent core
  bf16_t* pre[PPO_MAX_LAYERS] = {};         // conv outputs before the layer normalisation [CH*V][Ho*Wo*Co]
  float2* lnstat[PPO_MAX_LAYERS] = {};      // (mean, rstd) per image
  bf16_t* dpre = nullptr;                   // gradient w.r.t. one convolution's output (largest layer)
  bf16_t* embT = nullptr;                   // [flat][E]
  bf16_t* lstmWT[4] = {};                   // [lin + H][4H]
  bf16_t* xh[4] = {};                       // LSTM layer inputs [CH][lin + H]: x_t, then the h entering step t (xh[0] is the feature matrix)
  bf16_t* dxh[4] = {};                      // their gradients (side by side: the bottom layer's x half)
  float* gates[4] = {};                     // [CH][4H] gate activations
  float* c_enter[4] = {};                   // [CH][H] cell state entering each step
  float* lstm_pre = nullptr;                // [CHe][4H] gate pre-activations of one step
  bf16_t* da[4] = {};                       // [CH][4H] gate pre-activation gradients
  float* dc_carry[4] = {};                  // [CHe][H]
  float* lstm_part = nullptr;               // slices of the products of the layers that run side by side
  bf16_t* htop = nullptr;                   // [CH][H] top layer's h: the trunk's input
  int32_t* seqidx = nullptr;                // [CH] rollout sample of each row of a sequence chunk
  float *h0 = nullptr, *c0 = nullptr;       // [nl][N][H] state of every environment at the start of the rollout
  int PU = 0;                               // units the minibatch permutation shuffles: N environments (recurrent) or S samples
  int CHe = 0;                              // environments per sequence chunk
  ParamMap pmap;             // internal order <-> canonical order
  float* canon = nullptr;    // device staging in canonical order for parameter / gradient / moment I/O
  float* hstage = nullptr;   // pinned host staging of the same (slots of HSTAGE elements)
  hipEvent_t hstage_ev[8] = {};
  // device: parameters
  float *p = nullptr, *m = nullptr, *v = nullptr, *g = nullptr;
  bf16_t* shadow = nullptr;
  bf16_t* wd[PPO_MAX_LAYERS][2];  // transposed-conv weights per row parity (conv layers >= 1)
  bf16_t* wtap[PPO_MAX_LAYERS];   // the same weights transposed per tap: [9][Cin][Cout]
  uint32_t* abits[PPO_MAX_LAYERS] = {};  // sign bits of conv layer l's stored output for the current chunk (ReLU mask of the backward pass)
  bool abits_ok[PPO_MAX_LAYERS] = {};    // written by the forward kernel that ran for this chunk
  bool dry = false;                      // the launchers of the first two convolutions only say whether they cover the shapes
  int b0pitch = 0;                       // words per row of abits[0] when f01_train
  bool f01_fwd = false, f01_train = false;  // those two run in one kernel: forward only / forward and backward (act[0] then stays unused)
  int64_t wver = 0;                      // bumped whenever the weights change (every repack_weights call)
  int64_t wd_ver[PPO_MAX_LAYERS] = {};   // weight version that wd[l] holds (0: none): packed on demand the first time,
  bool wd_used[PPO_MAX_LAYERS] = {};     // with every other re-pack from then on
  bf16_t* fcT[PPO_MAX_LAYERS];    // [in][out]
  bf16_t* headT = nullptr;        // [hid][32]
  bf16_t *aux1T = nullptr, *aux2T = nullptr;  // auxiliary head: [hid][XH], [XH][32]
  bf16_t *auxact = nullptr, *dauxact = nullptr, *daux = nullptr;  // its hidden activation [CH][XH], that layer's gradient, its output gradient [CH][32]
  // device: rollout buffer (SoA)
  bf16_t *obs = nullptr, *proprio = nullptr;
  float *action = nullptr, *logp = nullptr, *value = nullptr, *reward = nullptr, *adv = nullptr, *ret = nullptr;
  uint8_t* done = nullptr;
  // device: permutation
  int32_t *perm = nullptr, *ptmp = nullptr, *phist = nullptr, *pstart = nullptr;
  int nb = 1, shift = 64;
  // device: workspaces for one chunk of CH samples
  int CH = 0;
  bf16_t* act[PPO_MAX_LAYERS] = {};  // conv outputs of layers 0..nconv-2, [CH*V][H][W][C]
  bf16_t* feat = nullptr;         // [CH][feat_ld]: last conv output per view, then proprio
  bf16_t* fcact[PPO_MAX_LAYERS];  // [CH][fout]
  float* headout = nullptr;       // [CH][32]
  bf16_t* dhead = nullptr;        // [CH][32]
  bf16_t* gbuf[2] = {nullptr, nullptr};
  float *partial = nullptr, *bias_partial = nullptr;
  bf16_t* zpage = nullptr;  // 64 KiB of zeros: source of out-of-range operand fetches (most kernels use its first KiB)
  // partial / bias_partial are cursors into the two workspaces and *_elems what is left behind them:
  // every weight-gradient kernel of a backward pass takes its partials from the cursor and queues its
  // reduction (defer_reduce); flush_reduces sums them all in one launch and rewinds the cursors
  int64_t partial_elems = 0, bias_partial_elems = 0;
  float *partial_base = nullptr, *bias_partial_base = nullptr;
  int64_t partial_cap = 0, bias_partial_cap = 0;
  ReduceJobs rjobs;
  LossFinalize lossfin = {};    // pending: rides as the last block of the next reduction launch
  GnormFinalize gnfin = {}; // pending: rides as the last block of the next re-pack launch
  int rjob_blocks = 0;
  float *stat_part = nullptr, *dls_part = nullptr, *sq_part = nullptr;
  float* lr_dev = nullptr;  // the KL-adaptive learning rate (desired_kl > 0); lr_live: an adaptive update has left a rate there
  bool lr_live = false;
  float* adv_n = nullptr;  // advantages normalised over the rollout (norm_adv)
  float* advn_part = nullptr;  // per-block (count, mean, squared deviations) of that normalisation
  int max_loss_blocks = 0, adam_blocks = 0;
  DevStats* dstats = nullptr;
  int max_steps = 4096;
  // state
  std::vector<char> written;                               // per step: 0 incomplete, 1 complete, 2 acted (outcome missing)
  std::vector<std::vector<std::pair<int, int>>> cover;     // per step: merged environment ranges of partial writes
  bool gae_done = false;
  int64_t step = 0, update_idx = 0;
  std::vector<void*> allocs;
  // optional per-kernel-class timing with HIP events on the context's stream
  bool prof_on = false;
  struct ProfClass { std::string name; int64_t launches = 0; double flops = 0, bytes = 0; };
  struct ProfRec { int cls; hipEvent_t a, b; };
  std::vector<ProfClass> prof_cls;
  std::map<std::string, int> prof_idx;
  std::vector<ProfRec> prof_recs;
  std::vector<hipEvent_t> prof_pool;
};

// Brackets the launches made during its lifetime with a pair of events (when profiling is on) and
// books the algorithmic FLOPs / bytes of the work under `name`.
struct ProfScope {
  Ctx* c; int rec = -1;
  ProfScope(Ctx* c_, const std::string& name, double flops, double bytes) : c(c_) {
    if (!c->prof_on) return;
    auto it = c->prof_idx.find(name);
    int id;
    if (it == c->prof_idx.end()) { id = (int)c->prof_cls.size(); c->prof_idx[name] = id; Ctx::ProfClass pc; pc.name = name; c->prof_cls.push_back(pc); }
    else id = it->second;
    c->prof_cls[id].launches += 1; c->prof_cls[id].flops += flops; c->prof_cls[id].bytes += bytes;
    hipEvent_t ev[2];
    for (int i = 0; i < 2; ++i) {
      if (!c->prof_pool.empty()) { ev[i] = c->prof_pool.back(); c->prof_pool.pop_back(); }
      else if (hipEventCreate(&ev[i]) != hipSuccess) return;
    }
    Ctx::ProfRec r; r.cls = id; r.a = ev[0]; r.b = ev[1];
    (void)hipEventRecord(r.a, c->stream);
    rec = (int)c->prof_recs.size();
    c->prof_recs.push_back(r);
  }
  ~ProfScope() { if (rec >= 0) (void)hipEventRecord(c->prof_recs[rec].b, c->stream); }
};

int fail(Ctx* c, int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  if (c) c->err = buf; else g_create_error = buf;
  return code;
}

#define HIPCHK(c, call)                                                                          \
  do {                                                                                           \
    hipError_t e_ = (call);                                                                      \
    if (e_ != hipSuccess) return fail(c, PPO_EHIP, "%s failed: %s", #call, hipGetErrorString(e_)); \
  } while (0)
#define LAUNCHCHK(c, what)                                                                              \
  do {                                                                                                  \
    hipError_t e_ = hipGetLastError();                                                                  \
    if (e_ != hipSuccess) return fail(c, PPO_EHIP, "launch of %s failed: %s", what, hipGetErrorString(e_)); \
  } while (0)

template <typename T>
int dalloc(Ctx* c, T** out, int64_t n) {
  void* p = nullptr;
  size_t bytes = (size_t)(n > 0 ? n : 1) * sizeof(T);
  hipError_t e = hipMalloc(&p, bytes);
  if (e != hipSuccess) return fail(c, e == hipErrorOutOfMemory ? PPO_ENOMEM : PPO_EHIP, "hipMalloc of %zu bytes failed: %s", bytes, hipGetErrorString(e));
  c->allocs.push_back(p);
  *out = (T*)p;
  return PPO_OK;
}
#define DALLOC(c, ptr, n)                          \
  do {                                             \
    int rc_ = dalloc(c, &(ptr), (int64_t)(n));     \
    if (rc_ != PPO_OK) return rc_;                 \
  } while (0)

inline int cdiv(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

// ---------------------------------------------------------------- validation (no HIP calls)
int validate_desc(const ppo_net_desc* d) {
  if (!d) return fail(nullptr, PPO_EINVAL, "desc is NULL");
  if (d->num_envs < 1 || d->horizon < 1) return fail(nullptr, PPO_ESHAPE, "num_envs and horizon must be >= 1");
  if ((int64_t)d->num_envs * d->horizon > (1 << 30)) return fail(nullptr, PPO_ESHAPE, "num_envs*horizon too large");
  if (d->n_views < 1 || d->n_views > 4) return fail(nullptr, PPO_ESHAPE, "n_views must be 1..4");
  if (d->in_c != 1 && d->in_c != 3) return fail(nullptr, PPO_ESHAPE, "in_c must be 1 (depth) or 3 (RGB)");
  if (d->in_h < 2 || d->in_w < 2 || d->in_h > 4096 || d->in_w > 4096) return fail(nullptr, PPO_ESHAPE, "image size out of range");
  if (d->obs_dtype != 0 && d->obs_dtype != 1) return fail(nullptr, PPO_EINVAL, "obs_dtype must be 0 (fp32) or 1 (bf16)");
  if (d->proprio_dim < 8 || d->proprio_dim % 8) return fail(nullptr, PPO_ESHAPE, "proprio_dim must be a positive multiple of 8");
  if (d->act_dim < 1 || d->act_dim > 31) return fail(nullptr, PPO_ESHAPE, "act_dim must be 1..31");
  if (d->conv_k != 3 || d->conv_stride != 2 || d->conv_pad != 1) return fail(nullptr, PPO_ESHAPE, "only 3x3 stride-2 pad-1 convolutions are supported");
  if (d->n_conv < 2 || d->n_conv > PPO_MAX_LAYERS) return fail(nullptr, PPO_ESHAPE, "n_conv must be 2..%d", PPO_MAX_LAYERS);
  for (int i = 0; i < d->n_conv; ++i)
    if (d->conv_ch[i] < 8 || d->conv_ch[i] > 1024 || (d->conv_ch[i] & (d->conv_ch[i] - 1))) return fail(nullptr, PPO_ESHAPE, "conv_ch[%d] must be a power of two in 8..1024", i);
  if (d->conv_ch[0] != 8 && d->conv_ch[0] != 16 && d->conv_ch[0] != 32 && d->conv_ch[0] != 64) return fail(nullptr, PPO_ESHAPE, "conv_ch[0] must be 8, 16, 32 or 64");
  if (d->n_fc < 1 || d->n_fc > PPO_MAX_LAYERS) return fail(nullptr, PPO_ESHAPE, "n_fc must be 1..%d", PPO_MAX_LAYERS);
  for (int i = 0; i < d->n_fc; ++i)
    if (d->fc_dim[i] < 8 || d->fc_dim[i] % 8 || d->fc_dim[i] > 16384) return fail(nullptr, PPO_ESHAPE, "fc_dim[%d] must be a multiple of 8 in 8..16384", i);
  if (d->has_value_head != 0 && d->has_value_head != 1) return fail(nullptr, PPO_EINVAL, "has_value_head must be 0 or 1");
  if (d->max_chunk < 0) return fail(nullptr, PPO_EINVAL, "max_chunk must be >= 0");
  if (d->aux_hidden < 0 || d->aux_hidden % 8 || d->aux_hidden > 4096) return fail(nullptr, PPO_ESHAPE, "aux_hidden must be a multiple of 8 in 0..4096");
  if (d->aux_hidden > 0 && d->has_value_head) return fail(nullptr, PPO_ESHAPE, "the auxiliary MLP head belongs to a distillation student (has_value_head = 0)");
  if (d->aux_hidden > 0 && (d->aux_dim < 1 || d->aux_dim >= d->act_dim)) return fail(nullptr, PPO_ESHAPE, "aux_dim must be in 1..act_dim-1 when aux_hidden > 0");
  if (d->aux_hidden == 0 && d->aux_dim != 0) return fail(nullptr, PPO_ESHAPE, "aux_dim without aux_hidden (for auxiliary columns of the linear head use ppo_hparams.aux_dim)");
  if (d->layer_norm != 0 && d->layer_norm != 1) return fail(nullptr, PPO_EINVAL, "layer_norm must be 0 or 1");
  if (d->embed_dim < 0 || d->embed_dim % 8 || d->embed_dim > 4096) return fail(nullptr, PPO_ESHAPE, "embed_dim must be a multiple of 8 in 0..4096");
  if (d->lstm_layers < 0 || d->lstm_layers > 4) return fail(nullptr, PPO_ESHAPE, "lstm_layers must be 0..4");
  if (d->lstm_layers > 0 && (d->lstm_units < 8 || d->lstm_units % 8 || d->lstm_units > 4096)) return fail(nullptr, PPO_ESHAPE, "lstm_units must be a multiple of 8 in 8..4096");
  if (d->lstm_layers == 0 && d->lstm_units != 0) return fail(nullptr, PPO_ESHAPE, "lstm_units without lstm_layers");
  if (d->lstm_layers > 0 && !d->has_value_head) return fail(nullptr, PPO_ESHAPE, "recurrent layers are built for the actor-critic teacher (has_value_head = 1)");
  // every convolution but the first, hidden layer, head, auxiliary, embedding and LSTM matrix has a transposed copy
  if (d->n_conv - 1 + d->n_fc + 1 + (d->aux_hidden > 0 ? 2 : 0) + (d->embed_dim > 0 ? 1 : 0) + d->lstm_layers > RepackJobs::MAXT)
    return fail(nullptr, PPO_ESHAPE, "too many layers for one re-pack launch");
  return PPO_OK;
}

int validate_hp(Ctx* c, const ppo_hparams* hp, bool distill) {
  if (!hp) return fail(c, PPO_EINVAL, "hparams is NULL");
  const float f[] = {hp->clip_eps, hp->vclip_eps, hp->vf_coef, hp->ent_coef, hp->lr, hp->beta1, hp->beta2, hp->adam_eps, hp->max_grad_norm, hp->desired_kl, hp->aux_coef};
  for (float x : f) if (!isfinite(x)) return fail(c, PPO_EINVAL, "non-finite hyper-parameter");
  if (!distill && !(hp->clip_eps > 0.f)) return fail(c, PPO_EINVAL, "clip_eps must be > 0");
  if (!(hp->lr >= 0.f) || !(hp->beta1 >= 0.f && hp->beta1 < 1.f) || !(hp->beta2 >= 0.f && hp->beta2 < 1.f) || !(hp->adam_eps > 0.f))
    return fail(c, PPO_EINVAL, "Adam hyper-parameters out of range");
  if (hp->norm_adv != 0 && hp->norm_adv != 1) return fail(c, PPO_EINVAL, "norm_adv must be 0 or 1");
  if (hp->lr_carry != 0 && hp->lr_carry != 1) return fail(c, PPO_EINVAL, "lr_carry must be 0 or 1");
  if (distill && (hp->aux_dim < 0 || hp->aux_dim >= c->A)) return fail(c, PPO_EINVAL, "aux_dim must be in [0, act_dim)");
  if (distill && hp->aux_dim > 0 && !(hp->aux_coef >= 0.f)) return fail(c, PPO_EINVAL, "aux_coef must be >= 0");
  if (distill && c->XH > 0 && hp->aux_dim != c->X) return fail(c, PPO_EINVAL, "this student has an auxiliary MLP head for %d outputs: hparams.aux_dim must be %d", c->X, c->X);
  if (!distill && hp->desired_kl > 0.f && !(isfinite(hp->lr_min) && isfinite(hp->lr_max) && hp->lr_min > 0.f && hp->lr_min <= hp->lr_max))
    return fail(c, PPO_EINVAL, "desired_kl > 0 needs 0 < lr_min <= lr_max");
  if (hp->epochs < 1 || hp->minibatches < 1) return fail(c, PPO_EINVAL, "epochs and minibatches must be >= 1");
  if (c->PU % hp->minibatches)
    return fail(c, PPO_ESHAPE, "%s = %d is not divisible by minibatches = %d", c->nl > 0 ? "num_envs (a recurrent net's minibatches are whole environments)" : "num_envs*horizon",
                c->PU, hp->minibatches);
  if ((int64_t)hp->epochs * hp->minibatches > c->max_steps) return fail(c, PPO_ESHAPE, "epochs*minibatches exceeds %d", c->max_steps);
  return PPO_OK;
}

// ---------------------------------------------------------------- geometry and parameter layout
void build_geometry(Ctx* c) {
  const ppo_net_desc& d = c->d;
  c->N = d.num_envs; c->T = d.horizon; c->S = c->N * c->T; c->V = d.n_views; c->A = d.act_dim; c->P = d.proprio_dim;
  c->XH = d.aux_hidden; c->X = d.aux_hidden > 0 ? d.aux_dim : 0; c->A_main = c->A - c->X;
  c->ln = d.layer_norm != 0; c->E = d.embed_dim; c->nl = d.lstm_layers; c->H = d.lstm_layers > 0 ? d.lstm_units : 0;
  c->NH = c->A_main + (d.has_value_head ? 1 : 0);
  c->nconv = d.n_conv; c->nfc = d.n_fc;
  // stored image rows are padded with zeros to a multiple of 8 pixels (k_write_obs); every kernel takes the padded
  // width for the image's own, the first layer's output width comes from the real one
  c->cC[0] = d.in_c; c->cH[0] = d.in_h; c->cW[0] = (d.in_w + 7) / 8 * 8;
  for (int l = 0; l < c->nconv; ++l) {
    c->cC[l + 1] = d.conv_ch[l];
    c->cH[l + 1] = (c->cH[l] + 2 - 3) / 2 + 1;
    c->cW[l + 1] = ((l == 0 ? d.in_w : c->cW[l]) + 2 - 3) / 2 + 1;
  }
  c->img_elems = (int64_t)d.in_c * d.in_h * c->cW[0];
  c->flat = c->cC[c->nconv] * c->cH[c->nconv] * c->cW[c->nconv];
  c->enc = c->E > 0 ? c->E : c->flat;
  c->feat_cols = c->V * c->enc + c->P;
  // recurrent nets: a feature row is followed by the h that enters the first LSTM layer at that step (the two
  // halves of that layer's GEMM operand side by side)
  c->feat_ld = c->feat_cols + (c->nl > 0 ? c->H : 0);
  int in = c->feat_cols;
  for (int l = 0; l < c->nl; ++l) { c->lin[l] = in; in = c->H; }
  for (int l = 0; l < c->nfc; ++l) { c->fin[l] = in; c->fout[l] = d.fc_dim[l]; in = d.fc_dim[l]; }
  c->hid = in;

  // canonical offsets: per conv W, b, [gain, shift]; [embedding W, b]; per LSTM layer W_ih, W_hh, b; per hidden
  // layer W, b; mean head W, b; [value head w, b; logstd]; [auxiliary head W1, b1, W2, b2]
  std::vector<int64_t> cConvW(c->nconv), cConvB(c->nconv), cLnG(c->nconv), cLnB(c->nconv), cFcW(c->nfc), cFcB(c->nfc);
  int64_t cWih[4], cWhh[4], cLb[4], cEmbW = -1, cEmbB = -1;
  int64_t off = 0;
  for (int l = 0; l < c->nconv; ++l) {
    cConvW[l] = off; off += (int64_t)c->cC[l + 1] * c->cC[l] * 9; cConvB[l] = off; off += c->cC[l + 1];
    if (c->ln) { cLnG[l] = off; off += c->cC[l + 1]; cLnB[l] = off; off += c->cC[l + 1]; }
  }
  if (c->E > 0) { cEmbW = off; off += (int64_t)c->E * c->flat; cEmbB = off; off += c->E; }
  for (int l = 0; l < c->nl; ++l) {
    cWih[l] = off; off += (int64_t)4 * c->H * c->lin[l]; cWhh[l] = off; off += (int64_t)4 * c->H * c->H; cLb[l] = off; off += 4 * c->H;
  }
  for (int l = 0; l < c->nfc; ++l) { cFcW[l] = off; off += (int64_t)c->fin[l] * c->fout[l]; cFcB[l] = off; off += c->fout[l]; }
  int64_t cMuW = off; off += (int64_t)c->A_main * c->hid;
  int64_t cMuB = off; off += c->A_main;
  int64_t cVW = -1, cVB = -1, cLs = -1;
  if (d.has_value_head) { cVW = off; off += c->hid; cVB = off; off += 1; cLs = off; off += c->A; }
  int64_t cA1W = -1, cA1B = -1, cA2W = -1, cA2B = -1;
  if (c->XH > 0) {
    cA1W = off; off += (int64_t)c->XH * c->hid; cA1B = off; off += c->XH;
    cA2W = off; off += (int64_t)c->X * c->XH; cA2B = off; off += c->X;
  }
  c->total = off;
  ParamMap& pm = c->pmap;
  pm.nseg = 0;
  int64_t io = 0;
  // appends the internal elements [io, io + n) of one kind (ParamMap) and returns their first index
  auto seg = [&](int kind, int64_t n, int64_t co, int a = 1, int64_t co2 = 0, int lin = 0, bool flat = false) {
    ParamMap::Seg& g = pm.seg[pm.nseg++];
    g.io = io; g.co = co; g.co2 = co2; g.kind = kind; g.a = a; g.lin = lin;
    g.nperm = flat ? c->V * c->flat : 0; g.flat = c->flat; g.ch = c->cC[c->nconv]; g.pix = c->cH[c->nconv] * c->cW[c->nconv];
    io += n;
    return g.io;
  };

  // internal layout: conv W as [Co][(u*3+v)*Ci + ci]; the first layer behind the convolutions reads the
  // channel-last flatten (view, pixel, channel); LSTM input and recurrent weights side by side per gate row;
  // heads stacked as one [NH][hid] matrix.  Every matrix starts at a multiple of 8 elements (16-byte operand
  // loads from the bf16 shadow) and every bias a bf16-output epilogue reads at a multiple of 4: the vectors of
  // odd length (head biases, log-std, the auxiliary output bias) come last.
  for (int l = 0; l < c->nconv; ++l) {
    const int Co = c->cC[l + 1], Ci = c->cC[l];
    c->convW[l] = seg(ParamMap::CONV, (int64_t)Co * 9 * Ci, cConvW[l], Ci);
    c->convB[l] = seg(ParamMap::SAME, Co, cConvB[l]);
    c->lnG[l] = c->lnB[l] = -1;
    if (c->ln) { c->lnG[l] = seg(ParamMap::SAME, Co, cLnG[l]); c->lnB[l] = seg(ParamMap::SAME, Co, cLnB[l]); }
  }
  if (c->E > 0) {  // reads the flatten of one view
    c->embW = seg(ParamMap::MATRIX, (int64_t)c->E * c->flat, cEmbW, c->flat);
    ParamMap::Seg& g = pm.seg[pm.nseg - 1];
    g.nperm = g.flat;
    c->embB = seg(ParamMap::SAME, c->E, cEmbB);
  }
  const bool first_flat = c->E == 0;  // the first layer behind [encoder(view 0), ..., proprioception] reads the flatten itself
  for (int l = 0; l < c->nl; ++l) {
    const int K = c->lin[l] + c->H;
    c->lstmW[l] = seg(ParamMap::LSTM, (int64_t)4 * c->H * K, cWih[l], K, cWhh[l], c->lin[l], l == 0 && first_flat);
    c->lstmB[l] = seg(ParamMap::SAME, 4 * c->H, cLb[l]);
  }
  for (int l = 0; l < c->nfc; ++l) {
    c->fcW[l] = seg(ParamMap::MATRIX, (int64_t)c->fin[l] * c->fout[l], cFcW[l], c->fin[l], 0, 0, l == 0 && c->nl == 0 && first_flat);
    c->fcB[l] = seg(ParamMap::SAME, c->fout[l], cFcB[l]);
  }
  if (c->XH > 0) {
    c->aux1W = seg(ParamMap::SAME, (int64_t)c->XH * c->hid, cA1W);
    c->aux1B = seg(ParamMap::SAME, c->XH, cA1B);
    c->aux2W = seg(ParamMap::SAME, (int64_t)c->X * c->XH, cA2W);
  }
  c->headW = seg(ParamMap::SAME, (int64_t)c->A_main * c->hid, cMuW);
  if (d.has_value_head) seg(ParamMap::SAME, c->hid, cVW);
  c->headB = seg(ParamMap::SAME, c->A_main, cMuB);
  if (d.has_value_head) {
    seg(ParamMap::SAME, 1, cVB);
    c->logstd = seg(ParamMap::SAME, c->A, cLs);
  }
  if (c->XH > 0) c->aux2B = seg(ParamMap::SAME, c->X, cA2B);
  pm.total = io;
}

// number of input pixels of parity `par` along an axis of length n
inline int class_len(int n, int par) { return (n - par + 1) / 2; }

// ---------------------------------------------------------------- launch helpers
inline int ilog2(int x) { int l = 0; while ((1 << l) < x) ++l; return l; }

// With few tiles and short rows (<= 512 tiles of 32 x 32 at K <= 512, <= 128 at K <= 2048) the latency of an LDS ring
// is the larger part of a product with plain rows, and k_gemm_small wins (64 x 64 x 1056: 7.9 -> 4.7 us; 1250 x 128 x 256:
// 5.1 -> 3.4 us; beyond these lines its operand traffic, 32 x 32 per tile, loses: 4096 x 256 x 512: 7.0 against 9.6 us).
bool gemm_small_covers(int M, int N, int K) {
  const int64_t t32 = (int64_t)cdiv(M, 32) * cdiv(N, 32);
  return (t32 <= 512 && K <= 512) || (t32 <= 128 && K <= 2048);
}
// How a product with plain rows (C [M][N] = A [M][K] B^T) and K >= 1024 is cut up otherwise.  Every form is a chain of k-steps of 64 per tile, of
// measured length (us, operands in L2 / the last-level cache, chip full): 0.34 for a 64 x 64 tile, 0.60 for 128 x 128, 1.0
// for 256 x 128, behind 3.5 us of launch, ring fill and epilogue; a reduction over `splits` slices of K costs another 3 us
// and its fp32 partials at 6 TB/s.  The plan is the form with the smallest sum, blocks counted in rounds of 256 CUs: e.g.
// 4096 x 512 x 10304 leaves two rounds of 64 x 64 tiles (107 us) for 64 tiles of 256 x 128 in four slices (53 us);
// 16384 x 512 x 10304 stays one round of undivided 256 x 128 tiles (157 us).
struct GemmPlan { int bm, bn, splits, W; };  // splits > 1: W k-steps per slice
GemmPlan plan_gemm(int M, int N, int K, int64_t partial_elems) {
  const int nk = cdiv(K, 64);
  GemmPlan best = {64, 64, 1, nk};
  double tbest = 1e30;
  auto consider = [&](int bm, int bn, double step) {
    const int64_t tiles = (int64_t)cdiv(M, bm) * cdiv(N, bn);
    for (int s = 1; s <= 16 && (s == 1 || nk / s >= 3); ++s) {
      const int W = cdiv(nk, s);
      if (s > 1 && (cdiv(nk, W) != s || s * tiles * bm * bn > partial_elems)) continue;
      double t = 3.5 + (double)cdiv(tiles * s, 256) * W * step;
      if (s > 1) t += 3.0 + 8e-6 * s * (double)tiles * bm * bn / 6.0;
      if (t < tbest - 1e-9) { tbest = t; best = {bm, bn, s, W}; }
    }
  };
  if (N <= 32) consider(128, 32, 0.45);
  else if (N <= 64) { consider(64, 64, 0.34); consider(128, 64, 0.48); }
  else { consider(64, 64, 0.34); consider(128, 128, 0.60); consider(256, 128, 1.0); }
  return best;
}

// The LDS-ring kernel on tiles of BM x BN, undivided or in plan.splits slices of K.
template <int BM, int BN, int WM, int WN, class EP>
int launch_gemm_ring(Ctx* c, const ARows& al, int M, const bf16_t* Bm, int64_t ldb, int N, int K, const EP& ep, const GemmPlan& plan) {
  constexpr int ncw = WM * WN, nst = (BM + BN) * 128 * 8 <= 128 * 1024 ? 8 : ((BM + BN) * 128 * 4 <= 128 * 1024 ? 4 : 3), lds = nst * (BM + BN) * 128;
  static uint64_t attr_devs[2] = {0, 0};  // bit d: set on device d
  const bool split = plan.splits > 1;
  auto kfn = k_gemm_rs<BM, BN, WM, WN, nst, ARows, EP>;
  auto kfs = k_gemm_rs<BM, BN, WM, WN, nst, ARows, EpSplit>;
  const void* k = split ? (const void*)kfs : (const void*)kfn;
  if (!((attr_devs[split] >> c->dev) & 1)) { HIPCHK(c, hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, lds)); attr_devs[split] |= 1ull << c->dev; }
  if (!split) {
    hipLaunchKernelGGL(kfn, dim3(cdiv(M, BM), cdiv(N, BN)), dim3((ncw + 4) * 64), lds, c->stream, al, Bm, ldb, N, ep, c->zpage);
    return PPO_OK;
  }
  EpSplit es;
  es.map = ep.map; es.part[0] = reinterpret_cast<float*>((reinterpret_cast<uintptr_t>(c->partial) + 15) & ~(uintptr_t)15);
  es.N[0] = N; es.W[0] = plan.W; es.gy[0] = cdiv(N, BN); es.tiles[0] = cdiv(M, BM) * es.gy[0]; es.blocks[0] = es.tiles[0] * plan.splits;
  hipLaunchKernelGGL(kfs, dim3(es.blocks[0]), dim3((ncw + 4) * 64), lds, c->stream, al, Bm, ldb, N, es, c->zpage);
  hipLaunchKernelGGL((k_gemm_split_reduce<BM, BN, EP>), dim3(cdiv((int64_t)es.tiles[0] * (BM / 32) * (BN / 32), 4)), dim3(256), 0, c->stream, es.part[0], plan.splits, es.tiles[0],
                     es.gy[0], M, N, ep);
  return PPO_OK;
}

template <class AL, class EP>
int launch_gemm(Ctx* c, const AL& al_, int M, const bf16_t* Bm, int64_t ldb, int N, int K, const EP& ep_, const std::string& name, double abytes,
                int zdim = 1, double flops = -1.0) {
  if (M <= 0) return PPO_OK;
  AL al = al_; EP ep = ep_;
  al.prepare(); ep.map.prepare();
  const char* what = name.c_str();
  ProfScope ps(c, name, flops >= 0.0 ? flops : 2.0 * M * (double)N * K, abytes);
  dim3 blk(256);
  constexpr bool rows = std::is_same<AL, ARows>::value;
  if constexpr (rows) {
    if (!al.plain) return fail(c, PPO_ESHAPE, "%s: rows of images have no product of their own", what);
    if (gemm_small_covers(M, N, K)) {
      const dim3 grid(cdiv(M, 32), cdiv(N, 32));
      if (K <= 512) hipLaunchKernelGGL((k_gemm_small<4, EP>), grid, dim3(256), 0, c->stream, al.a.base, al.a.stride_b, M, Bm, ldb, N, K, ep);
      else hipLaunchKernelGGL((k_gemm_small<8, EP>), grid, dim3(512), 0, c->stream, al.a.base, al.a.stride_b, M, Bm, ldb, N, K, ep);
      LAUNCHCHK(c, what);
      return PPO_OK;
    }
    if (K >= 1024) {
      const GemmPlan plan = plan_gemm(M, N, K, c->partial_elems > 4 ? c->partial_elems - 4 : 0);
      int rc = PPO_OK;
      if (plan.bn == 32) rc = launch_gemm_ring<128, 32, 4, 1>(c, al, M, Bm, ldb, N, K, ep, plan);
      else if (plan.bm == 64) rc = launch_gemm_ring<64, 64, 2, 2>(c, al, M, Bm, ldb, N, K, ep, plan);
      else if (plan.bn == 64) rc = launch_gemm_ring<128, 64, 2, 2>(c, al, M, Bm, ldb, N, K, ep, plan);
      else if (plan.bm == 128) rc = launch_gemm_ring<128, 128, 2, 2>(c, al, M, Bm, ldb, N, K, ep, plan);
      else rc = launch_gemm_ring<256, 128, 4, 2>(c, al, M, Bm, ldb, N, K, ep, plan);
      if (rc) return rc;
      LAUNCHCHK(c, what);
      return PPO_OK;
    }
  }
  // Very deep reductions of gathered rows stream their operands through an LDS ring of up to eight stages, filled by
  // four loader waves while four or eight other waves compute (k_gemm_rs; plain rows took plan_gemm's forms above);
  // medium ones take 64-wide steps through registers, where the smaller LDS footprint lets more blocks share a CU and
  // hide the prologue and epilogue of their short loops.
#define LAUNCH_GEMM_RS(BM_, BN_, WM_, WN_)                                                                              \
  do {                                                                                                                   \
    constexpr int ncw = WM_ * WN_;                                                                                       \
    constexpr int nst = (BM_ + BN_) * 128 * 8 <= 128 * 1024 ? 8 : ((BM_ + BN_) * 128 * 4 <= 128 * 1024 ? 4 : 3);            \
    auto kfn = k_gemm_rs<BM_, BN_, WM_, WN_, nst, AL, EP>;                                                               \
    constexpr int lds = nst * (BM_ + BN_) * 128;                                                                         \
    static uint64_t attr_devs = 0;  /* bit d: set on device d */                                                                                        \
    if (!((attr_devs >> c->dev) & 1)) { HIPCHK(c, hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, lds)); attr_devs |= 1ull << c->dev; } \
    hipLaunchKernelGGL(kfn, grid, dim3((ncw + 4) * 64), lds, c->stream, al, Bm, ldb, N, ep, c->zpage);                    \
  } while (0)
#define LAUNCH_GEMM(BM_, BN_, WM_, WN_, GX, GY)                                                                        \
  do {                                                                                                                   \
    dim3 grid(GX, GY, zdim);                                                                                             \
    if constexpr (!rows) { if (K >= 1024) { LAUNCH_GEMM_RS(BM_, BN_, WM_, WN_); break; } }                                \
    if constexpr (WM_ * WN_ == 4) {                                                                                      \
      if (K >= 128) hipLaunchKernelGGL((k_gemm<BM_, BN_, WM_, WN_, 64, AL, EP>), grid, blk, 0, c->stream, al, Bm, ldb, N, ep); \
      else hipLaunchKernelGGL((k_gemm<BM_, BN_, WM_, WN_, 32, AL, EP>), grid, blk, 0, c->stream, al, Bm, ldb, N, ep);      \
    }                                                                                                                    \
  } while (0)
  if (N > 64) {
    if (K >= 1024 && (int64_t)cdiv(M, 256) * cdiv(N, 128) * zdim >= 256) LAUNCH_GEMM(256, 128, 4, 2, cdiv(M, 256), cdiv(N, 128));
    else if ((int64_t)cdiv(M, 128) * cdiv(N, 128) * zdim >= 256 || M <= 64) LAUNCH_GEMM(128, 128, 2, 2, cdiv(M, 128), cdiv(N, 128));
    else LAUNCH_GEMM(64, 64, 2, 2, cdiv(M, 64), cdiv(N, 64));
  } else if (N > 32) {
    if ((int64_t)cdiv(M, 128) * zdim >= 256 || M <= 64) LAUNCH_GEMM(128, 64, 2, 2, cdiv(M, 128), 1);
    else LAUNCH_GEMM(64, 64, 2, 2, cdiv(M, 64), 1);
  } else {
    LAUNCH_GEMM(128, 32, 4, 1, cdiv(M, 128), 1);
  }
#undef LAUNCH_GEMM
#undef LAUNCH_GEMM_RS
  LAUNCHCHK(c, what);
  return PPO_OK;
}

ImgAddr plain_rows(const bf16_t* base, int64_t ld) { ImgAddr a; a.base = base; a.idx = nullptr; a.stride_b = ld; a.stride_v = 0; a.V = 1; return a; }
ARows plain_arows(const bf16_t* base, int64_t ld, int M, int K) {
  ARows r; r.a = plain_rows(base, ld); r.HW = 1; r.C = 0; r.M = M; r.K = K; r.plain = true; return r;
}
MapRows plain_map(int64_t ld, int M) { MapRows m; m.stride_b = ld; m.stride_v = 0; m.V = 1; m.HW = 1; m.C = 0; m.M = M; return m; }

// All queued partial-sum reductions in one launch; the partial workspaces are free again afterwards.
int flush_reduces(Ctx* c) {
  ReduceJobs& J = c->rjobs;
  if (J.njobs > 0 || c->lossfin.on) {
    double bytes = 0.0;
    for (int j = 0; j < J.njobs; ++j) bytes += 4.0 * ((double)J.splits[j] + 1.0) * (double)J.n[j];
    ProfScope ps(c, "wgrad_reduce", 0.0, bytes);
    for (int j = J.njobs; j <= ReduceJobs::MAXJ; ++j) J.first[j] = c->rjob_blocks;
    hipLaunchKernelGGL(k_reduce_batch, dim3(c->rjob_blocks + (c->lossfin.on ? 1 : 0)), dim3(256), 0, c->stream, J, c->lossfin);
    LAUNCHCHK(c, "k_reduce_batch");
    c->lossfin.on = 0;
  }
  J.njobs = 0; c->rjob_blocks = 0;
  c->partial = c->partial_base; c->partial_elems = c->partial_cap;
  c->bias_partial = c->bias_partial_base; c->bias_partial_elems = c->bias_partial_cap;
  return PPO_OK;
}
// Make room for a kernel that would like `need` partial and `bneed` bias-partial elements.
int ensure_partial(Ctx* c, int64_t need, int64_t bneed) {
  if (need > c->partial_elems || bneed > c->bias_partial_elems || c->rjobs.njobs + 3 > ReduceJobs::MAXJ) return flush_reduces(c);
  return PPO_OK;
}
// Queue the reduction of `splits` partials of n elements that start at the cursor (kind as in ReduceJobs) and
// move the cursor behind them; with bias: the same for `splits` bias partials of nb elements (plain sums).
void defer_reduce(Ctx* c, int kind, int splits, int64_t n, int N, int K, float* dst, float* dst2, bool accumulate, bool with_bias, int64_t nb, float* bdst) {
  ReduceJobs& J = c->rjobs;
  auto add = [&](int kd, const float* part, int64_t nn, float* d, float* d2) {
    const int j = J.njobs++;
    J.first[j] = c->rjob_blocks; J.kind[j] = kd; J.splits[j] = splits; J.N[j] = N; J.K[j] = K; J.accumulate[j] = accumulate ? 1 : 0;
    J.n[j] = nn; J.partial[j] = part; J.dst[j] = d; J.dst2[j] = d2;
    J.vec[j] = (nn % 4 != 0 || (reinterpret_cast<uintptr_t>(part) & 15) != 0) ? 0 : splits <= 8 ? 2 : 1;
    c->rjob_blocks += cdiv(nn, J.vec[j] == 2 ? 1024 : J.vec[j] ? 128 : 32);
  };
  add(kind, c->partial, n, dst, dst2);
  c->partial += (int64_t)splits * n; c->partial_elems -= (int64_t)splits * n;
  if (with_bias) {
    add(0, c->bias_partial, nb, bdst, nullptr);
    c->bias_partial += (int64_t)splits * nb; c->bias_partial_elems -= (int64_t)splits * nb;
  }
}

// Wide plain weight gradient through the LDS-ring kernel (wgrad_rs.hip.h); returns 1 when the shape is not covered.
int launch_wgrad_rs(Ctx* c, const bf16_t* dy, int64_t ld_dy, const bf16_t* x, int64_t ld_x, int Nn, int Kk, int M, float* gw, float* gb, bool accumulate,
                    const std::string& name, double abytes) {
  typedef WgradRsShape S;
  if (Nn < 128 || Kk < 1024 || Nn % 8 || Kk % 8 || ld_dy % 8 || ld_x % 8 || M < 128) return 1;
  const int tiles = cdiv(Kk, S::TK) * cdiv(Nn, S::TN);
  // few splits (their fp32 partials cost traffic), but enough blocks to fill the chip's 256 CUs in whole rounds
  int splits = 1;
  double best = 0.0;
  for (int sp = 1; sp <= 8; ++sp) {
    if (cdiv(M, sp) < 512 && sp > 1) break;
    const int blocks = tiles * sp;
    const double eff = (double)blocks / (double)(cdiv(blocks, 256) * 256) - 0.06 * (sp - 1);
    if (eff > best + 1e-9) { best = eff; splits = sp; }
  }
  const int64_t per = (int64_t)Nn * Kk;
  if (splits > 1) { const int erc = ensure_partial(c, (int64_t)splits * per, gb ? (int64_t)splits * Nn : 0); if (erc) return erc; }
  if (splits > 1 && ((int64_t)splits * per > c->partial_elems || (gb && (int64_t)splits * Nn > c->bias_partial_elems))) splits = 1;
  int rows = cdiv(M, splits);
  rows = (rows + S::ROWS - 1) / S::ROWS * S::ROWS;
  splits = cdiv(M, rows);
  WgradRsArgs a;
  a.dy = dy; a.ld_dy = ld_dy; a.x = x; a.ld_x = ld_x; a.M = M; a.Nn = Nn; a.Kk = Kk; a.rows_per_split = rows; a.zpage = c->zpage;
  a.direct = splits == 1 ? 1 : 0; a.accumulate = accumulate ? 1 : 0;
  a.out = a.direct ? gw : c->partial; a.bias_out = gb ? (a.direct ? gb : c->bias_partial) : nullptr;
  {
    ProfScope ps(c, name, 2.0 * M * (double)Nn * Kk, abytes);
    static uint64_t attr_devs = 0;  /* bit d: set on device d */
    if (!((attr_devs >> c->dev) & 1)) { HIPCHK(c, hipFuncSetAttribute((const void*)k_wgrad_rs, hipFuncAttributeMaxDynamicSharedMemorySize, S::LDS_BYTES)); attr_devs |= 1ull << c->dev; }
    hipLaunchKernelGGL(k_wgrad_rs, dim3(cdiv(Kk, S::TK), cdiv(Nn, S::TN), splits), dim3(S::THREADS), S::LDS_BYTES, c->stream, a);
    LAUNCHCHK(c, "k_wgrad_rs");
  }
  if (splits > 1) defer_reduce(c, 0, splits, per, 0, 0, gw, nullptr, accumulate, gb != nullptr, Nn, gb);
  return PPO_OK;
}

// A hidden layer's input gradient that may be taken beside its weight gradient (k_fc_backward).
struct DgradBeside {
  const bf16_t* wT;  // [Kk][Nn]
  Ep<MapRows, bf16_t, false, false, true> ep;
  double abytes;
  bool taken;        // set by launch_wgrad
};
// How k_wgrad's work on Nn x Kk outputs is cut: blocks of 64 x 128*ktw outputs, and slices of the rows.  Wide outputs (the first
// hidden layer) have enough tiles with narrow blocks and few slices: the fp32 partials, not the operands, are then the larger part
// of the traffic.  Slices of 128 rows or more, of 64 or more where those would make fewer than 64 blocks: shorter chains (256 rows
// of 64 x 1056 7.1 -> 5.3 us, 1250 of 128 x 256 8.3 -> 7.4; 4096 rows, 64 blocks: 0).
struct WgradCut {
  int ktw, tiles, most;
  WgradCut(int Nn, int Kk) {
    ktw = Kk <= 128 ? 1 : (Kk <= 256 ? 2 : (Kk >= 1024 ? 1 : 3));
    tiles = cdiv(Kk, 128 * ktw) * cdiv(Nn, 64);
    most = cdiv(Kk >= 1024 ? 512 : 768, tiles);
  }
  int splits(int64_t M) const { return std::min(most, (int64_t)tiles * cdiv(M, 128) < 64 ? cdiv(M, 64) : cdiv(M, 128)); }
  // the most slices of up to M rows: those of M, or of the most rows that are cut by 64
  int splits_up_to(int64_t M) const { return tiles > 63 ? splits(M) : std::max(splits(M), splits(std::min<int64_t>(M, 63 / tiles * 128))); }
};
// G[Nn][Kk] (+)= Dy^T * A over M rows, plus optional bias gradient gb[Nn].
template <class DL, class AL>
int launch_wgrad(Ctx* c, const DL& dl_, const AL& al_, int Nn, int Kk, int M, float* gw, float* gb, bool accumulate, const std::string& name, double abytes,
                 DgradBeside* beside = nullptr) {
  if (M <= 0) return PPO_OK;
  // the queued sums of one launch run side by side: one that this gradient is added to is taken first
  for (int j = 0; accumulate && j < c->rjobs.njobs; ++j)
    if (c->rjobs.dst[j] == gw) { const int erc = flush_reduces(c); if (erc) return erc; }
  if constexpr (std::is_same<DL, ARows>::value && std::is_same<AL, ARows>::value) {
    if (dl_.plain && al_.plain) {
      const int rc = launch_wgrad_rs(c, dl_.a.base, dl_.a.stride_b, al_.a.base, al_.a.stride_b, Nn, Kk, M, gw, gb, accumulate, name, abytes);
      if (rc != 1) return rc;
    }
  }
  DL dl = dl_; AL al = al_;
  dl.prepare(); al.prepare();
  const char* what = name.c_str();
  const WgradCut cut(Nn, Kk);
  const int ktw = cut.ktw;
  int splits = cut.splits(M);
  const int64_t per = (int64_t)Nn * Kk;
  { const int erc = ensure_partial(c, (int64_t)splits * per, (int64_t)splits * Nn); if (erc) return erc; }
  if ((int64_t)splits * per > c->partial_elems) splits = (int)(c->partial_elems / per);
  if ((int64_t)splits * Nn > c->bias_partial_elems) splits = (int)(c->bias_partial_elems / Nn);
  if (splits < 1) return fail(c, PPO_ENOMEM, "weight-gradient workspace too small for %s", what);
  int rows = cdiv(M, splits);
  rows = (rows + 31) / 32 * 32;
  splits = cdiv(M, rows);
  dim3 grid(cdiv(Kk, 128 * ktw), cdiv(Nn, 64), splits);
  float* bp = gb ? c->bias_partial : nullptr;
  if constexpr (std::is_same<DL, ARows>::value && std::is_same<AL, ARows>::value) {
    // One launch with the input gradient where that is k_gemm_small's on four waves and the blocks of both (two to a CU by their
    // LDS) are resident at once: each then hides behind the other.  Beyond that line nothing is hidden: the blocks queue.
    const int nw = (int)(grid.x * grid.y * grid.z), gm = cdiv(M, 32), ng = gm * cdiv(Kk, 32);
    if (beside && dl.plain && al.plain && Nn <= 512 && gemm_small_covers(M, Kk, Nn) && nw + ng <= 512) {
      ProfScope ps(c, name + "+dgrad", 4.0 * M * (double)Nn * Kk, abytes + beside->abytes);
      beside->ep.map.prepare();
      FcBackward a;
      a.dl = dl; a.al = al; a.Nn = Nn; a.Kk = Kk; a.M = M; a.rows = rows; a.nw = nw; a.gx = make_fastdiv(grid.x); a.gy = make_fastdiv(grid.y); a.gm = make_fastdiv(gm);
      a.partial = c->partial; a.bias_partial = bp; a.wT = beside->wT;
      using EP = Ep<MapRows, bf16_t, false, false, true>;
      if (ktw == 1) hipLaunchKernelGGL((k_fc_backward<1, EP>), dim3(nw + ng), dim3(256), 0, c->stream, a, beside->ep);
      else if (ktw == 2) hipLaunchKernelGGL((k_fc_backward<2, EP>), dim3(nw + ng), dim3(256), 0, c->stream, a, beside->ep);
      else hipLaunchKernelGGL((k_fc_backward<3, EP>), dim3(nw + ng), dim3(256), 0, c->stream, a, beside->ep);
      LAUNCHCHK(c, what);
      beside->taken = true;
    }
  }
  if (!beside || !beside->taken) {
    ProfScope ps(c, name, 2.0 * M * (double)Nn * Kk, abytes);
    if (ktw == 1) hipLaunchKernelGGL((k_wgrad<1, DL, AL>), grid, dim3(256), 0, c->stream, dl, al, Nn, Kk, M, rows, c->partial, bp);
    else if (ktw == 2) hipLaunchKernelGGL((k_wgrad<2, DL, AL>), grid, dim3(256), 0, c->stream, dl, al, Nn, Kk, M, rows, c->partial, bp);
    else hipLaunchKernelGGL((k_wgrad<3, DL, AL>), grid, dim3(256), 0, c->stream, dl, al, Nn, Kk, M, rows, c->partial, bp);
    LAUNCHCHK(c, what);
  }
  defer_reduce(c, 0, splits, per, 0, 0, gw, nullptr, accumulate, gb != nullptr, Nn, gb);
  return PPO_OK;
}

// Re-packs of the weights into the layouts the backward kernels read, collected into one launch (validate_desc bounds their number).
struct RepackList {
  RepackJobs jobs;
  int nblocks = 0;
  RepackList() { jobs.njobs = 0; }
  void add(int kind, const bf16_t* src, bf16_t* dst, int a, int b, int ld, int64_t elems) {
    const int j = jobs.njobs++;
    jobs.first[j] = nblocks; jobs.kind[j] = kind; jobs.src[j] = src; jobs.dst[j] = dst; jobs.a[j] = a; jobs.b[j] = b; jobs.ld[j] = ld;
    nblocks += kind == 0 ? cdiv(ld, 64) * cdiv(b, 64) : cdiv(elems, 256);
  }
  // parity-class-packed transposed-conv weights of layer l, read by the implicit-GEMM paths
  void add_packed_dgrad(Ctx* c, int l) {
    const int Co = c->cC[l + 1], Ci = c->cC[l];
    for (int py = 0; py < 2; ++py) add(2, c->shadow + c->convW[l], c->wd[l][py], Co, Ci, py, (int64_t)2 * Ci * (1 + py) * 2 * Co);
    c->wd_ver[l] = c->wver;
  }
  int launch(Ctx* c, const GnormFinalize& gn) {
    for (int j = jobs.njobs; j <= RepackJobs::MAXJ; ++j) jobs.first[j] = nblocks;
    hipLaunchKernelGGL(k_repack_all, dim3(nblocks + (gn.on ? 1 : 0)), dim3(256), 0, c->stream, jobs, gn);
    LAUNCHCHK(c, "weight repack");
    return PPO_OK;
  }
};
// The packed weights of layer l, built now if its current ones are not (the LDS-image kernels use the per-tap
// transposes instead, so a layer is packed only once an implicit-GEMM path has asked for it).
int ensure_packed_dgrad_weights(Ctx* c, int l) {
  if (c->wd_ver[l] == c->wver) return PPO_OK;
  c->wd_used[l] = true;
  RepackList r;
  r.add_packed_dgrad(c, l);
  GnormFinalize none;
  none.on = 0;
  return r.launch(c, none);
}

int repack_weights(Ctx* c) {
  c->wver += 1;
  ProfScope ps(c, "weight_repack", 0.0, 4.0 * (double)c->total);
  RepackList r;
  for (int l = 1; l < c->nconv; ++l) {
    r.add(1, c->shadow + c->convW[l], c->wtap[l], c->cC[l + 1], c->cC[l], 0, (int64_t)9 * c->cC[l] * c->cC[l + 1]);
    if (c->wd_used[l]) r.add_packed_dgrad(c, l);
  }
  for (int l = 0; l < c->nfc; ++l)
    r.add(0, c->shadow + c->fcW[l], c->fcT[l], c->fout[l], c->fin[l], c->fout[l], (int64_t)c->fin[l] * c->fout[l]);
  r.add(0, c->shadow + c->headW, c->headT, c->NH, c->hid, HEAD_LD, (int64_t)c->hid * HEAD_LD);
  if (c->XH > 0) {
    r.add(0, c->shadow + c->aux1W, c->aux1T, c->XH, c->hid, c->XH, (int64_t)c->hid * c->XH);
    r.add(0, c->shadow + c->aux2W, c->aux2T, c->X, c->XH, HEAD_LD, (int64_t)c->XH * HEAD_LD);
  }
  if (c->E > 0) r.add(0, c->shadow + c->embW, c->embT, c->E, c->flat, c->E, (int64_t)c->flat * c->E);
  for (int l = 0; l < c->nl; ++l)
    r.add(0, c->shadow + c->lstmW[l], c->lstmWT[l], 4 * c->H, c->lin[l] + c->H, 4 * c->H, (int64_t)(c->lin[l] + c->H) * 4 * c->H);
  const int rc = r.launch(c, c->gnfin);
  c->gnfin.on = 0;
  return rc;
}

int refresh_shadow(Ctx* c) {
  hipLaunchKernelGGL(k_cast_bf16, dim3(cdiv(c->total, 256)), dim3(256), 0, c->stream, c->p, c->shadow, c->total);
  LAUNCHCHK(c, "k_cast_bf16");
  return repack_weights(c);
}

ImgAddr conv_out_addr(Ctx* c, int l, const bf16_t* contiguous, const bf16_t* strided) {
  // output of conv layer l (0-based) for a chunk: the last layer lives inside the feature matrix
  ImgAddr a; a.idx = nullptr; a.V = c->V;
  if (l == c->nconv - 1) { a.base = strided; a.stride_b = c->feat_ld; a.stride_v = c->flat; }
  else { int64_t e = (int64_t)c->cC[l + 1] * c->cH[l + 1] * c->cW[l + 1]; a.base = contiguous; a.stride_b = e * c->V; a.stride_v = e; }
  return a;
}

// Tiles of output columns for result rows that the row-wise LDS-image kernels do not cover: the numbers of tiles side by
// side (parts) and one above the other (bands) that load the fewest pixels with their halos, among those of at most `maxpix`
// pixels whose `fits(columns, rows)` holds.  Parts of fewer than 8 columns are not tried (their halo is a quarter of what
// they load); false: none fits.
struct ColsPlan { int TC, NP, TR, NB; };
template <class FITS>
bool plan_cols(int Ho, int Wo, int maxpix, FITS fits, ColsPlan* out, int multiple = 1) {
  int64_t best = -1;
  for (int np = 1; np <= cdiv(Wo, 8); ++np) {
    const int tc = cdiv(cdiv(Wo, np), multiple) * multiple;
    if (tc > maxpix || (np > 1 && cdiv(Wo, tc) != np)) continue;
    int tr = std::min(maxpix / tc, Ho);
    while (tr > 0 && !fits(tc, tr)) --tr;
    if (tr == 0) continue;
    const int nb = cdiv(Ho, tr);
    tr = cdiv(Ho, nb);
    const int64_t loads = (int64_t)np * nb * (2 * tr + 1) * (2 * tc + 1);
    if (best < 0 || loads < best) { best = loads; *out = ColsPlan{tc, np, tr, nb}; }
  }
  return best >= 0;
}

// Bands of whole rows cut from each image (nb a piece), or from the stack of all images (common.hip.h)?  What a tile costs hardly
// depends on how full it is, so the stack is taken where the `blocks` of the grid then have at most `pct` per cent of the tiles to
// do one after another: heights that are no multiple of the rows a tile can hold, and images of less than a tile.  Its bands are
// then made no higher than that number of tiles asks for.  `fits(rows)`: a band fits.  Measured, layers of 64 channels, cut from
// each image -> stacked: 1250 images with 7x10 results (bands of 4 and 3 rows, of 6) forward 22.9 -> 18.7 us, input gradient 30.2
// -> 23.9, weight gradient 28.5 -> 24.0; 16384 images with 8x10 results of 128 channels forward 265 -> 209, weight gradient 414 ->
// 344; 4096 images with 15x20 results (5 rows, 6) from 32 channels: weight gradient 89 -> 85, input gradient 117 -> 108, but
// forward, whose loads fill the memory's rate already, 89 -> 94.  The input gradient from 128 channels stays with its images: its
// finishing waves, its longest role, do the same work either way (4800 images with 4x7 results 29 -> 33).
template <class FITS>
bool plan_stack(int nimg, int Ho, int Wo, int maxpix, int nb, int blocks, int pct, FITS fits, int* rows) {
  const int64_t total = (int64_t)nimg * Ho;
  if (Wo > maxpix || 2 * total * Wo >= ((int64_t)1 << 31)) return false;  // (stacked rows and pixels are 32-bit numbers)
  int tr = (int)std::min<int64_t>(maxpix / Wo, total);
  while (tr > 0 && !fits(tr)) --tr;
  if (tr < 1) return false;
  const int64_t each = cdiv(cdiv(total, tr), blocks), now = cdiv((int64_t)nimg * nb, blocks);
  if (100 * each > pct * now) return false;
  *rows = cdiv(total, each * blocks);
  return true;
}
bool dense_images(int64_t stride_b, int64_t stride_v, int V, int64_t elems) { return stride_b == V * elems && (V == 1 || stride_v == elems); }

// Bands of whole result rows for the forward kernel: *TR rows each, balanced, *NB of them; false where they do not fit (tiles
// of columns then).
template <int CIN, int WIDE>
bool plan_fwd_rows(int W, int Ho, int Wo, int* TR, int* NB) {
  typedef ConvTileShape<CIN, WIDE> S;
  if (Wo > S::BM) return false;
  *NB = cdiv(Ho, std::min(S::BM / Wo, Ho)); *TR = cdiv(Ho, *NB);
  const int segs = cdiv(W * S::PIX, 1024), ni = cdiv(2 * *TR + 1, 4) * segs;  // loads per loader wave per band
  return segs <= S::MAXSEG && ni <= 63 && S::lds_bytes(W + 2, *TR, 3) <= 160 * 1024;
}
// Forward convolution through the LDS-image kernel; returns 1 when the layer's shape is not one
// it covers (the caller then takes the implicit-GEMM path).
template <int CIN, int WIDE, bool RELU>
int launch_conv_fwd_tile_t(Ctx* c, ConvTileArgs a, const std::string& name, double flops, double abytes) {
  typedef ConvTileShape<CIN, WIDE> S;
  const int nimg = a.ntiles;  // passed in as the image count
  int slots = a.W + 2, form, ni;
  if (plan_fwd_rows<CIN, WIDE>(a.W, a.Ho, a.Wo, &a.TR, &a.NB)) {
    a.TC = a.Wo; a.NP = 1;
    ni = cdiv(2 * a.TR + 1, 4) * cdiv(a.W * S::PIX, 1024);
    // bands of four or more output rows share at most an eighth of their input rows with a neighbour: read once, non-temporal
    form = a.TR >= 4;
    int tr;
    if (CIN == 16 && form != 1) return 1;
    auto fits = [&](int r) { return S::lds_bytes(slots, r, 3) + S::ZERO_BYTES <= 160 * 1024 && cdiv(2 * r + 1, 4) * cdiv(a.W * S::PIX, 1024) <= 63; };
    if (CIN != 16 && dense_images(a.in.stride_b, a.in.stride_v, a.V, (int64_t)a.H * a.W * CIN) && plan_stack(nimg, a.Ho, a.Wo, S::BM, a.NB, 256 / cdiv(a.Cout, S::BN), CIN == 32 ? 80 : 95, fits, &tr)) {
      a.stk = make_stack(nimg, a.Ho, a.Wo, a.H, a.V);
      a.stk.dense = dense_images(a.out_stride_b, a.out_stride_v, a.V, (int64_t)a.Ho * a.Wo * a.Cout);
      a.TR = tr; ni = cdiv(2 * tr + 1, 4) * cdiv(a.W * S::PIX, 1024); form = 3;
    }
  } else {
    ColsPlan p;
    auto fits = [&](int tc, int tr) { return S::image_bytes(2 * tc + 1, tr) <= S::MAXLD * 4096 && S::lds_bytes(2 * tc + 1, tr, 3) <= 160 * 1024; };
    if (CIN == 16 || !plan_cols(a.Ho, a.Wo, S::BM, fits, &p)) return 1;
    a.TC = p.TC; a.NP = p.NP; a.TR = p.TR; a.NB = p.NB;
    slots = 2 * a.TC + 1; ni = cdiv(cdiv(S::image_bytes(slots, a.TR), 1024), 4); form = 2;
  }
  a.ntiles = form == 3 ? cdiv(a.stk.rows, a.TR) : nimg * a.NB * a.NP; a.dv_nb = make_fastdiv(a.NB); a.dv_np = make_fastdiv(a.NP);
  // as many ring images as fit: a loader wave has (nbuf - 2) * ni loads outstanding behind the band it waits for
  a.nbuf = S::MAXBUF;
  const int extra = form == 3 ? S::ZERO_BYTES : 0;
  while (a.nbuf > 3 && (S::lds_bytes(slots, a.TR, a.nbuf) + extra > 160 * 1024 || (a.nbuf - 2) * ni > 63)) --a.nbuf;
  const int lds = S::lds_bytes(slots, a.TR, a.nbuf) + extra;
  const int gy = cdiv(a.Cout, S::BN);
  int gx = 256 / gy; if (gx > a.ntiles) gx = a.ntiles; if (gx < 1) gx = 1;
  auto kfn = k_conv_fwd_tile<CIN, LOAD_NT, WIDE, RELU>;  // (16 channels: bands of four or more rows only)
  if constexpr (CIN != 16) kfn = form == 3 ? k_conv_fwd_tile<CIN, LOAD_NT, WIDE, RELU, false, 0, false, true> : form == 2 ? k_conv_fwd_tile<CIN, 0, WIDE, RELU, true> : form == 1 ? k_conv_fwd_tile<CIN, LOAD_NT, WIDE, RELU> : k_conv_fwd_tile<CIN, 0, WIDE, RELU>;
  static uint64_t attr_devs[4] = {0, 0, 0, 0};  // bit d: set on device d
  if (!((attr_devs[form] >> c->dev) & 1)) { HIPCHK(c, hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024)); attr_devs[form] |= 1ull << c->dev; }
  ProfScope ps(c, name, flops, abytes);
  hipLaunchKernelGGL(kfn, dim3(gx, gy), dim3(S::THREADS), lds, c->stream, a);
  LAUNCHCHK(c, "k_conv_fwd_tile");
  return PPO_OK;
}
int launch_conv_fwd_tile(Ctx* c, const AConvFwd& al, const ImgAddr& o, int Cout, const bf16_t* w, const float* bias, int nimg,
                         const std::string& name, double abytes, uint32_t* bits, bool relu = true) {
  if ((al.Cin != 16 && al.Cin != 32 && al.Cin != 64) || (al.Cin == 16 && Cout > 32) || Cout % 8 || nimg < 1 || al.in.idx) return 1;
  ConvTileArgs a;
  a.in = al.in; a.in.prepare();
  a.out = const_cast<bf16_t*>(o.base); a.out_stride_b = o.stride_b; a.out_stride_v = o.stride_v;
  a.w = w; a.bias = bias; a.zpage = c->zpage; a.bits = bits; a.V = o.V; a.H = al.H; a.W = al.W; a.Ho = al.Ho; a.Wo = al.Wo; a.Cout = Cout;
  a.TR = a.NB = a.TC = a.NP = 0; a.nbuf = 3;
  a.ntiles = nimg;  // image count; the template turns it into tiles
  const double flops = 2.0 * (double)al.M * Cout * al.K;
  // more than 64 output channels: the 64 x 128 form reads the input once
#define LAUNCH_FWD(R_)                                                                       \
  (al.Cin == 16 ? launch_conv_fwd_tile_t<16, 0, R_>(c, a, name, flops, abytes)                \
   : al.Cin == 32 ? launch_conv_fwd_tile_t<32, 0, R_>(c, a, name, flops, abytes)              \
   : Cout > 64  ? launch_conv_fwd_tile_t<64, 1, R_>(c, a, name, flops, abytes)                \
                : launch_conv_fwd_tile_t<64, 0, R_>(c, a, name, flops, abytes))
  return relu ? LAUNCH_FWD(true) : LAUNCH_FWD(false);
#undef LAUNCH_FWD
}

// Tiles of the second layer's kernels that make its input from the images (conv0_rows.hip.h): whole result rows where the
// tile's input fits the producer waves, else columns (an even number: a tile's image rows then start at a multiple of 16
// bytes).  Whole rows also where columns would save less than a tenth of the pixels to make: their tiles test for missing
// pixels only in the first and last band.  `lds(TC, TR)`: bytes of a tile's LDS with the shortest rings.
template <int C0, class LDS>
bool plan_conv01(int W1, int Ho, int Wo, int maxpix, LDS lds, ColsPlan* out, bool* cols) {
  typedef Conv0Shape1<C0> S0;
  auto fits = [&](int tc, int tr, int ncol) { return (2 * tr + 1) * ncol <= S0::MAXPIX && S0::fits(tc, tr) && lds(tc, tr) <= 160 * 1024; };
  ColsPlan pc;
  bool havec = plan_cols(Ho, Wo, maxpix, [&](int tc, int tr) { return fits(tc, tr, 2 * tc + 1); }, &pc, 2);
  int tr = Wo <= maxpix ? std::min(maxpix / Wo, Ho) : 0;
  while (tr > 0 && !fits(Wo, tr, W1)) --tr;
  if (tr > 0) {
    const int nb = cdiv(Ho, tr);
    tr = cdiv(Ho, nb);
    const double made = (double)nb * (2 * tr + 1) * W1;
    if (!havec || made <= 1.1 * pc.NB * pc.NP * (2.0 * pc.TR + 1) * (2 * pc.TC + 1)) { *out = ColsPlan{Wo, 1, tr, nb}; *cols = false; return true; }
  }
  *out = pc; *cols = true;
  return havec;
}
// The two first convolutions' forward in one kernel; returns 1 when the shapes are not covered.  bits0, bits1: the layers' mask
// bits (both or neither).
template <int C0, bool BITS>
int launch_conv01_fwd_t(Ctx* c, ConvTileArgs a, const std::string& name, double flops, double abytes) {
  typedef ConvTileShape<32> S;
  typedef Conv0Shape1<C0> S0;
  const int nimg = a.ntiles;  // passed in as the image count
  auto lds_of = [&](int tc, int tr, int ni) { return 2 * S0::act_bytes(tc, tr) + S::STAGE_BYTES + S::BN * 4 + ni * S0::image_bytes(tc, tr); };
  ColsPlan p;
  bool cols;
  if (!plan_conv01<C0>(a.W, a.Ho, a.Wo, S::BM, [&](int tc, int tr) { return lds_of(tc, tr, 3); }, &p, &cols)) return 1;
  if (c->dry) return PPO_OK;
  a.TC = p.TC; a.NP = p.NP; a.TR = p.TR; a.NB = p.NB; a.ntiles = nimg * p.NB * p.NP; a.dv_nb = make_fastdiv(p.NB); a.dv_np = make_fastdiv(p.NP); a.nbuf = 2;
  a.src0.nimage = lds_of(p.TC, p.TR, S0::AHEAD + 1) <= 160 * 1024 ? S0::AHEAD + 1 : 3;
  const int gx = std::min(256, a.ntiles);
  auto kfn = cols ? k_conv_fwd_tile<32, 0, 0, true, true, C0, BITS> : k_conv_fwd_tile<32, 0, 0, true, false, C0, BITS>;
  static uint64_t attr_devs[2] = {0, 0};  // bit d: set on device d
  if (!((attr_devs[cols] >> c->dev) & 1)) { HIPCHK(c, hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024)); attr_devs[cols] |= 1ull << c->dev; }
  ProfScope ps(c, name, flops, abytes);
  hipLaunchKernelGGL(kfn, dim3(gx), dim3(S::THREADS), lds_of(p.TC, p.TR, a.src0.nimage), c->stream, a);
  LAUNCHCHK(c, "k_conv_fwd_tile");
  return PPO_OK;
}
Conv0Src conv0_src(Ctx* c, const ImgAddr& in, uint32_t* bits) {
  Conv0Src s;
  s.img = in; s.img.prepare(); s.w = c->shadow + c->convW[0]; s.bias = c->p + c->convB[0]; s.bits = bits;
  s.H = c->cH[0]; s.rowbytes = c->cW[0] * c->cC[0] * 2; s.bpitch = c->b0pitch; s.nimage = 0;
  return s;
}
int launch_conv01_fwd(Ctx* c, const ImgAddr& in, const ImgAddr& o, const bf16_t* proprio, int n, bool train) {
  const int C0 = c->cC[0], Co = c->cC[2];
  if (c->nconv < 2 || (C0 != 1 && C0 != 3) || c->cC[1] != 32 || Co % 8 || Co > 64 || c->P % 8 || c->feat_ld % 8 || c->flat % 8) return 1;
  ConvTileArgs a = {};
  const int nimg = n * c->V;
  const bool bits1 = train && c->nconv > 2;  // the last layer's mask is applied by the first linear layer's input gradient
  a.out = const_cast<bf16_t*>(o.base); a.out_stride_b = o.stride_b; a.out_stride_v = o.stride_v;
  a.w = c->shadow + c->convW[1]; a.bias = c->p + c->convB[1]; a.zpage = c->zpage; a.bits = bits1 ? c->abits[1] : nullptr; a.V = c->V;
  a.H = c->cH[1]; a.W = c->cW[1]; a.Ho = c->cH[2]; a.Wo = c->cW[2]; a.Cout = Co; a.ntiles = nimg;
  a.src0 = conv0_src(c, in, train ? c->abits[0] : nullptr);
  a.n0 = n; a.P = c->P; a.proprio = proprio; a.feat = c->feat + c->V * c->flat; a.feat_ld = c->feat_ld;
  const double m0 = (double)nimg * a.H * a.W, m1 = (double)nimg * a.Ho * a.Wo;
  const double flops = 2.0 * (m0 * 32 * 9 * C0 + m1 * Co * 288), bytes = 2.0 * ((double)nimg * c->img_elems + m1 * Co + 288.0 * Co) + (train ? m0 * 4 : 0.0) + (bits1 ? m1 * Co / 8 : 0.0);
  if (train) return C0 == 1 ? launch_conv01_fwd_t<1, true>(c, a, "conv_fwd.0+1", flops, bytes) : launch_conv01_fwd_t<3, true>(c, a, "conv_fwd.0+1", flops, bytes);
  return C0 == 1 ? launch_conv01_fwd_t<1, false>(c, a, "conv_fwd.0+1", flops, bytes) : launch_conv01_fwd_t<3, false>(c, a, "conv_fwd.0+1", flops, bytes);
}
// The second convolution's weight gradient with its input made again from the images; returns 1 when the shapes are not covered.
template <int C0>
int launch_conv01_wgrad_t(Ctx* c, ConvWgradArgs a, float* gw, float* gb, bool accumulate, const std::string& name, double flops, double abytes) {
  typedef ConvWgradShape<32> S;
  typedef Conv0Shape1<C0> S0;
  const int nimg = a.ntiles;  // passed in as the image count
  auto lds_of = [&](int tc, int tr, int nb) { return 2 * S0::act_bytes(tc, tr) + nb * (cdiv(tc * tr, 16) * 16 * 128 + S0::image_bytes(tc, tr)); };
  ColsPlan p;
  bool cols;
  if (!plan_conv01<C0>(a.W, a.Ho, a.Wo, 16 * S::MAXSTEP, [&](int tc, int tr) { return lds_of(tc, tr, 3); }, &p, &cols)) return 1;
  if (c->dry) return PPO_OK;
  a.TC = p.TC; a.NP = p.NP; a.TR = p.TR; a.NB = p.NB; a.ntiles = nimg * p.NB * p.NP; a.dv_nb = make_fastdiv(p.NB); a.dv_np = make_fastdiv(p.NP); a.nstep = cdiv(p.TR * p.TC, 16);
  a.nbuf = a.src0.nimage = lds_of(p.TC, p.TR, 4) <= 160 * 1024 ? 4 : 3;
  const int K = 288;
  int gx = std::min(256, a.ntiles);
  const int64_t per = (int64_t)a.Cout * K;
  { const int erc = ensure_partial(c, (int64_t)gx * per, (int64_t)gx * a.Cout); if (erc) return erc; }
  gx = (int)std::min<int64_t>(gx, std::min(c->partial_elems / per, c->bias_partial_elems / a.Cout));
  if (gx < 1) return fail(c, PPO_ENOMEM, "weight-gradient workspace too small for the second convolution");
  a.partial = c->partial; a.bias_partial = c->bias_partial;
  constexpr int NS1 = S::MAXSTEP, NS2 = S::MAXSTEP - 1;
  const int form = (a.nstep == NS1 ? 1 : (a.nstep == NS2 ? 2 : 0)) + (cols ? 3 : 0);
  static decltype(&k_conv_wgrad_tile<32, 0>) const forms[6] = {
      k_conv_wgrad_tile<32, 0, false, C0>, k_conv_wgrad_tile<32, NS1, false, C0>, k_conv_wgrad_tile<32, NS2, false, C0>,
      k_conv_wgrad_tile<32, 0, true, C0>, k_conv_wgrad_tile<32, NS1, true, C0>, k_conv_wgrad_tile<32, NS2, true, C0>};
  static uint64_t attr_devs[6] = {};  /* bit d: set on device d */
  if (!((attr_devs[form] >> c->dev) & 1)) { HIPCHK(c, hipFuncSetAttribute((const void*)forms[form], hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024)); attr_devs[form] |= 1ull << c->dev; }
  {
    ProfScope ps(c, name, flops, abytes);
    hipLaunchKernelGGL(forms[form], dim3(gx), dim3(S::THREADS), lds_of(p.TC, p.TR, a.nbuf), c->stream, a);
    LAUNCHCHK(c, "k_conv_wgrad_tile");
  }
  defer_reduce(c, 1, gx, per, a.Cout, K, gw, nullptr, accumulate, true, a.Cout, gb);
  return PPO_OK;
}
int launch_conv01_wgrad(Ctx* c, const ImgAddr& in, const ImgAddr& dy, int nimg, bool accumulate) {
  if (c->cC[2] > 64) return 1;
  ConvWgradArgs a = {};
  a.dy = dy; a.dy.prepare(); a.zpage = c->zpage; a.src0 = conv0_src(c, in, nullptr);
  a.H = c->cH[1]; a.W = c->cW[1]; a.Ho = c->cH[2]; a.Wo = c->cW[2]; a.Cout = c->cC[2]; a.ntiles = nimg;
  const double m0 = (double)nimg * a.H * a.W, m1 = (double)nimg * a.Ho * a.Wo;
  const double flops = 2.0 * (m1 * a.Cout * 288 + m0 * 32 * 9 * c->cC[0]), bytes = 2.0 * (m1 * a.Cout + (double)nimg * c->img_elems) + 4.0 * 288 * a.Cout;
  float *gw = c->g + c->convW[1], *gb = c->g + c->convB[1];
  return c->cC[0] == 1 ? launch_conv01_wgrad_t<1>(c, a, gw, gb, accumulate, "conv_wgrad.1", flops, bytes) : launch_conv01_wgrad_t<3>(c, a, gw, gb, accumulate, "conv_wgrad.1", flops, bytes);
}

// Weight (and bias) gradient of conv layer with 32 or 64 input channels through the LDS-image
// kernel; returns 1 when the shape is not covered (the caller then takes the implicit-GEMM path).
template <int CIN>
int launch_conv_wgrad_tile_t(Ctx* c, ConvWgradArgs a, float* gw, float* gb, bool accumulate, const std::string& name, double flops, double abytes) {
  typedef ConvWgradShape<CIN> S;
  // largest band that fits the pixel-step table and three ring buffers, then balanced over the image
  const int nimg = a.ntiles;  // passed in as the image count
  const int segs = cdiv(a.W * S::PIX, 1024);
  int TR = 0, slots = a.W + 2, ni = 0;
  for (int tr = a.Ho; tr >= 1; --tr)
    if (tr * a.Wo <= 16 * S::MAXSTEP && S::lds_bytes(slots, tr, cdiv(tr * a.Wo, 16), 3) <= 158 * 1024) { TR = tr; break; }
  bool stack = false;
  if (TR > 0) {
    a.NB = cdiv(a.Ho, TR); a.TR = cdiv(a.Ho, a.NB); a.nstep = cdiv(a.TR * a.Wo, 16); a.TC = a.Wo; a.NP = 1;
    auto loads = [&](int tr) { return cdiv(2 * tr + 1, 4) * segs + cdiv(cdiv(tr * a.Wo, 16) * 2, 4); };  // per loader wave and band
    ni = loads(a.TR);
    int tr;
    auto fits = [&](int r) { return S::lds_bytes(slots, r, cdiv(r * a.Wo, 16), 3) <= 158 * 1024 && loads(r) <= 63; };
    if (segs <= S::MAXSEG && dense_images(a.in.stride_b, a.in.stride_v, a.in.V, (int64_t)a.H * a.W * CIN) && plan_stack(nimg, a.Ho, a.Wo, 16 * S::MAXSTEP, a.NB, 256 / cdiv(a.Cout, 64), 95, fits, &tr)) {
      a.stk = make_stack(nimg, a.Ho, a.Wo, a.H, a.in.V);
      a.stk.dense = dense_images(a.dy.stride_b, a.dy.stride_v, a.in.V, (int64_t)a.Ho * a.Wo * a.Cout);
      a.TR = tr; a.nstep = cdiv(tr * a.Wo, 16); ni = loads(tr); stack = true;
    }
  }
  const bool cols = TR == 0 || segs > S::MAXSEG || ni > 63;
  if (cols) {
    ColsPlan p;
    auto fits = [&](int tc, int tr) { return S::image_bytes(2 * tc + 1, tr) <= S::MAXLD * 4096 && S::lds_bytes(2 * tc + 1, tr, cdiv(tc * tr, 16), 3) <= 158 * 1024; };
    if (!plan_cols(a.Ho, a.Wo, 16 * S::MAXSTEP, fits, &p)) return 1;
    a.TC = p.TC; a.NP = p.NP; a.TR = p.TR; a.NB = p.NB; a.nstep = cdiv(a.TR * a.TC, 16);
    slots = 2 * a.TC + 1; ni = cdiv(cdiv(S::image_bytes(slots, a.TR), 1024), 4) + cdiv(a.nstep * 2, 4);
  }
  a.ntiles = stack ? cdiv(a.stk.rows, a.TR) : nimg * a.NB * a.NP; a.dv_nb = make_fastdiv(a.NB); a.dv_np = make_fastdiv(a.NP);
  a.nbuf = S::MAXBUF;  // as many ring buffers as fit (the balanced band may be smaller than the largest that fits three)
  while (a.nbuf > 3 && (S::lds_bytes(slots, a.TR, a.nstep, a.nbuf) > 158 * 1024 || (a.nbuf - 2) * ni > 63)) --a.nbuf;
  const int gy = cdiv(a.Cout, 64), K = 9 * CIN;
  int gx = 256 / gy; if (gx > a.ntiles) gx = a.ntiles; if (gx < 1) gx = 1;
  const int64_t per = (int64_t)a.Cout * K;
  { const int erc = ensure_partial(c, (int64_t)gx * per, gb ? (int64_t)gx * a.Cout : 0); if (erc) return erc; }
  if ((int64_t)gx * per > c->partial_elems) gx = (int)(c->partial_elems / per);
  if (gb && (int64_t)gx * a.Cout > c->bias_partial_elems) gx = (int)(c->bias_partial_elems / a.Cout);
  if (gx < 1) return 1;
  a.partial = c->partial; a.bias_partial = gb ? c->bias_partial : nullptr;
  const int lds = S::lds_bytes(slots, a.TR, a.nstep, a.nbuf);
  // full and nearly full tiles have a form of their own (branch-free tile loop); index 0: any number of steps
  constexpr int NS1 = S::MAXSTEP, NS2 = S::MAXSTEP - 1;
  const int form = (a.nstep == NS1 ? 1 : (a.nstep == NS2 ? 2 : 0)) + (cols ? 3 : stack ? 6 : 0);
  static decltype(&k_conv_wgrad_tile<CIN, 0>) const forms[9] = {k_conv_wgrad_tile<CIN, 0>, k_conv_wgrad_tile<CIN, NS1>, k_conv_wgrad_tile<CIN, NS2>,
                                                                 k_conv_wgrad_tile<CIN, 0, true>, k_conv_wgrad_tile<CIN, NS1, true>, k_conv_wgrad_tile<CIN, NS2, true>,
                                                                 k_conv_wgrad_tile<CIN, 0, false, 0, true>, k_conv_wgrad_tile<CIN, NS1, false, 0, true>,
                                                                 k_conv_wgrad_tile<CIN, NS2, false, 0, true>};
  auto kfn = forms[form];
  static uint64_t attr_devs[9] = {};  /* bit d: set on device d */
  if (!((attr_devs[form] >> c->dev) & 1)) { HIPCHK(c, hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024)); attr_devs[form] |= 1ull << c->dev; }
  {
    ProfScope ps(c, name, flops, abytes);
    hipLaunchKernelGGL(kfn, dim3(gx, gy), dim3(S::THREADS), lds, c->stream, a);
    LAUNCHCHK(c, "k_conv_wgrad_tile");
  }
  defer_reduce(c, 1, gx, per, a.Cout, K, gw, nullptr, accumulate, gb != nullptr, a.Cout, gb);
  return PPO_OK;
}
// The same for 16 input and up to 32 output channels (conv16_tile.hip.h).
int launch_conv16_wgrad_tile(Ctx* c, ConvWgradArgs a, float* gw, float* gb, bool accumulate, const std::string& name, double flops, double abytes) {
  typedef Conv16WgradShape S;
  const int nimg = a.ntiles, segs = cdiv(a.W * S::PIX, 1024);  // passed in as the image count
  if (segs > S::MAXSEG || a.Wo > 16 * S::MAXSTEP || a.Cout > 32) return 1;
  auto lds_of = [&](int tr, int nb) { return S::lds_bytes(a.W, tr, cdiv(tr * a.Wo, 16), nb); };
  auto loads = [&](int tr) { return cdiv(2 * tr + 1, 4) * segs + cdiv(cdiv(tr * a.Wo, 16), 4); };  // per loader wave and band
  int tr = std::min(16 * S::MAXSTEP / a.Wo, a.Ho);
  while (tr > 0 && (lds_of(tr, 3) > 160 * 1024 || loads(tr) > 63)) --tr;
  if (tr < 1) return 1;
  a.NB = cdiv(a.Ho, tr); a.TR = cdiv(a.Ho, a.NB); a.nstep = cdiv(a.TR * a.Wo, 16); a.ntiles = nimg * a.NB; a.dv_nb = make_fastdiv(a.NB);
  a.nbuf = S::MAXBUF;
  while (a.nbuf > 3 && (lds_of(a.TR, a.nbuf) > 160 * 1024 || (a.nbuf - 2) * loads(a.TR) > 63)) --a.nbuf;
  int gx = std::min(256, a.ntiles);
  const int64_t per = (int64_t)a.Cout * 144;
  { const int erc = ensure_partial(c, (int64_t)gx * per, gb ? (int64_t)gx * a.Cout : 0); if (erc) return erc; }
  gx = (int)std::min<int64_t>(gx, c->partial_elems / per);
  if (gb) gx = (int)std::min<int64_t>(gx, c->bias_partial_elems / a.Cout);
  if (gx < 1) return 1;
  a.partial = c->partial; a.bias_partial = gb ? c->bias_partial : nullptr;
  static uint64_t attr_devs = 0;  /* bit d: set on device d */
  if (!((attr_devs >> c->dev) & 1)) { HIPCHK(c, hipFuncSetAttribute((const void*)k_conv16_wgrad_tile, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024)); attr_devs |= 1ull << c->dev; }
  {
    ProfScope ps(c, name, flops, abytes);
    hipLaunchKernelGGL(k_conv16_wgrad_tile, dim3(gx), dim3(S::THREADS), lds_of(a.TR, a.nbuf), c->stream, a);
    LAUNCHCHK(c, "k_conv16_wgrad_tile");
  }
  defer_reduce(c, 1, gx, per, a.Cout, 144, gw, nullptr, accumulate, gb != nullptr, a.Cout, gb);
  return PPO_OK;
}
int launch_conv_wgrad_tile(Ctx* c, const ImgAddr& dy, const AConvFwd& xl, int Cout, int nimg, float* gw, float* gb, bool accumulate,
                           const std::string& name, double abytes) {
  if ((xl.Cin != 16 && xl.Cin != 32 && xl.Cin != 64) || Cout % 8 || nimg < 1 || xl.in.idx || dy.idx) return 1;
  ConvWgradArgs a;
  a.in = xl.in; a.in.prepare(); a.dy = dy; a.dy.prepare(); a.zpage = c->zpage; a.partial = nullptr; a.bias_partial = nullptr;
  a.H = xl.H; a.W = xl.W; a.Ho = xl.Ho; a.Wo = xl.Wo; a.Cout = Cout; a.TR = a.NB = a.TC = a.NP = 0; a.nstep = 0; a.nbuf = 3;
  a.ntiles = nimg;  // image count; the template turns it into tiles
  const double flops = 2.0 * (double)xl.M * Cout * xl.K;
  if (xl.Cin == 16) return launch_conv16_wgrad_tile(c, a, gw, gb, accumulate, name, flops, abytes);
  return xl.Cin == 32 ? launch_conv_wgrad_tile_t<32>(c, a, gw, gb, accumulate, name, flops, abytes)
                      : launch_conv_wgrad_tile_t<64>(c, a, gw, gb, accumulate, name, flops, abytes);
}

// Transposed convolution through the quad-organised LDS-image kernel; returns 1 when the shape is
// not covered (the caller then takes the implicit-GEMM path).  With C0 > 0 the kernel also forms
// the first layer's weight-gradient partials (a.img0, a.H0, a.W0 set by the caller) and *grid_out
// receives the number of partials.
template <int CI, int C0, bool MASK = true>
int launch_conv_dgrad_tile_t(Ctx* c, ConvDgradArgs a, int nimg, const std::string& name, double flops, double abytes, int* grid_out) {
  typedef ConvDgradShape<CI> S;
  if (a.Wo > S::BQ) return 1;
  auto lds_of = [&](int tq) { return S::lds_bytes(a.W, a.Wo, tq) + (C0 > 0 ? S::fused_extra(a.W, a.W0, C0, tq) : 0); };
  auto fits = [&](int tq) {
    if (S::stage_bytes(a.W, tq) > S::MAXCH * 256 * 16 || lds_of(tq) > 158 * 1024) return false;
    if (C0 > 0 && ((tq * a.W) % 2 != 0 || tq * a.W / 2 > 128)) return false;  // pixels per finishing wave: two per lane at most
    return true;
  };
  int TQ = S::BQ / a.Wo < a.Ho ? S::BQ / a.Wo : a.Ho;
  while (TQ > 1 && !fits(TQ)) --TQ;
  if (!fits(TQ)) return 1;
  a.NB = cdiv(a.Ho, TQ);
  if (C0 == 0 || fits(cdiv(a.Ho, a.NB))) TQ = cdiv(a.Ho, a.NB);  // balanced bands
  a.TQ = TQ; a.NB = cdiv(a.Ho, TQ); a.ntiles = nimg * a.NB;
  const int segs = cdiv(a.Wo * 128, 1024);
  int ni = cdiv(a.TQ + 1, 2) * segs;
  if (C0 > 0) {
    const int rb0 = a.W0 * C0 * 2;
    if (rb0 % 16) return 1;
    ni += cdiv(cdiv((4 * a.TQ + 1) * rb0, 1024), 2);
  }
  if (segs > S::MAXSEG || ni > 63) return 1;
  if (c->dry) return PPO_OK;
  bool stack = false;
  if constexpr (C0 == 0) {
    int tr;
    auto sfits = [&](int r) { return S::stage_bytes(a.W, r) <= S::MAXCH * 256 * 16 && lds_of(r) + S::ZERO_BYTES <= 158 * 1024 && cdiv(r + 1, 2) * segs <= 63; };
    stack = dense_images(a.x_stride_b, a.x_stride_v, a.V, (int64_t)a.H * a.W * CI) && plan_stack(nimg, a.Ho, a.Wo, S::BQ, a.NB, 256, 95, sfits, &tr);
    if (stack) {
      a.stk = make_stack(nimg, a.Ho, a.Wo, a.H, a.V);
      a.stk.dense = dense_images(a.dy.stride_b, a.dy.stride_v, a.V, (int64_t)a.Ho * a.Wo * 64);
      a.TQ = tr; a.NB = 1; a.ntiles = cdiv(a.stk.rows, tr);
    }
  }
  int gx = a.ntiles < 256 ? a.ntiles : 256;
  if (C0 > 0) {
    const int64_t npair = (int64_t)CI * (9 * C0 + 1);
    { const int erc = ensure_partial(c, gx * npair, 0); if (erc) return erc; }
    if (gx * npair > c->partial_elems) gx = (int)(c->partial_elems / npair);
    if (gx < 1) return 1;
    a.partial0 = c->partial;
    *grid_out = gx;
  }
  auto kfn = stack ? k_conv_dgrad_tile<CI, C0, MASK, C0 == 0> : k_conv_dgrad_tile<CI, C0, MASK>;
  static uint64_t attr_devs[2] = {0, 0};  /* bit d: set on device d */
  if (!((attr_devs[stack] >> c->dev) & 1)) { HIPCHK(c, hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024)); attr_devs[stack] |= 1ull << c->dev; }
  ProfScope ps(c, name, flops, abytes);
  hipLaunchKernelGGL(kfn, dim3(gx), dim3(S::THREADS), lds_of(a.TQ) + (stack ? S::ZERO_BYTES : 0), c->stream, a);
  LAUNCHCHK(c, "k_conv_dgrad_tile");
  return PPO_OK;
}
ConvDgradArgs conv_dgrad_args(Ctx* c, const ImgAddr& dy, const ImgAddr& xa, const uint32_t* xbits, bf16_t* dx, const bf16_t* wt, int H, int W, int Ho, int Wo) {
  ConvDgradArgs a;
  a.dy = dy; a.dy.prepare(); a.dx = dx; a.xbits = xbits; a.x_stride_b = xa.stride_b; a.x_stride_v = xa.stride_v;
  a.wt = wt; a.zpage = c->zpage; a.V = xa.V; a.H = H; a.W = W; a.Ho = Ho; a.Wo = a.WoR = Wo; a.TQ = 0; a.NB = 0; a.ntiles = 0; a.seg_split = 0; a.dv_wo = make_fastdiv(Wo);
  a.img0 = ImgAddr(); a.img0.base = nullptr; a.img0.idx = nullptr; a.img0.stride_b = 0; a.img0.stride_v = 0; a.img0.V = 1;
  a.H0 = 0; a.W0 = 0; a.partial0 = nullptr;
  return a;
}
// The form for 128 gradient channels and 64 result channels (the contraction split over two pairs of compute waves).
template <bool MASK, bool F32>
int launch_conv_dgrad_k2_tile(Ctx* c, ConvDgradArgs a, int nimg, const std::string& name, double flops, double abytes) {
  typedef ConvDgradK2Shape S;
  if (a.Wo > S::BQ) return 1;
  auto fits = [&](int tq) { return S::result_bytes(a.W, tq) <= S::MAXCH * S::NFT * 16 && S::lds_bytes(a.W, a.Wo, tq, F32) <= 158 * 1024; };
  int TQ = S::BQ / a.Wo < a.Ho ? S::BQ / a.Wo : a.Ho;
  while (TQ > 1 && !fits(TQ)) --TQ;
  if (!fits(TQ)) return 1;
  a.NB = cdiv(a.Ho, TQ); TQ = cdiv(a.Ho, a.NB);  // balanced bands (fewer, larger tiles beat fuller ones: the cost of a tile is mostly fixed)
  a.TQ = TQ; a.NB = cdiv(a.Ho, TQ); a.ntiles = nimg * a.NB;
  const int segs = cdiv(a.Wo * S::PB, 1024);
  if (segs > S::MAXSEG || (a.TQ + 1) * segs > 63) return 1;
  const int gx = a.ntiles < 256 ? a.ntiles : 256;
  auto kfn = k_conv_dgrad_k2_tile<MASK, F32>;
  static uint64_t attr_devs = 0;  /* bit d: set on device d */
  if (!((attr_devs >> c->dev) & 1)) { HIPCHK(c, hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024)); attr_devs |= 1ull << c->dev; }
  ProfScope ps(c, name, flops, abytes);
  hipLaunchKernelGGL(kfn, dim3(gx), dim3(S::THREADS), S::lds_bytes(a.W, a.Wo, a.TQ, F32), c->stream, a);
  LAUNCHCHK(c, "k_conv_dgrad_k2_tile");
  return PPO_OK;
}
// The form for 32 gradient channels and 16 result channels, unmasked (conv16_tile.hip.h).
int launch_conv16_dgrad_tile(Ctx* c, ConvDgradArgs a, int nimg, const std::string& name, double flops, double abytes) {
  typedef Conv16DgradShape S;
  if (a.Wo > S::BQ || cdiv(a.Wo * 64, 1024) > S::MAXSEG) return 1;
  int tq = std::min(S::BQ / a.Wo, a.Ho);
  while (tq > 1 && S::lds_bytes(a.W, a.Wo, tq) > 40 * 1024) --tq;  // four blocks to a CU
  if (S::lds_bytes(a.W, a.Wo, tq) > 80 * 1024) return 1;
  a.NB = cdiv(a.Ho, tq); a.TQ = cdiv(a.Ho, a.NB); a.ntiles = nimg * a.NB; a.dv_rb0 = make_fastdiv(a.NB);
  const int lds = S::lds_bytes(a.W, a.Wo, a.TQ), gx = std::min(a.ntiles, 256 * std::min(4, 160 * 1024 / lds));
  static uint64_t attr_devs = 0;  /* bit d: set on device d */
  if (!((attr_devs >> c->dev) & 1)) { HIPCHK(c, hipFuncSetAttribute((const void*)k_conv16_dgrad_tile, hipFuncAttributeMaxDynamicSharedMemorySize, 80 * 1024)); attr_devs |= 1ull << c->dev; }
  ProfScope ps(c, name, flops, abytes);
  hipLaunchKernelGGL(k_conv16_dgrad_tile, dim3(gx), dim3(S::THREADS), lds, c->stream, a);
  LAUNCHCHK(c, "k_conv16_dgrad_tile");
  return PPO_OK;
}
// (xbits NULL: the gradient is left unmasked; f32: partial sums stay fp32)
int launch_conv_dgrad_tile(Ctx* c, const ImgAddr& dy, const ImgAddr& xa, const uint32_t* xbits, bf16_t* dx, const bf16_t* wt, int Co, int Ci, int H, int W, int Ho, int Wo,
                           int nimg, const std::string& name, double flops, double abytes, bool f32) {
  if (dy.idx || nimg < 1) return 1;
  const ConvDgradArgs a = conv_dgrad_args(c, dy, xa, xbits, dx, wt, H, W, Ho, Wo);
  if (Co == 128 && Ci == 64) {
    if (!f32) return xbits ? launch_conv_dgrad_k2_tile<true, false>(c, a, nimg, name, flops, abytes) : 1;
    return xbits ? launch_conv_dgrad_k2_tile<true, true>(c, a, nimg, name, flops, abytes) : launch_conv_dgrad_k2_tile<false, true>(c, a, nimg, name, flops, abytes);
  }
  if (Co == 32 && Ci == 16 && !xbits) return launch_conv16_dgrad_tile(c, a, nimg, name, flops, abytes);
  if (Co != 64 || (Ci != 32 && Ci != 64)) return 1;
  if (xbits) return Ci == 32 ? launch_conv_dgrad_tile_t<32, 0>(c, a, nimg, name, flops, abytes, nullptr) : launch_conv_dgrad_tile_t<64, 0>(c, a, nimg, name, flops, abytes, nullptr);
  return Ci == 32 ? launch_conv_dgrad_tile_t<32, 0, false>(c, a, nimg, name, flops, abytes, nullptr) : launch_conv_dgrad_tile_t<64, 0, false>(c, a, nimg, name, flops, abytes, nullptr);
}
// Register-fused form of the same pair of layers (conv_dgrad_wgrad0_tile.hip.h); returns 1 when the shape is not covered.
template <int C0, int NCW, int WC = 0>
int launch_conv_dgrad_wgrad0_reg_t(Ctx* c, ConvDgradArgs a, int nimg, const std::string& name, double flops, double abytes, int* grid_out) {
  typedef ConvDgradW0Shape<NCW> S;
  const bool exact = a.W % 8 == 0 && a.Wo * 2 == a.W && a.W * 2 == a.W0;
  if (!exact && !c->dry && !c->f01_train) return 1;  // only the two layers' forward kernel stores mask rows of a rounded-up width
  a.WoR = a.Wo; a.W = cdiv(a.W, 8) * 8; a.Wo = a.W / 2;
  if (WC && (a.W != WC || a.W0 != 2 * WC || a.WoR * 2 != WC)) return 1;
  constexpr bool ones = C0 == 1 && WC != 0;  // the kernel's ONES
  const int rb0 = a.W0 * C0 * 2;
  if (rb0 % 16 || a.Wo > S::BQ || a.H != (a.H0 + 1) / 2) return 1;
  auto fits = [&](int tq) {
    return tq * a.Wo <= S::BQ && S::lds_bytes(a.W, a.Wo, a.W0, C0, tq, ones) <= 160 * 1024 && S::loads_fit(a.W, a.Wo, a.W0, C0, tq) &&
           S::dyimg_bytes(a.Wo, tq) <= 65536;  // offsets into the page of zeros
  };
  int TQ = S::BQ / a.Wo < a.Ho ? S::BQ / a.Wo : a.Ho;
  while (TQ > 1 && !fits(TQ)) --TQ;
  if (TQ < 1 || !fits(TQ)) return 1;
  a.NB = cdiv(a.Ho, TQ); a.TQ = cdiv(a.Ho, a.NB); a.NB = cdiv(a.Ho, a.TQ); a.ntiles = nimg * a.NB;
  a.dv_rb0 = make_fastdiv(rb0); a.dv_mrow = make_fastdiv(a.W * 4); a.seg_split = S::seg_split(a.Wo, a.TQ);
  if (c->dry) { c->b0pitch = a.W; return PPO_OK; }
  int gx = a.ntiles < 256 ? a.ntiles : 256;
  const int64_t npair = (int64_t)S::CI * (9 * C0 + 1);
  { const int erc = ensure_partial(c, gx * npair, 0); if (erc) return erc; }
  if (gx * npair > c->partial_elems) gx = (int)(c->partial_elems / npair);
  if (gx < 1) return 1;
  a.partial0 = c->partial;
  *grid_out = gx;
  auto kfn = k_conv_dgrad_wgrad0_tile<C0, NCW, WC>;
  static uint64_t attr_devs = 0;  /* bit d: set on device d */
  if (!((attr_devs >> c->dev) & 1)) { HIPCHK(c, hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024)); attr_devs |= 1ull << c->dev; }
  ProfScope ps(c, name, flops, abytes);
  hipLaunchKernelGGL(kfn, dim3(gx), dim3(S::THREADS), S::lds_bytes(a.W, a.Wo, a.W0, C0, a.TQ, ones), c->stream, a);
  LAUNCHCHK(c, "k_conv_dgrad_wgrad0_tile");
  return PPO_OK;
}
// The same with the first layer's weight gradient fused in (depth or RGB input, 32 channels after the first layer).
int launch_conv_dgrad_wgrad0_tile(Ctx* c, const ImgAddr& dy, const ImgAddr& xa, const uint32_t* xbits, const bf16_t* wt, int Co, int Ci, int H, int W, int Ho, int Wo,
                                  const ImgAddr& img0, int C0, int H0, int W0, int nimg, const std::string& name, double flops, double abytes, int* grid_out) {
  if (Co != 64 || Ci != 32 || (C0 != 1 && C0 != 3) || dy.idx || nimg < 1 || !xbits) return 1;
  ConvDgradArgs a = conv_dgrad_args(c, dy, xa, xbits, nullptr, wt, H, W, Ho, Wo);
  a.img0 = img0; a.img0.prepare(); a.H0 = H0; a.W0 = W0;
  if (c->dry) c->b0pitch = W;  // words per mask row, unless a form below rounds it up
  // eight compute waves (two per SIMD) when the larger tile fits, else four
  // (the 80-wide result of 120x160 depth images has a form of its own with the row pitches known at compile time)
  int rrc = C0 == 1 ? launch_conv_dgrad_wgrad0_reg_t<1, 8, 80>(c, a, nimg, name, flops, abytes, grid_out) : 1;
  if (rrc == 1)
    rrc = C0 == 1 ? launch_conv_dgrad_wgrad0_reg_t<1, 8>(c, a, nimg, name, flops, abytes, grid_out)
                  : launch_conv_dgrad_wgrad0_reg_t<3, 8>(c, a, nimg, name, flops, abytes, grid_out);
  if (rrc == 1)
    rrc = C0 == 1 ? launch_conv_dgrad_wgrad0_reg_t<1, 4>(c, a, nimg, name, flops, abytes, grid_out)
                  : launch_conv_dgrad_wgrad0_reg_t<3, 4>(c, a, nimg, name, flops, abytes, grid_out);
  if (rrc != 1) return rrc;
  if (!c->dry && c->f01_train && c->b0pitch != W) return fail(c, PPO_ENOMEM, "the input-gradient kernel does not fit the workspace it was chosen for");
  return C0 == 1 ? launch_conv_dgrad_tile_t<32, 1>(c, a, nimg, name, flops, abytes, grid_out)
                 : launch_conv_dgrad_tile_t<32, 3>(c, a, nimg, name, flops, abytes, grid_out);
}

// First convolution forward through the LDS-ring kernel; returns 1 when the shape is not covered.
template <int C0, bool RELU = true>
int launch_conv0_fwd_tile_t(Ctx* c, Conv0Args a, int nimg) {
  typedef Conv0Shape<C0> S;
  const int rb = a.W * C0 * 2;
  if (rb % 16 || ((int64_t)a.H * rb) % 16 || a.Cout % 8 || a.Cout > 64) return 1;
  int TR = 0;
  for (int tr = a.Ho; tr >= 1; --tr)
    if (cdiv((2 * tr + 1) * rb, 1024) <= 63 && tr * a.Wo <= 1024 && S::lds_bytes(a.W, tr, a.Cout) <= 64 * 1024) { TR = tr; break; }
  if (TR == 0) return 1;
  a.NB = cdiv(a.Ho, TR); a.TR = cdiv(a.Ho, a.NB); a.ntiles = nimg * a.NB;
  a.dv_wo = make_fastdiv(a.Wo);
  int gx = a.ntiles < 512 ? a.ntiles : 512;
  a.tile_blocks = gx;
  if (a.gather_blocks > 0) a.gather_blocks = (int)std::min<int64_t>(32, cdiv((int64_t)a.pB * a.P, 512));
  auto kfn = k_conv0_fwd_tile<C0, RELU>;
  static uint64_t attr_devs = 0;  /* bit d: set on device d */
  if (!((attr_devs >> c->dev) & 1)) { HIPCHK(c, hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, 64 * 1024)); attr_devs |= 1ull << c->dev; }
  hipLaunchKernelGGL(kfn, dim3(gx + a.gather_blocks), dim3(S::THREADS), S::lds_bytes(a.W, a.TR, a.Cout), c->stream, a);
  LAUNCHCHK(c, "k_conv0_fwd_tile");
  return PPO_OK;
}

// First convolution's weight and bias gradient from a stored output gradient through the LDS-ring kernel; returns 1 when
// the shape is not covered.  *grid_out receives the number of partials.
template <int C0, int CO>
int launch_conv0_wgrad_tile_t(Ctx* c, Conv0WgradArgs a, int nimg, int* grid_out) {
  typedef Conv0WgradShape<C0, CO> S;
  const int rb = a.W * C0 * 2;
  if (rb % 16) return 1;
  // two blocks of four compute waves per CU; as many rows per band as three ring slots of half the LDS hold
  int TR = 0;
  for (int tr = a.Ho; tr >= 1; --tr)
    if (S::lds_bytes(a.W, a.Wo, tr) <= 79 * 1024 && cdiv(cdiv((2 * tr + 1) * rb, 1024), 4) + cdiv(cdiv(S::dy_bytes(a.Wo, tr), 1024), 4) <= 63) { TR = tr; break; }
  if (TR == 0) return 1;
  a.NB = cdiv(a.Ho, TR); a.TR = cdiv(a.Ho, a.NB); a.ntiles = nimg * a.NB;
  a.dv_rb = make_fastdiv(rb);
  int gx = a.ntiles < 512 ? a.ntiles : 512;
  const int64_t npair = (int64_t)CO * (S::K0 + 1);
  { const int erc = ensure_partial(c, gx * npair, 0); if (erc) return erc; }
  if (gx * npair > c->partial_elems) gx = (int)(c->partial_elems / npair);
  if (gx < 1) return 1;
  a.partial = c->partial; *grid_out = gx;
  auto kfn = k_conv0_wgrad_tile<C0, CO>;
  static uint64_t attr_devs = 0;  /* bit d: set on device d */
  if (!((attr_devs >> c->dev) & 1)) { HIPCHK(c, hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, 80 * 1024)); attr_devs |= 1ull << c->dev; }
  hipLaunchKernelGGL(kfn, dim3(gx), dim3(S::THREADS), S::lds_bytes(a.W, a.Wo, a.TR), c->stream, a);
  LAUNCHCHK(c, "k_conv0_wgrad_tile");
  return PPO_OK;
}
// The same with any kernel: leaves the partials at the cursor and queues their reduction.
int conv0_wgrad(Ctx* c, ImgAddr in, const bf16_t* dy, int nimg, bool acc) {
  in.prepare();
  const int Co = c->cC[1], Ho = c->cH[1], Wo = c->cW[1], C0 = c->cC[0], K = 9 * C0, npair = Co * (K + 1);
  const int64_t M = (int64_t)nimg * Ho * Wo;
  ProfScope ps(c, "conv_wgrad.0", 2.0 * (double)M * Co * (K + 1), 2.0 * ((double)M * Co + (double)nimg * c->img_elems));
  Conv0WgradArgs wa;
  wa.in = in; wa.dy = dy; wa.zpage = c->zpage; wa.partial = nullptr; wa.H = c->cH[0]; wa.W = c->cW[0]; wa.Ho = Ho; wa.Wo = Wo; wa.TR = wa.NB = wa.ntiles = 0;
  int nblk = 0;
#define WGRAD0_CO(C0_) (Co == 8 ? launch_conv0_wgrad_tile_t<C0_, 8>(c, wa, nimg, &nblk) : Co == 16 ? launch_conv0_wgrad_tile_t<C0_, 16>(c, wa, nimg, &nblk) \
                        : Co == 32 ? launch_conv0_wgrad_tile_t<C0_, 32>(c, wa, nimg, &nblk) : Co == 64 ? launch_conv0_wgrad_tile_t<C0_, 64>(c, wa, nimg, &nblk) : 1)
  const int rc = C0 == 1 ? WGRAD0_CO(1) : WGRAD0_CO(3);
#undef WGRAD0_CO
  if (rc != PPO_OK && rc != 1) return rc;
  if (rc == 1) {
    { const int erc = ensure_partial(c, (int64_t)2048 * npair, 0); if (erc) return erc; }
    int64_t max_blocks = c->partial_elems / npair;
    if (max_blocks > 2048) max_blocks = 2048;
    if (max_blocks < 1) return fail(c, PPO_ENOMEM, "weight-gradient workspace too small for the first convolution");
    int64_t ppb = (M + max_blocks - 1) / max_blocks;
    ppb = (ppb + 63) / 64 * 64;
    nblk = cdiv(M, ppb);
    if (C0 == 1) hipLaunchKernelGGL((k_conv1_wgrad<1>), dim3(nblk), dim3(256), 0, c->stream, in, nimg, c->cH[0], c->cW[0], Ho, Wo, Co, dy, (int)ppb, c->partial);
    else hipLaunchKernelGGL((k_conv1_wgrad<3>), dim3(nblk), dim3(256), 0, c->stream, in, nimg, c->cH[0], c->cW[0], Ho, Wo, Co, dy, (int)ppb, c->partial);
    LAUNCHCHK(c, "k_conv1_wgrad");
  }
  defer_reduce(c, 2, nblk, npair, Co, K, c->g + c->convW[0], c->g + c->convB[0], acc, false, 0, nullptr);
  return PPO_OK;
}

// The student's auxiliary MLP head on the last hidden layer x [n][hid]: hidden layer (bias, ReLU) into auxact, its
// X outputs into the columns [A_main, A) of the head-output rows, behind the linear head's.
int aux_head_forward(Ctx* c, const bf16_t* x, int64_t ldx, int n) {
  if (c->XH <= 0) return PPO_OK;
  ARows al = plain_arows(x, ldx, n, c->hid);
  Ep<MapRows, bf16_t, true, true, false> e1;
  e1.map = plain_map(c->XH, n); e1.out = c->auxact; e1.bias = c->p + c->aux1B; e1.mask = nullptr; e1.N = c->XH;
  int rc = launch_gemm(c, al, n, c->shadow + c->aux1W, c->hid, c->XH, c->hid, e1, "aux_fwd.0", 2.0 * n * ((double)c->hid + c->XH) + 2.0 * c->hid * c->XH);
  if (rc) return rc;
  ARows a2 = plain_arows(c->auxact, c->XH, n, c->XH);
  Ep<MapRows, float, true, false, false> e2;
  e2.map = plain_map(HEAD_LD, n); e2.out = c->headout + c->A_main; e2.bias = c->p + c->aux2B; e2.mask = nullptr; e2.N = c->X;
  return launch_gemm(c, a2, n, c->shadow + c->aux2W, c->XH, c->X, c->XH, e2, "aux_fwd.1", 2.0 * n * c->XH + 4.0 * n * c->X);
}
// Its backward from the loss gradient rows dhead [n][32]: weight and bias gradients of both layers, and the
// gradient it sends into the last hidden layer h, added to what the linear head left in dh [n][hid]
// (scratch: another [n][hid] buffer).
int aux_head_backward(Ctx* c, const bf16_t* h, int n, bool acc, bf16_t* dh, bf16_t* scratch) {
  if (c->XH <= 0) return PPO_OK;
  hipLaunchKernelGGL(k_aux_cols, dim3(cdiv((int64_t)n * 32, 256)), dim3(256), 0, c->stream, n, c->A_main, c->X, c->dhead, c->daux);
  LAUNCHCHK(c, "k_aux_cols");
  ARows dl2 = plain_arows(c->daux, HEAD_LD, n, HEAD_LD);
  ARows x2 = plain_arows(c->auxact, c->XH, n, c->XH);
  int rc = launch_wgrad(c, dl2, x2, c->X, c->XH, n, c->g + c->aux2W, c->g + c->aux2B, acc, "aux_wgrad.1", 2.0 * n * (c->XH + HEAD_LD));
  if (rc) return rc;
  Ep<MapRows, bf16_t, false, false, true> e2;
  e2.map = plain_map(c->XH, n); e2.out = c->dauxact; e2.bias = nullptr; e2.mask = c->auxact; e2.N = c->XH;
  rc = launch_gemm(c, dl2, n, c->aux2T, HEAD_LD, c->XH, HEAD_LD, e2, "aux_dgrad.1", 2.0 * n * (2.0 * c->XH + HEAD_LD));
  if (rc) return rc;
  ARows dl1 = plain_arows(c->dauxact, c->XH, n, c->XH);
  ARows x1 = plain_arows(h, c->hid, n, c->hid);
  rc = launch_wgrad(c, dl1, x1, c->XH, c->hid, n, c->g + c->aux1W, c->g + c->aux1B, acc, "aux_wgrad.0", 2.0 * n * ((double)c->hid + c->XH));
  if (rc) return rc;
  Ep<MapRows, bf16_t, false, false, true> e1;
  e1.map = plain_map(c->hid, n); e1.out = scratch; e1.bias = nullptr; e1.mask = h; e1.N = c->hid;
  rc = launch_gemm(c, dl1, n, c->aux1T, c->XH, c->hid, c->XH, e1, "aux_dgrad.0", 2.0 * n * (2.0 * c->hid + c->XH));
  if (rc) return rc;
  hipLaunchKernelGGL(k_add_bf16, dim3(cdiv((int64_t)n * c->hid / 8, 256)), dim3(256), 0, c->stream, (int64_t)n * c->hid / 8, dh, scratch);
  LAUNCHCHK(c, "k_add_bf16");
  return PPO_OK;
}

// Both convolutions of a small network in one kernel (conv_small.hip.h): one-channel images whose pixels, activation and
// gradient fit half of the LDS (up to about 96 x 96).
bool conv_small_covers(const Ctx* c) {
  return c->nconv == 2 && c->cC[0] == 1 && c->cC[1] == 8 && c->cC[2] == 16 && !c->ln && c->E == 0 && c->nl == 0 &&
         ConvSmallShape::covers(c->cH[0], c->cW[0], c->cH[1], c->cH[2], c->cW[2]);
}
ConvSmallArgs conv_small_args(Ctx* c, const int32_t* idx, int nimg, int64_t first) {
  ConvSmallArgs a = {};
  a.in.base = c->obs + first * c->img_elems * c->V; a.in.idx = idx; a.in.stride_b = c->img_elems * c->V; a.in.stride_v = c->img_elems; a.in.V = c->V;
  a.in.prepare();
  a.w0 = c->shadow + c->convW[0]; a.w1 = c->shadow + c->convW[1]; a.w1t = c->wtap[1]; a.b0 = c->p + c->convB[0]; a.b1 = c->p + c->convB[1];
  a.feat_ld = c->feat_ld; a.V = c->V; a.flat = c->flat; a.nimg = nimg;
  a.H = c->cH[0]; a.W = c->cW[0]; a.Ho0 = c->cH[1]; a.Wo0 = c->cW[1]; a.Ho1 = c->cH[2]; a.Wo1 = c->cW[2];
  a.dv0 = make_fastdiv(a.Wo0); a.dv1 = make_fastdiv(a.Wo1); a.dvr = make_fastdiv(a.W / 8);
  return a;
}
// Blocks per CU: what the LDS and the registers (two waves per SIMD backward, three forward) hold at once.
int conv_small_grid(Ctx* c, const ConvSmallArgs& a, bool bwd, int* grid, int* lds, int* ch) {
  static uint64_t attr_devs = 0;  /* bit d: set on device d */
  if (!((attr_devs >> c->dev) & 1)) {
    for (const void* k : {(const void*)k_conv_small_fwd<1>, (const void*)k_conv_small_fwd<2>, (const void*)k_conv_small_fwd<ConvSmallShape::CHUNKS>,
                          (const void*)k_conv_small_bwd<1>, (const void*)k_conv_small_bwd<2>, (const void*)k_conv_small_bwd<ConvSmallShape::CHUNKS>})
      HIPCHK(c, hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, 80 * 1024));
    attr_devs |= 1ull << c->dev;
  }
  *ch = cdiv(std::max(a.H * (a.W / 8), bwd ? a.Ho1 * a.Wo1 * 2 : 0), 256);
  *lds = std::max(ConvSmallShape::block_bytes(a.W, a.Ho0, a.Ho1, a.Wo1, bwd), bwd ? 4 * ConvSmallShape::RED * 4 : 0);
  *grid = std::min(a.nimg, 256 * std::min(bwd ? 2 : 3, 160 * 1024 / *lds));
  return PPO_OK;
}
int conv_small_forward(Ctx* c, const int32_t* idx, int n, int64_t first) {
  const int nimg = n * c->V;
  ConvSmallArgs a = conv_small_args(c, idx, nimg, first);
  a.feat = c->feat; a.proprio = c->proprio + first * c->P; a.P = c->P;
  int grid, lds, ch;
  { const int erc = conv_small_grid(c, a, false, &grid, &lds, &ch); if (erc) return erc; }
  const double m0 = (double)nimg * a.Ho0 * a.Wo0, m1 = (double)nimg * a.Ho1 * a.Wo1;
  ProfScope ps(c, "conv_small_fwd", 2.0 * (m0 * 72 + m1 * 1152), 2.0 * ((double)nimg * c->img_elems + m1 * 16));
  if (ch <= 1) hipLaunchKernelGGL(k_conv_small_fwd<1>, dim3(grid), dim3(256), lds, c->stream, a);
  else if (ch <= 2) hipLaunchKernelGGL(k_conv_small_fwd<2>, dim3(grid), dim3(256), lds, c->stream, a);
  else hipLaunchKernelGGL(k_conv_small_fwd<ConvSmallShape::CHUNKS>, dim3(grid), dim3(256), lds, c->stream, a);
  LAUNCHCHK(c, "k_conv_small_fwd");
  c->abits_ok[0] = false;
  return PPO_OK;
}
// The forward of n samples in one kernel (small_net.hip.h): one hidden layer of 32 or 64 units behind one view, a product that the
// separate launch would give to k_gemm_small, and few samples (four to a block: 1024 environments 20.1 -> 14.8 us a policy step;
// with eight to a block it would take as long as the separate launches).
bool small_net_covers(const Ctx* c, int n) {
  return conv_small_covers(c) && c->V == 1 && c->nfc == 1 && (c->fout[0] == 32 || c->fout[0] == 64) && c->fin[0] <= 2048 && c->P % 8 == 0 && c->P > 0 &&
         c->fin[0] == c->flat + c->P && n <= 256 * SmallNetShape::MAXS && gemm_small_covers(n, c->fout[0], c->fin[0]);
}
template <typename InT, bool ACT>
int launch_small_net(Ctx* c, SmallNetArgs a) {
  a.K = c->fin[0]; a.S = cdiv(a.n, 256); a.w = c->shadow + c->fcW[0]; a.b = c->p + c->fcB[0];
  const int nw = a.K <= 512 ? 4 : 8, nk = cdiv(cdiv(a.K, 16), nw);  // k_gemm_small's slices
  a.per = nk * 16;
  const int lds = SmallNetShape::lds_bytes(a.cs, a.K, a.S, c->fout[0]);
#define LAUNCH_SMALL(HID_, NK_)                                                                                                           \
  do {                                                                                                                                      \
    static uint64_t attr_devs = 0;  /* bit d: set on device d */                                                                            \
    if (!((attr_devs >> c->dev) & 1)) { HIPCHK(c, hipFuncSetAttribute((const void*)k_small_net<InT, HID_, NK_, ACT>, hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024)); attr_devs |= 1ull << c->dev; } \
    hipLaunchKernelGGL((k_small_net<InT, HID_, NK_, ACT>), dim3(cdiv(a.n, a.S)), dim3(512), lds, c->stream, a);                              \
  } while (0)
  if (c->fout[0] == 32) { if (nk <= 9) LAUNCH_SMALL(32, 9); else LAUNCH_SMALL(32, 16); }
  else { if (nk <= 9) LAUNCH_SMALL(64, 9); else LAUNCH_SMALL(64, 16); }
#undef LAUNCH_SMALL
  LAUNCHCHK(c, "k_small_net");
  return PPO_OK;
}
// features and hidden activations of n samples of the buffer, chosen by idx (NULL: first ..)
int small_net_forward(Ctx* c, const int32_t* idx, int n, int64_t first) {
  SmallNetArgs a = {};
  if (idx) first = 0;
  a.cs = conv_small_args(c, idx, n, first); a.cs.feat = c->feat; a.cs.proprio = c->proprio + first * c->P; a.cs.P = c->P;
  a.n = n; a.hout = c->fcact[0];
  ProfScope ps(c, "small_net_fwd", 2.0 * n * ((double)a.cs.Ho0 * a.cs.Wo0 * 72 + (double)a.cs.Ho1 * a.cs.Wo1 * 1152 + (double)c->fin[0] * c->fout[0]),
               2.0 * n * ((double)c->img_elems + c->fin[0] + c->fout[0]));
  c->abits_ok[0] = false;
  return launch_small_net<bf16_t, false>(c, a);
}
// from the masked gradient of the feature matrix in gbuf[cur]
int conv_small_backward(Ctx* c, const int32_t* idx, int n, bool acc, int cur) {
  const int nimg = n * c->V;
  ConvSmallArgs a = conv_small_args(c, idx, nimg, 0);
  a.dfeat = c->gbuf[cur];
  int grid, lds, ch;
  { const int erc = conv_small_grid(c, a, true, &grid, &lds, &ch); if (erc) return erc; }
  { const int erc = ensure_partial(c, (int64_t)grid * (1152 + 80), (int64_t)grid * 16); if (erc) return erc; }
  grid = (int)std::min<int64_t>(grid, std::min(c->partial_elems / (1152 + 80), c->bias_partial_elems / 16));
  if (grid < 1) return fail(c, PPO_ENOMEM, "weight-gradient workspace too small for the convolutions");
  a.part1 = c->partial; a.bpart1 = c->bias_partial; a.part0 = c->partial + (int64_t)grid * 1152;
  {
    const double m0 = (double)nimg * a.Ho0 * a.Wo0, m1 = (double)nimg * a.Ho1 * a.Wo1;
    ProfScope ps(c, "conv_small_bwd", 2.0 * (2.0 * m0 * 72 + 2.0 * m1 * 1152), 2.0 * ((double)nimg * c->img_elems + m1 * 16));
    if (ch <= 1) hipLaunchKernelGGL(k_conv_small_bwd<1>, dim3(grid), dim3(256), lds, c->stream, a);
    else if (ch <= 2) hipLaunchKernelGGL(k_conv_small_bwd<2>, dim3(grid), dim3(256), lds, c->stream, a);
    else hipLaunchKernelGGL(k_conv_small_bwd<ConvSmallShape::CHUNKS>, dim3(grid), dim3(256), lds, c->stream, a);
    LAUNCHCHK(c, "k_conv_small_bwd");
  }
  defer_reduce(c, 0, grid, 1152, 0, 0, c->g + c->convW[1], nullptr, acc, true, 16, c->g + c->convB[1]);
  defer_reduce(c, 2, grid, 80, 8, 9, c->g + c->convW[0], c->g + c->convB[0], acc, false, 0, nullptr);
  return PPO_OK;
}

// Encoder of the feed-forward configurations: convolutions with fused bias + ReLU, the last one writing into the
// feature matrix, whose tail columns receive the proprioception.  `n` samples selected by device indices idx
// (NULL: samples first .. first + n - 1 of the buffer).
// train: a backward pass follows and wants the mask bits.
int encoder_forward_ff(Ctx* c, const int32_t* idx, int n, int64_t first, bool train) {
  const int V = c->V, nimg = n * V;
  bool proprio_done = false;
  if (idx) first = 0;
  if (conv_small_covers(c)) return conv_small_forward(c, idx, n, first);
  const bf16_t* const proprio = c->proprio + first * c->P;
  ImgAddr in; in.base = c->obs + first * c->img_elems * V; in.idx = idx; in.stride_b = c->img_elems * V; in.stride_v = c->img_elems; in.V = V;
  const bool both = train ? c->f01_train : c->f01_fwd;
  if (both) {
    const int rc = launch_conv01_fwd(c, in, conv_out_addr(c, 1, c->act[1], c->feat), proprio, n, train);
    if (rc) return rc == 1 ? fail(c, PPO_ESHAPE, "the first two convolutions' kernel does not cover the shapes it was chosen for") : rc;
    c->abits_ok[0] = train; c->abits_ok[1] = train && c->nconv > 2;
    proprio_done = true;
  } else {  // first convolution straight from the rollout buffer
    int Co = c->cC[1], Ho = c->cH[1], Wo = c->cW[1];
    int64_t M = (int64_t)nimg * Ho * Wo;
    ProfScope ps(c, "conv_fwd.0", 2.0 * (double)M * Co * 9 * c->cC[0], 2.0 * ((double)nimg * c->img_elems + (double)M * Co));
    constexpr int TPW = 4;
    const int grid = cdiv(M, 32 * 4 * TPW);
    Conv0Args ca;
    ca.in = in; ca.in.prepare(); ca.out = c->act[0]; ca.w = c->shadow + c->convW[0]; ca.bias = c->p + c->convB[0]; ca.zpage = c->zpage;
    ca.bits = train && c->nconv > 1 ? c->abits[0] : nullptr;
    ca.H = c->cH[0]; ca.W = c->cW[0]; ca.Ho = Ho; ca.Wo = Wo; ca.Cout = Co; ca.TR = 0; ca.NB = 0; ca.ntiles = 0;
    ca.tile_blocks = 0; ca.gather_blocks = 1; ca.pB = n; ca.P = c->P; ca.pcol0 = V * c->flat; ca.proprio = proprio; ca.feat = c->feat; ca.feat_ld = c->feat_ld;
    int trc = c->cC[0] == 1 ? launch_conv0_fwd_tile_t<1>(c, ca, nimg) : (c->cC[0] == 3 ? launch_conv0_fwd_tile_t<3>(c, ca, nimg) : 1);
    if (trc != PPO_OK && trc != 1) return trc;
    c->abits_ok[0] = trc == PPO_OK && ca.bits;
    proprio_done = trc == PPO_OK;
    if (trc != PPO_OK) {  // shapes the LDS-ring kernel does not cover
      if (c->cC[0] == 1)
        hipLaunchKernelGGL((k_conv1_fwd<1, TPW>), dim3(grid), dim3(256), 0, c->stream, in, nimg, c->cH[0], c->cW[0], Ho, Wo, Co, c->shadow + c->convW[0], c->p + c->convB[0], c->act[0]);
      else
        hipLaunchKernelGGL((k_conv1_fwd<3, TPW>), dim3(grid), dim3(256), 0, c->stream, in, nimg, c->cH[0], c->cW[0], Ho, Wo, Co, c->shadow + c->convW[0], c->p + c->convB[0], c->act[0]);
      LAUNCHCHK(c, "k_conv1_fwd");
    }
  }
  for (int l = both ? 2 : 1; l < c->nconv; ++l) {
    AConvFwd al;
    al.in = conv_out_addr(c, l - 1, c->act[l - 1], nullptr);
    al.H = c->cH[l]; al.W = c->cW[l]; al.Cin = c->cC[l]; al.lc = ilog2(al.Cin); al.Ho = c->cH[l + 1]; al.Wo = c->cW[l + 1];
    al.M = nimg * al.Ho * al.Wo; al.K = 9 * al.Cin;
    ImgAddr o = conv_out_addr(c, l, c->act[l], c->feat);
    Ep<MapRows, bf16_t, true, true, false> ep;
    ep.map.stride_b = o.stride_b; ep.map.stride_v = o.stride_v; ep.map.V = V; ep.map.HW = al.Ho * al.Wo; ep.map.C = c->cC[l + 1]; ep.map.M = al.M;
    ep.out = const_cast<bf16_t*>(o.base); ep.bias = c->p + c->convB[l]; ep.mask = nullptr; ep.N = c->cC[l + 1];
    double ab = 2.0 * ((double)nimg * al.H * al.W * al.Cin + (double)al.M * c->cC[l + 1] + (double)al.K * c->cC[l + 1]);
    const bool want_bits = train && l < c->nconv - 1;  // the last layer's mask is applied by the first linear layer's input gradient
    int rc = launch_conv_fwd_tile(c, al, o, c->cC[l + 1], c->shadow + c->convW[l], c->p + c->convB[l], nimg, "conv_fwd." + std::to_string(l), ab,
                                  want_bits ? c->abits[l] : nullptr);
    c->abits_ok[l] = want_bits && rc == PPO_OK;
    if (rc == PPO_OK + 1) rc = launch_gemm(c, al, al.M, c->shadow + c->convW[l], al.K, c->cC[l + 1], al.K, ep, "conv_fwd." + std::to_string(l), ab);
    if (rc) return rc;
  }
  if (!proprio_done) {  // (the first convolution's kernel copies the proprioception when it is the LDS-ring form)
    hipLaunchKernelGGL(k_gather_proprio, dim3(cdiv((int64_t)n * c->P, 256)), dim3(256), 0, c->stream, proprio, idx, n, c->P, c->feat, (int64_t)c->feat_ld, V * c->flat);
    LAUNCHCHK(c, "k_gather_proprio");
  }
  return PPO_OK;
}

// Hidden layers (bias, ReLU) on the trunk's input x [n][fin0] (row stride ldx), then the heads.
int trunk_forward(Ctx* c, const bf16_t* x, int64_t ldx, int n, bool with_head) {
  for (int l = 0; l < c->nfc; ++l) {
    ARows al = plain_arows(x, ldx, n, c->fin[l]);
    Ep<MapRows, bf16_t, true, true, false> ep;
    ep.map = plain_map(c->fout[l], n); ep.out = c->fcact[l]; ep.bias = c->p + c->fcB[l]; ep.mask = nullptr; ep.N = c->fout[l];
    double ab = 2.0 * ((double)n * c->fin[l] + (double)n * c->fout[l] + (double)c->fin[l] * c->fout[l]);
    int rc = launch_gemm(c, al, n, c->shadow + c->fcW[l], c->fin[l], c->fout[l], c->fin[l], ep, "fc_fwd." + std::to_string(l), ab);
    if (rc) return rc;
    x = c->fcact[l]; ldx = c->fout[l];
  }
  if (with_head) {
    ARows al = plain_arows(x, ldx, n, c->hid);
    Ep<MapRows, float, true, false, false> ep;
    ep.map = plain_map(HEAD_LD, n); ep.out = c->headout; ep.bias = c->p + c->headB; ep.mask = nullptr; ep.N = c->NH;
    int rc = launch_gemm(c, al, n, c->shadow + c->headW, c->hid, c->NH, c->hid, ep, "head_fwd", 2.0 * n * c->hid + 4.0 * n * c->NH);
    if (rc) return rc;
    rc = aux_head_forward(c, x, ldx, n);
    if (rc) return rc;
  }
  return PPO_OK;
}

int encoder_forward_generic(Ctx* c, const int32_t* idx, int n, int64_t first);

// Forward of `n` samples of a feed-forward network selected by device indices idx (NULL: samples first ..
// first + n - 1 of the buffer).
int forward_chunk(Ctx* c, const int32_t* idx, int n, bool train, bool with_head, int64_t first = 0) {
  if (!with_head && small_net_covers(c, n)) return small_net_forward(c, idx, n, first);
  const int rc = (c->ln || c->E > 0) ? encoder_forward_generic(c, idx, n, first) : encoder_forward_ff(c, idx, n, first, train);
  if (rc) return rc;
  return trunk_forward(c, c->feat, c->feat_ld, n, with_head);
}

// Backward of heads and hidden layers of a chunk whose forward activations are in the workspaces and whose
// head gradient is in dhead; xin [n][fin0] (row stride ldin) is the trunk's input.  Gradients land in c->g
// (overwritten, or added when `acc`); the gradient w.r.t. the trunk's input is left in gbuf[*cur_out] as
// [n][fin0], masked by xin > 0 when `mask_in` (xin is then a ReLU output).
int trunk_backward(Ctx* c, const bf16_t* xin, int64_t ldin, bool mask_in, int n, bool acc, bool with_head, int* cur_out) {
  int cur = 0;
  const bf16_t* hlast = c->fcact[c->nfc - 1];
  if (with_head) {  // heads (otherwise gbuf[0] already holds the gradient of the last hidden layer)
    ARows dl = plain_arows(c->dhead, HEAD_LD, n, HEAD_LD);
    ARows xl = plain_arows(hlast, c->hid, n, c->hid);
    int rc = launch_wgrad(c, dl, xl, c->NH, c->hid, n, c->g + c->headW, c->g + c->headB, acc, "head_wgrad", 2.0 * n * (c->hid + HEAD_LD));
    if (rc) return rc;
    Ep<MapRows, bf16_t, false, false, true> ep;
    ep.map = plain_map(c->hid, n); ep.out = c->gbuf[cur]; ep.bias = nullptr; ep.mask = hlast; ep.N = c->hid;
    rc = launch_gemm(c, dl, n, c->headT, HEAD_LD, c->hid, HEAD_LD, ep, "head_dgrad", 2.0 * n * (2.0 * c->hid + HEAD_LD));
    if (rc) return rc;
    rc = aux_head_backward(c, hlast, n, acc, c->gbuf[cur], c->gbuf[cur ^ 1]);
    if (rc) return rc;
  }
  for (int l = c->nfc - 1; l >= 0; --l) {
    const bf16_t* x = l ? c->fcact[l - 1] : xin;
    const int64_t ldx = l ? c->fin[l] : ldin;
    ARows dl = plain_arows(c->gbuf[cur], c->fout[l], n, c->fout[l]);
    ARows xl = plain_arows(x, ldx, n, c->fin[l]);
    const double ab = 2.0 * ((double)n * c->fout[l] + 2.0 * n * c->fin[l] + (double)c->fin[l] * c->fout[l]);
    const bool masked = l > 0 || mask_in;
    DgradBeside beside = {};
    beside.wT = c->fcT[l]; beside.abytes = ab;
    Ep<MapRows, bf16_t, false, false, true>& ep = beside.ep;
    ep.map = plain_map(c->fin[l], n); ep.out = c->gbuf[cur ^ 1]; ep.bias = nullptr; ep.mask = x; ep.N = c->fin[l];
    int rc = launch_wgrad(c, dl, xl, c->fout[l], c->fin[l], n, c->g + c->fcW[l], c->g + c->fcB[l], acc, "fc_wgrad." + std::to_string(l),
                          2.0 * n * ((double)c->fin[l] + c->fout[l]) + 4.0 * (double)c->fin[l] * c->fout[l], masked ? &beside : nullptr);
    if (rc) return rc;
    if (masked) {
      if (!beside.taken) rc = launch_gemm(c, dl, n, c->fcT[l], c->fout[l], c->fin[l], c->fout[l], ep, "fc_dgrad." + std::to_string(l), ab);
    } else {  // the trunk's input is not a ReLU output (an embedding, an LSTM's h): nothing to mask
      Ep<MapRows, bf16_t, false, false, false> ep;
      ep.map = plain_map(c->fin[l], n); ep.out = c->gbuf[cur ^ 1]; ep.bias = nullptr; ep.mask = nullptr; ep.N = c->fin[l];
      rc = launch_gemm(c, dl, n, c->fcT[l], c->fout[l], c->fin[l], c->fout[l], ep, "fc_dgrad." + std::to_string(l), ab);
    }
    if (rc) return rc;
    cur ^= 1;
  }
  *cur_out = cur;
  return PPO_OK;
}

// Backward of the feed-forward configurations' convolutions from d(feat) in gbuf[cur] ([n][feat_ld], already masked
// by the last conv layer's ReLU).
int encoder_backward_ff(Ctx* c, const int32_t* idx, int n, bool acc, int cur) {
  const int V = c->V, nimg = n * V;
  if (conv_small_covers(c)) {
    const int rc = conv_small_backward(c, idx, n, acc, cur);
    return rc ? rc : flush_reduces(c);
  }
  for (int l = c->nconv - 1; l >= 1; --l) {
    const int Co = c->cC[l + 1], Ci = c->cC[l], Ho = c->cH[l + 1], Wo = c->cW[l + 1], H = c->cH[l], W = c->cW[l];
    ImgAddr dy = conv_out_addr(c, l, c->gbuf[cur], c->gbuf[cur]);
    ARows dl; dl.a = dy; dl.HW = Ho * Wo; dl.C = Co; dl.M = nimg * Ho * Wo; dl.K = Co; dl.plain = false;
    AConvFwd xl; xl.in = conv_out_addr(c, l - 1, c->act[l - 1], nullptr);
    xl.H = H; xl.W = W; xl.Cin = Ci; xl.lc = ilog2(Ci); xl.Ho = Ho; xl.Wo = Wo; xl.M = dl.M; xl.K = 9 * Ci;
    const double wab = 2.0 * ((double)dl.M * Co + (double)nimg * H * W * Ci) + 4.0 * 9.0 * Ci * Co;
    ImgAddr in; in.base = c->obs; in.idx = idx; in.stride_b = c->img_elems * V; in.stride_v = c->img_elems; in.V = V;
    int rc;
    if (l == 1 && c->f01_train) {
      rc = launch_conv01_wgrad(c, in, dy, nimg, acc);
      if (rc == 1) return fail(c, PPO_ESHAPE, "the second convolution's weight-gradient kernel does not cover the shapes it was chosen for");
    } else {
      rc = launch_conv_wgrad_tile(c, dy, xl, Co, nimg, c->g + c->convW[l], c->g + c->convB[l], acc, "conv_wgrad." + std::to_string(l), wab);
      if (rc == PPO_OK + 1)
        rc = launch_wgrad(c, dl, xl, Co, 9 * Ci, dl.M, c->g + c->convW[l], c->g + c->convB[l], acc, "conv_wgrad." + std::to_string(l), wab);
    }
    if (rc) return rc;
    // transposed convolution over horizontal pixel pairs, both row parities in one launch (grid.z)
    AConvDgrad al; al.dy = dy; al.Ho = Ho; al.Wo = Wo; al.Cout = Co; al.lco = ilog2(Co); al.H = H; al.W = W; al.dy_imgs = nimg;
    al.w0 = c->wd[l][0]; al.w1 = c->wd[l][1];
    const int M0 = nimg * class_len(H, 0) * class_len(W, 0);  // the even-row parity sizes the grid
    ImgAddr xa = conv_out_addr(c, l - 1, c->act[l - 1], nullptr);
    Ep<MapDgrad, bf16_t, false, false, true> ep;
    ep.map.stride_b = xa.stride_b; ep.map.stride_v = xa.stride_v; ep.map.V = V; ep.map.H = H; ep.map.W = W; ep.map.Cin = Ci; ep.map.imgs = nimg;
    ep.out = c->gbuf[cur ^ 1]; ep.bias = nullptr; ep.mask = xa.base; ep.N = 2 * Ci;
    const bool dense_in = xa.stride_v == (int64_t)H * W * Ci && xa.stride_b == (int64_t)V * H * W * Ci;
    if (c->abits_ok[l - 1] && Ci % 32 == 0 && dense_in) ep.mbits = c->abits[l - 1];  // bit index = element offset of the dense activation
    const double pix = (double)nimg * H * W;
    const int N2 = 2 * Ci, BNf = N2 > 64 ? 128 : (N2 > 32 ? 64 : 32);
    const size_t wlds = (size_t)6 * Co * BNf * sizeof(bf16_t);  // both parities' packed weights, resident in LDS
    if (l == 1 && wlds <= 56 * 1024) {
      // fused with the first layer's weight gradient: its input gradient never leaves the chip
      in.prepare(); al.prepare(); ep.map.prepare();
      const int K0 = 9 * c->cC[0], npair = Ci * (K0 + 1), tpp = cdiv(M0, 128);
      int grid = 2 * tpp < 512 ? 2 * tpp : 512;
      { const int erc = ensure_partial(c, (int64_t)grid * npair, 0); if (erc) return erc; }
      if ((int64_t)grid * npair > c->partial_elems) grid = (int)(c->partial_elems / npair);
      const double fflops = 2.0 * (double)nimg * Ho * Wo * 9.0 * Ci * Co + 2.0 * pix * Ci * (K0 + 1);
      // the ReLU mask is one bit per element when the forward kernel left its sign-bit words, else the stored activation
      const double fbytes = 2.0 * ((double)nimg * Ho * Wo * Co + (double)nimg * c->img_elems + 9.0 * Ci * Co) + (c->abits_ok[l - 1] ? pix * Ci / 8.0 : 2.0 * pix * Ci);
      int tgrid = 0;
      rc = launch_conv_dgrad_wgrad0_tile(c, dy, xa, c->abits_ok[l - 1] ? c->abits[l - 1] : nullptr, c->wtap[l], Co, Ci, H, W, Ho, Wo, in, c->cC[0], c->cH[0], c->cW[0], nimg,
                                         "conv_dgrad.1+wgrad.0", fflops, fbytes, &tgrid);
      if (rc == PPO_OK) grid = tgrid;
      else if (rc != PPO_OK + 1) return rc;
      else if (c->f01_train) return fail(c, PPO_ESHAPE, "the second convolution's input-gradient kernel does not cover the shapes it was chosen for");  // (its mask is nowhere else)
      else {
        rc = ensure_packed_dgrad_weights(c, l);
        if (rc) return rc;
        ProfScope ps(c, "conv_dgrad.1+wgrad.0", 2.0 * (double)nimg * Ho * Wo * 9.0 * Ci * Co + 2.0 * pix * Ci * (K0 + 1),
                     2.0 * ((double)nimg * Ho * Wo * Co + pix * Ci + (double)nimg * c->img_elems + 9.0 * Ci * Co));
#define LAUNCH_FUSED(BN_, WM_, WN_, CI0_)                                                                                                  \
        do {                                                                                                                                 \
          auto kfn = k_dgrad1_wgrad0<BN_, WM_, WN_, CI0_>;                                                                                   \
          HIPCHK(c, hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)wlds));                            \
          hipLaunchKernelGGL(kfn, dim3(grid), dim3(256), wlds, c->stream, al, ep.map, xa.base, in, c->cH[0], c->cW[0], tpp, c->partial);      \
        } while (0)
        if (c->cC[0] == 1) {
          if (BNf == 128) LAUNCH_FUSED(128, 2, 2, 1); else if (BNf == 64) LAUNCH_FUSED(64, 2, 2, 1); else LAUNCH_FUSED(32, 4, 1, 1);
        } else {
          if (BNf == 128) LAUNCH_FUSED(128, 2, 2, 3); else if (BNf == 64) LAUNCH_FUSED(64, 2, 2, 3); else LAUNCH_FUSED(32, 4, 1, 3);
        }
#undef LAUNCH_FUSED
        LAUNCHCHK(c, "k_dgrad1_wgrad0");
      }
      defer_reduce(c, 2, grid, npair, Ci, K0, c->g + c->convW[0], c->g + c->convB[0], acc, false, 0, nullptr);
      return flush_reduces(c);
    }
    double ab = 2.0 * ((double)nimg * Ho * Wo * Co + pix * Ci + 9.0 * Ci * Co) + (c->abits_ok[l - 1] && (Co == 64 || ep.mbits) ? pix * Ci / 8.0 : 2.0 * pix * Ci);
    const double dflops = 2.0 * (double)nimg * Ho * Wo * 9.0 * Ci * Co;
    // From 128 channels: fp32 halves where the layer below reads rows that its forward cuts into columns (they hold the sum that
    // the implicit-GEMM form takes at once), else bf16 halves.
    int tr, nb;
    const bool f32 = l > 1 && !(c->cC[l - 1] == 32 ? plan_fwd_rows<32, 0>(c->cW[l - 1], H, W, &tr, &nb) : plan_fwd_rows<64, 0>(c->cW[l - 1], H, W, &tr, &nb));
    rc = !c->abits_ok[l - 1] ? 1 : launch_conv_dgrad_tile(c, dy, xa, c->abits[l - 1], c->gbuf[cur ^ 1], c->wtap[l], Co, Ci, H, W, Ho, Wo, nimg, "conv_dgrad." + std::to_string(l), dflops, ab, f32);
    if (rc == PPO_OK + 1) {
      rc = ensure_packed_dgrad_weights(c, l);
      if (rc) return rc;
      rc = launch_gemm(c, al, M0, nullptr, 0, 2 * Ci, 4 * Co, ep, "conv_dgrad." + std::to_string(l), ab, 2, dflops);
    }
    if (rc) return rc;
    cur ^= 1;
  }
  {  // first convolution: weight and bias gradient only
    ImgAddr in; in.base = c->obs; in.idx = idx; in.stride_b = c->img_elems * V; in.stride_v = c->img_elems; in.V = V;
    const int rc = conv0_wgrad(c, in, c->gbuf[cur], nimg, acc);
    if (rc) return rc;
  }
  return flush_reduces(c);
}

int encoder_backward_generic(Ctx* c, const int32_t* idx, int n, bool acc, int cur);
int encoder_forward_generic(Ctx* c, const int32_t* idx, int n, int64_t first);

// Backward of a feed-forward chunk whose forward activations are in the workspaces and whose head gradient is
// in dhead.  Gradients land in c->g (overwritten, or added when `acc`).
int backward_chunk(Ctx* c, const int32_t* idx, int n, bool acc, bool with_head = true) {
  int cur = 0;
  const bool generic = c->ln || c->E > 0;
  int rc = trunk_backward(c, c->feat, c->feat_ld, c->E == 0, n, acc, with_head, &cur);
  if (rc) return rc;
  return generic ? encoder_backward_generic(c, idx, n, acc, cur) : encoder_backward_ff(c, idx, n, acc, cur);
}

// ---------------------------------------------------------------- encoder with layer normalisation and / or embedding
// The LDS-image kernels where they cover a layer, else the implicit-GEMM ones; with layer_norm without the ReLU: the
// convolution's output is stored (pre), normalised per image and rectified by k_ln_fwd; without it the ReLU stays in the
// convolution's epilogue.  The last layer's activation goes into the feature matrix, or (embed_dim > 0) into a
// buffer of its own that the embedding GEMM reads, view by view.
static ImgAddrW as_w(const ImgAddr& a) { ImgAddrW w; w.base = const_cast<bf16_t*>(a.base); w.stride_b = a.stride_b; w.stride_v = a.stride_v; w.V = a.V; return w; }
static ImgAddr contiguous_imgs(const bf16_t* base, int64_t e, int V) { ImgAddr a; a.base = base; a.idx = nullptr; a.stride_b = e * V; a.stride_v = e; a.V = V; return a; }
// where the output activation of conv layer l lives for a chunk
static ImgAddr act_addr(Ctx* c, int l) {
  const int64_t e = (int64_t)c->cC[l + 1] * c->cH[l + 1] * c->cW[l + 1];
  if (l == c->nconv - 1 && c->E == 0) { ImgAddr a; a.base = c->feat; a.idx = nullptr; a.stride_b = c->feat_ld; a.stride_v = c->flat; a.V = c->V; return a; }
  return contiguous_imgs(c->act[l], e, c->V);
}

// First layer and its normalisation in one kernel per direction (ln0_tile.hip.h): 16 channels behind a one-channel image that a
// block's registers hold (4864 output pixels).
bool ln0_covers(const Ctx* c) { return c->ln && c->cC[0] == 1 && c->cC[1] == 16 && Ln0Shape::covers(c->cH[0], c->cW[0], c->cH[1]); }
Ln0Args ln0_args(Ctx* c, const ImgAddr& in, int nimg) {
  Ln0Args a = {};
  a.in = in; a.in.prepare(); a.w = c->shadow + c->convW[0]; a.bias = c->p + c->convB[0]; a.gain = c->p + c->lnG[0]; a.shift = c->p + c->lnB[0]; a.nimg = nimg;
  a.H = c->cH[0]; a.W = c->cW[0]; a.Ho = c->cH[1]; a.Wo = c->cW[1]; a.w4 = make_fastdiv(a.W / 8); a.stats = c->lnstat[0];
  return a;
}
template <bool BWD>
int launch_ln0(Ctx* c, const Ln0Args& a, int grid) {
  const int lds = Ln0Shape::lds_bytes(a.Ho, a.W, BWD), nt = cdiv(Ln0Shape::tiles(a.Ho, a.W), Ln0Shape::NW);
  const int f = (nt <= 10 ? 0 : nt <= 20 ? 1 : 2) + (2 * a.Wo == a.W ? 0 : 3);
  static decltype(&k_conv0_ln_fwd<10, false>) const fwd[6] = {k_conv0_ln_fwd<10, false>, k_conv0_ln_fwd<20, false>, k_conv0_ln_fwd<38, false>,
                                                              k_conv0_ln_fwd<10, true>, k_conv0_ln_fwd<20, true>, k_conv0_ln_fwd<38, true>};
  static decltype(&k_conv0_ln_fwd<10, false>) const bwd[6] = {k_conv0_ln_bwd<10, false>, k_conv0_ln_bwd<20, false>, k_conv0_ln_bwd<38, false>,
                                                              k_conv0_ln_bwd<10, true>, k_conv0_ln_bwd<20, true>, k_conv0_ln_bwd<38, true>};
  auto kfn = BWD ? bwd[f] : fwd[f];
  static uint64_t attr_devs[6] = {};  /* bit d: set on device d */
  if (!((attr_devs[f] >> c->dev) & 1)) { HIPCHK(c, hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024)); attr_devs[f] |= 1ull << c->dev; }
  hipLaunchKernelGGL(kfn, dim3(grid), dim3(Ln0Shape::THREADS), lds, c->stream, a);
  LAUNCHCHK(c, BWD ? "k_conv0_ln_bwd" : "k_conv0_ln_fwd");
  return PPO_OK;
}

int encoder_forward_generic(Ctx* c, const int32_t* idx, int n, int64_t first) {
  const int V = c->V, nimg = n * V;
  bool proprio_done = false;
  if (idx) first = 0;
  for (int l = 0; l < c->nconv; ++l) {
    bool have_bits = false;
    const int Co = c->cC[l + 1], Ho = c->cH[l + 1], Wo = c->cW[l + 1], Ci = c->cC[l];
    const int64_t e = (int64_t)Co * Ho * Wo, M = (int64_t)nimg * Ho * Wo;
    const ImgAddr oa = act_addr(c, l);
    const ImgAddr conv_to = c->ln ? contiguous_imgs(c->pre[l], e, V) : oa;
    const std::string name = "conv_fwd." + std::to_string(l);
    if (l == 0 && ln0_covers(c)) {
      ImgAddr in; in.base = c->obs + first * c->img_elems * V; in.idx = idx; in.stride_b = c->img_elems * V; in.stride_v = c->img_elems; in.V = V;
      Ln0Args a = ln0_args(c, in, nimg);
      a.out = as_w(oa); a.P = c->P; a.proprio = c->proprio + first * c->P; a.feat = c->feat + V * c->enc; a.feat_ld = c->feat_ld;
      ProfScope ps(c, "conv_fwd.0+layer_norm", 2.0 * (double)M * Co * 9 + 8.0 * (double)nimg * e, 2.0 * ((double)nimg * c->img_elems + (double)M * Co));
      const int rc = launch_ln0<false>(c, a, std::min(nimg, 256));
      if (rc) return rc;
      proprio_done = true;
      c->abits_ok[0] = false;
      continue;
    }
    if (l == 0) {
      ImgAddr in; in.base = c->obs + first * c->img_elems * V; in.idx = idx; in.stride_b = c->img_elems * V; in.stride_v = c->img_elems; in.V = V;
      in.prepare();
      if (conv_to.stride_v != e || conv_to.stride_b != e * V) return fail(c, PPO_ESHAPE, "the first convolution needs a contiguous output (n_conv >= 2 or an embedding)");
      ProfScope ps(c, name, 2.0 * (double)M * Co * 9 * Ci, 2.0 * ((double)nimg * c->img_elems + (double)M * Co));
      bf16_t* out = const_cast<bf16_t*>(conv_to.base);
      const bf16_t* w = c->shadow + c->convW[0];
      const float* b = c->p + c->convB[0];
      Conv0Args ca;
      ca.in = in; ca.out = out; ca.w = w; ca.bias = b; ca.zpage = c->zpage; ca.bits = !c->ln && c->nconv > 1 ? c->abits[0] : nullptr;
      ca.H = c->cH[0]; ca.W = c->cW[0]; ca.Ho = Ho; ca.Wo = Wo; ca.Cout = Co; ca.TR = 0; ca.NB = 0; ca.ntiles = 0;
      ca.tile_blocks = 0; ca.gather_blocks = 1; ca.pB = n; ca.P = c->P; ca.pcol0 = V * c->enc; ca.proprio = c->proprio + first * c->P; ca.feat = c->feat; ca.feat_ld = c->feat_ld;
      const int trc = c->ln ? (Ci == 1 ? launch_conv0_fwd_tile_t<1, false>(c, ca, nimg) : launch_conv0_fwd_tile_t<3, false>(c, ca, nimg))
                            : (Ci == 1 ? launch_conv0_fwd_tile_t<1>(c, ca, nimg) : launch_conv0_fwd_tile_t<3>(c, ca, nimg));
      if (trc != PPO_OK && trc != 1) return trc;
      proprio_done = trc == PPO_OK;
      have_bits = trc == PPO_OK && ca.bits;
      if (trc == 1) {
        constexpr int TPW = 4;
        const int grid = cdiv(M, 32 * 4 * TPW);
#define LAUNCH_C1(CIN_, RELU_) hipLaunchKernelGGL((k_conv1_fwd<CIN_, TPW, RELU_>), dim3(grid), dim3(256), 0, c->stream, in, nimg, c->cH[0], c->cW[0], Ho, Wo, Co, w, b, out)
        if (Ci == 1) { if (c->ln) LAUNCH_C1(1, false); else LAUNCH_C1(1, true); }
        else { if (c->ln) LAUNCH_C1(3, false); else LAUNCH_C1(3, true); }
#undef LAUNCH_C1
      }
      LAUNCHCHK(c, "k_conv1_fwd");
    } else {
      AConvFwd al;
      al.in = act_addr(c, l - 1);
      al.H = c->cH[l]; al.W = c->cW[l]; al.Cin = Ci; al.lc = ilog2(Ci); al.Ho = Ho; al.Wo = Wo; al.M = (int)M; al.K = 9 * Ci;
      const double ab = 2.0 * ((double)nimg * al.H * al.W * Ci + (double)M * Co + (double)al.K * Co);
      uint32_t* const bits = !c->ln && l < c->nconv - 1 ? c->abits[l] : nullptr;
      int rc = launch_conv_fwd_tile(c, al, conv_to, Co, c->shadow + c->convW[l], c->p + c->convB[l], nimg, name, ab, bits, !c->ln);
      have_bits = rc == PPO_OK && bits;
      if (rc != 1) {
      } else if (c->ln) {
        Ep<MapRows, bf16_t, true, false, false> ep;
        ep.map.stride_b = conv_to.stride_b; ep.map.stride_v = conv_to.stride_v; ep.map.V = V; ep.map.HW = Ho * Wo; ep.map.C = Co; ep.map.M = (int)M;
        ep.out = const_cast<bf16_t*>(conv_to.base); ep.bias = c->p + c->convB[l]; ep.mask = nullptr; ep.N = Co;
        rc = launch_gemm(c, al, (int)M, c->shadow + c->convW[l], al.K, Co, al.K, ep, name, ab);
      } else {
        Ep<MapRows, bf16_t, true, true, false> ep;
        ep.map.stride_b = conv_to.stride_b; ep.map.stride_v = conv_to.stride_v; ep.map.V = V; ep.map.HW = Ho * Wo; ep.map.C = Co; ep.map.M = (int)M;
        ep.out = const_cast<bf16_t*>(conv_to.base); ep.bias = c->p + c->convB[l]; ep.mask = nullptr; ep.N = Co;
        rc = launch_gemm(c, al, (int)M, c->shadow + c->convW[l], al.K, Co, al.K, ep, name, ab);
      }
      if (rc) return rc;
    }
    c->abits_ok[l] = have_bits;
    if (c->ln) {
      ProfScope ps(c, "layer_norm_fwd", 8.0 * (double)nimg * e, 4.0 * (double)nimg * e);
      // an image that fits one block's registers is read once
      const int64_t pch = cdiv(e / 8, LN_RTHREADS);  // 16-byte chunks per thread
      if (pch <= 2 && Co <= 512) hipLaunchKernelGGL(k_ln_fwd_reg<2>, dim3(nimg), dim3(LN_RTHREADS), 0, c->stream, c->pre[l], (int)e, Co, c->p + c->lnG[l], c->p + c->lnB[l], as_w(oa), c->lnstat[l]);
      else if (pch <= 5 && Co <= 512) hipLaunchKernelGGL(k_ln_fwd_reg<5>, dim3(nimg), dim3(LN_RTHREADS), 0, c->stream, c->pre[l], (int)e, Co, c->p + c->lnG[l], c->p + c->lnB[l], as_w(oa), c->lnstat[l]);
      else if (pch <= 10 && Co <= 512) hipLaunchKernelGGL(k_ln_fwd_reg<10>, dim3(nimg), dim3(LN_RTHREADS), 0, c->stream, c->pre[l], (int)e, Co, c->p + c->lnG[l], c->p + c->lnB[l], as_w(oa), c->lnstat[l]);
      else
      hipLaunchKernelGGL(k_ln_fwd, dim3(nimg), dim3(LN_THREADS), 0, c->stream, c->pre[l], (int)e, Co, c->p + c->lnG[l], c->p + c->lnB[l], as_w(oa), c->lnstat[l]);
      LAUNCHCHK(c, "k_ln_fwd");
    }
  }
  if (c->E > 0) {  // embedding of each view's flattened features: a linear layer, no activation
    for (int v = 0; v < V; ++v) {
      ARows al = plain_arows(c->act[c->nconv - 1] + (int64_t)v * c->flat, (int64_t)V * c->flat, n, c->flat);
      Ep<MapRows, bf16_t, true, false, false> ep;
      ep.map = plain_map(c->feat_ld, n); ep.out = c->feat + (int64_t)v * c->E; ep.bias = c->p + c->embB; ep.mask = nullptr; ep.N = c->E;
      const int rc = launch_gemm(c, al, n, c->shadow + c->embW, c->flat, c->E, c->flat, ep, "embed_fwd", 2.0 * ((double)n * c->flat + (double)n * c->E + (double)c->flat * c->E));
      if (rc) return rc;
    }
  }
  if (!proprio_done) {
    hipLaunchKernelGGL(k_gather_proprio, dim3(cdiv((int64_t)n * c->P, 256)), dim3(256), 0, c->stream, c->proprio + first * c->P, idx, n, c->P, c->feat,
                       (int64_t)c->feat_ld, V * c->enc);
    LAUNCHCHK(c, "k_gather_proprio");
  }
  return PPO_OK;
}

// Layer-normalisation backward in registers by the number of 16-byte chunks per thread.  A form for every number: one
// made for more chunks than the image has spends the others' instructions and registers on zeros (two layers, 2048
// images, the first of 4096 values per chunk, us: 1 chunk 58, in a form for three 79, read twice 63; 6 chunks 106, in a
// form for ten 156, read twice 127; 11 chunks 180, in a form for nineteen 219, read twice 200).
template <int... N>
decltype(&k_ln_bwd) ln_bwd_reg(int chunks, std::integer_sequence<int, N...>) {
  static const decltype(&k_ln_bwd) form[] = {k_ln_bwd_reg<N + 1>...};
  return form[chunks - 1];
}

// Its backward from d(features) in `dfeat` (row stride ld_df; with an embedding its columns [v*E, (v+1)*E) are the
// gradient of view v's embedding, without one the masked gradient of the last convolution's activation).
int encoder_backward_seq(Ctx* c, const int32_t* idx, int n, bool acc, const bf16_t* dfeat, int64_t ld_df, int cur) {
  const int V = c->V, nimg = n * V, L = c->nconv;
  // gradient w.r.t. the last convolution's activation, masked by its ReLU
  ImgAddr dy;
  if (c->E > 0) {
    bf16_t* dst = c->gbuf[cur ^ 1];
    for (int v = 0; v < V; ++v) {
      ARows dl = plain_arows(dfeat + (int64_t)v * c->E, ld_df, n, c->E);
      ARows xl = plain_arows(c->act[L - 1] + (int64_t)v * c->flat, (int64_t)V * c->flat, n, c->flat);
      int rc = launch_wgrad(c, dl, xl, c->E, c->flat, n, c->g + c->embW, c->g + c->embB, acc || v > 0, "embed_wgrad", 2.0 * n * ((double)c->flat + c->E));
      if (rc) return rc;
      Ep<MapRows, bf16_t, false, false, true> ep;
      ep.map = plain_map((int64_t)V * c->flat, n); ep.out = dst + (int64_t)v * c->flat; ep.bias = nullptr; ep.mask = c->act[L - 1] + (int64_t)v * c->flat; ep.N = c->flat;
      rc = launch_gemm(c, dl, n, c->embT, c->E, c->flat, c->E, ep, "embed_dgrad", 2.0 * n * (2.0 * c->flat + c->E));
      if (rc) return rc;
    }
    cur ^= 1;
    dy = contiguous_imgs(c->gbuf[cur], c->flat, V);
  } else {
    if (c->nl > 0 && !c->ln) {  // the LSTM's GEMM left this gradient unmasked, and no layer-norm backward will mask it
      hipLaunchKernelGGL(k_mask_rows, dim3(cdiv((int64_t)n * (V * c->flat / 8), 256)), dim3(256), 0, c->stream, (int64_t)n, V * c->flat, const_cast<bf16_t*>(dfeat), ld_df,
                         c->feat, (int64_t)c->feat_ld);
      LAUNCHCHK(c, "k_mask_rows");
    }
    dy.base = dfeat; dy.idx = nullptr; dy.stride_b = ld_df; dy.stride_v = c->flat; dy.V = V;
  }
  for (int l = L - 1; l >= 0; --l) {
    const int Co = c->cC[l + 1], Ci = c->cC[l], Ho = c->cH[l + 1], Wo = c->cW[l + 1], H = c->cH[l], W = c->cW[l];
    const int64_t e = (int64_t)Co * Ho * Wo;
    ImgAddr dconv = dy;  // gradient w.r.t. the convolution's output
    if (l == 0 && ln0_covers(c)) {
      ImgAddr in; in.base = c->obs; in.idx = idx; in.stride_b = c->img_elems * V; in.stride_v = c->img_elems; in.V = V;
      Ln0Args a = ln0_args(c, in, nimg);
      a.dy = dy; a.dy.prepare();
      int grid = std::min(nimg, 256);
      { const int erc = ensure_partial(c, (int64_t)grid * 192, 0); if (erc) return erc; }
      grid = (int)std::min<int64_t>(grid, c->partial_elems / 192);
      if (grid < 1) return fail(c, PPO_ENOMEM, "weight-gradient workspace too small for the first convolution");
      a.part_ln = c->partial; a.part_w = c->partial + (int64_t)grid * 32;
      {
        ProfScope ps(c, "layer_norm_bwd+conv_wgrad.0", 2.0 * (double)nimg * Ho * Wo * 16 * 19 + 14.0 * (double)nimg * e, 2.0 * ((double)nimg * c->img_elems + (double)nimg * e));
        const int rc = launch_ln0<true>(c, a, grid);
        if (rc) return rc;
      }
      defer_reduce(c, 0, grid, 32, 0, 0, c->g + c->lnG[0], nullptr, acc, false, 0, nullptr);
      defer_reduce(c, 2, grid, 160, 16, 9, c->g + c->convW[0], c->g + c->convB[0], acc, false, 0, nullptr);
      break;
    }
    if (c->ln) {
      int grid = nimg < 1024 ? nimg : 1024;
      { const int erc = ensure_partial(c, (int64_t)grid * 2 * Co, 0); if (erc) return erc; }
      if ((int64_t)grid * 2 * Co > c->partial_elems) grid = (int)(c->partial_elems / (2 * Co));
      if (grid < 1) return fail(c, PPO_ENOMEM, "weight-gradient workspace too small for the layer-norm gradients");
      {
        ProfScope ps(c, "layer_norm_bwd", 14.0 * (double)nimg * e, 6.0 * (double)nimg * e);
        dy.prepare();
        // an image whose input and gradient fit one block's registers is read once
        const int64_t pch = cdiv(e / 8, LN_THREADS);  // 16-byte chunks per thread
        const bool rows16 = dy.stride_b % 8 == 0 && dy.stride_v % 8 == 0;
        auto kfn = rows16 && pch <= LN_BWD_CHUNKS ? ln_bwd_reg((int)pch, std::make_integer_sequence<int, LN_BWD_CHUNKS>()) : k_ln_bwd;
        hipLaunchKernelGGL(kfn, dim3(grid), dim3(LN_THREADS), 0, c->stream, dy, c->pre[l], c->lnstat[l], nimg, (int)e, Co, c->p + c->lnG[l], c->p + c->lnB[l], c->dpre, c->partial);
        LAUNCHCHK(c, "k_ln_bwd");
      }
      defer_reduce(c, 0, grid, 2 * Co, 0, 0, c->g + c->lnG[l], nullptr, acc, false, 0, nullptr);  // gain and shift gradients are adjacent
      dconv = contiguous_imgs(c->dpre, e, V);
    }
    if (l == 0) {
      ImgAddr in; in.base = c->obs; in.idx = idx; in.stride_b = c->img_elems * V; in.stride_v = c->img_elems; in.V = V;
      if (dconv.stride_v != e || dconv.stride_b != e * V) return fail(c, PPO_ESHAPE, "the first convolution's gradient needs a contiguous layout");
      const int rc = conv0_wgrad(c, in, dconv.base, nimg, acc);
      if (rc) return rc;
      break;
    }
    ARows dl; dl.a = dconv; dl.HW = Ho * Wo; dl.C = Co; dl.M = nimg * Ho * Wo; dl.K = Co; dl.plain = false;
    AConvFwd xl; xl.in = act_addr(c, l - 1);
    xl.H = H; xl.W = W; xl.Cin = Ci; xl.lc = ilog2(Ci); xl.Ho = Ho; xl.Wo = Wo; xl.M = dl.M; xl.K = 9 * Ci;
    const double wab = 2.0 * ((double)dl.M * Co + (double)nimg * H * W * Ci) + 4.0 * 9.0 * Ci * Co;
    int rc = launch_conv_wgrad_tile(c, dconv, xl, Co, nimg, c->g + c->convW[l], c->g + c->convB[l], acc, "conv_wgrad." + std::to_string(l), wab);
    if (rc == 1) rc = launch_wgrad(c, dl, xl, Co, 9 * Ci, dl.M, c->g + c->convW[l], c->g + c->convB[l], acc, "conv_wgrad." + std::to_string(l), wab);
    if (rc) return rc;
    const double pix = (double)nimg * H * W, dflops = 2.0 * (double)nimg * Ho * Wo * 9.0 * Ci * Co;
    const double dab = 2.0 * ((double)nimg * Ho * Wo * Co + pix * Ci + 9.0 * Ci * Co);
    const ImgAddr xa = act_addr(c, l - 1);
    // with layer normalisation the gradient may stay unmasked: k_ln_bwd applies the ReLU itself
    const uint32_t* const xbits = c->ln ? nullptr : c->abits[l - 1];
    if (c->ln || c->abits_ok[l - 1]) {
      rc = launch_conv_dgrad_tile(c, dconv, xa, xbits, c->gbuf[cur ^ 1], c->wtap[l], Co, Ci, H, W, Ho, Wo, nimg, "conv_dgrad." + std::to_string(l), dflops,
                                  dab + (xbits ? pix * Ci / 8.0 : 0.0), true);
      if (rc != PPO_OK && rc != 1) return rc;
      if (rc == PPO_OK) {
        cur ^= 1;
        dy = contiguous_imgs(c->gbuf[cur], (int64_t)Ci * H * W, V);
        continue;
      }
    }
    AConvDgrad al; al.dy = dconv; al.Ho = Ho; al.Wo = Wo; al.Cout = Co; al.lco = ilog2(Co); al.H = H; al.W = W; al.dy_imgs = nimg;
    rc = ensure_packed_dgrad_weights(c, l);
    if (rc) return rc;
    al.w0 = c->wd[l][0]; al.w1 = c->wd[l][1];
    const int M0 = nimg * class_len(H, 0) * class_len(W, 0);
    auto gemm = [&](auto ep) {
      ep.map.stride_b = xa.stride_b; ep.map.stride_v = xa.stride_v; ep.map.V = V; ep.map.H = H; ep.map.W = W; ep.map.Cin = Ci; ep.map.imgs = nimg;
      ep.out = c->gbuf[cur ^ 1]; ep.bias = nullptr; ep.mask = xa.base; ep.N = 2 * Ci;
      const bool dense_in = xa.stride_v == (int64_t)H * W * Ci && xa.stride_b == (int64_t)V * H * W * Ci;
      if (c->abits_ok[l - 1] && Ci % 32 == 0 && dense_in) ep.mbits = c->abits[l - 1];  // bit index = element offset of the dense activation
      return launch_gemm(c, al, M0, nullptr, 0, 2 * Ci, 4 * Co, ep, "conv_dgrad." + std::to_string(l), dab + (c->ln ? 0.0 : 2.0 * pix * Ci), 2, dflops);
    };
    rc = c->ln ? gemm(Ep<MapDgrad, bf16_t, false, false, false, true>()) : gemm(Ep<MapDgrad, bf16_t, false, false, true>());
    if (rc) return rc;
    cur ^= 1;
    dy = contiguous_imgs(c->gbuf[cur], (int64_t)Ci * H * W, V);
  }
  return flush_reduces(c);
}
int encoder_backward_generic(Ctx* c, const int32_t* idx, int n, bool acc, int cur) {
  return encoder_backward_seq(c, idx, n, acc, c->gbuf[cur], c->fin[0], cur);
}

// ---------------------------------------------------------------- recurrent core
// The layers' steps side by side (recurrent.hip.h): needs units in multiples of 32.
bool lstm_side_by_side(const Ctx* c) { return c->H % 32 == 0; }
int64_t lstm_tiled_rows(const Ctx* c, int ne) { return (int64_t)cdiv(ne, 32) * 32; }  // rows of one step in the tiled arrays

struct LstmProducts {
  ARowsSet al;
  EpSplit ep;
  int n = 0;
  void add(const bf16_t* a, int64_t lda, int M, const bf16_t* w, int N, int K) {
    al.a[n] = a; al.lda[n] = lda; al.w[n] = w; al.M[n] = M; al.K[n] = K; ep.N[n] = N;
    ++n;
  }
};
// All products of an iteration in one launch.  Slices of one length W for all of them, so that the blocks finish
// together: the W with the smallest sum of k-steps per round of 256 blocks (lengths as in plan_gemm) and of the slices'
// way through memory (written and read once, 6 TB/s).
template <int BM, int BN>
int launch_lstm_products(Ctx* c, LstmProducts& P, LstmPart (&out)[EpSplit::MAXP], const std::string& name) {
  constexpr int nst = BM == 64 ? 8 : 4, lds = nst * (BM + BN) * 128;
  const double step = BM == 64 ? 0.34 : 0.60;  // us per k-step, as in plan_gemm
  int nk[EpSplit::MAXP], kmax = 0;
  double flops = 0.0, bytes = 0.0;
  for (int i = 0; i < P.n; ++i) {
    P.ep.gy[i] = cdiv(P.ep.N[i], BN); P.ep.tiles[i] = cdiv(P.al.M[i], BM) * P.ep.gy[i]; nk[i] = cdiv(P.al.K[i], 64);
    if (nk[i] > kmax) kmax = nk[i];
    flops += 2.0 * P.al.M[i] * (double)P.ep.N[i] * P.al.K[i];
    bytes += 2.0 * ((double)P.al.M[i] * P.al.K[i] + (double)P.ep.N[i] * P.al.K[i]);
  }
  int W = kmax;
  double tbest = 1e30;
  for (int w = kmax; w >= 3 || w == kmax; --w) {
    int64_t blocks = 0;
    for (int i = 0; i < P.n; ++i) blocks += (int64_t)P.ep.tiles[i] * cdiv(nk[i], w);
    if (w < kmax && blocks > 512) break;   // (what lstm_part holds)
    const double t = step * w * cdiv(blocks, 256) + 8e-6 * (double)blocks * BM * BN / 6.0;
    if (t < tbest - 1e-9) { tbest = t; W = w; }
  }
  int gx = 0;
  float* part = c->lstm_part;
  for (int i = 0; i < P.n; ++i) {
    P.ep.W[i] = W;
    const int splits = cdiv(nk[i], W);
    P.ep.blocks[i] = P.ep.tiles[i] * splits; P.ep.part[i] = part;
    out[i].part = reinterpret_cast<const float4*>(part); out[i].splits = splits; out[i].tiles = P.ep.tiles[i]; out[i].gy = P.ep.gy[i];
    part += (int64_t)P.ep.blocks[i] * BM * BN;
    if (P.ep.blocks[i] > gx) gx = P.ep.blocks[i];
  }
  P.ep.map = plain_map(0, 0);
  gx = (gx + 7) / 8 * 8;
  auto kfn = k_gemm_rs<BM, BN, 2, 2, nst, ARowsSet, EpSplit>;
  static uint64_t attr_devs = 0;  /* bit d: set on device d */
  if (!((attr_devs >> c->dev) & 1)) { HIPCHK(c, hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, lds)); attr_devs |= 1ull << c->dev; }
  ProfScope ps(c, name, flops, bytes);
  hipLaunchKernelGGL(kfn, dim3(gx, 1, P.n), dim3(512), lds, c->stream, P.al, (const bf16_t*)nullptr, (int64_t)0, 0, P.ep, c->zpage);
  LAUNCHCHK(c, "lstm products");
  return PPO_OK;
}
// room of lstm_part: the undivided tiles of every layer's largest product, or 512 blocks of slices
int64_t lstm_part_elems(const Ctx* c) {
  auto blocks = [&](int bm, int bn) {
    int64_t t = 0;
    for (int l = 0; l < c->nl; ++l) t += (int64_t)cdiv(c->CHe, bm) * std::max(cdiv(4 * c->H, bn), cdiv(c->lin[l] + c->H, bn));
    return std::max<int64_t>(t, 512) * bm * bn;
  };
  return std::max(blocks(64, 64), blocks(128, 128));
}

template <int BM, int BN>
int lstm_forward_side_by_side(Ctx* c, int ne) {
  const int T = c->T, H = c->H, L = c->nl;
  const int64_t R = lstm_tiled_rows(c, ne);
  for (int s = 0; s < T + L - 1; ++s) {
    LstmProducts P;
    LstmFwdJobs J;
    LstmPart parts[EpSplit::MAXP];
    int lay[4];
    for (int l = 0; l < L; ++l) {
      const int t = s - l, K = c->lin[l] + H;
      if (t < 0 || t >= T) continue;
      lay[P.n] = l;
      P.add(c->xh[l] + (int64_t)t * ne * K, K, ne, c->shadow + c->lstmW[l], 4 * H, K);
    }
    int rc = launch_lstm_products<BM, BN>(c, P, parts, "lstm_fwd");
    if (rc) return rc;
    J.ne = ne; J.H = H; J.done = c->done;
    for (int i = 0; i < P.n; ++i) {
      const int l = lay[i], t = s - l, K = c->lin[l] + H;
      const bool last = t == T - 1, top = l == L - 1;
      const int64_t r0 = (int64_t)t * ne;
      auto& q = J.job[i];
      q.pre = parts[i]; q.bias = c->p + c->lstmB[l]; q.idx = c->seqidx + r0;
      q.c_enter = reinterpret_cast<const float4*>(c->c_enter[l] + t * R * H);
      q.c_next = last ? nullptr : reinterpret_cast<float4*>(c->c_enter[l] + (t + 1) * R * H);
      q.gates = reinterpret_cast<float4*>(c->gates[l] + t * R * 4 * H);
      q.ld_out = top ? H : c->lin[l + 1] + H; q.h_out = (top ? c->htop : c->xh[l + 1]) + r0 * q.ld_out;
      q.ld_next = K; q.h_next = last ? nullptr : c->xh[l] + (r0 + ne) * K + c->lin[l];
    }
    ProfScope ps(c, "lstm_cell_fwd", 30.0 * P.n * ne * H, (double)P.n * ne * H * 44.0);
    hipLaunchKernelGGL((k_lstm_cells_fwd<BM, BN>), dim3((int)(R / 32) * (H / 32), P.n), dim3(256), 0, c->stream, J);
    LAUNCHCHK(c, "k_lstm_cells_fwd");
  }
  return PPO_OK;
}

// dtop [T*ne][H]: gradient of the top layer's h.  Leaves every layer's gate gradients in da.
template <int BM, int BN>
int lstm_backward_side_by_side(Ctx* c, const bf16_t* dtop, int ne) {
  const int T = c->T, H = c->H, L = c->nl;
  const int64_t R = lstm_tiled_rows(c, ne);
  LstmPart parts[EpSplit::MAXP], prev[EpSplit::MAXP];
  bool have[4] = {false, false, false, false};   // layer l's product of the previous iteration is in prev[l]
  for (int s = 0; s < T + L - 1; ++s) {
    LstmBwdJobs J;
    int lay[4], nj = 0;
    J.ne = ne; J.H = H; J.done = c->done;
    for (int l = L - 1; l >= 0; --l) {
      const int t = T - 1 - (s - (L - 1 - l));
      if (t < 0 || t >= T) continue;
      const int64_t r0 = (int64_t)t * ne;
      auto& q = J.job[nj];
      lay[nj++] = l;
      q.above.part = nullptr; q.dh = nullptr; q.ld_dh = H; q.rec.part = nullptr; q.rec_col = l > 0 ? c->lin[l] : 0;
      if (l == L - 1) q.dh = dtop + r0 * H;
      else q.above = prev[l + 1];
      if (t < T - 1 && have[l]) q.rec = prev[l];
      q.idx = c->seqidx + r0;
      q.c_enter = reinterpret_cast<const float4*>(c->c_enter[l] + t * R * H);
      q.gates = reinterpret_cast<const float4*>(c->gates[l] + t * R * 4 * H);
      q.dc = reinterpret_cast<float4*>(c->dc_carry[l]);
      q.da = c->da[l] + r0 * 4 * H;
    }
    {
      ProfScope ps(c, "lstm_cell_bwd", 40.0 * nj * ne * H, (double)nj * ne * H * 40.0);
      hipLaunchKernelGGL((k_lstm_cells_bwd<BM, BN>), dim3((int)(R / 32) * (H / 32), nj), dim3(256), 0, c->stream, J);
      LAUNCHCHK(c, "k_lstm_cells_bwd");
    }
    // gate gradients -> gradient of the operand row: of the h half for the step before, and of the x half for the layer
    // below (the bottom layer's x half is one product over all steps afterwards; at step 0 nothing needs the h half)
    LstmProducts P;
    int pl[4];
    for (int i = 0; i < nj; ++i) {
      const int l = lay[i], t = T - 1 - (s - (L - 1 - l));
      have[l] = false;
      if (t == 0 && l == 0) continue;
      const int64_t skip = l > 0 ? 0 : (int64_t)c->lin[0] * 4 * H;
      pl[P.n] = l;
      P.add(c->da[l] + (int64_t)t * ne * 4 * H, 4 * H, ne, c->lstmWT[l] + skip, l > 0 ? c->lin[l] + H : H, 4 * H);
    }
    if (P.n == 0) continue;
    const int rc = launch_lstm_products<BM, BN>(c, P, parts, "lstm_dgrad");
    if (rc) return rc;
    for (int i = 0; i < P.n; ++i) { prev[pl[i]] = parts[i]; have[pl[i]] = true; }
  }
  return PPO_OK;
}

// Forward of a chunk of `ne` whole environments (device list env) x T steps, rows time-major.  Encoder on all
// ne*T rows at once, then the LSTM (products of the operand rows [x_t, h_enter] with [W_ih, W_hh] and cell kernels: the
// layers side by side, or, for units that are no multiple of 32, one layer and step after the other), then hidden layers
// and heads on all rows.
int forward_seq_chunk(Ctx* c, const int32_t* env, int ne, bool with_head) {
  const int T = c->T, n = ne * T, H = c->H;
  hipLaunchKernelGGL(k_seq_index, dim3(cdiv(n, 256)), dim3(256), 0, c->stream, env, ne, T, c->N, c->seqidx);
  LAUNCHCHK(c, "k_seq_index");
  int rc = (c->ln || c->E > 0) ? encoder_forward_generic(c, c->seqidx, n, 0) : encoder_forward_ff(c, c->seqidx, n, 0, true);
  if (rc) return rc;
  const bool side = lstm_side_by_side(c);
  for (int l = 0; l < c->nl; ++l) {
    hipLaunchKernelGGL(k_lstm_init, dim3(cdiv(ne * H, 256)), dim3(256), 0, c->stream, env, ne, H, c->h0 + (int64_t)l * c->N * H, c->c0 + (int64_t)l * c->N * H,
                       c->xh[l], (int64_t)(c->lin[l] + H), c->lin[l], c->c_enter[l], side ? 1 : 0);
    LAUNCHCHK(c, "k_lstm_init");
  }
  if (side) {
    rc = ne <= 64 ? lstm_forward_side_by_side<64, 64>(c, ne) : lstm_forward_side_by_side<128, 128>(c, ne);
    if (rc) return rc;
  }
  for (int l = 0; l < c->nl && !side; ++l) {
    const int K = c->lin[l] + H;
    const bool top = l == c->nl - 1;
    bf16_t* outm = top ? c->htop : c->xh[l + 1];
    const int64_t ld_out = top ? H : c->lin[l + 1] + H;
    for (int t = 0; t < T; ++t) {
      const int64_t r0 = (int64_t)t * ne;
      ARows al = plain_arows(c->xh[l] + r0 * K, K, ne, K);
      Ep<MapRows, float, true, false, false> ep;
      ep.map = plain_map(4 * H, ne); ep.out = c->lstm_pre; ep.bias = c->p + c->lstmB[l]; ep.mask = nullptr; ep.N = 4 * H;
      rc = launch_gemm(c, al, ne, c->shadow + c->lstmW[l], K, 4 * H, K, ep, "lstm_fwd." + std::to_string(l), 2.0 * ((double)ne * K + (double)K * 4 * H) + 16.0 * ne * H);
      if (rc) return rc;
      ProfScope ps(c, "lstm_cell_fwd", 30.0 * ne * H, (double)ne * H * (16.0 + 16.0 + 8.0 + 4.0));
      const bool last = t == T - 1;
      hipLaunchKernelGGL(k_lstm_cell_fwd, dim3(cdiv(ne * H, 256)), dim3(256), 0, c->stream, ne, H, c->lstm_pre, c->c_enter[l] + r0 * H, c->done, c->seqidx + r0,
                         c->gates[l] + r0 * 4 * H, outm + r0 * ld_out, ld_out, last ? nullptr : c->xh[l] + (r0 + ne) * K + c->lin[l], (int64_t)K,
                         last ? nullptr : c->c_enter[l] + (r0 + ne) * H);
      LAUNCHCHK(c, "k_lstm_cell_fwd");
    }
  }
  return trunk_forward(c, c->nl > 0 ? c->htop : c->feat, c->nl > 0 ? (int64_t)H : c->feat_ld, n, with_head);
}

// Its backward: heads and hidden layers on all rows, then back-propagation through time: per step the cells' backward
// and a product that turns the gate gradients into the gradient of the operand row [x_t, h_enter] - its h half is what
// step t-1 receives -, the layers side by side or (other units) one after the other, the top one first; a layer's weight
// gradient is one contraction over all rows afterwards.  Then the encoder's backward on all rows.
int backward_seq_chunk(Ctx* c, int ne, bool acc, bool with_head) {
  const int T = c->T, n = ne * T, H = c->H;
  int cur = 0;
  int rc = trunk_backward(c, c->htop, H, false, n, acc, with_head, &cur);
  if (rc) return rc;
  const bf16_t* dabove = c->gbuf[cur];
  int64_t ld_above = H;
  const bool side = lstm_side_by_side(c);
  if (side) {
    rc = ne <= 64 ? lstm_backward_side_by_side<64, 64>(c, dabove, ne) : lstm_backward_side_by_side<128, 128>(c, dabove, ne);
    if (rc) return rc;
    // the bottom layer's input gradient, all steps at once
    ARows dl = plain_arows(c->da[0], 4 * H, n, 4 * H);
    Ep<MapRows, bf16_t, false, false, false> ep;
    ep.map = plain_map(c->lin[0] + H, n); ep.out = c->dxh[0]; ep.bias = nullptr; ep.mask = nullptr; ep.N = c->lin[0];
    rc = launch_gemm(c, dl, n, c->lstmWT[0], 4 * H, c->lin[0], 4 * H, ep, "lstm_dgrad.x", 2.0 * ((double)n * 4 * H + (double)n * c->lin[0] + (double)c->lin[0] * 4 * H));
    if (rc) return rc;
  }
  for (int l = c->nl - 1; l >= 0; --l) {
    const int K = c->lin[l] + H;
    for (int t = T - 1; t >= 0 && !side; --t) {
      const int64_t r0 = (int64_t)t * ne;
      const bool last = t == T - 1;
      {
        ProfScope ps(c, "lstm_cell_bwd", 40.0 * ne * H, (double)ne * H * (16.0 + 4.0 + 4.0 + 8.0 + 8.0));
        hipLaunchKernelGGL(k_lstm_cell_bwd, dim3(cdiv(ne * H, 256)), dim3(256), 0, c->stream, ne, H, c->gates[l] + r0 * 4 * H, c->c_enter[l] + r0 * H, c->done,
                           c->seqidx + r0, dabove + r0 * ld_above, ld_above, last ? nullptr : c->dxh[l] + (r0 + ne) * K + c->lin[l], (int64_t)K, c->dc_carry[l],
                           last ? 1 : 0, c->da[l] + r0 * 4 * H);
        LAUNCHCHK(c, "k_lstm_cell_bwd");
      }
      ARows dl = plain_arows(c->da[l] + r0 * 4 * H, 4 * H, ne, 4 * H);
      Ep<MapRows, bf16_t, false, false, false> ep;
      ep.map = plain_map(K, ne); ep.out = c->dxh[l] + r0 * K; ep.bias = nullptr; ep.mask = nullptr; ep.N = K;
      rc = launch_gemm(c, dl, ne, c->lstmWT[l], 4 * H, K, 4 * H, ep, "lstm_dgrad." + std::to_string(l), 2.0 * ((double)ne * 4 * H + (double)ne * K + (double)K * 4 * H));
      if (rc) return rc;
    }
    ARows dl = plain_arows(c->da[l], 4 * H, n, 4 * H);
    ARows xl = plain_arows(c->xh[l], K, n, K);
    rc = launch_wgrad(c, dl, xl, 4 * H, K, n, c->g + c->lstmW[l], c->g + c->lstmB[l], acc, "lstm_wgrad." + std::to_string(l), 2.0 * n * ((double)K + 4 * H) + 4.0 * (double)K * 4 * H);
    if (rc) return rc;
    dabove = c->dxh[l]; ld_above = K;   // the x half of this layer's operand gradient is the layer below's dh
  }
  return encoder_backward_seq(c, c->seqidx, n, acc, c->dxh[0], c->lin[0] + H, cur);
}

// The one-launch form for up to PERM_SMALL units on the current device.
hipError_t launch_perm_small(const PermStreams& ps, int S, int count, int32_t* perm, hipStream_t stream) {
  const int nb = perm_small_buckets(S);
  int lg = 0;
  while ((1 << lg) < nb) ++lg;
  static std::once_flag once[STATIC_MAX_DEVICES];
  static hipError_t attr[STATIC_MAX_DEVICES];
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= STATIC_MAX_DEVICES) return hipErrorInvalidDevice;
  std::call_once(once[dev], [&]() { attr[dev] = hipFuncSetAttribute((const void*)k_perm_small, hipFuncAttributeMaxDynamicSharedMemorySize, perm_small_lds(PERM_SMALL, PERM_SMALL)); });
  if (attr[dev] != hipSuccess) return attr[dev];
  hipLaunchKernelGGL(k_perm_small, dim3(count), dim3(1024), perm_small_lds(S, nb), stream, ps, S, nb, 64 - lg, perm);
  return hipGetLastError();
}

// The permutations of epochs epoch0 .. epoch0 + count - 1 (count <= PERM_BATCH) of (seed, update) into the slots
// 0 .. count - 1 of c->perm ([PERM_BATCH][S]): one launch for few units, five otherwise, whatever the count.
int gen_permutations(Ctx* c, uint64_t seed, uint64_t update, uint64_t epoch0, int count) {
  PermStreams ps;
  for (int e = 0; e < PERM_BATCH; ++e) ps.s[e] = perm_stream(seed, update, epoch0 + (uint64_t)(e < count ? e : 0));
  const int S = c->PU, g = cdiv(S, 256), nb = c->nb;  // the units a minibatch is made of: samples, or whole environments
  ProfScope pscope(c, "permutation", 0.0, 4.0 * S * count);
  if (S <= PERM_SMALL) {
    HIPCHK(c, launch_perm_small(ps, S, count, c->perm, c->stream));
    return PPO_OK;
  }
  hipLaunchKernelGGL(k_fill_i32, dim3(cdiv((int64_t)count * 2 * nb, 256)), dim3(256), 0, c->stream, c->phist, (int64_t)count * 2 * nb, 0);  // hist + cursor
  hipLaunchKernelGGL(k_perm_hist, dim3(g, count), dim3(256), 0, c->stream, ps, S, c->shift, nb, c->phist);
  hipLaunchKernelGGL(k_perm_scan, dim3(1, count), dim3(1024), 0, c->stream, c->phist, c->pstart, nb);
  hipLaunchKernelGGL(k_perm_scatter, dim3(g, count), dim3(256), 0, c->stream, ps, S, c->shift, nb, c->pstart, c->phist, c->ptmp);
  hipLaunchKernelGGL(k_perm_rank, dim3(g, count), dim3(256), 0, c->stream, ps, S, c->shift, nb, c->pstart, c->phist, c->ptmp, c->perm);
  LAUNCHCHK(c, "permutation kernels");
  return PPO_OK;
}
int gen_permutation(Ctx* c, uint64_t seed, uint64_t update, uint64_t epoch) { return gen_permutations(c, seed, update, epoch, 1); }

// Output layer forward, loss and output layer backward of a chunk in one kernel (head_loss.hip.h);
// returns 1 when the width of the last hidden layer or the workspaces do not allow it.
template <int HID>
int launch_head_loss_t(Ctx* c, const LossData& L, int n, bool acc, bool distill, float* sp, float* dp) {
  typedef HeadLossShape<HID> S;
  const int nblk = cdiv(n, 64);
  { const int erc = ensure_partial(c, (int64_t)nblk * c->NH * HID, (int64_t)nblk * c->NH); if (erc) return erc; }
  if ((int64_t)nblk * c->NH * HID > c->partial_elems || (int64_t)nblk * c->NH > c->bias_partial_elems) return 1;
  HeadLossArgs a;
  a.h = c->fcact[c->nfc - 1]; a.w = c->shadow + c->headW; a.wt = c->headT; a.bias = c->p + c->headB; a.dh = c->gbuf[0];
  a.wpart = c->partial; a.bpart = c->bias_partial; a.stat_part = sp; a.dls_part = dp; a.n = n; a.NH = c->NH;
  {
    ProfScope ps(c, "head+loss", 6.0 * n * (double)HID * HEAD_LD, (double)n * (4.0 * HID + 4.0 * c->A + 20.0));
    static uint64_t attr_devs[2] = {0, 0};  // bit d: set on device d
    if (distill) {
      auto kfn = k_head_loss<HID, true>;
      if (!((attr_devs[1] >> c->dev) & 1)) { HIPCHK(c, hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, S::LDS_BYTES)); attr_devs[1] |= 1ull << c->dev; }
      hipLaunchKernelGGL(kfn, dim3(nblk), dim3(256), S::LDS_BYTES, c->stream, a, L);
    } else {
      auto kfn = k_head_loss<HID, false>;
      if (!((attr_devs[0] >> c->dev) & 1)) { HIPCHK(c, hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, S::LDS_BYTES)); attr_devs[0] |= 1ull << c->dev; }
      hipLaunchKernelGGL(kfn, dim3(nblk), dim3(256), S::LDS_BYTES, c->stream, a, L);
    }
    LAUNCHCHK(c, "k_head_loss");
  }
  defer_reduce(c, 0, nblk, (int64_t)c->NH * HID, 0, 0, c->g + c->headW, nullptr, acc, true, c->NH, c->g + c->headB);
  return PPO_OK;
}
int launch_head_loss(Ctx* c, const LossData& L, int n, bool acc, bool distill, float* sp, float* dp) {
  if (c->NH > HEAD_LD || c->nfc < 1) return 1;
  switch (c->hid) {
    case 32: return launch_head_loss_t<32>(c, L, n, acc, distill, sp, dp);
    case 64: return launch_head_loss_t<64>(c, L, n, acc, distill, sp, dp);
    case 128: return launch_head_loss_t<128>(c, L, n, acc, distill, sp, dp);
    default: return 1;
  }
}
bool head_loss_covers(const Ctx* c) { return c->XH == 0 && c->NH <= HEAD_LD && c->nfc >= 1 && (c->hid == 32 || c->hid == 64 || c->hid == 128); }

// Output layer alone, of `n` samples whose last hidden activations are in the workspaces (k_head_act): with a.noise
// the policy's sample, else means and values.
bool head_act_covers(const Ctx* c) { return c->XH == 0 && c->NH <= HEAD_LD && c->A <= c->NH && (c->hid == 32 || c->hid == 64 || c->hid == 128); }
int launch_head_act(Ctx* c, HeadActArgs a, int n) {
  a.h = c->fcact[c->nfc - 1]; a.w = c->shadow + c->headW; a.bias = c->p + c->headB; a.n = n; a.A = c->A; a.NH = c->NH;
  ProfScope ps(c, a.noise ? "head+sample" : "head_fwd", 2.0 * n * (double)c->hid * c->NH, (double)n * (2.0 * c->hid + (a.noise ? 12.0 : 4.0) * c->A + 16.0));
  const dim3 grid(cdiv(n, 32)), blk(64);
#define LAUNCH_HEAD_ACT(HID_)                                                                                   \
  do {                                                                                                            \
    if (a.noise) hipLaunchKernelGGL((k_head_act<HID_, true>), grid, blk, 0, c->stream, a);                         \
    else hipLaunchKernelGGL((k_head_act<HID_, false>), grid, blk, 0, c->stream, a);                                \
  } while (0)
  if (c->hid == 32) LAUNCH_HEAD_ACT(32); else if (c->hid == 64) LAUNCH_HEAD_ACT(64); else LAUNCH_HEAD_ACT(128);
#undef LAUNCH_HEAD_ACT
  LAUNCHCHK(c, "k_head_act");
  return PPO_OK;
}

int run_update(Ctx* c, const ppo_hparams* hp, ppo_mb_stats* host_stats, bool distill) {
  // a minibatch is Bu units of L rows each: samples (L = 1), or whole environments of T steps (recurrent nets)
  const bool recurrent = c->nl > 0;
  const int L = recurrent ? c->T : 1, Bu = c->PU / hp->minibatches, CU = recurrent ? c->CHe : c->CH;
  const int B = Bu * L;
  const int steps = hp->epochs * hp->minibatches;
  const int blocks_per_chunk = cdiv(CU * L, LOSS_BLOCK);
  int k = 0;
  const bool adaptive = !distill && hp->desired_kl > 0.f;  // the learning rate lives on the device and follows approx_kl
  if (!distill && hp->norm_adv) {
    ProfScope ps(c, "adv_normalize", 0.0, 12.0 * c->S);
    int per = cdiv(c->S, ADVN_BLOCKS);
    if (per < 4096) per = 4096;  // a block is worth launching for a few samples per thread
    const int nblk = cdiv(c->S, per);
    hipLaunchKernelGGL(k_adv_stats, dim3(nblk), dim3(1024), 0, c->stream, c->S, per, c->adv, c->advn_part);
    hipLaunchKernelGGL(k_adv_apply, dim3(nblk), dim3(1024), 0, c->stream, c->S, per, nblk, c->adv, c->advn_part, c->adv_n);
    LAUNCHCHK(c, "advantage normalisation");
  }
  for (int e = 0; e < hp->epochs; ++e) {
    int rc = PPO_OK;
    // the permutations of the next PERM_BATCH epochs in one set of launches (those of the last set are no longer read)
    if (e % PERM_BATCH == 0) rc = gen_permutations(c, hp->seed, (uint64_t)c->update_idx, (uint64_t)e, hp->epochs - e < PERM_BATCH ? hp->epochs - e : PERM_BATCH);
    if (rc) return rc;
    for (int mb = 0; mb < hp->minibatches; ++mb, ++k) {
      const int32_t* units = c->perm + (int64_t)(e % PERM_BATCH) * c->PU + (int64_t)mb * Bu;
      int nblocks = 0;
      for (int c0 = 0, ci = 0; c0 < Bu; c0 += CU, ++ci) {
        const int nu = (Bu - c0 < CU) ? Bu - c0 : CU, n = nu * L;
        const bool fused_head = head_loss_covers(c);
        // the rollout samples of the chunk's rows: the permutation's entries themselves, or the index list that
        // forward_seq_chunk builds from the chunk's environments
        const int32_t* rows = recurrent ? c->seqidx : units + c0;
        rc = recurrent ? forward_seq_chunk(c, units + c0, nu, !fused_head) : forward_chunk(c, rows, n, true, !fused_head);
        if (rc) return rc;
        float* sp = c->stat_part + (int64_t)ci * blocks_per_chunk * LOSS_NSTAT;
        float* dp = c->dls_part + (int64_t)ci * blocks_per_chunk * 32;
        LossData L;
        L.Bfull = B; L.A = c->A; L.logstd = distill ? nullptr : c->p + c->logstd; L.idx = rows; L.action = c->action; L.logp_old = c->logp;
        L.v_old = c->value; L.adv = hp->norm_adv ? c->adv_n : c->adv; L.ret = c->ret; L.clip_eps = hp->clip_eps; L.vclip_eps = hp->vclip_eps; L.vf_coef = hp->vf_coef;
        L.aux_dim = distill ? hp->aux_dim : 0; L.aux_coef = hp->aux_coef;
        bool head_done = false;
        if (fused_head) {
          rc = launch_head_loss(c, L, n, c0 > 0, distill, sp, dp);
          if (rc != PPO_OK && rc != 1) return rc;
          head_done = rc == PPO_OK;
          if (!head_done) {  // workspaces too small for the fused form: the output layer as a GEMM after all
            ARows al = plain_arows(c->fcact[c->nfc - 1], c->hid, n, c->hid);
            Ep<MapRows, float, true, false, false> ep;
            ep.map = plain_map(HEAD_LD, n); ep.out = c->headout; ep.bias = c->p + c->headB; ep.mask = nullptr; ep.N = c->NH;
            rc = launch_gemm(c, al, n, c->shadow + c->headW, c->hid, c->NH, c->hid, ep, "head_fwd", 2.0 * n * c->hid + 4.0 * n * c->NH);
            if (rc) return rc;
          }
        }
        if (!head_done) {
        ProfScope ps(c, "loss", 0.0, (double)n * (HEAD_LD * 6.0 + 4.0 * c->A + 20.0));
        if (distill) hipLaunchKernelGGL(k_loss<true>, dim3(cdiv(n, LOSS_BLOCK)), dim3(LOSS_BLOCK), 0, c->stream, n, L, c->headout, c->dhead, sp, dp);
        else hipLaunchKernelGGL(k_loss<false>, dim3(cdiv(n, LOSS_BLOCK)), dim3(LOSS_BLOCK), 0, c->stream, n, L, c->headout, c->dhead, sp, dp);
        LAUNCHCHK(c, "loss kernel");
        }
        // partial slots of a ragged last chunk follow the full chunks contiguously
        nblocks = ci * blocks_per_chunk + cdiv(n, LOSS_BLOCK);
        if (c0 + CU >= Bu) {
          // last chunk: every loss partial of the minibatch exists; their sums (statistics, log-std gradient)
          // are taken by one more block of the backward pass's reduction launch
          LossFinalize& f = c->lossfin;
          f.on = 1; f.nblocks = nblocks; f.Bfull = B; f.A = c->A; f.distill = distill ? 1 : 0; f.stat_part = c->stat_part; f.dls_part = c->dls_part;
          f.logstd = distill ? nullptr : c->p + c->logstd; f.vf_coef = hp->vf_coef; f.ent_coef = hp->ent_coef; f.st = c->dstats + k;
          f.g_logstd = distill ? nullptr : c->g + c->logstd;
          f.desired_kl = adaptive ? hp->desired_kl : 0.f; f.lr_min = hp->lr_min; f.lr_max = hp->lr_max; f.lr_init = hp->lr; f.lr_dev = c->lr_dev;
          f.lr_reset = (k == 0 && !(hp->lr_carry && c->lr_live)) ? 1 : 0;
          f.aux_dim = distill ? hp->aux_dim : 0; f.aux_coef = hp->aux_coef;
        }
        rc = recurrent ? backward_seq_chunk(c, nu, c0 > 0, !head_done) : backward_chunk(c, rows, n, c0 > 0, !head_done);
        if (rc) return rc;
      }
      if (c->lossfin.on) { rc = flush_reduces(c); if (rc) return rc; }  // (a backward pass always ends with a flush; kept for safety)
      c->step += 1;
      {
      ProfScope ps(c, "adam", 0.0, 30.0 * (double)c->total);
      const double c1 = 1.0 - pow((double)hp->beta1, (double)c->step), c2 = 1.0 - pow((double)hp->beta2, (double)c->step);
      const bool clip = hp->max_grad_norm > 0.f;
      if (clip) {  // the norm has to be known before the step: one more pass over the gradient
        hipLaunchKernelGGL(k_gnorm_partial, dim3(c->adam_blocks), dim3(256), 0, c->stream, c->total, c->g, c->sq_part);
        LAUNCHCHK(c, "k_gnorm_partial");
      }
      GnormFinalize norm;
      norm.on = clip ? 1 : 0; norm.nb = c->adam_blocks; norm.sq_part = c->sq_part; norm.st = c->dstats + k; norm.max_norm = hp->max_grad_norm;
      hipLaunchKernelGGL(k_adam, dim3(c->adam_blocks), dim3(256), 0, c->stream, c->total, c->p, c->m, c->v, c->g, c->shadow, hp->lr, hp->beta1, hp->beta2,
                         hp->adam_eps, (float)(1.0 / c1), (float)(1.0 / c2), c->sq_part, norm,
                         adaptive ? c->lr_dev : nullptr);
      LAUNCHCHK(c, "k_adam");
      if (!clip) {  // the step's gradient norm: one more block of the re-pack launch that follows
        c->gnfin = norm;
        c->gnfin.on = 1;
      }
      }
      rc = repack_weights(c);
      if (rc) return rc;
    }
  }
  c->update_idx += 1;
  if (adaptive) c->lr_live = true;
  if (host_stats) {
    HIPCHK(c, hipMemcpyAsync(host_stats, c->dstats, sizeof(DevStats) * (size_t)steps, hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
  }
  return PPO_OK;
}

// The way back ends in ordinary host memory, by way of a ring of pinned pieces.  The calling thread queues every transfer
// (a stream handle may name another stream in another thread) and waits for each to arrive; a small team copies the pieces
// into the caller's memory, whose fresh pages fault on first touch, under the transfers that follow: 22 MB
// arrive in 0.79 ms, 43 MB in 1.64 (with every thread queueing its own transfers 0.79 and 1.61; pieces dealt to the team
// in turn 1.72: one thread's slow page faults then hold up the ring; a lone thread took 4.4 for 64 MB where a team
// took 1.6).  Vectors of a few pieces need no team.
// One piece has nothing to overlap with: straight into the caller's memory (70 k parameters 44 -> 38 us, 235 k 73 -> 66).
constexpr int64_t HSTAGE = 1 << 18;  // floats per slot (1 MiB)
constexpr int HSTAGE_TEAM = 4;
int64_t read_pieces(const Ctx* c) { return cdiv(c->total, HSTAGE); }
int read_team(const Ctx* c) { return read_pieces(c) < 2 * HSTAGE_TEAM ? 1 : HSTAGE_TEAM; }
int create_read_staging(Ctx* c) {
  const int64_t slots = std::min(read_pieces(c), (int64_t)2 * read_team(c));
  if (slots < 2) return PPO_OK;
  HIPCHK(c, hipHostMalloc((void**)&c->hstage, sizeof(float) * (size_t)slots * HSTAGE, hipHostMallocDefault));
  for (int i = 0; i < slots; ++i) HIPCHK(c, hipEventCreateWithFlags(&c->hstage_ev[i], hipEventDisableTiming));
  return PPO_OK;
}

// Which passes run the first two convolutions in one kernel per direction: the forward where its kernel covers the shapes; in
// training the weight gradient and the input gradient must as well (nothing then reads the first layer's output from memory).
void choose_conv01(Ctx* c) {
  c->f01_fwd = c->f01_train = false;
  if (c->ln || c->E > 0 || c->nl > 0 || c->nconv < 2 || conv_small_covers(c)) return;
  ImgAddr none; none.base = nullptr; none.idx = nullptr; none.stride_b = none.stride_v = 0; none.V = c->V;
  static const uint32_t some_bits = 0;
  int grid = 0;
  c->dry = true;
  c->f01_fwd = launch_conv01_fwd(c, none, none, nullptr, 1, false) == PPO_OK;
  c->f01_train = c->f01_fwd && launch_conv01_wgrad(c, none, none, 1, false) == PPO_OK &&
                 launch_conv_dgrad_wgrad0_tile(c, none, none, &some_bits, nullptr, c->cC[2], c->cC[1], c->cH[1], c->cW[1], c->cH[2], c->cW[2], none, c->cC[0], c->cH[0], c->cW[0], 1,
                                               "", 0.0, 0.0, &grid) == PPO_OK;
  c->dry = false;
}
int create_impl(Ctx* c) {
  build_geometry(c);
  HIPCHK(c, hipGetDevice(&c->dev));
  if (c->dev < 0 || c->dev >= 64) return fail(c, PPO_EHIP, "device number %d out of range", c->dev);
  { int32_t* ws = nullptr; HIPCHK(c, static_scratch(&ws)); }  // the static scratch of ppo_permutation_static on this device
  const int V = c->V;
  int CH = c->d.max_chunk > 0 ? c->d.max_chunk : 16384 / V;
  if (CH > c->S) CH = c->S;
  if (CH < 1) CH = 1;
  c->CH = CH;
  choose_conv01(c);
  // the kernels index rows with 32-bit integers
  if ((int64_t)CH * V * c->cH[1] * c->cW[1] >= (1LL << 31) || (int64_t)CH * c->feat_ld >= (1LL << 40))
    return fail(c, PPO_ESHAPE, "chunk of %d samples is too large for 32-bit row indices; lower max_chunk", CH);
  const int64_t S = c->S;
  c->PU = c->nl > 0 ? c->N : c->S;
  c->CHe = CH / c->T < 1 ? 1 : CH / c->T;
  if (c->CHe > c->N) c->CHe = c->N;
  if (c->nl > 0 && (int64_t)c->CHe * c->T > CH) return fail(c, PPO_ESHAPE, "max_chunk = %d holds no whole environment of %d steps", CH, c->T);
  // parameters
  DALLOC(c, c->p, c->total); DALLOC(c, c->m, c->total); DALLOC(c, c->v, c->total); DALLOC(c, c->g, c->total);
  DALLOC(c, c->shadow, c->total + 8);
  DALLOC(c, c->canon, c->total);
  for (int l = 1; l < c->nconv; ++l) {
    for (int py = 0; py < 2; ++py) DALLOC(c, c->wd[l][py], (int64_t)2 * c->cC[l] * (1 + py) * 2 * c->cC[l + 1]);
    DALLOC(c, c->wtap[l], (int64_t)9 * c->cC[l] * c->cC[l + 1]);
  }
  for (int l = 0; l < c->nfc; ++l) DALLOC(c, c->fcT[l], (int64_t)c->fin[l] * c->fout[l]);
  DALLOC(c, c->headT, (int64_t)c->hid * HEAD_LD);
  if (c->XH > 0) { DALLOC(c, c->aux1T, (int64_t)c->hid * c->XH); DALLOC(c, c->aux2T, (int64_t)c->XH * HEAD_LD); }
  // rollout buffer
  DALLOC(c, c->obs, S * V * c->img_elems);
  DALLOC(c, c->proprio, S * c->P); DALLOC(c, c->action, S * c->A);
  DALLOC(c, c->logp, S); DALLOC(c, c->value, S); DALLOC(c, c->reward, S); DALLOC(c, c->adv, S); DALLOC(c, c->adv_n, S); DALLOC(c, c->ret, S); DALLOC(c, c->done, S);
  // permutation of the PU units a minibatch is drawn from: about 32 keys per bucket
  int nb = 1, lg = 0;
  while ((int64_t)nb * 32 < c->PU && nb < (1 << 20)) { nb <<= 1; ++lg; }
  c->nb = nb; c->shift = 64 - lg;
  DALLOC(c, c->perm, (int64_t)PERM_BATCH * c->PU); DALLOC(c, c->ptmp, (int64_t)PERM_BATCH * c->PU);  // one slot per epoch of a batch
  DALLOC(c, c->phist, (int64_t)PERM_BATCH * 2 * nb); DALLOC(c, c->pstart, (int64_t)PERM_BATCH * nb);
  // workspaces
  int64_t gmax = (int64_t)CH * c->feat_ld;
  for (int l = 0; l < c->nconv - 1; ++l) {
    int64_t e = (int64_t)CH * V * c->cC[l + 1] * c->cH[l + 1] * c->cW[l + 1];
    const bool in_memory = l > 0 || !c->f01_train;  // else neither the first layer's output nor its gradient is
    if (in_memory) DALLOC(c, c->act[l], e);
    const int64_t words = (int64_t)CH * V * c->cH[l + 1] * (l == 0 && c->f01_train ? c->b0pitch : c->cW[l + 1]) * ((c->cC[l + 1] + 31) / 32);
    DALLOC(c, c->abits[l], words);
    if (l == 0 && c->f01_train) HIPCHK(c, hipMemsetAsync(c->abits[0], 0, (size_t)words * 4, c->stream));  // the words behind a row's last pixel stay zero
    if (in_memory && e > gmax) gmax = e;
  }
  DALLOC(c, c->feat, (int64_t)CH * c->feat_ld);
  if ((int64_t)CH * c->fin[0] > gmax) gmax = (int64_t)CH * c->fin[0];
  if (c->E > 0) {  // the last convolution's activation has a buffer of its own, read by the embedding
    const int l = c->nconv - 1;
    DALLOC(c, c->act[l], (int64_t)CH * V * c->flat);
    DALLOC(c, c->embT, (int64_t)c->flat * c->E);
    if ((int64_t)CH * V * c->flat > gmax) gmax = (int64_t)CH * V * c->flat;
  }
  if (c->ln) {
    int64_t emax = 0;
    for (int l = 0; l < c->nconv; ++l) {
      const int64_t e = (int64_t)CH * V * c->cC[l + 1] * c->cH[l + 1] * c->cW[l + 1];
      DALLOC(c, c->lnstat[l], (int64_t)CH * V);
      if (e > gmax) gmax = e;
      if (l == 0 && ln0_covers(c)) continue;  // the convolution's output and its gradient stay in registers
      DALLOC(c, c->pre[l], e);
      if (e > emax) emax = e;
    }
    DALLOC(c, c->dpre, emax);
  }
  if (c->nl > 0) {
    const int H = c->H;
    c->xh[0] = c->feat;
    for (int l = 0; l < c->nl; ++l) {
      const int64_t K = c->lin[l] + H;
      DALLOC(c, c->lstmWT[l], K * 4 * H);
      if (l > 0) DALLOC(c, c->xh[l], (int64_t)CH * K);
      if (l == 0 || !lstm_side_by_side(c)) DALLOC(c, c->dxh[l], (int64_t)CH * K);  // side by side, upper layers' stay in lstm_part
      const int64_t rows = std::max<int64_t>(CH, c->T * lstm_tiled_rows(c, c->CHe));
      DALLOC(c, c->gates[l], rows * 4 * H); DALLOC(c, c->c_enter[l], rows * H);
      DALLOC(c, c->da[l], (int64_t)CH * 4 * H); DALLOC(c, c->dc_carry[l], lstm_tiled_rows(c, c->CHe) * H);
    }
    if (lstm_side_by_side(c)) DALLOC(c, c->lstm_part, lstm_part_elems(c));
    else DALLOC(c, c->lstm_pre, (int64_t)c->CHe * 4 * H);
    DALLOC(c, c->htop, (int64_t)CH * H); DALLOC(c, c->seqidx, CH);
    DALLOC(c, c->h0, (int64_t)c->nl * c->N * H); DALLOC(c, c->c0, (int64_t)c->nl * c->N * H);
    HIPCHK(c, hipMemsetAsync(c->h0, 0, sizeof(float) * (size_t)c->nl * c->N * H, c->stream));
    HIPCHK(c, hipMemsetAsync(c->c0, 0, sizeof(float) * (size_t)c->nl * c->N * H, c->stream));
    if ((int64_t)CH * H > gmax) gmax = (int64_t)CH * H;
  }
  for (int l = 0; l < c->nfc; ++l) { DALLOC(c, c->fcact[l], (int64_t)CH * c->fout[l]); if ((int64_t)CH * c->fout[l] > gmax) gmax = (int64_t)CH * c->fout[l]; }
  DALLOC(c, c->headout, (int64_t)CH * HEAD_LD); DALLOC(c, c->dhead, (int64_t)CH * HEAD_LD);
  if (c->XH > 0) {
    DALLOC(c, c->auxact, (int64_t)CH * c->XH); DALLOC(c, c->dauxact, (int64_t)CH * c->XH); DALLOC(c, c->daux, (int64_t)CH * HEAD_LD);
    HIPCHK(c, hipMemsetAsync(c->headout, 0, sizeof(float) * (size_t)CH * HEAD_LD, c->stream));
  }
  DALLOC(c, c->gbuf[0], gmax); DALLOC(c, c->gbuf[1], gmax);
  // weight-gradient partials: room for every layer at its preferred split count, all layers of a backward
  // pass side by side (their sums are taken in one launch at the end of the pass)
  int64_t pe_sum = 2048LL * c->cC[1] * (9 * c->cC[0] + 1), bpe_sum = 0;
  // k_wgrad, of a chunk's rows or fewer.  (Of more than 256 columns also as many slices as blocks of 384 columns would take: the
  // products of wide layers that are cut into slices leave their partial sums here as well.)
  auto want = [&](int Nn, int Kk, int64_t M, int64_t& need, int64_t& bneed) {
    int splits = WgradCut(Nn, Kk).splits_up_to(M);
    if (Kk > 256) splits = std::max(splits, std::min(cdiv(768, cdiv(Kk, 384) * cdiv(Nn, 64)), cdiv(M, 128)));
    need = (int64_t)splits * Nn * Kk; bneed = (int64_t)splits * Nn;
  };
  for (int l = 1; l < c->nconv; ++l) {
    int64_t need, bneed;
    want(c->cC[l + 1], 9 * c->cC[l], (int64_t)CH * V * c->cH[l + 1] * c->cW[l + 1], need, bneed);
    // or one partial per block of the LDS-image weight-gradient kernel
    const int64_t gy = cdiv(c->cC[l + 1], 64), gx = 256 / gy > 0 ? 256 / gy : 1, per = (int64_t)c->cC[l + 1] * 9 * c->cC[l];
    if (gx * per > need) need = gx * per;
    if (gx * c->cC[l + 1] > bneed) bneed = gx * c->cC[l + 1];
    pe_sum += need; bpe_sum += bneed;
  }
  for (int l = 0; l < c->nfc; ++l) {
    int64_t need, bneed;
    want(c->fout[l], c->fin[l], CH, need, bneed);
    const int64_t per = (int64_t)c->fout[l] * c->fin[l];  // k_wgrad_rs: up to four splits are worth their partials
    if (4 * per > need) need = 4 * per;
    if (4 * (int64_t)c->fout[l] > bneed) bneed = 4 * (int64_t)c->fout[l];
    pe_sum += need; bpe_sum += bneed;
  }
  {
    int64_t need, bneed;
    want(c->NH, c->hid, CH, need, bneed);
    const int64_t nblk = cdiv(CH, 64);  // fused output-layer kernel: one partial per 64 samples
    if (nblk * c->NH * c->hid > need) need = nblk * c->NH * c->hid;
    if (nblk * c->NH > bneed) bneed = nblk * c->NH;
    pe_sum += need; bpe_sum += bneed;
  }
  if (c->E > 0) { int64_t need, bneed; want(c->E, c->flat, CH, need, bneed); pe_sum += need; bpe_sum += bneed; }
  for (int l = 0; l < c->nl; ++l) {
    int64_t need, bneed;
    want(4 * c->H, c->lin[l] + c->H, CH, need, bneed);
    const int64_t per = (int64_t)4 * c->H * (c->lin[l] + c->H);
    if (4 * per > need) need = 4 * per;
    if (16 * (int64_t)c->H > bneed) bneed = 16 * (int64_t)c->H;
    pe_sum += need; bpe_sum += bneed;
  }
  if (conv_small_covers(c)) { pe_sum += 1024LL * (1152 + 80); bpe_sum += 1024LL * 16; }
  if (c->ln) pe_sum += 1024LL * 2 * 1024;  // layer-norm gain / shift partials: one per block of k_ln_bwd
  if (c->XH > 0) {
    int64_t need, bneed;
    want(c->XH, c->hid, CH, need, bneed); pe_sum += need; bpe_sum += bneed;
    want(c->X, c->XH, CH, need, bneed); pe_sum += need; bpe_sum += bneed;
  }
  c->partial_cap = pe_sum; c->bias_partial_cap = bpe_sum > 0 ? bpe_sum : 1;
  DALLOC(c, c->partial_base, c->partial_cap); DALLOC(c, c->bias_partial_base, c->bias_partial_cap);
  c->partial = c->partial_base; c->partial_elems = c->partial_cap;
  c->bias_partial = c->bias_partial_base; c->bias_partial_elems = c->bias_partial_cap;
  c->rjobs.njobs = 0; c->rjob_blocks = 0;
  DALLOC(c, c->zpage, 32768);
  HIPCHK(c, hipMemsetAsync(c->zpage, 0, 65536, c->stream));
  // loss / Adam partials
  {
    const int CU = c->nl > 0 ? c->CHe : CH, Lr = c->nl > 0 ? c->T : 1;
    c->max_loss_blocks = (cdiv(c->PU, CU) + 1) * cdiv((int64_t)CU * Lr, LOSS_BLOCK) + 1;
  }
  DALLOC(c, c->stat_part, (int64_t)c->max_loss_blocks * LOSS_NSTAT); DALLOC(c, c->dls_part, (int64_t)c->max_loss_blocks * 32);
  c->adam_blocks = cdiv(c->total, 1024); if (c->adam_blocks > 2048) c->adam_blocks = 2048;
  DALLOC(c, c->sq_part, c->adam_blocks);
  DALLOC(c, c->lr_dev, 1); DALLOC(c, c->advn_part, 3 * ADVN_BLOCKS);
  DALLOC(c, c->dstats, c->max_steps);
  HIPCHK(c, hipMemsetAsync(c->p, 0, sizeof(float) * (size_t)c->total, c->stream));
  HIPCHK(c, hipMemsetAsync(c->m, 0, sizeof(float) * (size_t)c->total, c->stream));
  HIPCHK(c, hipMemsetAsync(c->v, 0, sizeof(float) * (size_t)c->total, c->stream));
  HIPCHK(c, hipMemsetAsync(c->g, 0, sizeof(float) * (size_t)c->total, c->stream));
  HIPCHK(c, hipMemsetAsync(c->shadow, 0, sizeof(bf16_t) * (size_t)(c->total + 8), c->stream));
  int rc = refresh_shadow(c);
  if (rc) return rc;
  rc = create_read_staging(c);
  if (rc) return rc;
  HIPCHK(c, hipStreamSynchronize(c->stream));
  c->written.assign((size_t)c->T, 0);
  c->cover.assign((size_t)c->T, {});
  return PPO_OK;
}

void free_all(Ctx* c) {
  for (void* p : c->allocs) (void)hipFree(p);
  c->allocs.clear();
  for (auto& e : c->hstage_ev) if (e) { (void)hipEventDestroy(e); e = nullptr; }
  if (c->hstage) { (void)hipHostFree(c->hstage); c->hstage = nullptr; }
}

// Parameter-shaped vectors cross the ABI in canonical order and live on the device in the internal one; the
// reordering is a device kernel over a staging vector in canonical order (k_param_map).
int to_internal(Ctx* c, const float* canon, float* dev) {
  HIPCHK(c, hipMemcpyAsync(c->canon, canon, sizeof(float) * (size_t)c->total, hipMemcpyHostToDevice, c->stream));
  hipLaunchKernelGGL(k_param_map<true>, dim3(cdiv(c->total, 256)), dim3(256), 0, c->stream, c->pmap, c->canon, dev);
  LAUNCHCHK(c, "k_param_map");
  HIPCHK(c, hipStreamSynchronize(c->stream));
  return PPO_OK;
}
int to_canonical(Ctx* c, const float* dev, float* canon) {
  hipLaunchKernelGGL(k_param_map<false>, dim3(cdiv(c->total, 256)), dim3(256), 0, c->stream, c->pmap, dev, c->canon);
  LAUNCHCHK(c, "k_param_map");
  const int64_t np = read_pieces(c);
  const int team = read_team(c);
  if (np == 1) {
    HIPCHK(c, hipMemcpyAsync(canon, c->canon, sizeof(float) * (size_t)c->total, hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    return PPO_OK;
  }
  const int slots = (int)std::min(np, (int64_t)2 * team);
  auto count = [&](int64_t k) { return std::min(HSTAGE, c->total - k * HSTAGE); };
  auto copy = [&](int64_t k, int slot) { memcpy(canon + k * HSTAGE, c->hstage + slot * HSTAGE, sizeof(float) * (size_t)count(k)); };
  // pieces arrive in order, in whichever slot was free; whoever of the team is idle copies the oldest one
  struct Piece { int64_t k; int slot; };
  std::mutex mu;
  std::condition_variable work, space;
  Piece arrived[2 * HSTAGE_TEAM], flight[2 * HSTAGE_TEAM];  // rings of `slots`
  int64_t n_arrived = 0, n_taken = 0, n_queued = 0, n_landed = 0;
  int spare[2 * HSTAGE_TEAM], n_spare = slots;
  for (int i = 0; i < slots; ++i) spare[i] = i;
  bool last = false;  // nothing arrives any more
  auto member = [&]() {
    for (;;) {
      Piece q;
      {
        std::unique_lock<std::mutex> lk(mu);
        work.wait(lk, [&]() { return n_taken < n_arrived || last; });
        if (n_taken == n_arrived) return;
        q = arrived[n_taken++ % slots];
      }
      copy(q.k, q.slot);
      { std::lock_guard<std::mutex> lk(mu); spare[n_spare++] = q.slot; }
      space.notify_one();
    }
  };
  std::thread members[HSTAGE_TEAM];
  bool helped = false;
  for (int t = 0; t < team && team > 1; ++t) {
    try {
      members[t] = std::thread(member);
      helped = true;
    } catch (...) {  // no thread to be had: the others do its share, or this one
    }
  }
  hipError_t e = hipSuccess;
  while (n_landed < np && e == hipSuccess) {
    while (n_queued < np && e == hipSuccess) {  // every transfer there is room for; at least one in flight
      int slot;
      {
        std::unique_lock<std::mutex> lk(mu);
        if (n_spare == 0 && n_queued > n_landed) break;
        space.wait(lk, [&]() { return n_spare > 0; });
        slot = spare[--n_spare];
      }
      const int64_t k = n_queued;
      e = hipMemcpyAsync(c->hstage + slot * HSTAGE, c->canon + k * HSTAGE, sizeof(float) * (size_t)count(k), hipMemcpyDeviceToHost, c->stream);
      if (e == hipSuccess) e = hipEventRecord(c->hstage_ev[slot], c->stream);
      flight[n_queued++ % slots] = Piece{k, slot};
    }
    if (e != hipSuccess) break;
    const Piece q = flight[n_landed++ % slots];
    e = hipEventSynchronize(c->hstage_ev[q.slot]);
    if (e != hipSuccess) break;
    if (helped) {
      { std::lock_guard<std::mutex> lk(mu); arrived[n_arrived++ % slots] = q; }
      work.notify_one();
    } else {
      copy(q.k, q.slot);
      spare[n_spare++] = q.slot;
    }
  }
  { std::lock_guard<std::mutex> lk(mu); last = true; }
  work.notify_all();
  for (std::thread& m : members) if (m.joinable()) m.join();
  HIPCHK(c, e);
  return PPO_OK;
}

}  // namespace

struct ppo_ctx : Ctx {};

extern "C" {

int ppo_create(ppo_ctx** out, const ppo_net_desc* desc, void* hip_stream) {
  if (!out) return fail(nullptr, PPO_EINVAL, "out is NULL");
  *out = nullptr;
  int rc = validate_desc(desc);
  if (rc) return rc;
  ppo_ctx* c = new (std::nothrow) ppo_ctx();
  if (!c) return fail(nullptr, PPO_ENOMEM, "host allocation failed");
  c->d = *desc;
  c->stream = (hipStream_t)hip_stream;
  rc = create_impl(c);
  if (rc) { g_create_error = c->err; free_all(c); delete c; return rc; }
  *out = c;
  return PPO_OK;
}

int ppo_destroy(ppo_ctx* c) {
  if (!c) return PPO_EINVAL;
  (void)hipStreamSynchronize(c->stream);
  for (auto& r : c->prof_recs) { (void)hipEventDestroy(r.a); (void)hipEventDestroy(r.b); }
  for (auto e : c->prof_pool) (void)hipEventDestroy(e);
  free_all(c);
  delete c;
  return PPO_OK;
}

const char* ppo_last_error(const ppo_ctx* c) { return c ? c->err.c_str() : g_create_error.c_str(); }

int64_t ppo_param_count(const ppo_ctx* c) { return c ? c->total : PPO_EINVAL; }
int64_t ppo_buffer_image_bytes(const ppo_ctx* c) { return c ? (int64_t)c->S * c->V * c->img_elems * (int64_t)sizeof(bf16_t) : PPO_EINVAL; }

int ppo_set_params(ppo_ctx* c, const float* h, int64_t n) {
  if (!c) return PPO_EINVAL;
  if (!h) return fail(c, PPO_EINVAL, "h_params is NULL");
  if (n != c->total) return fail(c, PPO_ESHAPE, "expected %lld parameters, got %lld", (long long)c->total, (long long)n);
  int rc = to_internal(c, h, c->p);
  if (rc) return rc;
  rc = refresh_shadow(c);
  if (rc) return rc;
  HIPCHK(c, hipStreamSynchronize(c->stream));
  return PPO_OK;
}
int ppo_get_params(ppo_ctx* c, float* h, int64_t n) {
  if (!c) return PPO_EINVAL;
  if (!h) return fail(c, PPO_EINVAL, "h_params is NULL");
  if (n != c->total) return fail(c, PPO_ESHAPE, "expected %lld parameters, got %lld", (long long)c->total, (long long)n);
  return to_canonical(c, c->p, h);
}
int ppo_get_grads(ppo_ctx* c, float* h, int64_t n) {
  if (!c) return PPO_EINVAL;
  if (!h) return fail(c, PPO_EINVAL, "h_grads is NULL");
  if (n != c->total) return fail(c, PPO_ESHAPE, "expected %lld parameters, got %lld", (long long)c->total, (long long)n);
  return to_canonical(c, c->g, h);
}
int ppo_set_opt_state(ppo_ctx* c, const float* hm, const float* hv, int64_t n, int64_t step, int64_t update_idx) {
  if (!c) return PPO_EINVAL;
  if (!hm || !hv) return fail(c, PPO_EINVAL, "h_m / h_v is NULL");
  if (n != c->total) return fail(c, PPO_ESHAPE, "expected %lld parameters, got %lld", (long long)c->total, (long long)n);
  if (step < 0 || update_idx < 0) return fail(c, PPO_EINVAL, "step and update_idx must be >= 0");
  int rc = to_internal(c, hm, c->m);
  if (rc) return rc;
  rc = to_internal(c, hv, c->v);
  if (rc) return rc;
  c->step = step; c->update_idx = update_idx;
  return PPO_OK;
}
int ppo_get_opt_state(ppo_ctx* c, float* hm, float* hv, int64_t n, int64_t* step, int64_t* update_idx) {
  if (!c) return PPO_EINVAL;
  if (!hm || !hv) return fail(c, PPO_EINVAL, "h_m / h_v is NULL");
  if (n != c->total) return fail(c, PPO_ESHAPE, "expected %lld parameters, got %lld", (long long)c->total, (long long)n);
  int rc = to_canonical(c, c->m, hm);
  if (rc) return rc;
  rc = to_canonical(c, c->v, hv);
  if (rc) return rc;
  if (step) *step = c->step;
  if (update_idx) *update_idx = c->update_idx;
  return PPO_OK;
}

int ppo_get_adaptive_lr(ppo_ctx* c, float* h_lr, int32_t* h_live) {
  if (!c) return PPO_EINVAL;
  if (!h_lr || !h_live) return fail(c, PPO_EINVAL, "h_lr / h_live is NULL");
  *h_live = c->lr_live ? 1 : 0;
  *h_lr = 0.f;
  if (c->lr_live) {
    HIPCHK(c, hipMemcpyAsync(h_lr, c->lr_dev, sizeof(float), hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
  }
  return PPO_OK;
}
int ppo_set_adaptive_lr(ppo_ctx* c, float lr, int32_t live) {
  if (!c) return PPO_EINVAL;
  if (live != 0 && live != 1) return fail(c, PPO_EINVAL, "live must be 0 or 1");
  if (live && !(isfinite(lr) && lr > 0.f)) return fail(c, PPO_EINVAL, "a live adaptive rate must be finite and > 0");
  if (live) {
    HIPCHK(c, hipMemcpyAsync(c->lr_dev, &lr, sizeof(float), hipMemcpyHostToDevice, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
  }
  c->lr_live = live != 0;
  return PPO_OK;
}

static int write_slab(ppo_ctx* c, int32_t t, int32_t n0, int32_t cnt, const void* d_obs, const float* d_proprio, const float* d_action,
                      const float* d_logp, const float* d_value, const float* d_reward, const uint8_t* d_done);
static int all_written(ppo_ctx* c);

int ppo_buffer_write(ppo_ctx* c, int32_t t, const void* d_obs, const float* d_proprio, const float* d_action, const float* d_logp,
                     const float* d_value, const float* d_reward, const uint8_t* d_done) {
  if (!c) return PPO_EINVAL;
  if (t < 0 || t >= c->T) return fail(c, PPO_EINVAL, "t = %d outside [0, %d)", t, c->T);
  if (!d_obs || !d_proprio || !d_action) return fail(c, PPO_EINVAL, "d_obs, d_proprio and d_action must not be NULL");
  if (c->d.has_value_head && (!d_logp || !d_value || !d_reward || !d_done))
    return fail(c, PPO_EINVAL, "an actor-critic buffer needs d_logp, d_value, d_reward and d_done");
  const int rc = write_slab(c, t, 0, c->N, d_obs, d_proprio, d_action, d_logp, d_value, d_reward, d_done);
  if (rc) return rc;
  if (t == 0) { c->written.assign((size_t)c->T, 0); c->cover.assign((size_t)c->T, {}); }
  c->written[(size_t)t] = 1;
  c->cover[(size_t)t].clear();
  c->gae_done = false;
  return PPO_OK;
}

int ppo_buffer_write_range(ppo_ctx* c, int32_t t, int32_t env_offset, int32_t count, const void* d_obs, const float* d_proprio,
                           const float* d_action, const float* d_logp, const float* d_value, const float* d_reward, const uint8_t* d_done) {
  if (!c) return PPO_EINVAL;
  if (t < 0 || t >= c->T) return fail(c, PPO_EINVAL, "t = %d outside [0, %d)", t, c->T);
  if (env_offset < 0 || count < 0 || (int64_t)env_offset + count > c->N)
    return fail(c, PPO_EINVAL, "environments [%d, %d + %d) outside [0, %d)", env_offset, env_offset, count, c->N);
  if (count == 0) return PPO_OK;
  if (!d_obs || !d_proprio || !d_action) return fail(c, PPO_EINVAL, "d_obs, d_proprio and d_action must not be NULL");
  if (c->d.has_value_head && (!d_logp || !d_value || !d_reward || !d_done))
    return fail(c, PPO_EINVAL, "an actor-critic buffer needs d_logp, d_value, d_reward and d_done");
  // a range that arrives while every step of the rollout is complete is the first slice of the NEXT rollout: from
  // here on no step counts as written until its own ranges have covered [0, N) again (the slabs still hold the
  // previous rollout's records)
  const bool new_rollout = all_written(c) != 0;
  const int rc = write_slab(c, t, env_offset, count, d_obs, d_proprio, d_action, d_logp, d_value, d_reward, d_done);
  if (rc) return rc;
  if (new_rollout) { c->written.assign((size_t)c->T, 0); c->cover.assign((size_t)c->T, {}); }
  // within a rollout, a write into a complete step starts that step afresh; the step is complete again once the
  // ranges cover [0, N)
  auto& cv = c->cover[(size_t)t];
  if (c->written[(size_t)t] == 1) cv.clear();
  cv.push_back({env_offset, env_offset + count});
  std::sort(cv.begin(), cv.end());
  std::vector<std::pair<int, int>> merged;
  for (const auto& r : cv) {
    if (!merged.empty() && r.first <= merged.back().second) merged.back().second = std::max(merged.back().second, r.second);
    else merged.push_back(r);
  }
  cv.swap(merged);
  const bool complete = cv.size() == 1 && cv[0].first == 0 && cv[0].second == c->N;
  c->written[(size_t)t] = complete ? 1 : 0;
  if (complete) cv.clear();
  c->gae_done = false;
  return PPO_OK;
}

int ppo_buffer_write_state(ppo_ctx* c, const float* d_h0, const float* d_c0) {
  if (!c) return PPO_EINVAL;
  if (c->nl <= 0) return fail(c, PPO_ESTATE, "this network has no recurrent layers");
  const size_t bytes = sizeof(float) * (size_t)c->nl * c->N * c->H;
  if (d_h0) HIPCHK(c, hipMemcpyAsync(c->h0, d_h0, bytes, hipMemcpyDeviceToDevice, c->stream));
  else HIPCHK(c, hipMemsetAsync(c->h0, 0, bytes, c->stream));
  if (d_c0) HIPCHK(c, hipMemcpyAsync(c->c0, d_c0, bytes, hipMemcpyDeviceToDevice, c->stream));
  else HIPCHK(c, hipMemsetAsync(c->c0, 0, bytes, c->stream));
  return PPO_OK;
}

int ppo_buffer_read_obs(ppo_ctx* c, int32_t t, void* d_obs_bf16) {
  if (!c) return PPO_EINVAL;
  if (t < 0 || t >= c->T) return fail(c, PPO_EINVAL, "t = %d outside [0, %d)", t, c->T);
  if (!d_obs_bf16) return fail(c, PPO_EINVAL, "d_obs_bf16 is NULL");
  if (!c->written[(size_t)t]) return fail(c, PPO_ESTATE, "step %d has not been written", t);
  const int64_t nimg = (int64_t)c->N * c->V, n = nimg * c->d.in_c * c->d.in_h * c->d.in_w;
  hipLaunchKernelGGL(k_read_obs, dim3(cdiv(n, 256)), dim3(256), 0, c->stream, c->obs + (int64_t)t * nimg * c->img_elems, (bf16_t*)d_obs_bf16, nimg, c->d.in_c,
                     c->d.in_h, c->d.in_w, c->cW[0]);
  LAUNCHCHK(c, "k_read_obs");
  return PPO_OK;
}

static int all_written(ppo_ctx* c) {
  for (char w : c->written) if (w != 1) return 0;  // 2: acted, outcome still missing
  return 1;
}

// Images, proprioception and (where given) the other fields of step t into the slab: one launch.
// Environments [n0, n0 + cnt) of the step; the caller's arrays hold cnt rows.
static int write_slab(ppo_ctx* c, int32_t t, int32_t n0, int32_t cnt, const void* d_obs, const float* d_proprio, const float* d_action,
                      const float* d_logp, const float* d_value, const float* d_reward, const uint8_t* d_done) {
  const int N = cnt, V = c->V, C = c->d.in_c;
  const int64_t nimg = (int64_t)N * V;
  const bool flat = c->cW[0] == c->d.in_w;  // no pad: an image is one row
  const int W = flat ? c->d.in_h * c->d.in_w : c->d.in_w, rows = flat ? 1 : c->d.in_h, groups = (W + 7) / 8;
  const int64_t off = (int64_t)t * c->N + n0;
  bf16_t* dst = c->obs + off * V * c->img_elems;
  ProfScope ps(c, "buffer_write", 0.0, (double)nimg * c->img_elems * (c->d.obs_dtype == 0 ? 6.0 : 4.0) + (double)N * (6.0 * c->P + 8.0 * c->A + 26.0));
  const int mx = c->P > c->A ? c->P : c->A;
  ScalarWrite sw;
  sw.N = N; sw.P = c->P; sw.A = c->A; sw.proprio = d_proprio; sw.action = d_action; sw.logp = d_logp; sw.value = d_value; sw.reward = d_reward; sw.done = d_done;
  sw.o_proprio = c->proprio + off * c->P; sw.o_action = c->action + off * c->A; sw.o_logp = c->logp + off; sw.o_value = c->value + off;
  sw.o_reward = c->reward + off; sw.o_done = c->done + off;
  // 32-bit group numbers: a slab of more images than that goes out in several launches, the last with the scalars
  const int64_t most = std::max<int64_t>(1, ((1LL << 31) - 256) / ((int64_t)rows * groups));
  for (int64_t i0 = 0; i0 < nimg; i0 += most) {
    const int64_t ni = std::min(most, nimg - i0), n_row = ni * rows;
    const int obs_blocks = cdiv(n_row * groups, 256), sc_blocks = i0 + ni == nimg ? cdiv((int64_t)N * mx, 256) : 0;
    const int64_t so = i0 * C * c->d.in_h * c->d.in_w;
    bf16_t* const d0 = dst + i0 * c->img_elems;
    const FastDiv dg = make_fastdiv(groups), dh = make_fastdiv(rows);
#define LAUNCH_WRITE(T_, C_) hipLaunchKernelGGL((k_write_obs<T_, C_>), dim3(obs_blocks + sc_blocks), dim3(256), 0, c->stream, (const T_*)d_obs + so, d0, n_row, W, dg, dh, obs_blocks, sw)
    if (c->d.obs_dtype == 0) { if (C == 1) LAUNCH_WRITE(float, 1); else LAUNCH_WRITE(float, 3); }
    else { if (C == 1) LAUNCH_WRITE(bf16_t, 1); else LAUNCH_WRITE(bf16_t, 3); }
#undef LAUNCH_WRITE
  }
  LAUNCHCHK(c, "k_write_obs");
  return PPO_OK;
}

int ppo_gae(ppo_ctx* c, const float* d_last_value, float gamma, float lambda) {
  if (!c) return PPO_EINVAL;
  if (!d_last_value) return fail(c, PPO_EINVAL, "d_last_value is NULL");
  if (!isfinite(gamma) || !isfinite(lambda) || gamma < 0.f || gamma > 1.f || lambda < 0.f || lambda > 1.f)
    return fail(c, PPO_EINVAL, "gamma and lambda must be in [0, 1]");
  if (!c->d.has_value_head) return fail(c, PPO_ESTATE, "this context has no value head (distillation student)");
  if (!all_written(c)) return fail(c, PPO_ESTATE, "ppo_gae needs all %d steps written", c->T);
  ProfScope ps(c, "gae", 6.0 * c->S, 17.0 * c->S + 4.0 * c->N);
  if (c->T <= 8) hipLaunchKernelGGL(k_gae<8>, dim3(cdiv(c->N, 64)), dim3(64), 0, c->stream, c->T, c->N, c->reward, c->done, c->value, d_last_value, gamma, lambda, c->adv, c->ret);
  else if (c->T <= 16) hipLaunchKernelGGL(k_gae<16>, dim3(cdiv(c->N, 64)), dim3(64), 0, c->stream, c->T, c->N, c->reward, c->done, c->value, d_last_value, gamma, lambda, c->adv, c->ret);
  else hipLaunchKernelGGL(k_gae<32>, dim3(cdiv(c->N, 64)), dim3(64), 0, c->stream, c->T, c->N, c->reward, c->done, c->value, d_last_value, gamma, lambda, c->adv, c->ret);
  LAUNCHCHK(c, "k_gae");
  c->gae_done = true;
  return PPO_OK;
}

int ppo_get_adv_ret(ppo_ctx* c, float* d_adv, float* d_ret) {
  if (!c) return PPO_EINVAL;
  if (!c->gae_done) return fail(c, PPO_ESTATE, "ppo_gae has not run on this rollout");
  if (d_adv) HIPCHK(c, hipMemcpyAsync(d_adv, c->adv, sizeof(float) * (size_t)c->S, hipMemcpyDeviceToDevice, c->stream));
  if (d_ret) HIPCHK(c, hipMemcpyAsync(d_ret, c->ret, sizeof(float) * (size_t)c->S, hipMemcpyDeviceToDevice, c->stream));
  return PPO_OK;
}

int ppo_permutation(ppo_ctx* c, uint64_t seed, uint64_t update_idx, uint64_t epoch, int32_t* h_perm) {
  if (!c) return PPO_EINVAL;
  if (!h_perm) return fail(c, PPO_EINVAL, "h_perm is NULL");
  int rc = gen_permutation(c, seed, update_idx, epoch);
  if (rc) return rc;
  HIPCHK(c, hipMemcpyAsync(h_perm, c->perm, sizeof(int32_t) * (size_t)c->PU, hipMemcpyDeviceToHost, c->stream));
  HIPCHK(c, hipStreamSynchronize(c->stream));
  return PPO_OK;
}

int ppo_permutation_static(int64_t S, uint64_t seed, uint64_t update_idx, uint64_t epoch, int32_t* d_perm, void* hip_stream) {
  if (S < 0) return fail(nullptr, PPO_EINVAL, "S must be >= 0");
  if (S > STATIC_PERM_MAX_S)
    return fail(nullptr, PPO_ESHAPE, "ppo_permutation_static handles at most %lld samples (got %lld); use a context's ppo_permutation",
                (long long)STATIC_PERM_MAX_S, (long long)S);
  if (S == 0) return PPO_OK;
  if (!d_perm) return fail(nullptr, PPO_EINVAL, "d_perm is NULL");
  int32_t* ws = nullptr;
  {
    const hipError_t e = static_scratch(&ws);
    if (e != hipSuccess) return fail(nullptr, PPO_EHIP, "address of the static scratch array: %s", hipGetErrorString(e));
  }
  // the bucket count of ppo_create (about 32 keys per bucket), so both entry points run the same kernels on the same grids
  int nb = 1, lg = 0;
  while ((int64_t)nb * 32 < S && nb < STATIC_PERM_MAX_NB) { nb <<= 1; ++lg; }
  const int shift = 64 - lg;
  int32_t* hist = ws;                  // [2 * nb]: counts, then scatter cursors
  int32_t* start = ws + 2 * (int64_t)STATIC_PERM_MAX_NB;  // [nb]
  int32_t* tmp = ws + 3 * (int64_t)STATIC_PERM_MAX_NB;    // [S]
  hipStream_t st = (hipStream_t)hip_stream;
  PermStreams ps;
  for (int e = 0; e < PERM_BATCH; ++e) ps.s[e] = perm_stream(seed, update_idx, epoch);
  if (S <= PERM_SMALL) {
    const hipError_t e = launch_perm_small(ps, (int)S, 1, d_perm, st);
    return e == hipSuccess ? PPO_OK : fail(nullptr, PPO_EHIP, "launch of k_perm_small failed: %s", hipGetErrorString(e));
  }
  const int g = cdiv(S, 256), Si = (int)S;
  // the array keeps the last call's contents: counts and cursors must start at zero (a fill kernel, so that a
  // caller may record this call into a graph); start and tmp are fully overwritten before they are read
  hipLaunchKernelGGL(k_fill_i32, dim3(cdiv((int64_t)2 * nb, 256)), dim3(256), 0, st, hist, (int64_t)2 * nb, 0);
  hipLaunchKernelGGL(k_perm_hist, dim3(g, 1), dim3(256), 0, st, ps, Si, shift, nb, hist);
  hipLaunchKernelGGL(k_perm_scan, dim3(1, 1), dim3(1024), 0, st, hist, start, nb);
  hipLaunchKernelGGL(k_perm_scatter, dim3(g, 1), dim3(256), 0, st, ps, Si, shift, nb, start, hist, tmp);
  hipLaunchKernelGGL(k_perm_rank, dim3(g, 1), dim3(256), 0, st, ps, Si, shift, nb, start, hist, tmp, d_perm);
  LAUNCHCHK(nullptr, "permutation kernels");
  return PPO_OK;
}

int ppo_update(ppo_ctx* c, const ppo_hparams* hp, ppo_mb_stats* host_stats) {
  if (!c) return PPO_EINVAL;
  if (!c->d.has_value_head) return fail(c, PPO_ESTATE, "ppo_update needs a value head; use distill_update for a student");
  int rc = validate_hp(c, hp, false);
  if (rc) return rc;
  if (!c->gae_done) return fail(c, PPO_ESTATE, "ppo_update needs ppo_gae on the current rollout");
  return run_update(c, hp, host_stats, false);
}

int distill_update(ppo_ctx* c, const ppo_hparams* hp, ppo_mb_stats* host_stats) {
  if (!c) return PPO_EINVAL;
  if (c->d.has_value_head) return fail(c, PPO_ESTATE, "distill_update needs a student context (has_value_head = 0)");
  int rc = validate_hp(c, hp, true);
  if (rc) return rc;
  if (!all_written(c)) return fail(c, PPO_ESTATE, "distill_update needs all %d steps written", c->T);
  return run_update(c, hp, host_stats, true);
}

__global__ void k_copy_heads(int n, int A, int has_v, const float* __restrict__ out, float* __restrict__ mu, float* __restrict__ v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)n * HEAD_LD) return;
  int b = (int)(i / HEAD_LD), j = (int)(i - (int64_t)b * HEAD_LD);
  if (j < A) mu[(int64_t)b * A + j] = out[i];
  else if (j == A && has_v && v) v[b] = out[i];
}

int ppo_forward(ppo_ctx* c, const int32_t* d_idx, int64_t count, float* d_mu, float* d_v) {
  if (!c) return PPO_EINVAL;
  if (!d_mu) return fail(c, PPO_EINVAL, "d_mu is NULL");
  if (count < 0 || (!d_idx && count > c->S)) return fail(c, PPO_EINVAL, "count out of range");
  if (c->nl > 0) return fail(c, PPO_ESTATE, "ppo_forward treats samples independently: not available for a recurrent net");
  if (!all_written(c)) return fail(c, PPO_ESTATE, "ppo_forward needs all %d steps written", c->T);
  for (int64_t c0 = 0; c0 < count; c0 += c->CH) {
    int n = (int)((count - c0 < c->CH) ? count - c0 : c->CH);
    const int32_t* idx = d_idx ? d_idx + c0 : nullptr;
    const bool fused = head_act_covers(c);
    int rc = forward_chunk(c, idx, n, false, !fused, c0);  // without indices: samples c0 .. c0 + n - 1
    if (rc) return rc;
    if (fused) {
      HeadActArgs a = {};
      a.c_action = d_mu + c0 * c->A; a.c_value = d_v ? d_v + c0 : nullptr;
      rc = launch_head_act(c, a, n);
      if (rc) return rc;
      continue;
    }
    hipLaunchKernelGGL(k_copy_heads, dim3(cdiv((int64_t)n * HEAD_LD, 256)), dim3(256), 0, c->stream, n, c->A, c->d.has_value_head, c->headout,
                       d_mu + c0 * c->A, d_v ? d_v + c0 : nullptr);
    LAUNCHCHK(c, "k_copy_heads");
  }
  return PPO_OK;
}

int ppo_act(ppo_ctx* c, int32_t t, const void* d_obs, const float* d_proprio, const float* d_noise, float* d_action, float* d_logp,
            float* d_value) {
  if (!c) return PPO_EINVAL;
  if (!c->d.has_value_head) return fail(c, PPO_ESTATE, "ppo_act needs an actor-critic context (has_value_head = 1)");
  if (c->nl > 0) return fail(c, PPO_ESTATE, "ppo_act keeps no recurrent state between calls: not available for a recurrent net");
  if (t < 0 || t >= c->T) return fail(c, PPO_EINVAL, "t = %d outside [0, %d)", t, c->T);
  if (!d_obs || !d_proprio || !d_noise) return fail(c, PPO_EINVAL, "d_obs, d_proprio and d_noise must not be NULL");
  const int64_t first = (int64_t)t * c->N;
  // One kernel reads a sample's observations while another sample's outputs are already written: a caller who takes the outputs
  // into the memory of the observations gets the separate launches.
  auto overlap = [&](const void* out, int64_t n) {
    const uintptr_t o = reinterpret_cast<uintptr_t>(out), b = reinterpret_cast<uintptr_t>(d_obs), p = reinterpret_cast<uintptr_t>(d_proprio);
    const uintptr_t on = (uintptr_t)(n * 4), bn = (uintptr_t)((int64_t)c->N * c->V * c->d.in_c * c->d.in_h * c->d.in_w * (c->d.obs_dtype == 0 ? 4 : 2)), pn = (uintptr_t)((int64_t)c->N * c->P * 4);
    return out && ((o < b + bn && b < o + on) || (o < p + pn && p < o + on));
  };
  const bool one = head_act_covers(c) && c->N <= c->CH && small_net_covers(c, c->N) && !overlap(d_action, (int64_t)c->N * c->A) && !overlap(d_logp, c->N) &&
                   !overlap(d_value, c->N);
  int rc = PPO_OK;
  if (one) {
    SmallNetArgs a = {};
    a.cs = conv_small_args(c, nullptr, c->N, first); a.cs.P = c->P;
    a.src = d_obs; a.psrc = d_proprio; a.slab = c->obs + first * c->img_elems; a.pslab = c->proprio + first * c->P; a.W0 = c->d.in_w; a.n = c->N;
    HeadActArgs& h = a.head;
    h.w = c->shadow + c->headW; h.bias = c->p + c->headB; h.n = c->N; h.A = c->A; h.NH = c->NH; h.logstd = c->p + c->logstd; h.noise = d_noise;
    h.o_action = c->action + first * c->A; h.o_logp = c->logp + first; h.o_value = c->value + first; h.c_action = d_action; h.c_logp = d_logp; h.c_value = d_value;
    ProfScope ps(c, "small_net_act", 2.0 * c->N * ((double)a.cs.Ho0 * a.cs.Wo0 * 72 + (double)a.cs.Ho1 * a.cs.Wo1 * 1152 + (double)c->fin[0] * c->fout[0]),
                 (double)c->N * (c->img_elems * (c->d.obs_dtype == 0 ? 6.0 : 4.0) + 6.0 * c->P + 12.0 * c->A + 16.0));
    rc = c->d.obs_dtype == 0 ? launch_small_net<float, true>(c, a) : launch_small_net<bf16_t, true>(c, a);
  } else rc = write_slab(c, t, 0, c->N, d_obs, d_proprio, nullptr, nullptr, nullptr, nullptr, nullptr);
  if (rc) return rc;
  if (t == 0) { c->written.assign((size_t)c->T, 0); c->cover.assign((size_t)c->T, {}); }
  c->written[(size_t)t] = 2;
  c->cover[(size_t)t].clear();
  c->gae_done = false;
  for (int64_t c0 = 0; !one && c0 < c->N; c0 += c->CH) {
    const int n = (int)((c->N - c0 < c->CH) ? c->N - c0 : c->CH);
    const bool fused = head_act_covers(c);
    rc = forward_chunk(c, nullptr, n, false, !fused, first + c0);
    if (rc) return rc;
    const int64_t s0 = first + c0;
    if (fused) {
      HeadActArgs a = {};
      a.logstd = c->p + c->logstd; a.noise = d_noise + c0 * c->A;
      a.o_action = c->action + s0 * c->A; a.o_logp = c->logp + s0; a.o_value = c->value + s0;
      a.c_action = d_action ? d_action + c0 * c->A : nullptr; a.c_logp = d_logp ? d_logp + c0 : nullptr; a.c_value = d_value ? d_value + c0 : nullptr;
      rc = launch_head_act(c, a, n);
      if (rc) return rc;
      continue;
    }
    ProfScope ps(c, "act_sample", 0.0, (double)n * (4.0 * HEAD_LD + 12.0 * c->A + 8.0));
    hipLaunchKernelGGL(k_act_sample, dim3(cdiv(n, 64)), dim3(64), 0, c->stream, n, c->A, c->headout, c->p + c->logstd, d_noise + c0 * c->A,
                       c->action + s0 * c->A, c->logp + s0, c->value + s0, d_action ? d_action + c0 * c->A : nullptr,
                       d_logp ? d_logp + c0 : nullptr, d_value ? d_value + c0 : nullptr);
    LAUNCHCHK(c, "k_act_sample");
  }
  return PPO_OK;
}

int ppo_buffer_write_outcome(ppo_ctx* c, int32_t t, const float* d_reward, const uint8_t* d_done) {
  if (!c) return PPO_EINVAL;
  if (t < 0 || t >= c->T) return fail(c, PPO_EINVAL, "t = %d outside [0, %d)", t, c->T);
  if (!d_reward || !d_done) return fail(c, PPO_EINVAL, "d_reward and d_done must not be NULL");
  if (!c->written[(size_t)t]) return fail(c, PPO_ESTATE, "step %d holds no record yet (ppo_act or ppo_buffer_write first)", t);
  hipLaunchKernelGGL(k_write_outcome, dim3(cdiv(c->N, 256)), dim3(256), 0, c->stream, c->N, d_reward, d_done, c->reward + (int64_t)t * c->N,
                     c->done + (int64_t)t * c->N);
  LAUNCHCHK(c, "k_write_outcome");
  c->written[(size_t)t] = 1;
  c->gae_done = false;
  return PPO_OK;
}

int ppo_profile(ppo_ctx* c, int32_t enable) {
  if (!c) return PPO_EINVAL;
  (void)hipStreamSynchronize(c->stream);
  for (auto& r : c->prof_recs) { c->prof_pool.push_back(r.a); c->prof_pool.push_back(r.b); }
  c->prof_recs.clear(); c->prof_cls.clear(); c->prof_idx.clear();
  c->prof_on = enable != 0;
  return PPO_OK;
}

int64_t ppo_profile_report(ppo_ctx* c, char* buf, int64_t cap) {
  if (!c || !buf || cap < 1) return PPO_EINVAL;
  if (hipStreamSynchronize(c->stream) != hipSuccess) return fail(c, PPO_EHIP, "hipStreamSynchronize failed");
  std::vector<double> ms(c->prof_cls.size(), 0.0);
  for (auto& r : c->prof_recs) {
    float t = 0.f;
    if (hipEventElapsedTime(&t, r.a, r.b) == hipSuccess) ms[(size_t)r.cls] += t;
  }
  std::string out;
  char line[256];
  for (size_t i = 0; i < c->prof_cls.size(); ++i) {
    const auto& pc = c->prof_cls[i];
    snprintf(line, sizeof line, "%s %lld %.6f %.6e %.6e\n", pc.name.c_str(), (long long)pc.launches, ms[i], pc.flops, pc.bytes);
    out += line;
  }
  if ((int64_t)out.size() + 1 > cap) return fail(c, PPO_EINVAL, "report needs %zu bytes", out.size() + 1);
  memcpy(buf, out.c_str(), out.size() + 1);
  return (int64_t)out.size();
}

int ppo_diag_gemm(int32_t M, int32_t N, int32_t K, const float* h_a, const float* h_b, float* h_c) {
  if (!h_a || !h_b || !h_c || M < 1 || N < 1 || K < 8 || K % 8) return PPO_EINVAL;
  Ctx tmp;
  Ctx* c = &tmp;
  if (hipGetDevice(&c->dev) != hipSuccess || c->dev < 0 || c->dev >= 64) return fail(nullptr, PPO_EHIP, "no usable HIP device");
  float *da = nullptr, *db = nullptr, *dc = nullptr;
  bf16_t *ba = nullptr, *bb = nullptr;
  int rc = PPO_OK;
  auto body = [&]() -> int {
    DALLOC(c, da, (int64_t)M * K); DALLOC(c, db, (int64_t)N * K); DALLOC(c, dc, (int64_t)M * N);
    DALLOC(c, ba, (int64_t)M * K); DALLOC(c, bb, (int64_t)N * K);
    DALLOC(c, c->zpage, 32768);
    // room for split reductions; what would need more fills the chip undivided (1 GiB: 32 tiles of 256 x 128 for every CU)
    c->partial_elems = std::min<int64_t>((int64_t)8 * (M + 256) * (N + 128), 1 << 28) + 4;
    DALLOC(c, c->partial, c->partial_elems);
    HIPCHK(c, hipMemset(c->zpage, 0, 65536));
    HIPCHK(c, hipMemcpy(da, h_a, sizeof(float) * (size_t)M * K, hipMemcpyHostToDevice));
    HIPCHK(c, hipMemcpy(db, h_b, sizeof(float) * (size_t)N * K, hipMemcpyHostToDevice));
    hipLaunchKernelGGL(k_cast_bf16, dim3(cdiv((int64_t)M * K, 256)), dim3(256), 0, c->stream, da, ba, (int64_t)M * K);
    hipLaunchKernelGGL(k_cast_bf16, dim3(cdiv((int64_t)N * K, 256)), dim3(256), 0, c->stream, db, bb, (int64_t)N * K);
    LAUNCHCHK(c, "k_cast_bf16");
    ARows al = plain_arows(ba, K, M, K);
    Ep<MapRows, float, false, false, false> ep;
    ep.map = plain_map(N, M); ep.out = dc; ep.bias = nullptr; ep.mask = nullptr; ep.N = N;
    int r = launch_gemm(c, al, M, bb, K, N, K, ep, "diag_gemm", 0.0);
    if (r) return r;
    HIPCHK(c, hipDeviceSynchronize());
    HIPCHK(c, hipMemcpy(h_c, dc, sizeof(float) * (size_t)M * N, hipMemcpyDeviceToHost));
    return PPO_OK;
  };
  rc = body();
  if (rc) g_create_error = c->err;
  free_all(c);
  return rc;
}

int ppo_diag_peak(int32_t kind, int64_t nbytes, int32_t iters, float* h_result) {
  if (!h_result || kind < PEAK_COPY || kind > PEAK_MFMA_VALU || iters < 1 || iters > 100000) return fail(nullptr, PPO_EINVAL, "ppo_diag_peak: bad argument");
  const bool streams = kind != PEAK_MFMA && kind != PEAK_MFMA_VALU;
  if (streams && (nbytes < (1 << 20) || nbytes > (16LL << 30) || nbytes % 16)) return fail(nullptr, PPO_EINVAL, "ppo_diag_peak: nbytes must be a multiple of 16 in [1 MiB, 16 GiB]");
  if (kind == PEAK_MFMA_VALU && (nbytes < 0 || nbytes > 8)) return fail(nullptr, PPO_EINVAL, "ppo_diag_peak: kind 5 takes the number of vector instructions per MFMA (0..8) in nbytes");
  Ctx tmp;
  Ctx* c = &tmp;
  auto body = [&]() -> int {
    uint4 *src = nullptr, *dst = nullptr;
    float* sink = nullptr;
    hipEvent_t e0, e1;
    DALLOC(c, sink, 4);
    const int64_t n16 = nbytes / 16;
    if (streams) {
      DALLOC(c, src, n16); DALLOC(c, dst, n16);
      HIPCHK(c, hipMemset(src, 0, (size_t)nbytes));
      HIPCHK(c, hipMemset(dst, 0, (size_t)nbytes));
    }
    HIPCHK(c, hipEventCreate(&e0)); HIPCHK(c, hipEventCreate(&e1));
    const int mfma_rounds = 4096;
    auto launch = [&]() {
      const dim3 grid(256 * 16), blk(256);
      switch (kind) {
        case PEAK_COPY: hipLaunchKernelGGL(k_peak_stream<PEAK_COPY>, grid, blk, 0, nullptr, src, dst, n16, (uint32_t*)sink); break;
        case PEAK_READ: hipLaunchKernelGGL(k_peak_stream<PEAK_READ>, grid, blk, 0, nullptr, src, dst, n16, (uint32_t*)sink); break;
        case PEAK_WRITE: hipLaunchKernelGGL(k_peak_stream<PEAK_WRITE>, grid, blk, 0, nullptr, src, dst, n16, (uint32_t*)sink); break;
        case PEAK_COPY_NT: hipLaunchKernelGGL(k_peak_stream<PEAK_COPY_NT>, grid, blk, 0, nullptr, src, dst, n16, (uint32_t*)sink); break;
        case PEAK_MFMA: hipLaunchKernelGGL(k_peak_mfma, dim3(256 * 2), dim3(512), 0, nullptr, mfma_rounds, sink); break;
        default:
          switch ((int)nbytes) {
#define PEAK_MV(K_) case K_: hipLaunchKernelGGL(k_peak_mfma_valu<K_>, dim3(256), dim3(512), 0, nullptr, mfma_rounds, sink); break;
            PEAK_MV(0) PEAK_MV(1) PEAK_MV(2) PEAK_MV(3) PEAK_MV(4) PEAK_MV(5) PEAK_MV(6) PEAK_MV(7) PEAK_MV(8)
#undef PEAK_MV
          }
          break;
      }
    };
    for (int i = 0; i < 2; ++i) launch();
    LAUNCHCHK(c, "peak kernel");
    HIPCHK(c, hipEventRecord(e0, nullptr));
    for (int i = 0; i < iters; ++i) launch();
    HIPCHK(c, hipEventRecord(e1, nullptr));
    HIPCHK(c, hipEventSynchronize(e1));
    LAUNCHCHK(c, "peak kernel");
    float ms = 0.f;
    HIPCHK(c, hipEventElapsedTime(&ms, e0, e1));
    (void)hipEventDestroy(e0); (void)hipEventDestroy(e1);
    const double sec = (double)ms * 1e-3 / iters;
    if (kind == PEAK_MFMA) *h_result = (float)(256.0 * 2 * 8 * mfma_rounds * 4 * 32768.0 / sec / 1e12);   // TFLOP/s
    else if (kind == PEAK_MFMA_VALU) *h_result = (float)(256.0 * 8 * mfma_rounds * 8 * 16384.0 / sec / 1e12);  // TFLOP/s of the MFMAs: 256 blocks of 8 waves
    else *h_result = (float)((kind == PEAK_COPY || kind == PEAK_COPY_NT ? 2.0 : 1.0) * (double)nbytes / sec / 1e9);  // GB/s
    return PPO_OK;
  };
  const int rc = body();
  if (rc) g_create_error = c->err;
  free_all(c);
  return rc;
}

}  // extern "C"
