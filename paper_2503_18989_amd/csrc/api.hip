// Host side of the middle-submodel library: configuration, workspace carving,
// the integer planner of a step (positions, page table, attention work lists)
// and the launch sequence of the decoder layers.  Interface and semantics are
// documented in include/hat_mid.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <set>
#include <string>
#include <vector>

#include "../../include/hat_mid.h"
#include "hat_kernels.h"
#include "hat_layout.h"

// ---- static scratch of hat_mid_kv_export_static -------------------------------------------------
// Page ids of the rows being exported, staged here instead of in the caller's workspace.  One copy
// of the array exists on every GPU the library is loaded on (16 KB each, held until the process
// ends).  In host code the array's NAME is only a handle for hipGetSymbolAddress: the address a
// kernel may use is the one that call returns, taken once per device with that device current.
constexpr int kStaticPageIds = 4096;   // 4096 pages = 65 536 cache rows per call
static __device__ __align__(256) int32_t scratch[kStaticPageIds];

namespace {

constexpr int kMaxGpus = 64;
std::mutex g_scratch_mu;
int32_t* g_scratch_ptr[kMaxGpus] = {};   // device address of `scratch` on each GPU (nullptr: not taken yet)

// Address of the current device's copy of `scratch`, taken on first use on that device.
hipError_t static_scratch(int device, int32_t** out) {
  if (device < 0 || device >= kMaxGpus) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[device]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[device] = (int32_t*)p;
  }
  *out = g_scratch_ptr[device];
  return hipSuccess;
}

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
inline int round_up(int x, int a) { return (x + a - 1) / a * a; }

constexpr int kCapAttnTarget = 2048;  // workgroup target that the work-list capacities are sized for
constexpr int kAttnTarget = 256;      // one 8-wave workgroup per CU

struct LayerDev {
  act_t *wqkv, *wo, *wgu, *wd;
  float *g_attn, *g_ffn;
};

struct Shapes {
  int L, d, H, hd, F, Fpad;
  int Nqkv, No, Ngu, Nd;  // padded weight rows
  int Tcap;               // row capacity of activation buffers (multiple of 256)
  int attn_target;        // workgroups a chunk-attention launch should reach
  int verify_target;      // workgroups a verify-attention launch should reach
  int chunk_items_cap, chunk_blocks_cap, verify_items_cap, merge_cap;
  int part_rows_cap;
  int part32_cap;         // fp32 partial rows (chunk items that stream the cache); their numbers follow those of the part_rows_cap others
  int gemm_part_rows;     // rows of the split-K partial-sum buffer
  size_t plan_words;
};

bool valid_cfg(const hat_mid_config_t* c) {
  if (!c) return false;
  if (c->n_layers <= 0 || c->n_heads <= 0 || c->d_ffn <= 0) return false;
  if (c->head_dim != 64 && c->head_dim != 128) return false;
  if (c->d_model != c->n_heads * c->head_dim || c->d_model % 64 != 0 || c->d_model > 8192) return false;
  if (c->page_size != HAT_PAGE_SIZE || c->n_pages <= 0) return false;
  if (c->max_devices <= 0 || c->max_step_tokens <= 0 || c->max_pos <= 0) return false;
  if (c->io_dtype != HAT_BF16 && c->io_dtype != HAT_F32) return false;
  if (c->kv_dtype != HAT_KV_BF16 && c->kv_dtype != HAT_KV_F16) return false;
  if (!(c->rms_eps > 0.f) || !(c->rope_theta > 0.f)) return false;
  return true;
}

Shapes make_shapes(const hat_mid_config_t& c) {
  Shapes s;
  s.L = c.n_layers; s.d = c.d_model; s.H = c.n_heads; s.hd = c.head_dim; s.F = c.d_ffn;
  s.Fpad = round_up(c.d_ffn, 64);
  s.Nqkv = round_up(3 * s.d, 256);
  s.No = round_up(s.d, 256);
  s.Ngu = round_up(2 * s.Fpad, 256);
  s.Nd = round_up(s.d, 256);
  s.Tcap = round_up(c.max_step_tokens, 256);
  s.attn_target = kAttnTarget;
  s.verify_target = 2048;
  // capacities are sized for this target; a larger one (hat_mid_debug_set_attn_targets) splits
  // only as far as they allow -- the planner checks every capacity before it splits
  const int per_head = (kCapAttnTarget + s.H - 1) / s.H;
  s.chunk_items_cap = 2 * per_head + s.Tcap / 128 + c.max_devices + 2;
  // row blocks of the chunk items that stream the cache: every key range once more, in launches that stay within a workgroup per CU
  s.chunk_blocks_cap = s.Tcap / HAT_NARROW_QROWS + c.max_devices + 256;
  s.verify_items_cap = 2 * per_head + c.max_devices + 2;
  s.merge_cap = s.Tcap / 16 + s.Tcap / 128 + 2 * c.max_devices + 2;
  // n narrow items wanted: key ranges of sum / n keys leave fewer than 2 n + 1 ranges in the items that have more than one
  s.part32_cap = HAT_NARROW_QROWS * (2 * (per_head * 3 / 8) + 2);
  s.part_rows_cap = HAT_CHUNK_QROWS * (2 * per_head + 2) + HAT_MAX_VERIFY * s.verify_items_cap;
  s.gemm_part_rows = 4096;
  s.plan_words = (size_t)3 * s.Tcap + 8 * ((size_t)s.Tcap / 16 + 2 * (size_t)c.max_devices + 2) + 8 * (size_t)c.max_devices + 16 + (size_t)c.n_pages + c.max_devices +
                 12 * ((size_t)s.chunk_items_cap + s.chunk_blocks_cap + s.verify_items_cap) + 8 * (size_t)s.merge_cap + 64;
  return s;
}

// carve the workspace; with base == nullptr only sizes are computed
struct Carver {
  unsigned char* base;
  size_t off = 0;
  explicit Carver(void* b) : base((unsigned char*)b) {}
  template <class T>
  T* take(size_t n) {
    off = align_up(off, 256);
    T* p = base ? (T*)(base + off) : nullptr;
    off += n * sizeof(T);
    return p;
  }
};

struct Buffers {
  std::vector<LayerDev> layers;
  double* inv_freq;
  float* resid;
  act_t *xn, *xn2, *qkv, *attn, *act;
  float2* table;
  act_t* part_o;
  float* part_o32;
  float2* part_ml;
  float* gemm_part;
  int32_t* plan_dev;
  int32_t* fixture_pages;
  float* stage_in[2];
  float* stage_out;
};

size_t carve(const hat_mid_config_t& c, const Shapes& s, void* base, Buffers* out) {
  Carver cv(base);
  Buffers b;
  b.layers.resize(s.L);
  for (int l = 0; l < s.L; ++l) {
    b.layers[l].wqkv = cv.take<act_t>((size_t)s.Nqkv * s.d);
    b.layers[l].wo = cv.take<act_t>((size_t)s.No * s.d);
    b.layers[l].wgu = cv.take<act_t>((size_t)s.Ngu * s.d);
    b.layers[l].wd = cv.take<act_t>((size_t)s.Nd * s.Fpad);
    b.layers[l].g_attn = cv.take<float>(s.d);
    b.layers[l].g_ffn = cv.take<float>(s.d);
  }
  b.inv_freq = cv.take<double>(s.hd / 2);
  b.resid = cv.take<float>((size_t)s.Tcap * s.d);
  b.xn = cv.take<act_t>((size_t)s.Tcap * s.d);
  b.xn2 = cv.take<act_t>((size_t)s.Tcap * s.d);
  b.qkv = cv.take<act_t>((size_t)s.Tcap * 3 * s.d);
  b.attn = cv.take<act_t>((size_t)s.Tcap * s.d);
  b.act = cv.take<act_t>((size_t)s.Tcap * s.Fpad);
  b.table = cv.take<float2>((size_t)s.Tcap * (s.hd / 2));
  b.part_o = cv.take<act_t>((size_t)s.part_rows_cap * s.d);
  b.part_o32 = cv.take<float>((size_t)s.part32_cap * s.d);
  b.part_ml = cv.take<float2>((size_t)(s.part_rows_cap + s.part32_cap) * s.H);
  b.gemm_part = cv.take<float>((size_t)s.gemm_part_rows * s.d);
  b.plan_dev = cv.take<int32_t>(s.plan_words);
  b.fixture_pages = cv.take<int32_t>((size_t)(c.max_pos + 15) / 16 + 2);
  // staging for steps whose hidden states live in host memory: two input slots (the upload of the
  // next step overlaps the current one) and one output slot, sized for fp32 rows
  b.stage_in[0] = cv.take<float>((size_t)s.Tcap * s.d);
  b.stage_in[1] = cv.take<float>((size_t)s.Tcap * s.d);
  b.stage_out = cv.take<float>((size_t)s.Tcap * s.d);
  if (out) *out = b;
  return align_up(cv.off, 256);
}

struct DeviceState {
  int len = 0;
  std::vector<int32_t> pages;
};

constexpr int kPlanBufs = 3;

}  // namespace

struct hat_mid {
  hat_mid_config_t cfg;
  Shapes s;
  Buffers b;
  kv_t* pool;
  size_t layer_pool_elems;

  std::set<int32_t> free_pages;
  std::vector<DeviceState> dev;

  int32_t* plan_host[kPlanBufs] = {nullptr, nullptr, nullptr};
  hipEvent_t plan_ev[kPlanBufs] = {nullptr, nullptr, nullptr};
  bool plan_ev_used[kPlanBufs] = {false, false, false};
  int plan_next = 0;

  hipEvent_t ev_begin = nullptr, ev_end = nullptr;
  bool have_step = false;
  int last_tokens = 0;

  bool profiling = false;
  struct Rec { int id; hipEvent_t a, b; };
  std::vector<Rec> recs;
  std::vector<hipEvent_t> ev_pool;

  // steps fed from host memory (hat_mid_forward_host)
  hipStream_t copy_stream = nullptr;
  hipEvent_t up_done[2] = {nullptr, nullptr}, slot_free[2] = {nullptr, nullptr};
  bool slot_used[2] = {false, false};
  int host_slot = 0;

  // what the step being planned has done to the page state, so that a failure after the pages
  // moved (plan capacity, a HIP call while enqueueing) can put everything back
  struct PageOp { int32_t page; bool taken; };   // taken: the page left the free set; else it entered it
  std::vector<PageOp> undo_pages;
  std::vector<std::pair<int32_t, DeviceState>> undo_dev;
  bool undo_on = false;

  // hat_mid_kv_export_static: this GPU's copy of the static scratch array, a pinned host buffer for
  // the page ids on their way there, and the event that says the last upload has read it
  int device = -1;
  int32_t* static_pages_dev = nullptr;
  int32_t* static_pages_host = nullptr;
  hipEvent_t static_ev = nullptr;
  bool static_ev_used = false;

  hipStream_t last_stream = nullptr;       // stream of the most recent enqueue (hat_mid_destroy waits for it)
  bool used_stream = false;
  size_t plan_limit = 0;                   // > 0: lowered plan capacity (hat_mid_debug_limit_plan)
  bool verify_probe = false;               // verify attention replaced by its loads-only twin (hat_mid_debug_set_verify_probe)

  bool host_only = false;                  // built by hat_mid_debug_create_host_only: no GPU memory, no HIP calls
  std::vector<int32_t> host_plan;          // its plan words
  int host_narrow = 0;                     // StepPlan::n_narrow of its last plan
  size_t host_blocks = 0;                  // StepPlan::o_cb
  int host_n_blocks = 0, host_block_waves = 0;   // n_cblocks and block_waves of it
  bool host_along = false, host_ring = false;
  int force_tile[4] = {-1, -1, -1, -1};   // tuning overrides per GEMM class (qkv, o, gate/up, down)
  int force_ksplit[4] = {0, 0, 0, 0};

  std::string err;
};

namespace {

hat_status_t fail(hat_mid* h, hat_status_t st, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  if (h) h->err = buf;
  return st;
}

#define HIP_TRY(h, expr)                                                                          \
  do {                                                                                            \
    hipError_t e_ = (expr);                                                                       \
    if (e_ != hipSuccess) return fail(h, HAT_EHIP, "%s failed: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

// node i sees itself and nothing later; its ancestors are one path (each ancestor's own mask is
// the ancestors before it plus itself)
bool valid_tree(const uint8_t* m, int n) {
  for (int i = 0; i < n; ++i) {
    if ((m[i] >> i) != 1) return false;
    unsigned path = 0;
    for (int j = 0; j < i; ++j) {
      if (!((m[i] >> j) & 1)) continue;
      if (m[j] != (path | (1u << j))) return false;
      path |= 1u << j;
    }
  }
  return true;
}

int32_t take_lowest(hat_mid* h) {
  auto it = h->free_pages.begin();
  int32_t id = *it;
  h->free_pages.erase(it);
  if (h->undo_on) h->undo_pages.push_back({id, true});
  return id;
}

void give_back(hat_mid* h, int32_t id) {
  h->free_pages.insert(id);
  if (h->undo_on) h->undo_pages.push_back({id, false});
}

// Page movements of one call are logged between undo_begin and undo_commit; undo_rollback puts
// lengths, page lists and the free set back to what they were at undo_begin.
void undo_begin(hat_mid* h) {
  h->undo_pages.clear();
  h->undo_dev.clear();
  h->undo_on = true;
}
void undo_save_device(hat_mid* h, int32_t id) { h->undo_dev.emplace_back(id, h->dev[id]); }
void undo_commit(hat_mid* h) {
  h->undo_on = false;
  h->undo_pages.clear();
  h->undo_dev.clear();
}
void undo_rollback(hat_mid* h) {
  h->undo_on = false;
  for (auto it = h->undo_pages.rbegin(); it != h->undo_pages.rend(); ++it) {
    if (it->taken) h->free_pages.insert(it->page);
    else h->free_pages.erase(it->page);
  }
  for (auto it = h->undo_dev.rbegin(); it != h->undo_dev.rend(); ++it) h->dev[it->first] = std::move(it->second);
  h->undo_pages.clear();
  h->undo_dev.clear();
}

void note_stream(hat_mid* h, hipStream_t st) {
  h->last_stream = st;
  h->used_stream = true;
}

hipEvent_t get_event(hat_mid* h) {
  if (!h->ev_pool.empty()) {
    hipEvent_t e = h->ev_pool.back();
    h->ev_pool.pop_back();
    return e;
  }
  hipEvent_t e;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}

// brackets one launch with events when profiling is on
struct Timed {
  hat_mid* h;
  hipStream_t st;
  int id;
  hipEvent_t a = nullptr, b = nullptr;
  Timed(hat_mid* h_, hipStream_t st_, int id_) : h(h_), st(st_), id(id_) {
    if (h->profiling) {
      a = get_event(h);
      b = get_event(h);
      if (a) (void)hipEventRecord(a, st);
    }
  }
  ~Timed() {
    if (h->profiling && a && b) {
      (void)hipEventRecord(b, st);
      h->recs.push_back({id, a, b});
    }
  }
};

#define LAUNCH(h, st, id, call)                                                                      \
  do {                                                                                               \
    hipError_t e_;                                                                                   \
    {                                                                                                \
      Timed t_(h, st, id);                                                                           \
      e_ = (call);                                                                                   \
    }                                                                                                \
    if (e_ != hipSuccess) return fail(h, HAT_EHIP, "%s failed: %s", #call, hipGetErrorString(e_));   \
  } while (0)

}  // namespace

extern "C" {

size_t hat_mid_kv_bytes(const hat_mid_config_t* cfg) {
  if (!valid_cfg(cfg)) return 0;
  return (size_t)cfg->n_layers * cfg->n_pages * kv_page_elems(cfg->n_heads, cfg->head_dim) * sizeof(kv_t);
}

size_t hat_mid_workspace_bytes(const hat_mid_config_t* cfg) {
  if (!valid_cfg(cfg)) return 0;
  Shapes s = make_shapes(*cfg);
  return carve(*cfg, s, nullptr, nullptr);
}

static hat_status_t create_impl(const hat_mid_config_t* cfg, const hat_mid_layer_weights_t* layers, void* kv_pool,
                                void* workspace, void* hip_stream, hat_mid_t** out) {
  if (out) *out = nullptr;
  if (!out || !valid_cfg(cfg) || !layers || !kv_pool || !workspace) return HAT_EINVAL;
  if (((uintptr_t)kv_pool | (uintptr_t)workspace) & 255) return HAT_EINVAL;
  for (int l = 0; l < cfg->n_layers; ++l) {
    const hat_mid_layer_weights_t& w = layers[l];
    if (!w.attn_norm || !w.wq || !w.wk || !w.wv || !w.wo || !w.ffn_norm || !w.w_gate || !w.w_up || !w.w_down)
      return HAT_EINVAL;
  }
  hipStream_t st = (hipStream_t)hip_stream;
  hat_mid* h = new hat_mid();
  h->cfg = *cfg;
  h->s = make_shapes(*cfg);
  carve(*cfg, h->s, workspace, &h->b);
  h->pool = (kv_t*)kv_pool;
  h->layer_pool_elems = (size_t)cfg->n_pages * kv_page_elems(cfg->n_heads, cfg->head_dim);
  for (int i = 0; i < cfg->n_pages; ++i) h->free_pages.insert(i);
  h->dev.resize(cfg->max_devices);

  auto bail = [&](hipError_t e, const char* what) {
    fprintf(stderr, "hat_mid_create: %s: %s\n", what, hipGetErrorString(e));
    hat_mid_destroy(h);
    return HAT_EHIP;
  };
  hipError_t e;
  if ((e = hat_gemm_init()) != hipSuccess) return bail(e, "gemm init");
  for (int i = 0; i < kPlanBufs; ++i) {
    if ((e = hipHostMalloc((void**)&h->plan_host[i], h->s.plan_words * sizeof(int32_t), hipHostMallocDefault)) !=
        hipSuccess)
      return bail(e, "pinned plan buffer");
    if ((e = hipEventCreateWithFlags(&h->plan_ev[i], hipEventDisableTiming)) != hipSuccess) return bail(e, "event");
  }
  if ((e = hipGetDevice(&h->device)) != hipSuccess) return bail(e, "current device");
  if ((e = static_scratch(h->device, &h->static_pages_dev)) != hipSuccess) return bail(e, "address of the static scratch array");
  if ((e = hipHostMalloc((void**)&h->static_pages_host, kStaticPageIds * sizeof(int32_t), hipHostMallocDefault)) != hipSuccess)
    return bail(e, "pinned page-id buffer");
  if ((e = hipEventCreateWithFlags(&h->static_ev, hipEventDisableTiming)) != hipSuccess) return bail(e, "event");
  if ((e = hipStreamCreateWithFlags(&h->copy_stream, hipStreamNonBlocking)) != hipSuccess) return bail(e, "copy stream");
  for (int i = 0; i < 2; ++i) {
    if ((e = hipEventCreateWithFlags(&h->up_done[i], hipEventDisableTiming)) != hipSuccess) return bail(e, "event");
    if ((e = hipEventCreateWithFlags(&h->slot_free[i], hipEventDisableTiming)) != hipSuccess) return bail(e, "event");
  }
  if ((e = hipEventCreate(&h->ev_begin)) != hipSuccess) return bail(e, "event");
  if ((e = hipEventCreate(&h->ev_end)) != hipSuccess) return bail(e, "event");

  // rotary frequencies theta^(-2i/hd), in double
  {
    std::vector<double> f(h->s.hd / 2);
    for (int i = 0; i < h->s.hd / 2; ++i) f[i] = std::pow((double)cfg->rope_theta, -2.0 * i / h->s.hd);
    if ((e = hipMemcpyAsync(h->b.inv_freq, f.data(), f.size() * sizeof(double), hipMemcpyHostToDevice, st)) !=
        hipSuccess)
      return bail(e, "inv_freq upload");
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return bail(e, "sync");
  }
  // weights -> P32 tiles
  const Shapes& s = h->s;
  for (int l = 0; l < s.L; ++l) {
    const hat_mid_layer_weights_t& w = layers[l];
    LayerDev& ld = h->b.layers[l];
    if ((e = hat_launch_retile(ld.wqkv, s.Nqkv, s.d, (const bf16_t*)w.wq, (const bf16_t*)w.wk, (const bf16_t*)w.wv,
                               s.d, s.d, s.hd == 64 ? HAT_RETILE_QKV64 : HAT_RETILE_QKV128, st)) != hipSuccess)
      return bail(e, "retile qkv");
    if ((e = hat_launch_retile(ld.wo, s.No, s.d, (const bf16_t*)w.wo, nullptr, nullptr, s.d, s.d, 0, st)) !=
        hipSuccess)
      return bail(e, "retile o");
    if ((e = hat_launch_retile(ld.wgu, s.Ngu, s.d, (const bf16_t*)w.w_gate, (const bf16_t*)w.w_up, nullptr, s.F, s.d,
                               2, st)) != hipSuccess)
      return bail(e, "retile gate/up");
    if ((e = hat_launch_retile(ld.wd, s.Nd, s.Fpad, (const bf16_t*)w.w_down, nullptr, nullptr, s.d, s.F, 0, st)) !=
        hipSuccess)
      return bail(e, "retile down");
    if ((e = hat_launch_bf16_to_f32((const bf16_t*)w.attn_norm, ld.g_attn, s.d, st)) != hipSuccess)
      return bail(e, "gain");
    if ((e = hat_launch_bf16_to_f32((const bf16_t*)w.ffn_norm, ld.g_ffn, s.d, st)) != hipSuccess)
      return bail(e, "gain");
  }
  note_stream(h, st);
  *out = h;
  return HAT_OK;
}

void hat_mid_destroy(hat_mid_t* h) {
  if (!h) return;
  if (h->host_only) {
    delete h;
    return;
  }
  // wait for this handle's work only: its copy stream and the stream of its last enqueue (calls on
  // one handle are stream-ordered, so that covers all of them)
  if (h->copy_stream) (void)hipStreamSynchronize(h->copy_stream);
  if (h->used_stream) (void)hipStreamSynchronize(h->last_stream);
  for (int i = 0; i < kPlanBufs; ++i) {
    if (h->plan_host[i]) (void)hipHostFree(h->plan_host[i]);
    if (h->plan_ev[i]) (void)hipEventDestroy(h->plan_ev[i]);
  }
  if (h->ev_begin) (void)hipEventDestroy(h->ev_begin);
  if (h->ev_end) (void)hipEventDestroy(h->ev_end);
  if (h->static_ev) (void)hipEventDestroy(h->static_ev);
  if (h->static_pages_host) (void)hipHostFree(h->static_pages_host);
  for (int i = 0; i < 2; ++i) {
    if (h->up_done[i]) (void)hipEventDestroy(h->up_done[i]);
    if (h->slot_free[i]) (void)hipEventDestroy(h->slot_free[i]);
  }
  if (h->copy_stream) (void)hipStreamDestroy(h->copy_stream);
  for (auto& r : h->recs) {
    (void)hipEventDestroy(r.a);
    (void)hipEventDestroy(r.b);
  }
  for (auto e : h->ev_pool) (void)hipEventDestroy(e);
  delete h;
}

const char* hat_mid_last_error(const hat_mid_t* h) { return h ? h->err.c_str() : "null handle"; }

hat_status_t hat_mid_release(hat_mid_t* h, int32_t device_id) {
  if (!h) return HAT_EINVAL;
  if (device_id < 0 || device_id >= h->cfg.max_devices) return fail(h, HAT_EDEVICE, "device id %d out of range", device_id);
  DeviceState& d = h->dev[device_id];
  for (int32_t p : d.pages) h->free_pages.insert(p);
  d.pages.clear();
  d.len = 0;
  return HAT_OK;
}

hat_status_t hat_mid_kv_compact(hat_mid_t* h, int32_t device_id, int32_t base_pos, const int32_t* keep,
                                int32_t n_keep, void* hip_stream) {
  if (!h) return HAT_EINVAL;
  const hat_mid_config_t& c = h->cfg;
  if (device_id < 0 || device_id >= c.max_devices) return fail(h, HAT_EDEVICE, "device id %d out of range", device_id);
  if (base_pos < 0 || n_keep < 0 || n_keep > HAT_MAX_VERIFY || (n_keep > 0 && !keep))
    return fail(h, HAT_EINVAL, "bad compact arguments");
  for (int i = 0; i < n_keep; ++i)
    if (keep[i] < 0 || keep[i] >= HAT_MAX_VERIFY || (i > 0 && keep[i] <= keep[i - 1]))
      return fail(h, HAT_EINVAL, "kept nodes must be ascending indices below %d", HAT_MAX_VERIFY);
  DeviceState& d = h->dev[device_id];
  if (base_pos > d.len || (n_keep > 0 && base_pos + keep[n_keep - 1] >= d.len))
    return fail(h, HAT_EPOS, "kept row beyond cache length %d", d.len);
  HatRowMoves mv{};
  for (int i = 0; i < n_keep; ++i) {
    const int src = base_pos + keep[i], dst = base_pos + i;
    if (src == dst) continue;
    mv.src[mv.n] = d.pages[src >> 4] * 16 + (src & 15);
    mv.dst[mv.n] = d.pages[dst >> 4] * 16 + (dst & 15);
    ++mv.n;
  }
  if (!h->host_only) note_stream(h, (hipStream_t)hip_stream);
  if (!h->host_only)
    HIP_TRY(h, hat_launch_kv_move(h->pool, h->layer_pool_elems, c.n_layers, c.n_pages, mv, c.n_heads, c.head_dim,
                                  (hipStream_t)hip_stream));
  d.len = base_pos + n_keep;
  const size_t want = (size_t)(d.len + 15) / 16;
  while (d.pages.size() > want) {
    h->free_pages.insert(d.pages.back());
    d.pages.pop_back();
  }
  return HAT_OK;
}

hat_status_t hat_mid_kv_query(const hat_mid_t* h, int32_t device_id, int32_t* kv_len, int32_t* pages_out, int32_t cap,
                              int32_t* n_pages_out) {
  if (!h) return HAT_EINVAL;
  if (device_id < 0 || device_id >= h->cfg.max_devices) return HAT_EDEVICE;
  const DeviceState& d = h->dev[device_id];
  if (kv_len) *kv_len = d.len;
  if (n_pages_out) *n_pages_out = (int32_t)d.pages.size();
  if (pages_out)
    for (int i = 0; i < cap && i < (int)d.pages.size(); ++i) pages_out[i] = d.pages[i];
  return HAT_OK;
}

// What the planning half of a step hands to the enqueueing half: where each array lies in the
// plan words, and how many work items there are.
struct StepPlan {
  int T = 0, S = 0, n_append = 0;
  size_t o_pos = 0, o_dst = 0, o_tseg = 0, o_toff = 0, o_sstart = 0, o_spt = 0, o_in = 0, o_out = 0, o_pt = 0, o_app = 0;
  size_t o_ci = 0, o_cb = 0, o_vi = 0, o_mi = 0, words = 0;
  int n_citems = 0, n_narrow = 0, n_cblocks = 0, block_waves = 0, n_vitems = 0, n_mitems = 0;
  bool heads_inner = false, along = false, ring = false;
};

// Time in us of a launch of streamed row blocks with 8 or 4 waves each (the two template forms of attn_verify_kernel), `keys`
// the keys that each block reads, `mbytes` the cache rows that the launch reads at least once.  One workgroup of eight waves, or two (head dim 64:
// three) of four, are resident on a CU; a wave takes `step` for 32 keys, more as its CU fills, and a workgroup `block` beside them.  Fitted to
// 2500 mixes of one to sixteen chunks of 20 .. 1024 rows over 0 .. 6000 keys with six head counts (error 5 .. 6 % on average), most of all to their order.
// Eight waves shorten a workgroup, four get more out of a full CU and leave less of the chip idle in the last round.  us with 4 | 8
// (workgroups; bf16 cache): 1 x 64 rows over 4000 keys of the 7B shape 64.9 | 46.0 (64), 1 x 256 over 1000 24.1 | 20.4 (256), 13B shape 29.8 | 33.1
// (320), 8 x 64 over 4000 174 | 166 (640), 4 x 512 over 500 of the 7B shape 76.4 | 97.2 (2048), 4 x 128 over 2000 at head dim 64 34.0 | 36.1 (512).
// These are times of the kernel before it read page ids ahead, which took 3 .. 9 % off all of them, and verify items that go along are not counted.  With the present kernel the choice
// is 0.4 % of a layer behind the best of staged, eight and four waves over 90 other mixes (1 .. 12 chunks of 33 .. 500 rows over 0 .. 6000 keys; 2.8 % at the most, 302 + 355 rows over 5000 .. 5700 keys of the 7B
// shape), where always staging is 3.8, always eight waves 2.0 and always four 0.6 % behind it.
// `waves` = 2: items of at most 64 rows, a workgroup of attn_ring_kernel each (head dim 128, fp16 cache; each of its two computing waves goes through all keys). Fitted to 88 mixes of 3 .. 24
// such items (5.6 % off on average).
static double stream_us(const Shapes& s, int kv_f16, int waves, const std::vector<int>& keys, double mbytes) {
  struct Cost { double launch, block, step, shared, per_mb; };
  static const Cost k4[2][2] = {{{3.92, 3.30, 0.776, 0.005, 0.176}, {4.23, 2.70, 0.690, 0.005, 0.163}}, {{4.58, 4.44, 1.327, 0.357, 0.102}, {4.45, 3.65, 1.176, 0.437, 0.109}}};
  static const Cost k8[2][2] = {{{4.91, 2.00, 1.069, 0, 0.126}, {4.79, 2.01, 0.826, 0, 0.143}}, {{4.52, 3.87, 1.831, 0, 0.090}, {3.96, 3.64, 1.686, 0, 0.102}}};
  static const Cost pair = {0, 8.89, 0.403, 0.400, 0.055};
  const Cost& c = waves == 2 ? pair : (waves == 8 ? k8 : k4)[s.hd == 128][kv_f16 != 0];
  const double n = (double)keys.size() * s.H, slots = waves == 8 ? 256 : s.hd == 128 ? 512 : 768;
  std::vector<double> steps;
  for (int k : keys) steps.push_back(std::max(1.0, (double)((k + 31) / 32) / (waves == 2 ? 1 : waves)));
  std::sort(steps.begin(), steps.end());
  auto mean = [&](size_t shortest) {
    double sum = 0;
    for (size_t i = 0; i < shortest; ++i) sum += steps[i];
    return sum / shortest;
  };
  auto block_us = [&](double workgroups, double n_steps) {
    return c.block + n_steps * (c.step + (waves == 8 ? 0 : c.shared * std::sqrt(std::min(1.0, std::max(0.0, workgroups - 256) / (slots - 256)))));
  };
  const double rounds = n / slots, whole = std::floor(rounds), rest = rounds - whole, longest = block_us(n, steps.back()), avg = block_us(n, mean(steps.size()));
  double us = longest;
  if (waves == 8) us = std::max(us, avg * std::ceil(rounds));
  else if (rounds > 1) {   // the last round is one of the shortest blocks, with fewer workgroups to a CU
    const size_t shortest = std::max<size_t>(1, (size_t)std::lround(rest * slots / s.H));
    const double tail = rest > 0 ? std::pow(rest, 0.15) * block_us(rest * slots, mean(shortest)) : 0;
    us = std::max(us, std::max(avg * rounds, avg * whole + tail) + 0.225 * (longest - avg));
  }
  return c.launch + us + c.per_mb * mbytes;
}

// A chunk item and its key ranges (ns of `step` keys each).
struct ChunkCut {
  int seg, q0, nq, need, ns, step, part_row;
  bool narrow;   // in the launch of the narrow items
};

// keys that each row block of the streamed items reads
static std::vector<int> block_keys(const std::vector<ChunkCut>& cuts, const hat_mid_segment_t* segs) {
  std::vector<int> keys;
  for (const ChunkCut& u : cuts) {
    if (u.narrow) continue;
    for (int r0 = 0; r0 < u.nq; r0 += HAT_NARROW_QROWS) {
      const int need = segs[u.seg].start_pos + u.q0 + std::min(r0 + HAT_NARROW_QROWS, u.nq);
      for (int k = 0; k < u.ns; ++k) keys.push_back(std::max(0, std::min(need, (k + 1) * u.step) - k * u.step));
    }
  }
  return keys;
}

// Time in us of the same items staged (attn_chunk_kernel): a workgroup takes `block`, and for each 64 keys `stage` and `wave` for each of its waves with
// rows.  Fitted like stream_us, as is merge_us.  Over an fp16 cache attn_ring_kernel takes the items of more than a few keys; the constants are those of attn_chunk_kernel there, which takes
// 8 .. 12 % longer with them, so that a step near the line may stream where staging has become the faster way.
static double staged_us(const Shapes& s, int kv_f16, const std::vector<ChunkCut>& cuts, double mbytes) {
  struct Cost { double launch, block, stage, wave, per_mb; };
  static const Cost k[2][2] = {{{0.02, 7.82, 0.768, 0.071, 0.054}, {3.64, 3.86, 0.565, 0.080, 0.150}}, {{0, 9.81, 0.951, 0.124, 0.068}, {0, 9.11, 1.377, 0.105, 0.004}}};
  const Cost& c = k[s.hd == 128][kv_f16 != 0];
  double longest = 0, sum = 0;
  int n = 0;
  for (const ChunkCut& u : cuts) {
    if (u.narrow) continue;
    for (int i = 0; i < u.ns; ++i, ++n) {
      const double t = c.block + (std::min(u.step, u.need - i * u.step) + 63) / 64 * (c.stage + c.wave * ((u.nq + 31) / 32));
      longest = std::max(longest, t);
      sum += t;
    }
  }
  const double rounds = n * s.H / 256.0, whole = std::floor(rounds), avg = sum / n;
  double us = longest;
  if (rounds > 1) us = std::max(us, avg * std::max(rounds, whole + std::pow(rounds - whole, 0.2)) + 0.4 * (longest - avg));
  return c.launch + us + c.per_mb * mbytes;
}
static double merge_us(const Shapes& s, const std::vector<ChunkCut>& cuts, bool fp32, bool launched) {
  double rows = 0;
  for (const ChunkCut& u : cuts)
    if (!u.narrow && u.ns > 1) rows += u.ns * u.nq;
  if (rows == 0) return 0;
  return (launched ? 0.0 : fp32 ? 5.5 : 6.0) + (fp32 ? 1.1e-6 : 0.8e-6) * rows * s.d;
}

// Host half of a step: validates every segment, commits the page movements, and writes the plan
// (positions, write targets, page lists, attention work lists) into P (capacity: plan_words).
// No GPU call: the same code serves the host-only handles that the planner's CPU tests use.
static hat_status_t plan_step(hat_mid_t* h, const hat_mid_segment_t* segs, int32_t n_segs, int32_t* P, StepPlan* sp) {
  if (!segs || n_segs < 0) return fail(h, HAT_EINVAL, "no segments");
  const hat_mid_config_t& c = h->cfg;
  const Shapes& s = h->s;

  // ---- validate everything before touching state
  if (n_segs > c.max_devices) return fail(h, HAT_EINVAL, "more segments (%d) than devices", n_segs);
  std::vector<char> seen(c.max_devices, 0);
  long total = 0;
  for (int i = 0; i < n_segs; ++i) {
    const hat_mid_segment_t& g = segs[i];
    if (g.device_id < 0 || g.device_id >= c.max_devices)
      return fail(h, HAT_EDEVICE, "segment %d: device id %d out of range", i, g.device_id);
    if ((g.kind != HAT_SEG_CHUNK && g.kind != HAT_SEG_VERIFY) || g.n <= 0 || g.start_pos < 0)
      return fail(h, HAT_EINVAL, "segment %d: bad kind/n/start", i);
    if (g.kind == HAT_SEG_VERIFY && g.n > HAT_MAX_VERIFY)
      return fail(h, HAT_EINVAL, "segment %d: verify segment of %d rows (max %d)", i, g.n, HAT_MAX_VERIFY);
    if (g.tree_mask) {
      if (g.kind != HAT_SEG_VERIFY) return fail(h, HAT_EINVAL, "segment %d: a tree needs a verify segment", i);
      if (!valid_tree(g.tree_mask, g.n)) return fail(h, HAT_EINVAL, "segment %d: tree_mask is not a parents-first forest", i);
    }
    if ((long)g.start_pos + g.n > c.max_pos) return fail(h, HAT_EINVAL, "segment %d: beyond max_pos", i);
    if (!g.hidden_in || !g.hidden_out) return fail(h, HAT_EINVAL, "segment %d: null hidden pointer", i);
    if (seen[g.device_id]) return fail(h, HAT_EDUP, "segment %d: device %d twice in one step", i, g.device_id);
    seen[g.device_id] = 1;
    if (g.start_pos > h->dev[g.device_id].len)
      return fail(h, HAT_EPOS, "segment %d: start %d beyond cache length %d", i, g.start_pos, h->dev[g.device_id].len);
    total += g.n;
  }
  if (total > c.max_step_tokens) return fail(h, HAT_EINVAL, "step of %ld rows exceeds max_step_tokens", total);
  {
    long free_after = (long)h->free_pages.size(), need = 0;
    for (int i = 0; i < n_segs; ++i) {
      const hat_mid_segment_t& g = segs[i];
      const long have = (long)h->dev[g.device_id].pages.size();
      const long keep = (g.start_pos + 15) / 16;
      free_after += have - keep;
      need += (g.start_pos + g.n + 15) / 16 - keep;
    }
    if (need > free_after) return fail(h, HAT_ENOMEM, "KV pool exhausted: need %ld pages, %ld free", need, free_after);
  }

  // ---- move the pages: all rollbacks, then all allocations.  Logged: the caller commits the
  // step once it has been planned and enqueued, and rolls it back otherwise.
  undo_begin(h);
  for (int i = 0; i < n_segs; ++i) undo_save_device(h, segs[i].device_id);
  for (int i = 0; i < n_segs; ++i) {
    DeviceState& d = h->dev[segs[i].device_id];
    const size_t keep = (size_t)(segs[i].start_pos + 15) / 16;
    while (d.pages.size() > keep) {
      give_back(h, d.pages.back());
      d.pages.pop_back();
    }
    d.len = segs[i].start_pos;
  }
  const int T = (int)total, S = n_segs;
  int np_total = 0;
  for (int i = 0; i < n_segs; ++i) {
    DeviceState& d = h->dev[segs[i].device_id];
    const size_t want = (size_t)(segs[i].start_pos + segs[i].n + 15) / 16;
    while (d.pages.size() < want) d.pages.push_back(take_lowest(h));
    d.len = segs[i].start_pos + segs[i].n;
    np_total += (int)d.pages.size();
  }

  // ---- plan words
  size_t w = 0;
  auto take = [&](size_t n, size_t align_words) {
    w = align_up(w, align_words);
    size_t o = w;
    w += n;
    return o;
  };
  const size_t o_pos = take(T, 1), o_dst = take(T, 1), o_tseg = take(T, 1);
  const size_t o_toff = take(S + 1, 1), o_sstart = take(S, 1), o_spt = take(S, 1);
  const size_t o_in = take(2 * (size_t)S, 2), o_out = take(2 * (size_t)S, 2);
  const size_t o_pt = take(np_total, 1);
  int n_append = 0;
  for (int i = 0; i < S; ++i) n_append += ((segs[i].start_pos + segs[i].n - 1) >> 4) - (segs[i].start_pos >> 4) + 1;
  const size_t o_app = take(8 * (size_t)n_append, 4);

  std::vector<HatAttnItem> citems, cblocks, vitems;
  std::vector<HatMergeItem> mitems;
  {
    int t = 0, pt = 0;
    for (int i = 0; i < S; ++i) {
      const hat_mid_segment_t& g = segs[i];
      const DeviceState& d = h->dev[g.device_id];
      P[o_toff + i] = t;
      P[o_sstart + i] = g.start_pos;
      P[o_spt + i] = pt;
      uint64_t ip = (uint64_t)(uintptr_t)g.hidden_in, op = (uint64_t)(uintptr_t)g.hidden_out;
      memcpy(&P[o_in + 2 * i], &ip, 8);
      memcpy(&P[o_out + 2 * i], &op, 8);
      for (size_t k = 0; k < d.pages.size(); ++k) P[o_pt + pt + k] = d.pages[k];
      for (int r = 0; r < g.n; ++r) {
        const int q = g.start_pos + r;   // cache row; also the position unless the rows form a tree
        P[o_pos + t] = g.tree_mask ? g.start_pos + __builtin_popcount(g.tree_mask[r]) - 1 : q;
        P[o_dst + t] = d.pages[q >> 4] * 16 + (q & 15);
        P[o_tseg + t] = i;
        ++t;
      }
      pt += (int)d.pages.size();
    }
    P[o_toff + S] = T;
    HatAppendItem* ap = (HatAppendItem*)&P[o_app];
    for (int i = 0; i < S; ++i) {
      const hat_mid_segment_t& g = segs[i];
      const DeviceState& d = h->dev[g.device_id];
      for (int pg = g.start_pos >> 4; pg <= (g.start_pos + g.n - 1) >> 4; ++pg) {
        HatAppendItem a{};
        a.page = d.pages[pg]; a.pos0 = pg * 16; a.row0 = P[o_toff + i] + (a.pos0 - g.start_pos);
        a.lo = std::max(g.start_pos, a.pos0); a.hi = std::min(g.start_pos + g.n, a.pos0 + 16);
        *ap++ = a;
      }
    }
  }

  // ---- attention work lists
  {
    const int per_head = (s.verify_target + s.H - 1) / s.H;  // verify items wanted
    int part_row = 0, part_row32 = s.part_rows_cap;
    // rows of a split item are merged in groups of 16 (one workgroup per group and head)
    auto push_merge = [&](int row0, int nrows, int prow, int nsplit) {
      for (int g0 = 0; g0 < nrows; g0 += 16) {
        HatMergeItem m{};
        m.row0 = row0 + g0; m.nrows = std::min(16, nrows - g0); m.part_row = prow + g0; m.nsplit = nsplit;
        m.stride = nrows;
        mitems.push_back(m);
      }
    };
    // verify segments: split each cache into key ranges of about equal size
    long vkeys = 0;
    int nver = 0;
    for (int i = 0; i < S; ++i)
      if (segs[i].kind == HAT_SEG_VERIFY) { vkeys += segs[i].start_pos + segs[i].n; ++nver; }
    if (nver) {
      long ch = (vkeys + per_head - 1) / per_head;
      ch = std::max<long>(256, (ch + 127) / 128 * 128);
      for (int i = 0; i < S; ++i) {
        if (segs[i].kind != HAT_SEG_VERIFY) continue;
        const int len = segs[i].start_pos + segs[i].n;
        int ns = (int)((len + ch - 1) / ch);
        ns = std::min(ns, 64);
        if ((int)vitems.size() + ns > s.verify_items_cap - 1 || part_row + ns * segs[i].n > s.part_rows_cap) ns = 1;
        const int step = round_up((len + ns - 1) / ns, 64);
        ns = (len + step - 1) / step;
        for (int k = 0; k < ns; ++k) {
          HatAttnItem it{};
          it.seg = i; it.q0 = 0; it.nq = segs[i].n;
          it.start = segs[i].start_pos; it.tok0 = P[o_toff + i]; it.kv_len = len; it.pt_off = P[o_spt + i];
          it.kv_begin = k * step; it.kv_end = std::min(len, (k + 1) * step);
          it.part_row = ns > 1 ? part_row + k * segs[i].n : -1;
          for (int r = 0; r < segs[i].n; ++r) {
            const uint32_t vis = segs[i].tree_mask ? segs[i].tree_mask[r] : (2u << r) - 1;
            (r < 4 ? it.vis_lo : it.vis_hi) |= vis << (8 * (r & 3));
          }
          vitems.push_back(it);
        }
        if (ns > 1) {
          push_merge(P[o_toff + i], segs[i].n, part_row, ns);
          part_row += ns * segs[i].n;
        }
      }
    }
    // chunk segments: tiles of HAT_CHUNK_QROWS rows, split along the keys so that no work item
    // is larger than a third of one workgroup slot's share of the launch (all heads do the same
    // work, so a head has attn_target / H slots): the items, sorted by cost, then pack evenly.
    // Items of at most HAT_NARROW_QROWS rows are bound by the cache stream: key ranges of about equal size instead, for
    // three eighths of verify_target workgroups (8 x 32 rows over 4096 keys: 118 us and 7 us of merging with 768 workgroups
    // wanted, 130 and 9 with 2048).
    // Next to larger items that is a merge, and next to staged ones a second launch (4 .. 14 us a layer with narrow items of 500 keys): only where a
    // narrow item is so long that the common launch, which does not split it, would wait for it.  Measured in whole layers over 30
    // mixes with a launch of their own (one or four items of 17 rows next to one to ten chunks of 128 .. 512 rows, three widths): streamed at 1000 keys
    // between 11 us ahead and 13 behind, at 1400 between 20 ahead and 3 behind, at 2000 ahead by 7 .. 31 in all of them.  Next to larger items that stream there is no second
    // launch, but still the merge: over 50 mixes with narrow items of 230 .. 1430 keys next to 1 .. 8
    // chunks of 40 .. 512 rows a bound of 1024, 512 or 0 keys instead of 1536 costs 0.4, 1.1 and 0.9 % a layer on average (ahead in 21, 16 and 18 of them).
    double total_cost = 0, narrow_cost = 0;   // (rows x visible keys)
    double block_cost = 0, narrow_block = 0;  // the same of the items that may stream, in whole blocks of rows
    double chunk_mb = 0;                      // cache rows that chunks read
    long narrow_keys = 0, blocks = 0, narrow_blocks = 0;
    int narrow_longest = 0, longest_chunk = 0;   // keys; rows
    for (int i = 0; i < S; ++i) {
      if (segs[i].kind != HAT_SEG_CHUNK) continue;
      chunk_mb += (segs[i].start_pos + segs[i].n) * 4e-6 * s.d;
      longest_chunk = std::max(longest_chunk, segs[i].n);
      for (int q0 = 0; q0 < segs[i].n; q0 += HAT_CHUNK_QROWS) {
        const int nq = std::min(HAT_CHUNK_QROWS, segs[i].n - q0);
        const int need = segs[i].start_pos + q0 + nq;
        const double cost = (double)nq * (need - 0.5 * nq);
        if (nq > HAT_NARROW_QROWS) {
          total_cost += cost;
          blocks += (nq + HAT_NARROW_QROWS - 1) / HAT_NARROW_QROWS;
          block_cost += round_up(nq, HAT_NARROW_QROWS) * (need - 0.5 * nq);
        } else {
          narrow_cost += cost;
          narrow_block += HAT_NARROW_QROWS * (need - 0.5 * nq);
          ++narrow_blocks;
          narrow_keys += need;
          narrow_longest = std::max(narrow_longest, need);
        }
      }
    }
    const bool any_wide = blocks > 0;
    const bool stream_narrow = !any_wide || narrow_longest >= 1536;
    const bool pairs_only = longest_chunk <= HAT_PAIR_QROWS && vitems.empty() && !(stream_narrow && narrow_blocks > 0);
    if (!stream_narrow) {
      total_cost += narrow_cost;
      block_cost += narrow_block;
      blocks += narrow_blocks;
    }
    const long narrow_step = std::max<long>(256, (narrow_keys / std::max(1, per_head * 3 / 8) + 127) / 128 * 128);
    const double cost_cap = std::max(256.0 * 256.0, total_cost / (3.0 * std::max(1, s.attn_target / s.H)));
    // The chunk items with their key ranges, the larger ones staged (ranges = 0) or streamed in that many ranges; an item for whose ranges a buffer has no room stays whole.
    auto cut_items = [&](int ranges) {
      std::vector<ChunkCut> cuts;
      int row16 = part_row, row32 = part_row32, n_items = 0, n_merges = (int)mitems.size();
      for (int i = 0; i < S; ++i) {
        if (segs[i].kind != HAT_SEG_CHUNK) continue;
        for (int q0 = 0; q0 < segs[i].n; q0 += HAT_CHUNK_QROWS) {
          ChunkCut u{};
          u.seg = i; u.q0 = q0; u.nq = std::min(HAT_CHUNK_QROWS, segs[i].n - q0);
          u.need = segs[i].start_pos + q0 + u.nq;
          u.narrow = stream_narrow && u.nq <= HAT_NARROW_QROWS;
          int ns = u.narrow ? (int)((u.need + narrow_step - 1) / narrow_step) : ranges > 0 ? ranges : (int)std::ceil(u.nq * (u.need - 0.5 * u.nq) / cost_cap);
          ns = std::max(1, std::min(std::min(ns, std::max(1, u.need / 256)), u.narrow ? 32 : 16));
          const bool fp32 = u.narrow || ranges > 0;
          int& row = fp32 ? row32 : row16;
          if (n_items + ns > s.chunk_items_cap - 1 || row + ns * u.nq > (fp32 ? s.part_rows_cap + s.part32_cap : s.part_rows_cap) ||
              n_merges + 9 >= s.merge_cap)
            ns = 1;
          u.step = round_up((u.need + ns - 1) / ns, 64);
          u.ns = (u.need + u.step - 1) / u.step;
          u.part_row = u.ns > 1 ? row : -1;
          if (u.ns > 1) {
            row += u.ns * u.nq;
            n_merges += (u.nq + 15) / 16;
          }
          n_items += u.ns;
          cuts.push_back(u);
        }
      }
      return cuts;
    };
    // Larger items are staged through LDS, cut along the keys and merged; or they stream the cache too, 32 rows to a
    // workgroup.  Staging moves an eighth of the bytes and shares the widening, but its workgroups of 256 rows
    // leave waves idle on shorter items, fill the chip in coarse rounds, and need the merge.  Neither the rows x keys of a step nor its
    // longest item says which is faster; the two times do.  Attention and merge in us, staged | streamed (bf16 cache):
    //   7B shape: 1 x 256 over 1000 30.8 | 20.4, 4 x 512 over 500 89.7 | 76.4, 10 of 64 and 256 over 1000 75 | 58, but 8 x 128 over 3000 128 | 134,
    //   8 of 87 .. 106 over 25 15.3 | 17.6; 64 heads: 12 of 200 .. 290 over 20 83 | 113, 1 x 1024 over 1000 135 | 125.
    // Streaming has to be predicted 3 % ahead, 7 % in launches of more than 95 M rows x keys x heads, whose staged items fill the chip better than the
    // prediction has it (8 x 128 over 3000).  Over 820 mixes that the times were not fitted to, the choice is on average 0.3 % behind the fastest
    // way; it is 3 % or more behind staging in 2 %, 23 % at the most.
    // The partial results of staged items are held in fp16.  So smaller launches than these stage only where staging leaves every
    // item whole: otherwise 2 % of the mixes would be faster staged, mostly single chunks over long caches (128 rows over 4000 keys of the 7B
    // shape 34.5 us, streamed in two ranges 35.7; 256 over 6000 of the 13B shape 95, streamed 105).
    // A raised or lowered attn_target is a wish for the staged kernel's key ranges.
    const int f16 = c.kv_dtype == HAT_KV_F16;
    std::vector<ChunkCut> cuts = cut_items(0);
    double chosen_us = 0;
    if (any_wide && s.attn_target == kAttnTarget) {
      const bool merges = !mitems.empty() || narrow_keys > narrow_step;   // that a launch is needed for anyway
      const double staged_merge = merge_us(s, cuts, false, merges);
      const bool large = block_cost * s.H * s.hd / 128 > 95e6;
      double best = staged_merge > 0 && !large ? 1e300 : (large ? 0.93 : 0.97) * (staged_us(s, f16, cuts, chunk_mb) + staged_merge);
      // Streamed items are cut along the keys where CUs are free and the shorter workgroups are worth the merge: 64 rows of the 7B shape over
      // 1000 keys 18.7 us whole, 18.9 in three ranges, over 4000 46.0 | 30.3, four 27.8.  Not next to narrow items, whose ranges have the fp32 partial rows.
      const int most = stream_narrow && narrow_keys > 0 ? 1 : std::max(1, std::min(8, (int)(256 / (blocks * s.H))));
      for (int ranges = 1; ranges <= most; ++ranges) {
        std::vector<ChunkCut> streamed = cut_items(ranges);
        const std::vector<int> keys = block_keys(streamed, segs);
        const double us8 = stream_us(s, f16, 8, keys, chunk_mb), us4 = ranges > 1 ? us8 : stream_us(s, f16, 4, keys, chunk_mb);
        const double us = std::min(us8, us4) + merge_us(s, streamed, true, merges);
        if (us >= best) continue;
        best = us;
        cuts.swap(streamed);
        sp->block_waves = us8 <= us4 ? 8 : 4;
      }
      chosen_us = best;
    }
    // Chunks of at most 64 rows with nothing beside them, fp16 cache, head dim 128: a small workgroup for each reads its pages once, where that is
    // predicted 3 % ahead of the way chosen above.  That is in large steps: of 88 mixes of 3 .. 24 chunks of 33 .. 64 rows over 30 .. 8000 keys (16, 32 and 40
    // heads) it takes 59, whose attention is 19 % faster on average and nowhere slower (8 x 64 over 4096 keys of the 13B shape 158 us streamed, 126);
    // few or unequal ones leave CUs idle that four or eight waves to a block fill (2 x 40 over 3900 .. 5000 58 | 90).  Over a bf16 cache both computing
    // waves have to widen what they read: 49 mixes, where predicted ahead 5 % on average but up to 13 % behind; at head dim 64 44 mixes, up to 15 % behind.
    if (any_wide && s.attn_target == kAttnTarget && f16 && s.hd == 128 && pairs_only) {
      std::vector<ChunkCut> whole = cut_items(1);
      std::vector<int> keys;
      for (const ChunkCut& u : whole) keys.push_back(u.need);
      if (stream_us(s, f16, 2, keys, chunk_mb) < 0.97 * chosen_us) {
        cuts.swap(whole);
        sp->block_waves = 2;
      }
    }
    for (const ChunkCut& u : cuts) {
      for (int k = 0; k < u.ns; ++k) {
        HatAttnItem it{};
        it.seg = u.seg; it.q0 = u.q0; it.nq = u.nq;
        it.start = segs[u.seg].start_pos; it.tok0 = P[o_toff + u.seg]; it.kv_len = segs[u.seg].start_pos + segs[u.seg].n;
        it.pt_off = P[o_spt + u.seg];
        it.kv_begin = k * u.step; it.kv_end = std::min(u.need, (k + 1) * u.step);
        it.part_row = u.ns > 1 ? u.part_row + k * u.nq : -1;
        citems.push_back(it);
      }
      if (u.ns > 1) push_merge(P[o_toff + u.seg] + u.q0, u.nq, u.part_row, u.ns);
    }
    auto by_cost = [](const HatAttnItem& a, const HatAttnItem& b) {
      return (long)(a.kv_end - a.kv_begin) * a.nq > (long)(b.kv_end - b.kv_begin) * b.nq;
    };
    std::stable_sort(citems.begin(), citems.end(), by_cost);
    std::stable_sort(vitems.begin(), vitems.end(), by_cost);
    const auto narrow0 = std::stable_partition(citems.begin(), citems.end(), [&](const HatAttnItem& a) { return !stream_narrow || a.nq > HAT_NARROW_QROWS; });
    sp->n_narrow = (int)(citems.end() - narrow0);
    // Staged over an fp16 cache: by the ring kernel where a workgroup has on average as many keys as make up for a stage of 64 KB, of which one
    // workgroup fits a CU; of the chunk kernel's, with stages of half (head dim 64: a quarter) of that, two do.  750 mixes of 1 .. 32 chunks of 33 .. 512 rows
    // over 0 .. 4000 keys at 128, 600 at 64, ring against chunk kernel by keys a workgroup: head dim 128 below 64 1.07 times its time, 64 .. 128 level, 128 .. 192 0.88, more 0.9;
    // head dim 64 below 64 1.33 (at the most 1.69), 64 .. 128 1.25, 128 .. 256 1.09, 256 .. 320 0.97, more 0.94.  With the lines here the choice is
    // 0.2 and 0.4 % behind the faster of the two, always the ring kernel 0.7 and 7.8 %; whole steps of 874 other mixes put the lines at the same place.  8 x 128 rows of new prompts at 64 heads of 64: chunk kernel 14.1 us, ring 18.8.
    if (f16 && sp->block_waves == 0 && narrow0 != citems.begin()) {
      double keys = 0;
      for (auto it = citems.begin(); it != narrow0; ++it) keys += it->kv_end - it->kv_begin;
      sp->ring = keys >= (s.hd == 128 ? 96.0 : 256.0) * (narrow0 - citems.begin());
    }
    if (sp->block_waves > 2) {
      for (auto it = citems.begin(); it != narrow0; ++it)
        for (int r0 = (it->nq - 1) / HAT_NARROW_QROWS * HAT_NARROW_QROWS; r0 >= 0; r0 -= HAT_NARROW_QROWS) {   // the block with the most keys first
          HatAttnItem b = *it;
          b.q0 += r0;
          b.nq = std::min(HAT_NARROW_QROWS, it->nq - r0);
          if (b.part_row >= 0) b.part_row += r0;
          cblocks.push_back(b);
        }
      // The blocks of one head read the same pages, which favours a head at a time; but with more than a workgroup per CU the last head then starts
      // its longest blocks when the others are nearly done.  So where the lengths differ by more than a tenth and the longest is 800 keys, the
      // heads of an XCD go through the list together: 227, 256, 13, 256 and 104 rows over 971 .. 1364 keys at 32 heads of 64 46.3 -> 42.6 us, 3 x 65
      // over 808 .. 2867 at 64 heads 71 -> 56, 5 % on average over 140 such mixes (between 22 % ahead and 5 behind).  Over 110 of fewer keys
      // it is level (14 % ahead to 8 behind; 576 rows of a new prompt at 32 heads of 64 7 % behind), of equal lengths 4 % behind (8 x 64 over 4096 at 40 heads).
      double longest = 0, sum = 0;
      for (const HatAttnItem& b : cblocks) {
        const int keys = std::max(0, std::min(b.kv_end, b.start + b.q0 + b.nq) - b.kv_begin);
        longest = std::max(longest, (double)keys);
        sum += keys;
      }
      sp->heads_inner = s.H % 8 == 0 && cblocks.size() * s.H > 256 && longest >= 800 && longest * cblocks.size() > 1.1 * sum;
    }
  }
  // Verify items go along in the launch of the streamed chunk items: they fill what its last round leaves idle, and a launch is less.
  // Layer in us, two launches | one, 57 mixes of chunks of 2 .. 230 rows with 1, 8 and 30 drafts over 200 .. 8000 keys (7B, 13B and head-dim-64 shapes): 1.8 .. 2.0 % less at
  // head dim 128, 4.7 % at 64; 100 rows next to 30 drafts over 1 .. 8 k 360 | 322 (head dim 64), 725 | 701 (7B).
  // With eight waves a verify item is short for them: as many items as leave each CU one gain the same, beyond a thousand
  // they lose 3 .. 13 %.  Next to narrow items alone the launch that is saved is what there is to gain, and at head dim 128 it no longer shows where the drafts read more
  // than 1.5 GB: over 36 mixes level on average, but 17 .. 32 rows with 30 or 58 drafts over 1 .. 8 k 0 .. 3 % behind in 10 of 12 (13B shape 1083 | 1121);
  // 16 such drafts (1.2 .. 1.5 GB) 0.7 % ahead.
  double verify_gb = 0;
  for (int i = 0; i < S; ++i)
    if (segs[i].kind == HAT_SEG_VERIFY) verify_gb += (segs[i].start_pos + segs[i].n) * 4e-9 * s.d;
  if (!vitems.empty() && (!cblocks.empty() || sp->n_narrow > 0))
    sp->along = sp->block_waves == 8 ? vitems.size() * s.H <= 256 : !cblocks.empty() || s.hd == 64 || verify_gb <= 1.5;
  const size_t o_ci = take(12 * citems.size(), 4), o_cb = take(12 * cblocks.size(), 4), o_vi = take(12 * vitems.size(), 4);
  const size_t o_mi = take(8 * mitems.size(), 8);
  const size_t plan_cap = h->plan_limit ? std::min(h->plan_limit, s.plan_words) : s.plan_words;
  if (w > plan_cap) {
    undo_rollback(h);
    return fail(h, HAT_EINVAL, "internal: plan of %zu words exceeds capacity %zu", w, plan_cap);
  }
  static_assert(sizeof(HatAttnItem) == 48 && sizeof(HatMergeItem) == 32, "plan item sizes");
  if (!citems.empty()) memcpy(&P[o_ci], citems.data(), citems.size() * sizeof(HatAttnItem));
  if (!cblocks.empty()) memcpy(&P[o_cb], cblocks.data(), cblocks.size() * sizeof(HatAttnItem));
  if (!vitems.empty()) memcpy(&P[o_vi], vitems.data(), vitems.size() * sizeof(HatAttnItem));
  if (!mitems.empty()) memcpy(&P[o_mi], mitems.data(), mitems.size() * sizeof(HatMergeItem));

  sp->T = T; sp->S = S; sp->n_append = n_append;
  sp->o_pos = o_pos; sp->o_dst = o_dst; sp->o_tseg = o_tseg; sp->o_toff = o_toff; sp->o_sstart = o_sstart;
  sp->o_spt = o_spt; sp->o_in = o_in; sp->o_out = o_out; sp->o_pt = o_pt; sp->o_app = o_app;
  sp->o_ci = o_ci; sp->o_cb = o_cb; sp->o_vi = o_vi; sp->o_mi = o_mi; sp->words = w;
  sp->n_citems = (int)citems.size(); sp->n_cblocks = (int)cblocks.size(); sp->n_vitems = (int)vitems.size(); sp->n_mitems = (int)mitems.size();
  return HAT_OK;
}

// Device half of a step: uploads the plan and enqueues the kernels of every layer on st.
static hat_status_t enqueue_step(hat_mid_t* h, const StepPlan& sp, const int32_t* P, int bi, hipStream_t st) {
  const hat_mid_config_t& c = h->cfg;
  const Shapes& s = h->s;
  const int T = sp.T, S = sp.S, n_append = sp.n_append;
  const size_t o_pos = sp.o_pos, o_dst = sp.o_dst, o_tseg = sp.o_tseg, o_toff = sp.o_toff, o_sstart = sp.o_sstart;
  const size_t o_spt = sp.o_spt, o_in = sp.o_in, o_out = sp.o_out, o_pt = sp.o_pt, o_app = sp.o_app;
  const size_t o_ci = sp.o_ci, o_vi = sp.o_vi, o_mi = sp.o_mi, w = sp.words;

  HIP_TRY(h, hipEventRecord(h->ev_begin, st));
  HIP_TRY(h, hipMemcpyAsync(h->b.plan_dev, P, w * sizeof(int32_t), hipMemcpyHostToDevice, st));
  HIP_TRY(h, hipEventRecord(h->plan_ev[bi], st));
  h->plan_ev_used[bi] = true;

  const int32_t* D = h->b.plan_dev;
  HatPlanDev pd{};
  pd.T = T; pd.S = S;
  pd.pos = D + o_pos; pd.kv_dst = D + o_dst; pd.tok_seg = D + o_tseg; pd.tok_off = D + o_toff;
  pd.seg_start = D + o_sstart; pd.seg_pt = D + o_spt; pd.page_tbl = D + o_pt;
  pd.in_ptr = (const uint64_t*)(D + o_in); pd.out_ptr = (const uint64_t*)(D + o_out);
  pd.append = (const HatAppendItem*)(D + o_app); pd.n_append = n_append;

  // the gather launch fills the rotary table and applies the first norm too, unless each is to be timed by itself
  const bool gather_norms = hat_gather_norms(T) && !h->profiling;
  if (gather_norms) pd.first = HatFirstNorm{h->b.inv_freq, h->b.table, s.hd / 2, h->b.layers[0].g_attn, h->b.xn, c.rms_eps};
  LAUNCH(h, st, HAT_K_GATHER, hat_launch_gather(pd, h->b.resid, s.d, c.io_dtype, st));
  if (!gather_norms) LAUNCH(h, st, HAT_K_ROPE_APPEND, hat_launch_rope_table(pd, h->b.inv_freq, h->b.table, s.hd / 2, st));

  const bool along = sp.along && !h->profiling && !h->verify_probe;   // (each kind to be timed by itself)

  int nparts = 0;  // split-K partial sums of the previous residual GEMM still to be folded in,
  int prow0 = 0;   // for the rows from this one on
  auto run_gemm = [&](int id, HatGemm& g) -> hat_status_t {
    const int cls = id == HAT_K_GEMM_QKV ? 0 : id == HAT_K_GEMM_O ? 1 : id == HAT_K_GEMM_GATEUP ? 2 : 3;
    g.force_tile = h->force_tile[cls];
    g.force_ksplit = h->force_ksplit[cls];
    const HatGemmPlan gp = hat_gemm_plan(g);
    if (g.epilogue == HAT_EPI_RESID) {
      nparts = gp.ksplit > 1 ? gp.ksplit : 0;
      int bt = 0;
      if (gp.full > 0) hat_gemm_tile_info(gp.tile, nullptr, &bt, nullptr, nullptr, nullptr);
      prow0 = gp.full * bt;
    }
    LAUNCH(h, st, id, hat_launch_gemm(g, gp, st));
    return HAT_OK;
  };
  // RMSNorm of all rows; rows from prow0 on first take in their partial sums
  auto run_norm = [&](const float* gain, act_t* out) -> hat_status_t {
    if (prow0 > 0) LAUNCH(h, st, HAT_K_RMSNORM, hat_launch_rmsnorm(h->b.resid, h->b.gemm_part, 0, gain, out, prow0, s.d, c.rms_eps, st));
    LAUNCH(h, st, HAT_K_RMSNORM,
           hat_launch_rmsnorm(h->b.resid + (size_t)prow0 * s.d, h->b.gemm_part, nparts, gain, out + p32_index(prow0, 0, s.d), T - prow0, s.d,
                              c.rms_eps, st));
    nparts = prow0 = 0;
    return HAT_OK;
  };
  for (int l = 0; l < s.L; ++l) {
    const LayerDev& ld = h->b.layers[l];
    kv_t* pool_l = h->pool + (size_t)l * h->layer_pool_elems;
    hat_status_t rc;
    if ((l > 0 || !gather_norms) && (rc = run_norm(ld.g_attn, h->b.xn)) != HAT_OK) return rc;
    HatGemm g{};
    g.W = ld.wqkv; g.X = h->b.xn; g.K = s.d; g.T = T; g.Nw = s.Nqkv; g.Nout = 3 * s.d; g.outP = h->b.qkv;
    g.epilogue = HAT_EPI_QKV;
    g.qkv = HatQkvOut{h->b.table, pd.kv_dst, pool_l, c.n_pages, s.H, s.hd, c.kv_dtype == HAT_KV_F16};
    g.force_tile = h->force_tile[0];
    HatGemmPlan qp = hat_gemm_plan(g);   // a streaming tile, or none
    const bool apart = h->force_tile[0] == HAT_APART_TILE;
    if (qp.tile < 0) {
      g.epilogue = HAT_EPI_P32;
      qp = hat_gemm_plan(g);
      if (!apart) g.epilogue = HAT_EPI_QKV;
    }
    LAUNCH(h, st, HAT_K_GEMM_QKV, hat_launch_gemm(g, qp, st));
    if (apart)
      LAUNCH(h, st, HAT_K_ROPE_APPEND, hat_launch_rope_append(pd, h->b.qkv, h->b.table, pool_l, c.n_pages, s.H, s.hd, c.kv_dtype == HAT_KV_F16, st));
    HatAttn a{};
    a.qkv = h->b.qkv; a.pool_layer = pool_l; a.outP = h->b.attn; a.part_o = h->b.part_o; a.part_o32 = h->b.part_o32; a.part_ml = h->b.part_ml;
    a.part32_row0 = s.part_rows_cap;
    a.H = s.H; a.hd = s.hd; a.d = s.d; a.n_pages = c.n_pages; a.kv_f16 = c.kv_dtype == HAT_KV_F16;
    if (sp.n_citems > 0) {
      a.items = (const HatAttnItem*)(D + o_ci); a.n_items = sp.n_citems; a.n_narrow = sp.n_narrow;
      a.blocks = (const HatAttnItem*)(D + sp.o_cb); a.n_blocks = sp.n_cblocks; a.block_waves = sp.block_waves; a.heads_inner = sp.heads_inner; a.ring = sp.ring;
      if (along) {
        a.verify = (const HatAttnItem*)(D + o_vi); a.n_verify = sp.n_vitems;
      }
      LAUNCH(h, st, HAT_K_ATTN_CHUNK, hat_launch_attn_chunk(pd, a, st));
    }
    if (sp.n_vitems > 0 && !along) {
      a.items = (const HatAttnItem*)(D + o_vi); a.n_items = sp.n_vitems;
      if (h->verify_probe)
        LAUNCH(h, st, HAT_K_ATTN_VERIFY, hat_launch_attn_verify_probe(pd, a, (uint32_t*)h->b.fixture_pages, st));
      else
        LAUNCH(h, st, HAT_K_ATTN_VERIFY, hat_launch_attn_verify(pd, a, st));
    }
    if (sp.n_mitems > 0)
      LAUNCH(h, st, HAT_K_ATTN_MERGE, hat_launch_attn_merge(a, (const HatMergeItem*)(D + o_mi), sp.n_mitems, st));
    g = HatGemm{};
    g.W = ld.wo; g.X = h->b.attn; g.K = s.d; g.T = T; g.Nw = s.No; g.Nout = s.d; g.resid = h->b.resid;
    g.part = h->b.gemm_part; g.part_rows = s.gemm_part_rows;
    g.epilogue = HAT_EPI_RESID;
    if ((rc = run_gemm(HAT_K_GEMM_O, g)) != HAT_OK || (rc = run_norm(ld.g_ffn, h->b.xn2)) != HAT_OK) return rc;
    g = HatGemm{};
    g.W = ld.wgu; g.X = h->b.xn2; g.K = s.d; g.T = T; g.Nw = s.Ngu; g.Nout = s.Fpad; g.outP = h->b.act;
    g.epilogue = HAT_EPI_SWIGLU;
    if ((rc = run_gemm(HAT_K_GEMM_GATEUP, g)) != HAT_OK) return rc;
    g = HatGemm{};
    g.W = ld.wd; g.X = h->b.act; g.K = s.Fpad; g.T = T; g.Nw = s.Nd; g.Nout = s.d; g.resid = h->b.resid;
    g.part = h->b.gemm_part; g.part_rows = s.gemm_part_rows;
    g.epilogue = HAT_EPI_RESID;
    if ((rc = run_gemm(HAT_K_GEMM_DOWN, g)) != HAT_OK) return rc;
  }
  pd.part_row0 = prow0;
  LAUNCH(h, st, HAT_K_SCATTER, hat_launch_scatter(pd, h->b.resid, h->b.gemm_part, nparts, s.d, c.io_dtype, st));
  HIP_TRY(h, hipEventRecord(h->ev_end, st));
  h->have_step = true;
  h->last_tokens = T;
  return HAT_OK;
}

static hat_status_t forward_impl(hat_mid_t* h, const hat_mid_segment_t* segs, int32_t n_segs, void* hip_stream) {
  if (!h) return HAT_EINVAL;
  if (n_segs == 0) return HAT_OK;  // an empty step: no work, no state change
  if (h->host_only) return fail(h, HAT_EINVAL, "a host-only handle plans steps, it does not run them");
  hipStream_t st = (hipStream_t)hip_stream;
  // the pinned plan buffers rotate; this one was last read by the upload of three steps ago
  const int bi = h->plan_next;
  if (h->plan_ev_used[bi]) HIP_TRY(h, hipEventSynchronize(h->plan_ev[bi]));
  int32_t* P = h->plan_host[bi];
  StepPlan sp;
  const hat_status_t prc = plan_step(h, segs, n_segs, P, &sp);
  if (prc != HAT_OK) return prc;   // nothing moved (plan_step undoes its own page movements)
  note_stream(h, st);
  const hat_status_t erc = enqueue_step(h, sp, P, bi, st);
  if (erc != HAT_OK) {
    // a HIP call failed part-way: lengths and pages go back to where they were; kernels already
    // enqueued may still write cache rows at or beyond the segments' start positions
    undo_rollback(h);
    return erc;
  }
  undo_commit(h);
  h->plan_next = (bi + 1) % kPlanBufs;
  return HAT_OK;
}

// No exception crosses the ABI: the entry points that allocate host memory (vectors, the handle)
// turn an allocation failure into a status.
hat_status_t hat_mid_create(const hat_mid_config_t* cfg, const hat_mid_layer_weights_t* layers, void* kv_pool,
                            void* workspace, void* hip_stream, hat_mid_t** out) {
  try {
    return create_impl(cfg, layers, kv_pool, workspace, hip_stream, out);
  } catch (...) {
    if (out) *out = nullptr;
    return HAT_EHIP;
  }
}

hat_status_t hat_mid_forward(hat_mid_t* h, const hat_mid_segment_t* segs, int32_t n_segs, void* hip_stream) {
  try {
    return forward_impl(h, segs, n_segs, hip_stream);
  } catch (...) {
    if (h && h->undo_on) undo_rollback(h);
    return fail(h, HAT_EHIP, "host allocation failed while planning the step");
  }
}

hat_status_t hat_mid_last_step_stats(hat_mid_t* h, int32_t* tokens, float* gpu_ms) {
  if (!h) return HAT_EINVAL;
  if (!h->have_step) return fail(h, HAT_EINVAL, "no step has run yet");
  HIP_TRY(h, hipEventSynchronize(h->ev_end));
  float ms = 0.f;
  HIP_TRY(h, hipEventElapsedTime(&ms, h->ev_begin, h->ev_end));
  if (tokens) *tokens = h->last_tokens;
  if (gpu_ms) *gpu_ms = ms;
  return HAT_OK;
}

hat_status_t hat_mid_set_profiling(hat_mid_t* h, int32_t on) {
  if (!h) return HAT_EINVAL;
  if (h->host_only) return fail(h, HAT_EINVAL, "a host-only handle has no GPU side");
  h->profiling = on != 0;
  return HAT_OK;
}

hat_status_t hat_mid_kernel_times(hat_mid_t* h, float* ms, int32_t* launches) {
  if (!h || !ms || !launches) return HAT_EINVAL;
  for (int i = 0; i < HAT_K_COUNT; ++i) { ms[i] = 0.f; launches[i] = 0; }
  for (auto& r : h->recs) {
    HIP_TRY(h, hipEventSynchronize(r.b));
    float t = 0.f;
    HIP_TRY(h, hipEventElapsedTime(&t, r.a, r.b));
    ms[r.id] += t;
    launches[r.id] += 1;
    h->ev_pool.push_back(r.a);
    h->ev_pool.push_back(r.b);
  }
  h->recs.clear();
  return HAT_OK;
}

static hat_status_t fixture_pages(hat_mid_t* h, const DeviceState& d, int pos0, int n, hipStream_t st) {
  const int p0 = pos0 >> 4, p1 = (pos0 + n - 1) >> 4;
  HIP_TRY(h, hipStreamSynchronize(st));  // the staging area below is reused by every fixture call
  HIP_TRY(h, hipMemcpy(h->b.fixture_pages, d.pages.data() + p0, (size_t)(p1 - p0 + 1) * sizeof(int32_t),
                       hipMemcpyHostToDevice));
  return HAT_OK;
}

static hat_status_t forward_host_impl(hat_mid_t* h, const hat_mid_segment_t* segs, int32_t n_segs, void* hip_stream) {
  if (!h) return HAT_EINVAL;
  if (h->host_only) return fail(h, HAT_EINVAL, "a host-only handle has no GPU side");
  if (n_segs == 0) return HAT_OK;
  if (!segs || n_segs < 0) return fail(h, HAT_EINVAL, "no segments");
  if (n_segs > h->cfg.max_devices) return fail(h, HAT_EINVAL, "more segments (%d) than devices", n_segs);
  const Shapes& s = h->s;
  const size_t rowb = (size_t)s.d * (h->cfg.io_dtype == HAT_F32 ? 4 : 2);
  long total = 0;
  for (int i = 0; i < n_segs; ++i) {
    if (segs[i].n <= 0 || !segs[i].hidden_in || !segs[i].hidden_out)
      return fail(h, HAT_EINVAL, "segment %d: n = %d or a null host pointer", i, segs[i].n);
    total += segs[i].n;
  }
  if (total > s.Tcap) return fail(h, HAT_EINVAL, "step of %ld rows exceeds max_step_tokens %d", total, s.Tcap);
  hipStream_t st = (hipStream_t)hip_stream;
  const int slot = h->host_slot;
  h->host_slot ^= 1;
  // this input slot was last read by the step two calls back
  if (h->slot_used[slot]) HIP_TRY(h, hipStreamWaitEvent(h->copy_stream, h->slot_free[slot], 0));
  std::vector<hat_mid_segment_t> dsegs(segs, segs + n_segs);
  unsigned char* in = (unsigned char*)h->b.stage_in[slot];
  unsigned char* out = (unsigned char*)h->b.stage_out;
  size_t off = 0;
  for (int i = 0; i < n_segs; ++i) {
    const size_t nb = (size_t)segs[i].n * rowb;
    HIP_TRY(h, hipMemcpyAsync(in + off, segs[i].hidden_in, nb, hipMemcpyHostToDevice, h->copy_stream));
    dsegs[i].hidden_in = in + off;
    dsegs[i].hidden_out = out + off;
    off += nb;
  }
  HIP_TRY(h, hipEventRecord(h->up_done[slot], h->copy_stream));
  HIP_TRY(h, hipStreamWaitEvent(st, h->up_done[slot], 0));
  const hat_status_t rc = forward_impl(h, dsegs.data(), n_segs, hip_stream);
  HIP_TRY(h, hipEventRecord(h->slot_free[slot], st));
  h->slot_used[slot] = true;
  if (rc != HAT_OK) return rc;
  off = 0;
  for (int i = 0; i < n_segs; ++i) {
    const size_t nb = (size_t)segs[i].n * rowb;
    HIP_TRY(h, hipMemcpyAsync(segs[i].hidden_out, out + off, nb, hipMemcpyDeviceToHost, st));
    off += nb;
  }
  return HAT_OK;
}

hat_status_t hat_mid_forward_host(hat_mid_t* h, const hat_mid_segment_t* segs, int32_t n_segs, void* hip_stream) {
  try {
    return forward_host_impl(h, segs, n_segs, hip_stream);
  } catch (...) {
    if (h && h->undo_on) undo_rollback(h);
    return fail(h, HAT_EHIP, "host allocation failed while planning the step");
  }
}

hat_status_t hat_mid_kv_import(hat_mid_t* h, int32_t device_id, int32_t layer, int32_t pos0, int32_t n, const void* k,
                               const void* v, void* hip_stream) {
  if (!h) return HAT_EINVAL;
  if (h->host_only) return fail(h, HAT_EINVAL, "a host-only handle has no GPU side");
  const hat_mid_config_t& c = h->cfg;
  if (device_id < 0 || device_id >= c.max_devices) return fail(h, HAT_EDEVICE, "device id %d out of range", device_id);
  if (layer < 0 || layer >= c.n_layers || n <= 0 || pos0 < 0 || !k || !v) return fail(h, HAT_EINVAL, "bad import arguments");
  if ((long)pos0 + n > c.max_pos) return fail(h, HAT_EINVAL, "import beyond max_pos");
  DeviceState& d = h->dev[device_id];
  if (pos0 > d.len) return fail(h, HAT_EPOS, "import at %d beyond cache length %d", pos0, d.len);
  const size_t want = (size_t)(pos0 + n + 15) / 16;
  if (want > d.pages.size() && want - d.pages.size() > h->free_pages.size())
    return fail(h, HAT_ENOMEM, "KV pool exhausted on import");
  undo_begin(h);
  undo_save_device(h, device_id);
  while (d.pages.size() < want) d.pages.push_back(take_lowest(h));
  d.len = std::max(d.len, pos0 + n);
  hipStream_t st = (hipStream_t)hip_stream;
  note_stream(h, st);
  hat_status_t rc = fixture_pages(h, d, pos0, n, st);
  if (rc == HAT_OK) {
    const hipError_t e = hat_launch_kv_import(h->pool + (size_t)layer * h->layer_pool_elems, c.n_pages, h->b.fixture_pages,
                                              pos0, n, (const bf16_t*)k, (const bf16_t*)v, c.n_heads, c.head_dim, c.kv_dtype == HAT_KV_F16, st);
    if (e != hipSuccess) rc = fail(h, HAT_EHIP, "kv import launch failed: %s", hipGetErrorString(e));
  }
  if (rc != HAT_OK) {
    undo_rollback(h);   // the pages taken for this import return to the pool, the length is as before
    return rc;
  }
  undo_commit(h);
  return HAT_OK;
}

hat_status_t hat_mid_kv_export(hat_mid_t* h, int32_t device_id, int32_t layer, int32_t pos0, int32_t n, void* k,
                               void* v, void* hip_stream) {
  if (!h) return HAT_EINVAL;
  if (h->host_only) return fail(h, HAT_EINVAL, "a host-only handle has no GPU side");
  const hat_mid_config_t& c = h->cfg;
  if (device_id < 0 || device_id >= c.max_devices) return fail(h, HAT_EDEVICE, "device id %d out of range", device_id);
  if (layer < 0 || layer >= c.n_layers || n <= 0 || pos0 < 0 || !k || !v) return fail(h, HAT_EINVAL, "bad export arguments");
  const DeviceState& d = h->dev[device_id];
  if (pos0 + n > d.len) return fail(h, HAT_EPOS, "export of rows %d..%d beyond cache length %d", pos0, pos0 + n, d.len);
  hipStream_t st = (hipStream_t)hip_stream;
  note_stream(h, st);
  hat_status_t rc = fixture_pages(h, d, pos0, n, st);
  if (rc != HAT_OK) return rc;
  HIP_TRY(h, hat_launch_kv_export(h->pool + (size_t)layer * h->layer_pool_elems, c.n_pages, h->b.fixture_pages, pos0, n,
                                  (bf16_t*)k, (bf16_t*)v, c.n_heads, c.head_dim, c.kv_dtype == HAT_KV_F16, st));
  return HAT_OK;
}

hat_status_t hat_mid_kv_export_static(hat_mid_t* h, int32_t device_id, int32_t layer, int32_t pos0, int32_t n, void* k,
                                      void* v, void* hip_stream) {
  if (!h) return HAT_EINVAL;
  if (h->host_only) return fail(h, HAT_EINVAL, "a host-only handle has no GPU side");
  const hat_mid_config_t& c = h->cfg;
  if (device_id < 0 || device_id >= c.max_devices) return fail(h, HAT_EDEVICE, "device id %d out of range", device_id);
  if (layer < 0 || layer >= c.n_layers || n <= 0 || pos0 < 0 || !k || !v) return fail(h, HAT_EINVAL, "bad export arguments");
  const DeviceState& d = h->dev[device_id];
  if ((long)pos0 + n > d.len) return fail(h, HAT_EPOS, "export of rows %d..%ld beyond cache length %d", pos0, (long)pos0 + n, d.len);
  const int p0 = pos0 >> 4, p1 = (pos0 + n - 1) >> 4, np = p1 - p0 + 1;
  if (np > kStaticPageIds)
    return fail(h, HAT_EINVAL, "export of %d rows spans %d pages: the static scratch holds %d page ids (%d rows)", n, np,
                kStaticPageIds, kStaticPageIds * HAT_PAGE_SIZE);
  hipStream_t st = (hipStream_t)hip_stream;
  // the pinned buffer is free again once the previous call's upload has read it
  if (h->static_ev_used) HIP_TRY(h, hipEventSynchronize(h->static_ev));
  memcpy(h->static_pages_host, d.pages.data() + p0, (size_t)np * sizeof(int32_t));
  note_stream(h, st);
  // from here on only the address taken with hipGetSymbolAddress is used for the array
  HIP_TRY(h, hipMemcpyAsync(h->static_pages_dev, h->static_pages_host, (size_t)np * sizeof(int32_t), hipMemcpyHostToDevice, st));
  HIP_TRY(h, hipEventRecord(h->static_ev, st));
  h->static_ev_used = true;
  HIP_TRY(h, hat_launch_kv_export(h->pool + (size_t)layer * h->layer_pool_elems, c.n_pages, h->static_pages_dev, pos0, n,
                                  (bf16_t*)k, (bf16_t*)v, c.n_heads, c.head_dim, c.kv_dtype == HAT_KV_F16, st));
  return HAT_OK;
}

hat_status_t hat_mid_debug_create_host_only(const hat_mid_config_t* cfg, hat_mid_t** out) {
  if (out) *out = nullptr;
  if (!out || !valid_cfg(cfg)) return HAT_EINVAL;
  try {
    hat_mid* h = new hat_mid();
    h->host_only = true;
    h->cfg = *cfg;
    h->s = make_shapes(*cfg);
    h->pool = nullptr;
    h->layer_pool_elems = (size_t)cfg->n_pages * kv_page_elems(cfg->n_heads, cfg->head_dim);
    for (int i = 0; i < cfg->n_pages; ++i) h->free_pages.insert(i);
    h->dev.resize(cfg->max_devices);
    h->host_plan.resize(h->s.plan_words);
    *out = h;
    return HAT_OK;
  } catch (...) {
    return HAT_EHIP;
  }
}

hat_status_t hat_mid_debug_plan(hat_mid_t* h, const hat_mid_segment_t* segs, int32_t n_segs, int32_t* pos,
                                int32_t* kv_dst, int32_t cap_rows, int32_t* chunk_items, int32_t* n_chunk_items,
                                int32_t* verify_items, int32_t* n_verify_items, int32_t* merge_items,
                                int32_t* n_merge_items, int32_t cap_items) {
  if (!h) return HAT_EINVAL;
  if (!h->host_only) return fail(h, HAT_EINVAL, "hat_mid_debug_plan needs a host-only handle");
  if (n_chunk_items) *n_chunk_items = 0;
  if (n_verify_items) *n_verify_items = 0;
  if (n_merge_items) *n_merge_items = 0;
  h->host_narrow = h->host_n_blocks = h->host_block_waves = 0;
  h->host_along = h->host_ring = false;
  if (n_segs == 0) return HAT_OK;
  try {
    StepPlan sp;
    const int32_t* P = h->host_plan.data();
    const hat_status_t rc = plan_step(h, segs, n_segs, h->host_plan.data(), &sp);
    if (rc != HAT_OK) return rc;
    undo_commit(h);
    h->host_narrow = sp.n_narrow;
    h->host_blocks = sp.o_cb;
    h->host_n_blocks = sp.n_cblocks;
    h->host_block_waves = sp.block_waves;
    h->host_along = sp.along;
    h->host_ring = sp.ring;
    if (sp.T > cap_rows || std::max(sp.n_citems, std::max(sp.n_vitems, sp.n_mitems)) > cap_items)
      return fail(h, HAT_EINVAL, "output arrays too small for %d rows / %d, %d, %d items (the step has been planned)", sp.T,
                  sp.n_citems, sp.n_vitems, sp.n_mitems);
    if (pos) memcpy(pos, P + sp.o_pos, sp.T * sizeof(int32_t));
    if (kv_dst) memcpy(kv_dst, P + sp.o_dst, sp.T * sizeof(int32_t));
    if (chunk_items) memcpy(chunk_items, P + sp.o_ci, (size_t)sp.n_citems * sizeof(HatAttnItem));
    if (verify_items) memcpy(verify_items, P + sp.o_vi, (size_t)sp.n_vitems * sizeof(HatAttnItem));
    if (merge_items) memcpy(merge_items, P + sp.o_mi, (size_t)sp.n_mitems * sizeof(HatMergeItem));
    if (n_chunk_items) *n_chunk_items = sp.n_citems;
    if (n_verify_items) *n_verify_items = sp.n_vitems;
    if (n_merge_items) *n_merge_items = sp.n_mitems;
    return HAT_OK;
  } catch (...) {
    if (h->undo_on) undo_rollback(h);
    return fail(h, HAT_EHIP, "host allocation failed while planning the step");
  }
}

hat_status_t hat_mid_debug_plan_narrow(const hat_mid_t* h, int32_t* n_narrow) {
  if (!h || !h->host_only || !n_narrow) return HAT_EINVAL;
  *n_narrow = h->host_narrow;
  return HAT_OK;
}

hat_status_t hat_mid_debug_plan_blocks(const hat_mid_t* h, int32_t* blocks, int32_t* n_blocks, int32_t cap_blocks,
                                       int32_t* waves) {
  if (!h || !h->host_only || !n_blocks) return HAT_EINVAL;
  *n_blocks = h->host_n_blocks;
  if (waves) *waves = h->host_block_waves;
  if (!blocks) return HAT_OK;
  if (h->host_n_blocks > cap_blocks) return HAT_EINVAL;
  if (h->host_n_blocks > 0) memcpy(blocks, h->host_plan.data() + h->host_blocks, (size_t)h->host_n_blocks * sizeof(HatAttnItem));
  return HAT_OK;
}

hat_status_t hat_mid_debug_plan_ring(const hat_mid_t* h, int32_t* ring) {
  if (!h || !h->host_only || !ring) return HAT_EINVAL;
  *ring = h->host_ring;
  return HAT_OK;
}
hat_status_t hat_mid_debug_plan_along(const hat_mid_t* h, int32_t* along) {
  if (!h || !h->host_only || !along) return HAT_EINVAL;
  *along = h->host_along;
  return HAT_OK;
}

hat_status_t hat_mid_debug_force_gemm(hat_mid_t* h, int32_t which, int32_t tile, int32_t ksplit) {
  if (!h || which < 0 || which > 3) return HAT_EINVAL;
  h->force_tile[which] = tile;
  h->force_ksplit[which] = ksplit;
  return HAT_OK;
}

int32_t hat_mid_debug_gemm_tile_count(void) { return hat_gemm_tile_count(); }

hat_status_t hat_mid_debug_gemm_tile_info(int32_t tile, int32_t* features, int32_t* tokens, int32_t* waves,
                                          int32_t* k_per_stage, int32_t* stages) {
  int bf, bt, w, bk, ns;
  if (!hat_gemm_tile_info(tile, &bf, &bt, &w, &bk, &ns)) return HAT_EINVAL;
  if (features) *features = bf;
  if (tokens) *tokens = bt;
  if (waves) *waves = w;
  if (k_per_stage) *k_per_stage = bk;
  if (stages) *stages = ns;
  return HAT_OK;
}
hat_status_t hat_mid_debug_gemm_tile_resources(int32_t tile, int32_t* loader_waves, int32_t* lds_bytes) {
  int nl, lds;
  if (!hat_gemm_tile_resources(tile, &nl, &lds)) return HAT_EINVAL;
  if (loader_waves) *loader_waves = nl;
  if (lds_bytes) *lds_bytes = lds;
  return HAT_OK;
}

hat_status_t hat_mid_debug_set_attn_targets(hat_mid_t* h, int32_t chunk_target, int32_t verify_target) {
  if (!h || chunk_target < 0 || verify_target < 0) return HAT_EINVAL;
  if (chunk_target > 0) h->s.attn_target = chunk_target;
  if (verify_target > 0) h->s.verify_target = verify_target;
  return HAT_OK;
}

hat_status_t hat_mid_debug_set_verify_probe(hat_mid_t* h, int32_t on) {
  if (!h) return HAT_EINVAL;
  if (h->host_only) return fail(h, HAT_EINVAL, "a host-only handle has no GPU side");
  h->verify_probe = on != 0;
  return HAT_OK;
}

hat_status_t hat_mid_debug_limit_plan(hat_mid_t* h, int64_t max_words) {
  if (!h || max_words < 0) return HAT_EINVAL;
  h->plan_limit = (size_t)max_words;
  return HAT_OK;
}

static HatGemmPlan auto_gemm_plan(int32_t T, int32_t Nw, int32_t Nout, int32_t K, int32_t epilogue, int32_t part_rows) {
  HatGemm g{};
  static float dummy;   // only its non-nullness is looked at
  g.T = T; g.Nw = Nw; g.Nout = Nout; g.K = K; g.epilogue = epilogue;
  g.part = part_rows > 0 ? &dummy : nullptr;
  g.part_rows = part_rows;
  g.force_tile = -1;
  return hat_gemm_plan(g);
}

hat_status_t hat_mid_debug_gemm_plan(int32_t T, int32_t Nw, int32_t Nout, int32_t K, int32_t epilogue,
                                     int32_t part_rows, int32_t* tile, int32_t* ksplit) {
  if (!tile || !ksplit) return HAT_EINVAL;
  const HatGemmPlan p = auto_gemm_plan(T, Nw, Nout, K, epilogue, part_rows);
  *tile = p.tile;
  *ksplit = p.full > 0 ? 1 : p.ksplit;   // of the whole product; hat_mid_debug_gemm_split reports a split tail
  return HAT_OK;
}

hat_status_t hat_mid_debug_gemm_split(int32_t T, int32_t Nw, int32_t Nout, int32_t K, int32_t part_rows, int32_t* tile,
                                      int32_t* first_row, int32_t* ksplit) {
  if (!tile || !first_row || !ksplit) return HAT_EINVAL;
  const HatGemmPlan p = auto_gemm_plan(T, Nw, Nout, K, HAT_EPI_RESID, part_rows);
  int bt = 0;
  hat_gemm_tile_info(p.tile, nullptr, &bt, nullptr, nullptr, nullptr);
  *tile = p.tile;
  *first_row = p.full * bt;
  *ksplit = p.ksplit;
  return HAT_OK;
}

hat_status_t hat_mid_debug_dump(hat_mid_t* h, int32_t which, void* dst, void* hip_stream) {
  if (!h || !dst) return HAT_EINVAL;
  if (!h->have_step) return fail(h, HAT_EINVAL, "no step has run yet");
  const Shapes& s = h->s;
  hipStream_t st = (hipStream_t)hip_stream;
  const int T = h->last_tokens;
  switch (which) {
    case HAT_DUMP_XNORM: HIP_TRY(h, hat_launch_unpack_p32(h->b.xn, s.d, 0, s.d, T, (float*)dst, st)); break;
    case HAT_DUMP_Q: HIP_TRY(h, hat_launch_unpack_p32(h->b.qkv, 3 * s.d, 0, s.d, T, (float*)dst, st)); break;
    case HAT_DUMP_ATTN: HIP_TRY(h, hat_launch_unpack_p32(h->b.attn, s.d, 0, s.d, T, (float*)dst, st)); break;
    case HAT_DUMP_XNORM2: HIP_TRY(h, hat_launch_unpack_p32(h->b.xn2, s.d, 0, s.d, T, (float*)dst, st)); break;
    case HAT_DUMP_ACT: HIP_TRY(h, hat_launch_unpack_p32(h->b.act, s.Fpad, 0, s.F, T, (float*)dst, st)); break;
    default: return fail(h, HAT_EINVAL, "unknown dump id %d", which);
  }
  return HAT_OK;
}

}  // extern "C"
