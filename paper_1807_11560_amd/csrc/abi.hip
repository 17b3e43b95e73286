// C-ABI entry points (include/lddmm.h): argument validation, the per-
// workspace record that ties lddmm_hessvec to the preceding
// lddmm_gradient, the Gauss-Newton-Krylov loop of lddmm_register, and the
// kernel-family timer.
#include "../../include/lddmm.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <coroutine>
#include <cstdio>
#include <cstring>
#include <functional>
#include <map>
#include <mutex>
#include <string>
#include <memory>
#include <vector>

#include "engine.h"
#include "sampler.h"

using namespace lddmm;

namespace {

thread_local std::string g_last_error;
thread_local int64_t g_last_hvps = 0;

int fail(int code, const std::string& msg) {
  g_last_error = msg;
  return code;
}

int hip_fail(hipError_t e, const char* where) {
  return fail(LDDMM_E_HIP, std::string(where) + ": " + hipGetErrorString(e));
}

// Record per workspace pointer: the parameters of the last gradient that
// prepared it for lddmm_hessvec.
struct WsRecord {
  bool prepared = false;
  Dims dims{};
};
std::mutex g_ws_mu;
std::map<const void*, WsRecord> g_ws;

bool same_dims(const Dims& a, const Dims& b) {
  for (int j = 0; j < 3; ++j)
    if (a.N[j] != b.N[j] || a.K[j] != b.K[j] || a.M[j] != b.M[j]) return false;
  return a.nt == b.nt && a.s == b.s && a.alpha == b.alpha && a.sigma == b.sigma &&
         a.hessian == b.hessian && a.state == b.state && a.integrator == b.integrator && a.prec == b.prec &&
         a.ckpt == b.ckpt;
}

void set_prepared(const void* ws, bool prepared, const Dims& d) {
  std::lock_guard<std::mutex> lk(g_ws_mu);
  WsRecord& r = g_ws[ws];
  r.prepared = prepared;
  r.dims = d;
}

// ---------------------------------------------------------------- tile table
// Launch shapes per (grid, band, spectral grid, precision, arch): set by
// lddmm_tiles_set / lddmm_autotune / lddmm_tiles_load, read when a call's
// parameters are validated.
struct TileKey {
  int N[3], K[3], M[3], prec;
  std::string arch;
  bool operator<(const TileKey& o) const {
    const int a[10] = {N[0], N[1], N[2], K[0], K[1], K[2], M[0], M[1], M[2], prec};
    const int b[10] = {o.N[0], o.N[1], o.N[2], o.K[0], o.K[1], o.K[2], o.M[0], o.M[1], o.M[2], o.prec};
    for (int i = 0; i < 10; ++i)
      if (a[i] != b[i]) return a[i] < b[i];
    return arch < o.arch;
  }
};
struct TileEntry {
  lddmm_tiles t{};
  double ms = 0.0;  // the autotuner's time per Hessian-vector product (0: not measured)
};
std::mutex g_tiles_mu;
std::map<TileKey, TileEntry> g_tiles;
std::atomic<bool> g_tiles_any{false};

// Architecture name of the current device ("gfx950"), "" without one.
std::string current_arch() {
  static std::mutex mu;
  static std::map<int, std::string> names;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) {
    (void)hipGetLastError();
    return "";
  }
  std::lock_guard<std::mutex> lk(mu);
  auto it = names.find(dev);
  if (it != names.end()) return it->second;
  hipDeviceProp_t prop;
  std::string name;
  if (hipGetDeviceProperties(&prop, dev) == hipSuccess) {
    name = prop.gcnArchName;
    name = name.substr(0, name.find(':'));
  } else {
    (void)hipGetLastError();
  }
  names[dev] = name;
  return name;
}

TileKey tile_key(const Dims& d, const std::string& arch) {
  TileKey k;
  for (int j = 0; j < 3; ++j) {
    k.N[j] = d.N[j];
    k.K[j] = d.K[j];
    k.M[j] = d.M[j];
  }
  k.prec = d.prec;
  k.arch = arch;
  return k;
}

int check_tiles(const Dims& d, const lddmm_tiles& t) {
  if (t.prod_rows < 0 || t.prod_rows > prod_rows_max(d))
    return fail(LDDMM_E_INVALID_ARG, "prod_rows must be in [0, " + std::to_string(prod_rows_max(d)) + "]");
  if (t.col_split < 0 || t.col_split > 3) return fail(LDDMM_E_INVALID_ARG, "col_split must be in [0, 3]");
  if (t.sl_threads != 0 && t.sl_threads != 64 && t.sl_threads != 128 && t.sl_threads != 256)
    return fail(LDDMM_E_INVALID_ARG, "sl_threads must be 0, 64, 128 or 256");
  return LDDMM_OK;
}

void apply_tiles(Dims& d) {
  if (!g_tiles_any.load()) return;
  const std::string arch = current_arch();
  if (arch.empty()) return;
  std::lock_guard<std::mutex> lk(g_tiles_mu);
  auto it = g_tiles.find(tile_key(d, arch));
  if (it == g_tiles.end()) return;
  d.tile_prod_rows = it->second.t.prod_rows;
  d.tile_col = it->second.t.col_split;
  d.tile_sl = it->second.t.sl_threads;
}

// ---- the table as JSON: {"format": "lddmm-tiles-1", "entries": [{"arch":
// "gfx950", "grid": [..], "band": [..], "spectral": [..], "precision":
// "fp32"|"bf16x3", "prod_rows": r, "col_split": c, "sl_threads": t,
// "ms_per_hvp": x}, ...]}.  The reader takes that form (any key order, extra
// keys ignored) and nothing else of JSON.
struct JsonValue {
  enum Kind { NUL, NUM, STR, ARR, OBJ, BOOL } kind = NUL;
  double num = 0.0;
  std::string str;
  std::vector<JsonValue> arr;
  std::vector<std::pair<std::string, JsonValue>> obj;
  const JsonValue* get(const char* key) const {
    for (auto& kv : obj)
      if (kv.first == key) return &kv.second;
    return nullptr;
  }
};

struct JsonReader {
  const std::string& s;
  size_t i = 0;
  int depth = 0;
  explicit JsonReader(const std::string& text) : s(text) {}
  void ws() {
    while (i < s.size() && (s[i] == ' ' || s[i] == '\n' || s[i] == '\t' || s[i] == '\r')) ++i;
  }
  bool str(std::string* out) {
    if (i >= s.size() || s[i] != '"') return false;
    ++i;
    out->clear();
    while (i < s.size() && s[i] != '"') {
      if (s[i] == '\\') {
        if (++i >= s.size()) return false;
        const char c = s[i];
        if (c != '"' && c != '\\' && c != '/') return false;
        out->push_back(c);
      } else {
        out->push_back(s[i]);
      }
      ++i;
    }
    if (i >= s.size()) return false;
    ++i;
    return true;
  }
  bool value(JsonValue* v) {
    ws();
    if (i >= s.size() || ++depth > 8) return false;
    bool ok = false;
    const char c = s[i];
    if (c == '{') {
      v->kind = JsonValue::OBJ;
      ++i;
      ws();
      if (i < s.size() && s[i] == '}') {
        ++i;
        ok = true;
      } else {
        for (;;) {
          ws();
          std::string key;
          JsonValue val;
          if (!str(&key)) break;
          ws();
          if (i >= s.size() || s[i] != ':') break;
          ++i;
          if (!value(&val)) break;
          v->obj.emplace_back(key, std::move(val));
          ws();
          if (i < s.size() && s[i] == ',') {
            ++i;
            continue;
          }
          if (i < s.size() && s[i] == '}') {
            ++i;
            ok = true;
          }
          break;
        }
      }
    } else if (c == '[') {
      v->kind = JsonValue::ARR;
      ++i;
      ws();
      if (i < s.size() && s[i] == ']') {
        ++i;
        ok = true;
      } else {
        for (;;) {
          JsonValue val;
          if (!value(&val)) break;
          v->arr.push_back(std::move(val));
          ws();
          if (i < s.size() && s[i] == ',') {
            ++i;
            continue;
          }
          if (i < s.size() && s[i] == ']') {
            ++i;
            ok = true;
          }
          break;
        }
      }
    } else if (c == '"') {
      v->kind = JsonValue::STR;
      ok = str(&v->str);
    } else if (s.compare(i, 4, "null") == 0) {
      v->kind = JsonValue::NUL;
      i += 4;
      ok = true;
    } else if (s.compare(i, 4, "true") == 0 || s.compare(i, 5, "false") == 0) {
      v->kind = JsonValue::BOOL;
      v->num = s[i] == 't';
      i += s[i] == 't' ? 4 : 5;
      ok = true;
    } else {
      const char* b = s.c_str() + i;
      char* e = nullptr;
      v->kind = JsonValue::NUM;
      v->num = std::strtod(b, &e);
      ok = e != b && std::isfinite(v->num);
      i += (size_t)(e - b);
    }
    --depth;
    return ok;
  }
};

bool json_int3(const JsonValue* v, int out[3]) {
  if (!v || v->kind != JsonValue::ARR || v->arr.size() != 3) return false;
  for (int j = 0; j < 3; ++j) {
    const JsonValue& x = v->arr[j];
    if (x.kind != JsonValue::NUM || x.num != (double)(int)x.num) return false;
    out[j] = (int)x.num;
  }
  return true;
}

bool json_int(const JsonValue* v, int* out) {
  if (!v || v->kind != JsonValue::NUM || v->num != (double)(int)v->num) return false;
  *out = (int)v->num;
  return true;
}

int validate(const lddmm_params* p, Dims* d) {
  if (!p) return fail(LDDMM_E_INVALID_ARG, "params is NULL");
  if (p->ndim != 3)
    return fail(LDDMM_E_SHAPE, p->ndim == 2 ? "two-dimensional problems are taken by the single-problem entry points only"
                                            : "ndim must be 2 or 3");
  if (!(p->alpha > 0.0) || !std::isfinite(p->alpha))
    return fail(LDDMM_E_INVALID_ARG, "alpha must be positive");
  if (!(p->sigma > 0.0) || !std::isfinite(p->sigma))
    return fail(LDDMM_E_INVALID_ARG, "sigma must be positive");
  if (p->s < 1 || p->s > 8) return fail(LDDMM_E_INVALID_ARG, "s must be in [1, 8]");
  if (p->time_steps < 1 || p->time_steps > 1000)
    return fail(LDDMM_E_INVALID_ARG, "time_steps must be in [1, 1000]");
  if (p->precision != LDDMM_FP32 && p->precision != LDDMM_FP32_BF16X3)
    return fail(LDDMM_E_INVALID_ARG, "unknown precision");
  if (p->hessian != LDDMM_GN_PAPER && p->hessian != LDDMM_GN_CLASSICAL && p->hessian != LDDMM_NEWTON &&
      p->hessian != LDDMM_GN_EXACT)
    return fail(LDDMM_E_INVALID_ARG, "unknown hessian mode");
  if (p->hessian == LDDMM_GN_EXACT && (p->state != LDDMM_STATE_IMAGE || p->integrator != LDDMM_EULER))
    return fail(LDDMM_E_INVALID_ARG, "LDDMM_GN_EXACT needs the image state and Euler steps");
  if (p->state != LDDMM_STATE_IMAGE && p->state != LDDMM_STATE_DEFORMATION)
    return fail(LDDMM_E_INVALID_ARG, "unknown state");
  if (p->integrator != LDDMM_EULER && p->integrator != LDDMM_RK4)
    return fail(LDDMM_E_INVALID_ARG, "unknown integrator");
  if (p->integrator == LDDMM_RK4 && p->state != LDDMM_STATE_IMAGE)
    return fail(LDDMM_E_INVALID_ARG, "LDDMM_RK4 integrates the image state only");
  Dims& o = *d;
  o = Dims{};
  for (int j = 0; j < 3; ++j) {
    const int N = p->grid[j], K = p->band[j];
    if (N < 8 || N > 2048) return fail(LDDMM_E_SHAPE, "grid sizes must be in [8, 2048]");
    if (K < 4 || K > kMaxBand || (K & 1) || K > N)
      return fail(LDDMM_E_SHAPE, "band sizes must be even, in [4, 64] and at most the grid size");
    const int M = p->spectral[j] ? p->spectral[j] : 3 * K / 2;
    if (M < 3 * K / 2 - 2 || M > kMaxPadded)
      return fail(LDDMM_E_SHAPE, "spectral grid must satisfy 3K/2 - 2 <= M <= 256");
    o.N[j] = N;
    o.K[j] = K;
    o.M[j] = M;
  }
  if (o.N[2] > kMaxRow) return fail(LDDMM_E_SHAPE, "the last grid axis must be at most 256");
  o.Kh = o.K[2] / 2;
  o.nb = o.K[0] * o.K[1] * o.Kh;
  o.nN = (long long)o.N[0] * o.N[1] * o.N[2];
  o.nM = (long long)o.M[0] * o.M[1] * o.M[2];
  o.nt = p->time_steps;
  o.s = p->s;
  o.alpha = p->alpha;
  o.sigma = p->sigma;
  o.hessian = p->hessian;
  o.state = p->state;
  o.integrator = p->integrator;
  o.prec = p->precision == LDDMM_FP32_BF16X3 ? 1 : 0;
  if (p->checkpoint < 0 || p->checkpoint > o.nt)
    return fail(LDDMM_E_INVALID_ARG, "checkpoint must be in [0, time_steps]");
  if (p->checkpoint > 0 && (p->state != LDDMM_STATE_IMAGE || p->integrator != LDDMM_EULER))
    return fail(LDDMM_E_INVALID_ARG, "checkpoints need the image state and Euler steps");
  o.ckpt = p->checkpoint;
  if (!band_sizes_taken(o)) return fail(LDDMM_E_SHAPE, "band and padded grid too large together");
  apply_tiles(o);
  return LDDMM_OK;
}

// Only lddmm_gradient_exact (and the workspace size) take checkpoints.
int no_checkpoint(const Dims& d) {
  if (d.ckpt) return fail(LDDMM_E_INVALID_ARG, "checkpoint is for lddmm_gradient_exact only");
  return LDDMM_OK;
}

// The adjoint sweeps are transposes of Euler steps: only shooting takes RK4.
int euler_only(const Dims& d) {
  if (d.integrator != LDDMM_EULER)
    return fail(LDDMM_E_INVALID_ARG, "LDDMM_RK4 is for lddmm_shoot and lddmm_geodesic_energy only");
  return LDDMM_OK;
}

// ------------------------------------------- the workspace of lddmm_shoot_static
// For callers that cannot allocate device memory: a fixed array in the
// library's device code, one copy per GPU, held until the process ends.  In
// host code the name `scratch` only stands for the symbol; its device address
// on the current GPU comes from hipGetSymbolAddress, taken once per device
// and kept.  Every lddmm_shoot_static call on one GPU uses that GPU's copy,
// so such calls that overlap on one GPU race.
// Above the documented size it holds what fragment tables of few k take more
// than plain ones, so that the documented size decides what is taken: at most
// 59280 + 58976 + 33728 bytes of the three axes over all sizes that validate()
// accepts (band, padded and image size 34, 241, 34 on the first axis, 4, 249, 385
// on the second, 8, 241, 241 on the third), and less than 256 of alignment.
constexpr size_t kScratchSlack = 160 << 10;
static __device__ __align__(256) unsigned char scratch[LDDMM_STATIC_SCRATCH_BYTES + kScratchSlack];
std::mutex g_scratch_mu;
std::map<int, void*> g_scratch_ptr;  // device -> its copy of scratch

// Address of the current GPU's copy of `scratch`.
hipError_t static_scratch(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  auto it = g_scratch_ptr.find(dev);
  if (it == g_scratch_ptr.end()) {
    void* p = nullptr;
    if ((e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch))) != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    it = g_scratch_ptr.emplace(dev, p).first;
  }
  *out = it->second;
  return hipSuccess;
}

int check_ws(const Dims& d, const void* ws, size_t ws_bytes) {
  if (!ws) return fail(LDDMM_E_INVALID_ARG, "workspace is NULL");
  size_t need = Engine::workspace_bytes(d);
  if (ws_bytes < need)
    return fail(LDDMM_E_WORKSPACE, "workspace too small: need " + std::to_string(need) + " bytes");
  return LDDMM_OK;
}

// ---------------------------------------------------------------- timer
using EventPair = std::pair<hipEvent_t, hipEvent_t>;
struct Timer {
  LaunchSampler smp;    // family, one launch in `every`, the per-thread decision
  std::mutex& mu = smp.mu;
  bool error = false;
  std::vector<EventPair> pending;
  std::vector<EventPair> pool;
  int64_t launches = 0;
  double ms = 0.0;
  double flops = 0.0, bytes = 0.0;
};
Timer g_timer;

// ---------------------------------------------------------------- graphs
// Launch-bound sequences (one CG iteration, the gradient at the head of a
// Gauss-Newton iteration, one line-search trial, one Hessian-vector
// product) are captured once per device, workspace, problem, external
// pointers and timed kernel family into a HIP graph on a library stream,
// and replayed on the caller's stream.  While a family is timed, its
// launches are bracketed by external event nodes inside the graph; the
// durations of a replay are collected before the next replay of the same
// graph and by lddmm_kernel_timer_read.  The event nodes are added to the
// captured graph around each kernel node of the family (event records made
// during capture would only order streams).
struct GraphEntry {
  hipGraphExec_t exec = nullptr;
  int family = 0;
  std::vector<hipGraphNode_t> knodes;  // kernel nodes of the timed family (during capture)
  std::vector<EventPair> pairs;
  double flops = 0.0, bytes = 0.0;
  bool unharvested = false;
};
bool g_use_graphs = false;
std::mutex g_graph_mu;
std::mutex g_capture_mu;
std::map<std::string, GraphEntry> g_graphs;  // entries live until the process ends
std::map<int, hipStream_t> g_cap_streams;
thread_local GraphEntry* t_capturing = nullptr;

bool take_pair(EventPair* ev) {
  if (!g_timer.pool.empty()) {
    *ev = g_timer.pool.back();
    g_timer.pool.pop_back();
    return true;
  }
  // device-scope release: recording the pair writes back no caches for the
  // host, so the interval holds the kernel and not a system-wide fence
  if (hipEventCreateWithFlags(&ev->first, hipEventReleaseToDevice) != hipSuccess) return false;
  if (hipEventCreateWithFlags(&ev->second, hipEventReleaseToDevice) != hipSuccess) return false;
  return true;
}

// Adds the durations of the last replay of a timed graph (waits for it).
// Call with g_timer.mu held.
void harvest(GraphEntry& g) {
  if (!g.unharvested) return;
  g.unharvested = false;
  for (auto& ev : g.pairs) {
    float ms = 0.f;
    if (hipEventSynchronize(ev.second) != hipSuccess || hipEventElapsedTime(&ms, ev.first, ev.second) != hipSuccess) {
      g_timer.error = true;
      return;
    }
    g_timer.ms += ms;
    g_timer.launches += 1;
  }
}

}  // namespace

namespace lddmm {
void timer_work(int family, double flops, double bytes) {
  g_timer.smp.account(family, [&] {
    double& f = t_capturing ? t_capturing->flops : g_timer.flops;
    double& b = t_capturing ? t_capturing->bytes : g_timer.bytes;
    f += flops;
    b += bytes;
  });
}
bool timer_events(int family, hipEvent_t* start, hipEvent_t* stop) {
  if (t_capturing || !g_timer.smp.sampled(family)) return false;
  std::lock_guard<std::mutex> lk(g_timer.mu);
  EventPair ev;
  if (!take_pair(&ev)) {
    g_timer.error = true;
    return false;
  }
  g_timer.pending.push_back(ev);
  *start = ev.first;
  *stop = ev.second;
  return true;
}
void timer_captured(int family, hipStream_t st) {
  if (!t_capturing || !g_timer.smp.sampled(family)) return;
  std::lock_guard<std::mutex> lk(g_timer.mu);
  // the node the next captured operation would depend on: the kernel just launched
  hipStreamCaptureStatus cs;
  const hipGraphNode_t* deps = nullptr;
  size_t nd = 0;
  if (hipStreamGetCaptureInfo_v2(st, &cs, nullptr, nullptr, &deps, &nd) != hipSuccess || nd != 1)
    g_timer.error = true;
  else
    t_capturing->knodes.push_back(deps[0]);
}
}  // namespace lddmm

namespace {

std::string graph_key(const Engine& e, const void* ws, int kind, std::initializer_list<const void*> ext) {
  const Dims& d = e.dims();
  int dev = -1;
  (void)hipGetDevice(&dev);
  // a timed graph samples the launches the timer picked while it was captured
  const int tf = g_timer.smp.family.load();
  const int fam = tf ? tf + 256 * g_timer.smp.every.load() : 0;
  std::string k;
  auto put = [&k](const void* p, size_t n) { k.append(static_cast<const char*>(p), n); };
  put(&dev, sizeof dev);
  put(&ws, sizeof ws);
  put(&kind, sizeof kind);
  put(&fam, sizeof fam);
  put(d.N, sizeof d.N);
  put(d.K, sizeof d.K);
  put(d.M, sizeof d.M);
  put(&d.nt, sizeof d.nt);
  put(&d.s, sizeof d.s);
  put(&d.alpha, sizeof d.alpha);
  put(&d.sigma, sizeof d.sigma);
  put(&d.hessian, sizeof d.hessian);
  put(&d.state, sizeof d.state);
  put(&d.integrator, sizeof d.integrator);
  put(&d.prec, sizeof d.prec);
  put(&d.ckpt, sizeof d.ckpt);
  put(&d.tile_prod_rows, sizeof d.tile_prod_rows);
  put(&d.tile_col, sizeof d.tile_col);
  put(&d.tile_sl, sizeof d.tile_sl);
  for (const void* p : ext) put(&p, sizeof p);
  return k;
}

hipError_t capture_stream(hipStream_t* out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lk(g_graph_mu);
  hipStream_t& s = g_cap_streams[dev];
  if (!s && (e = hipStreamCreateWithFlags(&s, hipStreamNonBlocking)) != hipSuccess) return e;
  *out = s;
  return hipSuccess;
}

// Brackets each recorded kernel node of a captured graph by two event
// record nodes: its dependencies -> start -> kernel -> stop -> its dependents.
hipError_t add_timing_nodes(hipGraph_t graph, GraphEntry& ne) {
  std::lock_guard<std::mutex> lk(g_timer.mu);
  hipError_t e;
  for (hipGraphNode_t K : ne.knodes) {
    EventPair ev;
    if (!take_pair(&ev)) return hipErrorOutOfMemory;
    ne.pairs.push_back(ev);
    size_t nd = 0, nn = 0;
    if ((e = hipGraphNodeGetDependencies(K, nullptr, &nd)) != hipSuccess) return e;
    if ((e = hipGraphNodeGetDependentNodes(K, nullptr, &nn)) != hipSuccess) return e;
    std::vector<hipGraphNode_t> deps(nd), dn(nn);
    if (nd && (e = hipGraphNodeGetDependencies(K, deps.data(), &nd)) != hipSuccess) return e;
    if (nn && (e = hipGraphNodeGetDependentNodes(K, dn.data(), &nn)) != hipSuccess) return e;
    hipGraphNode_t e1, e2;
    if ((e = hipGraphAddEventRecordNode(&e1, graph, deps.data(), nd, ev.first)) != hipSuccess) return e;
    if ((e = hipGraphAddDependencies(graph, &e1, &K, 1)) != hipSuccess) return e;
    if ((e = hipGraphAddEventRecordNode(&e2, graph, &K, 1, ev.second)) != hipSuccess) return e;
    for (hipGraphNode_t d : dn) {
      if ((e = hipGraphRemoveDependencies(graph, &K, &d, 1)) != hipSuccess) return e;
      if ((e = hipGraphAddDependencies(graph, &e2, &d, 1)) != hipSuccess) return e;
    }
  }
  ne.knodes.clear();
  return hipSuccess;
}

// Runs `body` (which enqueues on e.stream() and may fork onto the engine's
// auxiliary stream, joining back before it returns) through the graph of
// `key`, capturing it on first use; with graphs disabled, runs it directly.
hipError_t run_graph(Engine& e, const std::string& key, const std::function<hipError_t()>& body) {
  if (!g_use_graphs) return body();
  GraphEntry* g = nullptr;
  {
    std::lock_guard<std::mutex> lk(g_graph_mu);
    auto it = g_graphs.find(key);
    if (it != g_graphs.end()) g = &it->second;
  }
  const hipStream_t st = e.stream();
  hipError_t err;
  // captures run one at a time (the capture stream of a device is shared by
  // the host threads of a batch)
  std::unique_lock<std::mutex> cl(g_capture_mu, std::defer_lock);
  if (!g) {
    cl.lock();
    std::lock_guard<std::mutex> lk(g_graph_mu);
    auto it = g_graphs.find(key);
    if (it != g_graphs.end()) g = &it->second;
  }
  if (!g) {
    hipStream_t cap = nullptr;
    if ((err = capture_stream(&cap)) != hipSuccess) return err;
    if ((err = e.aux_init(e.dims().nt + 2)) != hipSuccess) return err;
    GraphEntry ne;
    ne.family = g_timer.smp.family.load();
    e.set_stream(cap);
    t_capturing = &ne;
    err = hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal);
    if (err == hipSuccess) {
      const hipError_t eb = body();
      hipGraph_t graph = nullptr;
      const hipError_t ee = hipStreamEndCapture(cap, &graph);
      err = eb != hipSuccess ? eb : ee;
      if (err == hipSuccess && !ne.knodes.empty()) err = add_timing_nodes(graph, ne);
      if (err == hipSuccess) err = hipGraphInstantiateWithFlags(&ne.exec, graph, 0);
      if (graph) (void)hipGraphDestroy(graph);
    }
    t_capturing = nullptr;
    e.set_stream(st);
    if (err != hipSuccess) {
      std::lock_guard<std::mutex> lk(g_timer.mu);
      for (auto& ev : ne.pairs) g_timer.pool.push_back(ev);
      return err;
    }
    std::lock_guard<std::mutex> lk(g_graph_mu);
    g = &(g_graphs[key] = std::move(ne));
  }
  if (cl.owns_lock()) cl.unlock();
  if (!g->pairs.empty()) {
    std::lock_guard<std::mutex> lk(g_timer.mu);
    harvest(*g);
  }
  if ((err = hipGraphLaunch(g->exec, st)) != hipSuccess) return err;
  if (g->family != 0 && g->family == g_timer.smp.family.load()) {
    std::lock_guard<std::mutex> lk(g_timer.mu);
    g_timer.flops += g->flops;
    g_timer.bytes += g->bytes;
    if (!g->pairs.empty()) g->unharvested = true;
  }
  return hipSuccess;
}

enum GraphKind { GK_HESSVEC = 1, GK_GN_HEAD = 2, GK_PCG_ITER = 3, GK_GN_HEAD_KEPT = 4, GK_TRIAL = 16 };

// ------------------------------------------------------ register loop
// batched registration: at most this many pairs per call, and by default
// this many running at a time; each pair's workspace slice is 256-aligned
constexpr int kMaxBatch = 4096;
constexpr int kBatchConcurrency = 8;
size_t batch_slice(size_t bytes) { return (bytes + 255) & ~(size_t)255; }

// 64 doubles of pinned, coherent host memory per host thread, through which
// the registration loop reads its scalars without a copy command: a kernel
// at the end of the work writes the values to words 1.. and then 1 to word
// 0, which the host cleared before enqueueing it and spins on.  A thread
// holds its block from its first use until it exits; the block then returns
// to a pool that later threads draw from, so the worker threads of
// successive batched calls reuse the same blocks (and the CG graphs captured
// with them).  Blocks are never freed; null if none can be had.
constexpr int kHostWords = 64;
struct HostWordsPool {
  std::mutex mu;
  std::vector<double*> free;
};
HostWordsPool g_host_words;
struct HostWordsLease {
  double* p = nullptr;
  bool tried = false;
  ~HostWordsLease() {
    if (!p) return;
    std::lock_guard<std::mutex> lk(g_host_words.mu);
    g_host_words.free.push_back(p);
  }
};
double* host_words() {
  thread_local HostWordsLease lease;
  if (!lease.tried) {
    lease.tried = true;
    {
      std::lock_guard<std::mutex> lk(g_host_words.mu);
      if (!g_host_words.free.empty()) {
        lease.p = g_host_words.free.back();
        g_host_words.free.pop_back();
      }
    }
    if (!lease.p && hipHostMalloc(reinterpret_cast<void**>(&lease.p), kHostWords * sizeof(double),
                                  hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent) !=
                        hipSuccess) {
      (void)hipGetLastError();
      lease.p = nullptr;
    }
  }
  return lease.p;
}

// Waits until the stream's kernel has set hf[0] (spinning on the host
// memory), or the stream has finished or failed.
hipError_t wait_host_flag(double* hf, hipStream_t st) {
  volatile double* f = hf;
  for (;;) {
    for (int i = 0; i < 2048; ++i)
      if (f[0] != 0.0) return hipSuccess;
    const hipError_t q = hipStreamQuery(st);
    if (q == hipErrorNotReady) continue;
    if (q != hipSuccess) return q;
    return f[0] != 0.0 ? hipSuccess : hipErrorUnknown;
  }
}

// ------------------------------------------------------ resumable loop
// The Gauss-Newton-Krylov loop is a C++ coroutine that enqueues device work
// and suspends wherever it needs a value back from the device (the energy
// and |g| of an iteration, the CG stop flag, the CG scalars, a trial's
// energy).  lddmm_register resumes it by waiting for each value in turn; the
// batch resumes many of them from one host thread, polling whichever pairs
// have a value ready, so that no pair's host work waits for another's device
// work.  What a suspended loop waits for: hf[0] set by the stream's last
// kernel (hf non-null), or the stream finished (hf null).
struct DeviceWait {
  double* hf = nullptr;
  hipStream_t st = nullptr;
};

struct RegTask {
  struct promise_type {
    int result = LDDMM_OK;
    DeviceWait wait;
    hipError_t wait_result = hipSuccess;
    RegTask get_return_object() { return RegTask{std::coroutine_handle<promise_type>::from_promise(*this)}; }
    std::suspend_always initial_suspend() noexcept { return {}; }
    std::suspend_always final_suspend() noexcept { return {}; }
    void return_value(int r) { result = r; }
    void unhandled_exception() { result = LDDMM_E_HIP; }
  };
  using handle = std::coroutine_handle<promise_type>;
  handle h;
  RegTask() = default;
  explicit RegTask(handle hh) : h(hh) {}
  RegTask(RegTask&& o) noexcept : h(o.h) { o.h = nullptr; }
  RegTask& operator=(RegTask&& o) noexcept {
    if (this != &o) {
      if (h) h.destroy();
      h = o.h;
      o.h = nullptr;
    }
    return *this;
  }
  RegTask(const RegTask&) = delete;
  ~RegTask() {
    if (h) h.destroy();
  }
  bool done() const { return !h || h.done(); }
  int result() const { return h.promise().result; }
};

// co_await DeviceReady{hf, st}: suspends the loop until the wait is over and
// yields the wait's status.
struct DeviceReady {
  DeviceWait w;
  RegTask::handle h{};
  bool await_ready() const noexcept { return false; }
  void await_suspend(RegTask::handle hh) noexcept {
    h = hh;
    hh.promise().wait = w;
  }
  hipError_t await_resume() const noexcept { return h.promise().wait_result; }
};

DeviceReady until(double* hf, hipStream_t st) { return DeviceReady{DeviceWait{hf, st}}; }

// Non-blocking test of a wait: true when it is over (status in *r).
bool wait_over(const DeviceWait& w, hipError_t* r, bool query_stream) {
  if (w.hf && static_cast<volatile double*>(w.hf)[0] != 0.0) {
    *r = hipSuccess;
    return true;
  }
  if (!query_stream) return false;
  const hipError_t q = hipStreamQuery(w.st);
  if (q == hipErrorNotReady) return false;
  if (q != hipSuccess) {
    *r = q;
    return true;
  }
  *r = (!w.hf || static_cast<volatile double*>(w.hf)[0] != 0.0) ? hipSuccess : hipErrorUnknown;
  return true;
}

// Resumes a loop to its end on the calling thread, waiting for each value.
int run_to_end(RegTask& t) {
  t.h.resume();
  while (!t.h.done()) {
    auto& pr = t.h.promise();
    pr.wait_result = pr.wait.hf ? wait_host_flag(pr.wait.hf, pr.wait.st) : hipStreamSynchronize(pr.wait.st);
    t.h.resume();
  }
  return t.result();
}

// Enqueues the copy of a[0 .. na), b[0 .. nb) (device) to the host: to
// hf[1 ..] with hf[0] set last when hf is non-null (hf[0] cleared here),
// else to fb by copy commands; then the loop awaits DeviceWait{hf, st} and
// reads the values with read_values.
hipError_t read_enqueue(double* hf, double* fb, const double* a, int na, const double* b, int nb, hipStream_t st) {
  hipError_t r;
  if (hf) {
    static_cast<volatile double*>(hf)[0] = 0.0;
    return launch_host_copy(a, na, b, nb, hf, st);
  }
  if ((r = hipMemcpyAsync(fb, a, na * sizeof(double), hipMemcpyDeviceToHost, st))) return r;
  if (nb && (r = hipMemcpyAsync(fb + na, b, nb * sizeof(double), hipMemcpyDeviceToHost, st))) return r;
  return hipSuccess;
}
void read_values(double* out, const double* hf, const double* fb, int n) {
  const volatile double* src = hf ? static_cast<const volatile double*>(hf + 1) : fb;
  for (int i = 0; i < n; ++i) out[i] = src[i];
}

// The Gauss-Newton-Krylov loop (see lddmm_register).  hf: the pinned host
// words of this loop (or null: copy commands instead).
RegTask register_loop(Engine& e, const void* ws, const float* I0, const float* I1, void* v0_inout, int gn_iters,
                      int pcg_iters, lddmm_stats* stats, int stats_len, int64_t* hvps, double* hf) {
  const Dims& d = e.dims();
  hipStream_t st = e.stream();
  const int n = 3 * d.nb;
  const double c1 = 1e-4;
  const int max_trials = 10;
  hipError_t err;
  double fb[kHostWords];  // values read by copy commands when hf is null
#define HTRY(x)                                     \
  do {                                              \
    err = (x);                                      \
    if (err != hipSuccess) co_return hip_fail(err, #x); \
  } while (0)
  // out[0 .. na + nb) = a[0 .. na), b[0 .. nb) once the work enqueued so far has finished
#define READ_BACK(out, a, na, b, nb)                        \
  do {                                                      \
    HTRY(read_enqueue(hf, fb, (a), (na), (b), (nb), st));   \
    HTRY(co_await until(hf, st));         \
    read_values((out), hf, fb, (na) + (nb));                \
  } while (0)
  HTRY(e.init_tables());
  HTRY(e.load_band(v0_inout, e.v0h));
  // ||I0 - I1||^2 for MSE_rel
  HTRY(launch_sqdiff(I0, I1, d.nN, e.partial, e.scal + 8, 1.0, st));
  double denom = 0.0;
  READ_BACK(&denom, e.scal + 8, 1, nullptr, 0);
  double g0_inf = -1.0;
  int status = LDDMM_OK;
  // the accepted line-search trial of the previous iteration ran the caching
  // forward at the new v0 and left its energy in scal[0..2]
  bool kept = false;
  for (int it = 0; it < gn_iters; ++it) {
    // energy and gradient at v0 (and max |g|)
    HTRY(run_graph(e, graph_key(e, ws, kept ? GK_GN_HEAD_KEPT : GK_GN_HEAD, {I0, I1}), [&]() -> hipError_t {
      hipError_t r;
      const hipStream_t s = e.stream();
      if (!kept) {
        if ((r = launch_copy(reinterpret_cast<const float*>(e.v0h), reinterpret_cast<float*>(e.V[0]), 2LL * n,
                             s)))
          return r;
        if ((r = e.forward(I0)) || (r = e.energy(e.final_state(), I1))) return r;
      }
      if ((r = e.backward(I1, e.gh))) return r;
      return launch_band_maxabs(e.gh, d, e.partial, e.scal + 3, s);
    }));
    kept = false;
    double sc[4];
    READ_BACK(sc, e.scal, 4, nullptr, 0);
    if (!std::isfinite(sc[0]) || !std::isfinite(sc[3]))
      co_return fail(LDDMM_E_NONFINITE, "energy or gradient is not finite");
    if (g0_inf < 0) g0_inf = sc[3];
    // CG in the V metric on H_V p = -g_V
    HTRY(launch_pcg_init(e.gh, e.ph, e.rh, e.dh, n, st));
    HTRY(launch_band_dot(e.rh, e.rh, e.Lsym, d, e.partial, e.pcg + SC_RR, 1.0, st));
    HTRY(launch_pcg_reset(e.pcg, st));
    const std::string iter_key = graph_key(e, ws, GK_PCG_ITER, {hf});
    for (int k = 0; k < pcg_iters; ++k) {
      if (hf) static_cast<volatile double*>(hf)[0] = 0.0;
      // H d, then the CG updates (decisions taken on the device)
      HTRY(run_graph(e, iter_key, [&]() -> hipError_t {
        hipError_t r;
        const hipStream_t s = e.stream();
        if ((r = e.hessvec(e.dh, e.Hdh))) return r;
        // <d, H d>_V, then phase a; <r, r>_V, then phase b (in the reductions' last blocks)
        if ((r = launch_band_dot(e.dh, e.Hdh, e.Lsym, d, e.partial, e.pcg + SC_DHD, 1.0, s, e.count, e.pcg, 1)))
          return r;
        if ((r = launch_pcg_update_pr(e.pcg, e.dh, e.Hdh, e.ph, e.rh, n, s))) return r;
        if ((r = launch_band_dot(e.rh, e.rh, e.Lsym, d, e.partial, e.pcg + SC_RRNEW, 1.0, s, e.count, e.pcg, 2,
                                 hf)))
          return r;
        return launch_pcg_update_d(e.pcg, e.rh, e.dh, n, s);
      }));
      ++*hvps;
      double stopped = 0.0;
      if (hf) {
        HTRY(co_await until(hf, st));
        stopped = static_cast<volatile double*>(hf)[1];
      } else {
        HTRY(hipMemcpyAsync(fb, e.pcg + SC_STOPPED, sizeof(double), hipMemcpyDeviceToHost, st));
        HTRY(co_await until(nullptr, st));
        stopped = fb[0];
      }
      if (stopped != 0.0) break;
    }
    // the CG scalars and the slope <g, p>_V; fall back to -g if p is not a
    // descent direction
    double pc[SC_COUNT + 1];
    HTRY(launch_band_dot(e.gh, e.ph, e.Lsym, d, e.partial, e.scal + 4, 1.0, st));
    READ_BACK(pc, e.pcg, SC_COUNT, e.scal + 4, 1);
    double slope = pc[SC_COUNT];
    if (!(slope < 0.0)) {
      HTRY(launch_axpy_band(e.tmph, e.gh, -1.f, e.ph, n, st));  // tmph is zero-filled below
      HTRY(launch_band_dot(e.gh, e.ph, e.Lsym, d, e.partial, e.scal + 4, 1.0, st));
      READ_BACK(&slope, e.scal + 4, 1, nullptr, 0);
    }
    // Armijo backtracking
    double eps = 1.0, Etry = 0.0;
    bool ok = false;
    int trials = 0;
    for (int t = 0; t < max_trials; ++t) {
      ++trials;
      // E(v0 + eps p), by the caching forward (it costs what the light one
      // does: the same fields are written, to their cache slots), so that an
      // accepted trial leaves the trajectories of the next gradient
      HTRY(run_graph(e, graph_key(e, ws, GK_TRIAL + t, {I0, I1}), [&]() -> hipError_t {
        hipError_t r;
        const hipStream_t s = e.stream();
        if ((r = launch_axpy_band(e.v0h, e.ph, (float)eps, e.vtry, n, s))) return r;
        if ((r = launch_copy(reinterpret_cast<const float*>(e.vtry), reinterpret_cast<float*>(e.V[0]), 2LL * n, s)))
          return r;
        if ((r = e.forward(I0))) return r;
        return e.energy(e.final_state(), I1);
      }));
      READ_BACK(&Etry, e.scal, 1, nullptr, 0);
      if (std::isfinite(Etry) && Etry <= sc[0] + c1 * eps * slope) {
        ok = true;
        break;
      }
      eps *= 0.5;
    }
    if (stats && it < stats_len) {
      lddmm_stats& s = stats[it];
      std::memset(&s, 0, sizeof(s));
      s.energy = sc[0];
      s.energy_reg = sc[1];
      s.energy_data = sc[2];
      s.mse_rel = denom > 0 ? 100.0 * sc[2] * d.sigma * d.sigma * (double)d.nN / denom : 0.0;
      s.grad_inf_rel = g0_inf > 0 ? sc[3] / g0_inf : 0.0;
      s.step = ok ? eps : 0.0;
      s.trials = trials;
      s.pcg_iters = (int)pc[SC_ITERS];
      s.pcg_guard = pc[SC_GUARD] != 0.0;
    }
    if (!ok) {
      status = LDDMM_W_LINESEARCH;
      break;
    }
    HTRY(launch_copy(reinterpret_cast<const float*>(e.vtry), reinterpret_cast<float*>(e.v0h), 2LL * n, st));
    kept = true;
  }
  HTRY(e.store_band(e.v0h, nullptr, 0.f, v0_inout));
  HTRY(co_await until(nullptr, st));
  co_return status;
#undef READ_BACK
#undef HTRY
}

// ------------------------------------------------ two-dimensional problems
// A problem on the plane (paper §3.1 with d = 2: grid N0 x N1, band K0 x K1,
// two velocity components) runs as the three-dimensional problem on
// kDepthN x N0 x N1 with band kDepthK x K0 x K1 whose fields do not depend on
// the new first coordinate: images repeated over the planes, band fields in
// components 1 and 2 at first-axis frequency 0.  That problem is the planar
// one exactly: every product, derivative and symbol of such fields keeps them
// independent of the first coordinate (the derivative along it and the
// first velocity component stay zero, the symbols at k = (0, k0, k1) are the
// planar ones), and the energy's mean over voxels and its band inner product
// are unchanged.  In floating point the forward transforms along the first
// axis leave rounding-level values at its nonzero frequencies, which the
// results do not read.  The staging buffers sit after the three-dimensional
// workspace in ws.
constexpr int kDepthN = 8, kDepthK = 4;

void lift2d(const lddmm_params* p, lddmm_params* q) {
  *q = *p;
  q->ndim = 3;
  q->grid[0] = kDepthN;
  q->grid[1] = p->grid[0];
  q->grid[2] = p->grid[1];
  q->band[0] = kDepthK;
  q->band[1] = p->band[0];
  q->band[2] = p->band[1];
  q->spectral[0] = 0;
  q->spectral[1] = p->spectral[0];
  q->spectral[2] = p->spectral[1];
}

struct Stage2D {
  lddmm_params q;
  size_t ws3 = 0, total = 0;
  long long plane = 0, plane2 = 0;  // N0 N1 and K0 K1
  float *I0e = nullptr, *I1e = nullptr;  // [kDepthN][N0][N1]
  float2 *A = nullptr, *B = nullptr;     // [3][kDepthK][K0][K1]
};

// Sizes (and, with ws, the buffers) of a planar problem's staging.
int stage2d(const lddmm_params* p, void* ws, size_t ws_bytes, Stage2D* s) {
  lift2d(p, &s->q);
  Dims d;
  int rc = validate(&s->q, &d);
  if (rc) return rc;
  s->ws3 = batch_slice(Engine::workspace_bytes(d));
  s->plane = (long long)d.N[1] * d.N[2];
  s->plane2 = (long long)d.K[1] * d.K[2];
  const size_t img = batch_slice((size_t)kDepthN * s->plane * sizeof(float));
  const size_t band = batch_slice((size_t)3 * kDepthK * s->plane2 * sizeof(float2));
  s->total = s->ws3 + 2 * img + 2 * band;
  if (!ws) return LDDMM_OK;
  if (ws_bytes < s->total)
    return fail(LDDMM_E_WORKSPACE, "workspace too small: need " + std::to_string(s->total) + " bytes");
  char* b = static_cast<char*>(ws) + s->ws3;
  s->I0e = reinterpret_cast<float*>(b);
  s->I1e = reinterpret_cast<float*>(b + img);
  s->A = reinterpret_cast<float2*>(b + 2 * img);
  s->B = reinterpret_cast<float2*>(b + 2 * img + band);
  return LDDMM_OK;
}

#define TRY2D(x)                                   \
  do {                                             \
    const hipError_t e2 = (x);                     \
    if (e2 != hipSuccess) return hip_fail(e2, #x); \
  } while (0)

}  // namespace

extern "C" {

int lddmm_workspace_bytes(const lddmm_params* p, size_t* bytes) {
  if (p && p->ndim == 2) {
    Stage2D st;
    int rc = stage2d(p, nullptr, 0, &st);
    if (rc) return rc;
    if (!bytes) return fail(LDDMM_E_INVALID_ARG, "bytes is NULL");
    *bytes = st.total;
    return LDDMM_OK;
  }
  Dims d;
  int rc = validate(p, &d);
  if (rc) return rc;
  if (!bytes) return fail(LDDMM_E_INVALID_ARG, "bytes is NULL");
  *bytes = Engine::workspace_bytes(d);
  return LDDMM_OK;
}

int lddmm_shoot(const lddmm_params* p, const float* I0, const void* v0, float* m1, void* v1,
                void* ws, size_t ws_bytes, void* stream) {
  if (p && p->ndim == 2) {
    Stage2D g;
    int rc = stage2d(p, ws, ws_bytes, &g);
    if (rc) return rc;
    if (!I0 || !v0 || !m1) return fail(LDDMM_E_INVALID_ARG, "null input or output");
    const hipStream_t st = static_cast<hipStream_t>(stream);
    TRY2D(launch_embed_image(I0, g.I0e, g.plane, kDepthN, st));
    TRY2D(launch_embed_band(static_cast<const float2*>(v0), g.A, kDepthK, g.plane2, st));
    if ((rc = lddmm_shoot(&g.q, g.I0e, g.A, g.I1e, v1 ? g.B : nullptr, ws, g.ws3, stream))) return rc;
    TRY2D(launch_copy(g.I1e, m1, g.plane, st));
    if (v1) TRY2D(launch_extract_band(g.B, static_cast<float2*>(v1), kDepthK, g.plane2, st));
    return LDDMM_OK;
  }
  Dims d;
  int rc = validate(p, &d);
  if (rc) return rc;
  if ((rc = no_checkpoint(d))) return rc;
  if (!I0 || !v0 || !m1) return fail(LDDMM_E_INVALID_ARG, "null input or output");
  if ((rc = check_ws(d, ws, ws_bytes))) return rc;
  set_prepared(ws, false, d);
  Engine e(d, ws, static_cast<hipStream_t>(stream));
  hipError_t err;
  if ((err = e.init_tables()) != hipSuccess) return hip_fail(err, "tables");
  if ((err = e.load_band(v0, e.V[0])) != hipSuccess) return hip_fail(err, "load v0");
  const float* mnt = nullptr;
  if ((err = e.forward_light(I0, &mnt)) != hipSuccess) return hip_fail(err, "shoot");
  if ((err = launch_copy(mnt, m1, d.nN, e.stream())) != hipSuccess) return hip_fail(err, "copy m1");
  if (v1 && (err = e.store_band(e.V[d.nt], nullptr, 0.f, v1)) != hipSuccess)
    return hip_fail(err, "store v1");
  g_last_error.clear();
  return LDDMM_OK;
}

int lddmm_shoot_static(const lddmm_params* p, const float* I0, const void* v0, float* m1, void* v1,
                       void* stream) {
  if (p && p->ndim == 2) return fail(LDDMM_E_SHAPE, "lddmm_shoot_static takes three-dimensional problems");
  Dims d;
  int rc = validate(p, &d);
  if (rc) return rc;
  if ((rc = no_checkpoint(d))) return rc;
  if (!I0 || !v0 || !m1) return fail(LDDMM_E_INVALID_ARG, "null input or output");
  const size_t need = Engine::workspace_bytes(d);
  if (need - Engine::table_surplus(d) > LDDMM_STATIC_SCRATCH_BYTES || need > sizeof(scratch))
    return fail(LDDMM_E_WORKSPACE, "problem needs " + std::to_string(need) + " bytes of workspace, more than the " +
                                       std::to_string((size_t)LDDMM_STATIC_SCRATCH_BYTES) +
                                       " of lddmm_shoot_static; use lddmm_shoot with a caller workspace");
  void* ws = nullptr;
  hipError_t err;
  if ((err = static_scratch(&ws)) != hipSuccess) return hip_fail(err, "static workspace");
  // the caller's stream only: no auxiliary stream or event is created
  Engine e(d, ws, static_cast<hipStream_t>(stream));
  e.set_one_stream(true);
  if ((err = e.init_tables()) != hipSuccess) return hip_fail(err, "tables");
  if ((err = e.load_band(v0, e.V[0])) != hipSuccess) return hip_fail(err, "load v0");
  const float* mnt = nullptr;
  if ((err = e.forward_light(I0, &mnt)) != hipSuccess) return hip_fail(err, "shoot");
  if ((err = launch_copy(mnt, m1, d.nN, e.stream())) != hipSuccess) return hip_fail(err, "copy m1");
  if (v1 && (err = e.store_band(e.V[d.nt], nullptr, 0.f, v1)) != hipSuccess) return hip_fail(err, "store v1");
  g_last_error.clear();
  return LDDMM_OK;
}

int lddmm_apply_symbol(const lddmm_params* p, int32_t which, const void* in, void* out, void* ws,
                       size_t ws_bytes, void* stream) {
  if (p && p->ndim == 2) {
    Stage2D g;
    int rc = stage2d(p, ws, ws_bytes, &g);
    if (rc) return rc;
    if (!in || !out) return fail(LDDMM_E_INVALID_ARG, "null input or output");
    const hipStream_t st = static_cast<hipStream_t>(stream);
    TRY2D(launch_embed_band(static_cast<const float2*>(in), g.A, kDepthK, g.plane2, st));
    if ((rc = lddmm_apply_symbol(&g.q, which, g.A, g.B, ws, g.ws3, stream))) return rc;
    TRY2D(launch_extract_band(g.B, static_cast<float2*>(out), kDepthK, g.plane2, st));
    return LDDMM_OK;
  }
  Dims d;
  int rc = validate(p, &d);
  if (rc) return rc;
  if (which != LDDMM_SYMBOL_L && which != LDDMM_SYMBOL_K) return fail(LDDMM_E_INVALID_ARG, "unknown symbol");
  if (!in || !out) return fail(LDDMM_E_INVALID_ARG, "null input or output");
  if ((rc = check_ws(d, ws, ws_bytes))) return rc;
  Engine e(d, ws, static_cast<hipStream_t>(stream));
  hipError_t err;
  if ((err = e.init_tables()) != hipSuccess) return hip_fail(err, "tables");
  if ((err = e.load_band(in, e.tmph)) != hipSuccess) return hip_fail(err, "load");
  if ((err = e.store_band(e.tmph, nullptr, 0.f, out, which == LDDMM_SYMBOL_L ? e.Lsym : e.Ksym)) != hipSuccess)
    return hip_fail(err, "store");
  g_last_error.clear();
  return LDDMM_OK;
}

int lddmm_geodesic_energy(const lddmm_params* p, const void* v0, double* energies, void* ws,
                          size_t ws_bytes, void* stream) {
  if (p && p->ndim == 2) {
    Stage2D g;
    int rc = stage2d(p, ws, ws_bytes, &g);
    if (rc) return rc;
    if (!v0 || !energies) return fail(LDDMM_E_INVALID_ARG, "null input or output");
    TRY2D(launch_embed_band(static_cast<const float2*>(v0), g.A, kDepthK, g.plane2, static_cast<hipStream_t>(stream)));
    return lddmm_geodesic_energy(&g.q, g.A, energies, ws, g.ws3, stream);
  }
  Dims d;
  int rc = validate(p, &d);
  if (rc) return rc;
  if ((rc = no_checkpoint(d))) return rc;
  if (!v0 || !energies) return fail(LDDMM_E_INVALID_ARG, "null input or output");
  if ((rc = check_ws(d, ws, ws_bytes))) return rc;
  set_prepared(ws, false, d);
  Engine e(d, ws, static_cast<hipStream_t>(stream));
  hipError_t err;
  if ((err = e.init_tables()) != hipSuccess) return hip_fail(err, "tables");
  if ((err = e.load_band(v0, e.V[0])) != hipSuccess) return hip_fail(err, "load v0");
  if ((err = e.geodesic_energies(energies)) != hipSuccess) return hip_fail(err, "geodesic energies");
  g_last_error.clear();
  return LDDMM_OK;
}

int lddmm_gradient(const lddmm_params* p, const float* I0, const float* I1, const void* v0,
                   void* grad, double* energy3, void* ws, size_t ws_bytes, void* stream) {
  if (p && p->ndim == 2) {
    Stage2D g;
    int rc = stage2d(p, ws, ws_bytes, &g);
    if (rc) return rc;
    if (!I0 || !I1 || !v0 || !grad) return fail(LDDMM_E_INVALID_ARG, "null input or output");
    const hipStream_t st = static_cast<hipStream_t>(stream);
    TRY2D(launch_embed_image(I0, g.I0e, g.plane, kDepthN, st));
    TRY2D(launch_embed_image(I1, g.I1e, g.plane, kDepthN, st));
    TRY2D(launch_embed_band(static_cast<const float2*>(v0), g.A, kDepthK, g.plane2, st));
    if ((rc = lddmm_gradient(&g.q, g.I0e, g.I1e, g.A, g.B, energy3, ws, g.ws3, stream))) return rc;
    TRY2D(launch_extract_band(g.B, static_cast<float2*>(grad), kDepthK, g.plane2, st));
    return LDDMM_OK;
  }
  Dims d;
  int rc = validate(p, &d);
  if (rc) return rc;
  if ((rc = no_checkpoint(d))) return rc;
  if ((rc = euler_only(d))) return rc;
  if (!I0 || !I1 || !v0 || !grad) return fail(LDDMM_E_INVALID_ARG, "null input or output");
  if ((rc = check_ws(d, ws, ws_bytes))) return rc;
  set_prepared(ws, false, d);
  Engine e(d, ws, static_cast<hipStream_t>(stream));
  hipError_t err;
  if ((err = e.init_tables()) != hipSuccess) return hip_fail(err, "tables");
  if ((err = e.load_band(v0, e.V[0])) != hipSuccess) return hip_fail(err, "load v0");
  if ((err = e.forward(I0)) != hipSuccess) return hip_fail(err, "forward");
  if ((err = e.energy(e.final_state(), I1)) != hipSuccess) return hip_fail(err, "energy");
  if ((err = e.backward(I1, nullptr)) != hipSuccess) return hip_fail(err, "backward");
  if ((err = e.store_band(e.V[0], e.W[0], 1.f, grad)) != hipSuccess) return hip_fail(err, "store");
  if (energy3 && (err = launch_scalar_copy(e.scal, energy3, 3, e.stream())) != hipSuccess)
    return hip_fail(err, "energy copy");
  set_prepared(ws, true, d);
  g_last_error.clear();
  return LDDMM_OK;
}

int lddmm_energy(const lddmm_params* p, const float* I0, const float* I1, const void* v0, double* energy3,
                 void* ws, size_t ws_bytes, void* stream) {
  if (p && p->ndim == 2) {
    Stage2D g;
    int rc = stage2d(p, ws, ws_bytes, &g);
    if (rc) return rc;
    if (!I0 || !I1 || !v0 || !energy3) return fail(LDDMM_E_INVALID_ARG, "null input or output");
    const hipStream_t st = static_cast<hipStream_t>(stream);
    TRY2D(launch_embed_image(I0, g.I0e, g.plane, kDepthN, st));
    TRY2D(launch_embed_image(I1, g.I1e, g.plane, kDepthN, st));
    TRY2D(launch_embed_band(static_cast<const float2*>(v0), g.A, kDepthK, g.plane2, st));
    return lddmm_energy(&g.q, g.I0e, g.I1e, g.A, energy3, ws, g.ws3, stream);
  }
  Dims d;
  int rc = validate(p, &d);
  if (rc) return rc;
  if (d.ckpt && (d.state != LDDMM_STATE_IMAGE || d.integrator != LDDMM_EULER))
    return fail(LDDMM_E_INVALID_ARG, "checkpoints need the image state and Euler steps");
  if (!I0 || !I1 || !v0 || !energy3) return fail(LDDMM_E_INVALID_ARG, "null input or output");
  if ((rc = check_ws(d, ws, ws_bytes))) return rc;
  set_prepared(ws, false, d);
  Engine e(d, ws, static_cast<hipStream_t>(stream));
  hipError_t err;
  if ((err = e.init_tables()) != hipSuccess) return hip_fail(err, "tables");
  if ((err = e.load_band(v0, e.V[0])) != hipSuccess) return hip_fail(err, "load v0");
  const float* mnt = nullptr;
  if (d.ckpt) {  // the checkpointed layout has no light-forward buffers
    if ((err = e.forward_ckpt(I0)) != hipSuccess) return hip_fail(err, "shoot");
    mnt = e.final_state();
  } else if ((err = e.forward_light(I0, &mnt)) != hipSuccess) {
    return hip_fail(err, "shoot");
  }
  if ((err = e.energy(mnt, I1)) != hipSuccess) return hip_fail(err, "energy");
  if ((err = launch_scalar_copy(e.scal, energy3, 3, e.stream())) != hipSuccess) return hip_fail(err, "energy copy");
  g_last_error.clear();
  return LDDMM_OK;
}

int lddmm_gradient_exact(const lddmm_params* p, const float* I0, const float* I1, const void* v0,
                         void* grad, double* energy3, void* ws, size_t ws_bytes, void* stream) {
  if (p && p->ndim == 2) {
    Stage2D g;
    int rc = stage2d(p, ws, ws_bytes, &g);
    if (rc) return rc;
    if (!I0 || !I1 || !v0 || !grad) return fail(LDDMM_E_INVALID_ARG, "null input or output");
    const hipStream_t st = static_cast<hipStream_t>(stream);
    TRY2D(launch_embed_image(I0, g.I0e, g.plane, kDepthN, st));
    TRY2D(launch_embed_image(I1, g.I1e, g.plane, kDepthN, st));
    TRY2D(launch_embed_band(static_cast<const float2*>(v0), g.A, kDepthK, g.plane2, st));
    if ((rc = lddmm_gradient_exact(&g.q, g.I0e, g.I1e, g.A, g.B, energy3, ws, g.ws3, stream))) return rc;
    TRY2D(launch_extract_band(g.B, static_cast<float2*>(grad), kDepthK, g.plane2, st));
    return LDDMM_OK;
  }
  Dims d;
  int rc = validate(p, &d);
  if (rc) return rc;
  if ((rc = euler_only(d))) return rc;
  if (d.state != LDDMM_STATE_IMAGE) return fail(LDDMM_E_INVALID_ARG, "the exact gradient is for the image state");
  if (!I0 || !I1 || !v0 || !grad) return fail(LDDMM_E_INVALID_ARG, "null input or output");
  if ((rc = check_ws(d, ws, ws_bytes))) return rc;
  set_prepared(ws, false, d);
  Engine e(d, ws, static_cast<hipStream_t>(stream));
  hipError_t err;
  if ((err = e.init_tables()) != hipSuccess) return hip_fail(err, "tables");
  if ((err = e.load_band(v0, e.V[0])) != hipSuccess) return hip_fail(err, "load v0");
  if ((err = e.forward_ckpt(I0)) != hipSuccess) return hip_fail(err, "forward");
  if ((err = e.energy(e.final_state(), I1)) != hipSuccess) return hip_fail(err, "energy");
  if ((err = e.backward_exact(I1, e.gh)) != hipSuccess) return hip_fail(err, "backward");
  if ((err = e.store_band(e.gh, nullptr, 0.f, grad)) != hipSuccess) return hip_fail(err, "store");
  if (energy3 && (err = launch_scalar_copy(e.scal, energy3, 3, e.stream())) != hipSuccess)
    return hip_fail(err, "energy copy");
  // the exact Gauss-Newton product may follow on an unchecked workspace
  if (d.hessian == LDDMM_GN_EXACT && d.ckpt == 0) set_prepared(ws, true, d);
  g_last_error.clear();
  return LDDMM_OK;
}

int lddmm_hessvec(const lddmm_params* p, const void* dv0, void* Hdv, void* ws, size_t ws_bytes,
                  void* stream) {
  if (p && p->ndim == 2) {
    Stage2D g;
    int rc = stage2d(p, ws, ws_bytes, &g);
    if (rc) return rc;
    if (!dv0 || !Hdv) return fail(LDDMM_E_INVALID_ARG, "null input or output");
    if (dv0 == Hdv) return fail(LDDMM_E_INVALID_ARG, "Hdv may not alias dv0");
    const hipStream_t st = static_cast<hipStream_t>(stream);
    TRY2D(launch_embed_band(static_cast<const float2*>(dv0), g.A, kDepthK, g.plane2, st));
    if ((rc = lddmm_hessvec(&g.q, g.A, g.B, ws, g.ws3, stream))) return rc;
    TRY2D(launch_extract_band(g.B, static_cast<float2*>(Hdv), kDepthK, g.plane2, st));
    return LDDMM_OK;
  }
  Dims d;
  int rc = validate(p, &d);
  if (rc) return rc;
  if ((rc = no_checkpoint(d))) return rc;
  if ((rc = euler_only(d))) return rc;
  if (!dv0 || !Hdv) return fail(LDDMM_E_INVALID_ARG, "null input or output");
  if (dv0 == Hdv) return fail(LDDMM_E_INVALID_ARG, "Hdv may not alias dv0");
  if ((rc = check_ws(d, ws, ws_bytes))) return rc;
  {
    std::lock_guard<std::mutex> lk(g_ws_mu);
    auto it = g_ws.find(ws);
    if (it == g_ws.end() || !it->second.prepared || !same_dims(it->second.dims, d))
      return fail(LDDMM_E_NOT_PREPARED, "no lddmm_gradient with these parameters on this workspace");
  }
  Engine e(d, ws, static_cast<hipStream_t>(stream));
  hipError_t err;
  if ((err = e.load_band(dv0, e.dV[0])) != hipSuccess) return hip_fail(err, "load dv0");
  if ((err = run_graph(e, graph_key(e, ws, GK_HESSVEC, {}), [&] { return e.hessvec(e.dV[0], e.Hdh); })) !=
      hipSuccess)
    return hip_fail(err, "hessvec");
  if ((err = e.store_band(e.Hdh, nullptr, 0.f, Hdv)) != hipSuccess) return hip_fail(err, "store");
  g_last_error.clear();
  return LDDMM_OK;
}

int lddmm_register(const lddmm_params* p, const float* I0, const float* I1, void* v0_inout,
                   int32_t gn_iters, int32_t pcg_iters, lddmm_stats* stats, int32_t stats_len,
                   void* ws, size_t ws_bytes, void* stream) {
  if (p && p->ndim == 2) {
    Stage2D g;
    int rc = stage2d(p, ws, ws_bytes, &g);
    if (rc) return rc;
    if (!I0 || !I1 || !v0_inout) return fail(LDDMM_E_INVALID_ARG, "null input or output");
    const hipStream_t st = static_cast<hipStream_t>(stream);
    TRY2D(launch_embed_image(I0, g.I0e, g.plane, kDepthN, st));
    TRY2D(launch_embed_image(I1, g.I1e, g.plane, kDepthN, st));
    TRY2D(launch_embed_band(static_cast<const float2*>(v0_inout), g.A, kDepthK, g.plane2, st));
    rc = lddmm_register(&g.q, g.I0e, g.I1e, g.A, gn_iters, pcg_iters, stats, stats_len, ws, g.ws3, stream);
    if (rc < 0) return rc;
    TRY2D(launch_extract_band(g.A, static_cast<float2*>(v0_inout), kDepthK, g.plane2, st));
    TRY2D(hipStreamSynchronize(st));
    return rc;
  }
  Dims d;
  int rc = validate(p, &d);
  if (rc) return rc;
  if ((rc = no_checkpoint(d))) return rc;
  if ((rc = euler_only(d))) return rc;
  if (!I0 || !I1 || !v0_inout) return fail(LDDMM_E_INVALID_ARG, "null input or output");
  if (gn_iters < 0 || pcg_iters < 1) return fail(LDDMM_E_INVALID_ARG, "bad iteration counts");
  if ((rc = check_ws(d, ws, ws_bytes))) return rc;
  set_prepared(ws, false, d);
  Engine e(d, ws, static_cast<hipStream_t>(stream));
  // zero-filled scratch used to negate the gradient
  hipError_t err = launch_fill(reinterpret_cast<float*>(e.tmph), 6LL * d.nb, 0.f, e.stream());
  if (err != hipSuccess) return hip_fail(err, "fill");
  g_last_hvps = 0;
  RegTask t = register_loop(e, ws, I0, I1, v0_inout, gn_iters, pcg_iters, stats, stats_len, &g_last_hvps,
                            host_words());
  rc = run_to_end(t);
  if (rc >= 0) g_last_error.clear();
  return rc;
}

int64_t lddmm_last_register_hvps(void) { return g_last_hvps; }

int lddmm_batch_workspace_bytes(int32_t n, const lddmm_params* p, size_t* bytes) {
  if (n < 1 || n > kMaxBatch) return fail(LDDMM_E_INVALID_ARG, "n must be in [1, 4096]");
  if (!p || !bytes) return fail(LDDMM_E_INVALID_ARG, "params or bytes is NULL");
  size_t total = 0;
  for (int i = 0; i < n; ++i) {
    Dims d;
    int rc = validate(&p[i], &d);
    if (!rc) rc = no_checkpoint(d);
    if (rc) return fail(rc, "pair " + std::to_string(i) + ": " + g_last_error);
    total += batch_slice(Engine::workspace_bytes(d));
  }
  *bytes = total;
  return LDDMM_OK;
}

int lddmm_register_batch(int32_t n, const lddmm_params* p, const float* const* I0, const float* const* I1,
                         void* const* v0_inout, int32_t gn_iters, int32_t pcg_iters, int32_t concurrency,
                         lddmm_stats* stats, int32_t stats_len, int32_t* status, int64_t* hvps, void* ws,
                         size_t ws_bytes, void* stream) {
  if (n < 1 || n > kMaxBatch) return fail(LDDMM_E_INVALID_ARG, "n must be in [1, 4096]");
  if (!p || !I0 || !I1 || !v0_inout || !ws) return fail(LDDMM_E_INVALID_ARG, "null argument");
  if (gn_iters < 0 || pcg_iters < 1) return fail(LDDMM_E_INVALID_ARG, "bad iteration counts");
  if (concurrency < 0 || concurrency > 64) return fail(LDDMM_E_INVALID_ARG, "concurrency must be in [0, 64]");
  if (stats && stats_len < 0) return fail(LDDMM_E_INVALID_ARG, "negative stats_len");
  std::vector<Dims> dims(n);
  std::vector<size_t> off(n);
  size_t total = 0;
  for (int i = 0; i < n; ++i) {
    int rc = validate(&p[i], &dims[i]);
    if (!rc) rc = euler_only(dims[i]);
    if (!rc) rc = no_checkpoint(dims[i]);
    if (rc) return fail(rc, "pair " + std::to_string(i) + ": " + g_last_error);
    if (!I0[i] || !I1[i] || !v0_inout[i])
      return fail(LDDMM_E_INVALID_ARG, "pair " + std::to_string(i) + ": null input or output");
    off[i] = total;
    total += batch_slice(Engine::workspace_bytes(dims[i]));
  }
  if (ws_bytes < total)
    return fail(LDDMM_E_WORKSPACE, "workspace too small: need " + std::to_string(total) + " bytes");
  int dev = 0;
  hipError_t err = hipGetDevice(&dev);
  if (err != hipSuccess) return hip_fail(err, "device");
  // the pairs start after the work already on the caller's stream
  hipEvent_t start = nullptr;
  if ((err = hipEventCreateWithFlags(&start, hipEventDisableTiming)) != hipSuccess) return hip_fail(err, "event");
  if ((err = hipEventRecord(start, static_cast<hipStream_t>(stream))) != hipSuccess) {
    (void)hipEventDestroy(start);
    return hip_fail(err, "event record");
  }
  std::vector<int> rcs(n, LDDMM_OK);
  std::vector<std::string> msgs(n);
  std::vector<int64_t> counts(n, 0);
  // largest pairs first (workspace size as the measure of work), so that the
  // last pairs to finish are small ones and the tail of the batch is short
  std::vector<int> order(n);
  for (int i = 0; i < n; ++i) order[i] = i;
  std::stable_sort(order.begin(), order.end(),
                   [&](int a, int b) { return Engine::workspace_bytes(dims[a]) > Engine::workspace_bytes(dims[b]); });
  // pinned host words per pair, drawn from the pool in pair order and
  // returned in reverse, so that a repeated call gives pair i the same block
  // (and replays the CG graphs captured with it)
  std::vector<double*> words(n, nullptr);
  {
    std::lock_guard<std::mutex> lk(g_host_words.mu);
    for (int i = 0; i < n; ++i) {
      if (!g_host_words.free.empty()) {
        words[i] = g_host_words.free.back();
        g_host_words.free.pop_back();
      } else if (hipHostMalloc(reinterpret_cast<void**>(&words[i]), kHostWords * sizeof(double),
                               hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess) {
        (void)hipGetLastError();
        words[i] = nullptr;
      }
    }
  }
  // `concurrency` slots, each with a stream of its own; every slot runs one
  // pair's loop at a time and takes the next pair of that order when it ends.
  // All loops are resumed from this thread (see register_loop).
  struct Slot {
    hipStream_t s = nullptr;
    int pair = -1;
    std::unique_ptr<Engine> eng;
    RegTask task;
  };
  const int nw = std::min<int>(n, concurrency ? concurrency : kBatchConcurrency);
  std::vector<Slot> slots(nw);
  for (Slot& sl : slots) {
    if (err == hipSuccess) err = hipStreamCreateWithFlags(&sl.s, hipStreamNonBlocking);
    if (err == hipSuccess) err = hipStreamWaitEvent(sl.s, start, 0);
  }
  int next = 0;
  auto finish = [&](Slot& sl) {
    const int i = sl.pair;
    rcs[i] = sl.task.result();
    if (rcs[i] < 0) msgs[i] = g_last_error;
    sl.task = RegTask();
    sl.eng.reset();
    sl.pair = -1;
  };
  // starts the next pair in the slot; false when none is left
  auto start_pair = [&](Slot& sl) -> bool {
    while (next < n) {
      const int i = order[next++];
      void* w = static_cast<char*>(ws) + off[i];
      set_prepared(w, false, dims[i]);
      sl.eng = std::make_unique<Engine>(dims[i], w, sl.s);
      sl.eng->set_one_stream(true);
      const hipError_t fe = launch_fill(reinterpret_cast<float*>(sl.eng->tmph), 6LL * dims[i].nb, 0.f, sl.s);
      sl.pair = i;
      if (fe != hipSuccess) {
        rcs[i] = hip_fail(fe, "fill");
        msgs[i] = g_last_error;
        sl.eng.reset();
        sl.pair = -1;
        continue;
      }
      sl.task = register_loop(*sl.eng, w, I0[i], I1[i], v0_inout[i], gn_iters, pcg_iters,
                              stats ? stats + (size_t)i * stats_len : nullptr, stats ? stats_len : 0, &counts[i],
                              words[i]);
      sl.task.h.resume();
      if (!sl.task.done()) return true;
      finish(sl);
    }
    return false;
  };
  if (err == hipSuccess) {
    int active = 0;
    for (Slot& sl : slots)
      if (start_pair(sl)) ++active;
    // a loop waiting for a flag is resumed once the flag is set; its stream
    // is queried (for a failure that would leave the flag unset) every 64th
    // round, a loop waiting for its stream to finish every round
    for (unsigned round = 1; active > 0; ++round) {
      const bool query = round % 64 == 0;
      for (Slot& sl : slots) {
        if (sl.pair < 0) continue;
        auto& pr = sl.task.h.promise();
        hipError_t r;
        if (!wait_over(pr.wait, &r, query || !pr.wait.hf)) continue;
        pr.wait_result = r;
        sl.task.h.resume();
        if (!sl.task.done()) continue;
        finish(sl);
        if (!start_pair(sl)) --active;
      }
    }
  } else {
    for (int i = 0; i < n; ++i) {
      rcs[i] = hip_fail(err, "batch stream");
      msgs[i] = g_last_error;
    }
  }
  for (Slot& sl : slots)
    if (sl.s) {
      (void)hipStreamSynchronize(sl.s);
      (void)hipStreamDestroy(sl.s);
    }
  (void)hipEventDestroy(start);
  {
    std::lock_guard<std::mutex> lk(g_host_words.mu);
    for (int i = n - 1; i >= 0; --i)
      if (words[i]) g_host_words.free.push_back(words[i]);
  }
  int result = LDDMM_OK;
  int64_t sum = 0;
  for (int i = 0; i < n; ++i) {
    if (status) status[i] = rcs[i];
    if (hvps) hvps[i] = counts[i];
    sum += counts[i];
    if (rcs[i] < 0 && result >= 0) {
      result = rcs[i];
      g_last_error = "pair " + std::to_string(i) + ": " + msgs[i];
    } else if (rcs[i] == LDDMM_W_LINESEARCH && result == LDDMM_OK) {
      result = LDDMM_W_LINESEARCH;
    }
  }
  g_last_hvps = sum;
  if (result >= 0) g_last_error.clear();
  return result;
}

int lddmm_kernel_timer(int32_t family, int32_t every) {
  if (family < LDDMM_KF_NONE || family > KF_LAST) return fail(LDDMM_E_INVALID_ARG, "unknown kernel family");
  if (every < 1 || every > 1000) return fail(LDDMM_E_INVALID_ARG, "every must be in [1, 1000]");
  std::lock_guard<std::mutex> lg(g_graph_mu);
  std::lock_guard<std::mutex> lk(g_timer.mu);
  for (auto& ev : g_timer.pending) g_timer.pool.push_back(ev);
  g_timer.pending.clear();
  for (auto& kv : g_graphs) kv.second.unharvested = false;
  g_timer.error = false;
  g_timer.smp.family.store(family);
  g_timer.smp.every.store(every);
  g_timer.smp.seen = 0;
  g_timer.launches = 0;
  g_timer.ms = 0.0;
  g_timer.flops = 0.0;
  g_timer.bytes = 0.0;
  return LDDMM_OK;
}

int lddmm_kernel_timer_read(int64_t* launches, double* total_ms, double* flops, double* bytes) {
  std::lock_guard<std::mutex> lg(g_graph_mu);
  std::lock_guard<std::mutex> lk(g_timer.mu);
  for (auto& kv : g_graphs) harvest(kv.second);
  for (auto& ev : g_timer.pending) {
    if (hipEventSynchronize(ev.second) != hipSuccess) return fail(LDDMM_E_HIP, "event sync");
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, ev.first, ev.second) != hipSuccess)
      return fail(LDDMM_E_HIP, "event elapsed");
    g_timer.ms += ms;
    g_timer.launches += 1;
    g_timer.pool.push_back(ev);
  }
  g_timer.pending.clear();
  if (g_timer.error) return fail(LDDMM_E_HIP, "a timing event could not be created, recorded or read");
  if (launches) *launches = g_timer.launches;
  if (total_ms) *total_ms = g_timer.ms;
  if (flops) *flops = g_timer.flops;
  if (bytes) *bytes = g_timer.bytes;
  return LDDMM_OK;
}

int lddmm_use_graphs(int32_t enable) {
  if (enable != 0 && enable != 1) return fail(LDDMM_E_INVALID_ARG, "enable must be 0 or 1");
  g_use_graphs = enable != 0;
  return LDDMM_OK;
}

const char* lddmm_status_string(int code) {
  switch (code) {
    case LDDMM_OK: return "ok";
    case LDDMM_W_LINESEARCH: return "line search failed; last accepted iterate returned";
    case LDDMM_E_INVALID_ARG: return "invalid argument";
    case LDDMM_E_SHAPE: return "unsupported shape";
    case LDDMM_E_WORKSPACE: return "workspace too small";
    case LDDMM_E_HIP: return "HIP runtime error";
    case LDDMM_E_NOT_PREPARED: return "hessvec needs a preceding gradient on this workspace";
    case LDDMM_E_NONFINITE: return "non-finite energy or gradient";
    default: return "unknown status";
  }
}

const char* lddmm_last_error(void) { return g_last_error.c_str(); }

int lddmm_tiles_set(const lddmm_params* p, const char* arch, const lddmm_tiles* t) {
  Dims d;
  int rc = validate(p, &d);
  if (rc) return rc;
  if (!t) return fail(LDDMM_E_INVALID_ARG, "tiles is NULL");
  if ((rc = check_tiles(d, *t))) return rc;
  const std::string a = arch ? std::string(arch) : current_arch();
  if (a.empty()) return fail(LDDMM_E_INVALID_ARG, "no arch given and no current device");
  std::lock_guard<std::mutex> lk(g_tiles_mu);
  TileEntry& e = g_tiles[tile_key(d, a)];
  e.t = *t;
  e.ms = 0.0;
  g_tiles_any.store(true);
  return LDDMM_OK;
}

int lddmm_tiles_get(const lddmm_params* p, const char* arch, lddmm_tiles* t, int32_t* found) {
  Dims d;
  int rc = validate(p, &d);
  if (rc) return rc;
  if (!t || !found) return fail(LDDMM_E_INVALID_ARG, "tiles or found is NULL");
  const std::string a = arch ? std::string(arch) : current_arch();
  std::lock_guard<std::mutex> lk(g_tiles_mu);
  auto it = g_tiles.find(tile_key(d, a));
  *found = it != g_tiles.end();
  *t = *found ? it->second.t : lddmm_tiles{};
  return LDDMM_OK;
}

int lddmm_tiles_clear(void) {
  std::lock_guard<std::mutex> lk(g_tiles_mu);
  g_tiles.clear();
  g_tiles_any.store(false);
  return LDDMM_OK;
}

int lddmm_tiles_save(const char* path) {
  if (!path) return fail(LDDMM_E_INVALID_ARG, "path is NULL");
  std::string out = "{\"format\": \"lddmm-tiles-1\", \"entries\": [";
  {
    std::lock_guard<std::mutex> lk(g_tiles_mu);
    bool first = true;
    for (auto& kv : g_tiles) {
      const TileKey& k = kv.first;
      char buf[512];
      std::snprintf(buf, sizeof buf,
                    "%s\n  {\"arch\": \"%s\", \"grid\": [%d, %d, %d], \"band\": [%d, %d, %d], "
                    "\"spectral\": [%d, %d, %d], \"precision\": \"%s\", \"prod_rows\": %d, \"col_split\": %d, "
                    "\"sl_threads\": %d, \"ms_per_hvp\": %.6f}",
                    first ? "" : ",", k.arch.c_str(), k.N[0], k.N[1], k.N[2], k.K[0], k.K[1], k.K[2], k.M[0],
                    k.M[1], k.M[2], k.prec ? "bf16x3" : "fp32", kv.second.t.prod_rows, kv.second.t.col_split,
                    kv.second.t.sl_threads, kv.second.ms);
      out += buf;
      first = false;
    }
  }
  out += "\n]}\n";
  FILE* f = std::fopen(path, "wb");
  if (!f) return fail(LDDMM_E_INVALID_ARG, std::string("cannot write ") + path);
  const bool ok = std::fwrite(out.data(), 1, out.size(), f) == out.size();
  if (std::fclose(f) != 0 || !ok) return fail(LDDMM_E_INVALID_ARG, std::string("write failed: ") + path);
  return LDDMM_OK;
}

int lddmm_tiles_load(const char* path) {
  if (!path) return fail(LDDMM_E_INVALID_ARG, "path is NULL");
  FILE* f = std::fopen(path, "rb");
  if (!f) return fail(LDDMM_E_INVALID_ARG, std::string("cannot read ") + path);
  std::string text;
  char buf[4096];
  size_t n;
  while ((n = std::fread(buf, 1, sizeof buf, f)) > 0 && text.size() < (1u << 24)) text.append(buf, n);
  std::fclose(f);
  JsonReader r(text);
  JsonValue root;
  const bool parsed = r.value(&root);
  r.ws();
  if (!parsed || r.i != text.size() || root.kind != JsonValue::OBJ)
    return fail(LDDMM_E_INVALID_ARG, "not a tile table (JSON object expected)");
  const JsonValue* fmt = root.get("format");
  const JsonValue* ents = root.get("entries");
  if (!fmt || fmt->kind != JsonValue::STR || fmt->str != "lddmm-tiles-1" || !ents || ents->kind != JsonValue::ARR)
    return fail(LDDMM_E_INVALID_ARG, "tile table: format \"lddmm-tiles-1\" and an entries array expected");
  // every entry is checked before any is taken
  std::vector<std::pair<TileKey, TileEntry>> add;
  for (size_t k = 0; k < ents->arr.size(); ++k) {
    const JsonValue& e = ents->arr[k];
    const std::string where = "tile table entry " + std::to_string(k) + ": ";
    lddmm_params p{};
    int grid[3], band[3], spec[3];
    const JsonValue* arch = e.get("arch");
    const JsonValue* prec = e.get("precision");
    lddmm_tiles t{};
    if (e.kind != JsonValue::OBJ || !arch || arch->kind != JsonValue::STR || arch->str.empty() ||
        !json_int3(e.get("grid"), grid) || !json_int3(e.get("band"), band) || !json_int3(e.get("spectral"), spec) ||
        !prec || prec->kind != JsonValue::STR || (prec->str != "fp32" && prec->str != "bf16x3") ||
        !json_int(e.get("prod_rows"), &t.prod_rows) || !json_int(e.get("col_split"), &t.col_split) ||
        !json_int(e.get("sl_threads"), &t.sl_threads))
      return fail(LDDMM_E_INVALID_ARG, where + "arch, grid, band, spectral, precision, prod_rows, col_split and "
                                               "sl_threads expected");
    p.ndim = 3;
    for (int j = 0; j < 3; ++j) {
      p.grid[j] = grid[j];
      p.band[j] = band[j];
      p.spectral[j] = spec[j];
    }
    p.time_steps = 1;
    p.s = 2;
    p.alpha = 1.0;
    p.sigma = 1.0;
    p.precision = prec->str == "bf16x3" ? LDDMM_FP32_BF16X3 : LDDMM_FP32;
    Dims d;
    int rc = validate(&p, &d);
    if (!rc) rc = check_tiles(d, t);
    if (rc) return fail(rc, where + g_last_error);
    TileEntry te;
    te.t = t;
    const JsonValue* ms = e.get("ms_per_hvp");
    te.ms = (ms && ms->kind == JsonValue::NUM) ? ms->num : 0.0;
    add.emplace_back(tile_key(d, arch->str), te);
  }
  std::lock_guard<std::mutex> lk(g_tiles_mu);
  for (auto& kv : add) g_tiles[kv.first] = kv.second;
  if (!g_tiles.empty()) g_tiles_any.store(true);
  return LDDMM_OK;
}

int lddmm_autotune(const lddmm_params* p, const float* I0, const float* I1, const void* v0, int32_t reps,
                   lddmm_tiles* best, double* ms_best, double* ms_default, void* ws, size_t ws_bytes, void* stream) {
  Dims d;
  int rc = validate(p, &d);
  if (rc) return rc;
  if ((rc = no_checkpoint(d))) return rc;
  if ((rc = euler_only(d))) return rc;
  if (!I0 || !I1 || !v0) return fail(LDDMM_E_INVALID_ARG, "null input");
  if (reps < 1 || reps > 1000) return fail(LDDMM_E_INVALID_ARG, "reps must be in [1, 1000]");
  if ((rc = check_ws(d, ws, ws_bytes))) return rc;
  const std::string arch = current_arch();
  if (arch.empty()) return fail(LDDMM_E_HIP, "no current device");
  const hipStream_t st = static_cast<hipStream_t>(stream);
  // the built-in rule prepares the workspace (the layout does not depend on the tiles)
  d.tile_prod_rows = d.tile_col = d.tile_sl = 0;
  set_prepared(ws, false, d);
  hipError_t err;
  {
    Engine e(d, ws, st);
    if ((err = e.init_tables()) || (err = e.load_band(v0, e.V[0])) || (err = e.forward(I0)) ||
        (err = e.energy(e.final_state(), I1)) || (err = e.backward(I1, nullptr)) ||
        (err = launch_copy(reinterpret_cast<const float*>(e.V[0]), reinterpret_cast<float*>(e.dV[0]), 6LL * d.nb,
                           st)))
      return hip_fail(err, "autotune gradient");
  }
  hipEvent_t ev[2] = {nullptr, nullptr};
  for (auto& x : ev)
    if ((err = hipEventCreate(&x)) != hipSuccess) return hip_fail(err, "event");
  // The built-in rule's product is kept (in the line search's trial buffer,
  // unused here) and every candidate's product must equal it bit for bit; a
  // candidate that differs is rejected.  Mismatches are counted in the
  // reduction scratch.
  Engine e0(d, ws, st);
  float2* ref = e0.vtry;
  unsigned* nbad = reinterpret_cast<unsigned*>(e0.partial);
  const long long nfl = 6LL * d.nb;
  // time per Hessian-vector product (direction v0) with the given tiles; 0
  // mismatches in *bad if its product equals the reference
  auto measure = [&](const lddmm_tiles& t, double* ms, unsigned* bad) -> hipError_t {
    Dims dc = d;
    dc.tile_prod_rows = t.prod_rows;
    dc.tile_col = t.col_split;
    dc.tile_sl = t.sl_threads;
    Engine e(dc, ws, st);
    hipError_t r;
    if ((r = e.hessvec(e.dV[0], e.Hdh))) return r;  // first launches of the variant
    if (bad) {
      if ((r = launch_fill(reinterpret_cast<float*>(nbad), 1, 0.f, st)) ||
          (r = launch_count_ne(reinterpret_cast<const float*>(e.Hdh), reinterpret_cast<const float*>(ref), nfl,
                               nbad, st)) ||
          (r = hipMemcpyAsync(bad, nbad, sizeof(unsigned), hipMemcpyDeviceToHost, st)))
        return r;
    }
    if ((r = hipEventRecord(ev[0], st))) return r;
    for (int k = 0; k < reps; ++k)
      if ((r = e.hessvec(e.dV[0], e.Hdh))) return r;
    if ((r = hipEventRecord(ev[1], st)) || (r = hipEventSynchronize(ev[1]))) return r;
    float el = 0.f;
    if ((r = hipEventElapsedTime(&el, ev[0], ev[1]))) return r;
    *ms = el / reps;
    return hipSuccess;
  };
  // one field at a time, from the built-in rule; a candidate replaces the
  // current choice only if it is at least 1 % faster (the built-in rule is
  // timed twice, the first time to bring clocks and caches to their state)
  lddmm_tiles cur{};
  double tcur = 0.0, t0 = 0.0;
  err = measure(cur, &t0, nullptr);
  if (err == hipSuccess)
    err = launch_copy(reinterpret_cast<const float*>(e0.Hdh), reinterpret_cast<float*>(ref), nfl, st);
  if (err == hipSuccess) err = measure(cur, &t0, nullptr);
  tcur = t0;
  auto trial = [&](lddmm_tiles t) {
    double tt = 0.0;
    unsigned bad = 1;
    if (err == hipSuccess) err = measure(t, &tt, &bad);
    if (err == hipSuccess && bad == 0 && tt < 0.99 * tcur) {
      cur = t;
      tcur = tt;
    }
  };
  for (int th : {64, 128}) {
    lddmm_tiles t = cur;
    t.sl_threads = th;
    trial(t);
  }
  // only where a product launches k_prods: in the sweeps that k_step does not
  // serve, and at t = 1 of the deformation state
  const bool prods = !step_fused(d) || d.state != LDDMM_STATE_IMAGE;
  for (int r = 1; prods && r < prod_rows_max(d); ++r) {
    lddmm_tiles t = cur;
    t.prod_rows = r;
    trial(t);
  }
  for (int c = 1; c <= 3; ++c) {
    lddmm_tiles t = cur;
    t.col_split = c;
    trial(t);
  }
  for (auto& x : ev) (void)hipEventDestroy(x);
  if (err != hipSuccess) return hip_fail(err, "autotune");
  // the workspace stays prepared for lddmm_hessvec with these parameters
  set_prepared(ws, true, d);
  {
    std::lock_guard<std::mutex> lk(g_tiles_mu);
    TileEntry& e = g_tiles[tile_key(d, arch)];
    e.t = cur;
    e.ms = tcur;
    g_tiles_any.store(true);
  }
  if (best) *best = cur;
  if (ms_best) *ms_best = tcur;
  if (ms_default) *ms_default = t0;
  g_last_error.clear();
  return LDDMM_OK;
}

}  // extern "C"
