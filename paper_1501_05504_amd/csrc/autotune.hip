// Tile-configuration autotuner (host C++).
//
// Dense GEMMs: on the first product of a given shape class (precision,
// operand layouts, M, N, K, batch) every tile configuration and the size
// rule's own choice (wave tiles among them) are timed with HIP events on the
// context's stream and the fastest is kept in the context's cache (and appended
// to an optional on-disk cache file of "key:how cfg" lines, loaded when
// autotuning is switched on).  Where the rule would run GEMM-1 and the W-map of
// H_eff in one launch, that is timed against the tuned GEMM-1 and the launches
// around it (whole product in FP64, d = 4, w = 6, with the rule's choices among the
// candidates and without: 37 x 29 11.3 / 27.0 us, 256 x 250 43.6 / 62.0).
// Grouped block plans: all six tile configurations of the grouped launch are
// timed on scratch buffers right after the plan is built.
// Tuning is skipped while a stream is being captured into a graph and for
// products that accumulate into C (beta != 0).
#include <fstream>
#include <sstream>

#include "d3s_internal.h"

namespace d3s {

namespace {

std::string gemm_key(d3s_prec p, const GemmArgs& g) {
  std::ostringstream o;
  o << "gemm:" << (int)p << ':' << g.a_kc << ':' << g.b_kc << ':' << g.M << ':' << g.N << ':' << g.K << ':'
    << g.batch;
  return o.str();
}

bool capturing(Ctx* c) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(c->stream, &st) != hipSuccess) {
    (void)hipGetLastError();
    return true;
  }
  return st != hipStreamCaptureStatusNone;
}

template <typename F>
double time_ms(Ctx* c, F&& launch, int reps) {
  hipEvent_t e0, e1;
  D3S_HIP(hipEventCreate(&e0));
  D3S_HIP(hipEventCreate(&e1));
  launch();   // warm-up
  D3S_HIP(hipEventRecord(e0, c->stream));
  for (int r = 0; r < reps; ++r) launch();
  D3S_HIP(hipEventRecord(e1, c->stream));
  D3S_HIP(hipEventSynchronize(e1));
  float ms = 0.f;
  D3S_HIP(hipEventElapsedTime(&ms, e0, e1));
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  return ms / reps;
}

// A decision is the fastest fixed configuration, plus one of these where
// something else was faster still
enum { kRule = 8, kFused = 16 };   // no fixed configuration; GEMM-1 and W-map in one launch

void remember(Ctx* c, const std::string& key, int code) {
  c->tune_cache[key] = code;
  if (!c->tune_path.empty()) {
    std::ofstream f(c->tune_path, std::ios::app);
    const char* how = (code & kFused) ? ":fused " : (code & kRule) ? ":rule " : ":tile ";
    if (f) f << key << how << (code & 7) << '\n';
  }
}

// with a tile configuration chosen for the time of a call
struct WithTile {
  Ctx* c;
  WithTile(Ctx* ctx, int cfg) : c(ctx) { c->tile_config = cfg; }
  ~WithTile() { c->tile_config = -1; }
};

void gemm_as(Ctx* c, d3s_prec p, const GemmArgs& g, int code) {
  WithTile w(c, (code < 0 || (code & kRule)) ? -1 : (code & 7));
  gemm(c, p, g);
}

int time_gemm(Ctx* c, d3s_prec p, const GemmArgs& g) {
  double best = 1e300;
  int code = 0;
  for (int k = 0; k <= 4; ++k) {
    const double ms = time_ms(c, [&] { gemm_as(c, p, g, k); }, 3);
    if (ms < best) {
      best = ms;
      code = k;
    }
  }
  // in BF16 the rule is one of the configurations
  if (p != D3S_BF16 && time_ms(c, [&] { gemm_as(c, p, g, -1); }, 3) < best) code |= kRule;
  return code;
}

}  // namespace

// Lines without ":tile", ":rule" or ":fused" behind the key compared the fixed
// configurations only: their shapes are timed again.
void autotune_load(Ctx* c) {
  if (c->tune_path.empty()) return;
  std::ifstream f(c->tune_path);
  std::string key;
  int cfg;
  while (f >> key >> cfg) {
    const size_t at = key.rfind(':');
    if (at == std::string::npos || cfg < 0 || cfg > 4) continue;
    const std::string how = key.substr(at + 1);
    if (how != "tile" && how != "rule" && how != "fused") continue;
    c->tune_cache[key.substr(0, at)] = cfg | (how == "fused" ? kFused : how == "rule" ? kRule : 0);
  }
}

void tuned_gemm(Ctx* c, d3s_prec p, const GemmArgs& g) {
  if (!c->autotune || c->tile_config >= 0) {
    gemm(c, p, g);
    return;
  }
  const std::string key = gemm_key(p, g);
  auto it = c->tune_cache.find(key);
  int code = -1;
  if (it != c->tune_cache.end()) {
    code = it->second;
  } else if (g.beta == 0.0 && !capturing(c)) {
    code = time_gemm(c, p, g);
    remember(c, key, code);
  }
  gemm_as(c, p, g, code);
}

bool tuned_first(Ctx* c, d3s_prec p, const GemmArgs& g1, int d, const std::function<bool()>& fused,
                 const std::function<void(const std::function<void()>&)>& separate) {
  const std::string key = gemm_key(p, g1) + ":d" + std::to_string(d);
  auto it = c->tune_cache.find(key);
  int code;
  if (it != c->tune_cache.end()) {
    code = it->second;
  } else {
    const bool ran = fused();
    if (!ran) separate([&] { tuned_gemm(c, p, g1); });
    if (!ran || capturing(c)) return ran;
    code = time_gemm(c, p, g1);
    const double ms = time_ms(c, [&] { separate([&] { gemm_as(c, p, g1, code); }); }, 3);
    if (time_ms(c, [&] { fused(); }, 3) < ms) code |= kFused;
    remember(c, key, code);
  }
  if ((code & kFused) && fused()) return true;
  separate([&] { gemm_as(c, p, g1, code); });
  return false;
}

void tune_grouped(Ctx* c, GroupedPlan& g, const void* A, const void* B, void* C) {
  if (!c->autotune || g.ntasks == 0 || capturing(c)) return;
  double best = 1e300;
  int best_cfg = g.cfg;
  for (int cfg = 0; cfg <= 5; ++cfg) {
    g.cfg = cfg;
    grouped_retile(c, g);
    const double ms = time_ms(c, [&] { grouped_gemm(c, c->tune_prec, g, A, B, C, 1.0); }, 2);
    if (ms < best) {
      best = ms;
      best_cfg = cfg;
    }
  }
  if (g.cfg != best_cfg) {
    g.cfg = best_cfg;
    grouped_retile(c, g);
  }
}

}  // namespace d3s
