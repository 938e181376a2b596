// Autotuner for the MFMA tile variant of each GEMM step (an extension; the
// paper leaves each step's kernel to its library).
//
// For every distinct step shape (precision, form, output store, h, m, n, k)
// the candidate workgroup shapes are timed with HIP events on a stand-in
// problem of the same structure, filled with hashed uniform values (m, then
// K down to 8192, then the batch cut so that a trial stays near 2e13 FLOP
// while keeping enough tiles to show the step's wave quantization), and the
// fastest is kept.  Choices live in a per-context cache, optionally backed
// by a text file (TNC_AUTOTUNE_CACHE) so later processes skip the timing.
// Without tuning a shape-based default is used.
#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <fstream>
#include <initializer_list>
#include <sstream>

#include "core.hpp"

namespace tnc {

namespace {

int64_t tiles_for(int variant, int64_t h, int64_t m, int64_t n) {
  int bm = 0, bnc = 0;
  gemm_variant_tile(variant, &bm, &bnc);
  return h * ((m + bm - 1) / bm) * ((n + bnc - 1) / bnc);
}

double padding_waste(int variant, int64_t m, int64_t n) {
  int bm = 0, bnc = 0;
  gemm_variant_tile(variant, &bm, &bnc);
  const double pm = static_cast<double>((m + bm - 1) / bm * bm);
  const double pn = static_cast<double>((n + bnc - 1) / bnc * bnc);
  return 1.0 - static_cast<double>(m) * n / (pm * pn);
}

// complex64 runs the 4M kernels in both forms
bool runs_4m(int prec, int form) { return prec == TNC_PREC_C64 || form == TNC_GEMM_4M; }

// Ranking of the variants by measured per-tile throughput on large shapes.
const std::vector<int>& ranking(tnc_prec prec, tnc_cgemm form) {
  static const std::vector<int> r4m = {3, 2, 0, 1, 4, 5, 6, kDirect64x32, kDirect32x32, kDirect32x16};
  static const std::vector<int> r3m = {2, 0, 1, 4, 5, 6};
  return runs_4m(prec, form) ? r4m : r3m;
}

std::vector<int> candidates(tnc_prec prec, tnc_cgemm form, int64_t h, int64_t m, int64_t n) {
  std::vector<int> out;
  for (int v : ranking(prec, form)) {
    if (v >= kGemmVariants && tiles_for(v, h, m, n) > 2048) continue;  // the few-tile shapes
    if (tiles_for(v, h, m, n) * 64 < (int64_t{1} << 32) && padding_waste(v, m, n) < 0.5) out.push_back(v);
  }
  if (out.empty()) out.push_back(0);
  return out;
}

}  // namespace

// What a tile takes: `alone` ns per complex k where its workgroup has a CU to
// itself, `full` ns per k and workgroup where `at_once` of them share one.
struct TileCost {
  double alone, full;
  int at_once;
};

// The variant whose launch takes least.  The CU with the most tiles, q of
// them, runs them at_once by at_once, each batch for max(alone, batch x full)
// per k and a prologue worth k0 of it; a tile's store takes a time of its own
// where nothing else runs beside it (a shape of one workgroup per CU), less
// where something does.  Fitted to forced variants over some 105 random
// shapes in each form (h 1..8192, m, n 16..4000, k 16..2500): on average 0.2 %
// behind the best in 3M, 0.4 % in 4M.
static int least_time(const TileCost* cost, std::initializer_list<int> variants, double k0, double store_alone, double store,
                      int64_t h, int64_t m, int64_t n, int64_t k) {
  int best = *variants.begin();
  double top = 0.0;
  for (int v : variants) {
    const TileCost& c = cost[v];
    const int64_t q = (tiles_for(v, h, m, n) + 255) / 256;
    auto batch = [&](int64_t b) { return b ? std::max(c.alone, static_cast<double>(b) * c.full) : 0.0; };
    int bm = 0, bnc = 0;
    gemm_variant_tile(v, &bm, &bnc);
    const double t = (static_cast<double>(q / c.at_once) * batch(c.at_once) + batch(q % c.at_once)) * (static_cast<double>(k) + k0) * 1e-3 +
                     (c.at_once == 1 ? store_alone : store) * static_cast<double>(q) * bm * bnc / 8192;
    if (top == 0.0 || t < 0.99 * top) {
      top = t;
      best = v;
    }
  }
  return best;
}

// Split 3M (before: 128 x 64 unless a small tile padded next to nothing and had
// 1024 workgroups, so 579 x 33 x 51 x 460 ran 66 us on it, 64 x 64 takes 47; 134 x
// 35 x 193 x 308 48 and, on 64 x 32, 34; 4096 x 32 x 32 x 128 110 and 81).
static int default_variant_3m(int64_t h, int64_t m, int64_t n, int64_t k) {
  static const TileCost cost[kGemmVariants] = {{55, 39, 2}, {99, 99, 1}, {69, 69, 1}, {0, 0, 1}, {82, 26.4, 3}, {89, 16.8, 2}, {88, 8.65, 4}};
  return least_time(cost, {0, 2, 4, 5, 6}, 45, 0.74, 0.30, h, m, n, k);
}

// 4M kernels.  With few tiles the shapes that share K out (us per launch,
// 128 x 64 tile before and the chosen shape: 256 x 256 x 256 26.6, 7.0;
// 512 x 512 x 512 47, 14.6; 8 x 1024 x 64 x 128 17.3, 10.7; from 2048
// 32 x 16 tiles on the tiles win: 1024 x 1024 x 64 12.5, 13.4), the one with
// the least rounds, weighed by what a round takes (1 x 1000 x 500 x 200: 1024
// tiles of 32 x 16, two to a CU, 15.9; 512 of 32 x 32 15.7; 256 of 64 x 32
// 12.4; where 64 x 32 pads into a second round, 3 x 138 x 1067 x 79: 12.1, 11.9,
// 15.2).  Else in complex64 the
// tile with the largest product of what it reaches on large shapes (relative
// to 256 x 128), the share of it that is not padding, how evenly its
// workgroups fill 256 CUs, and how well one CU's waves hide each other's
// latency (fewer than two per SIMD do not: 2 x 4096 x 256 x 128 runs 20.5 us
// on 256 workgroups of four waves, 28.0 on 512 of two, 24.8 on 128 of eight).
// In split precision the tile of the least predicted time (by rates as in
// complex64 5 x 1699 x 917 x 2208 ran on 64 x 64, 525 us, 472 on 128 x 64; 246 x
// 130 x 42 x 1239 174, now 126).  Its 256 x 128 tile (3) has one sum for all
// three products where the others keep the cross products apart (error
// against 64 bits at k = 1024, 4096, 16384: 1.005, 1.02 and 1.08 times
// theirs), so nobody gets it unasked except planned steps that give every CU
// four tiles of it.
int default_variant(tnc_prec prec, tnc_cgemm form, int64_t h, int64_t m, int64_t n, int64_t k, bool planned) {
  if (!runs_4m(prec, form)) return default_variant_3m(h, m, n, k);
  const int64_t few = tiles_for(kDirect32x16, h, m, n);
  if (few <= 256) return kDirect32x16;
  if (few <= 1024) {
    auto rounds = [&](int v, int64_t at_once) { return static_cast<double>((tiles_for(v, h, m, n) + at_once - 1) / at_once); };
    const double t7 = 1.2 * rounds(kDirect32x16, 512), t8 = rounds(kDirect32x32, 256), t9 = 1.4 * rounds(kDirect64x32, 256);
    return t9 <= t8 && t9 <= t7 ? kDirect64x32 : t8 <= t7 ? kDirect32x32 : kDirect32x16;
  }
  if (prec == TNC_PREC_BF16X3) {
    static const TileCost cost[kGemmVariants] = {{42, 44, 2}, {86, 86, 1}, {71.5, 71.5, 1}, {155, 155, 1}, {85, 27.7, 4}, {47, 30.5, 4}, {74.5, 18.3, 8}};
    if (planned && tiles_for(3, h, m, n) >= 1024 && padding_waste(3, m, n) <= 0.125)
      return least_time(cost, {3, 0, 1, 2, 4, 5, 6}, 37, 0.82, 0.24, h, m, n, k);
    return least_time(cost, {0, 1, 2, 4, 5, 6}, 37, 0.82, 0.24, h, m, n, k);
  }
  static const double rate[kGemmVariants] = {0.86, 0.83, 0.97, 1.0, 0.74, 0.70, 0.575};  // 8192 x 8192 x 4096
  static const int waves[kGemmVariants] = {4, 4, 8, 8, 2, 2, 1};
  int best = 4;
  double top = 0.0;
  for (int v : {3, 2, 0, 1, 4, 5, 6}) {
    const int64_t t = tiles_for(v, h, m, n), q = (t + 255) / 256;
    const int64_t w = q * waves[v];
    const double hide = w >= 8 ? 1.0 : w >= 4 ? 0.58 : w >= 2 ? 0.32 : 0.2;
    const double e = rate[v] * (1.0 - padding_waste(v, m, n)) * (static_cast<double>(t) / (256.0 * q)) * hide;
    if (e > 1.01 * top) {
      top = e;
      best = v;
    }
  }
  return best;
}

// Entries of the file count only for the kernels they were measured on: the
// first field is "generation:precision", and a line of another generation
// (or of none) is passed over.  The generation goes up whenever kernels behind
// the variants' numbers change (2: complex64 and split 4M on the bf16 pipe,
// the shapes for few tiles; 3: split 4M with two stages on their way).
static constexpr int kTuneGeneration = 3;

std::string TuneKey::str() const {
  std::ostringstream o;
  o << kTuneGeneration << ':' << prec << ' ' << form << ' ' << perm << ' ' << h << ' ' << m << ' ' << n << ' ' << k;
  return o.str();
}

void load_tune_cache(Ctx& c) {
  const char* path = std::getenv("TNC_AUTOTUNE_CACHE");
  if (!path) return;
  std::ifstream f(path);
  std::string line;
  while (std::getline(f, line)) {
    std::istringstream in(line);
    TuneKey key;
    int generation = 0, v = 0;
    char colon = 0;
    if (!(in >> generation >> colon >> key.prec >> key.form >> key.perm >> key.h >> key.m >> key.n >> key.k >> v)) continue;
    if (generation != kTuneGeneration || colon != ':') continue;
    if (v >= 0 && v < (runs_4m(key.prec, key.form) ? kAllVariants : kGemmVariants)) c.tune_cache[key] = v;
  }
}

static void save_tune_entry(const TuneKey& key, int v) {
  const char* path = std::getenv("TNC_AUTOTUNE_CACHE");
  if (!path) return;
  std::ofstream f(path, std::ios::app);
  f << key.str() << ' ' << v << '\n';
}

int tune_shape(Ctx& c, const TuneKey& key, int64_t k, bool perm_store) {
  {
    std::lock_guard<std::mutex> g(c.tune_mu);
    auto it = c.tune_cache.find(key);
    if (it != c.tune_cache.end()) return it->second;
  }
  const tnc_prec prec = static_cast<tnc_prec>(key.prec);
  const tnc_cgemm form = static_cast<tnc_cgemm>(key.form);
  const std::vector<int> cand = candidates(prec, form, key.h, key.m, key.n);
  int best = cand.front();
  if (cand.size() > 1) {
    // stand-in problem near 2e13 FLOP (about 0.15 s).  m is cut first while
    // the grid keeps 8 or more rounds of the largest workgroup (256 x 128)
    // over the 256 CUs, so wave quantization -- which separates the shapes on
    // few-tile steps -- stays that of the step; K stays whole there, since
    // whether a K panel fits an XCD's 4 MiB L2 also ranks the shapes (3M
    // (2,2) leads (2,4) at k = 2048 and trails it by 5 % at k = 16384).
    // Then K (down to 8192), the batch, and m below that bound.
    int64_t h = key.h, m = key.m;
    const double target = 2e13;
    auto flop = [&] { return 8.0 * h * m * key.n * k; };
    auto half_m = [](int64_t x) { return (x / 2 + 255) / 256 * 256; };
    while (m > 8192 && flop() > target && h * ((half_m(m) + 255) / 256) * ((key.n + 127) / 128) >= 2048)
      m = half_m(m);
    while (k > 8192 && k % 32 == 0 && flop() > target) k /= 2;
    while (h > 1 && flop() > target) h = (h + 1) / 2;
    while (m > 4096 && flop() > target) m = half_m(m);
    // and its operands stay within 8 GiB beside the caller's arena (the
    // batch shrinks; 2048 or more tiles remain for batches of this size)
    auto bytes = [&] { return 8.0 * h * (m * k + key.n * k + m * key.n); };
    while (h > 1 && bytes() > 8.0 * (int64_t{1} << 30)) h = (h + 1) / 2;
    DeviceBuf a, b, cc, offm, offn;
    a.alloc(static_cast<size_t>(h * m * k) * 8);
    b.alloc(static_cast<size_t>(h * key.n * k) * 8);
    cc.alloc(static_cast<size_t>(h * m * key.n) * 8);
    check_hip(launch_fill_hash(static_cast<float*>(a.ptr), h * m * k * 2, 0x5eed0001u, c.stream), "tune fill");
    check_hip(launch_fill_hash(static_cast<float*>(b.ptr), h * key.n * k * 2, 0x5eed0002u, c.stream), "tune fill");
    GemmDesc d;
    std::memset(&d, 0, sizeof(d));
    d.A = static_cast<const float2*>(a.ptr);
    d.B = static_cast<const float2*>(b.ptr);
    d.C = static_cast<float2*>(cc.ptr);
    d.m = m;
    d.n = key.n;
    d.k = k;
    d.h = h;
    if (h > 1) {
      d.nbd = 1;
      d.bext[0] = static_cast<int32_t>(h);
      d.bsA[0] = m * k;
      d.bsB[0] = key.n * k;
      d.pow2 = 0;
    }
    if (perm_store) {  // a permuted store with the natural offsets: same access count
      std::vector<int64_t> om(m), on(key.n);
      for (int64_t i = 0; i < m; ++i) om[i] = i * key.n;
      for (int64_t j = 0; j < key.n; ++j) on[j] = j;
      offm.alloc(om.size() * 8);
      offn.alloc(on.size() * 8);
      check_hip(hipMemcpy(offm.ptr, om.data(), om.size() * 8, hipMemcpyHostToDevice), "tune tables");
      check_hip(hipMemcpy(offn.ptr, on.data(), on.size() * 8, hipMemcpyHostToDevice), "tune tables");
      d.offM = static_cast<const int64_t*>(offm.ptr);
      d.offN = static_cast<const int64_t*>(offn.ptr);
    }
    const Form f = form == TNC_GEMM_3M ? Form::M3 : Form::M4;
    const Prec p = prec == TNC_PREC_BF16X3 ? Prec::BF16X3 : Prec::C64;
    hipEvent_t e0, e1;
    check_hip(hipEventCreate(&e0), "event");
    check_hip(hipEventCreate(&e1), "event");
    float best_ms = 1e30f;
    for (int v : cand) {
      check_hip(launch_gemm(d, GemmKernel::MFMA, v, f, p, c.stream), "tune launch");  // warm-up
      check_hip(hipEventRecord(e0, c.stream), "event");
      for (int r = 0; r < 2; ++r) check_hip(launch_gemm(d, GemmKernel::MFMA, v, f, p, c.stream), "tune launch");
      check_hip(hipEventRecord(e1, c.stream), "event");
      check_hip(hipEventSynchronize(e1), "event");
      float ms = 0;
      check_hip(hipEventElapsedTime(&ms, e0, e1), "event");
      // candidates come in ranking order (full-size sweeps); a later one
      // must win by more than 1 %, the spread of repeated trials
      if (ms < 0.99f * best_ms) {
        best_ms = ms;
        best = v;
      }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
  }
  {
    std::lock_guard<std::mutex> g(c.tune_mu);
    c.tune_cache[key] = best;
  }
  save_tune_entry(key, best);
  return best;
}

void assign_variants(const Plan& plan, ChunkPlan& cp, bool tune) {
  Ctx& c = *plan.net->ctx;
  for (StepPlan& sp : cp.steps) {
    if (sp.kind != GemmKernel::MFMA) continue;
    const GemmDesc& d = sp.desc;
    const bool perm = !sp.offM.empty() && sp.split == 1;
    const TuneKey key{static_cast<int>(plan.prec), static_cast<int>(plan.form), perm ? 1 : 0, d.h, d.m, d.n, d.k};
    bool cached = false;
    {
      std::lock_guard<std::mutex> g(c.tune_mu);
      auto it = c.tune_cache.find(key);
      if (it != c.tune_cache.end()) {
        sp.variant = it->second;
        cached = true;
      }
    }
    if (cached) continue;
    if (tune && !c.host_only)
      sp.variant = tune_shape(c, key, d.k, perm);
    else
      sp.variant = default_variant(plan.prec, plan.form, d.h, d.m, d.n, d.k, true);
  }
  summarize_steps(cp);
}

}  // namespace tnc
