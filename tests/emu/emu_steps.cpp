// CPU emulation of sim_kernel's forms that emu_wg.cpp does not take: per-trial
// thresholds (the coin filter and its binary64 resolution) as well as tables,
// turn-off times as well as one-step burns, from any ignitions and parameter
// vectors, with burn maps. Built with AddressSanitizer and
// UndefinedBehaviorSanitizer; every buffer, the spill area of each workgroup's
// queues and its life bytes among them, has exactly the size the host gives it.
//
// usage: emu_steps CASE_DIR W H WINDOW QUEUE_CAP WORKGROUPS SEED TABLE TURN_OFF GLOBAL
// WINDOW 0: one whole-lattice launch; else the window launch and the
// whole-lattice launch over the simulations it lists. GLOBAL: the whole-lattice
// launch keeps its bitsets in global memory.
// CASE_DIR holds veg.bin (uint8), elev.bin, slope.bin, aspect.bin, wind.bin
// (float32), betas.bin (float64 rows of 5), steps.bin (uint8 [256]) and sims.bin
// (fire_sim). The kernel source's own functions make the cell records and the
// tables; out: tables.bin (uint32 [n_params][H][W][8], what the oracle is to
// take), results.bin and maps.bin.
#include "kernel.inc"
#include <chrono>
#include <fstream>
#include <string>
#include <thread>
#ifndef EMU_BLOCK
#define EMU_BLOCK 128
#endif
thread_local Dim3 threadIdx, blockIdx;
Dim3 blockDim, gridDim;
thread_local uint32_t *g_lds;
thread_local WgCtx *g_wg;
thread_local int *g_where;
std::atomic<long> g_progress{0};
std::mutex g_atomic_mu;
using namespace firegpu;
constexpr int BLOCK = EMU_BLOCK;

template <class T> std::vector<T> load(const std::string &path) {
  std::ifstream f(path, std::ios::binary | std::ios::ate);
  if (!f) { fprintf(stderr, "missing %s\n", path.c_str()); exit(2); }
  std::vector<T> v((size_t)f.tellg() / sizeof(T));
  f.seekg(0);
  f.read(reinterpret_cast<char *>(v.data()), v.size() * sizeof(T));
  return v;
}

template <class T> void save(const std::string &path, const std::vector<T> &v) {
  std::ofstream(path, std::ios::binary).write(reinterpret_cast<const char *>(v.data()), v.size() * sizeof(T));
}

template <bool TABLE, bool DUR, bool WIN, bool GB>
void run_workgroup(const SimArgs &a, int b) {
  // lds_bytes_for of the host
  const size_t words = (size_t)(GB ? 0 : a.bitset_words) + 2 * (size_t)a.queue_cap + 16;
  std::vector<uint32_t> lds(words + (DUR ? (2 * (size_t)a.queue_cap + 3) / 4 : 0), 0xDEADBEEFu);
  WgCtx ctx;
  Barrier block(BLOCK);
  ctx.block = &block;
  for (int w = 0; w < BLOCK / 64; ++w) ctx.wave.push_back(new Barrier(64));
  std::vector<int> where(BLOCK, 0);
  std::vector<std::thread> th;
  for (int t = 0; t < BLOCK; ++t)
    th.emplace_back([&, t] {
      threadIdx.x = t;
      blockIdx.x = b;
      g_wg = &ctx;
      g_lds = lds.data();
      g_where = &where[t];
      sim_kernel<BLOCK, TABLE, DUR, WIN, GB>(a);
      block.arrive_and_drop();
    });
  for (auto &x : th) x.join();
  for (auto *p : ctx.wave) delete p;
}

template <bool WIN, bool GB>
void launch(const SimArgs &a, int groups, bool table, bool dur) {
  blockDim.x = BLOCK;
  gridDim.x = groups;
  std::vector<std::thread> wgs;
  for (int b = 0; b < groups; ++b)
    wgs.emplace_back([&, b] {
      if (table) dur ? run_workgroup<true, true, WIN, GB>(a, b) : run_workgroup<true, false, WIN, GB>(a, b);
      else dur ? run_workgroup<false, true, WIN, GB>(a, b) : run_workgroup<false, false, WIN, GB>(a, b);
    });
  for (auto &x : wgs) x.join();
}

int main(int argc, char **argv) {
  if (argc != 11) { fprintf(stderr, "see the head of emu_steps.cpp\n"); return 2; }
  const std::string d = argv[1];
  const int W = atoi(argv[2]), H = atoi(argv[3]), win = atoi(argv[4]), cap = atoi(argv[5]), groups = atoi(argv[6]);
  const uint64_t seed = strtoull(argv[7], nullptr, 0);
  const bool table = atoi(argv[8]) != 0, dur = atoi(argv[9]) != 0, global = atoi(argv[10]) != 0;
  auto veg = load<uint8_t>(d + "/veg.bin");
  auto elev = load<float>(d + "/elev.bin"), slope = load<float>(d + "/slope.bin");
  auto aspect = load<float>(d + "/aspect.bin"), wind = load<float>(d + "/wind.bin");
  auto betas = load<double>(d + "/betas.bin");
  auto steps = load<uint8_t>(d + "/steps.bin");
  auto sims = load<fire_sim>(d + "/sims.bin");
  const int64_t n = (int64_t)W * H;
  const int stride = (W + 31) / 32, n_sims = (int)sims.size(), n_params = (int)betas.size() / 5;
  std::vector<uint4> rec(n), fcov(n);
  std::vector<double> ps(2 * n), omega(8 * n);
  std::vector<uint32_t> blocked((size_t)H * stride);
  threadIdx.x = 0; blockIdx.x = 0; blockDim.x = 1; gridDim.x = 1;
  preprocess_kernel(veg.data(), elev.data(), slope.data(), aspect.data(), wind.data(), W, H, stride, rec.data(),
                    ps.data(), omega.data(), blocked.data());
  fcov_kernel(rec.data(), ps.data(), omega.data(), n, 1u, fcov.data());
  if (dur) set_life_kernel(rec.data(), n, steps.data());
  std::vector<uint32_t> tables((size_t)n_params * n * 8);
  for (int p = 0; p < n_params; ++p)
    for (int64_t c = 0; c < n; ++c)
      for (int k = 0; k < 8; ++k) {
        const int x = (int)(c % W) + dir_dx(k), y = (int)(c / W) + dir_dy(k);
        const bool in = x >= 0 && x < W && y >= 0 && y < H;
        const int64_t t = (int64_t)y * W + x;
        tables[((size_t)p * n + c) * 8 + k] =
            in ? edge_threshold(&betas[5 * p], rec[t].w, ps.data(), omega.data(), t, k, 1u) : 0u;
      }
  save(d + "/tables.bin", tables);
  std::vector<LandscapeDev> lsd(1);
  LandscapeDev &L = lsd[0];
  L.W = W; L.H = H; L.stride = stride; L.valid = 1; L.rec = rec.data(); L.ps = ps.data();
  L.omega = omega.data(); L.blocked = blocked.data(); L.burn_steps = dur ? steps.data() : nullptr;
  L.forest_class = 1; L.fcov = fcov.data();
  std::vector<fire_result> out(n_sims);
  std::vector<uint32_t> maps((size_t)n_sims * H * stride, 0xDEADBEEFu);
  std::vector<uint32_t> work(2, 0), err(1, 0), retry(1 + n_sims, 0);
  const int64_t ovf_cap = std::max<int64_t>(1, n - cap);
  std::vector<uint32_t> spill((size_t)groups * 2 * ovf_cap);
  std::vector<uint8_t> life(dur ? (size_t)groups * 2 * ovf_cap : 0);
  std::vector<uint32_t> gbits(global ? (size_t)groups * H * stride : 0, 0xDEADBEEFu);
  SimArgs a{};
  a.ls = lsd.data(); a.n_ls = 1; a.tg = nullptr; a.n_tg = 0;
  a.betas = betas.data(); a.n_params = n_params;
  a.sims = sims.data(); a.order = nullptr; a.n_sims = n_sims;
  a.key0 = (uint32_t)seed; a.key1 = (uint32_t)(seed >> 32);
  a.tables = table ? tables.data() : nullptr; a.table_stride = n * 8; a.table_ls = table ? 0 : -1;
  a.out = out.data(); a.maps = maps.data(); a.map_words = (int64_t)H * stride;
  a.work = &work[0]; a.error_flag = err.data(); a.ovf = spill.data();
  a.ovf_life = dur ? life.data() : nullptr; a.ovf_cap = ovf_cap; a.queue_cap = cap;
  if (win > 0) {
    a.win = win;
    a.bitset_words = std::min(win, H) * std::min(win / 32, stride);
    a.retry = retry.data();
    launch<true, false>(a, groups, table, dur);
    a.work = &work[1]; a.order = retry.data() + 1; a.n_dev = retry.data(); a.win = 0;
  }
  a.bitset_words = H * stride;
  a.gbits = global ? gbits.data() : nullptr;
  if (global) launch<false, true>(a, groups, table, dur);
  else launch<false, false>(a, groups, table, dur);
  save(d + "/results.bin", out);
  save(d + "/maps.bin", maps);
  printf("error flag %u, re-runs %u of %d\n", err[0], retry[0], n_sims);
  return err[0] != 0;
}
