// Host-only check of the tile lists that launches really run on (built with
// g++ from csrc/plan.cpp by tests/test_exec_tiles.py).  A launch with too few
// tiles of its class to fill the chip runs on smaller tiles: for every group
// and kind of launch, the run's list must store every cell of the group's padded
// outputs exactly once with a tile that divides the padding (lower tiles: a
// tile on the diagonal, a pair of mirror tiles, or, inside a diagonal tile of a
// class that stores those whole, every tile in its mirror place), and large
// groups must keep their class tiles.  Arguments: precision.  Prints "OK", how
// many runs use each kernel, and how many waves have each mode.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <string>
#include <vector>

#include "../paper_2606_27153_amd/csrc/muon_internal.h"

using namespace muon;

static int fail(const std::string& m) {
  std::printf("FAIL %s\n", m.c_str());
  return 1;
}

int main(int argc, char** argv) {
  std::vector<muon_matrix_desc> descs;
  long long r, c;
  while (std::scanf("%lld %lld", &r, &c) == 2) descs.push_back(muon_matrix_desc{r, c, MUON_BF16, MUON_BF16, MUON_F32, 0});
  muon_plan_opts o{};
  o.precision = argc > 1 ? std::atoi(argv[1]) : 0;
  o.max_ns_steps = 5;
  o.a = 3.4445f;
  o.b = -4.775f;
  o.c = 2.0315f;
  o.eps = 1e-7f;
  o.small_m_threshold = 64;
  o.gram_min_aspect = 1.4f;
  Plan p;
  std::string err;
  if (build_plan(descs.data(), int32_t(descs.size()), o, p, err) != MUON_OK) return fail("build_plan: " + err);
  static const int kTile[EX_COUNT] = {256, 128, 128, 64};
  int used[EX_COUNT] = {}, modes[3] = {};
  for (const WaveHost& w : p.waves)
    for (const ClassLaunch& cl : w.launches) {
      const ClassInfo& ci = class_info(cl.kclass);
      // a merged wave runs on its groups' 64-tile lists (the others serve
      // launch timing)
      const StageRun runs[5] = {cl.run_gram, cl.run_square, cl.run_full, cl.merged_lower, cl.merged_full};
      if (w.mode != WAVE_APART && (w.launches.size() < 2 || w.launches.size() > size_t(kMaxParts)))
        return fail("merged groups");
      modes[w.mode] += &cl == &w.launches[0];
      const bool carried = w.mode == WAVE_MERGED || (w.mode == WAVE_SIDES_MERGED && cl.side);
      for (int kind = 0; kind < (carried ? 5 : 3); ++kind) {
        const StageRun& run = runs[kind];
        const bool full = kind == 2 || kind == 4;
        if (kind > 2 && run.exec != EX_64_RING3) return fail("merged tile");
        const int t = kTile[run.exec];
        used[run.exec]++;
        if (t > ci.tile) return fail("tile larger than the class's");
        if (ci.fp32 && (run.exec == EX_256 || run.exec == EX_128_RING3)) return fail("kernel without fp32 form");
        if (run.off < 0 || run.off + run.n > int64_t(p.h_tiles.size())) return fail("list out of range");
        if ((full ? cl.n_full + cl.n_strip_full : cl.n_lower) > 1024 && t != ci.tile)
          return fail("a launch that fills the chip left its class tile");
        if (t == ci.tile) {   // the class lists themselves
          if (run.off != (full ? cl.full_off : cl.lower_off) || run.n != (full ? cl.n_full : cl.n_lower))
            return fail("class list");
          continue;
        }
        std::map<int, std::vector<int>> cells;
        for (int s = 0; s < w.count; ++s) {
          const MatHost& h = p.mats[size_t(p.order[size_t(w.first + s)])];
          if (h.kclass != cl.kclass || h.gram != cl.gram) continue;
          if (h.m_pad % t || h.n_pad % t) return fail("tile does not divide the padding");
          cells[w.first + s].assign(size_t(h.m_pad / t) * size_t((full ? h.n_pad : h.m_pad) / t), 0);  // stores
        }
        for (int32_t i = 0; i < run.n; ++i) {
          const TileEntry& e = p.h_tiles[size_t(run.off + i)];
          auto it = cells.find(e.mat);
          if (it == cells.end()) return fail("tile of another group");
          const MatHost& h = p.mats[size_t(p.order[size_t(e.mat)])];
          const long long cm = h.m_pad / t, cn = (full ? h.n_pad : h.m_pad) / t;
          if (e.ti < 0 || e.tj < 0 || e.ti >= cm || e.tj >= cn) return fail("tile out of range");
          // which half of a product is stored follows the class: its diagonal
          // tiles whole, but for matrices of several 256 tiles
          const int per = ci.tile / t;
          const bool whole = !full && e.ti / per == e.tj / per && (ci.tile < 256 || h.m_pad == 256);
          if (e.flags != (whole ? kTileWhole : 0)) return fail("rule of the diagonal tiles");
          if (!full && !whole && e.tj > e.ti) return fail("tile above the diagonal");
          if (full || !whole) ++it->second[size_t(e.ti * cn + e.tj)];
          if (!full && (whole || e.ti != e.tj)) ++it->second[size_t(e.tj * cn + e.ti)];
        }
        for (const auto& kv : cells) {
          for (int v : kv.second)
            if (v != 1) return fail("outputs not stored exactly once");
        }
      }
    }
  std::printf("OK %d %d %d %d %d %d %d\n", used[0], used[1], used[2], used[3], modes[0], modes[1],
              modes[2]);
  return 0;
}
