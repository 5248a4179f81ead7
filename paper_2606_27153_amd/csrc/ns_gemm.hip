// Host side of the grouped Newton-Schulz GEMMs: one stage of one (kernel
// class, iteration form) group over its tile lists.  The kernels are in
// ns_gemm_kernel.h, launched through the per-group launchers of ns_gemm.h.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "muon_internal.h"
#include "ns_gemm.h"

namespace muon {
namespace {

// One grouped launch over the tiles of `run` (twice that for a paired ST_SYM
// step, whose second half computes the second product), on the kernels of
// class kc's operand type.
int launch_tiles(const Plan& p, int32_t kc, bool padded, int32_t stage, const StageRun& run, bool pair, GemmArgs g,
                 hipStream_t st) {
  if (run.n == 0) return 0;
  g.tiles = p.d_tiles + run.off;
  g.split = pair ? run.n : INT32_MAX;
  const unsigned grid = unsigned(run.n) * (stage == ST_SYM && pair ? 2u : 1u);
  const ClassInfo& ci = class_info(kc);
  if (run.exec == EX_256) {
    // the 256 tile puts two waves on each SIMD, so a skipped wave speeds up
    // its partner (the PAD instantiation)
    if (ci.f16)
      return stage == ST_BX ? launch_t256_f16_bx(padded, grid, g, st) : launch_t256_f16_sq(padded, stage, grid, g, st);
    return stage == ST_BX ? launch_t256_bf16_bx(padded, grid, g, st) : launch_t256_bf16_sq(padded, stage, grid, g, st);
  }
  return ci.fp32  ? launch_tile_f32(run.exec, stage, grid, g, st)
         : ci.f16 ? launch_tile_f16(run.exec, stage, grid, g, st)
                  : launch_tile_bf16(run.exec, stage, grid, g, st);
}

// What every launch of a wave shares.
GemmArgs wave_args(const Plan& p, const WaveHost& w, char* ws, const StepScalars& sc) {
  GemmArgs g{};
  g.mats = p.d_mats;
  g.ws = ws;
  g.scale = reinterpret_cast<const float*>(ws + w.scale_off);
  g.flag = reinterpret_cast<const int32_t*>(ws + w.flag_off);
  g.mat_base = w.first;
  g.ptrs = p.d_ptrs;
  g.lr = sc.lr;
  g.decay = sc.decay;
  return g;
}

}  // namespace

int launch_ns_gemm(const Plan& p, const WaveHost& w, const ClassLaunch& cl, int32_t stage, const GemmStep& gs,
                   char* ws, const StepScalars& sc, void* stream) {
  GemmArgs g = wave_args(p, w, ws, sc);
  g.fcoef = gs.fcoef;
  g.diag = gs.diag;
  g.oscale = gs.oscale;
  g.first = gs.first;
  g.pin = gs.pin;
  g.last = gs.last;
  g.l = gs.l;
  g.r = gs.r;
  g.out = gs.out;
  g.l2 = gs.l2;
  g.r2 = gs.r2;
  g.out2 = gs.out2;
  hipStream_t st = hipStream_t(stream);
  // a 256-tile B*X is followed by the edge strips of the same matrices on
  // 128 tiles (their outputs are disjoint); any other launch covers its
  // matrices' whole padded outputs
  const StageRun& run = stage == ST_GRAM ? cl.run_gram : stage == ST_BX ? cl.run_full : cl.run_square;
  int e = launch_tiles(p, cl.kclass, cl.padded, stage, run, gs.pair != 0, g, st);
  if (e == 0 && stage == ST_BX && run.exec == EX_256)
    e = launch_tiles(p, cl.kclass, false, stage, StageRun{EX_128_RING2, cl.strip_full_off, cl.n_strip_full}, false, g,
                     st);
  return e;
}

int launch_merged(const Plan& p, const WaveHost& w, const GemmOp* const* ops, char* ws, const StepScalars& sc,
                  void* stream) {
  MultiArgs m{};
  m.common = wave_args(p, w, ws, sc);
  int64_t blocks = 0;
  bool f16 = false;
  for (size_t i = 0; i < w.launches.size(); ++i) {
    if (!ops[i]) continue;
    const ClassLaunch& cl = w.launches[i];
    const StageRun& run = ops[i]->stage == ST_BX ? cl.merged_full : cl.merged_lower;
    const bool pair = ops[i]->stage == ST_SYM && ops[i]->g.pair != 0;
    blocks += int64_t(run.n) * (pair ? 2 : 1);
    MultiPart& q = m.part[m.n++];
    q.tiles = p.d_tiles + run.off;
    q.g = ops[i]->g;
    q.stage = ops[i]->stage;
    q.fp32 = class_info(cl.kclass).fp32;
    q.split = pair ? run.n : INT32_MAX;
    q.end = int32_t(blocks);
    f16 = f16 || class_info(cl.kclass).f16 != 0;
  }
  if (m.n == 0) return 0;
  hipStream_t st = hipStream_t(stream);
  return f16 ? launch_multi_f16(unsigned(blocks), m, st) : launch_multi_bf16(unsigned(blocks), m, st);
}

}  // namespace muon
