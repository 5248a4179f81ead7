// The small-tile Newton-Schulz GEMM kernel: 128 x 128 and 64 x 64 output
// tiles (bf16, fp16 and fp32 operands), the same stages and operand layouts
// as the 256-tile kernel of ns_gemm_kernel.h, whose building blocks it uses.
//
// It runs the matrices whose own class is a small tile, the column and row
// edge strips of the 256 class, and launches of the 256 class that would
// leave much of the chip idle (see exec_tile in plan.cpp).  Such launches
// are bound by the latency of one block's chain of slabs -- direct-to-LDS
// load, barrier, fragment reads, MFMAs -- not by a rate.  The K loop
// therefore keeps NST slabs in a ring and issues the loads of slab k + NST - 1
// while slab k is multiplied, waiting (vmcnt) only for slab k's own loads.
#ifndef MUON_NS_TILE_KERNEL_H
#define MUON_NS_TILE_KERNEL_H

#include "ns_gemm_kernel.h"

namespace muon {
namespace {

// Waits until at most N of this wave's vector memory operations are in
// flight and its LDS reads have returned, then meets the block's barrier.
template <int N>
__device__ __forceinline__ void wait_vm_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// LDS bytes of one slab of both operands, in any operand type.
constexpr int tile_slab_bytes(int tile) { return 2 * tile * 128; }

// Tile number `block` of one launch, in the NST * tile_slab_bytes(TILE) bytes
// of LDS at lds.
template <typename E, int TILE, int STAGE, int NST>
__device__ __forceinline__ void run_tile(const GemmArgs& args, int block, char* lds) {
  using C = Cfg<E, TILE, 2, 2>;
  constexpr bool TRB = STAGE == ST_BX && sizeof(E) == 2;
  constexpr int STG = tile_slab_bytes(TILE);

  const bool second = STAGE == ST_SYM && block >= args.split;
  const TileEntry te = args.tiles[second ? block - args.split : block];
  const int32_t bl = second ? args.l2 : args.l, br = second ? args.r2 : args.r, bo = second ? args.out2 : args.out;
  const MatDev& d = args.mats[te.mat];
  const int32_t slot = te.mat - args.mat_base;
  const int32_t mflag = args.flag[slot];
  const bool zero = mflag != FLAG_LIVE;
  if (mflag == FLAG_SKIP || (zero && !(STAGE == ST_BX && args.last))) return;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
  const int ti = te.ti, tj = te.tj;
  const int wm = wid / 2, wn = wid % 2;
  const int wrow = wm * C::WTM;
  // The two halves of a symmetric product round differently, so which of them
  // is stored follows the matrix's class, not the tile that this launch runs
  // on.  Where the class stores diagonal tiles whole, the tiles inside one
  // (kTileWhole) are stored as computed, in the one pass that the transposed
  // copy is.  Elsewhere (256 classes of several tiles) a diagonal tile keeps
  // the 32 x 32 blocks on or below the diagonal (bmask), stored transposed in
  // their mirror position, and those below it (rmask) also as computed.
  const bool diag = STAGE != ST_BX && ti == tj;
  const bool whole = STAGE != ST_BX && (te.flags & kTileWhole) != 0;
  const bool dtile = diag && !whole;
  uint32_t bmask = 0, rmask = 0;
  if (dtile) {
#pragma unroll
    for (int i = 0; i < C::NBM; ++i)
#pragma unroll
      for (int j = 0; j < C::NBN; ++j) {
        const int rb = wm * C::NBM + i, cb = wn * C::NBN + j;
        if (rb >= cb) bmask |= 1u << (i * C::NBN + j);
        if (rb > cb) rmask |= 1u << (i * C::NBN + j);
      }
  }
  const int64_t mp = d.m_pad, np = d.n_pad;
  // What the epilogue needs of the descriptor and the scale is loaded here: a
  // load after the K loop, whose assembly the compiler moves no load across,
  // would add its latency to every tile.
  const int m = uniform(d.m);
  ApplyDesc ad{};
  if (STAGE == ST_BX && args.last) ad = apply_desc(args.ptrs, d);
  const float sc = args.first ? args.scale[slot] : 1.f;
  E* out_t = nullptr;        // transposed output (leading dimension mp)
  E* out_r = nullptr;        // row-major output
  int64_t ld_r = mp;
  if (STAGE != ST_BX) {
    out_t = reinterpret_cast<E*>(args.ws + d.sq_off[bo]);
    out_r = out_t;
  } else {
    out_t = TRB ? nullptr : reinterpret_cast<E*>(args.ws + d.xt_off[args.pin ^ 1]);
    out_r = reinterpret_cast<E*>(args.ws + d.x_off[args.pin ^ 1]);
    ld_r = np;
  }

  const E* opa;
  const E* opb;
  int64_t K;
  if (STAGE == ST_GRAM) {
    const E* x = reinterpret_cast<const E*>(args.ws + d.x_off[args.pin]);
    K = np;
    opa = x + int64_t(ti) * TILE * K;
    opb = x + int64_t(tj) * TILE * K;
  } else if (STAGE == ST_POLY || STAGE == ST_SYM) {
    K = mp;
    opa = reinterpret_cast<const E*>(args.ws + d.sq_off[bl]) + int64_t(ti) * TILE * K;
    opb = reinterpret_cast<const E*>(args.ws + d.sq_off[STAGE == ST_POLY ? bl : br]) + int64_t(tj) * TILE * K;
  } else {
    K = mp;
    opa = reinterpret_cast<const E*>(args.ws + d.sq_off[bl]) + int64_t(ti) * TILE * K;
    if (TRB)
      opb = reinterpret_cast<const E*>(args.ws + d.x_off[args.pin]) + int64_t(tj) * TILE;
    else
      opb = reinterpret_cast<const E*>(args.ws + d.xt_off[args.pin]) + int64_t(tj) * TILE * K;
  }

  f32x16 acc[C::NBM][C::NBN];
  // fp32 operands: each slab's products are summed into a zeroed partial
  // accumulator, which is added to the result after the slab.  This
  // two-level sum keeps the rounding error of long K loops (K = n up to
  // 14336 for the Gram product) near sqrt(K / 32) + sqrt(32) roundings
  // instead of sqrt(K / 2), the chain of one accumulator through every
  // 32x32x2 step.  The 16-bit classes accumulate directly.
  f32x16 part[C::NBM][C::NBN];
#pragma unroll
  for (int i = 0; i < C::NBM; ++i)
#pragma unroll
    for (int j = 0; j < C::NBN; ++j)
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        acc[i][j][q] = 0.f;
        if constexpr (sizeof(E) == 4) part[i][j][q] = 0.f;
      }

  // K loop up to the last slab that holds a real row or column (the padding
  // is zero and adds nothing)
  const int64_t kreal = STAGE == ST_GRAM ? int64_t(d.rows > d.cols ? d.rows : d.cols) : int64_t(d.m);
  // (a tile that lies wholly in the padding only stores zeros)
  const int64_t nreal = STAGE == ST_BX ? int64_t(d.rows > d.cols ? d.rows : d.cols) : int64_t(d.m);
  const bool pad_tile = int64_t(ti) * TILE >= d.m || int64_t(tj) * TILE >= nreal;
  const int nk = pad_tile ? 0 : int((kreal + C::BK - 1) / C::BK);
  // a*X (B*X) and b*A (A*A, as b/c * A, the product is scaled by c at the
  // end) are folded in while the slab holding them is in LDS.
  const bool FUSE = (STAGE == ST_POLY || STAGE == ST_BX) && args.fcoef != 0.f;
  const float fcoef = args.fcoef;
  const int frow0 = ti * TILE + wrow;
  if (!zero) {
    constexpr int L = 2 * C::CPW;  // loads of one slab per wave
    const E* srca = lane_src<C>(opa, K, wid, lane);
    const E* srcb;
    if constexpr (TRB)
      srcb = lane_src_rows<C, E>(opb, np, wid, lane);
    else
      srcb = lane_src<C>(opb, K, wid, lane);
    int oa[4], ob[4], ot[2 * C::NBN];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      oa[ks] = frag_off(wrow, lane, ks);
      ob[ks] = frag_off(wn * C::WTN, lane, ks);
    }
    if constexpr (TRB) tr_offsets<C>(wn, lane, ot);
    auto load = [&](int kt, char* st) {
      load_slab<C>(srca, K, kt, st, wid);
      if constexpr (TRB)
        load_slab_rows<C>(srcb, np, kt, st + C::OPB, wid);
      else
        load_slab<C>(srcb, K, kt, st + C::OPB, wid);
    };
    int rs = 0, wr = (NST - 1) * STG;  // stage read, stage written this trip
    typename Frag<E>::T fa[2][C::NBM], fb[2][C::NBN];
    auto body = [&](const char* st, int kt) {
      auto rd = [&](int ks, auto& a, auto& b) {
        if constexpr (TRB)
          read_frags_tr<C, E>(st, st + C::OPB, oa[ks], ot, ks, a, b);
        else
          read_frags<C, E>(st, st + C::OPB, oa[ks], ob[ks], a, b);
      };
      // the first fragments are read ahead of the next loads' issue
      rd(0, fa[0], fb[0]);
      if (kt + NST - 1 < nk) load(kt + NST - 1, lds + wr);
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        if (ks < 3) rd(ks + 1, fa[(ks + 1) & 1], fb[(ks + 1) & 1]);
        if constexpr (sizeof(E) == 4)
          mfma_frags<C, E>(fa[ks & 1], fb[ks & 1], part);
        else
          mfma_frags<C, E>(fa[ks & 1], fb[ks & 1], acc);
      }
      if constexpr (sizeof(E) == 4) {
#pragma unroll
        for (int i = 0; i < C::NBM; ++i)
#pragma unroll
          for (int j = 0; j < C::NBN; ++j)
#pragma unroll
            for (int q = 0; q < 16; ++q) {
              acc[i][j][q] += part[i][j][q];
              part[i][j][q] = 0.f;
            }
      }
      if (FUSE) fuse_input<C, E, TRB>(st + C::OPB, kt, frow0, wn, lane, fcoef, acc);
    };
#pragma unroll
    for (int s = 0; s < NST - 1; ++s)
      if (s < nk) load(s, lds + s * STG);
    for (int kt = 0; kt < nk; ++kt) {
      // slab kt has landed once only the loads of the (at most NST - 2) slabs
      // issued after it are in flight; the barrier publishes it and retires
      // the stage that was read in the previous trip
      const int after = nk - 1 - kt < NST - 2 ? nk - 1 - kt : NST - 2;
      static_assert(NST == 2 || NST == 3, "the waits below cover one slab in flight");
      if (NST > 2 && after == 1)
        wait_vm_barrier<L>();
      else
        wait_vm_barrier<0>();
      body(lds + rs, kt);
      __builtin_amdgcn_sched_barrier(0);
      rs = rs == (NST - 1) * STG ? 0 : rs + STG;
      wr = wr == (NST - 1) * STG ? 0 : wr + STG;
    }
    wait_vm_barrier<0>();  // the stages become the epilogue's staging area
  }

  // Epilogue, as in the 256-tile kernel.
  const int64_t row0 = int64_t(ti) * TILE + wrow;
  const int64_t col0 = int64_t(tj) * TILE + wn * C::WTN;
  char* region = lds + wid * C::WAVE_LDS;
  if (STAGE == ST_POLY && diag && args.diag != 0.f) {
    // diag * I on the real diagonal (the padding stays zero)
#pragma unroll
    for (int i = 0; i < C::NBM; ++i)
#pragma unroll
      for (int j = 0; j < C::NBN; ++j)
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          const int r = wrow + 32 * i + 8 * (q >> 2) + 4 * (lane >> 5) + (q & 3);
          const int c = wn * C::WTN + 32 * j + (lane & 31);
          if (r == c && ti * TILE + r < m) acc[i][j][q] += args.diag;
        }
  }
  const float mul = STAGE == ST_GRAM ? args.oscale * sc * sc : STAGE == ST_BX ? args.oscale * sc : args.oscale;
#pragma unroll
  for (int i = 0; i < C::NBM; ++i)
#pragma unroll
    for (int j = 0; j < C::NBN; ++j)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[i][j][q] *= mul;
  if (STAGE == ST_BX && args.last) {
    apply_update_tile<C>(acc, region, args, ad, row0, col0, lane);
  } else if (dtile) {
    if (bmask) store_t_via_lds<C, E, true>(acc, region, out_t, mp, row0, col0, lane, bmask);
    if (rmask) store_rows_via_lds<C, E, true>(acc, region, out_r, ld_r, row0, col0, lane, rmask);
  } else {
    if (!TRB) store_t_via_lds<C, E>(acc, region, out_t, mp, row0, col0, lane);
    if (!whole) store_rows_via_lds<C, E>(acc, region, out_r, ld_r, row0, col0, lane);
  }
}

template <typename E, int TILE, int STAGE, int NST>
__global__ __launch_bounds__(256) void ns_tile_kernel(GemmArgs args) {
  __shared__ __attribute__((aligned(1024))) char lds[NST * tile_slab_bytes(TILE)];
  run_tile<E, TILE, STAGE, NST>(args, int(blockIdx.x), lds);
}

// One launch that carries the current product of several groups of a wave,
// whatever their stage and operand type (16-bit E or fp32), all on 64 tiles.
// Block b belongs to the first part whose `end` exceeds it.
template <typename E>
__global__ __launch_bounds__(256) void ns_multi_kernel(MultiArgs m) {
  __shared__ __attribute__((aligned(1024))) char lds[3 * tile_slab_bytes(64)];
  const int b = int(blockIdx.x);
  int i = 0, begin = 0;
  while (i + 1 < m.n && b >= m.part[i].end) begin = m.part[i++].end;
  const MultiPart& q = m.part[i];
  GemmArgs a = m.common;
  a.tiles = q.tiles;
  a.fcoef = q.g.fcoef;
  a.diag = q.g.diag;
  a.oscale = q.g.oscale;
  a.first = q.g.first;
  a.pin = q.g.pin;
  a.last = q.g.last;
  a.l = q.g.l;
  a.r = q.g.r;
  a.out = q.g.out;
  a.l2 = q.g.l2;
  a.r2 = q.g.r2;
  a.out2 = q.g.out2;
  a.split = q.split;
  const int t = b - begin;
  if (q.fp32) {
    switch (q.stage) {
      case ST_GRAM: run_tile<float, 64, ST_GRAM, 3>(a, t, lds); break;
      case ST_POLY: run_tile<float, 64, ST_POLY, 3>(a, t, lds); break;
      default: run_tile<float, 64, ST_BX, 3>(a, t, lds); break;
    }
  } else {
    switch (q.stage) {
      case ST_GRAM: run_tile<E, 64, ST_GRAM, 3>(a, t, lds); break;
      case ST_POLY: run_tile<E, 64, ST_POLY, 3>(a, t, lds); break;
      case ST_SYM: run_tile<E, 64, ST_SYM, 3>(a, t, lds); break;
      default: run_tile<E, 64, ST_BX, 3>(a, t, lds); break;
    }
  }
}

template <typename E>
int launch_multi(unsigned nblocks, const MultiArgs& m, hipStream_t st) {
  hipLaunchKernelGGL(ns_multi_kernel<E>, dim3(nblocks), dim3(256), 0, st, m);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Any stage of one class.
template <typename E, int TILE, int NST>
int launch_tile(int32_t stage, unsigned nblocks, const GemmArgs& g, hipStream_t st) {
  switch (stage) {
    case ST_GRAM:
      hipLaunchKernelGGL((ns_tile_kernel<E, TILE, ST_GRAM, NST>), dim3(nblocks), dim3(256), 0, st, g);
      break;
    case ST_POLY:
      hipLaunchKernelGGL((ns_tile_kernel<E, TILE, ST_POLY, NST>), dim3(nblocks), dim3(256), 0, st, g);
      break;
    case ST_BX:
      hipLaunchKernelGGL((ns_tile_kernel<E, TILE, ST_BX, NST>), dim3(nblocks), dim3(256), 0, st, g);
      break;
    case ST_SYM:
      // fp32 matrices never take the Gram-space form
      if constexpr (sizeof(E) == 2)
        hipLaunchKernelGGL((ns_tile_kernel<E, TILE, ST_SYM, NST>), dim3(nblocks), dim3(256), 0, st, g);
      else
        return -1;
      break;
    default: return -1;
  }
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace
}  // namespace muon

#endif  // MUON_NS_TILE_KERNEL_H
