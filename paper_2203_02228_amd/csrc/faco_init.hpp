// faco_init.hpp -- the initial solution's local search with 3-opt (gfx950;
// included by ant_in8.hip).
//
// Alg. 2 starts from a nearest-neighbour tour improved with 2-opt and 3-opt
// (Sec. 4.3).  With FACO_LS_INIT_3OPT the ant kernel leaves the plain
// nearest-neighbour tour in ant slot 0 (route, pos, tour coordinates) and the
// whole initial search runs here: every city listed in ascending original
// number, best improvement per listed city trying 2-opt, then Or-opt, then the
// pure 3-opt reconnection (two adjacent blocks exchange places, both keep their
// orientation), and sweeps over all cities until none improves or n changes
// were made.  It is the ants' team search (team_local_search) with the 3-opt
// trial added, one 8-wave workgroup, and its sweeps are launches over the
// whole chip (a wave per city), chained as for the search without 3-opt.
#pragma once
#include "faco_kernels.hpp"

namespace faco {

// The search's workgroup.  mode: MODE_INIT_FIRST (from the nearest-neighbour
// tour) or MODE_INIT_MORE (from the cities the sweep marked).  LDS as run_ant.
template <int KT>
__global__ void __launch_bounds__(64 * kMaxTeam) init_search_kernel(Inst I, int mode) {
  extern __shared__ uint32_t lds[];
  constexpr int TW = kMaxTeam;
  const bool more = mode == MODE_INIT_MORE;
  if (more && uniform_i(I.st->init_done)) return;
  const int W = (I.n + 31) >> 5, lane = lane_id();
  const int w = uniform_i((int)(threadIdx.x >> 6));
  TeamLds *tl = (TeamLds *)lds;
  uint32_t *vis = lds + team_words<TW>();
  uint32_t *inq = vis + W, *ord = inq + W;
  LaneCounters cnt, tk;
  DevState *st = I.st;
  const int64_t t0 = w == 0 ? (more ? st->init_clock : ticks()) : 0;
  int changes = more ? uniform_i(st->init_changes) : 0;
  const int changes0 = changes;
  int64_t len = more ? st->init_cur : st->gb_len;
  Queue Q;
  Q.lr = (int32_t *)(ord + W);
  Q.gr = I.ring;
  int listed = 0;
  if (w == 0) {
    if (more) {
      cnt[CNT_SWEEPS] = 1;
      tk[TK_SWEEP_CITIES] = I.n;
      tk[TK_SWEEP_TESTS] = ticks() - t0;
    }
    search_setup(I, mode, W, 0, I.ring, vis, inq, ord, Q, cnt);
    listed = Q.count;
    if (more) tk[3] = ticks() - t0;
    queue_share(tl, Q);
  }
  team_sync();
  queue_take(tl, Q);
  const uint32_t flags = LS_2OPT | (I.ls_flags & LS_OROPT);
  len -= team_local_search<KT, TW, true>(I, flags, I.routes, I.pos, I.rxy, inq, vis, ord, tl, W, Q,
                                         cnt, tk, -1, w, changes);
  if (w > 0) return;
  init_finish(I, mode, I.routes, len, changes, changes0, listed, more, true, t0, cnt, tk);
  (void)lane;
}

// A sweep over all cities, a wave per city in label order (256 threads).
template <int KT>
__global__ void __launch_bounds__(256) init_sweep3_kernel(Inst I) {
  constexpr int GS = KT <= 16 ? 16 : 32;
  __shared__ alignas(16) int rec[4][kDescWords];
  if (I.st->init_done) return;
  const int w = uniform_i((int)(threadIdx.x >> 6));
  const int x = uniform_i((int)blockIdx.x * 4 + w);
  if (x >= I.n) return;
  const TeamLane T = team_lane<GS>(I, LS_2OPT | (I.ls_flags & LS_OROPT));
  const TeamPre P = team_pre<GS>(I, x);
  int best = team_eval<GS>(I, T, P, I.routes, I.pos, I.rxy, rec[w]);
  if (best == 0) best = team_eval3(I, x, I.routes, I.pos, I.rxy, rec[w]);
  if (best > 0 && lane_id() == 0) {
    const int o = I.orig_of[x];
    atomicOr(&I.marks[o >> 5], 1u << (o & 31));
  }
}

}  // namespace faco
