// faco_kernels.hpp -- HIP kernels of the FACO hot path for gfx950.
//
// One workgroup owns one ant: a team of 8 or 4 waves (or one wave, in large
// batches).  The candidate row of the current city is spread over the lanes, the
// Eq. (1) cumulative sums are formed lane-wise in slot order, the choice is a
// ballot.  In the construction wave 0 decides and the others take shares of its
// wide steps (windows, copies, scans) by command; in the local search every wave
// runs the same loop (faco_team_ls.hpp).  Visited and "on the checklist" sets are
// bitmaps in LDS; tours live in HBM.
#pragma once
#include "device_common.hpp"
#include "faco_device.hpp"
#include "faco_update.hpp"

namespace faco {

// q mod n; the common cases (q within one period of [0, n)) avoid a division
FACO_DEV int64_t ticks() { return (int64_t)wall_clock64(); }

// Clock reads inside the local-search rounds and the construction steps (the
// per-phase breakdown); each one waits for the wave's outstanding LDS and
// scalar operations.  Building with FACO_FINE_TICKS=0 leaves only the
// per-ant totals.
#ifndef FACO_FINE_TICKS
#define FACO_FINE_TICKS 1
#endif
FACO_DEV int64_t fine_ticks() { return FACO_FINE_TICKS ? ticks() : 0; }

// Per-ant event counters and tick sums, one per lane (lane c holds entry c)
// instead of one scalar register pair each: the local search needs the
// scalar registers for its own state.  Updates take the first active lane's
// increment, which is the wave's (every update sits in uniform control flow).
struct LaneCounters {
  int64_t v = 0;
  struct Ref {
    int64_t &v;
    int c;
    FACO_DEV void operator+=(int64_t d) {
      d = (int64_t)uniform_u64((uint64_t)d);
      v += lane_id() == c ? d : 0;
    }
    FACO_DEV void operator++(int) { v += lane_id() == c ? 1 : 0; }
    FACO_DEV void operator=(int64_t x) {
      x = (int64_t)uniform_u64((uint64_t)x);
      v = lane_id() == c ? x : v;
    }
  };
  FACO_DEV Ref operator[](int c) { return Ref{v, c}; }
};

FACO_DEV int wrapn(int q, int n) {
  if (q >= n) {
    q -= n;
    if (q >= n) q %= n;
  } else if (q < 0) {
    q += n;
    if (q < 0) {
      q %= n;
      q = q < 0 ? q + n : q;
    }
  }
  return q;
}
// for -n <= q < 2n
FACO_DEV int wrapc(int q, int n) {
  q += q < 0 ? n : 0;
  return q >= n ? q - n : q;
}
// for 0 <= q < 2n
FACO_DEV int wrap1(int q, int n) { return q >= n ? q - n : q; }

// Offset a source position by |off| <= 4096 (cheap form when n >= 4096).
FACO_DEV int wrap_off(int q, int off, int n) {
  if (n >= 4096) {
    q += off;
    return q >= n ? q - n : (q < 0 ? q + n : q);
  }
  return wrapn(q + off, n);
}

// ===================================================================== //
// Ant teams.  An ant may own TW waves of one workgroup.  In the construction
// (and in the local search on segment lists) wave 0, the leader, runs every
// decision; the other waves wait at a workgroup barrier for a command posted
// in LDS and take a share of the wide steps: source-following windows, copies,
// nearest-city scans, and on segment lists the record passes, Or-opt variants
// and sweep tests.  The local search on flat arrays is run by every wave alike
// (faco_team_ls.hpp).  Who computes a step never changes its result.
//   protocol: leader writes op + arguments, barrier; every wave does its
//   share (a step with a read/write hazard has barriers of its own, taken by
//   every wave alike); barrier; the leader reads what the op left in LDS.
// ===================================================================== //
constexpr int kMaxTeam = 8;
enum TeamOp {
  OP_EXIT, OP_WINDOW, OP_SWEEP, OP_COPY, OP_LENGTH, OP_NEAREST, OP_NEAREST_LABEL, OP_OROPT,
  OP_SEGPERM, OP_SEGMAT, OP_SEARCH, OP_GREEDY
};
constexpr int kDraws = 1024;     // a power of two
constexpr int kDescWords = 36;  // a wave's move record in the team local search
struct TeamLds {
  int op;
  int arg[11];
  uint64_t arg64[2];
  int f[2 * kMaxTeam];           // window: per-wave first stop, by round parity; nearest: per-wave
                                 // original number and index; sweep: per-wave counts
  int res[4];                    // window: [1] the choice that ended it
  int64_t part[kMaxTeam];        // nearest: per-wave distances; length: per-wave cost sums
  int64_t ub[kMaxTeam];          // nearest: per-wave bounds
  int cities[kMaxTeam * kWave];  // sweep: the batch of cities to test
  int disp[4];                   // persistent batches: the next task
  float draws[kDraws];           // roulette draws of the coming steps, by step
  int64_t okey[kMaxTeam][4];     // Or-opt: per-wave maxima of each listed city
  union {
    int orx[14][kWave];          // segment lists' Or-opt: the leader's loaded neighbourhoods
    struct {                     // local search by all waves (team_local_search)
      alignas(16) int desc[2][kMaxTeam * kDescWords];  // each wave's best move, by round parity
      int pushed;                // cities wave 0 listed after the move (bit 8: queue spilled)
      int cnt[2];                // sweep: cities gathered, by pass parity
    } ls;
  };
  int sgs[4];                    // segment-list tour: live buffer, epoch, last move's records
  int sov[9];                    // segment-list move: link overrides
};
template <int TW>
constexpr int team_words() {
  return TW > 1 ? (int)((sizeof(TeamLds) + 15) / 16) * 4 : 0;
}

FACO_DEV void team_post(TeamLds *tl, int op, int a0 = 0, int a1 = 0, int a2 = 0, int a3 = 0,
                        int a4 = 0) {
  if (lane_id() == 0) {
    tl->op = op;
    tl->arg[0] = a0;
    tl->arg[1] = a1;
    tl->arg[2] = a2;
    tl->arg[3] = a3;
    tl->arg[4] = a4;
  }
  team_sync();
}
FACO_DEV int team_arg(const TeamLds *tl, int i) { return uniform_i(tl->arg[i]); }

#include "faco_construct.hpp"

// ===================================================================== //
// Local search (Alg. 3 + Or-opt + sweep)
// ===================================================================== //
// Loads of a segment-list evaluation a split city may come from: the city a
// itself, a neighbour of it, a candidate b, b's successor.
enum { SL_A = 0, SL_NB = 1, SL_B = 2, SL_BS = 3 };
struct Move {
  int kind;  // 0 none, 1 2-opt, 2 Or-opt
  int gain;
  int w, x, y, z;     // 2-opt: remove (w,x), (y,z)
  int px, py, pz;     // positions of x, y, z
  int f, l, p, q, a, o, b, e, L;  // Or-opt
  int fpos, pq, pp, pb, side;     // positions of f, q, p, b; e = succ(b) if side 0
  int s0, s1, s2;     // segment in array order
  int2 xs0, xs1, xs2; // and its coordinates
  // where a segment-list tour finds the cities a move splits at (2-opt: x, z;
  // Or-opt: the segment's first city, q, the insertion edge's second city):
  // the lane holding it and which of its loads (SegEval)
  int ln[3], lk[3];
};

// Or-opt variants in evaluation order, one fixed slot each:
// slot 0..2 = forward L = 1..3, slot 3..4 = backward L = 2..3.
// For slot (dir, L) and nb[j] = route[pa + j - 3]: lanes of f, l, p, q.
constexpr int kOrSlots = 5;
FACO_DEV void or_slot_lanes(int slot, int &dir, int &L, int &lf, int &ll, int &lp, int &lq) {
  dir = slot < 3 ? 0 : 1;
  L = slot < 3 ? slot + 1 : slot - 1;
  if (dir == 0) {
    lf = 3; ll = 3 + L - 1; lp = 2; lq = 3 + L;
  } else {
    lf = 3 - L + 1; ll = 3; lp = 3 - L; lq = 4;
  }
}
FACO_DEV int or_lmax(const Inst &I) {
  return I.oropt_max < I.n - 3 ? I.oropt_max : I.n - 3;
}

FACO_DEV int2 shfl_i2(int2 v, int l) { return make_int2(__shfl(v.x, l), __shfl(v.y, l)); }

// Lane j (constant after unrolling) of the lane's group of GS lanes.
template <int GS>
FACO_DEV int grp_lane(int v, int j) {
  if (GS == 16) return row_bcast(v, j);
  return __shfl(v, (lane_id() & ~(GS - 1)) + j);
}
template <int GS>
FACO_DEV int2 grp_lane2(int2 v, int j) {
  return make_int2(grp_lane<GS>(v.x, j), grp_lane<GS>(v.y, j));
}

// Maximum over the GS lanes of a group (GS = 16: one DPP row; 32: two).
template <int GS>
FACO_DEV int64_t group_max(int64_t v) {
  v = row_reduce_i64(v, OpMax());
  if (GS == 32) {
    const int64_t o = shfl_xor_i64(v, 16);
    v = o > v ? o : v;
  }
  return v;
}

// Per-lane state of a grouped evaluation: GS lanes evaluate one city a
// (slot s = lane % GS handles candidate s), 64 / GS cities per wave.
struct GroupEval {
  int a, pa, b, pb, pbs, pbp, bs, bp, nb, d_ab;
  int uc;          // lane s < 11: neighbourhood cost s of the group's city
  int d_bs, d_bp;  // costs of b's tour edges
  int2 xa, xnb, xb, xbs, xbp;
  int64_t key2, keyo;  // group maxima: 2-opt, Or-opt (0 = none)
};

template <int GS>
FACO_DEV void group_keys(uint32_t flags, bool act, GroupEval &R);

// All loads for both move kinds of every city of the wave are issued
// together (4 dependent levels).  Keys order candidates as the sequential
// evaluation does: 2-opt loop 1 over the list, loop 2 over the list; Or-opt
// variants, list slots, succ before pred.
template <int GS>
FACO_DEV GroupEval eval_group(const Inst &I, uint32_t flags, int a, bool gvalid,
                              const int32_t *route, const int32_t *pos, const int2 *rxy) {
  const int n = I.n, K = I.k, lane = lane_id();
  const int s = lane & (GS - 1);
  const bool act = gvalid && s < K;
  const size_t row = (size_t)a * (size_t)K;
  GroupEval R;
  R.a = a;
  // level 1: indexed by a
  const int pa = pos[a];
  const int b = act ? I.cl[row + s] : a;
  const int d_ab = act ? I.cl_d[row + s] : 0;
  const int2 xa = I.xy[a];
  // level 2
  const int pn = wrapc(pa + (s < 7 ? s : 3) - 3, n);
  const int nb = s < 7 ? route[pn] : a;
  const int2 xnb = s < 7 ? rxy[pn] : xa;
  const int pb = pos[b];
  const int2 xb = I.xy[b];
  // level 3
  const int pbs = pb + 1 == n ? 0 : pb + 1, pbp = pb == 0 ? n - 1 : pb - 1;
  const int bs = route[pbs], bp = route[pbp];
  const int2 xbs = rxy[pbs], xbp = rxy[pbp];
  R.pa = pa; R.b = b; R.pb = pb; R.pbs = pbs; R.pbp = pbp; R.bs = bs; R.bp = bp;
  R.nb = nb; R.xa = xa; R.xnb = xnb; R.xb = xb; R.xbs = xbs; R.xbp = xbp; R.d_ab = d_ab;
  group_keys<GS>(flags, act, R);
  return R;
}

// The loads of a group that never change along a local search: the city's
// candidate row (candidate and cost) and its coordinates.  Loaded for the
// next group while the current move is applied.
struct GroupStatic {
  int a;       // the group's city (-1: none)
  int b, d_ab;
  int2 xa;
};
template <int GS>
FACO_DEV GroupStatic group_static(const Inst &I, int a, bool gvalid) {
  const int K = I.k, s = lane_id() & (GS - 1);
  const bool act = gvalid && s < K;
  const size_t row = (size_t)a * (size_t)K;
  GroupStatic P;
  P.a = gvalid ? a : -1;
  P.b = act ? I.cl[row + s] : a;
  P.d_ab = act ? I.cl_d[row + s] : 0;
  P.xa = I.xy[a];
  return P;
}

// eval_group with the static loads in registers: the positions of a and of
// its candidates are then the first level of loads, and the tour neighbours
// of both the second.
template <int GS>
FACO_DEV GroupEval eval_group_pre(const Inst &I, uint32_t flags, int a, bool gvalid,
                                  const GroupStatic &P, const int32_t *route,
                                  const int32_t *pos, const int2 *rxy) {
  const int n = I.n, K = I.k, lane = lane_id();
  const int s = lane & (GS - 1);
  const bool act = gvalid && s < K;
  GroupEval R;
  R.a = a;
  const int b = P.b, d_ab = P.d_ab;
  const int2 xa = P.xa;
  // level 1
  const int pa = pos[a];
  const int pb = pos[b];
  const int2 xb = I.xy[b];
  // level 2
  const int pn = wrapc(pa + (s < 7 ? s : 3) - 3, n);
  const int nb = s < 7 ? route[pn] : a;
  const int2 xnb = s < 7 ? rxy[pn] : xa;
  const int pbs = pb + 1 == n ? 0 : pb + 1, pbp = pb == 0 ? n - 1 : pb - 1;
  const int bs = route[pbs], bp = route[pbp];
  const int2 xbs = rxy[pbs], xbp = rxy[pbp];
  R.pa = pa; R.b = b; R.pb = pb; R.pbs = pbs; R.pbp = pbp; R.bs = bs; R.bp = bp;
  R.nb = nb; R.xa = xa; R.xnb = xnb; R.xb = xb; R.xbs = xbs; R.xbp = xbp; R.d_ab = d_ab;
  group_keys<GS>(flags, act, R);
  return R;
}

// The part of a group evaluation after the loads: neighbourhood costs and
// the 2-opt keys.
template <int GS>
FACO_DEV void group_keys(uint32_t flags, bool act, GroupEval &R) {
  const int lane = lane_id();
  const int gb = lane & ~(GS - 1);
  const int s = lane & (GS - 1);
  const int2 xnb = R.xnb, xb = R.xb, xbs = R.xbs, xbp = R.xbp;
  const int d_ab = R.d_ab;
  const int2 xas = grp_lane2<GS>(xnb, 4), xap = grp_lane2<GS>(xnb, 2);
  // Costs that depend only on the city's neighbourhood nb_0..nb_6 (tour
  // positions pa-3..pa+3), one per lane of the group: the tour edges
  // (nb_j, nb_j+1), j = 0..5, and the shortcuts (nb_2, nb_4), (nb_2, nb_5),
  // (nb_2, nb_6), (nb_1, nb_4), (nb_0, nb_4) that close the gap a removed
  // Or-opt segment leaves.  Consumers read them from the group's lanes.
  {
    const int su = s <= 5 ? s : (s <= 8 ? 2 : (s == 9 ? 1 : 0));
    const int sv = s <= 5 ? s + 1 : (s <= 8 ? s - 2 : 4);
    R.uc = cost(shfl_i2(xnb, gb + su), shfl_i2(xnb, gb + sv));
  }
  R.d_bs = cost(xb, xbs);
  R.d_bp = cost(xbp, xb);
  R.key2 = 0;
  if (flags & LS_2OPT) {
    const int d_as = grp_lane<GS>(R.uc, 3), d_ap = grp_lane<GS>(R.uc, 2);
    int g1 = 0, g2 = 0;
    if (act && d_as > d_ab) g1 = d_as + R.d_bs - d_ab - cost(xas, xbs);
    if (act && d_ap > d_ab) g2 = d_ap + R.d_bp - d_ab - cost(xap, xbp);
    const int64_t k1 = g1 > 0 ? (((int64_t)g1 << 8) | (int64_t)(255 - s)) : 0;
    const int64_t k2 = g2 > 0 ? (((int64_t)g2 << 8) | (int64_t)(255 - 32 - s)) : 0;
    R.key2 = group_max<GS>(k1 > k2 ? k1 : k2);
  }
  R.keyo = 0;
}

// Or-opt keys for the cities of the groups with `want` set (the others get 0).
// slot_mask selects the segment variants (slots) to evaluate.
template <int GS>
FACO_DEV void eval_group_oropt(const Inst &I, bool want, GroupEval &R,
                               uint32_t slot_mask = (1u << kOrSlots) - 1u) {
  const int n = I.n, K = I.k, lane = lane_id();
  const int s = lane & (GS - 1);
  const bool act = want && s < K;
  const int pa = R.pa, pb = R.pb, pbs = R.pbs, pbp = R.pbp, d_ab = R.d_ab;
  const int2 xnb = R.xnb, xbs = R.xbs, xbp = R.xbp;
  const int Lmax = or_lmax(I);
  int lbest = 0, lidx = 0;
  const int d_bs = R.d_bs, d_bp = R.d_bp;
  int u[11];
#pragma unroll
  for (int j = 0; j < 11; ++j) u[j] = grp_lane<GS>(R.uc, j);
#pragma unroll
  for (int vi = 0; vi < kOrSlots; ++vi) {
    int dir, L, lf, ll, lp, lq;
    or_slot_lanes(vi, dir, L, lf, ll, lp, lq);
    if (L > Lmax || !((slot_mask >> vi) & 1u)) continue;
    const int2 xf = grp_lane2<GS>(xnb, lf), xl = grp_lane2<GS>(xnb, ll);
    const int2 xo = dir == 0 ? xl : xf;
    const int fpos = dir == 0 ? pa : wrapc(pa - L + 1, n);
    // removal: (p, f) + (l, q) - (p, q); rem_a: the edge at a it removes
    const int rem_a = dir == 0 ? u[2] : u[3];
    const int g_rem = dir == 0 ? u[2] + u[2 + L] - u[5 + L]
                               : u[3 - L] + u[3] - (L == 2 ? u[9] : u[10]);
    if (!act) continue;
    if (!(d_ab < rem_a)) continue;
    if (wrapc(pb - fpos, n) < L) continue;
    // costs are >= 0: a variant whose gain without the new edge's cost
    // cannot beat lbest needs no cost
    if (wrapc(pbs - fpos, n) >= L && g_rem + d_bs - d_ab > lbest) {
      const int g = g_rem + d_bs - d_ab - cost(xo, xbs);
      if (g > lbest) {
        lbest = g;
        lidx = (vi * K + s) * 2 + 0;
      }
    }
    if (wrapc(pbp - fpos, n) >= L && g_rem + d_bp - d_ab > lbest) {
      const int g = g_rem + d_bp - d_ab - cost(xo, xbp);
      if (g > lbest) {
        lbest = g;
        lidx = (vi * K + s) * 2 + 1;
      }
    }
  }
  const int64_t key = lbest > 0 ? (((int64_t)lbest << 16) | (int64_t)(0xFFFF - lidx)) : 0;
  R.keyo = group_max<GS>(key);
}

// The move found for the city of group j (uniform j), from the group's lanes.
template <int GS>
FACO_DEV Move extract_move(const Inst &I, const GroupEval &R, int j) {
  const int n = I.n, K = I.k, base = j * GS;
  Move mv = {};
  const int64_t key2 = readlane_i64(R.key2, base);
  const int a = readlane_i(R.a, base);
  const int pa = readlane_i(R.pa, base);
  if (key2 > 0) {
    const int idx = 255 - (int)(key2 & 255);
    mv.kind = 1;
    mv.gain = (int)(key2 >> 8);
    if (idx < 32) {  // loop 1: (a, succ a, b, succ b), flip succ a .. b
      const int l = base + idx;
      mv.w = a; mv.x = readlane_i(R.nb, base + 4);
      mv.y = readlane_i(R.b, l); mv.z = readlane_i(R.bs, l);
      mv.px = pa + 1 == n ? 0 : pa + 1;
      mv.py = readlane_i(R.pb, l);
      mv.pz = readlane_i(R.pbs, l);
      mv.ln[0] = base + 4; mv.lk[0] = SL_NB;
      mv.ln[1] = l; mv.lk[1] = SL_BS;
    } else {         // loop 2: (pred a, a, pred b, b), flip a .. pred b
      const int l = base + idx - 32;
      mv.w = readlane_i(R.nb, base + 2); mv.x = a;
      mv.y = readlane_i(R.bp, l); mv.z = readlane_i(R.b, l);
      mv.px = pa;
      mv.py = readlane_i(R.pbp, l);
      mv.pz = readlane_i(R.pb, l);
      mv.ln[0] = base; mv.lk[0] = SL_A;
      mv.ln[1] = l; mv.lk[1] = SL_B;
    }
    return mv;
  }
  const int64_t keyo = readlane_i64(R.keyo, base);
  if (keyo <= 0) return mv;
  const int idx = 0xFFFF - (int)(keyo & 0xFFFF);
  const int side = idx & 1;
  const int s = (idx >> 1) % K;
  const int vi = (idx >> 1) / K;
  int dir, L, lf, ll, lp, lq;
  or_slot_lanes(vi, dir, L, lf, ll, lp, lq);
  const int l = base + s;
  mv.kind = 2;
  mv.gain = (int)(keyo >> 16);
  mv.L = L;
  mv.a = a;
  mv.f = readlane_i(R.nb, base + lf);
  mv.l = readlane_i(R.nb, base + ll);
  mv.p = readlane_i(R.nb, base + lp);
  mv.q = readlane_i(R.nb, base + lq);
  mv.o = dir == 0 ? mv.l : mv.f;
  mv.b = readlane_i(R.b, l);
  mv.e = side ? readlane_i(R.bp, l) : readlane_i(R.bs, l);
  mv.side = side;
  mv.pb = readlane_i(R.pb, l);
  mv.fpos = dir == 0 ? pa : wrapc(pa - L + 1, n);
  mv.pq = wrapc(mv.fpos + L, n);
  mv.pp = mv.fpos == 0 ? n - 1 : mv.fpos - 1;
  mv.s0 = readlane_i(R.nb, base + lf);
  mv.s1 = readlane_i(R.nb, base + lf + (L > 1 ? 1 : 0));
  mv.s2 = readlane_i(R.nb, base + lf + (L > 2 ? 2 : 0));
  mv.xs0 = readlane_i2(R.xnb, base + lf);
  mv.xs1 = readlane_i2(R.xnb, base + lf + (L > 1 ? 1 : 0));
  mv.xs2 = readlane_i2(R.xnb, base + lf + (L > 2 ? 2 : 0));
  mv.ln[0] = base + lf; mv.lk[0] = SL_NB;
  mv.ln[1] = base + lq; mv.lk[1] = SL_NB;
  mv.ln[2] = l; mv.lk[2] = side ? SL_B : SL_BS;
  return mv;
}

// Lane-serial test used by the sweep (one city per lane): does x have an
// improving move?  Candidate lists are sorted by distance and every move
// through candidate b needs d(x, b) below the longer tour edge at x, so only
// a prefix of the list matters.  The candidates are taken CK at a time (a
// chunk is loaded, then tested), while a lane of the wave still needs them;
// inside a chunk every array index is a compile-time constant, so nothing
// is indexed at run time.
// candidates per chunk of the sweep's test (4: the test stops sooner than
// with 8, measured on the sweeps of the 100k workload; 16 at once spills)
#ifndef FACO_SWEEP_CK
#define FACO_SWEEP_CK 4
#endif
template <int KT>
FACO_DEV bool has_improving(const Inst &I, uint32_t flags, int x,
                            const int32_t *route, const int32_t *pos, const int2 *rxy) {
  constexpr int CK = KT < FACO_SWEEP_CK ? KT : FACO_SWEEP_CK;
  const int n = I.n, K = I.k;
  const int row = x * K;
  // first chunk of the list with the city's own data
  int cb[CK], cd[CK];
#pragma unroll
  for (int j = 0; j < CK; ++j) {
    cb[j] = j < K ? at(I.cl, row + j) : x;
    cd[j] = j < K ? at(I.cl_d, row + j) : 0x7fffffff;
  }
  const int px = at(pos, x);
  const int2 cx = at(I.xy, x);
  int xnx[7], xny[7];
#pragma unroll
  for (int j = 0; j < 7; ++j) {
    const int2 q = at(rxy, wrapc(px + j - 3, n));
    xnx[j] = q.x; xny[j] = q.y;
  }
#define XN(j) make_int2(xnx[j], xny[j])
  const bool two = (flags & LS_2OPT) != 0, orr = (flags & LS_OROPT) != 0;
  const int d_s = cost(cx, XN(4)), d_p = cost(XN(2), cx);
  // Or-opt, per segment slot: where the segment starts, its length, the
  // endpoint that meets the insertion edge, the removed edge at x (0 when
  // the slot cannot apply: no candidate cost is below it) and the removal
  // gain
  int sf[kOrSlots], sl[kOrSlots], srem[kOrSlots], sg[kOrSlots], sox[kOrSlots], soy[kOrSlots];
  int lim = two ? (d_s > d_p ? d_s : d_p) : 0;
  const int Lmax = or_lmax(I);
#pragma unroll
  for (int vi = 0; vi < kOrSlots; ++vi) {
    int dir, L, lf, ll, lp, lq;
    or_slot_lanes(vi, dir, L, lf, ll, lp, lq);
    sl[vi] = L;
    sf[vi] = dir == 0 ? px : wrapc(px - L + 1, n);
    const int2 xo = dir == 0 ? XN(ll) : XN(lf);
    sox[vi] = xo.x;
    soy[vi] = xo.y;
    const int rem = dir == 0 ? d_p : d_s;
    srem[vi] = (orr && L <= Lmax && cd[0] < rem) ? rem : 0;
    sg[vi] = cost(XN(lp), XN(lf)) + cost(XN(ll), XN(lq)) - cost(XN(lp), XN(lq));
    lim = srem[vi] > lim ? srem[vi] : lim;
  }
  bool found = false;
  for (int c0 = 0;;) {
    int pb[CK], xbx[CK], xby[CK];
#pragma unroll
    for (int j = 0; j < CK; ++j) {
      pb[j] = at(pos, cb[j]);
      const int2 q = at(I.xy, cb[j]);
      xbx[j] = q.x; xby[j] = q.y;
    }
    int sx[CK], sy[CK], qx[CK], qy[CK];  // succ and pred of b
#pragma unroll
    for (int j = 0; j < CK; ++j) {
      const int2 q1 = at(rxy, pb[j] + 1 == n ? 0 : pb[j] + 1);
      const int2 q2 = at(rxy, pb[j] == 0 ? n - 1 : pb[j] - 1);
      sx[j] = q1.x; sy[j] = q1.y;
      qx[j] = q2.x; qy[j] = q2.y;
    }
#pragma unroll
    for (int j = 0; j < CK; ++j) {
      const int d_xb = cd[j];
      if (!found && c0 + j < K && d_xb < lim) {
        const int2 xb = make_int2(xbx[j], xby[j]);
        const int2 xbs = make_int2(sx[j], sy[j]), xbp = make_int2(qx[j], qy[j]);
        const int es = cost(xb, xbs) - d_xb, ep = cost(xbp, xb) - d_xb;
        if (two && d_s > d_xb && d_s + es - cost(XN(4), xbs) > 0) found = true;
        if (two && d_p > d_xb && d_p + ep - cost(XN(2), xbp) > 0) found = true;
        const int pbs = pb[j] + 1 == n ? 0 : pb[j] + 1, pbp = pb[j] == 0 ? n - 1 : pb[j] - 1;
#pragma unroll
        for (int vi = 0; vi < kOrSlots; ++vi) {
          const int L = sl[vi], fpos = sf[vi];
          if (!found && d_xb < srem[vi] && wrapc(pb[j] - fpos, n) >= L) {
            const int2 xo = make_int2(sox[vi], soy[vi]);
            // costs are >= 0: no cost of the new edge is needed unless the
            // rest of the gain is positive
            if (wrapc(pbs - fpos, n) >= L) {
              const int rest = sg[vi] + es;
              if (rest > 0 && rest - cost(xo, xbs) > 0) found = true;
            }
            if (wrapc(pbp - fpos, n) >= L) {
              const int rest = sg[vi] + ep;
              if (rest > 0 && rest - cost(xo, xbp) > 0) found = true;
            }
          }
        }
      }
    }
    c0 += CK;
    if (c0 >= K) break;
    // the next chunk, if a lane of the wave still needs it
    const int dn = at(I.cl_d, row + c0);
    if (!ballot(!found && dn < lim)) break;
#pragma unroll
    for (int j = 0; j < CK; ++j) {
      cb[j] = c0 + j < K ? at(I.cl, row + c0 + j) : x;
      cd[j] = c0 + j < K ? at(I.cl_d, row + c0 + j) : 0x7fffffff;
    }
  }
#undef XN
  return found;
}

// The flat tour (arrays in array order) as the sweep's test reads it.
struct FlatT {
  const int32_t *route, *pos;
  const int2 *rxy;
};
template <int KT>
FACO_DEV bool has_improving(const Inst &I, uint32_t flags, int x, const FlatT &T) {
  return has_improving<KT>(I, flags, x, T.route, T.pos, T.rxy);
}

#include "faco_seg.hpp"

// 64-element chunks in flight per wave and round of a team's rewrite.  More hide
// more of a long rewrite's latency and take eight registers each: 8-wave teams,
// one a CU at any tour length, hold 16, which keeps 2 waves per SIMD; 4-wave teams
// 8, so that the many ants of a batch run beside each other (4 waves per SIMD).  A
// batch of 64 instances of 200..5000 cities takes 0.71 ms an iteration on 4-wave
// teams with 8 chunks and 0.83 with 16; a 100k run 4.25 ms on 8-wave teams with 16
// and 4.28 with 8.  (Lone waves: see lone_reverse.)
template <int TW>
constexpr int team_chunks() { return TW == 8 ? 16 : 8; }

// Reverse the cyclic array range of length L starting at s: pairs (i,
// L-1-i) are disjoint, so the 64-pair chunks are dealt to the waves of a
// team of TW in turn (chunk c to wave c mod TW), CH per wave in flight.
template <int TW, int CH = team_chunks<TW>()>
FACO_DEV void reverse_part(int n, int s, int L, int w, int32_t *route, int32_t *pos,
                           int2 *rxy) {
  const int lane = lane_id();
  const int half = L >> 1;
  const int nch = (half + kWave - 1) / kWave;
  for (int c0 = w; c0 < nch; c0 += TW * CH) {
    int p1[CH], p2[CH], v1[CH], v2[CH];
    int c1x[CH], c1y[CH], c2x[CH], c2y[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int i = (c0 + c * TW) * kWave + lane;
      if (i < half) {
        p1[c] = wrap1(s + i, n);
        p2[c] = wrap1(s + L - 1 - i, n);
        v1[c] = at(route, p1[c]);
        v2[c] = at(route, p2[c]);
        const int2 a1 = at(rxy, p1[c]), a2 = at(rxy, p2[c]);
        c1x[c] = a1.x; c1y[c] = a1.y;
        c2x[c] = a2.x; c2y[c] = a2.y;
      }
    }
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int i = (c0 + c * TW) * kWave + lane;
      if (i < half) {
        at(route, p1[c]) = v2[c];
        at(route, p2[c]) = v1[c];
        at(rxy, p1[c]) = make_int2(c2x[c], c2y[c]);
        at(rxy, p2[c]) = make_int2(c1x[c], c1y[c]);
        at(pos, v2[c]) = p1[c];
        at(pos, v1[c]) = p2[c];
      }
    }
  }
}

// Move the cyclic block of D elements at src to dst = src -+ L (L <= 3,
// D + L < n), keeping its order.  down: dst below src, rounds ascend; else
// rounds descend.  A round reads TW * CH * 64 elements, then (after a
// barrier when TW > 1) writes them: no round reads what a later-starting
// write of another wave could clobber.
template <int TW, int CH = team_chunks<TW>()>
FACO_DEV void shift_part(int n, int src, int dst, int D, bool down, int w, int32_t *route,
                         int32_t *pos, int2 *rxy) {
  const int lane = lane_id();
  constexpr int R = TW * CH * kWave;
  const int nr = (D + R - 1) / R;
  for (int r = 0; r < nr; ++r) {
    // round r covers elements [rb, rb + R); its chunks go to the waves in turn
    const int rb = (down ? r : nr - 1 - r) * R;
    int v[CH], cvx[CH], cvy[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int i = rb + (w + c * TW) * kWave + lane;
      if (i < D) {
        const int sp = wrap1(src + i, n);
        v[c] = at(route, sp);
        const int2 q = at(rxy, sp);
        cvx[c] = q.x; cvy[c] = q.y;
      }
    }
    if (TW > 1) team_sync();
#pragma unroll
    for (int c = 0; c < CH; ++c) {
      const int i = rb + (w + c * TW) * kWave + lane;
      if (i < D) {
        const int d = wrap1(dst + i, n);
        at(route, d) = v[c];
        at(rxy, d) = make_int2(cvx[c], cvy[c]);
        at(pos, v[c]) = d;
      }
    }
  }
}

// Rewrites by a lone wave: 4 chunks in flight, and 8 where that leaves rounds.  8
// throughout cost batches of short tours 1..3% (256 instances of 200..5000 cities
// 1322 against 1289 us an iteration); 4 throughout cost long tours 1..4% (200 000
// cities, lists of 12, 4.46 against 4.28 ms).
constexpr int kLoneShort = 4 * kWave;
FACO_DEV void lone_reverse(int n, int s, int L, int32_t *route, int32_t *pos, int2 *rxy) {
  if (L >> 1 <= kLoneShort)
    reverse_part<1, 4>(n, s, L, 0, route, pos, rxy);
  else
    reverse_part<1, 8>(n, s, L, 0, route, pos, rxy);
}
FACO_DEV void lone_shift(int n, int src, int dst, int D, bool down, int32_t *route, int32_t *pos,
                         int2 *rxy) {
  if (D <= kLoneShort)
    shift_part<1, 4>(n, src, dst, D, down, 0, route, pos, rxy);
  else
    shift_part<1, 8>(n, src, dst, D, down, 0, route, pos, rxy);
}

// "Flip a section between x and y": the shorter of the paths x..y and z..w.
// px, py, pz: array positions of x, y, z.
FACO_DEV int apply_2opt(int n, int px, int py, int pz, int32_t *route, int32_t *pos,
                        int2 *rxy) {
  const int L1 = wrapc(py - px, n) + 1;
  const bool first = 2 * L1 <= n;
  const int L = first ? L1 : n - L1;
  lone_reverse(n, first ? px : pz, L, route, pos, rxy);
  wave_fence();
  return L;
}

// Or-opt: the segment and the shorter block between its old place and the
// insertion edge exchange places (block keeps its orientation).
FACO_DEV int apply_oropt(int n, int L, int a, int f, int b, int e, int side,
                         int pb, int fpos, int pq, int pp, int s0, int s1, int s2,
                         int2 xs0, int2 xs1, int2 xs2, int32_t *route, int32_t *pos,
                         int2 *rxy) {
  const int lane = lane_id();
  int x1, px1, px2;
  if (side == 0) {  // e = succ(b): edge (b, e)
    x1 = b;
    px1 = pb;
    px2 = pb + 1 == n ? 0 : pb + 1;
  } else {          // e = pred(b): edge (e, b)
    x1 = e;
    px1 = pb == 0 ? n - 1 : pb - 1;
    px2 = pb;
  }
  // segment in array order, then in the inserted orientation
  int segv = s0;
  segv = lane == 1 ? s1 : segv;
  segv = lane == 2 ? s2 : segv;
  int2 segx = xs0;
  segx = lane == 1 ? xs1 : segx;
  segx = lane == 2 ? xs2 : segx;
  const bool rev = (a != f) != (x1 != b);
  int src_lane = rev ? (L - 1 - lane) : lane;
  src_lane = src_lane < 0 ? 0 : (src_lane > 2 ? 2 : src_lane);
  const int ins = __shfl(segv, src_lane);
  const int2 insx = shfl_i2(segx, src_lane);
  const int D1 = wrapc(px1 - pq, n) + 1;
  const int D2 = wrapc(pp - px2, n) + 1;
  int moved;
  if (D1 <= D2) {
    // block q..x1 moves back by L to start at fpos; segment follows it
    lone_shift(n, pq, fpos, D1, true, route, pos, rxy);
    wave_fence();
    if (lane < L) {
      const int d = wrapc(fpos + D1 + lane, n);
      route[d] = ins;
      rxy[d] = insx;
      pos[ins] = d;
    }
    moved = D1 + L;
  } else {
    // block x2..p moves forward by L; segment goes in front of it
    lone_shift(n, px2, wrap1(px2 + L, n), D2, false, route, pos, rxy);
    wave_fence();
    if (lane < L) {
      const int d = wrap1(px2 + lane, n);
      route[d] = ins;
      rxy[d] = insx;
      pos[ins] = d;
    }
    moved = D2 + L;
  }
  wave_fence();
  return moved;
}

// Work queue of listed cities (FIFO).  Entries sit in an LDS ring while they
// fit (capacity I.lcap <= n), else in the ant's global ring (capacity n);
// a full LDS ring moves its entries to the global ring, oldest first, and
// the queue stays there.  Entries are written by lane 0; LDS operations of
// one wave complete in order, and the global ring is read by lane 0 only.
struct Queue {
  int head, tail, count;
  int cap;      // capacity of the ring in use
  int in_lds;   // 1: the LDS ring
  int32_t *lr;  // LDS ring
  int32_t *gr;  // global ring
};

FACO_DEV void q_spill(Queue &Q, int n) {
  const int lane = lane_id();
  for (int i = lane; i < Q.count; i += kWave) {
    int h = Q.head + i;
    h = h >= Q.cap ? h - Q.cap : h;
    Q.gr[i] = Q.lr[h];
  }
  wave_fence();
  Q.head = 0;
  Q.tail = Q.count == n ? 0 : Q.count;
  Q.cap = n;
  Q.in_lds = 0;
}

// push() of the cities x of the lanes with `take`, in lane order, all at once
// (the cities are distinct).
FACO_DEV int push_lanes(int n, int x, bool take, Queue &Q, uint32_t *inq, uint32_t *touched) {
  const int lane = lane_id();
  take = take && !bit_get(inq, x);
  const uint64_t pm = ballot(take);
  const int np = __builtin_popcountll(pm);
  if (np == 0) return 0;
  if (Q.in_lds && Q.count + np > Q.cap) q_spill(Q, n);
  if (take) {
    int t = Q.tail + __builtin_popcountll(pm & ((1ull << lane) - 1ull));
    t = t >= Q.cap ? t - Q.cap : t;
    bit_set(inq, x);
    bit_set(touched, x);
    (Q.in_lds ? Q.lr : Q.gr)[t] = x;
  }
  if (!Q.in_lds) wave_fence();  // the global ring is read back by lane 0
  Q.tail = Q.tail + np >= Q.cap ? Q.tail + np - Q.cap : Q.tail + np;
  Q.count += np;
  return np;
}

// push() of c[0], c[1], ... in that order, all at once: lane i takes c[i];
// it is listed unless it already is or an earlier lane holds the same city,
// and goes to the tail plus the number of listed lanes before it.
template <int NP>
FACO_DEV void push_all(int n, const int *c, Queue &Q, uint32_t *inq, uint32_t *touched) {
  const int lane = lane_id();
  int x = 0;
#pragma unroll
  for (int i = 0; i < NP; ++i) x = lane == i ? c[i] : x;
  bool take = lane < NP && !bit_get(inq, x);
#pragma unroll
  for (int i = 0; i < NP; ++i)
    if (i < lane && c[i] == x) take = false;
  const uint64_t pm = ballot(take);
  const int np = __builtin_popcountll(pm);
  if (np == 0) return;
  if (Q.in_lds && Q.count + np > Q.cap) q_spill(Q, n);
  if (take) {
    int t = Q.tail + __builtin_popcountll(pm & ((1ull << lane) - 1ull));
    t = t >= Q.cap ? t - Q.cap : t;
    bit_set(inq, x);
    bit_set(touched, x);
    (Q.in_lds ? Q.lr : Q.gr)[t] = x;
  }
  if (!Q.in_lds) wave_fence();  // the global ring is read back by lane 0
  Q.tail = Q.tail + np >= Q.cap ? Q.tail + np - Q.cap : Q.tail + np;
  Q.count += np;
}

// Sweep: test every touched city and list the improvable ones in ascending
// original number.  The touched cities are tested in label order, 64 TW at a
// time (wave w takes the w-th 64): labels follow a space-filling curve, so the
// cities of a batch have nearby candidate rows and tour neighbourhoods.  Each
// improvable city's original number is marked in the `ord` bitmap; `ord` is
// then read in ascending order and the marked cities are listed in that
// order (and `ord` is left clear).  The tour does not change during a sweep,
// so the order of the tests does not matter.
template <int KT, int TW, class TT>
FACO_DEV void sweep_part(const Inst &I, uint32_t flags, int count, int w, TeamLds *tl,
                         uint32_t *ord, const TT &T) {
  const int i = w * kWave + lane_id();
  if (i < count) {
    const int x = tl->cities[i];
    const int ox = I.orig_of[x];
    if (has_improving<KT>(I, flags, x, T)) bit_set(ord, ox);
  }
}

// Sweep tick slots (per ant): ticks in the move tests, ticks in listing the
// improvable cities, cities tested.
enum { TK_SWEEP_TESTS = 24, TK_SWEEP_LIST = 25, TK_SWEEP_CITIES = 26 };

// List the cities marked in `ord` (by original number) in ascending order, 64
// at a time, and leave `ord` clear; the number listed.  One wave.
FACO_DEV int list_marked(const Inst &I, int W, Queue &Q, uint32_t *inq, uint32_t *touched,
                         uint32_t *ord) {
  const int lane = lane_id();
  int pushed = 0, bo = -1;
  int bcount = 0;
  auto list = [&](int cnt) {
    const int x = lane < cnt ? I.int_of[bo] : 0;
    pushed += cnt;
    push_lanes(I.n, x, lane < cnt, Q, inq, touched);
  };
  for (int w0 = 0; w0 < W; w0 += kWave) {
    const uint32_t word = (w0 + lane < W) ? ord[w0 + lane] : 0u;
    if (w0 + lane < W) ord[w0 + lane] = 0u;
    uint64_t nz = ballot(word != 0u);
    while (nz) {
      const int l = ctz64(nz);
      nz &= nz - 1;
      uint32_t bits = (uint32_t)readlane_i((int)word, l);
      while (bits) {
        const int bpos = __builtin_ctz(bits);
        bits &= bits - 1;
        if (lane == bcount) bo = (w0 + l) * 32 + bpos;
        if (++bcount == kWave) {
          list(kWave);
          bcount = 0;
        }
      }
    }
  }
  if (bcount) list(bcount);
  return pushed;
}

template <int KT, int TW, class TT>
FACO_DEV int sweep(const Inst &I, uint32_t flags, int W, Queue &Q, const TT &T,
                   uint32_t *inq, uint32_t *touched, uint32_t *ord, TeamLds *tl,
                   LaneCounters &tk) {
  const int lane = lane_id();
  int bx = -1, bcount = 0;
  auto test = [&](int cnt) {
    const int64_t t0 = fine_ticks();
    tk[TK_SWEEP_CITIES] += cnt;
    if (TW == 1) {
      if (lane < cnt) {
        const int ox = I.orig_of[bx];
        if (has_improving<KT>(I, flags, bx, T)) bit_set(ord, ox);
      }
      tk[TK_SWEEP_TESTS] += fine_ticks() - t0;
      return;
    }
    // cnt cities sit in tl->cities[0..cnt)
    team_post(tl, OP_SWEEP, cnt, (int)flags);
    sweep_part<KT, TW>(I, flags, cnt, 0, tl, ord, T);
    team_sync();
    tk[TK_SWEEP_TESTS] += fine_ticks() - t0;
  };
  if (TW == 1) {
    for (int w0 = 0; w0 < W; w0 += kWave) {
      const uint32_t word = (w0 + lane < W) ? touched[w0 + lane] : 0u;
      uint64_t nz = ballot(word != 0u);
      while (nz) {
        const int l = ctz64(nz);
        nz &= nz - 1;
        uint32_t bits = (uint32_t)readlane_i((int)word, l);
        while (bits) {
          const int bpos = __builtin_ctz(bits);
          bits &= bits - 1;
          if (lane == bcount) bx = (w0 + l) * 32 + bpos;
          if (++bcount == kWave) {
            test(kWave);
            bcount = 0;
          }
        }
      }
    }
    if (bcount) test(bcount);
  } else {
    // every lane with touched bits in its word places its lowest one per
    // pass (the order of the tests does not matter), slots by rank
    constexpr int cap = TW * kWave;
    int fill = 0;
    for (int w0 = 0; w0 < W; w0 += kWave) {
      uint32_t word = (w0 + lane < W) ? touched[w0 + lane] : 0u;
      for (;;) {
        const uint64_t m = ballot(word != 0u);
        if (!m) break;
        const int room = cap - fill;
        const int r = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        if (word != 0u && r < room) {
          tl->cities[fill + r] = (w0 + lane) * 32 + __builtin_ctz(word);
          word &= word - 1u;
        }
        const int np = __builtin_popcountll(m);
        fill += np < room ? np : room;
        if (fill == cap) {
          test(cap);
          fill = 0;
        }
      }
    }
    if (fill) test(fill);
  }
  wave_fence();
  const int64_t tl0 = fine_ticks();
  const int pushed = list_marked(I, W, Q, inq, touched, ord);
  tk[TK_SWEEP_LIST] += fine_ticks() - tl0;
  return pushed;
}

// The Or-opt evaluation of an LS round, shared by the helper waves of a team.
// The leader has loaded the listed cities' neighbourhoods and evaluated the
// 2-opt moves; when a city before the first one with a 2-opt move needs
// Or-opt, it leaves what the evaluation needs in tl->orx (lane by lane) and
// helper wave w (1 <= w < TW) takes segment variants w - 1, w - 1 + (TW - 1),
// ... for the cities before arg[0], leaving each city's maximum key in
// tl->okey[w].  Keys order variants as the sequential evaluation does, so the
// maximum over the waves is the sequential evaluation's result.
template <int TW>
FACO_DEV uint32_t or_slot_mask(int w) {
  uint32_t m = 0;
  for (int vi = w - 1; vi >= 0 && vi < kOrSlots; vi += TW - 1) m |= 1u << vi;
  return m;
}

FACO_DEV void or_share(TeamLds *tl, const GroupEval &R) {
  const int l = lane_id();
  tl->orx[0][l] = R.pa;
  tl->orx[1][l] = R.pb;
  tl->orx[2][l] = R.pbs;
  tl->orx[3][l] = R.pbp;
  tl->orx[4][l] = R.d_ab;
  tl->orx[5][l] = R.d_bs;
  tl->orx[6][l] = R.d_bp;
  tl->orx[7][l] = R.uc;
  tl->orx[8][l] = R.xnb.x;
  tl->orx[9][l] = R.xnb.y;
  tl->orx[10][l] = R.xbs.x;
  tl->orx[11][l] = R.xbs.y;
  tl->orx[12][l] = R.xbp.x;
  tl->orx[13][l] = R.xbp.y;
}

template <int KT, int TW>
FACO_DEV void oropt_part(const Inst &I, int w, TeamLds *tl) {
  constexpr int GS = KT <= 16 ? 16 : 32;
  const uint32_t mask = or_slot_mask<TW>(w);
  if (!mask) return;
  const int l = lane_id(), grp = l / GS;
  const int j2 = team_arg(tl, 0);
  GroupEval R;
  R.pa = tl->orx[0][l];
  R.pb = tl->orx[1][l];
  R.pbs = tl->orx[2][l];
  R.pbp = tl->orx[3][l];
  R.d_ab = tl->orx[4][l];
  R.d_bs = tl->orx[5][l];
  R.d_bp = tl->orx[6][l];
  R.uc = tl->orx[7][l];
  R.xnb = make_int2(tl->orx[8][l], tl->orx[9][l]);
  R.xbs = make_int2(tl->orx[10][l], tl->orx[11][l]);
  R.xbp = make_int2(tl->orx[12][l], tl->orx[13][l]);
  eval_group_oropt<GS>(I, grp < j2, R, mask);
  if ((l & (GS - 1)) == 0) tl->okey[w][grp] = R.keyo;
}

// The first fault of the instance keeps its ant (-1: the initial solution)
// and the iteration being built.
FACO_DEV void record_fault(const Inst &I, int32_t bit, int ant) {
  if (lane_id() == 0) {
    if (atomicOr(&I.st->fault, bit) == 0) {
      I.st->fault_ant = ant;
      I.st->fault_iter = I.st->iter + 1;
    }
  }
}

// SEG: the tour is a segment list (SQ); else the flat arrays route, pos, rxy.
// changes: moves made before (in) and by the end (out).
template <int KT, int TW, bool SEG>
FACO_DEV int64_t local_search(const Inst &I, uint32_t flags, int32_t *route,
                              int32_t *pos, int2 *rxy, uint32_t *inq, uint32_t *touched,
                              uint32_t *ord, TeamLds *tl, int W, Queue Q, LaneCounters &cnt,
                              LaneCounters &tk, int ant, SegState &SQ, int &changes) {
  constexpr int GS = KT <= 16 ? 16 : 32;  // lanes per evaluated city
  constexpr int G = kWave / GS;           // cities evaluated together
  const int n = I.n, lane = lane_id();
  const int grp = lane / GS;
  flags = (uint32_t)uniform_i((int)flags);
  int changes_at_sweep = -1;
  int64_t gain = 0;
  // The next round's static loads (its groups' candidate rows and
  // coordinates), issued during this round for the groups it will most
  // likely hold; used if it holds them.
  GroupStatic pre;
  pre.a = -1;
  pre.b = pre.d_ab = 0;
  pre.xa = make_int2(0, 0);
  for (;;) {
    for (;;) {
      Q.count = uniform_i(Q.count);
      Q.head = uniform_i(Q.head);
      Q.tail = uniform_i(Q.tail);
      Q.cap = uniform_i(Q.cap);
      Q.in_lds = uniform_i(Q.in_lds);
      changes = uniform_i(changes);
      if (!(Q.count > 0 && changes < n)) break;
      // Evaluate the next G listed cities on the current tour.  The first one
      // with a move is applied; the ones before it are popped with no move;
      // the ones after it stay listed (their evaluation is discarded).
      const int gcount = Q.count < G ? Q.count : G;
      int e[G];
      if (Q.in_lds) {
        int h = Q.head + lane;
        h = h >= Q.cap ? h - Q.cap : h;
        const int hv = lane < gcount ? Q.lr[h] : 0;
#pragma unroll
        for (int g = 0; g < G; ++g) e[g] = readlane_i(hv, g);
      } else {
#pragma unroll
        for (int g = 0; g < G; ++g) {
          int h = Q.head + g;
          h = h >= Q.cap ? h - Q.cap : h;
          e[g] = readlane_i(lane == 0 && g < gcount ? Q.gr[h] : 0, 0);
        }
      }
      int a = e[0];
#pragma unroll
      for (int g = 1; g < G; ++g) a = grp == g ? e[g] : a;
      const int64_t t0 = fine_ticks();
      SegEval Z;
      GroupEval R;
      if constexpr (SEG) {
        R = eval_group_seg<GS>(I, flags, a, grp < gcount, SQ.T, Z);
      } else {
        // the prefetched loads serve if every group is full and holds the
        // city they were loaded for
        const bool hit = ballot(!(grp < gcount && pre.a == a)) == 0ull;
        if (hit)
          R = eval_group_pre<GS>(I, flags, a, true, pre, route, pos, rxy);
        else
          R = eval_group<GS>(I, flags, a, grp < gcount, route, pos, rxy);
        pre.a = -1;
      }
      // Or-opt is only tried where no 2-opt move exists, and only cities
      // before the first one with a 2-opt move can be the chosen one
      const uint64_t h2 = ballot((lane & (GS - 1)) == 0 && grp < gcount && R.key2 > 0);
      const int j2 = uniform_i(h2 ? ctz64(h2) / GS : gcount);
      // Most likely the move is the first 2-opt one (j2) and the next round
      // holds the G listed cities after it: load their static data now,
      // beside the rest of this round (a wrong guess only costs the loads).
      if constexpr (!SEG) {
        const int np_guess = j2 < gcount ? j2 + 1 : gcount;
        if (Q.in_lds && j2 < gcount && Q.count - np_guess >= G) {
          int h = Q.head + np_guess + grp;
          h = h >= Q.cap ? h - Q.cap : h;
          pre = group_static<GS>(I, Q.lr[h], true);
        }
      }
      if (TW > 1 && (flags & LS_OROPT) && j2 > 0) {
        // the team's helpers evaluate the Or-opt variants from the leader's loads
        const int64_t to = fine_ticks();
        or_share(tl, R);
        team_post(tl, OP_OROPT, j2);
        team_sync();
        int64_t k = 0;
#pragma unroll
        for (int w = 1; w < TW; ++w)
          if (or_slot_mask<TW>(w)) {
            const int64_t kw = tl->okey[w][grp];
            k = kw > k ? kw : k;
          }
        R.keyo = grp < j2 ? k : 0;
        tk[14]++;
        tk[13] += fine_ticks() - to;
      } else if ((flags & LS_OROPT) && j2 > 0) {
        const int64_t to = fine_ticks();
        eval_group_oropt<GS>(I, grp < j2, R);
        tk[13] += fine_ticks() - to;
        tk[14]++;
      }
      const int64_t t1 = fine_ticks();
      tk[1] += t1 - t0;
      tk[12]++;
      const uint64_t hm = ballot((lane & (GS - 1)) == 0 && grp < gcount &&
                                 (R.key2 > 0 || R.keyo > 0));
      const int j = hm ? ctz64(hm) / GS : gcount;
      const int npop = j < gcount ? j + 1 : gcount;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        if (g < npop) {
          if (lane == 0) bit_clear(inq, e[g]);
          Q.head = Q.head + 1 == Q.cap ? 0 : Q.head + 1;
          Q.count--;
        }
      }
      cnt[CNT_LS_POPS] += npop;
      if (j >= gcount) continue;
      const Move mv = extract_move<GS>(I, R, j);
      const int64_t ta = fine_ticks();
      if (uniform_i(mv.kind) == 1) {
        if constexpr (SEG)
          cnt[CNT_MOVED_ELEMS] += seg_apply_2opt<TW>(I, SQ, tl, mv, Z, tk);
        else
          cnt[CNT_MOVED_ELEMS] += apply_2opt(n, uniform_i(mv.px), uniform_i(mv.py),
                                             uniform_i(mv.pz), route, pos, rxy);
        tk[15] += fine_ticks() - ta;
        const int pc[4] = {mv.w, mv.x, mv.y, mv.z};
        push_all<4>(n, pc, Q, inq, touched);
        cnt[CNT_MOVES_2OPT]++;
      } else {
        if constexpr (SEG)
          cnt[CNT_MOVED_ELEMS] += seg_apply_oropt<TW>(I, SQ, tl, mv, Z, tk);
        else
          cnt[CNT_MOVED_ELEMS] +=
              apply_oropt(n, uniform_i(mv.L), mv.a, mv.f, mv.b, mv.e, uniform_i(mv.side),
                          uniform_i(mv.pb), uniform_i(mv.fpos), uniform_i(mv.pq),
                          uniform_i(mv.pp), mv.s0, mv.s1, mv.s2, mv.xs0, mv.xs1, mv.xs2,
                          route, pos, rxy);
        tk[15] += fine_ticks() - ta;
        const int pc[6] = {mv.p, mv.q, mv.b, mv.e, mv.f, mv.l};
        push_all<6>(n, pc, Q, inq, touched);
        cnt[CNT_MOVES_OROPT]++;
      }
      if constexpr (SEG) {
        // room for the next move's splits
        if (uniform_i(SQ.S) + 3 > I.seg_max) seg_materialize<TW>(I, ant < 0 ? 0 : ant, SQ, tl, tk);
      }
      tk[2] += fine_ticks() - t1;
      ++changes;
      gain += mv.gain;
    }
    changes = uniform_i(changes);
    if (!(flags & LS_SWEEP) || changes >= n) break;
    // Every city a sweep lists has an improving move, so a sweep that was
    // followed by no change can only come from the two move tests
    // disagreeing: stop instead of spinning, and report it.
    if (changes == changes_at_sweep) {
      record_fault(I, FAULT_LS_STALL, ant);
      break;
    }
    changes_at_sweep = changes;
    cnt[CNT_SWEEPS]++;
    const int64_t t2 = ticks();
    int pushed;
    if constexpr (SEG)
      pushed = uniform_i(sweep<KT, TW>(I, flags, W, Q, SQ.T, inq, touched, ord, tl, tk));
    else
      pushed = uniform_i(sweep<KT, TW>(I, flags, W, Q, FlatT{route, pos, rxy}, inq, touched,
                                       ord, tl, tk));
    tk[3] += ticks() - t2;
    if (pushed == 0) break;
  }
  cnt[CNT_LS_GAIN] += gain;
  return gain;
}

#include "faco_team_ls.hpp"

// ===================================================================== //
// Helper waves of a team: wait for a command, take this wave's share, repeat
// until the leader posts OP_EXIT or OP_SEARCH (returned).
// ===================================================================== //
template <int KT, int TW, bool SEG>
FACO_DEV int team_helper(const Inst &I, int ant, int w, TeamLds *tl, uint32_t *vis,
                          uint32_t *ord, int32_t *route, int32_t *pos, int2 *rxy, int4 *rec) {
  int64_t lane_len = 0;  // costs of the edges this wave's lanes appended
  // a segment-list move's record whose cities this wave labels after the move
  int rl_h = -1, rl_lo = 0, rl_hi = -1;
  SegT rl_T;
  for (;;) {
    if (SEG && rl_h >= 0) {
      seg_relabel(rl_T, rl_lo, rl_hi, rl_h);
      rl_h = -1;
    }
    team_sync();
    const int op = uniform_i(tl->op);
    if (op == OP_EXIT || op == OP_SEARCH) return op;
    if (op == OP_WINDOW) {
      WinOut o;
      int have = team_arg(tl, 4);
      window_rounds<KT, TW>(I, uniform_u64(tl->arg64[0]), (uint64_t)ant, team_arg(tl, 3),
                            team_arg(tl, 0), team_arg(tl, 1), team_arg(tl, 2), w, have, tl, vis,
                            route, pos, rxy, lane_len, o);
      continue;  // the command ended at its own last barrier
    } else if (op == OP_COPY) {
      copy_part<TW>(I, team_arg(tl, 0), team_arg(tl, 1), team_arg(tl, 2), team_arg(tl, 3), w,
                    route, pos, rxy, lane_len);
    } else if (op == OP_LENGTH) {
      const int64_t sum = wave_sum_i64(lane_len);
      if (lane_id() == 0) tl->part[w] = sum;
    } else if (op == OP_NEAREST || op == OP_NEAREST_LABEL) {
      int64_t md;
      int mj;
      if (op == OP_NEAREST)
        nearest_part<true, TW>(I, team_arg(tl, 0), w, vis, tl, md, mj);
      else
        nearest_part<false, TW>(I, team_arg(tl, 0), w, vis, tl, md, mj);
    } else if (op == OP_GREEDY) {
      if (w == 1) greedy_rows(I, tl);
    } else if (SEG && op == OP_SWEEP) {
      sweep_part<KT, TW>(I, (uint32_t)team_arg(tl, 1), team_arg(tl, 0), w, tl, ord,
                         seg_view(I, ant, rec, uniform_i(tl->sgs[0]), uniform_i(tl->sgs[1]),
                                  uniform_i(tl->sgs[2]), uniform_i(tl->sgs[3])));
    } else if (SEG && op == OP_SEGPERM) {
      const SegT T = seg_view(I, ant, rec, uniform_i(tl->sgs[0]), uniform_i(tl->sgs[1]));
      const int rv = team_arg(tl, 5);
      const int S0 = team_arg(tl, 0), S = team_arg(tl, 1);
      // the new record this wave labels: read before the pass's barrier (the
      // leader may change records again once the move is over)
      if (S0 + w - 1 < S) {
        const int4 r = rec[S0 + w - 1];
        rl_h = S0 + w - 1;
        rl_lo = uniform_i(r.x);
        rl_hi = uniform_i(r.y);
        rl_T = T;
      }
      SegOv O;
#pragma unroll
      for (int j = 0; j < kSovPre + kSovPost; ++j) O.v[j] = uniform_i(tl->sov[j]);
      seg_perm_part(T, w * kWave + lane_id(), kWave * TW, S, team_arg(tl, 2), team_arg(tl, 3),
                    team_arg(tl, 4), rv & 1, (rv >> 1) & 1, O, team_arg(tl, 6),
                    team_arg(tl, 7));
      if (!FACO_SEG_DEFER && rl_h >= 0) {
        seg_relabel(rl_T, rl_lo, rl_hi, rl_h);
        rl_h = -1;
      }
    } else if (SEG && op == OP_SEGMAT) {
      const int live = uniform_i(tl->sgs[0]);
      const SegT T = seg_view(I, ant, rec, live, uniform_i(tl->sgs[1]), uniform_i(tl->sgs[2]),
                              uniform_i(tl->sgs[3]));
      const size_t o = (size_t)ant * (size_t)I.n;
      const int tid = w * kWave + lane_id();
      seg_mat_part(T, tid, kWave * TW, (live ? I.routes : I.r2) + o, (live ? I.rxy : I.x2) + o,
                   (live ? I.pos : I.p2) + o);
      team_sync();
      seg_reset_part(rec, tid, kWave * TW, (I.n + (1 << I.seg_shift) - 1) >> I.seg_shift, I.n,
                     I.seg_shift);
    } else if (SEG && op == OP_OROPT) {
      oropt_part<KT, TW>(I, w, tl);
    }
    team_sync();
  }
}

// ===================================================================== //
// One ant: construction + local search.  MODE_ANT: ant `ant` of iteration
// st->iter + 1.  MODE_INIT: initial solution (nearest neighbour + LS over all
// cities) written to the global best.  MODE_INIT_FIRST, MODE_INIT_MORE: the
// same with the sweeps in launches of their own (init_sweep_kernel, the whole
// chip instead of one workgroup): the first launch searches until no city is
// listed, each later one lists what the sweep before it marked and goes on;
// one that finds nothing marked ends the search (DevState.init_done).
//   lds: [team area][visited W][listed W][sweep order W]
//        [SEG: segment records, I.seg_max int4 at a 16-byte boundary]
//        [queue ring I.lcap].
// ===================================================================== //
enum { MODE_ANT = 0, MODE_INIT = 1, MODE_INIT_FIRST = 2, MODE_INIT_MORE = 3 };
__host__ __device__ inline int seg_lds_words(int tw_words, int W) { return (tw_words + 3 * W + 3) & ~3; }

// The queue and bitmaps the local search starts from (leader wave); returns
// the flags it runs with.
FACO_DEV uint32_t search_setup(const Inst &I, int mode, int W, int nchk, int32_t *ring,
                               uint32_t *vis, uint32_t *inq, uint32_t *ord, Queue &Q,
                               LaneCounters &cnt) {
  const int n = I.n, lane = lane_id();
  uint32_t flags = I.ls_flags;
  const int lcap = I.lcap;
  if (mode == MODE_INIT_MORE) {
    // the cities the sweep marked, in ascending original number
    for (int w = lane; w < W; w += kWave) {
      ord[w] = I.marks[w];
      inq[w] = 0u;
      vis[w] = 0u;
      I.marks[w] = 0u;
    }
    Q.in_lds = 1;
    Q.cap = lcap;
    Q.head = Q.tail = Q.count = 0;
    wave_fence();
    list_marked(I, W, Q, inq, vis, ord);
    wave_fence();
    return LS_2OPT | (I.ls_flags & LS_OROPT);
  }
  if (mode != MODE_ANT) {
    // the initial solution reports only its local-search counters
#pragma unroll
    for (int c = 0; c < CNT_LS_POPS; ++c) cnt[c] = 0;
    // with 3-opt, the initial search runs in init_search_kernel afterwards
    flags = LS_2OPT | (mode == MODE_INIT ? LS_SWEEP : 0u) | (I.ls_flags & LS_OROPT);
    if (I.ls_flags & LS_INIT_3OPT) flags = 0u;
    if (mode == MODE_INIT_FIRST)
      for (int w = lane; w < W; w += kWave) I.marks[w] = 0u;
    Q.in_lds = n <= lcap ? 1 : 0;
    Q.cap = Q.in_lds ? lcap : n;
    // every city listed, in ascending original number
    for (int i = lane; i < n; i += kWave) (Q.in_lds ? Q.lr : ring)[i] = I.int_of[i];
    for (int w = lane; w < W; w += kWave) {
      const int rem = n - w * 32;
      const uint32_t full = rem >= 32 ? 0xFFFFFFFFu : ((1u << rem) - 1u);
      inq[w] = full;
      vis[w] = full;  // touched
    }
    Q.count = n;
    cnt[CNT_CHECKLIST0] = n;
  } else {
    for (int w = lane; w < W; w += kWave) vis[w] = 0u;
    wave_fence();
    Q.in_lds = nchk <= lcap ? 1 : 0;
    Q.cap = Q.in_lds ? lcap : n;
    for (int i = lane; i < nchk; i += kWave) {
      const int c = ring[i];
      bit_set(vis, c);
      if (Q.in_lds) Q.lr[i] = c;
    }
    Q.count = nchk;
    if (flags & (LS_2OPT | LS_OROPT)) cnt[CNT_CHECKLIST0] = nchk;
  }
  Q.head = 0;
  Q.tail = Q.count == Q.cap ? 0 : Q.count;
  for (int w = lane; w < W; w += kWave) ord[w] = 0u;  // sweeps leave it clear
  wave_fence();
  flags = (uint32_t)uniform_i((int)flags);
  Q.head = uniform_i(Q.head);
  Q.tail = uniform_i(Q.tail);
  Q.count = uniform_i(Q.count);
  Q.cap = uniform_i(Q.cap);
  Q.in_lds = uniform_i(Q.in_lds);
  return flags;
}

// End of a launch of the initial search (wave 0): its state, counters and ticks
// (added to the earlier launches' with add_cnt, add_tk), and the global best
// once the search has ended: in MODE_INIT, when the sweep marked nothing, or at
// n moves.  Marked cities without a move are the two move tests disagreeing.
FACO_DEV void init_finish(const Inst &I, int mode, const int32_t *route, int64_t len, int changes,
                          int changes0, int listed, bool add_cnt, bool add_tk, int64_t t0,
                          LaneCounters &cnt, LaneCounters &tk) {
  const int n = I.n, lane = lane_id();
  DevState *st = I.st;
  bool done = mode == MODE_INIT || changes >= n;
  if (mode == MODE_INIT_MORE && changes == changes0) {
    done = true;
    if (uniform_i(listed) > 0) record_fault(I, FAULT_LS_STALL, -1);
  }
  if (done)
    for (int i = lane; i < n; i += kWave) I.gb_route[i] = route[i];
  const int64_t t1 = ticks();
  tk[4] = t1 - t0;
  if (lane == 0) {
    st->init_done = done ? 1 : 0;
    st->init_changes = changes;
    st->init_cur = len;
    st->init_clock = t1;
    if (done) {
      st->gb_len = len;
      st->init_len = len;
    }
  }
  if (lane < NCNT) st->init_cnt[lane] = cnt.v + (add_cnt ? st->init_cnt[lane] : 0);
  if (lane < kTicks) st->init_ticks[lane] = tk.v + (add_tk ? st->init_ticks[lane] : 0);
}

template <int KT, int TW, bool SEG = false>
FACO_DEV void run_ant(const Inst &I, int ant, int mode, uint32_t *lds) {
  const int n = I.n, lane = lane_id();
  const int W = (n + 31) >> 5;
  TeamLds *tl = (TeamLds *)lds;
  uint32_t *vis = lds + team_words<TW>();
  uint32_t *inq = vis + W;
  uint32_t *ord = inq + W;
  int4 *rec = (int4 *)(lds + seg_lds_words(team_words<TW>(), W));
  int32_t *route = I.routes + (size_t)ant * (size_t)n;
  int32_t *pos = I.pos + (size_t)ant * (size_t)n;
  int32_t *ring = I.ring + (size_t)ant * (size_t)n;
  int2 *rxy = I.rxy + (size_t)ant * (size_t)n;
  const int w = TW > 1 ? uniform_i((int)(threadIdx.x >> 6)) : 0;
  const bool init = mode != MODE_ANT, more = mode == MODE_INIT_MORE;
  if (more && uniform_i(I.st->init_done)) return;
  LaneCounters cnt, tk;
  // a later launch of the initial search counts the sweep before it
  const int64_t t0 = w == 0 ? (more ? I.st->init_clock : ticks()) : 0;
  int64_t len = 0;
  uint32_t flags = 0;
  int changes = more ? uniform_i(I.st->init_changes) : 0, listed = 0;
  const int changes0 = changes;
  Queue Q;
  Q.lr = SEG ? (int32_t *)(rec + I.seg_max) : (int32_t *)(ord + W);
  Q.gr = ring;
  SegState SQ;
  if (TW > 1 && w > 0) {
    if (team_helper<KT, TW, SEG>(I, ant, w, tl, vis, ord, route, pos, rxy, rec) == OP_EXIT)
      return;
  } else {
    int nchk = 0;
    if (more) {
      len = I.st->init_cur;
      cnt[CNT_SWEEPS] = 1;
      tk[TK_SWEEP_CITIES] = n;
      tk[TK_SWEEP_TESTS] = ticks() - t0;
    } else {
      len = init ? construct_greedy<TW>(I, route, pos, rxy, vis, inq, tl, W, cnt)
                 : construct<KT, TW>(I, (uint64_t)I.st->iter + 1, ant, route, pos, rxy, ring,
                                     vis, inq, tl, W, nchk, cnt, tk);
      tk[0] = ticks() - t0;
    }
    flags = search_setup(I, mode, W, nchk, ring, vis, inq, ord, Q, cnt);
    listed = Q.count;
    if (more) tk[3] = ticks() - t0;
    if constexpr (SEG || TW == 1) {
      if constexpr (SEG) seg_begin(I, ant, rec, tl, TW > 1, SQ);
      if (flags & (LS_2OPT | LS_OROPT))
        len -= local_search<KT, TW, SEG>(I, flags, route, pos, rxy, inq, vis, ord, tl, W, Q, cnt,
                                         tk, init ? -1 : ant, SQ, changes);
    }
  }
  if constexpr (TW > 1 && !SEG) {
    // the whole team runs the local search
    if (w == 0) {
      const bool search = (flags & (LS_2OPT | LS_OROPT)) != 0;
      queue_share(tl, Q);
      if (lane == 0) {
        tl->op = search ? OP_SEARCH : OP_EXIT;
        tl->arg[5] = (int)flags;
      }
      team_sync();
      if (!search) flags = 0;
    }
    if (w > 0 || flags) {
      queue_take(tl, Q);
      flags = (uint32_t)team_arg(tl, 5);
      len -= team_local_search<KT, TW>(I, flags, route, pos, rxy, inq, vis, ord, tl, W, Q, cnt,
                                       tk, init ? -1 : ant, w, changes);
      if (w > 0) return;
    }
  }
  int live = 0;
  if constexpr (SEG) {
    if (uniform_i(SQ.dirty)) seg_materialize<TW>(I, ant, SQ, tl, tk);
    live = uniform_i(SQ.live);
    if (lane == 0) I.sepoch[ant] = SQ.T.epoch;
  }
  if (TW > 1 && SEG) {
    if (lane == 0) tl->op = OP_EXIT;
    team_sync();
  }
  if (init) {
    const int32_t *fr = (live ? I.r2 : I.routes) + (size_t)ant * (size_t)n;
    init_finish(I, mode, fr, len, changes, changes0, listed, more, more, t0, cnt, tk);
  } else {
    if (lane == 0) {
      I.lens[ant] = len;
      I.rsel[ant] = live;
    }
    if (lane < NCNT) {
      I.cnt[(size_t)ant * NCNT + lane] = cnt.v;
      I.cnt_acc[(size_t)ant * NCNT + lane] += cnt.v;
    }
    tk[4] = ticks() - t0;
    if (lane < kTicks) I.ticks[(size_t)ant * kTicks + lane] += tk.v;
  }
}

// One sweep of the initial search over all cities (its tour is ant slot 0's),
// a city per lane in label order: marks the improvable ones by original
// number.  The tour does not change meanwhile, so the whole chip shares it: a
// sweep of 100k cities takes 52 us (launch included) instead of one 8-wave
// workgroup's 5.7 ms.
template <int KT>
__global__ void __launch_bounds__(256) init_sweep_kernel(Inst I) {
  if (I.st->init_done) return;
  const int x = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (x >= I.n) return;
  const uint32_t flags = LS_2OPT | (I.ls_flags & LS_OROPT);
  if (has_improving<KT>(I, flags, x, I.routes, I.pos, I.rxy)) {
    const int o = I.orig_of[x];
    atomicOr(&I.marks[o >> 5], 1u << (o & 31));
  }
}

// One workgroup of TW waves per ant.  4-wave teams on flat arrays are held to 128
// registers (here and in ant_batch_kernel), so that a CU runs four of them; with
// lists of 12/16/24/32, 1000 cities and 1024 ants take 497/442/509/565 us an
// iteration, and 574/510/682/747 without the bound.  It spills 2 to 36 registers
// (most with long lists), which costs where a CU gets no four teams anyhow: 10 000
// cities and 1000 ants (LDS holds three) 756/770/822/917 against 754/752/790/880, a
// batch of 20 of 4000..16 000 cities 603/597/660/752 against 583/571/627/692.
template <int KT, int TW, bool SEG = false>
__global__ void __launch_bounds__(64 * TW, TW == 4 && !SEG ? 4 : 1) ant_kernel(Inst I, int mode) {
  extern __shared__ uint32_t lds[];
  run_ant<KT, TW, SEG>(I, (int)blockIdx.x, mode, lds);
}

// ===================================================================== //
// Batched execution: one launch per phase covers every ant of every instance
// of a batch.  Each instance reads only its own Inst, so it evolves exactly as
// it would alone.
//   insts  Inst [count]
//   amap   int2 [total ants]: (instance, ant) of wave w = block * apb + wave
//          (TW > 1: of block w, whose TW waves form the ant's team)
// ===================================================================== //
template <int KT, int TW>
__global__ void __launch_bounds__(TW > 1 ? 64 * TW : 256, TW == 4 ? 4 : 1)
    ant_batch_kernel(const Inst *insts, const int2 *amap, int total, int apb, int lds_words) {
  extern __shared__ uint32_t lds[];
  if (TW > 1) {
    // one workgroup of TW waves per ant
    const int2 m = amap[blockIdx.x];
    run_ant<KT, TW>(insts[m.x], m.y, 0, lds);
    return;
  }
  const int wave = (int)(threadIdx.x / kWave);
  const int w = (int)blockIdx.x * apb + wave;
  if (w >= total) return;
  const int2 m = amap[w];
  run_ant<KT, 1>(insts[m.x], m.y, 0, lds + (size_t)wave * (size_t)lds_words);
}

// ===================================================================== //
// Persistent batched execution.  One launch runs `iterations` iterations of
// every instance of a batch, and each instance advances on its own: the ants
// of its next iteration become available as soon as its own update is done,
// whatever the other instances are doing.  Per instance (BatchCtl):
//   ticket  ant tasks handed out in this launch (iteration e + 1 of the
//           launch owns tickets e A .. e A + A - 1)
//   done    ants of the current iteration that have finished
//   epoch   iterations completed (update included) in this launch
// Workers (a workgroup of TW waves when TW > 1, else each wave) take an ant
// task by compare-and-swap on a ticket of the current iteration, so no ant
// of iteration e + 2 can start before the update of iteration e + 1 is
// published.  The worker that finishes an instance's last ant runs the
// instance's update (colony, source, pheromone: the same functions as the
// per-phase kernels) and publishes the next epoch.  Workers leave once every
// instance has completed; a worker that sees no ant finish anywhere for
// kStallPolls polls records a stall fault in every unfinished instance and
// leaves, so no wait is unbounded.
// ===================================================================== //
constexpr int kStallPolls = 1 << 21;  // ~7 s of polls without any ant finishing

// An ant task of the current iteration of some instance, largest instances
// first (the host orders the table by tour length, descending).  The whole
// wave scans 64 instances at a time; the lanes of instances with tickets
// left try them in order, one at a time.  Uniform result.
FACO_DEV bool grab_task(BatchCtl *ctl, int count, int iters, int &inst, int &ant) {
  const int lane = lane_id();
  for (int base = 0; base < count; base += kWave) {
    const int i = base + lane;
    int e = 0;
    int64_t A = 0, t = 0;
    bool avail = false;
    if (i < count) {
      e = ld_agent(&ctl[i].epoch);
      if (e < iters) {
        A = ctl[i].ants;
        t = ld_agent64(&ctl[i].ticket);
        avail = t < ((int64_t)e + 1) * A;
      }
    }
    uint64_t m = ballot(avail);
    while (m) {
      const int l = ctz64(m);
      m &= m - 1;
      int won = 0, a = 0;
      if (lane == l) {
        const int64_t lim = ((int64_t)e + 1) * A;
        while (t < lim) {
          const int64_t seen = cas_agent64(&ctl[i].ticket, t, t + 1);
          if (seen == t) {
            won = 1;
            a = (int)(t - (int64_t)e * A);
            break;
          }
          t = seen;
        }
      }
      if (readlane_i(won, l)) {
        inst = base + l;
        ant = readlane_i(a, l);
        return true;
      }
    }
  }
  return false;
}

// After an ant: count it; true for the instance's last ant of the iteration.
// One lane.
FACO_DEV bool finish_ant(BatchCtl *ctl, BatchRun *run, int inst) {
  fence_release_agent();
  const int d = add_agent(&ctl[inst].done, 1) + 1;
  add_agent(&run->progress, 1);
  return d == ctl[inst].ants;
}

// After the update: publish the next epoch.  One lane.
FACO_DEV void publish_epoch(BatchCtl *ctl, BatchRun *run, int inst, int iters) {
  st_agent(&ctl[inst].done, 0);
  fence_release_agent();
  const int e = ld_agent(&ctl[inst].epoch) + 1;
  st_agent(&ctl[inst].epoch, e);
  if (e == iters) add_agent(&run->finished, 1);
}

// The update of one instance by the worker's NT threads (thread tid).
template <int TW>
FACO_DEV void worker_update(const Inst &I, int tid, int nt) {
  if (tid < kWave) run_colony(I);
  if (TW > 1) team_sync(); else wave_fence();
  for (int i = tid; i - lane_id() < I.n; i += nt) run_source(I, i, 0);
  if (TW > 1) team_sync(); else wave_fence();
  const uint32_t slots = (uint32_t)I.n * (uint32_t)I.ks;
  for (uint32_t s = (uint32_t)tid; s < slots; s += (uint32_t)nt) run_pheromone(I, s, 0);
  if (TW > 1) team_sync(); else wave_fence();
}

FACO_DEV void mark_stall(const Inst *insts, BatchCtl *ctl, int count, int iters) {
  for (int i = 0; i < count; ++i)
    if (ld_agent(&ctl[i].epoch) < iters) atomicOr(&insts[i].st->fault, FAULT_BATCH_STALL);
}

template <int KT, int TW>
__global__ void __launch_bounds__(TW > 1 ? 64 * TW : 256)
    ant_persist_kernel(const Inst *insts, BatchCtl *ctl, BatchRun *run, int lds_words) {
  extern __shared__ uint32_t lds[];
  const int count = run->count, iters = run->iterations;
  const int lane = lane_id(), w = (int)(threadIdx.x >> 6);
  int polls = 0, seen = -1;
  if (TW > 1) {
    // the workgroup is one worker; wave 0 takes the tasks
    TeamLds *tl = (TeamLds *)lds;
    for (;;) {
      if (w == 0) {
        int cmd = 2, inst = 0, ant = 0;  // 0 ant, 1 idle, 2 leave, 3 stalled
        if (uniform_i(ld_agent(&run->finished)) < count) {
          if (grab_task(ctl, count, iters, inst, ant)) {
            cmd = 0;
          } else {
            const int pr = uniform_i(ld_agent(&run->progress));
            if (pr != seen) {
              seen = pr;
              polls = 0;
            }
            cmd = ++polls > kStallPolls ? 3 : 1;
          }
        }
        if (lane == 0) {
          tl->disp[0] = cmd;
          tl->disp[1] = inst;
          tl->disp[2] = ant;
        }
      }
      team_sync();
      const int cmd = uniform_i(tl->disp[0]);
      const int inst = uniform_i(tl->disp[1]), ant = uniform_i(tl->disp[2]);
      team_sync();  // every wave has read the task before it is replaced
      if (cmd == 2) break;
      if (cmd == 3) {
        if (w == 0 && lane == 0) mark_stall(insts, ctl, count, iters);
        break;
      }
      if (cmd == 1) {
        __builtin_amdgcn_s_sleep(127);
        continue;
      }
      fence_acquire_agent();
      run_ant<KT, TW>(insts[inst], ant, 0, lds);
      team_sync();
      if (w == 0 && lane == 0) tl->disp[3] = finish_ant(ctl, run, inst) ? 1 : 0;
      team_sync();
      if (uniform_i(tl->disp[3])) {
        fence_acquire_agent();
        worker_update<TW>(insts[inst], (int)threadIdx.x, 64 * TW);
        if (w == 0 && lane == 0) publish_epoch(ctl, run, inst, iters);
      }
    }
  } else {
    // every wave is a worker with its own slice of LDS
    uint32_t *mine = lds + (size_t)w * (size_t)lds_words;
    for (;;) {
      int cmd = 2, inst = 0, ant = 0;  // 0 ant, 1 idle, 2 leave, 3 stalled
      if (uniform_i(ld_agent(&run->finished)) < count) {
        if (grab_task(ctl, count, iters, inst, ant)) {
          cmd = 0;
        } else {
          const int pr = uniform_i(ld_agent(&run->progress));
          if (pr != seen) {
            seen = pr;
            polls = 0;
          }
          cmd = ++polls > kStallPolls ? 3 : 1;
        }
      }
      cmd = uniform_i(cmd);
      inst = uniform_i(inst);
      ant = uniform_i(ant);
      if (cmd == 2) break;
      if (cmd == 3) {
        if (lane == 0) mark_stall(insts, ctl, count, iters);
        break;
      }
      if (cmd == 1) {
        __builtin_amdgcn_s_sleep(127);
        continue;
      }
      fence_acquire_agent();
      run_ant<KT, 1>(insts[inst], ant, 0, mine);
      int last = 0;
      if (lane == 0) last = finish_ant(ctl, run, inst) ? 1 : 0;
      if (readlane_i(last, 0)) {
        fence_acquire_agent();
        worker_update<1>(insts[inst], lane, kWave);
        if (lane == 0) publish_epoch(ctl, run, inst, iters);
      }
    }
  }
}

}  // namespace faco
