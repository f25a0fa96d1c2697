// faco_team_ls.hpp -- the local search of an ant whose team has several waves,
// on flat arrays (included by faco_kernels.hpp after the array rewrites).
//
// Every wave of the team runs the same loop on the same (wave-uniform) state
// and no wave waits for commands: a round takes the next TW listed cities,
// wave w evaluates the w-th one (2-opt and every Or-opt variant at once) and
// leaves its best move in LDS; after one barrier every wave sees all TW
// moves, takes the first city with one (the ones before it are popped without
// a move, the ones after it stay listed: the order of one city at a time),
// rewrites its share of the arrays, and a second barrier ends the round.
// Wave 0 meanwhile pushes the move's cities.
//
// What bounds a round is its chain: two dependent levels of loads (positions,
// then tour neighbours; 64 ants' arrays are 100 MB at 100k cities, so they
// mostly miss L2), its instructions, one every four cycles, and the barriers.  A leader
// that evaluated four cities and handed the Or-opt variants to helper waves
// through LDS paid two more barriers and 14 words a lane for the hand-over.
// Measured on the 100k workload (64 ants, iterations 100..200): 649 rounds of 8
// cities an ant at 1.84 us instead of 797 of 4 at 2.04, a move 2.1 us instead
// of 3.0; the ant kernel 7.1 ms instead of 9.6.
#pragma once

// Move record of a wave (9 int4):
//   [0] gain (0: none), code, b, bn   [1] pb, pbn, pa, a
//   [2 + j] city and coordinates at tour position pa - 3 + j (j = 0..6)
// code: 0/1 2-opt through (a, succ a)/(pred a, a); 2 + 2 slot + side: Or-opt
// (slots of or_slot_lanes).  bn: succ b (2-opt code 0, Or-opt side 0) or
// pred b; pb, pbn, pa: positions of b, bn, a.

// The loads of a wave's next city that never change along a local search.
struct TeamPre {
  int a;
  int b, d;
};
template <int GS>
FACO_DEV TeamPre team_pre(const Inst &I, int a) {
  const int s = lane_id() & (GS - 1);
  TeamPre P;
  P.a = a;
  P.b = a;
  P.d = 0;
  if (s < I.k) {
    P.b = at(I.cl + (size_t)a * (size_t)I.k, s);
    P.d = at(I.cl_d + (size_t)a * (size_t)I.k, s);
  }
  return P;
}

// What a lane evaluates, fixed along a local search.  lane = (part, candidate
// slot s), part p of 64 / GS: even parts try the moves through (b, succ b),
// odd parts those through (pred b, b).  With four parts (lists of up to 16)
// the first pair of parts tries the 2-opt move and Or-opt slots 0, 1 and the
// second slots 2, 3, 4; with two parts every lane tries all six.
// A variant's segment is a range of tour positions pa - 3 + j; its mask holds
// those j as bits (all bits: the lane does not try the variant).
struct TeamLane {
  int su, sv;            // ends (j) of this lane's neighbourhood cost
  int ja, jb, jc;        // j of the end of the variants' second new edge
  uint32_t ma, mb, mc;
  int step;              // 1: b's neighbour is succ b; -1: pred b
  int m2nd, mrem;        // all ones: second pair of parts; removed edge (pred a, a)
};
// m ? x : y for an all-ones or zero mask in a vector register
FACO_DEV int pick(int m, int x, int y) { return (m & x) | (~m & y); }
constexpr uint32_t kSegMask[kOrSlots] = {0x08u, 0x18u, 0x38u, 0x0Cu, 0x0Eu};
constexpr int kTwoBit = 1 << 30;  // above every Or-opt gain: 2-opt goes first

template <int GS>
FACO_DEV TeamLane team_lane(const Inst &I, uint32_t flags) {
  const int lane = lane_id();
  const int side = (lane / GS) & 1;
  const bool second = lane / GS >= 2;
  const int r = lane & 15;
  TeamLane T;
  // costs 0..5: tour edges (j, j + 1); 6..10: (6, 2), (2, 5), (2, 4), (1, 4),
  // (0, 4), the edges that close the gap of a removed segment
  T.su = r <= 6 ? r : (r <= 8 ? 2 : (r == 9 ? 1 : (r == 10 ? 0 : 3)));
  T.sv = r <= 5 ? r + 1 : (r == 6 ? 2 : (r == 7 ? 5 : (r <= 10 ? 4 : 3)));
  const int two = side ? 2 : 4;
  T.ja = second ? 5 : two;
  T.jb = second ? 2 : 3;
  T.jc = second ? 1 : 4;
  const int lmax = (flags & LS_OROPT) ? or_lmax(I) : 0;
  const bool act = (lane & (GS - 1)) < I.k;
  const uint32_t none = 0xFFFFFFFFu;
  T.ma = second ? (lmax >= 3 ? kSegMask[2] : none) : ((flags & LS_2OPT) ? 0u : none);
  T.mb = second ? (lmax >= 2 ? kSegMask[3] : none) : (lmax >= 1 ? kSegMask[0] : none);
  T.mc = second ? (lmax >= 3 ? kSegMask[4] : none) : (lmax >= 2 ? kSegMask[1] : none);
  T.step = side ? -1 : 1;
  T.m2nd = second ? -1 : 0;
  T.mrem = second || side ? -1 : 0;
  T.ma = act ? T.ma : none;
  T.mb = act ? T.mb : none;
  T.mc = act ? T.mc : none;
  return T;
}

// Evaluate city a with the whole wave.  The result is the best move in the
// order of the sequential evaluation: 2-opt first (loop 1 over the list, then
// loop 2), else Or-opt by gain, then slot, list position, succ before pred.
// Leaves the move in desc and returns its gain (0: none; uniform).
template <int GS>
FACO_DEV int team_eval(const Inst &I, const TeamLane &T, const TeamPre &P,
                        const int32_t *route, const int32_t *pos, const int2 *rxy, int *desc) {
  const int n = I.n;
  // opaque: masks of lanes are compared afresh instead of kept (and spilled)
  // in scalar register pairs across the whole kernel
  int lane = lane_id();
  asm volatile("" : "+v"(lane));
  const int s = lane & (GS - 1), side = (lane / GS) & 1;
  const int a = P.a, b = P.b, d_ab = P.d;
  // level 1
  const int pb = at(pos, b);
  const int2 xb = at(I.xy, b);
  const int pa = uniform_i(at(pos, a));
  // level 2: a's neighbourhood and b's neighbour
  const int32_t *rb = route + (pa - 3);
  const int2 *xr = rxy + (pa - 3);
  uint32_t ou = 8u * (uint32_t)T.su, ov = 8u * (uint32_t)T.sv;
  uint32_t oa = 8u * (uint32_t)T.ja, ob = 8u * (uint32_t)T.jb, oc = 8u * (uint32_t)T.jc;
  int pbn = pb + T.step;
  pbn = pbn == n ? 0 : pbn;
  pbn = (int)min((uint32_t)pbn, (uint32_t)(n - 1));  // -1: the last position
  // which of the positions pa - 3 + j hold b and bn (rj, rn; others: any
  // value outside 0..6, kept apart by the shift's 31)
  int rj = pb - pa + 3, rn = rj + T.step;
  uint32_t wrap_bits = 0u;
  if (pa < 8 || pa + 8 >= n) {
    rb = route;
    xr = rxy;
    ou = 8u * (uint32_t)wrapc(pa - 3 + T.su, n);
    ov = 8u * (uint32_t)wrapc(pa - 3 + T.sv, n);
    oa = 8u * (uint32_t)wrapc(pa - 3 + T.ja, n);
    ob = 8u * (uint32_t)wrapc(pa - 3 + T.jb, n);
    oc = 8u * (uint32_t)wrapc(pa - 3 + T.jc, n);
    rj = wrapc(rj, n);
    rn = wrapc(rj + T.step, n);
    if (n < 7)  // a tour shorter than the neighbourhood
      wrap_bits = (1u << (rj + n)) | (1u << (rn + n));
  }
  const int2 xbn = at(rxy, pbn);
  const int2 U = at_byte(xr, ou), V = at_byte(xr, ov);
  const int2 xA = at_byte(xr, oa), xB = at_byte(xr, ob), xC = at_byte(xr, oc);
  const int bn = at(route, pbn);
  const int nb = at_byte(rb, ou >> 1);
  const uint32_t M = (1u << min((uint32_t)rj, 31u)) | (1u << min((uint32_t)rn, 31u)) | wrap_bits;
  const int uc = cost_ne(U, V);
  const int in = cost_ne(xb, xbn) - d_ab;  // edge freed at b minus the new edge (a, b)
  int u[11];
#pragma unroll
  for (int j = 0; j < 11; ++j) u[j] = row_bcast(uc, j);
  int g2, go, vo;
  if (GS == 16) {
    const int cA = cost_ne(xA, xbn), cB = cost_ne(xB, xbn), cC = cost_ne(xC, xbn);
    // removal gains; the removed edge at a: pred a for the forward slots and
    // the 2-opt move through pred b, succ a otherwise
    const int m = T.m2nd;
    const int remA = pick(T.mrem, u[2], u[3]), remB = pick(m, u[3], u[2]);
    int gA = pick(m, u[2] + u[5] - u[6], remA) + in - cA;
    int gB = pick(m, u[1] - u[9], u[2] - u[8]) + u[3] + in - cB;
    int gC = pick(m, u[3] + u[0] - u[10], u[2] + u[4] - u[7]) + in - cC;
    gA = ((M & T.ma) == 0u && d_ab < remA) ? gA : 0;
    gB = ((M & T.mb) == 0u && d_ab < remB) ? gB : 0;
    gC = ((M & T.mc) == 0u && d_ab < remB) ? gC : 0;
    g2 = gA & ~m;
    go = gA & m;
    vo = m & 2;
    vo = gB > go ? (m & 3) : vo;
    go = gB > go ? gB : go;
    vo = gC > go ? 1 + (m & 3) : vo;
    go = gC > go ? gC : go;
  } else {
    // ma, mb, mc hold the masks of the 2-opt move and slots 0, 1: the others
    // follow from the same limits
    const int remA = side ? u[2] : u[3];
    g2 = remA + in - cost_ne(xA, xbn);
    g2 = ((M & T.ma) == 0u && d_ab < remA) ? g2 : 0;
    const int lmax = T.mc != 0xFFFFFFFFu ? (or_lmax(I) >= 3 ? 3 : 2) : (T.mb != 0xFFFFFFFFu ? 1 : 0);
    const int su[5] = {u[2] + u[3] - u[8], u[2] + u[4] - u[7], u[2] + u[5] - u[6],
                       u[3] + u[1] - u[9], u[3] + u[0] - u[10]};
    const int je[5] = {3, 4, 5, 2, 1};
    go = 0;
    vo = 0;
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      const int2 xo = make_int2(row_bcast(U.x, je[v]), row_bcast(U.y, je[v]));
      const int L = v < 3 ? v + 1 : v - 1;
      const int g = su[v] + in - cost_ne(xo, xbn);
      const bool ok = L <= lmax && (M & kSegMask[v]) == 0u && d_ab < (v < 3 ? u[2] : u[3]) && g > go;
      vo = ok ? v : vo;
      go = ok ? g : go;
    }
  }
  const int key = g2 > 0 ? g2 + kTwoBit : go;
  const int best = wave_max_i32(key);
  uint64_t m = ballot(key == best);  // 2-opt: lane order is the order of the two loops
  const bool two = best >= kTwoBit;
  if (!two && best > 0 && (m & (m - 1))) {
    const int idx = key == best ? (vo * I.k + s) * 2 + side : 0x7fffffff;
    const int low = wave_min_i32(idx);
    m = ballot(idx == low);
  }
  int4 *d4 = reinterpret_cast<int4 *>(desc);
  if (lane == ctz64(m)) {
    d4[0] = make_int4(two ? best - kTwoBit : best, two ? side : 2 + 2 * vo + side, b, bn);
    d4[1] = make_int4(pb, pbn, pa, a);
  }
  if (lane < 7) d4[2 + lane] = make_int4(nb, U.x, U.y, 0);
  return best;
}

// The 3-opt trial of the initial search, by the whole wave, for a city a
// without 2-opt or Or-opt move: remove (t1, t2), (t3, t4), (t5, t6), add (t2,
// t3), (t4, t5), (t6, t1), with t1 = a, t2 its neighbour in direction dir, t3 =
// slot s of t2's list, t5 = slot r of t4's list, all positive partial gains, t5
// on the path t2 .. t3 before t3.  Variant (dir K + s) K + r; best gain, first
// variant.  Lane: a pair (dir, s) and every second r, eight r at a time, so
// the four levels of dependent loads are taken by all variants together (a
// loop over single variants per lane took them eight times over).
// Record: [0] gain, code kThreeOpt + dir   [1] position of t2, offsets of t3
// and t5 from it, a   [2 + j] t_(j+1).  Returns the gain (0: none; uniform).
constexpr int kThreeOpt = 32;
FACO_DEV int team_eval3(const Inst &I, int a, const int32_t *route, const int32_t *pos,
                        const int2 *rxy, int *desc) {
  constexpr int RB = 8;
  const int n = I.n, K = I.k, lane = lane_id();
  const int pa = uniform_i(at(pos, a));
  const int2 xa = at(rxy, pa);
  int best = 0, bc = 0, bdir = 0, bp2 = 0, bo3 = 0, bo5 = 0;
  int b2 = 0, b3 = 0, b4 = 0, b5 = 0, b6 = 0;
  for (int q0 = 0; q0 < 2 * K; q0 += kWave / 2) {
    const int q = q0 + (lane >> 1), qc = q < 2 * K ? q : 0;
    const int dir = qc >= K ? 1 : 0, s = qc - dir * K, fwd = dir ? -1 : 1;
    const int p2 = wrapc(pa + fwd, n);
    const int t2 = at(route, p2);
    const int t3 = at(I.cl, t2 * K + s);
    int g1 = cost(xa, at(rxy, p2)) - at(I.cl_d, t2 * K + s);
    const int p3 = at(pos, t3), p4 = wrapc(p3 + fwd, n);
    const int t4 = at(route, p4);
    const bool ok = q < 2 * K && g1 > 0 && t3 != a && t4 != a;
    g1 += cost(at(rxy, p3), at(rxy, p4));
    const int off3 = wrapc(dir ? p2 - p3 : p3 - p2, n);
    for (int r0 = 0; r0 < K; r0 += 2 * RB) {
      int t5[RB], g2[RB];
#pragma unroll
      for (int i = 0; i < RB; ++i) {
        const int r = r0 + 2 * i + (lane & 1);
        const bool in = ok && r < K;
        t5[i] = in ? at(I.cl, t4 * K + r) : a;
        g2[i] = in ? g1 - at(I.cl_d, t4 * K + r) : 0;
      }
      int p5[RB];
#pragma unroll
      for (int i = 0; i < RB; ++i) p5[i] = at(pos, t5[i]);
      int t6[RB];
      int2 x5[RB], x6[RB];
#pragma unroll
      for (int i = 0; i < RB; ++i) {
        const int p6 = wrapc(p5[i] + fwd, n);
        t6[i] = at(route, p6);
        x5[i] = at(rxy, p5[i]);
        x6[i] = at(rxy, p6);
      }
#pragma unroll
      for (int i = 0; i < RB; ++i) {
        const int off5 = wrapc(dir ? p2 - p5[i] : p5[i] - p2, n);
        const int g = g2[i] + cost(x5[i], x6[i]) - cost(x6[i], xa);
        if (g2[i] > 0 && off5 < off3 && g > best) {
          best = g;
          bc = q * K + r0 + 2 * i + (lane & 1);
          bdir = dir;
          bp2 = p2;
          bo3 = off3;
          bo5 = off5;
          b2 = t2;
          b3 = t3;
          b4 = t4;
          b5 = t5[i];
          b6 = t6[i];
        }
      }
    }
  }
  const int top = wave_max_i32(best);
  if (top == 0) return 0;
  const int first = wave_min_i32(best == top ? bc : 0x7fffffff);
  if (best == top && bc == first) {
    int4 *d4 = reinterpret_cast<int4 *>(desc);
    d4[0] = make_int4(top, kThreeOpt + bdir, 0, 0);
    d4[1] = make_int4(bp2, bo3, bo5, a);
    d4[2].x = a;
    d4[3].x = b2;
    d4[4].x = b3;
    d4[5].x = b4;
    d4[6].x = b5;
    d4[7].x = b6;
  }
  return top;
}

// This wave's share of a reversal (see reverse_part): few chunks take the
// variant with few in flight.  Chunks start at wave 1: wave 0 has the pushes.
template <int TW>
FACO_DEV void team_reverse_share(int n, int s, int L, int w, int32_t *route, int32_t *pos,
                                 int2 *rxy) {
  const int half = L >> 1;
  const int ww = w == 0 ? TW - 1 : w - 1;
  if (half <= TW * kWave)
    reverse_part<TW, 1>(n, s, L, ww, route, pos, rxy);
  else if (half <= 4 * TW * kWave)
    reverse_part<TW, 4>(n, s, L, ww, route, pos, rxy);
  else
    reverse_part<TW>(n, s, L, ww, route, pos, rxy);
}

// A block move by the team, or by wave 1 alone while it holds the whole block
// in registers (no barrier between its reads and writes needed).
constexpr int kSoloShift = 2 * kWave;
template <int TW>
FACO_DEV void team_shift_share(int n, int src, int dst, int D, bool down, int w, int32_t *route,
                               int32_t *pos, int2 *rxy) {
  if (D <= kSoloShift) {
    if (w == 1) shift_part<1, kSoloShift / kWave>(n, src, dst, D, down, 0, route, pos, rxy);
    return;
  }
  const int ww = w == 0 ? TW - 1 : w - 1;
  if (D <= TW * kWave)
    shift_part<TW, 1>(n, src, dst, D, down, ww, route, pos, rxy);
  else if (D <= 4 * TW * kWave)
    shift_part<TW, 4>(n, src, dst, D, down, ww, route, pos, rxy);
  else
    shift_part<TW>(n, src, dst, D, down, ww, route, pos, rxy);
}

// The queue's state from wave 0 to the other waves (a barrier between).
FACO_DEV void queue_share(TeamLds *tl, const Queue &Q) {
  if (lane_id() == 0) {
    tl->arg[0] = Q.head;
    tl->arg[1] = Q.tail;
    tl->arg[2] = Q.count;
    tl->arg[3] = Q.cap;
    tl->arg[4] = Q.in_lds;
  }
}
FACO_DEV void queue_take(const TeamLds *tl, Queue &Q) {
  Q.head = team_arg(tl, 0);
  Q.tail = team_arg(tl, 1);
  Q.count = team_arg(tl, 2);
  Q.cap = team_arg(tl, 3);
  Q.in_lds = team_arg(tl, 4);
}

// Cities per wave up to which a sweep evaluates them one after the other, each
// by a whole wave (0.7 us a city), instead of 64 at once, a lane each (10 to 13
// us a step, up to four dependent chunks of candidates).  Sweeps of the slowest
// ant per iteration, in us: 35 cities (200-city tours) 7.2 against 24.8, 123
// (1000) 31 against 36.  Thresholds 8/16/32/64 give iterations of 1000 cities
// in 257/248/246/246 us and of 5000 in 582/581/581/591.
constexpr int kWaveSweep = 32;

// Sweep by all waves (see sweep()): the touched cities are gathered into a
// list in LDS (the queue's ring, empty during a sweep; all of them at once
// when they fit, else a range of bitmap words at a time), every wave tests 64
// of them per step with no barrier between steps, and wave 0 lists the
// improvable ones.  Returns the number listed; Q is updated in every wave.
template <int KT, int TW>
FACO_DEV int team_sweep(const Inst &I, uint32_t flags, int W, Queue &Q, const FlatT &T,
                        uint32_t *inq, uint32_t *touched, uint32_t *ord, TeamLds *tl, int w,
                        const TeamLane &tlane, LaneCounters &tk) {
  constexpr int GS = KT <= 16 ? 16 : 32;
  const int lane = lane_id(), tid = w * kWave + lane;
  constexpr int NT = TW * kWave;
  const int64_t t0 = ticks();
  // a small ring (a configured capacity) is replaced by the team's city list
  const bool ring = I.lcap >= 4 * NT;
  int32_t *list = ring ? Q.lr : tl->cities;
  const int cap = ring ? I.lcap : NT;
  int own = 0;
  for (int wi = tid; wi < W; wi += NT) own += __builtin_popcount(touched[wi]);
  own = wave_sum_i32(own);
  if (lane == 0) {
    tl->f[w] = own;
    if (w == 0) tl->ls.cnt[0] = 0;
  }
  team_sync();
  const int total = uniform_i(wave_sum_i32(lane < TW ? tl->f[lane] : 0));
  const int step = total <= cap ? W : cap / 32;
  int p = 0;
  for (int w0 = 0; w0 < W; w0 += step, p ^= 1) {
    const int w1 = w0 + step < W ? w0 + step : W;
    if (w == 0 && lane == 0) tl->ls.cnt[p ^ 1] = 0;
    for (int g = w0 + w * kWave; g < w1; g += NT) {
      uint32_t word = g + lane < w1 ? touched[g + lane] : 0u;
      const int c = wave_sum_i32(__builtin_popcount(word));
      if (c == 0) continue;
      int at = 0;
      if (lane == 0) at = atomicAdd(&tl->ls.cnt[p], c);
      at = uniform_i(at);
      for (;;) {
        const uint64_t m = ballot(word != 0u);
        if (!m) break;
        const int r = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        if (word != 0u) {
          list[at + r] = (g + lane) * 32 + __builtin_ctz(word);
          word &= word - 1u;
        }
        at += __builtin_popcountll(m);
      }
    }
    team_sync();
    const int cnt = uniform_i(tl->ls.cnt[p]);
    if (cnt <= kWaveSweep * TW) {
      int x = w < cnt ? uniform_i(list[w]) : 0;
      TeamPre P = team_pre<GS>(I, x);
      for (int i = w; i < cnt; i += TW) {
        const int xn = i + TW < cnt ? uniform_i(list[i + TW]) : x;
        const TeamPre Pn = team_pre<GS>(I, xn);
        const int ox = I.orig_of[x];
        if (team_eval<GS>(I, tlane, P, T.route, T.pos, T.rxy, tl->ls.desc[0] + w * kDescWords) > 0 &&
            lane == 0)
          bit_set(ord, ox);
        x = xn;
        P = Pn;
      }
    } else {
      for (int i0 = w * kWave; i0 < cnt; i0 += NT) {
        const int i = i0 + lane;
        if (i < cnt) {
          const int x = list[i];
          const int ox = I.orig_of[x];
          if (has_improving<KT>(I, flags, x, T)) bit_set(ord, ox);
        }
      }
    }
    team_sync();
  }
  if (w == 0) {
    tk[TK_SWEEP_CITIES] += total;
    tk[TK_SWEEP_TESTS] += ticks() - t0;
  }
  int marks = 0;
  for (int wi = tid; wi < W; wi += NT) marks += __builtin_popcount(ord[wi]);
  marks = wave_sum_i32(marks);
  if (lane == 0) tl->f[w] = marks;
  team_sync();
  const int listed = uniform_i(wave_sum_i32(lane < TW ? tl->f[lane] : 0));
  if (listed > 0) {
    if (w == 0) {
      const int64_t tl0 = ticks();
      list_marked(I, W, Q, inq, touched, ord);
      queue_share(tl, Q);
      tk[TK_SWEEP_LIST] += ticks() - tl0;
    }
    team_sync();
    queue_take(tl, Q);
  }
  return listed;
}

// The local search (Alg. 3 + Or-opt + sweeps), called by every wave w of the
// team with the same arguments; cnt, tk and the return value (the gain) are
// wave 0's.  changes: moves made before (in) and by the end (out).  OPT3: the
// initial search with 3-opt (no sweeps of its own).
template <int KT, int TW, bool OPT3 = false>
FACO_DEV int64_t team_local_search(const Inst &I, uint32_t flags, int32_t *route, int32_t *pos,
                                   int2 *rxy, uint32_t *inq, uint32_t *touched, uint32_t *ord,
                                   TeamLds *tl, int W, Queue Q, LaneCounters &cnt,
                                   LaneCounters &tk, int ant, int w, int &changes) {
  constexpr int GS = KT <= 16 ? 16 : 32;
  const int n = I.n, lane = lane_id();
  flags = (uint32_t)uniform_i((int)flags);
  const int changes0 = changes;
  int changes_at_sweep = -1, par = 0;
  int pops = 0, m2 = 0, m3 = 0, sweeps = 0, rounds = 0;
  int64_t gain = 0, moved = 0, t_eval = 0, t_apply = 0, t_sweep = 0;
  const TeamLane tlane = team_lane<GS>(I, flags);
  TeamPre pre;
  int pre_a = -1;
  pre.a = pre.b = pre.d = 0;
  int64_t t0 = w == 0 ? ticks() : 0;
  for (;;) {
    for (;;) {
      Q.count = uniform_i(Q.count);
      Q.head = uniform_i(Q.head);
      Q.tail = uniform_i(Q.tail);
      Q.cap = uniform_i(Q.cap);
      Q.in_lds = uniform_i(Q.in_lds);
      changes = uniform_i(changes);
      if (!(Q.count > 0 && changes < n)) break;
      const int gcount = Q.count < TW ? Q.count : TW;
      int *desc = tl->ls.desc[par];
      par ^= 1;
      if (w < gcount) {
        pre_a = uniform_i(pre_a);
        if (pre_a < 0) {
          int h = Q.head + w;
          h = h >= Q.cap ? h - Q.cap : h;
          int a = Q.lr[Q.in_lds ? h : 0];
          if (!Q.in_lds) a = Q.gr[h];
          pre_a = uniform_i(a);
          pre = team_pre<GS>(I, pre_a);
        }
        pre.a = pre_a;
        const int found = team_eval<GS>(I, tlane, pre, route, pos, rxy, desc + w * kDescWords);
        if (OPT3 && found == 0) team_eval3(I, pre.a, route, pos, rxy, desc + w * kDescWords);
      }
      team_sync();
      // lanes 2 v and 2 v + 1 hold the head of wave v's record
      // (the records of waves without a city are old ones)
      const int vl = lane & (2 * TW - 1);
      const int4 v = reinterpret_cast<const int4 *>(desc)[(vl >> 1) * (kDescWords / 4) + (vl & 1)];
      const uint64_t hm = ballot(v.x > 0) & 0x5555u & ((1u << (2 * gcount)) - 1u);
      const int j = uniform_i(hm ? ctz64(hm) >> 1 : gcount);
      const int npop = j < gcount ? j + 1 : gcount;
      // wave 0 unlists the popped cities
      if (w == 0 && (lane & 1) == 1 && (lane >> 1) < npop) bit_clear(inq, v.w);
      Q.head = Q.head + npop >= Q.cap ? Q.head + npop - Q.cap : Q.head + npop;
      Q.count -= npop;
      pops += npop;
      ++rounds;
      // the next round's city of this wave, if it is listed already (the
      // move's cities go to the tail)
      pre_a = -1;
      if (w < Q.count) {
        int h = Q.head + w;
        h = h >= Q.cap ? h - Q.cap : h;
        int a = Q.lr[Q.in_lds ? h : 0];
        if (!Q.in_lds) a = Q.gr[h];
        pre_a = uniform_i(a);
        pre = team_pre<GS>(I, pre_a);
      }
      if (w == 0) {
        const int64_t t1 = fine_ticks();
        t_eval += t1 - t0;
        t0 = t1;
      }
      if (j >= gcount) continue;
      const int jb = 2 * j;
      const int code = readlane_i(v.y, jb);
      const int g = readlane_i(v.x, jb);
      const int pb = readlane_i(v.x, jb + 1), pbn = readlane_i(v.y, jb + 1);
      const int pa = readlane_i(v.z, jb + 1);
      const int *rec = desc + j * kDescWords;
      const bool two = code < 2, three = OPT3 && code >= kThreeOpt;
      const int side = code & 1, slot = (code - 2) >> 1;
      int dir, L, lf, ll, lp, lq;
      or_slot_lanes(slot, dir, L, lf, ll, lp, lq);
      if (w == 0) {
        // cities to list, in order: 2-opt (w, x, y, z), Or-opt (p, q, b, e,
        // first, last); words of the record
        int k;
        if (two) {
          // side 0: a, succ a, b, succ b; side 1: pred a, a, pred b, b
          k = lane == 0 ? (side ? 8 + 4 * 2 : 8 + 4 * 3)
                        : (lane == 1 ? (side ? 8 + 4 * 3 : 8 + 4 * 4)
                                     : ((lane == 2) == (side == 0) ? 2 : 3));
        } else {
          // 3-opt: t1 .. t6
          const int jn = three ? lane
                               : (lane == 0 ? lp : (lane == 1 ? lq : (lane == 4 ? lf : ll)));
          k = !three && (lane == 2 || lane == 3) ? lane : 8 + 4 * jn;
        }
        const int np = two ? 4 : 6;
        const int x = rec[lane < np ? k : 0];
        bool take = lane < np && !bit_get(inq, lane < np ? x : 0);
        // the ends of a 2-opt move are four cities; an Or-opt move's may repeat
        if (!two) {
#pragma unroll
          for (int i = 0; i < 5; ++i) {
            const int xi = readlane_i(x, i);
            if (i < lane && xi == x) take = false;
          }
        }
        const uint64_t pm = ballot(take);
        const int cntp = __builtin_popcountll(pm);
        const int spill = Q.in_lds && Q.count + cntp > Q.cap ? 1 : 0;
        if (spill) q_spill(Q, n);
        if (take) {
          int t = Q.tail + __builtin_popcountll(pm & ((1ull << lane) - 1ull));
          t = t >= Q.cap ? t - Q.cap : t;
          bit_set(inq, x);
          bit_set(touched, x);
          (Q.in_lds ? Q.lr : Q.gr)[t] = x;
        }
        if (lane == 0) tl->ls.pushed = cntp | (spill << 8);
      }
      int mv;
      if (two) {
        // flip x..y, x = succ a or a, y = b or pred b, or the complement from
        // z = succ b or b: the shorter
        const int px = side ? pa : (pa + 1 == n ? 0 : pa + 1);
        const int py = side ? pbn : pb, pz = side ? pb : pbn;
        const int L1 = wrapc(py - px, n) + 1;
        const bool first = 2 * L1 <= n;
        mv = first ? L1 : n - L1;
        team_reverse_share<TW>(n, uniform_i(first ? px : pz), uniform_i(mv), w, route, pos, rxy);
        ++m2;
      } else if (three) {
        // the blocks t2 .. t5 and t6 .. t3 (in direction dir) exchange places:
        // the whole range reversed, then each block
        const int p2 = pb, off3 = pbn, off5 = pa;
        const int s0 = side ? wrapc(p2 - off3, n) : p2;
        const int L1 = side ? off3 - off5 : off5 + 1, L2 = side ? off5 + 1 : off3 - off5;
        mv = L1 + L2;
        team_reverse_share<TW>(n, uniform_i(s0), uniform_i(mv), w, route, pos, rxy);
        team_sync();
        team_reverse_share<TW>(n, uniform_i(s0), uniform_i(L2), w, route, pos, rxy);
        team_reverse_share<TW>(n, uniform_i(wrapc(s0 + L2, n)), uniform_i(L1), w, route, pos, rxy);
        ++m3;
      } else {
        // the segment and the shorter block between its old place and the
        // insertion edge (x1, x2) exchange places
        const int fpos = dir == 0 ? pa : wrapc(pa - L + 1, n);
        const int pq = wrapc(fpos + L, n), pp = fpos == 0 ? n - 1 : fpos - 1;
        const int px1 = side ? pbn : pb, px2 = side ? pb : pbn;
        const int D1 = wrapc(px1 - pq, n) + 1, D2 = wrapc(pp - px2, n) + 1;
        const bool down = D1 <= D2;
        const int D = uniform_i(down ? D1 : D2);
        const int src = uniform_i(down ? pq : px2);
        const int dst = uniform_i(down ? fpos : wrapc(px2 + L, n));
        // the segment in its inserted orientation
        const bool rev = (dir == 1) != (side == 1);
        const int i = lane < L ? lane : 0;
        const int ei = lf + (rev ? L - 1 - i : i);
        const int4 ins = reinterpret_cast<const int4 *>(rec)[2 + ei];
        team_shift_share<TW>(n, src, dst, D, down, w, route, pos, rxy);
        if (w == 1 && lane < L) {
          const int d = wrapc((down ? wrapc(fpos + D1, n) : px2) + lane, n);
          at(route, d) = ins.x;
          at(rxy, d) = make_int2(ins.y, ins.z);
          at(pos, ins.x) = d;
        }
        mv = D + L;
      }
      ++changes;
      gain += g;
      moved += mv;
      team_sync();
      const int pushed = uniform_i(tl->ls.pushed);
      const int np = pushed & 255;
      if (w == 0) {
        const int64_t t1 = fine_ticks();
        t_apply += t1 - t0;
        t0 = t1;
      } else if (pushed >> 8) {  // wave 0's queue moved to the global ring
        Q.head = 0;
        Q.tail = Q.count == n ? 0 : Q.count;
        Q.cap = n;
        Q.in_lds = 0;
      }
      Q.tail = Q.tail + np >= Q.cap ? Q.tail + np - Q.cap : Q.tail + np;
      Q.count += np;
    }
    changes = uniform_i(changes);
    if (OPT3 || !(flags & LS_SWEEP) || changes >= n) break;
    // Every city a sweep lists has an improving move, so a sweep that was
    // followed by no change can only come from the two move tests
    // disagreeing: stop instead of spinning, and report it.
    if (changes == changes_at_sweep) {
      if (w == 0) record_fault(I, FAULT_LS_STALL, ant);
      break;
    }
    changes_at_sweep = changes;
    ++sweeps;
    const int pushed = uniform_i(team_sweep<KT, TW>(I, flags, W, Q, FlatT{route, pos, rxy}, inq,
                                                    touched, ord, tl, w, tlane, tk));
    pre_a = -1;
    if (w == 0) {
      const int64_t t1 = ticks();
      t_sweep += t1 - t0;
      t0 = t1;
    }
    if (pushed == 0) break;
  }
  if (w == 0) {
    cnt[CNT_LS_POPS] += pops;
    cnt[CNT_MOVES_2OPT] += m2;
    cnt[CNT_MOVES_OROPT] += changes - changes0 - m2 - m3;
    if (OPT3) cnt[CNT_MOVES_3OPT] += m3;
    cnt[CNT_MOVED_ELEMS] += moved;
    cnt[CNT_SWEEPS] += sweeps;
    cnt[CNT_LS_GAIN] += gain;
    tk[1] += t_eval;
    tk[2] += t_apply;
    tk[3] += t_sweep;
    tk[12] += rounds;
    tk[14] += (flags & LS_OROPT) ? rounds : 0;
    tk[15] += t_apply;
  }
  return gain;
}
