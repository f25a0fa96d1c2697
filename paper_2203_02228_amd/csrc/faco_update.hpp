// faco_update.hpp -- the per-instance update after the ants (colony: iteration
// best, global best + limits, source choice; source materialisation; Eq. (2)
// pheromone update) as device functions: run_update for the update launch (lone
// and batched), run_colony, run_source and run_pheromone for the persistent batched
// kernel, the last two also for the state before the first iteration.
#pragma once
#include "device_common.hpp"
#include "faco_device.hpp"

namespace faco {

// ===================================================================== //
// Colony update (after the ants): iteration best, global best + limits
// (Sec. 4.5), source choice.  One wave.
// ===================================================================== //
FACO_DEV void limits(const Inst &I, int64_t gb_len, float &tmin_f, float &tmax_f) {
  const double tmax = 1.0 / ((double)gb_len * (1.0 - (double)I.rho));
  const double num = 1.0 - I.p_root;
  const double den = (double)(I.k - 1) * I.p_root;
  double tmin = tmax * num / den;
  if (tmin > tmax) tmin = tmax;
  tmax_f = (float)tmax;
  tmin_f = (float)tmin;
}

// What the colony decides after an iteration's ants (uniform).
struct Colony {
  int64_t iter, gb_len, src_len;
  float tmin, tmax, delta;
  int ib;
  bool improved, use_gb;
};

FACO_DEV Colony colony_decide(const Inst &I) {
  const int lane = lane_id();
  const DevState *st = I.st;
  Colony C;
  const uint64_t t = (uint64_t)st->iter + 1;
  int64_t bl = INT64_MAX;
  int ba = 0x7fffffff;
  for (int a = lane; a < I.A; a += kWave) {
    const int64_t L = I.lens[a];
    if (L < bl) {
      bl = L;
      ba = a;
    }
  }
  const int64_t minL = wave_min_i64(bl);
  C.ib = wave_min_i32(bl == minL ? ba : 0x7fffffff);
  C.iter = (int64_t)t;
  C.gb_len = st->gb_len;
  C.improved = minL < C.gb_len;
  C.tmin = st->tau_min;
  C.tmax = st->tau_max;
  if (C.improved) {
    C.gb_len = minL;
    limits(I, C.gb_len, C.tmin, C.tmax);
  }
  const uint64_t x = philox_word0(I.seed, t, ~0ull, 0, kPurposeSource);
  C.use_gb = (double)(uint32_t)(x >> 40) < I.p_gb * 16777216.0;
  C.src_len = C.use_gb ? C.gb_len : minL;
  C.delta = (float)(1.0 / (double)C.src_len);
  return C;
}

FACO_DEV void colony_write(const Inst &I, const Colony &C) {
  DevState *st = I.st;
  st->gb_len = C.gb_len;
  st->tau_min = C.tmin;
  st->tau_max = C.tmax;
  st->ib = C.ib;
  st->improved = C.improved ? 1 : 0;
  st->src_gb = C.use_gb ? 1 : 0;
  st->src_len = C.src_len;
  st->delta = C.delta;
  st->iter = C.iter;
}

FACO_DEV void run_colony(const Inst &I) {
  const Colony C = colony_decide(I);
  if (lane_id() == 0) colony_write(I, C);
}

// Bounding box of each half wave's 32 points (uniform over the half).
FACO_DEV int4 half_wave_box(int2 x) {
  int4 b = make_int4(x.x, x.y, x.x, x.y);
#pragma unroll
  for (int o = 1; o < 32; o <<= 1) {
    b.x = min(b.x, __shfl_xor(b.x, o));
    b.y = min(b.y, __shfl_xor(b.y, o));
    b.z = max(b.z, __shfl_xor(b.z, o));
    b.w = max(b.w, __shfl_xor(b.w, o));
  }
  return b;
}

// Source materialisation: the chosen tour becomes source_solution (route and
// its inverse), the iteration best becomes the global best when it improved.
// init: source := global best (before the first iteration).  Called with
// whole waves on 64 consecutive i (a multiple of 64 first), past n too.
FACO_DEV void run_source(const Inst &I, int i, int init) {
  const int n = I.n;
  if (i - lane_id() >= n) return;
  const DevState *st = I.st;
  const bool valid = i < n;
  const int ic = valid ? i : n - 1;
  const int i1 = ic + 1 == n ? 0 : ic + 1, i0 = ic == 0 ? n - 1 : ic - 1;
  const int32_t *from;
  if (init) {
    from = I.gb_route;
  } else {
    const int32_t *ibr = ant_route(I, st->ib);
    from = (st->src_gb && !st->improved) ? I.gb_route : ibr;
  }
  const int node = from[ic], next = from[i1], prev = from[i0];
  const int2 xn = I.xy[node];
  if (valid) {
    if (!init && st->improved) I.gb_route[i] = node;
    if (init || st->improved) I.gb_pos[node] = i;
    I.src_route[i] = node;
    I.src_pos[node] = i;
    I.src_adj[node] = make_int2(next, prev);
    I.src_xy[i] = xn;
    I.src_d[i] = cost(xn, I.xy[next]);
  }
  // bounding box of each half wave's 32 positions (those past n repeat the
  // last city)
  const int4 b = half_wave_box(xn);
  if (valid && (i & 31) == 0) I.sbox[i >> 5] = b;
}

// Eq. (2) with the deposit on the source edges: tau' = clamp(rho tau + delta
// [edge in source]).  init: tau = tau_max everywhere.  Slot s of city i's
// padded source-ordered row; pos: source positions of the cities, adj: city
// i's source neighbours.
FACO_DEV void pheromone_slot(const Inst &I, uint32_t i, uint32_t s, const int32_t *pos, int2 adj,
                             float tmin, float tmax, float delta, int init) {
  const uint32_t K = (uint32_t)I.k;
  // candidate row of city i moved to row pos(i), read by the next
  // construction: its Eq. (1) weight and the candidate's source position
  const int pi = pos[i];
  const size_t o = srow(pi, (int)s, I.ks);
  if (s >= K) {
    I.sw[o] = 0.0f;
    I.ssp[o] = pi;
    return;
  }
  const uint32_t idx = i * K + s;
  const int j = I.cl[idx];
  float tnew;
  if (init) {
    tnew = tmax;
  } else {
    const float t1 = I.rho * I.tau[idx];
    float t2 = (j == adj.x || j == adj.y) ? t1 + delta : t1;
    if (t2 > tmax) t2 = tmax;
    if (t2 < tmin) t2 = tmin;
    tnew = t2;
  }
  I.tau[idx] = tnew;
  I.sw[o] = tnew * I.eta[idx];
  I.ssp[o] = pos[j];
}

// slot: (city, slot of its padded source-ordered row).
FACO_DEV void run_pheromone(const Inst &I, uint32_t slot, int init) {
  const uint32_t n = (uint32_t)I.n, KS = (uint32_t)I.ks;
  if (slot >= n * KS) return;
  const uint32_t i = slot / KS, s = slot - i * KS;
  const DevState *st = I.st;
  const int2 adj = init ? make_int2(0, 0) : I.src_adj[i];
  pheromone_slot(I, i, s, I.src_pos, adj, st->tau_min, st->tau_max, st->delta, init);
}

// ===================================================================== //
// The whole update of an iteration in one launch (block `block` of
// update_blocks()): every block makes the colony's decision for itself from
// the ants' lengths, the first blocks update the pheromone, the padded rows and
// the source's inverse by (city, slot), the rest write the source's route, edge
// costs, coordinates and boxes by position.  Both read the
// chosen tour's own arrays (route and pos of the iteration best, or of the
// global best), so no block waits for another.  The state all blocks read is
// written by the last block that has read it.  As three dependent launches the
// update cost two more gaps of 7 us an iteration.  The decision takes a block
// about 2 us, and the blocks count themselves off at one address (about 13 ns
// each), so larger instances have a thread take several slots.  The launch with at
// most 256 + 64, 512 + 128 and 1024 + 256 blocks, lists of 16, in us: 10 000 cities
// 11.5/13.9/15.1, 20 000 13.6/16.1/21.0, 50 000 22.5/20.1/24.8, 100 000
// 37.8/27.1/30.2, 200 000 67.5/43.5/41.7 (the three launches 20.8, 22.8, 29.6, 39.7
// and 60.8): 512 + 128 until threads have 8 slots and 4 positions.
// ===================================================================== //
constexpr int kUpdateBlock = 256;
// blocks for `items` threads: one each, but at most `lo` of them while a thread has
// up to `most` items, and `hi` altogether
__host__ __device__ inline unsigned update_part(unsigned items, unsigned most, unsigned lo,
                                                unsigned hi) {
  const unsigned all = (items + kUpdateBlock - 1) / kUpdateBlock;
  unsigned cap = items / (most * kUpdateBlock);
  cap = cap < lo ? lo : (cap > hi ? hi : cap);
  return all < cap ? all : cap;
}
__host__ __device__ inline unsigned update_slot_blocks(int n, int ks) {
  return update_part((unsigned)n * (unsigned)ks, 8, 512, 1024);
}
__host__ __device__ inline unsigned update_pos_blocks(int n) {
  return update_part((unsigned)n, 4, 128, 256);
}
__host__ __device__ inline unsigned update_blocks(int n, int ks) {
  return update_slot_blocks(n, ks) + update_pos_blocks(n);
}

FACO_DEV void run_update(const Inst &I, unsigned block) {
  const int n = I.n;
  const uint32_t KS = (uint32_t)I.ks, slots = (uint32_t)n * KS;
  const unsigned nslot = update_slot_blocks(n, I.ks), npos = update_pos_blocks(n);
  const Colony C = colony_decide(I);
  const bool from_gb = C.use_gb && !C.improved;
  const int32_t *route = from_gb ? I.gb_route : ant_route(I, C.ib);
  const int32_t *pos = from_gb ? I.gb_pos : ant_pos(I, C.ib);
  if (block < nslot) {
    for (uint32_t slot = block * kUpdateBlock + threadIdx.x; slot < slots;
         slot += nslot * kUpdateBlock) {
      const uint32_t i = slot / KS, s = slot - i * KS;
      const int p = pos[i];
      const int2 adj = make_int2(route[p + 1 == n ? 0 : p + 1], route[p == 0 ? n - 1 : p - 1]);
      pheromone_slot(I, i, s, pos, adj, C.tmin, C.tmax, C.delta, 0);
      if (s == 0) {
        I.src_pos[i] = p;
        if (C.improved) I.gb_pos[i] = p;
      }
    }
  } else {
    for (int i = (int)((block - nslot) * kUpdateBlock + threadIdx.x); i - lane_id() < n;
         i += (int)npos * kUpdateBlock) {
      const int ic = i < n ? i : n - 1;
      const int node = route[ic], next = route[ic + 1 == n ? 0 : ic + 1];
      const int2 xn = I.xy[node];
      if (i < n) {
        if (C.improved) I.gb_route[i] = node;
        I.src_route[i] = node;
        I.src_xy[i] = xn;
        I.src_d[i] = cost(xn, I.xy[next]);
      }
      const int4 b = half_wave_box(xn);
      if (i < n && (i & 31) == 0) I.sbox[i >> 5] = b;
    }
  }
  __syncthreads();  // the whole block has read the state
  if (threadIdx.x == 0 && atomicAdd(&I.st->updates, 1) == (int)(nslot + npos) - 1) {
    colony_write(I, C);
    I.st->updates = 0;
  }
}

}  // namespace faco
