// faco_aux.hpp -- the per-iteration update kernel and its batched form, the
// tour-length verification and the candidate/backup list builder (gfx950).
#pragma once
#include "device_common.hpp"
#include "faco_device.hpp"
#include "faco_update.hpp"

namespace faco {

__global__ void __launch_bounds__(kUpdateBlock) update_kernel(Inst I) {
  run_update(I, blockIdx.x);
}

// Source and pheromone before the first iteration.
__global__ void __launch_bounds__(256) init_source_kernel(Inst I) {
  run_source(I, (int)(blockIdx.x * blockDim.x + threadIdx.x), 1);
}

__global__ void __launch_bounds__(256) init_pheromone_kernel(Inst I) {
  run_pheromone(I, blockIdx.x * blockDim.x + threadIdx.x, 1);
}

// Limits of the initial solution; state before the first iteration.
__global__ void init_state_kernel(Inst I) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  DevState *st = I.st;
  float tmin, tmax;
  limits(I, st->gb_len, tmin, tmax);
  st->tau_min = tmin;
  st->tau_max = tmax;
  st->src_len = st->gb_len;
  st->delta = 0.0f;
  st->ib = -1;
  st->src_gb = 0;
  st->improved = 0;
  st->iter = 0;
}


// ===================================================================== //
// Tour-length verification: every ant's tour (when `ants` is set) and the
// global best are summed again from the stored tours and the coordinates
// (int64, exact), and each ant's route is checked against its inverse
// (route[pos[c]] = c for every position: a permutation).  The sums are
// compared with the lengths the construction and local search tracked; a
// mismatch sets a fault.  Partial sums accumulate in vsum/vbad (zero
// between verifications; the finishing kernel reads and clears them).
//   verify: grid (chunks, A + 1 tours), block kVerifyBlock
// ===================================================================== //
constexpr int kVerifyBlock = 256;

FACO_DEV void verify_part(const Inst &I, int tour, int ants, int chunk, int nchunks) {
  const int n = I.n;
  const bool gb = tour == I.A;
  if (!gb && !ants) return;
  const int32_t *r = gb ? I.gb_route : ant_route(I, tour);
  const int32_t *pos = gb ? nullptr : ant_pos(I, tour);
  int64_t s = 0;
  bool bad = false;
  for (int i = chunk * kVerifyBlock + (int)threadIdx.x; i < n; i += nchunks * kVerifyBlock) {
    const int c = r[i], d = r[i + 1 == n ? 0 : i + 1];
    if ((unsigned)c >= (unsigned)n || (unsigned)d >= (unsigned)n) {
      bad = true;
      continue;
    }
    if (pos && pos[c] != i) bad = true;
    s += cost(I.xy[c], I.xy[d]);
  }
  s = wave_sum_i64(s);
  const bool wbad = ballot(bad) != 0;
  if (lane_id() == 0) {
    if (s) atomicAdd((unsigned long long *)&I.vsum[tour], (unsigned long long)s);
    if (wbad) atomicOr(&I.vbad[tour], 1);
  }
}

// Compare, publish the recomputed lengths in vout, clear the partial sums.
// iter_ahead: 1 when the ants being checked belong to the iteration in
// progress (before the colony update counts it), else 0.
FACO_DEV void verify_finish(const Inst &I, int ants, int iter_ahead) {
  DevState *st = I.st;
  for (int t = (int)threadIdx.x; t <= I.A; t += (int)blockDim.x) {
    if (t < I.A && !ants) continue;
    const int64_t L = I.vsum[t];
    const bool bad = I.vbad[t] != 0;
    const int64_t want = t < I.A ? I.lens[t] : st->gb_len;
    I.vout[t] = bad ? -1 : L;
    if (bad || L != want) {
      const int32_t bit = bad ? FAULT_PERMUTATION : FAULT_LENGTH;
      if (atomicOr(&st->fault, bit) == 0) {
        st->fault_ant = t < I.A ? t : -1;
        st->fault_iter = st->iter + iter_ahead;
      }
    }
    I.vsum[t] = 0;
    I.vbad[t] = 0;
  }
  if (threadIdx.x == 0) st->verified += (ants ? I.A : 0) + 1;
}

__global__ void __launch_bounds__(kVerifyBlock) verify_kernel(Inst I, int ants) {
  verify_part(I, (int)blockIdx.y, ants, (int)blockIdx.x, (int)gridDim.x);
}
__global__ void __launch_bounds__(kVerifyBlock) verify_finish_kernel(Inst I, int ants,
                                                                     int iter_ahead) {
  verify_finish(I, ants, iter_ahead);
}

// chunks per tour of a verification launch
__host__ __device__ inline unsigned verify_chunks(int n) {
  const int c = (n + 4 * kVerifyBlock - 1) / (4 * kVerifyBlock);
  return (unsigned)(c < 1 ? 1 : (c > 128 ? 128 : c));
}

// ===================================================================== //
// Batched forms: blockIdx selects the instance; each instance reads only
// its own Inst.
// ===================================================================== //
// blockIdx.y = instance; blocks past an instance's own return
__global__ void __launch_bounds__(kUpdateBlock) update_batch_kernel(const Inst *insts) {
  const Inst &I = insts[blockIdx.y];
  if (blockIdx.x < update_blocks(I.n, I.ks)) run_update(I, blockIdx.x);
}

// blockIdx.z = instance; instances without verification, and tours or
// chunks past an instance's own, return
__global__ void __launch_bounds__(kVerifyBlock) verify_batch_kernel(const Inst *insts) {
  const Inst &I = insts[blockIdx.z];
  if (!I.verify || (int)blockIdx.y > I.A) return;
  const unsigned nc = verify_chunks(I.n);
  if (blockIdx.x >= nc) return;
  verify_part(I, (int)blockIdx.y, 1, (int)blockIdx.x, (int)nc);
}
__global__ void __launch_bounds__(kVerifyBlock) verify_finish_batch_kernel(const Inst *insts) {
  const Inst &I = insts[blockIdx.x];
  if (I.verify) verify_finish(I, 1, 1);
}

// ===================================================================== //
// Candidate + backup lists (Sec. 4.1): the KK = K + BL nearest cities by
// (squared distance, original number); eta = 1/d.  A wave per query city, its
// candidates in LDS.  Labels follow the Hilbert curve, so the kKnnWin labels
// around the query's give KK candidates and a bound close to the last one's
// distance, and every run of 32 labels is a compact box (wbox).  The wave then
// tests the boxes of 64 runs at a time and examines the runs that are not
// strictly beyond the bound, two at a time, a city per lane; cities before the
// bound are appended, and a full buffer is ranked (each entry counts the entries
// before it), cut to the first KK in order, and gives a nearer bound.  A run
// beyond the bound holds no city of the list (a tie at the bound's distance is
// examined), and the kept set does not depend on the visiting order: the lists
// are exactly those of a scan over all cities.
// A query per lane with an insertion sort in LDS was bound by its serial
// chains, at any size: lists of 80 took 1.08 ms for 200 cities, 2.41 for 1021,
// 2.80 for 20 000, 21.7 for 200 000.
// ===================================================================== //
constexpr int kKnnRun = 32, kKnnWin = 192, kKnnCap = 256, kKnnWaves = 4;

// Rank the M entries by (distance, number) and keep the first KK in order.
template <int Q>
FACO_DEV void knn_rank(double *kd, int32_t *ko, int M, int KK) {
  const int lane = lane_id();
  double d[Q];
  int o[Q], before[Q], same[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int i = q * kWave + lane;
    d[q] = i < M ? kd[i] : __builtin_huge_val();
    o[q] = i < M ? ko[i] : 0x7fffffff;
    before[q] = same[q] = 0;
  }
  for (int j = 0; j < M; ++j) {
    const double dj = kd[j];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      before[q] += dj < d[q] ? 1 : 0;
      same[q] += dj == d[q] ? 1 : 0;
    }
  }
  bool tie = false;
#pragma unroll
  for (int q = 0; q < Q; ++q) tie = tie || same[q] > 1;
  if (ballot(tie)) {
    for (int j = 0; j < M; ++j) {
      const double dj = kd[j];
      const int oj = ko[j];
#pragma unroll
      for (int q = 0; q < Q; ++q) before[q] += dj == d[q] && oj < o[q] ? 1 : 0;
    }
  }
  wave_lds_sync();
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    if (q * kWave + lane < M && before[q] < KK) {
      kd[before[q]] = d[q];
      ko[before[q]] = o[q];
    }
  }
  wave_lds_sync();
}

__global__ void __launch_bounds__(kWave * kKnnWaves)
    knn_kernel(const int2 *xy, const int32_t *orig_of, const int32_t *int_of, const int4 *wbox,
               int n, int K, int BL, int32_t *cl, int32_t *bll, float *eta, int32_t *cl_d,
               DevState *st) {
  __shared__ double lds_d[kKnnWaves][kKnnCap];
  __shared__ int32_t lds_o[kKnnWaves][kKnnCap];
  const int lane = lane_id(), KK = K + BL;
  const int w = uniform_i((int)(threadIdx.x >> 6));
  const int i = uniform_i((int)blockIdx.x * kKnnWaves + w);
  if (i >= n) return;
  double *kd = lds_d[w];
  int32_t *ko = lds_o[w];
  const int2 xi = xy[i];
  const int win = n < kKnnWin ? n : kKnnWin;
  int lo = i - win / 2;
  lo = lo > n - win ? n - win : lo;
  lo = lo < 0 ? 0 : lo;
  // the window without the query itself
  for (int q = lane; q < win; q += kWave) {
    const int j = lo + q;
    if (j != i) {
      const int at_q = j < i ? q : q - 1;
      kd[at_q] = sqd(xi, xy[j]);
      ko[at_q] = orig_of[j];
    }
  }
  wave_lds_sync();
  int cnt = win - 1;
  double bound = __builtin_huge_val();
  int bound_o = 0x7fffffff;
  auto rank = [&]() {
    if (cnt <= 2 * kWave)
      knn_rank<2>(kd, ko, cnt, KK);
    else
      knn_rank<kKnnCap / kWave>(kd, ko, cnt, KK);
    if (cnt >= KK) {
      cnt = KK;
      bound = kd[KK - 1];
      bound_o = ko[KK - 1];
    }
  };
  rank();
  const int nrun = (n + kKnnRun - 1) / kKnnRun;
  bool sorted = true;
  for (int c0 = 0; c0 < nrun; c0 += kWave) {
    const int c = c0 + lane;
    bool need = false;
    if (c < nrun && (c * kKnnRun < lo || (c + 1) * kKnnRun > lo + win)) {
      const int4 b = wbox[c];
      const int dx = max(max(b.x - xi.x, xi.x - b.z), 0);
      const int dy = max(max(b.y - xi.y, xi.y - b.w), 0);
      need = !((double)dx * (double)dx + (double)dy * (double)dy > bound);
    }
    uint64_t m = ballot(need);
    while (m) {
      const int r0 = ctz64(m);
      m &= m - 1;
      const int r1 = m ? ctz64(m) : -1;
      if (m) m &= m - 1;
      const int r = lane < 32 ? r0 : r1;
      const int j = (c0 + r) * kKnnRun + (lane & 31);
      bool take = r >= 0 && j < n && (j < lo || j >= lo + win);
      double d = 0.0;
      int o = 0;
      if (take) {
        d = sqd(xi, xy[j]);
        take = d <= bound;
      }
      if (take) {
        o = orig_of[j];
        take = d < bound || o < bound_o;
      }
      const uint64_t tm = ballot(take);
      if (!tm) continue;
      if (take) {
        const int p = cnt + __builtin_popcountll(tm & ((1ull << lane) - 1ull));
        kd[p] = d;
        ko[p] = o;
      }
      cnt += __builtin_popcountll(tm);
      sorted = false;
      wave_lds_sync();
      if (cnt > kKnnCap - kWave) {
        rank();
        sorted = true;
      }
    }
  }
  if (!sorted) rank();
  for (int s = lane; s < KK; s += kWave) {
    const int c = int_of[ko[s]];
    if (s < K) {
      const int d = nint_sqrt(kd[s]);
      cl[(size_t)i * K + s] = c;
      cl_d[(size_t)i * K + s] = d;
      eta[(size_t)i * K + s] = (float)(1.0 / (double)d);
    } else {
      bll[(size_t)i * BL + (s - K)] = c;
    }
  }
  if (lane == 0 && kd[0] == 0.0) atomicOr(&st->dup, 1);
}

// ===================================================================== //
// Device-to-device copies of a list of blocks (the autotuner's snapshot and
// restore of its trial instances): one workgroup per block at a time, 16-byte
// words while both addresses are 16-byte aligned, single bytes for the rest.
// ===================================================================== //
struct CopySeg {
  const unsigned char *src;
  unsigned char *dst;
  uint64_t bytes;
};

__global__ void __launch_bounds__(256) copy_segments_kernel(const CopySeg *segs, int nseg) {
  for (int s = blockIdx.x; s < nseg; s += gridDim.x) {
    const CopySeg g = segs[s];
    const bool vec = (((uintptr_t)g.src | (uintptr_t)g.dst) & 15u) == 0;
    const uint64_t nv = vec ? g.bytes / 16 : 0;
    const uint4 *sv = reinterpret_cast<const uint4 *>(g.src);
    uint4 *dv = reinterpret_cast<uint4 *>(g.dst);
    for (uint64_t k = threadIdx.x; k < nv; k += blockDim.x) dv[k] = sv[k];
    for (uint64_t k = nv * 16 + threadIdx.x; k < g.bytes; k += blockDim.x) g.dst[k] = g.src[k];
  }
}

}  // namespace faco
