// Particle storage and cell binning.
//
// Storage: one 64-byte record per particle (position, momentum, 1/T, id,
// replica), so that gathering a neighbour touches one cache line instead of
// one line per array; the internal energy, read only by its own particle,
// lives in a separate array.
//
// Order: particles are kept sorted by the composite key (cell, id).  The sort
// is a two-level MSD radix sort: digit 1 is the whole cell index (one
// counting pass: histogram of cells with integer atomics, which also chains
// each cell's particles, then an exclusive scan to cell offsets); digit 2 is
// the particle identifier: every particle counts the smaller identifiers of
// its cell's chain (of its cell's bucket, where one block does it all or a large
// state has just been set).  The resulting order is a pure function of the positions,
// independent of the previous order and of atomic arrival order, so
// trajectories are bit reproducible and a resumed run continues exactly.
#pragma once

#include "common.h"

namespace dpde {

struct alignas(64) Rec {
  double qx, qy, qz;
  double px, py, pz;
  double invT;
  uint32_t id;   // identifier inside the replica
  uint32_t rep;  // replica index
};
static_assert(sizeof(Rec) == 64, "particle record must be one 64-byte block");

struct PState {
  Rec* r;
  double* eps;
};

// Neighbour-list build control for one step.  The kick kernel raises dmax to
// the largest squared displacement since the last build (bit pattern of a
// non-negative double, so integer max is float max); the binning and list
// build kernels run when force is set or dmax exceeds (skin/2)^2, and do
// nothing otherwise.  The decision is read from device memory by every
// kernel, so a captured graph replays it faithfully.
struct BuildCtl {
  unsigned long long dmax_bits;
  uint32_t force;
  uint32_t pad;
  unsigned long long qmax_bits;  // largest |coordinate| outside the box this step
};

// The same maxima of a step whose kick ran at the end of the previous one,
// spread over a wave's worth of slots (a cache line each) that the end of that
// step takes the maximum of.
constexpr int kNextSlots = kWave;
// What such a kick finds wrong belongs to the step it begins, so it waits here
// until the present one is counted.
struct alignas(128) NextMax {
  unsigned long long dmax_bits;
  unsigned long long qmax_bits;
  uint32_t status;
};

__device__ __forceinline__ bool rebuild_now(const BuildCtl* c, double half_skin2) {
  return c->force != 0u || __longlong_as_double((long long)c->dmax_bits) > half_skin2;
}

// Position (FP32) and identifier of a particle in 16 bytes: what the list
// build's candidate scans read (written by the reorder), and the reference
// of the kick's displacement test until the next build.  The FP32 distance
// test is widened by a bound on its rounding error, so a list still holds
// every pair within rc + skin; the exact r < rc filter of each step is FP64.
struct alignas(16) QIdF {
  float x, y, z;
  uint32_t id;
};

// XCD-aware tile order: the hardware deals workgroups round-robin over the 8
// XCDs (each with its own L2); the remap makes XCD x work through one
// contiguous share of the cell-sorted particles, a slab of the box whose
// neighbour data stays in that XCD's L2.  It is a bijection on [0, nb).
__device__ __forceinline__ unsigned xcd_tile(unsigned b, unsigned nb) {
  constexpr unsigned kXcd = 8;
  const unsigned q = nb / kXcd, r = nb % kXcd;
  const unsigned x = b % kXcd, k = b / kXcd;
  // workgroups b = x + 8k with k < q + (x < r) land on XCD x; give them the
  // consecutive tiles first(x) .. first(x) + q + (x < r) - 1
  const unsigned first = x * q + (x < r ? x : r);
  return first + k;
}

// ---- initial load: AoS rows in identifier order -> records --------------------
// Row k belongs to the replica r with geo[r].first <= k < geo[r].first + n.
__global__ void k_load_state(const double* __restrict__ q, const double* __restrict__ p,
                             const double* __restrict__ eps, const Geo* __restrict__ geo, int nrep,
                             int64_t n, PState s, uint32_t* status) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  int lo = 0, hi = nrep - 1;
  while (lo < hi) {  // last replica whose first row <= k
    const int mid = (lo + hi + 1) >> 1;
    if (geo[mid].first <= k) lo = mid; else hi = mid - 1;
  }
  Rec rc;
  rc.qx = q[3 * k]; rc.qy = q[3 * k + 1]; rc.qz = q[3 * k + 2];
  rc.px = p[3 * k]; rc.py = p[3 * k + 1]; rc.pz = p[3 * k + 2];
  rc.invT = 0.0;
  rc.id = (uint32_t)(k - geo[lo].first);
  rc.rep = (uint32_t)lo;
  const double e = eps[k];
  s.r[k] = rc;
  s.eps[k] = e;
  const bool fin = isfinite(rc.qx) && isfinite(rc.qy) && isfinite(rc.qz) && isfinite(rc.px) &&
                   isfinite(rc.py) && isfinite(rc.pz) && isfinite(e);
  if (!fin) atomicOr(status, ST_NONFINITE);
  else if (!(e > 0.0)) atomicOr(status, ST_NEG_EINT);
}

// ---- state out: records -> AoS rows in identifier order -----------------------
__global__ void k_store_state(PState s, const Geo* __restrict__ geo, int64_t n, double* q,
                              double* p, double* eps) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const Rec rc = s.r[i];
  const int64_t row = geo[rc.rep].first + (int64_t)rc.id;
  if (q) { q[3 * row] = rc.qx; q[3 * row + 1] = rc.qy; q[3 * row + 2] = rc.qz; }
  if (p) { p[3 * row] = rc.px; p[3 * row + 1] = rc.py; p[3 * row + 2] = rc.pz; }
  if (eps) eps[row] = s.eps[i];
}

__global__ void k_store_vec3(PState s, const Geo* __restrict__ geo, int64_t n,
                             const double* __restrict__ x, const double* __restrict__ y,
                             const double* __restrict__ z, double* out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const Rec& rc = s.r[i];
  const int64_t row = geo[rc.rep].first + (int64_t)rc.id;
  out[3 * row] = x[i]; out[3 * row + 1] = y[i]; out[3 * row + 2] = z[i];
}

// 1/T_i of every particle into out (identifier order).
__global__ void k_store_inv_temperature(PState s, const Geo* __restrict__ geo, int64_t n,
                                        double* out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const Rec& rc = s.r[i];
  out[geo[rc.rep].first + (int64_t)rc.id] = rc.invT;
}

// Length of every particle's list of the step into out (identifier order).
__global__ void k_store_list_length(PState s, const Geo* __restrict__ geo, int64_t n,
                                    const uint32_t* __restrict__ count, int32_t* out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const Rec& rc = s.r[i];
  out[geo[rc.rep].first + (int64_t)rc.id] = (int32_t)count[i];
}

constexpr int kAuxMaxThreads = 1024;  // largest block of the per-particle kernels

// A coordinate moved by one step at momentum p.
__device__ __forceinline__ double drifted(double q, double p, const Phys& P) {
  return q + P.dt * p / P.mass;
}

// First half of velocity-Verlet (Sec. 3.1) on one record: p += dt/2 F and
// q += dt p / m (kick != 0), then the periodic wrap into [0, L).  Returns in
// d2 the square of an upper bound on the displacement since the last list
// build and, for a coordinate outside [0, box) (free boundaries), the
// largest such |q| in qa; a non-finite p or q raises the status.  The one
// definition of this arithmetic: k_kick and the end of a step's last pair pass
// both call it.
__device__ __forceinline__ void kick_record(Rec& rc, const double F[3], const Geo& g,
                                            const Phys& P, int kick,
                                            const QIdF* __restrict__ ref, int64_t i,
                                            double& d2, double& qa, uint32_t* status) {
  double q[3] = {rc.qx, rc.qy, rc.qz};
  if (kick) {
    double p[3] = {rc.px, rc.py, rc.pz};
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      p[d] = p[d] + P.half_dt * F[d];
      q[d] = drifted(q[d], p[d], P);
    }
    rc.px = p[0]; rc.py = p[1]; rc.pz = p[2];
    if (!(isfinite(p[0]) && isfinite(p[1]) && isfinite(p[2]))) atomicOr(status, ST_NONFINITE);
  }
#pragma unroll
  for (int d = 0; d < 3; ++d)
    if (g.periodic[d]) q[d] = wrap_coord(q[d], g.box[d]);
  rc.qx = q[0]; rc.qy = q[1]; rc.qz = q[2];
  if (!(isfinite(q[0]) && isfinite(q[1]) && isfinite(q[2]))) {
    atomicOr(status, ST_NONFINITE);
  } else {
    // coordinates outside [0, box) (free boundaries) for the list build's
    // rounding margin; inside, the box side bounds them already
#pragma unroll
    for (int d = 0; d < 3; ++d)
      if (!(q[d] >= 0.0 && q[d] < g.box[d])) qa = fmax(qa, fabs(q[d]));
    // The reference is the build-time position rounded to FP32, each
    // coordinate within 2^-24 |x| of the exact one, which is below
    // 2^-23 |x_f| for its FP32 value x_f (2^-149 covers subnormals); the sum
    // of those bounds and 2^-50 of the FP64 distance for its own rounding
    // make d an upper bound on the true displacement.
    const QIdF r0 = ref[i];
    double dx = q[0] - (double)r0.x, dy = q[1] - (double)r0.y, dz = q[2] - (double)r0.z;
    if (g.periodic[0]) dx = min_image(dx, g.box[0], g.half_box[0]);
    if (g.periodic[1]) dy = min_image(dy, g.box[1], g.half_box[1]);
    if (g.periodic[2]) dz = min_image(dz, g.box[2], g.half_box[2]);
    const double slack =
        0x1p-23 * ((double)fabsf(r0.x) + (double)fabsf(r0.y) + (double)fabsf(r0.z)) + 0x1p-147;
    const double d = sqrt(dx * dx + dy * dy + dz * dz) * (1.0 + 0x1p-50) + slack;
    d2 = d * d;
  }
}

// Raise a running maximum of non-negative doubles kept as bits (they order
// like their bit patterns); one atomic, and only when it raises the value (a
// stale read can only be smaller than the true value, never skip a raise).
__device__ __forceinline__ void raise_max_bits(unsigned long long* where, double v) {
  const unsigned long long bits = (unsigned long long)__double_as_longlong(v);
  const unsigned long long cur = __hip_atomic_load(where, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (bits > cur) atomicMax(where, bits);
}

// The kick of every particle (kick == 0: only the wrap), with the maxima the
// next list-build decision reads.
template <bool BATCH>
__global__ void k_kick(PState s, const double* __restrict__ Fx, const double* __restrict__ Fy,
                       const double* __restrict__ Fz, int64_t n, const Geo* __restrict__ geo,
                       Phys P, int kick, const QIdF* __restrict__ ref, BuildCtl* ctl,
                       uint32_t* status) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  // no early return: every thread reaches the block barrier below (another
  // block may raise the status while this one runs)
  const bool run = !status_set(status);
  double d2 = 0.0, qa = 0.0;
  if (run && i < n) {
    Rec rc = s.r[i];
    const Geo& g = geo[BATCH ? rc.rep : 0u];
    double F[3] = {0.0, 0.0, 0.0};
    if (kick) {
      F[0] = Fx[i];
      F[1] = Fy[i];
      F[2] = Fz[i];
    }
    kick_record(rc, F, g, P, kick, ref, i, d2, qa, status);
    s.r[i] = rc;
  }
  // |q| outside the box only occurs with free boundaries: waves that have
  // any take their maximum and one atomic (when it raises the running one)
  if (__any(qa > 0.0)) {
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) qa = fmax(qa, __shfl_xor(qa, off, kWave));
    if ((threadIdx.x % kWave) == 0 && run) raise_max_bits(&ctl->qmax_bits, qa);
  }
  // block maximum of the displacement, then one atomic per block
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) d2 = fmax(d2, __shfl_xor(d2, off, kWave));
  __shared__ double wmax[kAuxMaxThreads / kWave];
  const int nw = blockDim.x / kWave;
  if ((threadIdx.x % kWave) == 0) wmax[threadIdx.x / kWave] = d2;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < nw; ++w) d2 = fmax(d2, wmax[w]);
    if (run) raise_max_bits(&ctl->dmax_bits, d2);
  }
}

// Runs of equal keys among consecutive lanes of a wave: the lane that heads
// this lane's run and the lane behind the run's last.  Every lane of the wave
// calls (dead lanes with live = false).
struct LaneRun {
  bool head;
  int from, end;
};
__device__ __forceinline__ LaneRun lane_run(uint32_t c, bool live) {
  const int lane = threadIdx.x % kWave;
  const uint32_t prev = __shfl_up(c, 1, kWave);
  LaneRun r;
  r.head = live && (lane == 0 || prev != c);
  const unsigned long long heads = __ballot(r.head);
  const unsigned long long below = (lane == 63) ? ~0ull : ((1ull << (lane + 1)) - 1ull);
  r.from = 63 - __clzll(heads & below);             // last head at or below this lane
  const unsigned long long above = heads & ~below;  // heads strictly above
  r.end = above ? __ffsll((long long)above) - 1 : kWave;
  // the run of a head ends before the next head or at the first dead lane
  const unsigned long long dead_above = ~__ballot(live) & ~below;
  if (dead_above) r.end = min(r.end, __ffsll((long long)dead_above) - 1);
  return r;
}

// Histogram increment with one atomic per run; the run's lanes take
// consecutive tickets.
__device__ __forceinline__ uint32_t run_ticket(uint32_t c, bool live, uint32_t* count) {
  const int lane = threadIdx.x % kWave;
  const LaneRun r = lane_run(c, live);
  uint32_t base = 0;
  if (r.head) base = atomicAdd(&count[c], (uint32_t)(r.end - lane));
  base = __shfl(base, r.from, kWave);
  return base + (uint32_t)(lane - r.from);
}

// ---- exclusive scan of the cell histogram -> cell offsets --------------------
constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanThreads * kScanItems;

// Exclusive scan of one value per thread across the block; returns the block
// total through *total.
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* smem,
                                                         uint32_t* total) {
  const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave, nw = blockDim.x / kWave;
  uint32_t x = v;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const uint32_t y = __shfl_up(x, off, kWave);
    if (lane >= off) x += y;
  }
  if (lane == kWave - 1) smem[wid] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t run = 0;
    for (int w = 0; w < nw; ++w) {
      const uint32_t t = smem[w];
      smem[w] = run;
      run += t;
    }
    smem[nw] = run;
  }
  __syncthreads();
  const uint32_t excl = smem[wid] + x - v;
  *total = smem[nw];
  __syncthreads();
  return excl;
}

// out[c] = sum_{c' < c} in[c'] for c <= n by one block of up to 1024 threads.
constexpr int kScanWavesMax = kAuxMaxThreads / kWave;
__device__ __forceinline__ void scan_in_block(const uint32_t* __restrict__ in, int64_t n,
                                              uint32_t* __restrict__ out,
                                              uint32_t* smem /* waves + 1 */) {
  uint32_t offset = 0;
  const int64_t chunk = (int64_t)blockDim.x * kScanItems;
  for (int64_t b0 = 0; b0 < n; b0 += chunk) {
    const int64_t base = b0 + (int64_t)threadIdx.x * kScanItems;
    uint32_t v[kScanItems], s = 0, total;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      v[k] = base + k < n ? in[base + k] : 0u;
      s += v[k];
    }
    uint32_t run = block_exclusive_scan(s, smem, &total) + offset;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
      if (base + k < n) out[base + k] = run;
      run += v[k];
    }
    offset += total;
  }
  if (threadIdx.x == 0) out[n] = offset;
}

__global__ void k_scan_tiles(const uint32_t* __restrict__ in, int64_t n,
                             uint32_t* __restrict__ tile_sums, const BuildCtl* ctl,
                             double half_skin2) {
  if (!rebuild_now(ctl, half_skin2)) return;
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  uint32_t s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k)
    if (base + k < n) s += in[base + k];
  __shared__ uint32_t smem[kScanThreads / kWave + 1];
  uint32_t total;
  block_exclusive_scan(s, smem, &total);
  if (threadIdx.x == 0) tile_sums[blockIdx.x] = total;
}

// out[c] = sum_{c' < c} in[c'] for c <= n; the histogram is cleared for the
// next step.  Each block first adds the totals of the tiles before it (at
// most 1024 * 8 tiles: 32 per thread), so no separate pass scans them.
__global__ void k_scan_apply(uint32_t* __restrict__ in, int64_t n,
                             const uint32_t* __restrict__ tile_sums, uint32_t* __restrict__ out,
                             const BuildCtl* ctl, double half_skin2) {
  if (!rebuild_now(ctl, half_skin2)) return;
  __shared__ uint32_t smem[kScanThreads / kWave + 1];
  uint32_t before = 0;
  for (unsigned t = threadIdx.x; t < blockIdx.x; t += blockDim.x) before += tile_sums[t];
  uint32_t offset;
  block_exclusive_scan(before, smem, &offset);
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  uint32_t v[kScanItems];
  uint32_t s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    v[k] = (base + k < n) ? in[base + k] : 0u;
    s += v[k];
  }
  uint32_t total;
  uint32_t run = block_exclusive_scan(s, smem, &total) + offset;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    if (base + k < n) {
      out[base + k] = run;
      in[base + k] = 0u;
    }
    run += v[k];
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) out[n] = offset + total;
}

// ---- the list build's binning -------------------------------------------------
// Cells: the histogram and, per cell, a chain of its particles (link[i] = the
// identifier and the next particle; `first` heads it), both left cleared by the
// list build.  In crowded cells, as steps meet them, the chains are no slower than
// the buckets of particle numbers that they replaced, whose identifiers had to be
// gathered (3000 particles in one cell 302 against 390 us per build, 12,000 1175
// against 1500).
struct CellBins {
  uint32_t* count;
  uint32_t* first;
  uint32_t* start;  // exclusive scan of the histogram, ncells + 1
  uint2* link;
  uint32_t* key;    // cell of every particle
  uint2* bucket;    // by cell: particle and identifier, or null (chains)
  int64_t ncells;
};
constexpr uint32_t kChainEnd = 0xFFFFFFFFu;

// Digit 2 and the move into the new order: particle i counts the smaller
// identifiers of its cell's chain, which is its place in the cell, and its
// record and internal energy go there in the spare buffer, with the build-time
// position (FP32) and the memory index of its identifier row (for the
// neighbour-list build).  The list build then returns the records to the
// working buffer, so the buffer roles never depend on whether this step
// rebuilt.
template <bool BATCH>
__device__ __forceinline__ void rank_move(const PState& src, const PState& dst, const CellBins& cb,
                                          int64_t i, const Geo* __restrict__ geo,
                                          QIdF* __restrict__ qid, uint32_t* __restrict__ slot) {
  const uint32_t c = cb.key[i];
  const uint32_t b = cb.start[c];
  // The record as four 16-byte words: copied as a structure, half of it went
  // through LDS (32 KB per block, bank conflicts on every access; the first
  // build of an unordered state at N = 1M 166 -> 150 us here, N = 65,536 75.7 ->
  // 74.8 us per step).
  const uint4* from = reinterpret_cast<const uint4*>(src.r + i);
  const uint4 w0 = from[0], w1 = from[1], w2 = from[2], w3 = from[3];
  const uint32_t id = w3.z;
  const double e = src.eps[i];
  uint32_t p = b;
  if (cb.bucket) {  // uniform
    const uint32_t end = cb.start[c + 1];
    for (uint32_t m = b; m < end; ++m) p += cb.bucket[m].y < id ? 1u : 0u;
  } else {
    for (uint32_t j = cb.first[c]; j != kChainEnd;) {
      const uint2 l = cb.link[j];
      p += l.x < id ? 1u : 0u;
      j = l.y;
    }
  }
  uint4* to = reinterpret_cast<uint4*>(dst.r + p);
  to[0] = w0;
  to[1] = w1;
  to[2] = w2;
  to[3] = w3;
  dst.eps[p] = e;
  qid[p] = QIdF{(float)__hiloint2double((int)w0.y, (int)w0.x),
                (float)__hiloint2double((int)w0.w, (int)w0.z),
                (float)__hiloint2double((int)w1.y, (int)w1.x), id};
  slot[(BATCH ? (uint32_t)geo[w3.w].first : 0u) + id] = p;
}

// The buckets: each cell's particles side by side, in the order of their tickets
// (link = the identifier and the ticket).
__device__ __forceinline__ void bucket_in(const CellBins& cb, int64_t i) {
  const uint2 l = cb.link[i];
  cb.bucket[cb.start[cb.key[i]] + l.y] = make_uint2((uint32_t)i, l.x);
}

// Digit 1 (list-build steps only): the cell of every particle, the histogram
// and the chains, with one atomic of each kind per run of equal keys inside a
// wave (the particles are still nearly in cell order).  Tiles follow the
// XCD-aware order, so each XCD's atomics touch its own slab of counters.
//
// On most steps the kernels of a build only find that none is due, and each
// such launch costs a few microseconds, so a build takes as few as its size
// allows (BinPlan): with `scan` the last block to finish also scans the
// histogram, and with `whole` (one block) it goes on to rank and move the
// particles, by buckets, which cost it no launch (1000 of 1800 particles in one
// cell: 218 -> 159 us).  The histogram is complete there: every block's atomics
// are ordered before its ticket.
template <bool BATCH>
__global__ __launch_bounds__(kAuxMaxThreads) void k_bin(
    PState s, PState dst, int64_t n, const Geo* __restrict__ geo, CellBins cb, int scan, int whole,
    uint32_t* ticket, QIdF* __restrict__ qid, uint32_t* __restrict__ slot, const BuildCtl* ctl,
    double half_skin2, const uint32_t* status) {
  if (status_set(status) || !rebuild_now(ctl, half_skin2)) return;  // uniform
  __shared__ uint32_t smem[kScanWavesMax + 1];
  __shared__ uint32_t last;
  const int64_t turn = (int64_t)gridDim.x * blockDim.x;
  const int64_t i0 = (int64_t)xcd_tile(blockIdx.x, gridDim.x) * blockDim.x;
  for (int64_t b0 = i0; b0 < n; b0 += turn) {  // uniform in the block
    const int64_t i = b0 + threadIdx.x;
    const bool live = i < n;
    uint32_t c = 0xFFFFFFFFu, id = 0u;
    if (live) {
      const Rec& rc = s.r[i];
      const Geo& g = geo[BATCH ? rc.rep : 0u];
      const int cx = cell_coord(rc.qx, g.scale[0], g.nc[0]);
      const int cy = cell_coord(rc.qy, g.scale[1], g.nc[1]);
      const int cz = cell_coord(rc.qz, g.scale[2], g.nc[2]);
      c = (uint32_t)(g.cell_base + cell_key(g, cx, cy, cz));
      id = rc.id;
      cb.key[i] = c;
    }
    if (cb.bucket) {  // uniform
      const uint32_t t = run_ticket(c, live, cb.count);
      if (live) cb.link[i] = make_uint2(id, t);
      continue;
    }
    const int lane = threadIdx.x % kWave;
    const LaneRun r = lane_run(c, live);
    uint32_t behind = kChainEnd;
    if (r.head) {
      atomicAdd(&cb.count[c], (uint32_t)(r.end - lane));
      behind = atomicExch(&cb.first[c], (uint32_t)i);
    }
    behind = __shfl(behind, r.from, kWave);
    if (live) cb.link[i] = make_uint2(id, lane + 1 < r.end ? (uint32_t)i + 1u : behind);
  }
  if (!scan) return;  // uniform
  if (gridDim.x > 1u) {
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) last = atomicAdd(ticket, 1u) == gridDim.x - 1u;
    __syncthreads();
    if (!last) return;  // uniform in the block
    __threadfence();
    if (threadIdx.x == 0) *ticket = 0u;
  } else {
    __threadfence_block();
    __syncthreads();
  }
  scan_in_block(cb.count, cb.ncells, cb.start, smem);
  if (!whole) return;  // uniform
  __threadfence_block();
  __syncthreads();
  for (int64_t i = threadIdx.x; i < n; i += blockDim.x) bucket_in(cb, i);
  __threadfence_block();
  __syncthreads();
  for (int64_t i = threadIdx.x; i < n; i += blockDim.x)
    rank_move<BATCH>(s, dst, cb, i, geo, qid, slot);
}

// The scan of a histogram too long for one block but short enough for each
// block to add up all counts before its own tile (no pass over tile sums).
constexpr int kScanWideThreads = 1024;
constexpr int kScanWideTile = kScanWideThreads * kScanItems;
__global__ __launch_bounds__(kScanWideThreads) void k_scan_cells(CellBins cb, const BuildCtl* ctl,
                                                                 double half_skin2) {
  if (!rebuild_now(ctl, half_skin2)) return;
  __shared__ uint32_t smem[kScanWideThreads / kWave + 1];
  const int64_t tile = (int64_t)blockIdx.x * kScanWideTile;
  uint32_t before = 0;
  const uint4* in4 = reinterpret_cast<const uint4*>(cb.count);
  for (int64_t k = threadIdx.x; k < tile / 4; k += kScanWideThreads) {
    const uint4 v = in4[k];
    before += (v.x + v.y) + (v.z + v.w);
  }
  uint32_t offset, total;
  block_exclusive_scan(before, smem, &offset);
  const int64_t base = tile + (int64_t)threadIdx.x * kScanItems;
  uint32_t v[kScanItems], s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    v[k] = base + k < cb.ncells ? cb.count[base + k] : 0u;
    s += v[k];
  }
  uint32_t run = block_exclusive_scan(s, smem, &total) + offset;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    if (base + k < cb.ncells) cb.start[base + k] = run;
    run += v[k];
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) cb.start[cb.ncells] = offset + total;
}

__global__ void k_bin_scatter(CellBins cb, int64_t n, const BuildCtl* ctl, double half_skin2,
                              const uint32_t* status) {
  if (status_set(status) || !rebuild_now(ctl, half_skin2)) return;  // uniform
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) bucket_in(cb, i);
}

// A particle per lane: those of the present memory order, or with buckets those
// of the new one's cells, so that the records, read wherever they lie, are
// written side by side.
template <bool BATCH>
__global__ void k_rank_gather(PState src, PState dst, CellBins cb, int64_t n,
                              const Geo* __restrict__ geo, QIdF* __restrict__ qid,
                              uint32_t* __restrict__ slot, const BuildCtl* ctl, double half_skin2,
                              const uint32_t* status) {
  if (status_set(status) || !rebuild_now(ctl, half_skin2)) return;  // uniform
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < n) rank_move<BATCH>(src, dst, cb, cb.bucket ? cb.bucket[k].x : k, geo, qid, slot);
}

}  // namespace dpde
