// Pair passes of one DPDE step over cell-sorted particles.
//
//   pass A  conservative forces at the new positions, neighbour list build,
//           second half-kick of velocity-Verlet (Sec. 3.1);
//   pass B  SER sweep 1: dp_ij and dp_i = sum_j dp_ij (eq. SER_p);
//   pass C  SER sweep 2: internal-energy reinjection
//           (eq. SER_eint_discretization), p <- p + dp, eps <- eps + d eps,
//           next 1/T_i.
//
// A few lanes per particle.  In the both-sides form each pair term is evaluated
// on both of its particles' lanes in the canonical orientation (lower identifier first) and
// negated on the higher one, so dp_ji = -dp_ij bit for bit and the particle
// sums are plain gathers: no atomics, fixed summation order.
//
// Sweep 2 needs the same dp_ij as sweep 1.  The paper regenerates the noise
// from (i, j, n) to avoid storing the increments; with HBM to spare, sweep 1
// here stores dp_ij per neighbour-list entry and sweep 2 reads it back, which
// removes the random-number generation and the pair geometry from sweep 2.
// The regenerating form is kept (Phys::regen) and gives identical bits.
#pragma once

#include "bin.h"
#include "eos.h"
#include "mlp.h"

namespace dpde {

constexpr int kPairBlockMax = 256;

enum : int { PREC_F64 = 0, PREC_F32 = 1 };

struct alignas(32) DP {
  double x, y, z, pad;
};

// Momentum after the conservative half-kick and the sweep-1 increment of one
// particle, packed so that sweep 2 gathers one line per neighbour.
// Per-particle results of SER sweep 1: dp_i = sum_j dp_ij, and
// h_i = (p_i + dp_i / 2) / m, so that the velocity combination of sweep 2,
// v_ij + (dp_i - dp_j)/(2m), is h_i - h_j (exactly antisymmetric).
struct alignas(32) Vec4 {
  double x, y, z, w;
};

// Neighbour lists: 32 particles side by side, entry after entry, so that for a
// given k the lanes of a wave touch consecutive words and a wave's lists lie in
// one stretch of memory.  (With entry k of all particles side by side the
// entries of one list were n words apart, each on pages of its own, and the
// sweeps over long lists, which also stream the increments of every entry, were
// bound by that and not by their arithmetic or cache accesses: 1,061,208
// particles of the Lennard-Jones fluid, ~53 entries, sweep 1 805 -> 751 us,
// sweep 2 513 -> 469, list of the step 477 -> 458; with ~13 entries neutral.)
constexpr int kRow = 32;
__host__ __device__ inline int64_t list_entry(int64_t i, int64_t k, int64_t cap) {
  return ((i / kRow) * cap + k) * kRow + i % kRow;
}
// Entries to allocate for n particles.
inline size_t list_size(int64_t n, int64_t cap) {
  return (size_t)((n + kRow - 1) / kRow) * kRow * (size_t)cap;
}

struct NList {
  uint32_t* idx;
  uint32_t* count;
  double* de;   // dp_ij per entry (stored-increment form): x, y, z of 32 entries each
  int64_t cap;  // capacity per particle
};

__device__ __forceinline__ bool wrap_cell(int& c, int nc, int periodic) {
  if (c < 0) {
    if (!periodic) return false;
    c += nc;
  } else if (c >= nc) {
    if (!periodic) return false;
    c -= nc;
  }
  return true;
}

// Separation q_i - q_j with the minimum image along periodic dimensions.
__device__ __forceinline__ void separation(const Geo& g, double xi, double yi, double zi,
                                           double xj, double yj, double zj, double& dx,
                                           double& dy, double& dz) {
  dx = xi - xj;
  dy = yi - yj;
  dz = zi - zj;
  if (g.periodic[0]) dx = min_image(dx, g.box[0], g.half_box[0]);
  if (g.periodic[1]) dy = min_image(dy, g.box[1], g.half_box[1]);
  if (g.periodic[2]) dz = min_image(dz, g.box[2], g.half_box[2]);
}

// A particle farther than the list reach from every periodic face sees all of
// its listed neighbours at their stored (wrapped) positions: the minimum
// image is then the identity.  Waves whose particles all qualify skip it.
__device__ __forceinline__ bool away_from_faces(const Geo& g, const Phys& P, double x, double y,
                                                double z) {
  const double q[3] = {x, y, z};
  bool ok = true;
#pragma unroll
  for (int d = 0; d < 3; ++d)
    if (g.periodic[d]) ok = ok && q[d] >= P.reach && q[d] <= g.box[d] - P.reach;
  return ok;
}

__device__ __forceinline__ void separation_mi(const Geo& g, bool mi, double xi, double yi,
                                              double zi, double xj, double yj, double zj,
                                              double& dx, double& dy, double& dz) {
  if (mi) {
    separation(g, xi, yi, zi, xj, yj, zj, dx, dy, dz);
  } else {
    dx = xi - xj;
    dy = yi - yj;
    dz = zi - zj;
  }
}

// ---------------------------------------------------------------------------
// Lane groups.  Every particle is served by kSub consecutive lanes of one
// wave: lane `sub` of the group takes the list entries sub, sub + kSub, ...,
// and partial sums meet in a fixed xor butterfly.  The butterfly adds the same
// two operands on both partner lanes (in swapped order, which addition does
// not see), so all lanes of a group end with the same, reproducible sum.
// Compaction into a list keeps the candidates' order: each trip the group
// ballots its predicates and a lane's slot is the count of set bits below it.
// ---------------------------------------------------------------------------
constexpr int kSub = 4;
constexpr uint32_t kSubMask = (1u << kSub) - 1u;
// The SER sweeps (passes B and C) use pairs of lanes: with ~12 neighbours
// their pair terms keep more lanes busy per trip, while the filters over the
// ~27 skin candidates (pass A, and the list build where cells hold few
// particles) are faster with four.
constexpr int kSubSer = 2;
constexpr int kListLds = 64;  // list entries per particle staged in LDS
// Particles per tile (= block) of the unique-pair passes: 128, and smaller ones
// in systems whose tiles of 128 leave the chip idle (TileShape in api.hip).
constexpr int kUniqTile = 128;

// In the tile form a pair joining two particles of one tile (consecutive
// memory indices) is listed for one of them only: for the lower memory index
// when the two indices differ in parity, else for the higher one, so that
// about half of every particle's pairs inside its tile stay in its list
// whatever its place in the tile (the lanes of the passes stay evenly
// loaded); a pair joining two tiles is in both lists.  Which side evaluates a
// pair changes no sum: every per-particle sum of the tile form is an exact
// fixed-point sum, so neither does the size of the tiles.

// Exclusive prefix of v over the wave and the wave total.
__device__ __forceinline__ uint32_t wave_prefix(uint32_t v, uint32_t& total) {
  const int lane = threadIdx.x % kWave;
  uint32_t incl = v;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const uint32_t up = (uint32_t)__shfl_up((int)incl, off, kWave);
    if (lane >= off) incl += up;
  }
  total = (uint32_t)__shfl((int)incl, kWave - 1, kWave);
  return incl - v;
}

struct Lanes {
  int64_t i;     // particle
  int sub;       // lane within the group
  int pib;       // group within the block
  int ppb;       // groups per block
  int shift;     // position of the group's bits in a wave ballot
};

template <int KS = kSub>
__device__ __forceinline__ Lanes lanes() {
  Lanes L;
  const int64_t t = (int64_t)xcd_tile(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
  L.i = t / KS;
  L.sub = threadIdx.x % KS;
  L.pib = threadIdx.x / KS;
  L.ppb = blockDim.x / KS;
  L.shift = (threadIdx.x % kWave) & ~(KS - 1);
  return L;
}

template <int KS = kSub>
__device__ __forceinline__ double group_sum(double x) {
#pragma unroll
  for (int off = 1; off < KS; off <<= 1) x += __shfl_xor(x, off, kWave);
  return x;
}

// Group bits of a wave ballot.
__device__ __forceinline__ uint32_t group_ballot(const Lanes& L, bool pred) {
  return (uint32_t)(__ballot(pred) >> L.shift) & kSubMask;
}

// Neighbour lists with a skin.  On a build step every particle collects the
// particles within rs = rc + skin through the 27-cell stencil (k_build_skin),
// and the list is sorted by neighbour identifier.  Every step then keeps the
// entries with r < rc, in list order: the pair set is exactly the stencil's,
// and every per-particle sum below runs in identifier order, so the
// trajectory does not depend on memory order, skin width or build schedule.
// A build is due when some particle has moved more than skin/2 since the last
// one (then no pair within rc can be missing from the lists).
// ---------------------------------------------------------------------------
struct SkinList {
  uint32_t* idx;  // as NList
  uint32_t* count;
  int64_t cap;    // capacity per particle
};

// Square of the FP32 test radius: rs plus a bound on the rounding of the FP32
// distance (conversions of coordinates up to Q = max(|q|, box), their
// difference, the minimum image and the squared sum stay below
// 8 2^-24 (Q + rs); twice that is added), rounded up.
__device__ __forceinline__ float build_radius2(const BuildCtl* ctl, double rs, double box_max) {
  const double Q = fmax(__longlong_as_double((long long)ctl->qmax_bits), box_max);
  const double thr = rs + 16.0 * 0x1p-24 * (Q + rs);
  float thr2 = (float)(thr * thr);
  if ((double)thr2 < thr * thr) thr2 = nextafterf(thr2, INFINITY);
  return thr2;
}

// Entries k0, k0 + step, ... of particle i's list of `count` (memory indices)
// that tiles of 128 would list too.
__device__ __forceinline__ uint32_t listed_in_128(const SkinList& sl, int64_t i, int count, int k0,
                                                  int step) {
  uint32_t listed = 0;
  for (int k = k0; k < count; k += step) {
    const uint32_t j = sl.idx[list_entry(i, k, sl.cap)], x = (uint32_t)i ^ j;
    const bool mine = (x & 1u) ? (uint32_t)i < j : (uint32_t)i > j;
    listed += x >= (uint32_t)kUniqTile || mine ? 1u : 0u;
  }
  return listed;
}

// The build's block serves a tile of 128 consecutive particles.  Particles of
// one cell share their 27-cell stencil, so the unit of work is a piece: up to
// kPiece particles of the tile in one cell, taken by one wave.  The wave lists
// the stencil's candidates once (27 lanes, a cell each), holds up to
// kBuildChunks of them per lane in registers, and tests them against the
// piece's particles one after the other, whose position is then uniform (in
// scalar registers); the accepted ones take their places from the ballot.
// Per candidate and particle that leaves the FP32 distance and the list
// ownership, some 15 vector instructions for 64 candidates; four lanes per
// particle walking the stencil each for itself took ~75 and issued at 0.88 of
// the VALU's rate (N = 1M in blocked order, per build: 496 us, 275 so; the
// both-sides lists 441 us, 234 so; 256 replicas 524 us, 297 so; N = 1000 on 16
// waves per block 36.9 us, 18.6 so).  The lists are staged in LDS and
// written row by row (entries beyond the staged rows go straight to memory).
//
// UNIQ (the tile form, tiles of `tile` particles): the list keeps only the pairs
// that the rule above assigns to this particle, holds memory indices, and is not sorted: the passes that
// read it add their pair terms in fixed point, in any order.  Otherwise it
// holds identifier rows (first + id) until k_sort_skin has ordered them and
// turned them into memory indices.
// A list longer than `limit`, the capacity the caller asked for, is an
// overflow.  Tiles below 128 list more of the pairs on both sides (at most
// (128 - tile) / 2 per particle, for which the lists have room: sl.cap), so
// what counts there is the list that tiles of 128 would hold: whether a system
// fits does not depend on the tile (NARROW: tile < 128).
// A run reached across a periodic face holds images one box length away: its
// candidates are compared after that shift (d - s with s = +-L), which for
// every candidate within the list radius is the minimum image itself, with
// the same two roundings.
// s holds the records the reorder has just written in cell order (its
// candidates come from qid); the block also returns its particles' records
// and internal energies to the working buffer `work`.
constexpr int kPiece = 32;       // particles of a piece (a cell holds ~7 at density 3)
constexpr int kBuildChunks = 4;  // candidates per lane held at once
constexpr int kBuildWindow = kBuildChunks * kWave;
constexpr int kBuildMaxThreads = 1024;

// LDS of a block beyond its static arrays: the staged rows, and per wave a
// window's candidate indices and their stencil cells.
inline size_t build_lds(int rows, int threads) {
  return (size_t)rows * kUniqTile * sizeof(uint32_t) +
         (size_t)(threads / kWave) * kBuildWindow * (sizeof(uint32_t) + sizeof(uint8_t));
}

template <bool BATCH, bool UNIQ, bool NARROW>
__global__ __launch_bounds__(kBuildMaxThreads) void k_build_skin(
    PState s, PState work, const QIdF* __restrict__ qid, const uint32_t* __restrict__ start,
    int64_t n, const Geo* __restrict__ geo, double rs, double box_max, SkinList sl,
    const BuildCtl* ctl, double half_skin2, int rows, int tile, uint32_t limit, CellBins cells,
    uint32_t* status) {
  extern __shared__ uint32_t dyn[];  // see build_lds
  __shared__ uint32_t cell_s[kUniqTile];
  __shared__ int cx_s[kUniqTile], cy_s[kUniqTile], cz_s[kUniqTile];
  __shared__ int first_s[kUniqTile + 1];   // first particle of every piece
  __shared__ uint32_t count_s[kUniqTile];  // list lengths
  __shared__ unsigned long long head_s[2], piece_s[2];
  __shared__ int next_s;       // next piece to take
  __shared__ uint32_t most_s;  // longest list
  __shared__ uint32_t run_s, stop_s;
  if (threadIdx.x == 0) {
    run_s = rebuild_now(ctl, half_skin2);
    stop_s = *status;
    next_s = 0;
    most_s = 0u;
  }
  __syncthreads();
  // a status from before the binning kept that from running too
  if (!run_s || (stop_s & ~ST_OVERFLOW)) return;  // uniform in the block
  const int64_t tb = (int64_t)xcd_tile(blockIdx.x, gridDim.x) * kUniqTile;
  const int np = (int)(n - tb < kUniqTile ? n - tb : kUniqTile);
  const int t = threadIdx.x;
  uint32_t* lst = dyn;
  const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  uint32_t* src = dyn + rows * kUniqTile + w * kBuildWindow;  // the window's candidates
  uint8_t* src_cell = reinterpret_cast<uint8_t*>(dyn + rows * kUniqTile +
                                                 (blockDim.x / kWave) * kBuildWindow) +
                      w * kBuildWindow;
  const Rec* __restrict__ R = s.r + tb;
  // the tile's cells: a piece starts where the cell changes, and every kPiece
  // particles inside one
  if (t < kUniqTile) {
    uint32_t c = 0xFFFFFFFFu;
    if (t < np) {
      const Geo& g = geo[BATCH ? R[t].rep : 0u];
      const int cx = cell_coord(R[t].qx, g.scale[0], g.nc[0]);
      const int cy = cell_coord(R[t].qy, g.scale[1], g.nc[1]);
      const int cz = cell_coord(R[t].qz, g.scale[2], g.nc[2]);
      cx_s[t] = cx;
      cy_s[t] = cy;
      cz_s[t] = cz;
      c = (uint32_t)(g.cell_base + cell_key(g, cx, cy, cz));
    }
    cell_s[t] = c;
  }
  // records back to the working buffer, 16 bytes per thread and turn
  if (!stop_s) {
    for (int c = t; c < 4 * np; c += blockDim.x)
      reinterpret_cast<uint4*>(work.r + tb)[c] = reinterpret_cast<const uint4*>(R)[c];
    for (int c = t; c < np; c += blockDim.x) work.eps[tb + c] = s.eps[tb + c];
  }
  __syncthreads();
  const bool head = t < np && (t == 0 || cell_s[t] != cell_s[t - 1]);
  // the cells' histogram entries and chains cleared for the next build (start
  // stays), also where another block has found an overflow; by the tile's own
  // cells, since a sparse box has many more (the few blocks of 100 particles
  // took 560 us to clear its 6.9M)
  if (head) {
    cells.count[cell_s[t]] = 0u;
    cells.first[cell_s[t]] = kChainEnd;
  }
  if (stop_s) return;  // uniform in the block
  const unsigned long long heads = __ballot(head);
  if (w < 2 && lane == 0) head_s[w] = heads;
  __syncthreads();
  bool piece = false;
  if (t < np) {
    const unsigned long long own = head_s[w] & (~0ull >> (63 - lane));  // heads at or below t
    const int from = own ? kWave * w + 63 - __clzll(own) : 63 - __clzll(head_s[0]);
    // pieces of 8 where those of 32 would leave waves idle (few cells in the tile)
    const int cells_met = __popcll(head_s[0]) + __popcll(head_s[1]);
    const int per = cells_met + np / kPiece < (int)blockDim.x / kWave ? 8 : kPiece;
    piece = ((t - from) % per) == 0;
  }
  const unsigned long long pieces = __ballot(piece);
  if (w < 2 && lane == 0) piece_s[w] = pieces;
  __syncthreads();
  const int npieces = __popcll(piece_s[0]) + __popcll(piece_s[1]);
  if (piece) {
    const int before = (w ? __popcll(piece_s[0]) : 0) +
                       __popcll(pieces & ((1ull << lane) - 1ull));
    first_s[before] = t;
  }
  if (t == 0) first_s[npieces] = np;
  __syncthreads();
  const float thr2 = build_radius2(ctl, rs, box_max);
  const uint32_t cap = (uint32_t)sl.cap;
  for (;;) {
    int pc = 0;
    if (lane == 0) pc = atomicAdd(&next_s, 1);
    pc = __builtin_amdgcn_readfirstlane(pc);
    if (pc >= npieces) break;
    const int p0 = __builtin_amdgcn_readfirstlane(first_s[pc]);
    const int p1 = __builtin_amdgcn_readfirstlane(first_s[pc + 1]);
    const int cx = cx_s[p0], cy = cy_s[p0], cz = cz_s[p0];
    const Geo& g =
        geo[BATCH ? (uint32_t)__builtin_amdgcn_readfirstlane((int)R[p0].rep) : 0u];
    // lanes l and l + 32, l < 27: cell l of the stencil, its candidates and
    // its image
    const int cell = lane % 32;
    uint32_t cb = 0, cn = 0;
    float sx = 0.0f, sy = 0.0f, sz = 0.0f;
    if (cell < 27) {
      int x = cx + cell % 3 - 1, y = cy + (cell / 3) % 3 - 1, z = cz + cell / 9 - 1;
      auto image = [](int c, int nc, double l) {
        return c >= nc ? (float)l : (c < 0 ? -(float)l : 0.0f);
      };
      sx = image(x, g.nc[0], g.box[0]);
      sy = image(y, g.nc[1], g.box[1]);
      sz = image(z, g.nc[2], g.box[2]);
      if (wrap_cell(x, g.nc[0], g.periodic[0]) && wrap_cell(y, g.nc[1], g.periodic[1]) &&
          wrap_cell(z, g.nc[2], g.periodic[2])) {
        const int64_t c = g.cell_base + cell_key(g, x, y, z);
        cb = start[c];
        cn = start[c + 1] - cb;
      }
    }
    const bool images = __any(cn && (sx != 0.0f || sy != 0.0f || sz != 0.0f));
    uint32_t pre = cn;  // this cell's first candidate position (prefix over the half-wave)
#pragma unroll
    for (int off = 1; off < 32; off <<= 1) {
      const uint32_t up = (uint32_t)__shfl_up((int)pre, off, 32);
      if (cell >= off) pre += up;
    }
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)pre, 31);
    pre -= cn;
    const QIdF own = qid[tb + (lane < p1 - p0 ? p0 + lane : p0)];  // lane q: particle p0 + q
    uint32_t counts = 0;  // lane q: entries of particle p0 + q so far
    const uint32_t first = (uint32_t)g.first;
    for (uint32_t w0 = 0; w0 < total; w0 += kBuildWindow) {
      const uint32_t lo = pre > w0 ? pre : w0;
      const uint32_t hi = pre + cn < w0 + kBuildWindow ? pre + cn : w0 + kBuildWindow;
      // the cells' two lanes write the window's candidate indices in turn, but
      // all lanes together a crowded cell's (its two would take up to 128 turns;
      // with pieces of 8, 12,000 particles in one cell 2420 -> 895 us per build)
      const bool crowded = lo + 32u < hi;
      for (unsigned long long left = __ballot(crowded && lane < 32); left; left &= left - 1ull) {
        const int c = __builtin_ctzll(left);
        const uint32_t b = (uint32_t)__builtin_amdgcn_readlane((int)(cb - pre), c);
        const uint32_t end = (uint32_t)__builtin_amdgcn_readlane((int)hi, c);
        for (uint32_t f = (uint32_t)__builtin_amdgcn_readlane((int)lo, c) + lane; f < end;
             f += kWave) {
          src[f - w0] = b + f;
          if (images) src_cell[f - w0] = (uint8_t)c;  // uniform
        }
      }
      if (!crowded) {
        for (uint32_t f = lo + lane / 32; f < hi; f += 2) {
          src[f - w0] = cb + (f - pre);
          if (images) src_cell[f - w0] = (uint8_t)cell;  // uniform
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
      const uint32_t left = total - w0;  // uniform
      float qx[kBuildChunks], qy[kBuildChunks], qz[kBuildChunks];
      float ix[kBuildChunks], iy[kBuildChunks], iz[kBuildChunks];
      uint32_t row[kBuildChunks], rel[kBuildChunks];
      unsigned long long live[kBuildChunks], odd[kBuildChunks];
#pragma unroll
      for (int c = 0; c < kBuildChunks; ++c) {
        const uint32_t f = (uint32_t)(c * kWave + lane);
        const bool have = f < left;
        const uint32_t j = have ? src[f] : (uint32_t)tb;
        const QIdF cand = qid[j];
        qx[c] = cand.x;
        qy[c] = cand.y;
        qz[c] = cand.z;
        ix[c] = iy[c] = iz[c] = 0.0f;
        if (images) {  // uniform
          const int from = have ? src_cell[f] : 0;
          ix[c] = __shfl(sx, from, kWave);
          iy[c] = __shfl(sy, from, kWave);
          iz[c] = __shfl(sz, from, kWave);
        }
        row[c] = UNIQ ? j : first + cand.id;
        rel[c] = j - (uint32_t)tb;
        live[c] = __ballot(have);
        odd[c] = __ballot((rel[c] & 1u) != 0u);
      }
      // one particle against the window
      auto test = [&](int q, auto mi) {
        const float xi = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(own.x), q));
        const float yi = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(own.y), q));
        const float zi = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(own.z), q));
        uint32_t base = (uint32_t)__builtin_amdgcn_readlane((int)counts, q);
        const uint32_t tq = (uint32_t)(p0 + q);
#pragma unroll
        for (int c = 0; c < kBuildChunks; ++c) {
          if ((uint32_t)(c * kWave) >= left) break;  // uniform
          float dx = xi - qx[c], dy = yi - qy[c], dz = zi - qz[c];
          if constexpr (decltype(mi)::value) {
            dx -= ix[c];
            dy -= iy[c];
            dz -= iz[c];
          }
          unsigned long long m = __ballot((dx * dx + dy * dy) + dz * dz < thr2) & live[c];
          if constexpr (UNIQ) {
            // in the tile, the lower index lists a pair of different parity,
            // the higher one a pair of equal parity
            const unsigned long long out = __ballot((rel[c] ^ tq) >= (uint32_t)tile);
            const unsigned long long below = __ballot(rel[c] < tq), above = __ballot(rel[c] > tq);
            const unsigned long long same = (tq & 1u) ? odd[c] : ~odd[c];
            m &= out | (same & below) | (~same & above);
          } else {
            m &= __ballot(rel[c] != tq);
          }
          const uint32_t pos =
              __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                        __builtin_amdgcn_mbcnt_lo((uint32_t)m, base));
          base += (uint32_t)__popcll(m);
          if (base <= (uint32_t)rows) {  // uniform: every place is staged
            if (__builtin_amdgcn_inverse_ballot_w64(m)) lst[pos * kUniqTile + tq] = row[c];
          } else if (__builtin_amdgcn_inverse_ballot_w64(m)) {
            if (pos < (uint32_t)rows) lst[pos * kUniqTile + tq] = row[c];
            else if (pos < cap) sl.idx[list_entry(tb + tq, pos, sl.cap)] = row[c];
          }
        }
        counts = lane == q ? base : counts;
      };
      if (images) {
        for (int q = 0; q < p1 - p0; ++q) test(q, std::true_type{});
      } else {
        for (int q = 0; q < p1 - p0; ++q) test(q, std::false_type{});
      }
      __builtin_amdgcn_wave_barrier();  // the next window overwrites src
    }
    if (lane < p1 - p0) {
      if (counts > (NARROW ? cap : limit)) atomicOr(status, ST_OVERFLOW);
      counts = counts < cap ? counts : cap;
      count_s[p0 + lane] = counts;
      atomicMax(&most_s, counts);
    }
  }
  __syncthreads();
  const uint32_t most = most_s < (uint32_t)rows ? most_s : (uint32_t)rows;
  for (uint32_t c = t; c < most * kUniqTile; c += blockDim.x) {
    const uint32_t k = c / kUniqTile, p = c % kUniqTile;
    if ((int)p < np && k < count_s[p]) sl.idx[list_entry(tb + p, k, sl.cap)] = lst[c];
  }
  if (t < np) sl.count[tb + t] = count_s[t];
  if constexpr (NARROW) {
    if (most_s > limit) {  // uniform
      __threadfence_block();
      __syncthreads();  // the lists are written
      if (t < np && count_s[t] > limit &&
          listed_in_128(sl, tb + t, (int)count_s[t], 0, 1) > limit)
        atomicOr(status, ST_OVERFLOW);
    }
  }
}

// ---- the same lists where cells hold few particles ----------------------------
// With one or two particles to a cell a piece leaves most of its wave idle in the
// candidate tests and every particle pays for a stencil by itself.  There four
// lanes per particle walk the stencil each for their own particle (the rule
// stands at the launch).
// Up to two contiguous cell ranges along x for the stencil row (y, z).
struct Row {
  int a0, b0, a1, b1;  // inclusive cell x-ranges; a1 > b1 means "no second range"
};

__device__ __forceinline__ Row stencil_row(int cx, int nc, int periodic) {
  Row r;
  r.a1 = 1;
  r.b1 = 0;
  if (periodic) {
    if (cx == 0) { r.a0 = 0; r.b0 = 1; r.a1 = nc - 1; r.b1 = nc - 1; }
    else if (cx == nc - 1) { r.a0 = nc - 2; r.b0 = nc - 1; r.a1 = 0; r.b1 = 0; }
    else { r.a0 = cx - 1; r.b0 = cx + 1; }
  } else {
    r.a0 = cx > 0 ? cx - 1 : 0;
    r.b0 = cx < nc - 1 ? cx + 1 : nc - 1;
  }
  return r;
}

// Visit the 27-cell stencil.  Its cells come as runs of consecutive memory
// (three cells of an x-row in row-major order; one run per cell block an
// x-row crosses in blocked order; a periodic wrap splits a row), which the
// group first lists in LDS (`runs`: the runs' first indices, then their
// cumulative ends with the run's periodic image in the top bits); the
// group's lanes then take the concatenated candidates four at a time (lane
// sub takes position F + sub), so a trip is cut short only at the end of the
// stencil, not at the end of every run.  A run reached across a periodic face
// holds images one box length away: its candidates are compared after that
// shift (d - s with s = +-L), which for every candidate within the list
// radius is the minimum image itself, with the same two roundings.
// `sink(take, j, id_j)` is called on every trip, `take` being r^2 < thr2 and
// j != i; the trips are uniform across the group, so `sink` may ballot.
constexpr int kRunsMax = 28;  // runs per stencil: 9 rows x at most 3 pieces
constexpr int kRunEndBits = 26;  // cumulative end; above it 2 bits per axis: 1 = +L, 2 = -L

template <bool MI, typename Sink>
__device__ __forceinline__ bool scan_candidates(const Lanes& L, const Geo& g,
                                                const uint32_t* __restrict__ start,
                                                const QIdF* __restrict__ qid, float xi, float yi,
                                                float zi, int cx, int cy, int cz, float thr2,
                                                uint32_t* runs, Sink&& sink) {
  const float bx = (float)g.box[0], by = (float)g.box[1], bz = (float)g.box[2];
  // the runs, in stencil order (uniform across the group; lane 0 records)
  uint32_t nr = 0, tot = 0;
  bool whole = true;  // false: the stencil holds more candidates than the run ends can count
  constexpr uint32_t kEndMask = (1u << kRunEndBits) - 1u;
  auto add = [&](uint32_t jb, uint32_t je, uint32_t image) {
    if (je > jb && je - jb > kEndMask - tot) whole = false;
    if (je > jb && whole) {
      tot += je - jb;
      if (L.sub == 0) {
        runs[nr] = jb;
        runs[kRunsMax + nr] = tot | (image << kRunEndBits);
      }
      ++nr;
    }
  };
  // the image code of a neighbour cell index before wrapping: +L from above,
  // -L from below (2 bits)
  auto code = [](int c, int nc) -> uint32_t { return c >= nc ? 1u : (c < 0 ? 2u : 0u); };
  const Row row = stencil_row(cx, g.nc[0], g.periodic[0]);
  const int B = g.oblk;
  // the x image of the second range of a periodic row: the cell left of
  // cx = 0 or right of cx = nc - 1
  const uint32_t cx1 = cx == 0 ? 2u : 1u;
  for (int dz = -1; dz <= 1; ++dz) {
    int z = cz + dz;
    const uint32_t iz = code(z, g.nc[2]) << 4;
    if (!wrap_cell(z, g.nc[2], g.periodic[2])) continue;
    for (int dy = -1; dy <= 1; ++dy) {
      int y = cy + dy;
      const uint32_t iyz = iz | (code(y, g.nc[1]) << 2);
      if (!wrap_cell(y, g.nc[1], g.periodic[1])) continue;
      if (B == 1) {  // row-major cells: each x range is one run of memory
        const int64_t base = g.cell_base + (int64_t)g.nc[0] * (y + (int64_t)g.nc[1] * z);
        add(start[base + row.a0], start[base + row.b0 + 1], iyz);
        if (row.a1 <= row.b1) add(start[base + row.a1], start[base + row.b1 + 1], iyz | cx1);
      } else {
        // blocked order: an x range is one run per cell block it crosses
        auto xrun = [&](int a, int b, uint32_t image) {
          for (int x = a; x <= b;) {
            const int e = min(b, block_of(x, g) * B + B - 1);
            const int64_t k0 = g.cell_base + cell_key(g, x, y, z);
            add(start[k0], start[k0 + (e - x) + 1], image);
            x = e + 1;
          }
        };
        xrun(row.a0, row.b0, iyz);
        if (row.a1 <= row.b1) xrun(row.a1, row.b1, iyz | cx1);
      }
    }
  }
  // the group's lanes read what lane 0 wrote (one wave: a fence suffices)
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  auto shift = [](uint32_t c2, float l) { return c2 == 1u ? l : (c2 == 2u ? -l : 0.0f); };
  // lane-local cursor: run r covers concatenated positions [prev, end) and
  // holds images shifted by (sx, sy, sz)
  uint32_t r = 0, prev = 0, word = nr ? runs[kRunsMax] : 0u;
  uint32_t end = word & kEndMask;
  float sx = 0.0f, sy = 0.0f, sz = 0.0f;
  auto image = [&]() {
    if constexpr (MI) {
      const uint32_t c = word >> kRunEndBits;
      sx = shift(c & 3u, bx);
      sy = shift((c >> 2) & 3u, by);
      sz = shift(c >> 4, bz);
    }
  };
  image();
  for (uint32_t F = 0; F < tot; F += kSub) {
    const uint32_t f = F + L.sub;
    bool take = false;
    uint32_t j = 0, idj = 0;
    if (f < tot) {
      if (f >= end) {
        do {
          prev = end;
          ++r;
          word = runs[kRunsMax + r];
          end = word & kEndMask;
        } while (f >= end);
        image();
      }
      j = runs[r] + (f - prev);
      const QIdF c = qid[j];
      float dx = xi - c.x, dy = yi - c.y, dz = zi - c.z;
      if constexpr (MI) {
        dx -= sx;
        dy -= sy;
        dz -= sz;
      }
      idj = c.id;
      take = (dx * dx + dy * dy) + dz * dz < thr2 && j != (uint32_t)L.i;
    }
    sink(take, j, idj);
  }
  return whole;
}

__device__ __forceinline__ bool interior_dim(int c, int nc, int periodic) {
  // cells c-1..c+1 exist without wrapping
  return !periodic || (c >= 1 && c <= nc - 2);
}

// Lists, limit and the records returned as in k_build_skin.
constexpr int kBuildLds = 32;  // list entries per particle staged in LDS

template <bool BATCH, bool UNIQ, bool NARROW>
__global__ __launch_bounds__(kPairBlockMax) void k_build_lanes(
    PState s, PState work, const QIdF* __restrict__ qid, const uint32_t* __restrict__ start,
    int64_t n, const Geo* __restrict__ geo, double rs, double box_max, SkinList sl,
    const BuildCtl* ctl, double half_skin2, int tile, uint32_t limit, CellBins cells,
    uint32_t* status) {
  __shared__ uint32_t lst[kBuildLds * (kPairBlockMax / kSub)];
  __shared__ uint32_t runs_s[2 * kRunsMax * (kPairBlockMax / kSub)];
  const uint32_t st = *status;  // another block may find an overflow: uniform in the wave only
  if (!rebuild_now(ctl, half_skin2) || (st & ~ST_OVERFLOW)) return;
  const Lanes L = lanes();
  if (L.i >= n) return;  // uniform in the group
  uint32_t* runs = runs_s + 2 * kRunsMax * L.pib;
  const int64_t i = L.i;
  const Rec* __restrict__ R = s.r;
  const Geo& g = geo[BATCH ? R[i].rep : 0u];
  const int cx = cell_coord(R[i].qx, g.scale[0], g.nc[0]);
  const int cy = cell_coord(R[i].qy, g.scale[1], g.nc[1]);
  const int cz = cell_coord(R[i].qz, g.scale[2], g.nc[2]);
  if (L.sub == 0) {  // the cell cleared, as in k_build_skin
    const int64_t c = g.cell_base + cell_key(g, cx, cy, cz);
    cells.count[c] = 0u;
    cells.first[c] = kChainEnd;
  }
  if (st) return;
  if (L.sub == 0) {
    work.r[i] = R[i];
    work.eps[i] = s.eps[i];
  }
  const float thr2 = build_radius2(ctl, rs, box_max);
  const QIdF own = qid[i];
  uint32_t nn = 0;
  const uint32_t cap = (uint32_t)sl.cap;
  const uint32_t first = (uint32_t)g.first;
  auto sink = [&](bool take, uint32_t j, uint32_t idj) {
    if constexpr (UNIQ) {
      const uint32_t x = (uint32_t)i ^ j;
      const bool mine = (x & 1u) ? (uint32_t)i < j : (uint32_t)i > j;
      take = take && (x >= (uint32_t)tile || mine);
    }
    const uint32_t bits = group_ballot(L, take);
    if (take) {
      const uint32_t pos = nn + __popc(bits & ((1u << L.sub) - 1u));
      const uint32_t row = UNIQ ? j : first + idj;
      if (pos < (uint32_t)kBuildLds) lst[pos * L.ppb + L.pib] = row;
      else if (pos < cap) sl.idx[list_entry(i, pos, sl.cap)] = row;
    }
    nn += __popc(bits);
  };
  // waves whose particles all sit away from the periodic faces meet no
  // image across them
  const bool interior = interior_dim(cx, g.nc[0], g.periodic[0]) &&
                        interior_dim(cy, g.nc[1], g.periodic[1]) &&
                        interior_dim(cz, g.nc[2], g.periodic[2]);
  const bool whole =
      __all(interior)
          ? scan_candidates<false>(L, g, start, qid, own.x, own.y, own.z, cx, cy, cz, thr2, runs,
                                   sink)
          : scan_candidates<true>(L, g, start, qid, own.x, own.y, own.z, cx, cy, cz, thr2, runs,
                                  sink);
  // a stencil too full to count is a list overflow
  if (!whole || nn > (NARROW ? cap : limit)) {
    if (L.sub == 0) atomicOr(status, ST_OVERFLOW);
  }
  nn = nn < cap ? nn : cap;
  const uint32_t staged = nn < (uint32_t)kBuildLds ? nn : (uint32_t)kBuildLds;
  for (uint32_t k = L.sub; k < staged; k += kSub)
    sl.idx[list_entry(i, k, sl.cap)] = lst[k * L.ppb + L.pib];
  if (L.sub == 0) sl.count[i] = nn;
  if constexpr (NARROW) {
    if (nn > limit) {  // uniform in the group
      __threadfence_block();  // the list is written
      uint32_t listed = listed_in_128(sl, i, (int)nn, L.sub, kSub);
#pragma unroll
      for (int off = 1; off < kSub; off <<= 1)
        listed += (uint32_t)__shfl_xor((int)listed, off, kWave);
      if (listed > limit && L.sub == 0) atomicOr(status, ST_OVERFLOW);
    }
  }
}

// Sort each skin list by neighbour identifier and replace the identifier
// rows by memory indices (slot[row], written by the reorder).  One list per
// lane, held in registers padded with all-ones and sorted by a bitonic
// network of 32, 64 or (for long lists, MAXW = 128) 128 words (the wave's
// longest list picks the width; rows are unique, so the order is total).
// Longer lists are insertion-sorted in place in global memory.
template <int N>
__device__ __forceinline__ void bitonic_sort(uint32_t (&v)[N]) {
#pragma unroll
  for (int k = 2; k <= N; k <<= 1) {
#pragma unroll
    for (int j = k >> 1; j > 0; j >>= 1) {
#pragma unroll
      for (int e = 0; e < N; ++e) {
        const int l = e ^ j;
        if (l > e) {
          const uint32_t x = v[e], y = v[l];
          const bool up = (e & k) == 0;
          v[e] = up ? min(x, y) : max(x, y);
          v[l] = up ? max(x, y) : min(x, y);
        }
      }
    }
  }
}

template <int N>
__device__ __forceinline__ void sort_list_regs(const SkinList& sl, const uint32_t* __restrict__ slot,
                                               int64_t i, uint32_t nn) {
  uint32_t v[N];
  uint32_t* l = sl.idx + list_entry(i, 0, sl.cap);
#pragma unroll
  for (int k = 0; k < N; ++k) v[k] = (uint32_t)k < nn ? l[k * kRow] : 0xFFFFFFFFu;
  bitonic_sort<N>(v);
#pragma unroll
  for (int k = 0; k < N; ++k)
    if ((uint32_t)k < nn) l[k * kRow] = slot[v[k]];
}

template <int MAXW>
__global__ __launch_bounds__(256) void k_sort_skin(int64_t n, SkinList sl,
                                                   const uint32_t* __restrict__ slot,
                                                   const BuildCtl* ctl, double half_skin2,
                                                   const uint32_t* status) {
  if (status_set(status) || !rebuild_now(ctl, half_skin2)) return;  // uniform
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint32_t nn = i < n ? sl.count[i] : 0u;
  uint32_t wmax = nn;
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1)
    wmax = max(wmax, (uint32_t)__shfl_xor((int)wmax, off, kWave));
  if (i >= n || nn == 0) return;
  if (wmax <= 32u) {
    sort_list_regs<32>(sl, slot, i, nn);
  } else if (nn <= 64u && (MAXW == 64 || wmax <= 64u)) {
    sort_list_regs<64>(sl, slot, i, nn);
  } else if (MAXW >= 128 && nn <= 128u) {
    sort_list_regs<MAXW>(sl, slot, i, nn);
  } else {
    uint32_t* l = sl.idx + list_entry(i, 0, sl.cap);
    for (uint32_t m = 1; m < nn; ++m) {
      const uint32_t x = l[(int64_t)m * kRow];
      uint32_t q = m;
      while (q > 0) {
        const uint32_t y = l[(int64_t)(q - 1) * kRow];
        if (y <= x) break;
        l[(int64_t)q * kRow] = y;
        --q;
      }
      l[(int64_t)q * kRow] = x;
    }
    for (uint32_t m = 0; m < nn; ++m) l[(int64_t)m * kRow] = slot[l[(int64_t)m * kRow]];
  }
}

// Pass A: neighbour list of the step (skin entries with r < rc, in identifier
// order, staged in LDS and written out coalesced), forces
// F_i = -sum_j v'(r_ij) d_ij / r_ij, U_i = 1/2 sum_j v(r_ij) and the Laplacian
// share L_i = sum_j (v'' + 2 v'/r) (eq. Tcon); mode 1 also applies
// p += dt/2 F (end of velocity-Verlet).  v is the soft potential
// (a rc/2)(1 - r/rc)^2 or the splined LJ of eq. Ep.
template <bool BATCH, int PREC>
__global__ __launch_bounds__(kPairBlockMax) void k_pass_a(
    PState s, int64_t n, const Geo* __restrict__ geo, Phys P, int mode,
    double* __restrict__ Fx, double* __restrict__ Fy, double* __restrict__ Fz,
    double* __restrict__ Ui, double* __restrict__ Li, SkinList sl, NList nl, uint32_t* status) {
  __shared__ uint32_t lst[kListLds * (kPairBlockMax / kSub)];
  const Lanes L = lanes();
  if (L.i >= n) return;  // uniform in the group
  if (status_set(status)) return;
  const int64_t i = L.i;
  const Rec* __restrict__ R = s.r;
  const double xi = R[i].qx, yi = R[i].qy, zi = R[i].qz;
  const GeoRef<BATCH> g = geo[BATCH ? R[i].rep : 0u];
  const uint32_t ns = sl.count[i];
  const uint32_t cap = (uint32_t)P.cap;
  const bool mi = !__all(away_from_faces(g, P, xi, yi, zi));  // uniform in the wave
  uint32_t nn = 0;
  double fx = 0.0, fy = 0.0, fz = 0.0, u = 0.0, lap = 0.0;
  const float inv_rc_f = (float)P.inv_rc, a_f = (float)P.a;
  uint32_t jn = (uint32_t)L.sub < ns ? sl.idx[list_entry(i, L.sub, sl.cap)] : 0u;
  double qnx = 0.0, qny = 0.0, qnz = 0.0;
  if ((uint32_t)L.sub < ns) {
    qnx = R[jn].qx;
    qny = R[jn].qy;
    qnz = R[jn].qz;
  }
  for (uint32_t base = 0; base < ns; base += kSub) {
    const uint32_t k = base + L.sub;
    const uint32_t j = jn;
    const double qjx = qnx, qjy = qny, qjz = qnz;
    if (k + kSub < ns) {
      jn = sl.idx[list_entry(i, k + kSub, sl.cap)];
      qnx = R[jn].qx;
      qny = R[jn].qy;
      qnz = R[jn].qz;
    }
    bool take = false;
    double dx = 0.0, dy = 0.0, dz = 0.0, r2 = 0.0;
    if (k < ns) {
      separation_mi(g, mi, xi, yi, zi, qjx, qjy, qjz, dx, dy, dz);
      r2 = dist2(dx, dy, dz);
      take = r2 < P.rc2;
    }
    const uint32_t bits = group_ballot(L, take);
    const uint32_t c = __popc(bits);
    if (take) {
      const uint32_t pos = nn + __popc(bits & ((1u << L.sub) - 1u));
      if (pos < (uint32_t)kListLds) lst[pos * L.ppb + L.pib] = j;
      else if (pos < cap) nl.idx[list_entry(i, pos, nl.cap)] = j;
    }
    // the pair at list position p is summed by lane p mod kSub (as in passes
    // B and C), whichever lane tested it: lane sub owns rank r of this trip
    const uint32_t r = (uint32_t)(L.sub - (int)nn) & (uint32_t)(kSub - 1);
    uint32_t b = bits;
    for (uint32_t q = 0; q < r; ++q) b &= b - 1u;
    const int src = L.shift + (b ? __ffs(b) - 1 : 0);
    const double ox = __shfl(dx, src, kWave), oy = __shfl(dy, src, kWave);
    const double oz = __shfl(dz, src, kWave), orr = __shfl(r2, src, kWave);
    if (r < c) {
      if constexpr (PREC == PREC_F64) {
        const double ir = inv_sqrt_f64(orr);  // 0 at r = 0
        const double rr = orr * ir;
        double f;
        if (P.potential == 0) {
          const double w = 1.0 - rr * P.inv_rc;
          u += P.half_a_rc * w * w;
          f = P.a * w * ir;  // -v'(r)/r
          lap += ir > 0.0 ? P.a * P.inv_rc - 2.0 * P.a * w * ir : 0.0;
        } else {
          const double ir2 = ir * ir;
          const double s2 = P.r_lj2 * ir2;
          const double s6 = s2 * s2 * s2, s12 = s6 * s6;
          u += P.lj4e * (s12 - s6) - P.lj_vc - P.lj_dvc * (rr - P.rc);
          const double dv = -6.0 * P.lj4e * (2.0 * s12 - s6) * ir - P.lj_dvc;
          f = -dv * ir;
          lap += P.lj4e * (156.0 * s12 - 42.0 * s6) * ir2 + 2.0 * dv * ir;
        }
        fx += f * ox;
        fy += f * oy;
        fz += f * oz;
      } else {
        const float rr = __builtin_sqrtf((float)orr);
        const float ir = rr > 0.0f ? 1.0f / rr : 0.0f;
        float f;
        if (P.potential == 0) {
          const float w = 1.0f - rr * inv_rc_f;
          u += (double)((float)P.half_a_rc * w * w);
          f = a_f * w * ir;
          lap += (double)(rr > 0.0f ? a_f * inv_rc_f - 2.0f * a_f * w * ir : 0.0f);
        } else {
          const float ir2 = ir * ir;
          const float s2 = (float)P.r_lj2 * ir2;
          const float s6 = s2 * s2 * s2, s12 = s6 * s6;
          const float e4 = (float)P.lj4e;
          u += (double)(e4 * (s12 - s6) - (float)P.lj_vc - (float)P.lj_dvc * (rr - (float)P.rc));
          const float dv = -6.0f * e4 * (2.0f * s12 - s6) * ir - (float)P.lj_dvc;
          f = -dv * ir;
          lap += (double)(e4 * (156.0f * s12 - 42.0f * s6) * ir2 + 2.0f * dv * ir);
        }
        fx += (double)(f * (float)ox);
        fy += (double)(f * (float)oy);
        fz += (double)(f * (float)oz);
      }
    }
    nn += c;
  }
  fx = group_sum(fx);
  fy = group_sum(fy);
  fz = group_sum(fz);
  u = group_sum(u);
  lap = group_sum(lap);
  if (nn > cap) {
    if (L.sub == 0) atomicOr(status, ST_OVERFLOW);
    nn = cap;
  }
  const uint32_t staged = nn < (uint32_t)kListLds ? nn : (uint32_t)kListLds;
  for (uint32_t k = L.sub; k < staged; k += kSub)
    nl.idx[list_entry(i, k, nl.cap)] = lst[k * L.ppb + L.pib];
  if (L.sub == 0) {
    nl.count[i] = nn;
    Fx[i] = fx;
    Fy[i] = fy;
    Fz[i] = fz;
    Ui[i] = 0.5 * u;
    Li[i] = lap;
    if (mode) {
      Rec* W = s.r;
      W[i].px = W[i].px + P.half_dt * fx;
      W[i].py = W[i].py + P.half_dt * fy;
      W[i].pz = W[i].pz + P.half_dt * fz;
    }
  }
}

// ---------------------------------------------------------------------------
// The SER momentum increment of one pair as seen by particle i (eq. SER_p):
//   dp_ij = -gamma_ij chi v_ij dt + sigma sqrt(chi) G_ij sqrt(dt)
// with chi = w^2, w = 1 - r/rc, gamma_ij = (gamma kT/2)(1/T_i + 1/T_j) and
// G_ij = +G(lo,hi) for i = lo, -G(lo,hi) for i = hi.  Every factor is either
// symmetric in (i,j) or flips sign exactly, so the result for (j,i) is the
// exact negative.
// ---------------------------------------------------------------------------
struct PairOut {
  double dp[3];
  double gdotv;  // noise . velocity term of the SEM energy update
  double v2;     // squared velocity term of the SEM energy update
  double chi;
  double w;
  double gij;
};

// Model 1 (the original DPDE model, Sec. 2.1): friction and noise along
// e_ij = d_ij / r with one scalar normal xi_ij = xi_ji per pair,
//   dp_ij = (-gamma_ij chi (e_ij . v_ij) dt + sigma w xi_ij sqrt(dt)) e_ij,
// antisymmetric through e_ji = -e_ij; a coincident pair does not interact.
template <bool BATCH, int PREC, int MODEL>
__device__ __forceinline__ void ser_pair(const Phys& P, const Geo& g, double dx, double dy,
                                         double dz, double r2, double vx, double vy, double vz,
                                         double invT_sum, uint32_t idi, uint32_t idj,
                                         uint64_t step, PairOut& o) {
  const bool i_lo = idi < idj;
  uint32_t wd[4];
  pair_words<!BATCH>(g, i_lo ? idi : idj, i_lo ? idj : idi, step, wd);
  if constexpr (PREC == PREC_F64) {
    const double ir = inv_sqrt_f64(r2);
    const double r = r2 * ir;
    double w = 1.0 - r * P.inv_rc;
    const double gij = P.gkT_half * invT_sum;
    if constexpr (MODEL == 1) {
      if (!(r2 > 0.0)) w = 0.0;
      const double chi = w * w;
      const double ex = dx * ir, ey = dy * ir, ez = dz * ir;
      const double ev = ex * vx + ey * vy + ez * vz;
      const double xi = normal1_f64(wd);
      const double mag = -gij * chi * ev * P.dt + P.sigma * w * xi * P.sqrt_dt;
      o.dp[0] = mag * ex;
      o.dp[1] = mag * ey;
      o.dp[2] = mag * ez;
      o.gdotv = ev * xi;
      o.v2 = ev * ev;
      o.chi = chi;
      o.w = w;
      o.gij = gij;
      return;
    }
    const double chi = w * w;
    double G[3];
    box_muller_f64(wd, G);
    const double c1 = -gij * chi * P.dt;
    const double c2 = (i_lo ? P.sigma : -P.sigma) * w * P.sqrt_dt;
    o.dp[0] = c1 * vx + c2 * G[0];
    o.dp[1] = c1 * vy + c2 * G[1];
    o.dp[2] = c1 * vz + c2 * G[2];
    o.gdotv = (i_lo ? 1.0 : -1.0) * (G[0] * vx + G[1] * vy + G[2] * vz);
    o.v2 = vx * vx + vy * vy + vz * vz;
    o.chi = chi;
    o.w = w;
    o.gij = gij;
  } else {
    const float r = __builtin_sqrtf((float)r2);
    float w = 1.0f - r * (float)P.inv_rc;
    const float gij = (float)(P.gkT_half * invT_sum);
    const float v0 = (float)vx, v1 = (float)vy, v2 = (float)vz;
    if constexpr (MODEL == 1) {
      if (!(r > 0.0f)) w = 0.0f;
      const float chi = w * w;
      const float ir = r > 0.0f ? 1.0f / r : 0.0f;
      const float ex = (float)dx * ir, ey = (float)dy * ir, ez = (float)dz * ir;
      const float ev = ex * v0 + ey * v1 + ez * v2;
      const float xi = normal1_f32(wd);
      const float mag = -gij * chi * ev * (float)P.dt + (float)P.sigma * w * xi * (float)P.sqrt_dt;
      o.dp[0] = (double)(mag * ex);
      o.dp[1] = (double)(mag * ey);
      o.dp[2] = (double)(mag * ez);
      o.gdotv = (double)(ev * xi);
      o.v2 = (double)(ev * ev);
      o.chi = (double)chi;
      o.w = (double)w;
      o.gij = (double)gij;
      return;
    }
    const float chi = w * w;
    float G[3];
    box_muller_f32(wd, G);
    const float c1 = -gij * chi * (float)P.dt;
    const float c2 = (i_lo ? (float)P.sigma : -(float)P.sigma) * w * (float)P.sqrt_dt;
    o.dp[0] = (double)(c1 * v0 + c2 * G[0]);
    o.dp[1] = (double)(c1 * v1 + c2 * G[1]);
    o.dp[2] = (double)(c1 * v2 + c2 * G[2]);
    o.gdotv = (double)((i_lo ? 1.0f : -1.0f) * (G[0] * v0 + G[1] * v1 + G[2] * v2));
    o.v2 = vx * vx + vy * vy + vz * vz;
    o.chi = (double)chi;
    o.w = (double)w;
    o.gij = (double)gij;
  }
}

// dp_ij of neighbour j seen from the record of particle i.
template <bool BATCH, int PREC, int MODEL>
__device__ __forceinline__ void pair_from_records(const Phys& P, const Geo& g, bool mi,
                                                  const Rec& a, const Rec& b, uint64_t step,
                                                  double& vx, double& vy, double& vz,
                                                  PairOut& o) {
  double dx, dy, dz;
  separation_mi(g, mi, a.qx, a.qy, a.qz, b.qx, b.qy, b.qz, dx, dy, dz);
  const double r2 = dist2(dx, dy, dz);
  vx = a.px * P.inv_mass - b.px * P.inv_mass;
  vy = a.py * P.inv_mass - b.py * P.inv_mass;
  vz = a.pz * P.inv_mass - b.pz * P.inv_mass;
  ser_pair<BATCH, PREC, MODEL>(P, g, dx, dy, dz, r2, vx, vy, vz, a.invT + b.invT, a.id, b.id, step, o);
}

// Stored increments dp_ij: FP64, or FP32 for the FP32 pair terms, whose
// increments are FP32 values to begin with (exact either way).  They are
// written once and read once, so both go non-temporal: the stream does not
// evict the neighbour data the gathers of both sweeps reuse from L2.
// The x components of a row of 32 entries, then the y and the z components.
__device__ __forceinline__ int64_t dp_at(int64_t e) { return e + 2 * kRow * (e / kRow); }

template <int PREC>
__device__ __forceinline__ void store_dp(const NList& nl, int64_t e, double x, double y, double z) {
  if constexpr (PREC == PREC_F32) {
    float* d = reinterpret_cast<float*>(nl.de) + dp_at(e);
    __builtin_nontemporal_store((float)x, d);
    __builtin_nontemporal_store((float)y, d + kRow);
    __builtin_nontemporal_store((float)z, d + 2 * kRow);
  } else {
    double* d = nl.de + dp_at(e);
    __builtin_nontemporal_store(x, d);
    __builtin_nontemporal_store(y, d + kRow);
    __builtin_nontemporal_store(z, d + 2 * kRow);
  }
}

template <int PREC>
__device__ __forceinline__ void load_dp(const NList& nl, int64_t e, double& x, double& y,
                                        double& z) {
  if constexpr (PREC == PREC_F32) {
    const float* d = reinterpret_cast<const float*>(nl.de) + dp_at(e);
    x = (double)__builtin_nontemporal_load(d);
    y = (double)__builtin_nontemporal_load(d + kRow);
    z = (double)__builtin_nontemporal_load(d + 2 * kRow);
  } else {
    const double* d = nl.de + dp_at(e);
    x = __builtin_nontemporal_load(d);
    y = __builtin_nontemporal_load(d + kRow);
    z = __builtin_nontemporal_load(d + 2 * kRow);
  }
}

// h_i = (p_i + dp_i/2)/m packed in 24 bytes (gathered by sweep 2)
struct H3 {
  double x, y, z;
};

// ---------------------------------------------------------------------------
// Inverse temperature of the updated internal energy.
// ---------------------------------------------------------------------------
__device__ __forceinline__ double inv_temperature(const Phys& P, double eps, uint32_t* status) {
  if (P.eos == 0) return P.cv / eps;
  int it;
  const double th = theta_newton_dev(P, eps, theta_start_dev(P, eps), it);
  if (!(th > 0.0) || !isfinite(th)) atomicOr(status, ST_EOS);
  return 1.0 / th;
}

// Observables of a step (the energy of Sec. 2.1, the temperatures of
// Sec. 2.2) are sums over particles of
// U, K, sum eps, Px, Py, Pz, sum 1/T, |grad U|^2, Laplacian U, out-of-range count
constexpr int kStatVals = 10;
constexpr int kStatBad = 9;
constexpr int kRecLen = 12;  // record: U K sum-eps E Px Py Pz Tkin Tint n |gradU|^2 lapU

// The per-particle terms of those sums, defined once so that both producers
// of the partial sums give the same bits.
__device__ __forceinline__ double sq3(double x, double y, double z) {
  return x * x + y * y + z * z;
}
__device__ __forceinline__ double kinetic(double px, double py, double pz, double mass) {
  return sq3(px, py, pz) / (2.0 * mass);
}
// A value's fixed-point form; a value outside the range adds one to the
// out-of-range count instead (the record is then NaN).
__device__ __forceinline__ Fix stat_fix(double x, int& bad) {
  if (fabs(x) < 0x1p30) return fix_of(x);
  ++bad;
  return fix_zero();
}

// The end of a step fused into its last pair pass (sweep 2, or the one sweep
// of SEM): each block's partial sums of the finished step's observables, and
// the next step's kick and drift on the records it writes, with the maxima of
// that step's list-build decision.  Kicking requires the sums (the separate
// observables pass reads the records, which would then be kicked).  In a batch
// every replica holds at least a tile's particles, so a block spans at most
// two replicas.
struct StepTail {
  const double* Fx;  // F of the step (pass A)
  const double* Fy;
  const double* Fz;
  const double* Ui;  // per-particle shares of U and of its Laplacian
  const double* Li;
  const QIdF* ref;   // positions at the last list build (FP32)
  NextMax* next;     // the next step's maxima; the step's end moves them into the build control
  Fix* partials;     // kStatVals per slot, cleared by their reader
  int slots;         // slots per replica: tile t adds into slot t % slots of its replica(s)
  int stats;         // add the partial sums (kTailAll, or kTailNoTheta)
  int kick;          // kick and drift the written records
};
// Every sum, or all but that of 1/T: with the projection, which follows, sets
// the energies and temperatures anew.
constexpr int kTailAll = 1, kTailNoTheta = 2;

// Slots of the partial sums: tiles in flight together (consecutive ones) add
// into different slots, and the final pass reads two per lane; a batch's
// replicas take a few each.
constexpr int kTailSlots = 128;
constexpr int kTailSlotsPerReplica = 4;

// dst += v exactly, in any order of the adds to dst: the low words add
// modulo 2^64, and the add that wraps them (known from the old value the
// atomic returns) carries one into the high word.
__device__ __forceinline__ void fix_atomic_add(Fix* dst, Fix v) {
  unsigned long long* lo = reinterpret_cast<unsigned long long*>(&dst->lo);
  unsigned long long* hi = reinterpret_cast<unsigned long long*>(&dst->hi);
  const unsigned long long old = atomicAdd(lo, (unsigned long long)v.lo);
  const unsigned long long carry = (old + (unsigned long long)v.lo < old) ? 1ull : 0ull;
  const unsigned long long h = (unsigned long long)v.hi + carry;
  if (h) atomicAdd(hi, h);
}

// Waves of a sweep's block: a tile of T particles with LPP lanes each.
template <int T, int LPP>
constexpr int tile_waves() {
  return T * LPP / kWave;
}
constexpr int kBothWaves = kPairBlockMax / kWave;  // most waves of a both-sides block

// One sum over the wave's even lanes and another over its odd lanes (the
// butterfly rounds never pair an even lane with an odd one); lanes 0 and 1
// store them as values ke and ko of wave w.
template <int W>
__device__ __forceinline__ void wave_pair_sums(Fix f, Fix (*out)[W], int ke, int ko, int w) {
#pragma unroll
  for (int off = kWave / 2; off > 1; off >>= 1) {
    Fix b;
    b.lo = (uint64_t)__shfl_xor((long long)f.lo, off, kWave);
    b.hi = (int64_t)__shfl_xor((long long)f.hi, off, kWave);
    f = fix_add(f, b);
  }
  const int lane = threadIdx.x % kWave;
  if (lane == 0) out[ke][w] = f;
  if (lane == 1) out[ko][w] = f;
}

// The work of a StepTail in one block of at most W waves: two lanes of every
// particle, of which `ev` is the first (live is false on the others).
template <bool BATCH, int W>
struct TailSums {
  Fix (*stat)[kStatVals][W];  // LDS, a set of sums per replica met (two in a batch)
  uint32_t rep0 = 0u, rep1 = 0u;
  bool two = false, in0 = true, live = false, ev = true;
  int bad = 0, w = 0;

  // The block's particles are the slots first .. last; a batch's block: the
  // replica of its first particle (set 0) and, when the last one differs,
  // the next replica (set 1).
  __device__ __forceinline__ TailSums(const StepTail& tail, Fix (*lds)[kStatVals][W],
                                      const Rec* __restrict__ R, int64_t first, int64_t last,
                                      uint32_t rep, bool live_, bool ev_)
      : stat(lds), live(live_), ev(ev_), w(threadIdx.x / kWave) {
    if constexpr (BATCH) {
      if (tail.stats) {
        rep0 = R[first].rep;
        rep1 = R[last].rep;
      }
      two = rep1 != rep0;
      in0 = rep == rep0;
    }
  }

  __device__ __forceinline__ void add(Fix f, int ke, int ko) {
    wave_pair_sums(in0 ? f : fix_zero(), stat[0], ke, ko, w);
    if constexpr (BATCH) {
      if (two) wave_pair_sums(in0 ? fix_zero() : f, stat[1], ke, ko, w);
    }
  }

  // The particle's values but 1/T split over its two lanes (first lane: U,
  // sum eps, Py, |grad U|^2, later 1/T; second: K, Px, Pz, Laplacian U and
  // the particle's out-of-range count), each pair summed over the wave's
  // first and second lanes apart.
  __device__ __forceinline__ void state(const StepTail& tail, const Rec& o, double e,
                                        const double F[3], double mass, int64_t i) {
    auto put = [&](double xe, double xo, int ke, int ko) {
      add(live ? stat_fix(ev ? xe : xo, bad) : fix_zero(), ke, ko);
    };
    put(live && ev ? tail.Ui[i] : 0.0, kinetic(o.px, o.py, o.pz, mass), 0, 1);
    put(e, o.px, 2, 3);
    put(o.py, o.pz, 4, 5);
    put(sq3(F[0], F[1], F[2]), live && !ev ? tail.Li[i] : 0.0, 7, 8);
  }

  // 1/T and the out-of-range count, then the block's sums into its slot.
  // Every thread of the block calls (barrier).
  __device__ __forceinline__ void finish(const StepTail& tail, double inv_t, int64_t tile) {
    const Fix ft =
        live && ev && tail.stats == kTailAll ? stat_fix(inv_t, bad) : fix_zero();
    const int nbad = bad + __shfl_xor(bad, 1, kWave);  // both lanes of the particle
    add(ev ? ft : Fix{(uint64_t)(uint32_t)nbad, 0ll}, 6, kStatBad);
    __syncthreads();
    if (threadIdx.x < (two ? 2 : 1) * kStatVals) {
      const int set = threadIdx.x / kStatVals, k = threadIdx.x % kStatVals;
      const int nw = blockDim.x / kWave;
      Fix t = fix_zero();
#pragma unroll
      for (int q = 0; q < W; ++q)
        if (q < nw) t = fix_add(t, stat[BATCH ? set : 0][k][q]);
      const int64_t slot = (int64_t)(set ? rep1 : rep0) * tail.slots + tile % tail.slots;
      fix_atomic_add(&tail.partials[slot * kStatVals + k], t);
    }
  }
};

// The kick and drift of the record o (on its particle's own lane), and the
// wave's maxima into one of the slots, with its status: one address for all of
// them made the raises queue up behind each other (N = 65,536: sweep 2 23.9 us,
// 18.4 so).
template <bool BATCH>
__device__ __forceinline__ void tail_kick(const StepTail& tail, bool own, Rec& o,
                                          const double F[3], const Geo* __restrict__ geo,
                                          const Phys& P, int64_t i, int64_t tile) {
  double d2 = 0.0, qa = 0.0;
  NextMax* next = tail.next + tile % kNextSlots;
  if (own) {
    const GeoRef<BATCH> g = geo[BATCH ? o.rep : 0u];
    kick_record(o, F, g, P, 1, tail.ref, i, d2, qa, &next->status);
  }
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) d2 = fmax(d2, __shfl_xor(d2, off, kWave));
  if (threadIdx.x % kWave == 0) raise_max_bits(&next->dmax_bits, d2);
  if (__any(qa > 0.0)) {
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) qa = fmax(qa, __shfl_xor(qa, off, kWave));
    if (threadIdx.x % kWave == 0) raise_max_bits(&next->qmax_bits, qa);
  }
}

// Block status flag made uniform: one read, shared through LDS.
__device__ __forceinline__ bool block_status_set(const uint32_t* status, uint32_t* flag) {
  if (threadIdx.x == 0) *flag = *status;
  __syncthreads();
  return *flag != 0u;
}

// ---------------------------------------------------------------------------
// Pass B (SER sweep 1, and the whole SEM update of eq. SEM_fd).
// ---------------------------------------------------------------------------
// SCHEME = 1, SEM: the sweep is the whole update, so its particles' new records
// (p += dp, eps += d eps, the next 1/T_i where the EOS is inline) go to `out`
// here, and the end of the step with them; no pass rereads the records.
template <bool BATCH, int PREC, int SCHEME, int MODEL>
__global__ __launch_bounds__(kPairBlockMax)
__attribute__((amdgpu_waves_per_eu(SCHEME == 1 && PREC == PREC_F64 && MODEL == 0 && !BATCH ? 6 : 1, 8))) void k_pass_b(
    PState s, NList nl, int64_t n, const Geo* __restrict__ geo, Phys P,
    const uint64_t* __restrict__ d_step, Vec4* __restrict__ dpi, H3* __restrict__ hv, int store,
    int eos_inline, Rec* __restrict__ out, StepTail tail, uint32_t* status) {
  constexpr int kSets = SCHEME == 1 ? (BATCH ? 2 : 1) : 0;
  const Lanes L = lanes<kSubSer>();
  const bool live = L.i < n;  // uniform in the group
  if constexpr (SCHEME == 1) {
    __shared__ uint32_t st_flag;
    if (block_status_set(status, &st_flag)) return;  // uniform in the block
  } else {
    if (!live) return;
    if (status_set(status)) return;
  }
  const int64_t i = live ? L.i : n - 1;
  const uint64_t step = *d_step;
  const Rec* __restrict__ R = s.r;
  const Rec a = R[i];
  const GeoRef<BATCH> g = geo[BATCH ? a.rep : 0u];
  const bool mi = !__all(away_from_faces(g, P, a.qx, a.qy, a.qz));  // uniform in the wave
  const uint32_t nn = live ? nl.count[i] : 0u;
  const int64_t cap = nl.cap;
  double ax = 0.0, ay = 0.0, az = 0.0, de = 0.0;
  // no software pipeline: the registers a prefetched record would hold buy
  // one more wave per SIMD, which hides the gather latency better
  for (uint32_t k = L.sub; k < nn; k += kSubSer) {
    const int64_t e = list_entry(i, k, cap);
    const uint32_t j = nl.idx[e];
    const Rec b = R[j];
    double vx, vy, vz;
    PairOut o;
    pair_from_records<BATCH, PREC, MODEL>(P, g, mi, a, b, step, vx, vy, vz, o);
    ax += o.dp[0];
    ay += o.dp[1];
    az += o.dp[2];
    if (store) store_dp<PREC>(nl, e, o.dp[0], o.dp[1], o.dp[2]);
    if constexpr (SCHEME == 1) {
      de += 0.5 * (o.gij * o.v2 - P.dsigma2_m) * o.chi * P.dt -
            0.5 * P.sigma * o.w * o.gdotv * P.sqrt_dt;
    }
  }
  ax = group_sum<kSubSer>(ax);
  ay = group_sum<kSubSer>(ay);
  az = group_sum<kSubSer>(az);
  if constexpr (SCHEME == 1) {
    __shared__ Fix stat_s[kSets][kStatVals][kBothWaves];
    de = group_sum<kSubSer>(de);
    const bool own = live && L.sub == 0;
    Rec o = a;
    o.px += ax;
    o.py += ay;
    o.pz += az;
    const double e = s.eps[i] + de;
    const bool need_t = own && e > 0.0 && eos_inline;
    if (own) {
      s.eps[i] = e;
      if (!(e > 0.0)) atomicOr(status, ST_NEG_EINT);
    }
    const int64_t tile = L.i / L.ppb;  // uniform in the block
    const int64_t first = tile * L.ppb;
    TailSums<BATCH, kBothWaves> ts(tail, stat_s, R, first, (first + L.ppb < n ? first + L.ppb : n) - 1, a.rep,
                       live, L.sub == 0);
    double F[3] = {0.0, 0.0, 0.0};
    if (tail.stats || tail.kick) {
      F[0] = tail.Fx[i];
      F[1] = tail.Fy[i];
      F[2] = tail.Fz[i];
    }
    if (tail.stats) ts.state(tail, o, e, F, P.mass, i);  // uniform
    if (tail.kick) tail_kick<BATCH>(tail, own, o, F, geo, P, i, tile);  // uniform
    // the new 1/T_i once the record (with the old one) is written, so that
    // only e and i stay live across the EOS
    if (own) out[i] = o;
    double inv_t = o.invT;
    if (need_t) {
      inv_t = inv_temperature(P, e, status);
      out[i].invT = inv_t;
    }
    if (tail.stats) ts.finish(tail, inv_t, tile);  // uniform
  } else if (L.sub == 0) {
    dpi[i] = Vec4{ax, ay, az, 0.0};
    hv[i] = H3{fma(ax, P.inv_2m, a.px * P.inv_mass), fma(ay, P.inv_2m, a.py * P.inv_mass),
                 fma(az, P.inv_2m, a.pz * P.inv_mass)};
  }
}

// ---------------------------------------------------------------------------
// The SER sweeps with each pair inside a tile evaluated once.
//
// Tiles are 128 consecutive particles of the cell order (one block of the
// sweeps, two lanes per particle; smaller tiles with more lanes in small
// systems).  With cells of side rc + skin about half
// of all pairs join two particles of one tile.  Pass A leaves such a pair in
// the list of one of its particles only, so the sweeps evaluate it once:
// that particle adds the pair term to its own sum and, with an LDS atomic,
// to the partner's (negated in sweep 1, as dp_ji = -dp_ij exactly; unchanged
// in sweep 2, as the reinjection term is symmetric).  A pair joining two
// tiles stays in both lists and is evaluated for each particle, as before.
//
// The per-particle sums are exact integer sums of the terms rounded once to
// the grid 2^-46 (sums of 64-bit integers do not depend on the order of their
// terms).  A particle's sum is therefore the same bits whichever lane, wave
// or tile contributes each term, so trajectories still do not depend on the
// memory order, the neighbour-list skin, the rebuild schedule or the
// batching.  The conversion is exact-range for |term| < 32 (a momentum or
// energy increment of one pair in one step); a larger term stops the step
// with DPDE_ERANGE.
// ---------------------------------------------------------------------------
// Fixed-point pair sums.  x 2^46 is exact, and adding M = 1.5 2^52 rounds it
// to an integer held in the low mantissa bits while |x| < 32: the bit
// pattern of x 2^46 + M minus that of M is round(x 2^46).  A lane adds the
// raw bit patterns and subtracts count * M once at the end.  The range is
// tracked as the largest high word of |x| (a NaN or infinity exceeds it too).
constexpr long long kFixMagicBits = 0x4338000000000000ll;  // bits of 1.5 2^52
constexpr uint32_t kFixRangeHi = 0x40400000u;               // high word of 32.0

__device__ __forceinline__ long long pair_fix_raw(double x) {
  return __double_as_longlong(fma(x, 0x1p46, 0x1.8p52));
}

__device__ __forceinline__ void pair_fix_range(double x, uint32_t& hi_max) {
  hi_max = max(hi_max, (uint32_t)(__double_as_longlong(x) >> 32) & 0x7FFFFFFFu);
}

__device__ __forceinline__ double pair_fix_value(long long v) { return (double)v * 0x1p-46; }

// The same on the grid 2^-G (|x| < 2^(51-G)): pass A's forces and potential
// shares on 2^-40 (|term| < 2048), the Laplacian shares on 2^-30.
template <int G>
__device__ __forceinline__ long long fix_raw_g(double x) {
  return __double_as_longlong(fma(x, __builtin_ldexp(1.0, G), 0x1.8p52));
}
template <int G>
__device__ __forceinline__ double fix_value_g(long long v) {
  return (double)v * __builtin_ldexp(1.0, -G);
}
template <int G>
constexpr uint32_t fix_range_hi() {  // high word of 2^(51-G)
  return (uint32_t)(1023 + 51 - G) << 20;
}

// Particle j's place in the tile of T particles that starts at tb; T or more
// outside it.
__device__ __forceinline__ uint32_t in_tile(uint32_t j, int64_t tb) {
  return j - (uint32_t)tb;
}

// Conservative pair terms of one pair at squared distance r2 (r < rc), as
// seen by particle i: f * d_ij with f = -v'(r)/r, the potential v(r) and the
// Laplacian term v'' + 2 v'/r (eq. Tcon).  A coincident pair adds v(0) and
// no force.
template <int PREC>
__device__ __forceinline__ void pair_conservative(const Phys& P, double dx, double dy, double dz,
                                                  double r2, double& gx, double& gy, double& gz,
                                                  double& v, double& lap) {
  if constexpr (PREC == PREC_F64) {
    const double ir = inv_sqrt_f64(r2);  // 0 at r = 0
    const double rr = r2 * ir;
    double f;
    if (P.potential == 0) {
      const double w = 1.0 - rr * P.inv_rc;
      v = P.half_a_rc * w * w;
      f = P.a * w * ir;  // -v'(r)/r
      lap = ir > 0.0 ? P.a * P.inv_rc - 2.0 * P.a * w * ir : 0.0;
    } else {
      const double ir2 = ir * ir;
      const double s2 = P.r_lj2 * ir2;
      const double s6 = s2 * s2 * s2, s12 = s6 * s6;
      v = P.lj4e * (s12 - s6) - P.lj_vc - P.lj_dvc * (rr - P.rc);
      const double dv = -6.0 * P.lj4e * (2.0 * s12 - s6) * ir - P.lj_dvc;
      f = -dv * ir;
      lap = P.lj4e * (156.0 * s12 - 42.0 * s6) * ir2 + 2.0 * dv * ir;
    }
    gx = f * dx;
    gy = f * dy;
    gz = f * dz;
  } else {
    const float inv_rc_f = (float)P.inv_rc, a_f = (float)P.a;
    const float rr = __builtin_sqrtf((float)r2);
    const float ir = rr > 0.0f ? 1.0f / rr : 0.0f;
    float f;
    if (P.potential == 0) {
      const float w = 1.0f - rr * inv_rc_f;
      v = (double)((float)P.half_a_rc * w * w);
      f = a_f * w * ir;
      lap = (double)(rr > 0.0f ? a_f * inv_rc_f - 2.0f * a_f * w * ir : 0.0f);
    } else {
      const float ir2 = ir * ir;
      const float s2 = (float)P.r_lj2 * ir2;
      const float s6 = s2 * s2 * s2, s12 = s6 * s6;
      const float e4 = (float)P.lj4e;
      v = (double)(e4 * (s12 - s6) - (float)P.lj_vc - (float)P.lj_dvc * (rr - (float)P.rc));
      const float dv = -6.0f * e4 * (2.0f * s12 - s6) * ir - (float)P.lj_dvc;
      f = -dv * ir;
      lap = (double)(e4 * (156.0f * s12 - 42.0f * s6) * ir2 + 2.0f * dv * ir);
    }
    gx = (double)(f * (float)dx);
    gy = (double)(f * (float)dy);
    gz = (double)(f * (float)dz);
  }
}

// Pass A in the tile form: the tile's particles, four or eight lanes each, walk
// their skin lists (each pair inside the tile in one of them); every
// pair with r < rc goes to the work list of the step and its conservative
// terms are added once, in fixed point, to both particles (the partner's
// share through LDS when it lies in the tile; a pair joining two tiles is in
// both lists and adds to its own particle only).  Forces and potential shares
// (U_i = 1/2 sum_j v(r_ij)) on the grid 2^-g chosen from a (2^-46 for a < 16,
// 2^-45 for a = 25): the form is used with the soft potential, whose pair
// force and potential are bounded by a;
// the Laplacian shares, which grow as 1/r, in two words: the term on the grid
// 2^-20 and its remainder on 2^-50.  Mode 1 also applies p += dt/2 F (end of
// velocity-Verlet).
constexpr int kTileListLds = 16;  // work-list entries per particle staged in LDS
constexpr int kTileSkinLds = 28;  // skin-list entries per particle staged in LDS (a block loads every row)

// In a batch a wave walks its particles one replica at a time, with that
// replica's geometry uniform (in scalar registers).  Replicas of at least a
// wave's kWave / KS particles (SMALL false) let a wave meet at most two, walked in
// straight-line code; with smaller ones (SMALL) a loop takes as many as the
// wave meets, at the cost of registers.
// Tiles of T particles with KS lanes each (see TileShape in api.hip).
template <bool BATCH, int PREC, bool SMALL, int T, int KS>
__global__ __launch_bounds__(KS * T) __attribute__((
    amdgpu_waves_per_eu(T != kUniqTile ? 1 : BATCH && SMALL ? 4 : 6, 8))) void k_pass_a_uniq(
    PState s, int64_t n, const Geo* __restrict__ geo, Phys P, int mode,
    double* __restrict__ Fx, double* __restrict__ Fy, double* __restrict__ Fz,
    double* __restrict__ Ui, double* __restrict__ Li, SkinList sl, NList nl, uint32_t* status) {
  // staged skin entries per particle: whole trips of the KS lanes
  constexpr int kStage = (kTileSkinLds + KS - 1) / KS * KS;
  constexpr int GH = 20, GR = 50;
  const double fsc = P.fix_scale_f;  // forces and potential shares: grid 1/fsc
  auto fix_f = [&](double x) { return __double_as_longlong(fma(x, fsc, 0x1.8p52)); };
  __shared__ unsigned long long acc[6][T];  // Fx Fy Fz U Lhi Llo, two's complement
  __shared__ uint32_t lst[kTileListLds * T];
  __shared__ uint32_t skin[kStage * T];  // the tile's skin lists, entry-major
  __shared__ uint32_t st_flag;
  for (int c = threadIdx.x; c < 6 * T; c += blockDim.x) acc[c / T][c % T] = 0;
  if (block_status_set(status, &st_flag)) return;  // uniform in the block
  const int64_t tb = (int64_t)xcd_tile(blockIdx.x, gridDim.x) * T;
  {
    // the first kStage entries of every skin list of the tile, loaded
    // entry by entry (runs of kRow consecutive words), all loads in flight at once
    constexpr int kPer = kStage / KS;
    uint32_t v[kPer];
#pragma unroll
    for (int r = 0; r < kPer; ++r) {
      const int c = r * (KS * T) + threadIdx.x;
      const int k = min(c / T, (int)sl.cap - 1);  // inside the list
      const int t = c % T;
      const int64_t row = tb + t < n ? tb + t : n - 1;
      v[r] = sl.idx[list_entry(row, k, sl.cap)];
    }
#pragma unroll
    for (int r = 0; r < kPer; ++r) skin[r * (KS * T) + threadIdx.x] = v[r];
    __syncthreads();
  }
  const int pl = threadIdx.x / KS, sub = threadIdx.x % KS;
  const int shift = (threadIdx.x % kWave) & ~(KS - 1);
  const int64_t i = tb + pl;
  const bool live = i < n;
  const Rec* __restrict__ R = s.r;
  double xi = 0.0, yi = 0.0, zi = 0.0;
  uint32_t ns = 0, rep = 0u;
  if (live) {
    xi = R[i].qx;
    yi = R[i].qy;
    zi = R[i].qz;
    ns = sl.count[i];
    if constexpr (BATCH) rep = R[i].rep;
  }
  const uint32_t cap = (uint32_t)nl.cap;
  long long XF0 = 0, XF1 = 0, XF2 = 0, XU = 0, XLh = 0, XLl = 0;  // raw fixed-point words
  uint32_t terms = 0u;
  uint32_t hi_l = 0u;
  uint32_t nn = 0;
  // The walk of the lanes in `mine` over their lists, with the geometry g of
  // their replica uniform in the wave (every pair term is a fixed-point sum,
  // so splitting a wave between replicas leaves the results' bits alone).
  auto walk = [&](const Geo& g, bool mine) {
    const bool mi = !__all(!mine || away_from_faces(g, P, xi, yi, zi));  // uniform in the wave
    if (!mine) return;
    // one trip of the group over entries base + sub (uniform in the group)
    auto trip = [&](uint32_t k, uint32_t j, double qjx, double qjy, double qjz) {
      bool take = false;
      double dx = 0.0, dy = 0.0, dz = 0.0, r2 = 0.0;
      if (k < ns) {
        separation_mi(g, mi, xi, yi, zi, qjx, qjy, qjz, dx, dy, dz);
        r2 = dist2(dx, dy, dz);
        take = r2 < P.rc2;
      }
      const uint32_t bits = (uint32_t)(__ballot(take) >> shift) & ((1u << KS) - 1u);
      if (take) {
        const uint32_t pos = nn + __popc(bits & ((1u << sub) - 1u));
        if (pos < (uint32_t)kTileListLds) lst[pos * T + pl] = j;
        else if (pos < cap) nl.idx[list_entry(i, pos, nl.cap)] = j;
        double gx, gy, gz, v, lap;
        pair_conservative<PREC>(P, dx, dy, dz, r2, gx, gy, gz, v, lap);
        const long long f0 = fix_f(gx), f1 = fix_f(gy), f2 = fix_f(gz);
        const long long fu = fix_f(0.5 * v);
        // Laplacian term: 2^-20 grid, then the (exact) remainder on 2^-50
        const long long fh = fix_raw_g<GH>(lap);
        const double rem = lap - (double)(fh - kFixMagicBits) * 0x1p-20;
        const long long fr = fix_raw_g<GR>(rem);
        // forces and potential shares are within the grid's range by its
        // choice (|f d| <= a, v/2 <= a rc/4); the Laplacian share grows as 1/r
        pair_fix_range(lap, hi_l);
        XF0 += f0;
        XF1 += f1;
        XF2 += f2;
        XU += fu;
        XLh += fh;
        XLl += fr;
        ++terms;
        const uint32_t rel = in_tile(j, tb);
        if (rel < (uint32_t)T) {  // the partner's share of a pair inside the tile
          atomicAdd(&acc[0][rel], (unsigned long long)(kFixMagicBits - f0));
          atomicAdd(&acc[1][rel], (unsigned long long)(kFixMagicBits - f1));
          atomicAdd(&acc[2][rel], (unsigned long long)(kFixMagicBits - f2));
          atomicAdd(&acc[3][rel], (unsigned long long)(fu - kFixMagicBits));
          atomicAdd(&acc[4][rel], (unsigned long long)(fh - kFixMagicBits));
          atomicAdd(&acc[5][rel], (unsigned long long)(fr - kFixMagicBits));
        }
      }
      nn += __popc(bits);
    };
    // entries staged in LDS: the next trip's position is requested before
    // this trip's pair terms
    const uint32_t ns0 = ns < (uint32_t)kStage ? ns : (uint32_t)kStage;
    uint32_t jn = (uint32_t)sub < ns0 ? skin[sub * T + pl] : 0u;
    double qnx = 0.0, qny = 0.0, qnz = 0.0;
    if ((uint32_t)sub < ns0) {
      qnx = R[jn].qx;
      qny = R[jn].qy;
      qnz = R[jn].qz;
    }
    uint32_t base = 0;
    for (; base < ns0; base += KS) {
      const uint32_t k = base + sub;
      const uint32_t j = jn;
      const double qjx = qnx, qjy = qny, qjz = qnz;
      if (k + KS < ns0) {
        jn = skin[(k + KS) * T + pl];
        qnx = R[jn].qx;
        qny = R[jn].qy;
        qnz = R[jn].qz;
      }
      trip(k, j, qjx, qjy, qjz);
    }
    // longer lists: the rest from memory
    for (; base < ns; base += KS) {
      const uint32_t k = base + sub;
      uint32_t j = 0u;
      double qjx = 0.0, qjy = 0.0, qjz = 0.0;
      if (k < ns) {
        j = sl.idx[list_entry(i, k, sl.cap)];
        qjx = R[j].qx;
        qjy = R[j].qy;
        qjz = R[j].qz;
      }
      trip(k, j, qjx, qjy, qjz);
    }
  };
  if constexpr (BATCH && SMALL) {
    bool todo = live;
    while (__any(todo)) {
      const uint32_t r = (uint32_t)__builtin_amdgcn_readlane((int)rep, __builtin_ctzll(__ballot(todo)));
      const bool mine = todo && rep == r;
      walk(geo[r], mine);
      todo = todo && !mine;
    }
  } else if constexpr (BATCH) {
    // the wave's first replica, then the next one if the wave reaches it
    const uint32_t r0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)rep);
    walk(geo[r0], live && rep == r0);
    const bool rest = live && rep != r0;
    if (__any(rest)) {
      const uint32_t r1 = (uint32_t)__builtin_amdgcn_readlane((int)rep, __builtin_ctzll(__ballot(rest)));
      walk(geo[r1], rest);
    }
  } else {
    walk(geo[0], live);
  }
  const long long m = (long long)terms * kFixMagicBits;
  XF0 -= m;
  XF1 -= m;
  XF2 -= m;
  XU -= m;
  XLh -= m;
  XLl -= m;
#pragma unroll
  for (int off = 1; off < KS; off <<= 1) {
    XF0 += __shfl_xor(XF0, off, kWave);
    XF1 += __shfl_xor(XF1, off, kWave);
    XF2 += __shfl_xor(XF2, off, kWave);
    XU += __shfl_xor(XU, off, kWave);
    XLh += __shfl_xor(XLh, off, kWave);
    XLl += __shfl_xor(XLl, off, kWave);
  }
  if (hi_l >= fix_range_hi<GH>()) atomicOr(status, ST_RANGE);
  __syncthreads();
  if (!live) return;
  if (nn > cap) {
    if (sub == 0) atomicOr(status, ST_OVERFLOW);
    nn = cap;
  }
  const uint32_t staged = nn < (uint32_t)kTileListLds ? nn : (uint32_t)kTileListLds;
  for (uint32_t k = sub; k < staged; k += KS)
    nl.idx[list_entry(i, k, nl.cap)] = lst[k * T + pl];
  if (sub == 0) {
    const double fx = (double)(long long)((unsigned long long)XF0 + acc[0][pl]) * P.fix_inv_f;
    const double fy = (double)(long long)((unsigned long long)XF1 + acc[1][pl]) * P.fix_inv_f;
    const double fz = (double)(long long)((unsigned long long)XF2 + acc[2][pl]) * P.fix_inv_f;
    nl.count[i] = nn;
    Fx[i] = fx;
    Fy[i] = fy;
    Fz[i] = fz;
    Ui[i] = (double)(long long)((unsigned long long)XU + acc[3][pl]) * P.fix_inv_f;
    Li[i] = fix_value_g<GH>((long long)((unsigned long long)XLh + acc[4][pl])) +
            fix_value_g<GR>((long long)((unsigned long long)XLl + acc[5][pl]));
    if (mode) {
      Rec* W = s.r;
      W[i].px = W[i].px + P.half_dt * fx;
      W[i].py = W[i].py + P.half_dt * fy;
      W[i].pz = W[i].pz + P.half_dt * fz;
    }
  }
}

// A wave of the tile sweeps serves 64 / LPP particles, LPP lanes each.  The
// first kTileRegular entries of every list go through the lane-group loop; the
// entries beyond them, few and unevenly spread over the particles, are dealt
// evenly over all 64 lanes of the wave, so the wave does not wait for its
// longest list.
constexpr int kTileRegular = 8;

// The particle (within the wave's PW) of overflow item x: the last p with
// first[p] <= x, first[] ascending in LDS.
template <int PW>
__device__ __forceinline__ int overflow_owner(const uint32_t* first, uint32_t x) {
  int lo = 0, hi = PW - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (first[mid] <= x) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// Occupancy: the FP64 vector-model instance fits 6 waves per SIMD only when
// asked (77 VGPRs), the batched one, which holds its replica's geometry per
// lane, 5 (81; at 6 it spills), without spills; the FP32 and projected-model
// instances keep the compiler's choice.
template <bool BATCH, int PREC, int MODEL, int T, int LPP>
__global__ __launch_bounds__(LPP * T)
__attribute__((amdgpu_waves_per_eu(
    PREC == PREC_F64 && MODEL == 0 && LPP == 2 ? (BATCH ? 5 : 6) : 1, 8)))
void k_pass_b_uniq(
    PState s, NList nl, int64_t n, const Geo* __restrict__ geo, Phys P,
    const uint64_t* __restrict__ d_step, Vec4* __restrict__ dpi, H3* __restrict__ hv, int store,
    uint32_t* status) {
  // two's-complement sums in unsigned words (the atomic add is modular)
  __shared__ unsigned long long acc[3][T];
  constexpr int PW = kWave / LPP;
  __shared__ uint32_t first_s[tile_waves<T, LPP>()][PW];
  __shared__ uint32_t st_flag;
  for (int c = threadIdx.x; c < 3 * T; c += blockDim.x) acc[c / T][c % T] = 0;
  if (block_status_set(status, &st_flag)) return;  // uniform in the block
  const int64_t tb = (int64_t)xcd_tile(blockIdx.x, gridDim.x) * T;
  const int pl = threadIdx.x / LPP, sub = threadIdx.x % LPP;
  const int w = threadIdx.x / kWave;
  uint32_t* first = first_s[w];
  const int64_t i = tb + pl;
  const bool live = i < n;
  const uint64_t step = *d_step;
  const Rec* __restrict__ R = s.r;
  const int64_t cap = nl.cap;
  long long X0 = 0, X1 = 0, X2 = 0;  // raw sums of fixed-point bit patterns
  uint32_t terms = 0u;
  uint32_t hi_max = 0u;
  Rec a{};
  uint32_t nn = 0;
  bool away = true;
  if (live) {
    a = R[i];
    nn = nl.count[i];
    const GeoRef<BATCH> g = geo[BATCH ? a.rep : 0u];
    away = away_from_faces(g, P, a.qx, a.qy, a.qz);
  }
  const bool mi = !__all(away);  // uniform in the wave
  // the pair term of entry k (partner j) of particle ii (record ra): stored,
  // its share added to the partner inside the tile; returns the raw
  // fixed-point words
  auto term = [&](const Rec& ra, int64_t ii, uint32_t k, uint32_t j, long long& f0,
                  long long& f1, long long& f2) {
    const int64_t e = list_entry(ii, k, cap);
    const Rec b = R[j];
    const GeoRef<BATCH> g = geo[BATCH ? ra.rep : 0u];
    double vx, vy, vz;
    PairOut o;
    pair_from_records<BATCH, PREC, MODEL>(P, g, mi, ra, b, step, vx, vy, vz, o);
    if (store) store_dp<PREC>(nl, e, o.dp[0], o.dp[1], o.dp[2]);
    f0 = pair_fix_raw(o.dp[0]);
    f1 = pair_fix_raw(o.dp[1]);
    f2 = pair_fix_raw(o.dp[2]);
    pair_fix_range(o.dp[0], hi_max);
    pair_fix_range(o.dp[1], hi_max);
    pair_fix_range(o.dp[2], hi_max);
    const uint32_t rel = in_tile(j, tb);
    if (rel < (uint32_t)T) {  // the partner's share of a pair inside the tile
      atomicAdd(&acc[0][rel], (unsigned long long)(kFixMagicBits - f0));
      atomicAdd(&acc[1][rel], (unsigned long long)(kFixMagicBits - f1));
      atomicAdd(&acc[2][rel], (unsigned long long)(kFixMagicBits - f2));
    }
  };
  const uint32_t nreg = nn < (uint32_t)kTileRegular ? nn : (uint32_t)kTileRegular;
  // this lane's regular entries sub, sub + LPP, ...: every index load in
  // flight at once (addresses clamped to the list, so no load needs a branch)
  uint32_t jr[kTileRegular / LPP];
#pragma unroll
  for (int q = 0; q < kTileRegular / LPP; ++q) {
    const uint32_t k = (uint32_t)(sub + LPP * q);
    const uint32_t kc = k < nreg ? k : (nreg ? nreg - 1u : 0u);
    jr[q] = nreg ? nl.idx[list_entry(i, kc, cap)] : 0u;
  }
  for (int q = 0; q < kTileRegular / LPP; ++q) {
    const uint32_t k = (uint32_t)(sub + LPP * q);
    if (k >= nreg) break;
    long long f0, f1, f2;
    term(a, i, k, jr[q], f0, f1, f2);
    X0 += f0;
    X1 += f1;
    X2 += f2;
    ++terms;
  }
  // the entries beyond kTileRegular, dealt over the wave
  uint32_t total;
  const uint32_t extra = (sub == 0 && nn > (uint32_t)kTileRegular) ? nn - kTileRegular : 0u;
  const uint32_t pre = wave_prefix(extra, total);
  if (total) {  // uniform in the wave
    if (sub == 0) first[pl % PW] = pre;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    for (uint32_t x = threadIdx.x % kWave; x < total; x += kWave) {
      const int p = overflow_owner<PW>(first, x);
      const int slot = PW * w + p;
      const int64_t ii = tb + slot;
      const uint32_t k = (uint32_t)kTileRegular + (x - first[p]);
      const Rec ra = R[ii];
      long long f0, f1, f2;
      term(ra, ii, k, nl.idx[list_entry(ii, k, cap)], f0, f1, f2);
      atomicAdd(&acc[0][slot], (unsigned long long)(f0 - kFixMagicBits));
      atomicAdd(&acc[1][slot], (unsigned long long)(f1 - kFixMagicBits));
      atomicAdd(&acc[2][slot], (unsigned long long)(f2 - kFixMagicBits));
    }
  }
  X0 -= (long long)terms * kFixMagicBits;
  X1 -= (long long)terms * kFixMagicBits;
  X2 -= (long long)terms * kFixMagicBits;
#pragma unroll
  for (int off = 1; off < LPP; off <<= 1) {
    X0 += __shfl_xor(X0, off, kWave);
    X1 += __shfl_xor(X1, off, kWave);
    X2 += __shfl_xor(X2, off, kWave);
  }
  if (hi_max >= kFixRangeHi) atomicOr(status, ST_RANGE);
  __syncthreads();
  if (!live || sub) return;
  const double ax = pair_fix_value((long long)((unsigned long long)X0 + acc[0][pl]));
  const double ay = pair_fix_value((long long)((unsigned long long)X1 + acc[1][pl]));
  const double az = pair_fix_value((long long)((unsigned long long)X2 + acc[2][pl]));
  dpi[i] = Vec4{ax, ay, az, 0.0};
  hv[i] = H3{fma(ax, P.inv_2m, a.px * P.inv_mass), fma(ay, P.inv_2m, a.py * P.inv_mass),
             fma(az, P.inv_2m, a.pz * P.inv_mass)};
}

// ---------------------------------------------------------------------------
// Pass C (SER sweep 2): d eps_i = -1/2 sum_j dp_ij . (v_ij + (dp_i - dp_j)/(2m))
// in FP64 for both precisions, then p <- p + dp, eps <- eps + d eps and the
// next 1/T_i.  The new records go to `out`, never over the records this pass
// gathers from.
// ---------------------------------------------------------------------------
// THETA = 1: the surrogate network gives the next 1/T_i inside this pass
// (the learned-EOS modes): the block's particles put their inputs in LDS,
// one wave evaluates the network for all of them on the matrix cores, and
// each particle finishes as the stand-alone theta kernel does (Newton outside
// the training range).  The block therefore meets at barriers and takes no
// early exit before them.
template <bool BATCH, int PREC, int REGEN, int MODEL, int THETA>
__global__ __launch_bounds__(kPairBlockMax)
__attribute__((amdgpu_waves_per_eu(!REGEN && THETA ? 6 : 1, 8))) void k_pass_c(
    PState s, NList nl, int64_t n, const Geo* __restrict__ geo, Phys P,
    const uint64_t* __restrict__ d_step, const Vec4* __restrict__ dpi,
    const H3* __restrict__ hv, int eos_inline, MlpDev m, int mlp_mode, Rec* __restrict__ out,
    StepTail tail, uint32_t* status) {
  __shared__ float net_x[kPairBlockMax / kSubSer];
  __shared__ float net_y[kPairBlockMax / kSubSer];
  __shared__ Fix stat_s[BATCH ? 2 : 1][kStatVals][kBothWaves];
  __shared__ uint32_t st_flag;
  const Lanes L = lanes<kSubSer>();
  const bool live = L.i < n;  // uniform in the group
  if (block_status_set(status, &st_flag)) return;  // uniform in the block
  const int64_t i = live ? L.i : 0;
  double de = 0.0;
  Rec a{};
  Vec4 di{};
  if (live) {
    const uint64_t step = *d_step;
    const Rec* __restrict__ R = s.r;
    a = R[i];
    const GeoRef<BATCH> g = geo[BATCH ? a.rep : 0u];
    const bool mi = REGEN ? !__all(away_from_faces(g, P, a.qx, a.qy, a.qz)) : true;
    di = dpi[i];
    const H3 hi = hv[i];
    const uint32_t nn = nl.count[i];
    const int64_t cap = nl.cap;
    uint32_t jn = (uint32_t)L.sub < nn ? nl.idx[list_entry(i, L.sub, cap)] : 0u;
    double hx = 0.0, hy = 0.0, hz = 0.0;
    if ((uint32_t)L.sub < nn) {
      hx = hv[jn].x;
      hy = hv[jn].y;
      hz = hv[jn].z;
    }
    for (uint32_t k = L.sub; k < nn; k += kSubSer) {
      const int64_t e = list_entry(i, k, cap);
      const uint32_t j = jn;
      const double ux = hi.x - hx, uy = hi.y - hy, uz = hi.z - hz;
      if (k + kSubSer < nn) {
        jn = nl.idx[e + kSubSer * kRow];
        hx = hv[jn].x;
        hy = hv[jn].y;
        hz = hv[jn].z;
      }
      double ex, ey, ez;
      if constexpr (REGEN) {
        const Rec b = R[j];
        double vx, vy, vz;
        PairOut o;
        pair_from_records<BATCH, PREC, MODEL>(P, g, mi, a, b, step, vx, vy, vz, o);
        ex = o.dp[0];
        ey = o.dp[1];
        ez = o.dp[2];
      } else {
        load_dp<PREC>(nl, e, ex, ey, ez);
      }
      de += -0.5 * (ex * ux + ey * uy + ez * uz);
    }
    de = group_sum<kSubSer>(de);
  }
  const double e = live ? s.eps[i] + de : 1.0;
  // the particle's updated record, formed on both of its lanes; the first
  // lane writes it
  const bool own = live && L.sub == 0;
  bool need_t = false;
  Rec o = a;
  o.px = a.px + di.x;
  o.py = a.py + di.y;
  o.pz = a.pz + di.z;
  if (own) {
    s.eps[i] = e;
    if (!(e > 0.0)) {
      atomicOr(status, ST_NEG_EINT);
    } else {
      need_t = THETA || eos_inline;
    }
  }
  const int64_t tile = L.i / L.ppb;  // uniform in the block
  const int64_t first = tile * L.ppb;
  TailSums<BATCH, kBothWaves> ts(tail, stat_s, s.r, first, (first + L.ppb < n ? first + L.ppb : n) - 1, a.rep,
                     live, L.sub == 0);
  double F[3] = {0.0, 0.0, 0.0};
  if ((tail.stats || tail.kick) && live) {
    F[0] = tail.Fx[i];
    F[1] = tail.Fy[i];
    F[2] = tail.Fz[i];
  }
  if (tail.stats) ts.state(tail, o, e, F, P.mass, i);  // uniform
  if (tail.kick) tail_kick<BATCH>(tail, own, o, F, geo, P, i, tile);  // uniform
  // The record (with the old 1/T_i) is written before the EOS, so that only e
  // and i stay live across it; the new 1/T_i follows.
  if (own) out[i] = o;
  double inv_t = o.invT;
  if constexpr (THETA) {
    float y = 0.0f;
    if (mlp_mode != 0) {  // uniform
      if (L.sub == 0) net_x[L.pib] = mlp_input(m, e);
      __syncthreads();
      // wave w takes particles 32 w .. 32 w + 31 of the block
      const int w = threadIdx.x / kWave, col = threadIdx.x % 32;
      if (32 * w < L.ppb) {  // uniform in the wave
        const int p = 32 * w + col;
        const float yw = mlp_wave32(m.wf, m.wb, p < L.ppb ? net_x[p] : 0.0f);
        if (threadIdx.x % kWave < 32) net_y[p] = yw;
      }
      __syncthreads();
      y = net_y[L.pib];
    }
    if (need_t) {
      int it;
      const double th = theta_from_net(P, m, mlp_mode, e, y, it);
      if (!(th > 0.0) || !isfinite(th)) atomicOr(status, ST_EOS);
      inv_t = 1.0 / th;
      out[i].invT = inv_t;
    }
  } else if (need_t) {
    inv_t = inv_temperature(P, e, status);
    out[i].invT = inv_t;
  }
  if (tail.stats) ts.finish(tail, inv_t, tile);  // uniform
}

// Pass C over the tile's unique pairs: the reinjection term
//   e_ij = -1/2 dp_ij . (h_i - h_j),   h = (p + dp/2)/m
// is symmetric in (i, j), so a pair inside the tile adds the same e_ij to both
// internal energies (eq. SER_eint_discretization); then p <- p + dp,
// eps <- eps + d eps and the next 1/T_i as in k_pass_c (THETA = 1: the
// surrogate network inside the pass); with a StepTail also the observables'
// partial sums and the next step's kick.  Occupancy, with stored increments:
// the record is written before the EOS, so that neither the network nor the
// inline EOS (its exponentials) adds to the tail's registers, and 6 waves per
// SIMD fit without scratch (92 VGPRs and 5 waves with the record held across
// the inline EOS; 256 replicas: 174 -> 155 us).  The instances that regenerate the noise hold the pair term's
// registers as well and keep the compiler's choice (asked for 5 or 6 they
// spill).
template <bool BATCH, int PREC, int REGEN, int MODEL, int THETA, int T, int LPP>
__global__ __launch_bounds__(LPP * T)
__attribute__((amdgpu_waves_per_eu(REGEN || LPP != 2 ? 1 : 6, 8))) void k_pass_c_uniq(
    PState s, NList nl, int64_t n, const Geo* __restrict__ geo, Phys P,
    const uint64_t* __restrict__ d_step, const Vec4* __restrict__ dpi,
    const H3* __restrict__ hv, int eos_inline, MlpDev m, int mlp_mode, Rec* __restrict__ out,
    StepTail tail, uint32_t* status) {
  __shared__ unsigned long long acc[T];  // two's-complement sums (modular adds)
  __shared__ float net_x[T];
  __shared__ float net_y[T];
  constexpr int PW = kWave / LPP;
  constexpr int W = tile_waves<T, LPP>();
  __shared__ uint32_t first_s[W][PW];
  __shared__ double hs[3][T];  // the tile's h: partners inside the tile read it here
  __shared__ Fix stat_s[BATCH ? 2 : 1][kStatVals][W];
  __shared__ uint32_t st_flag;
  for (int c = threadIdx.x; c < T; c += blockDim.x) acc[c] = 0;
  const int64_t tb = (int64_t)xcd_tile(blockIdx.x, gridDim.x) * T;
  if (threadIdx.x < T && tb + threadIdx.x < n) {
    const H3 h = hv[tb + threadIdx.x];
    hs[0][threadIdx.x] = h.x;
    hs[1][threadIdx.x] = h.y;
    hs[2][threadIdx.x] = h.z;
  }
  if (block_status_set(status, &st_flag)) return;  // uniform in the block (and hs visible)
  const int pl = threadIdx.x / LPP, sub = threadIdx.x % LPP;
  const int w = threadIdx.x / kWave;
  uint32_t* first = first_s[w];
  const int64_t i = tb + pl;
  const bool live = i < n;
  const uint64_t step = *d_step;
  const Rec* __restrict__ R = s.r;
  const int64_t cap = nl.cap;
  long long X = 0;  // raw sum of fixed-point bit patterns
  uint32_t terms = 0u;
  uint32_t hi_max = 0u;
  Rec a{};
  Vec4 di{};
  uint32_t nn = 0;
  bool away = true;
  if (live) {
    a = R[i];
    di = dpi[i];
    nn = nl.count[i];
    if constexpr (REGEN) {
      const GeoRef<BATCH> g = geo[BATCH ? a.rep : 0u];
      away = away_from_faces(g, P, a.qx, a.qy, a.qz);
    }
  }
  const bool mi = REGEN ? !__all(away) : true;  // uniform in the wave
  // h_j of a partner: from LDS inside the tile, else from memory
  auto gather_h = [&](uint32_t j, double& x, double& y, double& z) {
    const uint32_t rel = in_tile(j, tb);
    if (rel < (uint32_t)T) {
      x = hs[0][rel];
      y = hs[1][rel];
      z = hs[2][rel];
    } else {
      const H3 h = hv[j];
      x = h.x;
      y = h.y;
      z = h.z;
    }
  };
  // e_ij of entry k of particle ii (record ra, h_i = hi), given the
  // partner's index j and h_j; its share added to the partner inside the tile
  // (dx, dy, dz: the stored increment when the caller has loaded it, with
  // `have`)
  auto term = [&](const Rec& ra, const H3& hi, int64_t ii, uint32_t k, uint32_t j, double hx,
                  double hy, double hz, bool have = false, double dx = 0.0, double dy = 0.0,
                  double dz = 0.0) -> long long {
    const int64_t e = list_entry(ii, k, cap);
    const double ux = hi.x - hx, uy = hi.y - hy, uz = hi.z - hz;
    double ex = dx, ey = dy, ez = dz;
    if constexpr (REGEN) {
      const Rec b = R[j];
      const GeoRef<BATCH> g = geo[BATCH ? ra.rep : 0u];
      double vx, vy, vz;
      PairOut o;
      pair_from_records<BATCH, PREC, MODEL>(P, g, mi, ra, b, step, vx, vy, vz, o);
      ex = o.dp[0];
      ey = o.dp[1];
      ez = o.dp[2];
    } else {
      if (!have) load_dp<PREC>(nl, e, ex, ey, ez);
    }
    const double eij = -0.5 * (ex * ux + ey * uy + ez * uz);
    const long long f = pair_fix_raw(eij);
    pair_fix_range(eij, hi_max);
    const uint32_t rel = in_tile(j, tb);
    if (rel < (uint32_t)T) atomicAdd(&acc[rel], (unsigned long long)(f - kFixMagicBits));
    return f;
  };
  if (live) {
    const H3 hi = hv[i];
    const uint32_t nreg = nn < (uint32_t)kTileRegular ? nn : (uint32_t)kTileRegular;
    // this lane's regular entries: every index load in flight at once, then
    // each partner's h requested one entry ahead
    uint32_t jr[kTileRegular / LPP];
#pragma unroll
    for (int q = 0; q < kTileRegular / LPP; ++q) {
      const uint32_t k = (uint32_t)(sub + LPP * q);
      const uint32_t kc = k < nreg ? k : (nreg ? nreg - 1u : 0u);
      jr[q] = nreg ? nl.idx[list_entry(i, kc, cap)] : 0u;
    }
    double hx = 0.0, hy = 0.0, hz = 0.0;
    double sx = 0.0, sy = 0.0, sz = 0.0;  // the stored increment, likewise one entry ahead
    if ((uint32_t)sub < nreg) {
      gather_h(jr[0], hx, hy, hz);
      if constexpr (!REGEN) load_dp<PREC>(nl, list_entry(i, sub, cap), sx, sy, sz);
    }
#pragma unroll
    for (int q = 0; q < kTileRegular / LPP; ++q) {
      const uint32_t k = (uint32_t)(sub + LPP * q);
      if (k >= nreg) break;
      const double cx = hx, cy = hy, cz = hz;
      const double ex = sx, ey = sy, ez = sz;
      if (q + 1 < kTileRegular / LPP && k + LPP < nreg) {
        gather_h(jr[q + 1], hx, hy, hz);
        if constexpr (!REGEN) load_dp<PREC>(nl, list_entry(i, k + LPP, cap), sx, sy, sz);
      }
      X += term(a, hi, i, k, jr[q], cx, cy, cz, !REGEN, ex, ey, ez);
      ++terms;
    }
  }
  // the entries beyond kTileRegular, dealt over the wave
  uint32_t total;
  const uint32_t extra = (sub == 0 && nn > (uint32_t)kTileRegular) ? nn - kTileRegular : 0u;
  const uint32_t pre = wave_prefix(extra, total);
  if (total) {  // uniform in the wave
    if (sub == 0) first[pl % PW] = pre;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    for (uint32_t x = threadIdx.x % kWave; x < total; x += kWave) {
      const int p = overflow_owner<PW>(first, x);
      const int slot = PW * w + p;
      const int64_t ii = tb + slot;
      const uint32_t k = (uint32_t)kTileRegular + (x - first[p]);
      const uint32_t j = nl.idx[list_entry(ii, k, cap)];
      const H3 hj = hv[j];
      const Rec ra = REGEN ? R[ii] : Rec{};
      const long long f = term(ra, hv[ii], ii, k, j, hj.x, hj.y, hj.z);
      atomicAdd(&acc[slot], (unsigned long long)(f - kFixMagicBits));
    }
  }
  X -= (long long)terms * kFixMagicBits;
#pragma unroll
  for (int off = 1; off < LPP; off <<= 1) X += __shfl_xor(X, off, kWave);
  if (hi_max >= kFixRangeHi) atomicOr(status, ST_RANGE);
  __syncthreads();
  const double de =
      live ? pair_fix_value((long long)((unsigned long long)X + acc[pl])) : 0.0;
  const double e = live ? s.eps[i] + de : 1.0;
  const bool own = live && sub == 0;
  bool need_t = false;
  // the particle's updated record, formed on all of its lanes; the first
  // lane writes it
  Rec o = a;
  o.px = a.px + di.x;
  o.py = a.py + di.y;
  o.pz = a.pz + di.z;
  if (own) {
    s.eps[i] = e;
    if (!(e > 0.0)) {
      atomicOr(status, ST_NEG_EINT);
    } else {
      need_t = THETA || eos_inline;
    }
  }
  const int64_t tile = tb / T;
  TailSums<BATCH, W> ts(tail, stat_s, R, tb, (tb + T < n ? tb + T : n) - 1, a.rep,
                        live && sub < 2, sub == 0);
  double F[3] = {0.0, 0.0, 0.0};
  if ((tail.stats || tail.kick) && live) {
    F[0] = tail.Fx[i];
    F[1] = tail.Fy[i];
    F[2] = tail.Fz[i];
  }
  if (tail.stats) ts.state(tail, o, e, F, P.mass, i);  // uniform
  if (tail.kick) tail_kick<BATCH>(tail, own, o, F, geo, P, i, tile);  // uniform
  // The record (with the old 1/T_i) is written before the EOS, so that only e
  // and i stay live across it; the new 1/T_i follows.
  if (own) out[i] = o;
  double inv_t = o.invT;
  if constexpr (THETA) {
    float y = 0.0f;
    if (mlp_mode != 0) {  // uniform
      if (sub == 0) net_x[pl] = mlp_input(m, e);
      __syncthreads();
      // wave w < 4 takes particles 32 w .. 32 w + 31 of the tile
      if (32 * w < T) {  // uniform in the wave
        const int col = threadIdx.x % 32;
        const float yw = mlp_wave32(m.wf, m.wb, net_x[32 * w + col]);
        if (threadIdx.x % kWave < 32) net_y[32 * w + col] = yw;
      }
      __syncthreads();
      y = net_y[pl];
    }
    if (need_t) {
      int it;
      const double th = theta_from_net(P, m, mlp_mode, e, y, it);
      if (!(th > 0.0) || !isfinite(th)) atomicOr(status, ST_EOS);
      inv_t = 1.0 / th;
      out[i].invT = inv_t;
    }
  } else if (need_t) {
    inv_t = inv_temperature(P, e, status);
    out[i].invT = inv_t;
  }
  if (tail.stats) ts.finish(tail, inv_t, tile);  // uniform
}

// 1/T_i for every particle (initialisation and the separate-EOS path).
__global__ void k_inv_temperature(PState s, int64_t n, Phys P, uint32_t* status) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double e = s.eps[i];
  if (!(e > 0.0)) {
    atomicOr(status, ST_NEG_EINT);
    return;
  }
  s.r[i].invT = inv_temperature(P, e, status);
}

// ---------------------------------------------------------------------------
// Observables: per-tile partial sums (k_stats_tiles, or the end of the tile
// sweep 2), then one block per replica, all in the fixed-point form above, so
// a record does not depend on the particles' memory order (list rebuild
// schedule, batching, resume).
// Record: U, K, sum eps, E, Px, Py, Pz, T_kin, T_int, step.
// ---------------------------------------------------------------------------
constexpr int kStatThreads = 512;

__global__ __launch_bounds__(kStatThreads) void k_stats_tiles(
    PState s, const double* __restrict__ Ui, const double* __restrict__ Li,
    const double* __restrict__ Fx, const double* __restrict__ Fy, const double* __restrict__ Fz,
    const int64_t* __restrict__ tile_begin, Phys P, Fix* __restrict__ partials) {
  const int64_t b = tile_begin[blockIdx.x], e = tile_begin[blockIdx.x + 1];
  Fix v[kStatVals];
#pragma unroll
  for (int k = 0; k < kStatVals; ++k) v[k] = fix_zero();
  for (int64_t i = b + threadIdx.x; i < e; i += blockDim.x) {
    const Rec& rc = s.r[i];
    const double px = rc.px, py = rc.py, pz = rc.pz;
    const double x[9] = {Ui[i], kinetic(px, py, pz, P.mass), s.eps[i], px, py, pz, rc.invT,
                         sq3(Fx[i], Fy[i], Fz[i]), Li[i]};
    int bad = 0;
#pragma unroll
    for (int k = 0; k < 9; ++k) v[k] = fix_add(v[k], stat_fix(x[k], bad));
    v[kStatBad] = fix_add(v[kStatBad], Fix{(uint64_t)(uint32_t)bad, 0ll});
  }
  __shared__ Fix smem[kStatVals * (kStatThreads / kWave)];
  block_sum_fix<kStatVals>(v, smem);
  if (threadIdx.x == 0)
    for (int k = 0; k < kStatVals; ++k) partials[blockIdx.x * kStatVals + k] = v[k];
}

// End of the step: count a list build, reset the build control for the next
// step, advance the step and history counters (nothing but the reset of the
// next step's maxima when the status is raised).  The
// counters' values were read before (no other block writes them).
struct StepNow {
  uint64_t step;
  int64_t hist;
  unsigned long long builds;
  unsigned long long next_d, next_q;  // the next step's maxima
  uint32_t next_status;               // and what its kick found wrong
  bool rebuilt, failed;
};

__device__ __forceinline__ void step_end(const StepNow& c, uint64_t* d_step, int64_t* d_hist_count,
                                         BuildCtl* ctl, unsigned long long* builds,
                                         uint32_t* status, int advance) {
  if (c.failed) return;
  if (c.rebuilt) *builds = c.builds + 1ull;
  // the next step's maxima (nonzero when its kick ran at the end of this
  // step's last pair pass) become the build control
  ctl->dmax_bits = c.next_d;
  ctl->force = 0u;
  ctl->qmax_bits = c.next_q;
  if (advance) {
    *d_step = c.step + 1;
    *d_hist_count = c.hist + 1;
  }
  if (c.next_status) atomicOr(status, c.next_status);  // the next step is the one that fails
}

// The slots' maxima by the first wave (non-negative doubles order like their bits).
__device__ __forceinline__ void next_maxima(StepNow& c, const NextMax* next) {
  const NextMax v = next[threadIdx.x];
  c.next_d = v.dmax_bits;
  c.next_q = v.qmax_bits;
  c.next_status = v.status;
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) {
    const unsigned long long d = __shfl_xor(c.next_d, off, kWave);
    const unsigned long long q = __shfl_xor(c.next_q, off, kWave);
    c.next_d = d > c.next_d ? d : c.next_d;
    c.next_q = q > c.next_q ? q : c.next_q;
    c.next_status |= (uint32_t)__shfl_xor((int)c.next_status, off, kWave);
  }
}

// Per replica: sum the tile partials, write the record (and the history
// row).  The slots that a step's last pair pass adds into are left zero
// (kClearAll), or, before the projection, only the sums that it takes anew
// (kClearEnergy: sum eps and sum 1/T).  With `finish`, the last block to complete also ends the step: a
// ticket taken after each block's reads of the step and history counters
// tells it that every other block is done with them.
constexpr int kStatFinalThreads = kStatVals * kWave;  // one wave per recorded sum
enum : int { kClearNone = 0, kClearAll = 1, kClearEnergy = 2 };
// Only the block that ends the step needs the next step's maxima.  Up to this
// many replicas every block requests them before its sums; with more the last
// one does after them (3000 replicas: 9 us less, few ones: 0.6 us more).
constexpr unsigned kFewReplicas = 64;

__global__ __launch_bounds__(kStatFinalThreads) void k_stats_final(
    Fix* __restrict__ partials, int clear, const int32_t* __restrict__ rep_tile0,
    const Geo* __restrict__ geo, uint64_t* d_step, int advance,
    double* __restrict__ rec, double* __restrict__ hist, int64_t hist_cap,
    int64_t* d_hist_count, int nrep, int finish, uint32_t* ticket, BuildCtl* ctl,
    NextMax* next, unsigned long long* builds, double half_skin2, uint32_t* status) {
  const int r = blockIdx.x;
  const int t0 = rep_tile0[r], t1 = rep_tile0[r + 1];
  // the values the record and the end of the step need, requested before
  // the reduction so that their latency overlaps it
  StepNow now{*d_step, *d_hist_count, 0ull, 0ull, 0ull, 0u, false, false};
  if (finish) {
    now.builds = *builds;
    now.rebuilt = rebuild_now(ctl, half_skin2);
    now.failed = status_set(status);
    if (gridDim.x <= kFewReplicas && threadIdx.x < kWave) next_maxima(now, next);
  }
  const double N = (double)geo[r].n;
  // wave k adds value k over the replica's tiles
  const int k0 = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  // eight partials per lane in flight, then their slots zeroed where asked
  constexpr int kAhead = 8;
  const bool zero = clear == kClearAll || (clear == kClearEnergy && (k0 == 2 || k0 == 6));
  Fix acc = fix_zero();
  for (int tb = t0 + lane; tb < t1; tb += kAhead * kWave) {
    Fix v[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int t = tb + u * kWave;
      v[u] = t < t1 ? partials[t * kStatVals + k0] : fix_zero();
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) acc = fix_add(acc, v[u]);
    if (zero) {
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const int t = tb + u * kWave;
        if (t < t1) partials[t * kStatVals + k0] = fix_zero();
      }
    }
  }
  acc = wave_sum_fix(acc);
  __shared__ Fix tot[kStatVals];
  uint32_t ends = 0u;  // (first lane) this block ends the step
  if (lane == 0) tot[k0] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    Fix f[kStatVals];
    for (int k = 0; k < kStatVals; ++k) f[k] = tot[k];
    const bool bad = f[kStatBad].lo != 0ull || f[kStatBad].hi != 0ll;
    double v[9];
    for (int k = 0; k < 9; ++k) v[k] = bad ? __builtin_nan("") : fix_to_double(f[k]);
    double o[kRecLen];
    o[0] = v[0];
    o[1] = v[1];
    o[2] = v[2];
    o[3] = v[0] + v[1] + v[2];
    o[4] = v[3];
    o[5] = v[4];
    o[6] = v[5];
    o[7] = 2.0 * v[1] / (3.0 * (N - 1.0));
    o[8] = N / v[6];
    o[9] = (double)(now.step + (uint64_t)advance);
    o[10] = v[7];
    o[11] = v[8];
    double* hrow = nullptr;
    if (advance) hrow = hist + ((now.hist % hist_cap) * nrep + r) * kRecLen;
    for (int k = 0; k < kRecLen; ++k) {
      rec[r * kRecLen + k] = o[k];
      if (hrow) hrow[k] = o[k];
    }
    if (finish) {
      // one replica: this block is the last one, and the end of the kernel
      // publishes its writes (no device-wide fence needed)
      if (gridDim.x > 1u) __threadfence();
      if (gridDim.x == 1u || atomicAdd(ticket, 1u) == gridDim.x - 1u) {
        if (gridDim.x > 1u) __threadfence();
        if (gridDim.x <= kFewReplicas)
          step_end(now, d_step, d_hist_count, ctl, builds, status, advance);
        atomicExch(ticket, 0u);
        ends = 1u;
      }
    }
  }
  // the first wave alone waits for the ticket and clears the slots (one a lane)
  if (!finish || threadIdx.x >= kNextSlots) return;
  if (__builtin_amdgcn_readfirstlane((int)ends)) {
    if (gridDim.x > kFewReplicas) {
      next_maxima(now, next);
      if (threadIdx.x == 0) step_end(now, d_step, d_hist_count, ctl, builds, status, advance);
    }
    next[threadIdx.x].dmax_bits = 0ull;  // the slots are left cleared
    next[threadIdx.x].qmax_bits = 0ull;
    next[threadIdx.x].status = 0u;
  }
}

// Projection on the internal energies (Sec. 4.2): eps_i <- eps_i - (E - E0)/N
// per replica, E from the record of the unconstrained update, then the new
// 1/T_i when the EOS is evaluated inline.  With `slots` (where the step's last
// pair pass has added the other sums) each wave also adds the new sum eps and
// sum 1/T of its particles, so that no further pass over the records is
// needed; a batch's replicas then hold at least a tile, so a wave meets at
// most two of them.
template <bool BATCH>
__global__ void k_project(PState s, int64_t n, const Geo* __restrict__ geo, Phys P,
                          const double* __restrict__ rec, const double* __restrict__ E0,
                          int eos_inline, Fix* __restrict__ partials, int slots,
                          uint32_t* status) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (status_set(status)) return;  // another block may raise it: uniform in the wave only
  const bool live = i < n;
  uint32_t r = 0u;
  double e = 0.0, inv_t = 0.0;
  if (live) {
    r = BATCH ? s.r[i].rep : 0u;
    const double shift = (rec[r * kRecLen + 3] - E0[r]) / (double)geo[r].n;
    e = s.eps[i] - shift;
    s.eps[i] = e;
    if (!(e > 0.0)) {
      atomicOr(status, ST_NEG_EINT);
    } else if (eos_inline) {
      inv_t = inv_temperature(P, e, status);
      s.r[i].invT = inv_t;
    }
  }
  if (!slots) return;  // uniform
  int bad = 0;
  const Fix fe = live ? stat_fix(e, bad) : fix_zero(), ft = live ? stat_fix(inv_t, bad) : fix_zero();
  const int lane = threadIdx.x % kWave;
  const int64_t wave = i / kWave;
  auto sums = [&](bool mine, uint32_t rep) {
    const Fix z = fix_zero();
    const Fix se = wave_sum_fix(mine ? fe : z), st = wave_sum_fix(mine ? ft : z),
              sb = wave_sum_fix(mine ? Fix{(uint64_t)(uint32_t)bad, 0ll} : z);
    Fix* p = partials + ((int64_t)rep * slots + wave % slots) * kStatVals;
    if (lane == 0) fix_atomic_add(p + 2, se);
    if (lane == 1) fix_atomic_add(p + 6, st);
    if (lane == 2 && (sb.lo | (uint64_t)sb.hi)) fix_atomic_add(p + kStatBad, sb);
  };
  if constexpr (BATCH) {
    const uint32_t r0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)r);
    sums(live && r == r0, r0);
    const bool rest = live && r != r0;
    const unsigned long long others = __ballot(rest);
    if (others) sums(rest, (uint32_t)__builtin_amdgcn_readlane((int)r, __builtin_ctzll(others)));
  } else {
    sums(live, 0u);
  }
}

// After a call whose failing step's last pair pass kicked the records it wrote
// (to `out`, from `src`): the state goes back to that step.  A record that the
// pass wrote is where its own momentum takes it from the step's position; it
// gets that position and the momentum before the kick again (p + dp_i of the
// sweeps; SEM, which keeps no dp_i: by the kick backwards, to rounding).  The
// pass leaves out the particles of blocks that already met the raised status:
// they keep the record it read.
__global__ void k_unkick(Rec* out, const Rec* __restrict__ src, const Vec4* __restrict__ dpi,
                         const double* __restrict__ Fx, const double* __restrict__ Fy,
                         const double* __restrict__ Fz, int64_t n, const Geo* __restrict__ geo,
                         Phys P) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const Rec o = out[i];
  Rec a = src[i];
  const Geo& g = geo[a.rep];
  double q[3] = {drifted(a.qx, o.px, P), drifted(a.qy, o.py, P), drifted(a.qz, o.pz, P)};
#pragma unroll
  for (int d = 0; d < 3; ++d)
    if (g.periodic[d]) q[d] = wrap_coord(q[d], g.box[d]);
  if (o.id == a.id && o.rep == a.rep && o.qx == q[0] && o.qy == q[1] && o.qz == q[2]) {
    if (dpi) {
      a.px = a.px + dpi[i].x;
      a.py = a.py + dpi[i].y;
      a.pz = a.pz + dpi[i].z;
    } else {
      a.px = o.px - P.half_dt * Fx[i];
      a.py = o.py - P.half_dt * Fy[i];
      a.pz = o.pz - P.half_dt * Fz[i];
    }
    a.invT = o.invT;
  }
  out[i] = a;
}

// Target energy of the projection: the energy in the current record.
__global__ void k_capture_e0(const double* __restrict__ rec, double* __restrict__ E0, int nrep) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r < nrep) E0[r] = rec[r * kRecLen + 3];
}

// ---------------------------------------------------------------------------
// Test hooks.
// ---------------------------------------------------------------------------
__global__ void k_debug_cells(PState s, int64_t n, const Geo* __restrict__ geo, int32_t* out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const Rec& rc = s.r[i];
  const Geo& g = geo[rc.rep];
  const int cx = cell_coord(rc.qx, g.scale[0], g.nc[0]);
  const int cy = cell_coord(rc.qy, g.scale[1], g.nc[1]);
  const int cz = cell_coord(rc.qz, g.scale[2], g.nc[2]);
  out[g.first + rc.id] = cx + g.nc[0] * (cy + g.nc[1] * cz);
}

// The identifier row (replica's first row + ID) of the particle in every
// memory slot.
__global__ void k_debug_order(PState s, int64_t n, const Geo* __restrict__ geo, int32_t* out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const Rec& rc = s.r[i];
  out[i] = (int32_t)(geo[rc.rep].first + rc.id);
}

// Every pair of the lists once, as (lower id, higher id) rows.  A pair
// joining two tiles is in both lists (taken from the lower identifier); with
// the tile work lists (tile > 0) a pair inside a tile is in one list only.
__global__ void k_debug_pairs(PState s, NList nl, int64_t n, const Geo* __restrict__ geo,
                              int tile, int32_t* out, int64_t cap,
                              unsigned long long* counter) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const Rec& a = s.r[i];
  const Geo& g = geo[a.rep];
  for (uint32_t k = 0; k < nl.count[i]; ++k) {
    const uint32_t j = nl.idx[list_entry(i, k, nl.cap)];
    const uint32_t idj = s.r[j].id;
    const bool once = ((uint32_t)i ^ j) < (uint32_t)tile;
    if (once || a.id < idj) {
      const unsigned long long slot = atomicAdd(counter, 1ull);
      if ((int64_t)slot < cap) {
        out[2 * slot] = (int32_t)(g.first + (a.id < idj ? a.id : idj));
        out[2 * slot + 1] = (int32_t)(g.first + (a.id < idj ? idj : a.id));
      }
    }
  }
}

__global__ void k_debug_rng(uint32_t key0, uint32_t key1, uint64_t step,
                            const uint32_t* __restrict__ lo, const uint32_t* __restrict__ hi,
                            int64_t n, uint32_t* raw, double* g, float* g32) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  Geo geo;
  geo.key0 = key0;
  geo.key1 = key1;
  uint32_t w[4];
  pair_words<true>(geo, lo[k], hi[k], step, w);
  if (raw)
    for (int c = 0; c < 4; ++c) raw[4 * k + c] = w[c];
  if (g) {
    double G[3];
    box_muller_f64(w, G);
    for (int c = 0; c < 3; ++c) g[3 * k + c] = G[c];
  }
  if (g32) {
    float G[3];
    box_muller_f32(w, G);
    for (int c = 0; c < 3; ++c) g32[3 * k + c] = G[c];
  }
}

}  // namespace dpde
