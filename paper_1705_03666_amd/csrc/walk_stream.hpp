// The forward walk (values only) as a stream of paths through a wavefront,
// shared by the single-problem kernel k_walk_fwd below and the heterogeneous
// batch (walk_batch.hip).
//
// One path per lane.  A wavefront takes work items (a node and a range of
// its paths) from the queue and hands the paths out to its lanes in order; a
// lane whose path has ended takes the next path of the stream, whichever item
// that belongs to, so lanes stay busy until the queue is empty (they used to
// idle while each item's last paths ended, about five mean path lengths an
// item: a quarter of the time at 1024 paths an item).
//
// Order of the sums.  Paths end in any order, but an item's statistics are
// sums over its paths in path order, so they depend neither on the schedule
// nor on what else the wavefront ran.  An ended path's value goes to its
// place in a ring of kRing positions in LDS; the open items leave the ring
// first in, first out, 64 paths at a time once all 64 are there, path p0 + k
// of the item being added to lane k mod 64's shifted FP64 sums.  A path more
// than kRing positions behind the newest one stops the hand-out until it has
// ended: with 1024 positions and 64 lanes that is a path of 15 mean lengths.
//
// Draining.  When the queue is empty and at most a quarter (half, where a
// path's draws allow it) of the lanes still run a path, the idle lanes draw for
// the running ones: the generator is counter-based, so a path's next L blocks
// are drawn by L lanes at once, pass through LDS, and the path's own lane is
// left with the steps.  What bounds a
// small call (and the end of a large one) is the longest path's chain of
// dependent instructions, most of which are the ten Philox rounds and
// Box-Muller: 7 nodes x 300 paths on an interval took 300 cycles a step of
// the longest path with every lane on its own, 43 this way.
//
// Measured (MI355X, whole calls, before -> after this design): 4096 nodes
// over 8 subdomain shapes, budgets 1e3..1e5, dt 1e-3: 27.6 -> 21.4 ms; ball
// with cubic killing and source, 4096 x 1e4: 31.5 -> 26.2 ms; disk with terms,
// 256 x 1e4, dt 1e-4: 47.9 -> 33.5 ms; 7 x 300 on an interval: 377 -> 83 us.
#pragma once
#ifndef __HIPCC_RTC__
#include <hip/hip_runtime.h>
#endif

#include "pdd_device.hpp"
#include "walk_kernels.hpp"

namespace pdd {

// Ring positions per wavefront and open items.  FP64 values take twice the
// LDS, so their ring is half as long.
template <typename R>
constexpr int stream_ring() { return sizeof(R) == 4 ? 1024 : 512; }
constexpr int kOpenItems = 8;
// a record's ring position and open-item index share one word
constexpr uint32_t kPosBits = 28, kPosMask = (1u << kPosBits) - 1u;

// Exit record fields: X, with killing or a source Y and Z, and as words the
// tag (position, item) and the step count with the censored bit on top.
template <typename R, int DIM, bool YZ>
constexpr int stream_rec_bytes() { return (DIM + (YZ ? 2 : 0)) * kWave * (int)sizeof(R) + 2 * kWave * 4; }
// The Gaussians in LDS: the 64 blocks that the lanes draw for the remaining
// paths share the records' area (the records are flushed before); heavy steps
// (ROLL, see stream_walk) read every group's Gaussians from there, next to
// the records.
template <typename R, int DIM, int LAYOUT, bool YZ, bool ROLL>
constexpr int stream_area_bytes() {
  using NZr = Normals<R, LAYOUT>;
  constexpr int rec = stream_rec_bytes<R, DIM, YZ>();
  constexpr int z = kWave * (int)sizeof(R) * (ROLL ? GroupShape<DIM, NZr::kPerBlock>::NZ : NZr::kPerBlock);
  return ROLL ? rec + z : (rec > z ? rec : z);
}

struct OpenItem {
  uint32_t base, count, p0;
  int32_t node, slot;
  uint32_t cens;
  unsigned long long steps;
};

template <typename R, int AREA>
struct StreamLds {
  R ring[stream_ring<R>()];
  uint32_t have[stream_ring<R>() / 32];
  OpenItem open[kOpenItems];
  __attribute__((aligned(16))) unsigned char area[AREA];
};

// Philox counters of one path: (block, 0, path, node) -- the second word,
// block >> 32, is zero for every step count a path can reach.  Of the first
// three rounds, everything that depends on the path and the node alone is
// kept per lane, so a block takes 18 products instead of 20, and its first
// three rounds read no scalar register.
struct PathKey {
  uint32_t d1, b1, c1, c3;
};

constexpr uint32_t kPhM0 = 0xD2511F53u, kPhM1 = 0xCD9E8D57u, kPhW0 = 0x9E3779B9u, kPhW1 = 0xBB67AE85u;

__device__ __forceinline__ PathKey path_key(uint32_t path, uint32_t node, uint32_t k0, uint32_t k1) {
  const uint64_t p = (uint64_t)kPhM1 * (uint64_t)path;
  const uint32_t a = (uint32_t)(p >> 32) ^ k0;
  const uint64_t q = (uint64_t)kPhM0 * (uint64_t)a;
  PathKey k;
  k.d1 = node ^ k1;
  k.b1 = (uint32_t)p ^ (k0 + kPhW0);
  k.c1 = (uint32_t)(q >> 32) ^ (k1 + kPhW1);
  k.c3 = (uint32_t)q ^ (k1 + 2u * kPhW1);
  return k;
}

// The four words of block `blk` of a path: philox4x32_10(blk, 0, path, node).
__device__ __forceinline__ void path_block(const PathKey& K, uint32_t blk, uint32_t k0, uint32_t k1, uint32_t* w) {
  const uint64_t p = (uint64_t)kPhM0 * (uint64_t)blk;
  const uint32_t n2 = (uint32_t)(p >> 32) ^ K.d1;
  const uint64_t q = (uint64_t)kPhM1 * (uint64_t)n2;
  const uint32_t c0 = (uint32_t)(q >> 32) ^ K.b1;
  const uint32_t c2 = K.c1 ^ (uint32_t)p;
  const uint64_t p0 = (uint64_t)kPhM0 * (uint64_t)c0;
  const uint64_t p1 = (uint64_t)kPhM1 * (uint64_t)c2;
  w[0] = xor3((uint32_t)(p1 >> 32), (uint32_t)q, k0 + 2u * kPhW0);
  w[1] = (uint32_t)p1;
  w[2] = (uint32_t)(p0 >> 32) ^ K.c3;
  w[3] = (uint32_t)p0;
  k0 += 3u * kPhW0;
  k1 += 3u * kPhW1;
#pragma unroll
  for (int r = 3; r < 10; ++r) {
    const uint64_t a = (uint64_t)kPhM0 * (uint64_t)w[0];
    const uint64_t b = (uint64_t)kPhM1 * (uint64_t)w[2];
    w[0] = xor3((uint32_t)(b >> 32), w[1], k0);
    w[2] = xor3((uint32_t)(a >> 32), w[3], k1);
    w[1] = (uint32_t)b;
    w[3] = (uint32_t)a;
    k0 += kPhW0;
    k1 += kPhW1;
  }
}

template <typename R, int LAYOUT, bool LIBM>
__device__ __forceinline__ void path_normals(const PathKey& K, uint32_t blk, uint32_t k0, uint32_t k1, R* z) {
  uint32_t w[4];
  // opaque copies of the key: the round keys are rebuilt with scalar adds at
  // each use instead of living in registers
  uint32_t ka = k0, kb = k1;
  asm volatile("" : "+s"(ka), "+s"(kb));
  path_block(K, blk, ka, kb, w);
  Normals<R, LAYOUT, LIBM>::from_words(w, z);
}

// compile-time truth values, as arguments of generic lambdas
struct Yes { static constexpr bool value = true; };
struct No { static constexpr bool value = false; };

// What a launch gives every wavefront besides its problem.
struct StreamArgs {
  const WorkItem* items;
  int n_items;
  uint32_t* qhead;
  ItemStat* istat;
  double* dump_phi;
  int64_t* dump_steps;
  const int64_t* dump_off;
  uint32_t k0, k1;
  int refill_groups;
};

// Runs the items of one problem's queue to its end.  The launch's (or the
// problem's) first n_first wavefronts start with the item of their own number
// `first` (none if it is n_first), the rest of the queue is popped: with one
// item per wavefront or less, the queue's atomic, on which all wavefronts
// would otherwise start (70000 cycles for 2500 of them), is not touched.  PROB
// gives the problem:
//   kWos, kFree (pure diffusion: b = c = f = 0), kYZ (records carry Y and Z),
//   kRoll (heavy steps: one copy of the step's code, in a loop that reads its
//   Gaussians from LDS; unrolled, FP64 steps with generic terms took 90 KB of
//   code and 250 VGPRs);
//   start(node, x): the node's coordinates;  max_steps;  D: the domain
//   inside(x): the exit test, and Extremes, the same test for several
//   positions at once;  distance(x): to the boundary of D
//   sdt: sigma sqrt(dt);  dt: the step, or the shell width of walk on spheres
//   step(X, Y, Z, z): one Euler step with drift, killing and source
//   g(x): the boundary data
template <typename R, int DIM, int LAYOUT, class PROB, class LDS>
__device__ __forceinline__ void stream_walk(const PROB& prob, const StreamArgs& A, LDS* L, int lane, uint32_t first,
                                            uint32_t n_first) {
  using NZr = Normals<R, LAYOUT>;
  using GS = GroupShape<DIM, NZr::kPerBlock>;
  constexpr int PB = NZr::kPerBlock;
  constexpr int kRing = stream_ring<R>();
  constexpr bool kYZ = PROB::kYZ;
  // the area is reused with other types: every access may alias
  typedef R __attribute__((may_alias)) Ra;
  typedef uint32_t __attribute__((may_alias)) Ua;
  Ra* const rec = (Ra*)L->area;
  Ua* const rec_tag = (Ua*)(L->area + (DIM + (kYZ ? 2 : 0)) * kWave * sizeof(R));
  Ua* const rec_n = rec_tag + kWave;
  Ra* const zbuf = (Ra*)(L->area + (PROB::kRoll ? stream_rec_bytes<R, DIM, kYZ>() : 0));
  // pure diffusion: steps taken as one unit while draining
  constexpr int kFreeUnit = sizeof(R) == 4 ? (DIM == 1 ? 16 : (DIM == 2 ? 8 : 4))
                                           : (DIM == 1 ? 8 : (DIM == 2 || PB == 4 ? 4 : 2));
  // lanes that may still run a path when the draining starts: each of them
  // needs at least one group's (one unit's) blocks drawn at once
  constexpr int kDrain = kWave / (GS::NB > 2 || PROB::kFree ? 4 : 2);
  const uint32_t max_steps = prob.max_steps;

  // ring and open items (scalars)
  uint32_t next_pos = 0, tail = 0;       // positions handed out / retired
  int open_head = 0, open_n = 0;
  uint32_t h_row = 0;                    // paths of the head item retired
  int nrec = 0;
  // the item being handed out
  bool more = true;
  int c_node = 0, c_idx = 0;
  uint32_t c_path = 0, c_left = 0;
  R x0[DIM];
  bool c_in = false;
  // per lane: sums of the head item's values (shift = the lane's first)
  double sk = 0.0, s1 = 0.0, s2 = 0.0;
  // per lane: the path
  R X[DIM], Y = (R)1, Z = (R)0;
#pragma unroll
  for (int k = 0; k < DIM; ++k) X[k] = x0[k] = (R)0;
  PathKey key{0u, 0u, 0u, 0u};
  uint32_t n = 0, tag = 0;
  bool alive = false, fin = false, cens = false;

  for (int i = lane; i < kRing / 32; i += kWave) L->have[i] = 0u;
  __builtin_amdgcn_wave_barrier();

  // Adds up the head items' paths that have all arrived, 64 at a time.
  auto retire = [&]() {
    while (open_n > 0) {
      const OpenItem& it = L->open[open_head];
      const uint32_t base = (uint32_t)__builtin_amdgcn_readfirstlane((int)it.base);
      const uint32_t count = (uint32_t)__builtin_amdgcn_readfirstlane((int)it.count);
      const uint32_t left = count - h_row;
      const bool in = (uint32_t)lane < left;
      const uint32_t at = (base + h_row + (uint32_t)lane) & (uint32_t)(kRing - 1);
      const bool here = ((L->have[at >> 5] >> (at & 31u)) & 1u) != 0u;
      if (!__all(!in || here)) break;
      if (in) {
        const double v = (double)L->ring[at];
        sk = h_row == 0 ? v : sk;
        const double dv = v - sk;
        s1 += dv;
        s2 += dv * dv;
        atomicAnd(&L->have[at >> 5], ~(1u << (at & 31u)));
      }
      __builtin_amdgcn_wave_barrier();
      const uint32_t m = left < (uint32_t)kWave ? left : (uint32_t)kWave;
      tail += m;
      h_row += m;
      if (h_row < count) continue;
      // the item is complete: its statistics
      const uint32_t cnt = count / (uint32_t)kWave + ((uint32_t)lane < count % (uint32_t)kWave ? 1u : 0u);
      double wn = (double)cnt, wmean = 0.0, wm2 = 0.0;
      if (cnt > 0u) {
        const double a = s1 / wn;
        wmean = sk + a;
        wm2 = s2 - s1 * a;
        wm2 = wm2 < 0.0 ? 0.0 : wm2;
      }
      wave_welford(wn, wmean, wm2);
      if (lane == 0) {
        ItemStat st;
        st.mean = wmean;
        st.m2 = wm2;
        st.n = (int64_t)count;
        st.steps = (int64_t)it.steps;
        st.censored = (int64_t)it.cens;
        st.redrawn = 0;
        A.istat[it.slot] = st;
      }
      __builtin_amdgcn_wave_barrier();
      sk = s1 = s2 = 0.0;
      h_row = 0;
      open_head = (open_head + 1) & (kOpenItems - 1);
      --open_n;
    }
  };

  // The parked records, one per lane: projection, g, the path value, to the
  // value's place in the ring.
  auto flush = [&]() {
    __builtin_amdgcn_wave_barrier();
    if (lane < nrec) {
      R xe[DIM], xr[3];
#pragma unroll
      for (int k = 0; k < DIM; ++k) xe[k] = rec[k * kWave + lane];
      const R y = kYZ ? rec[DIM * kWave + lane] : (R)1, z = kYZ ? rec[(DIM + 1) * kWave + lane] : (R)0;
      const uint32_t tg = rec_tag[lane], nr = rec_n[lane];
      const uint32_t steps = nr & 0x7FFFFFFFu;
      project<R, DIM>(prob.D, xe, xr);
      const R gv = prob.g(xr);
      const R phi = gv * y + z;
      const uint32_t at = tg & (uint32_t)(kRing - 1);
      L->ring[at] = phi;
      OpenItem& it = L->open[tg >> kPosBits];
      atomicAdd(&it.steps, (unsigned long long)steps);
      if (nr >> 31) atomicAdd(&it.cens, 1u);
      if (A.dump_phi != nullptr) {
        const int64_t o = A.dump_off[it.node] + (int64_t)(it.p0 + ((tg - it.base) & kPosMask));
        A.dump_phi[o] = (double)phi;
        if (A.dump_steps != nullptr) A.dump_steps[o] = (int64_t)steps;
      }
      atomicOr(&L->have[at >> 5], 1u << (at & 31u));
    }
    __builtin_amdgcn_wave_barrier();
    nrec = 0;
  };

  // Hands the stream's next paths to the idle lanes; true if room for them
  // has to be made first by a flush of the parked records.
  auto refill = [&]() -> bool {
    for (;;) {
      const uint64_t idle = ballot(!alive && !fin);
      if (idle == 0) return false;
      if (c_left == 0u) {
        if (!more) return false;
        if (open_n == kOpenItems) return nrec > 0;
        uint32_t q = first;
        first = n_first;
        if (q >= n_first) q = n_first < (uint32_t)A.n_items ? n_first + pop_item(A.qhead) : n_first;
        if (q >= (uint32_t)A.n_items) {
          more = false;
          return false;
        }
        const WorkItem it = A.items[q];
        c_node = __builtin_amdgcn_readfirstlane(it.node);
        c_path = (uint32_t)__builtin_amdgcn_readfirstlane((int)it.p0);
        c_left = (uint32_t)__builtin_amdgcn_readfirstlane((int)it.count);
        c_idx = (open_head + open_n) & (kOpenItems - 1);
        ++open_n;
        if (lane == 0) {
          OpenItem o;
          o.base = next_pos;
          o.count = it.count;
          o.p0 = it.p0;
          o.node = it.node;
          o.slot = it.slot;
          o.cens = 0u;
          o.steps = 0ull;
          L->open[c_idx] = o;
        }
        __builtin_amdgcn_wave_barrier();
        prob.start(c_node, x0);
        c_in = prob.inside(x0);
      }
      const uint32_t room = (uint32_t)kRing - (next_pos - tail);
      if (room == 0u) return nrec > 0;
      uint32_t take = (uint32_t)__popcll(idle);
      take = take < c_left ? take : c_left;
      take = take < room ? take : room;
      const uint32_t rank = (uint32_t)lane_rank(idle);
      if (!alive && !fin && rank < take) {
        tag = ((next_pos + rank) & kPosMask) | ((uint32_t)c_idx << kPosBits);
        key = path_key(c_path + rank, (uint32_t)c_node, A.k0, A.k1);
#pragma unroll
        for (int k = 0; k < DIM; ++k) X[k] = x0[k];
        Y = (R)1;
        Z = (R)0;
        n = 0;
        alive = c_in;
        fin = !c_in;
      }
      next_pos += take;
      c_path += take;
      c_left -= take;
    }
  };

  // One step of every running lane.  CAP: the lane may reach max_steps.
  auto step = [&](auto cap, const R* z) {
    constexpr bool CAP = decltype(cap)::value;
    const bool act = CAP ? (alive && n < max_steps) : alive;
    if constexpr (PROB::kWos) {
      // jump by the distance to the boundary in the direction of this jump's
      // Gaussians, or stop inside the shell; predicated: a lane that stops or
      // is idle jumps by a radius of 0
      const R r = prob.distance(X);
      const bool jump = act && (r >= prob.dt);
      const R z2 = sum_squares<R, DIM>(z);
      jump_sphere<R, DIM>(X, jump ? r : (R)0, z2, z);
      n += jump ? 1u : 0u;
      alive = alive && !(act && !jump);
    } else if constexpr (PROB::kFree) {
      // pure diffusion, predicated: an idle lane adds 0 z
      const R m = act ? prob.sdt : (R)0;
#pragma unroll
      for (int k = 0; k < DIM; ++k) X[k] = X[k] + m * z[k];
      n += act ? 1u : 0u;
      alive = CAP ? (alive && !(act && !prob.inside(X))) : (act && prob.inside(X));
    } else if (act) {
      prob.step(X, Y, Z, z);
      ++n;
      if (!prob.inside(X)) alive = false;
    }
  };
  auto window = [&](auto cap) {
    for (int gi = 0; gi < A.refill_groups; ++gi) {
      if (!__any(alive)) break;
      R z[GS::NZ];
      const uint32_t blk = (uint32_t)(((uint64_t)n * DIM) / PB);
#pragma unroll
      for (int b = 0; b < GS::NB; ++b) path_normals<R, LAYOUT, PROB::kWos>(key, blk + (uint32_t)b, A.k0, A.k1, &z[b * PB]);
#pragma unroll
      for (int s = 0; s < GS::G; ++s) step(cap, &z[s * DIM]);
    }
  };

  // Draws `nb` blocks from `blk` on into this lane's part of zbuf, then takes
  // `nst` steps with the Gaussians from zr on, kUnit at a time, the next
  // unit's read from LDS ahead of the steps.  kUnit divides nst; long units
  // keep the branches and the waits of a lone wavefront off its steps.
  // (Pure diffusion: V is the position of the running paths, whose mask is
  // `run`, `steps` their steps since n was last brought up to date.)
  constexpr int kUnit = PROB::kFree ? kFreeUnit : 1;
  auto draw_and_step = [&](auto cap, const PathKey& K, uint32_t blk, int nb, const Ra* zr, int nst, R* V,
                           uint64_t& run, int steps) {
#pragma unroll 1
    for (int b = 0; b < nb; ++b) {
      R z[PB];
      path_normals<R, LAYOUT, PROB::kWos>(K, blk + (uint32_t)b, A.k0, A.k1, z);
#pragma unroll
      for (int k = 0; k < PB; ++k) zbuf[(lane * nb + b) * PB + k] = z[k];
    }
    __builtin_amdgcn_wave_barrier();
    R zn[kUnit * DIM];
#pragma unroll
    for (int k = 0; k < kUnit * DIM; ++k) zn[k] = zr[k];
#pragma unroll 1
    for (int s = 0; s < nst; s += kUnit) {
      R z[kUnit * DIM];
      const Ra* nx = zr + (s + kUnit < nst ? s + kUnit : s) * DIM;
#pragma unroll
      for (int k = 0; k < kUnit * DIM; ++k) {
        z[k] = zn[k];
        zn[k] = nx[k];
      }
      if constexpr (PROB::kFree) {
        // the chain from step to step is the fused multiply-add alone: the
        // unit's moves run on whether a path has left or not, one test covers
        // the unit (its extreme positions), and only if a path has left are
        // its exit step and position picked out
        R W[kUnit][DIM];
        typename PROB::Extremes ext(V);
#pragma unroll
        for (int q = 0; q < kUnit; ++q) {
#pragma unroll
          for (int k = 0; k < DIM; ++k) W[q][k] = V[k] = V[k] + prob.sdt * z[q * DIM + k];
          ext.add(prob, V);
        }
        if ((run & ~ballot(ext.inside(prob))) != 0) {
#pragma unroll
          for (int q = 0; q < kUnit; ++q) {
            const bool mine = alive && !prob.inside(W[q]);
#pragma unroll
            for (int k = 0; k < DIM; ++k) X[k] = mine ? W[q][k] : X[k];
            n += mine ? (uint32_t)(steps + s + q + 1) : 0u;
            alive = alive && !mine;
          }
          run = ballot(alive);
        }
      } else {
#pragma unroll
        for (int q = 0; q < kUnit; ++q) step(cap, &z[q * DIM]);
      }
    }
    __builtin_amdgcn_wave_barrier();
  };

  // The remaining paths (at most half the lanes) with every lane drawing:
  // path of rank j gets the blocks of lanes j Lp .. j Lp + Lp - 1.
  // Lp = 1: a window of groups, every lane drawing for itself.
  auto drain = [&](int na, uint64_t amask, bool shared) {
    int lg = 0;
    if (shared) {
      while ((na << (lg + 1)) <= kWave) ++lg;
    }
    __builtin_amdgcn_wave_barrier();
    const int Lp = 1 << lg;
    const int nblk = shared ? (Lp / GS::NB) * GS::NB : GS::NB;   // of a path and turn
    const int nst = nblk * PB / DIM;
    uint32_t blk = (uint32_t)(((uint64_t)n * DIM) / PB);
    PathKey hk = key;
    int zoff = lane * GS::NZ;
    if (shared) {
      // owner of this lane's draws: the lane of the running path of rank lane / Lp
      const int rank = lane_rank(amask);
      Ua* const who = (Ua*)zbuf;
      if (alive) who[rank] = (uint32_t)lane;
      __builtin_amdgcn_wave_barrier();
      const int j = lane >> lg;
      const int own = (int)(j < na ? who[j] : (uint32_t)lane);
      __builtin_amdgcn_wave_barrier();
      hk.d1 = (uint32_t)__shfl((int)key.d1, own, kWave);
      hk.b1 = (uint32_t)__shfl((int)key.b1, own, kWave);
      hk.c1 = (uint32_t)__shfl((int)key.c1, own, kWave);
      hk.c3 = (uint32_t)__shfl((int)key.c3, own, kWave);
      blk = (uint32_t)__shfl((int)blk, own, kWave) + (uint32_t)(lane & (Lp - 1));
      zoff = alive ? rank * Lp * PB : 0;
    }
    const int nb = shared ? 1 : GS::NB;
    R V[DIM];
#pragma unroll
    for (int k = 0; k < DIM; ++k) V[k] = X[k];
    uint64_t run = amask;
    int steps = 0;
    for (int turn = 0;; ++turn) {
      if (PROB::kRoll) draw_and_step(Yes{}, hk, blk, nb, zbuf + zoff, nst, V, run, steps);
      else draw_and_step(No{}, hk, blk, 1, zbuf + zoff, nst, V, run, steps);
      blk += (uint32_t)nblk;
      if (PROB::kFree) steps += nst;
      const int left = __popcll(ballot(alive));
      if (left == 0) break;
      if (shared) {
        if ((left << (lg + 1)) <= kWave || __any(alive && n + (uint32_t)(steps + nst) > max_steps)) break;
      } else if (turn + 1 >= A.refill_groups) {
        break;
      }
    }
    if (PROB::kFree && alive) {
      n += (uint32_t)steps;
#pragma unroll
      for (int k = 0; k < DIM; ++k) X[k] = V[k];
    }
  };

  const uint32_t span = (uint32_t)(A.refill_groups * GS::G);
  bool full = false;   // the records are to be flushed
  for (;;) {
    // park ended paths; process the records when they are 64 (or asked for)
    const uint64_t fmask = ballot(fin);
    const int nf = __popcll(fmask);
    if (full || nrec + nf > kWave) {
      flush();
      retire();
      full = false;
    }
    if (fmask != 0) {
      if (fin) {
        const int s = nrec + lane_rank(fmask);
#pragma unroll
        for (int k = 0; k < DIM; ++k) rec[k * kWave + s] = X[k];
        if constexpr (kYZ) {
          rec[DIM * kWave + s] = Y;
          rec[(DIM + 1) * kWave + s] = Z;
        }
        rec_tag[s] = tag;
        rec_n[s] = n | (cens ? 0x80000000u : 0u);
      }
      nrec += nf;
      fin = false;
      cens = false;
    }
    full = refill();
    if (full) continue;
    const uint64_t am = ballot(alive);
    if (am == 0) {
      if (ballot(fin) != 0) continue;
      if (nrec == 0) break;
      full = true;
      continue;
    }
    const int na = __popcll(am);
    const bool was = alive;
    const bool shared = !more && c_left == 0u && na <= kDrain && !__any(fin) &&
                        !__any(alive && n + (uint32_t)(kWave * PB) > max_steps);
    if (!PROB::kRoll && shared && nrec > 0) {   // the Gaussians take the records' place
      full = true;
      continue;
    }
    bool cap = PROB::kRoll;
    if (PROB::kRoll || shared) {
      drain(na, am, shared);
    } else {
      // (steps with drift, killing or a source: one copy, with the cap's test)
      cap = PROB::kYZ || __any(alive && n + span > max_steps);
      if (PROB::kYZ) window(Yes{});
      else if (cap) window(Yes{});
      else window(No{});
    }
    if (cap && alive && n >= max_steps) {
      alive = false;
      // walk on spheres: a path already inside the shell exits normally
      cens = PROB::kWos ? (prob.distance(X) >= prob.dt) : true;
    }
    fin = fin || (was && !alive);
  }
}

// ---------------------------------------------------------------------------
// The exit test.  KIND >= 0 (pure diffusion and walk on spheres, whose steps
// are short): a problem whose domain kind is KIND, with the bounds (box) or
// the centre and squared radius (ball) held in vector registers in FP32, so
// the comparisons that read them can share an issue slot; the same arithmetic
// as inside().  KIND = kAnyKind: inside() itself.
constexpr int kAnyKind = -1;
template <typename R, int DIM, int KIND>
struct ExitTest {
  Dom<R> dom;
  R lo[DIM], hi[DIM], ctr[DIM], rad2;
  __device__ __forceinline__ explicit ExitTest(const Dom<R>& D) : dom(D) {
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
      lo[k] = D.lo[k];
      hi[k] = D.hi[k];
      ctr[k] = D.ctr[k];
    }
    rad2 = D.rad2;
    if constexpr (sizeof(R) == 4 && KIND != kAnyKind) {
#pragma unroll
      for (int k = 0; k < DIM; ++k) {
        if constexpr (KIND == DOM_BOX) asm volatile("" : "+v"(lo[k]), "+v"(hi[k]));
        else asm volatile("" : "+v"(ctr[k]));
      }
      if constexpr (KIND != DOM_BOX) asm volatile("" : "+v"(rad2));
    }
  }
  __device__ __forceinline__ bool inside(const R* x) const {
    if constexpr (KIND == kAnyKind) {
      return pdd::inside<R, DIM>(dom, x);
    } else if constexpr (KIND == DOM_BOX) {
      bool in = true;
#pragma unroll
      for (int k = 0; k < DIM; ++k) in = in && (x[k] > lo[k]) && (x[k] < hi[k]);
      return in;
    } else {
      R d[DIM];
#pragma unroll
      for (int k = 0; k < DIM; ++k) d[k] = x[k] - ctr[k];
      return norm2<R, DIM>(d) < rad2;
    }
  }
};

// Whether every one of several positions is inside: the largest and smallest
// coordinates (box) or the largest squared distance from the centre (ball)
// decide, with the comparisons of the exit test.
template <typename R, int DIM, int KIND>
struct ExitExtremes {
  R hi[DIM], lo[DIM];
  __device__ __forceinline__ explicit ExitExtremes(const R* x) {
#pragma unroll
    for (int k = 0; k < DIM; ++k) hi[k] = lo[k] = KIND == DOM_BOX ? x[k] : (R)0;
  }
  template <class PROB>
  __device__ __forceinline__ void add(const PROB& P, const R* x) {
    if constexpr (KIND == DOM_BOX) {
#pragma unroll
      for (int k = 0; k < DIM; ++k) {
        hi[k] = fmax(hi[k], x[k]);
        lo[k] = fmin(lo[k], x[k]);
      }
    } else {
      R d[DIM];
#pragma unroll
      for (int k = 0; k < DIM; ++k) d[k] = x[k] - P.test.ctr[k];
      hi[0] = fmax(hi[0], norm2<R, DIM>(d));
    }
  }
  template <class PROB>
  __device__ __forceinline__ bool inside(const PROB& P) const {
    if constexpr (KIND == DOM_BOX) {
      bool in = true;
#pragma unroll
      for (int k = 0; k < DIM; ++k) in = in && (lo[k] > P.test.lo[k]) && (hi[k] < P.test.hi[k]);
      return in;
    } else {
      return hi[0] < P.test.rad2;
    }
  }
};

// One linear problem (the kernel's argument) as stream_walk's PROB.
template <typename R, int DIM, int DFC, bool TERMS, bool WOS, class TP, int KIND>
struct SingleProblem {
  static constexpr bool kWos = WOS, kFree = DFC < 0 && !TERMS && !WOS, kYZ = !WOS && !kFree;
  static constexpr bool kRoll = kYZ && (TERMS || sizeof(R) == 8);
  // FP32 walks without generic terms: the dense coefficients of c and f sit
  // in LDS (rows of kNMp), so the step's products read no scalar register
  static constexpr int NM = GradedLex<DIM, DFC>::N;
  static constexpr bool kLdsPoly = sizeof(R) == 4 && !TERMS && !WOS && DFC >= 0;
  static constexpr int kNMp = ((GradedLex<DIM, (DFC >= 0 ? DFC : 0)>::N + 3) / 4) * 4;
  typedef const __attribute__((address_space(3))) R* LdsR;
  typedef ExitExtremes<R, DIM, KIND> Extremes;

  const LinearParams& P;
  const Dom<R> D;                      // projection of exit points
  const ExitTest<R, DIM, KIND> test;   // exit test
  R dt, sdt;
  const uint32_t max_steps;
  const typename TP::template State<R> tst;
  LdsR lpoly;

  __device__ __forceinline__ SingleProblem(const LinearParams& p, const R* lp)
      : P(p), D(make_dom<R>(p)), test(make_test_dom<R>(p)), dt(dt_of<R>(p)), sdt(sdt_of<R>(p)),
        max_steps((uint32_t)p.max_steps), tst(TP::template load<R>(p)), lpoly((LdsR)lp) {
    // FP32: the step sizes in VGPRs, so the products that use them read no
    // SGPR and can share an issue slot with another wavefront's instruction
    if constexpr (sizeof(R) == 4) asm volatile("" : "+v"(dt), "+v"(sdt));
  }
  __device__ __forceinline__ void start(int node, R* x) const {
#pragma unroll
    for (int k = 0; k < DIM; ++k) x[k] = to_r<R>(P.nodes[(size_t)node * DIM + k]);
  }
  __device__ __forceinline__ bool inside(const R* x) const { return test.inside(x); }
  __device__ __forceinline__ R distance(const R* x) const {
    Dom<R> d = D;
    d.kind = KIND;
    return boundary_distance<R, DIM>(d, x);
  }
  __device__ __forceinline__ R g(const R* x) const { return g_value_tp<R, DIM, TP, true>(P, tst, x); }
  __device__ __forceinline__ void step(R* X, R& Y, R& Z, const R* z) const {
    R mono[NM > 0 ? NM : 1];
    if constexpr (DFC >= 0) monomials<R, DIM, DFC>(X, mono);
    R fv, cv;
    if constexpr (kLdsPoly) {
      fv = P.f.poly_deg >= 0 ? poly_dot_lds<R, NM>(lpoly + kNMp, mono) : (R)0;
      cv = P.c.poly_deg >= 0 ? poly_dot_lds<R, NM>(lpoly, mono) : (R)0;
    } else {
      fv = bcf_value<R, DIM, DFC, TERMS, TP, FUN_F>(P, tst, P.f, X, mono);
      cv = bcf_value<R, DIM, DFC, TERMS, TP, FUN_C>(P, tst, P.c, X, mono);
    }
    // terms known to vanish are skipped: X + 0 dt, Z + 0 and Y exp(0) leave
    // the same bits as evaluating them
    if (P.has_f) Z = Z + fv * Y * dt;
    if (P.has_c) Y = Y * fexp(-cv * dt);
    if (P.has_b) {
      R bv[DIM];
      if constexpr (TERMS) {
        bv[0] = bcf_value<R, DIM, DFC, TERMS, TP, FUN_B0>(P, tst, P.b[0], X, mono);
        if constexpr (DIM >= 2) bv[1] = bcf_value<R, DIM, DFC, TERMS, TP, FUN_B1>(P, tst, P.b[1], X, mono);
        if constexpr (DIM >= 3) bv[2] = bcf_value<R, DIM, DFC, TERMS, TP, FUN_B2>(P, tst, P.b[2], X, mono);
      } else {
#pragma unroll
        for (int k = 0; k < DIM; ++k) bv[k] = bcf_value<R, DIM, DFC, false, TP, FUN_B0>(P, tst, P.b[k], X, mono);
      }
#pragma unroll
      for (int k = 0; k < DIM; ++k) X[k] = X[k] + bv[k] * dt + sdt * z[k];
    } else {
#pragma unroll
      for (int k = 0; k < DIM; ++k) X[k] = X[k] + sdt * z[k];
    }
  }
};

// Occupancy request: the FP32 kernels without generic terms fit in 80 VGPRs
// (pure diffusion, walk on spheres: six waves per SIMD) or, with a polynomial
// part, in 96 (five), those with terms in 256 (two); the FP64
// kernels are left unconstrained.
template <typename R, int DFC, bool TERMS>
constexpr int fwd_min_waves() { return sizeof(R) == 4 ? (TERMS ? 2 : (DFC < 0 ? 6 : 5)) : 1; }

template <typename R, int DIM, int DFC, int LAYOUT, bool TERMS, bool WOS = false, class TP = TableTerms>
__global__ void __launch_bounds__(kBlock, (fwd_min_waves<R, DFC, TERMS>()))
k_walk_fwd(const LinearParams P, const StreamArgs A) {
  constexpr int kWaves = kBlock / kWave;
  using Any = SingleProblem<R, DIM, DFC, TERMS, WOS, TP, kAnyKind>;
  using Lds = StreamLds<R, stream_area_bytes<R, DIM, LAYOUT, Any::kYZ, Any::kRoll>()>;
  __shared__ Lds lds[kWaves];
  __shared__ __attribute__((aligned(16))) R lpoly[Any::kLdsPoly ? 2 * Any::kNMp : 4];   // row 0: c, row 1: f
  const int lane = (int)(threadIdx.x & (kWave - 1));
  const int wid = (int)(threadIdx.x / kWave);
  if constexpr (Any::kLdsPoly) {
    constexpr int kNMp = Any::kNMp;
    for (int i = (int)threadIdx.x; i < 2 * kNMp; i += kBlock) {
      const DevFun& F = i < kNMp ? P.c : P.f;
      const int m = i % kNMp;
      lpoly[i] = (F.poly_deg >= 0 && m < Any::NM) ? P.cf[F.poly_off + m] : (R)0;
    }
    __syncthreads();
  }
  const uint32_t wave = blockIdx.x * kWaves + (uint32_t)__builtin_amdgcn_readfirstlane(wid);
  const uint32_t n_waves = gridDim.x * kWaves;
  if constexpr (Any::kYZ) {
    stream_walk<R, DIM, LAYOUT>(
        SingleProblem<R, DIM, DFC, TERMS, WOS, TP, TP::kKind>(P, lpoly), A, &lds[wid], lane, wave, n_waves);
  } else if (P.dom_kind == DOM_BOX) {
    stream_walk<R, DIM, LAYOUT>(SingleProblem<R, DIM, DFC, TERMS, WOS, TP, DOM_BOX>(P, lpoly), A, &lds[wid], lane,
                                wave, n_waves);
  } else {
    stream_walk<R, DIM, LAYOUT>(SingleProblem<R, DIM, DFC, TERMS, WOS, TP, DOM_BALL>(P, lpoly), A, &lds[wid], lane,
                                wave, n_waves);
  }
}

}  // namespace pdd
