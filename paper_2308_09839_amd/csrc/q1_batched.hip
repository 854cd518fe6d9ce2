// Batched persistent Jacobi-PCG: many independent scalar-Laplace problems,
// each with up to four right-hand sides, solved by ONE cooperative launch.
//
// Each problem p owns a contiguous range of workgroups of one or four
// wavefronts (sized in proportion to its expected work), which meet at
// a barrier of global counters and flags; problems never wait for each
// other.  Vectors are stored interleaved [node][R] so that one gather of a
// node serves all R right-hand sides.  Per iteration (the CG operations of
// Table 4, regrouped):
//   P1  over the operator's LDS tiles (as in q1_tile.hip): the direction
//       update p = D^{-1} r + beta p_old on each tile's nodes into LDS (the
//       node's writer entry also stores it), then the tile's part of q = A p
//       from the staged p, written to the tile's slot of each of its free nodes,
//       with the partials of p^T A p (p times the tile's sums, and p^2 on
//       Dirichlet nodes by the writer entry).  p alternates between two buffers,
//       so reading p_old and writing p needs no barrier in between.
//   P2  q of a node = the sum of its slots (contiguous, in tile order; p on a
//       Dirichlet node); alpha = rho / p^T A p; x += alpha p; r -= alpha q;
//       partials of rho' = r^T D^{-1} r and r^T r; then the convergence test
//       and beta = rho'/rho for the next P1
// with one barrier after each phase.  In the mixed-precision form the search
// directions p, q and the applies of P1 are FP32 (the FP32 operator's
// coordinates and coefficients), while x, r and every dot product stay FP64;
// whenever the recurrence residual has fallen by delta since the last refresh
// (and before convergence is declared) the true residual r = b - A64 x is
// recomputed with an FP64 apply of x inside the same launch (two more
// barriers), and the recurrences continue from it with p kept.
// The barrier itself sums the partials in a fixed order (per sub-group of
// waves, then over sub-groups) and every wave reads the same totals, so all
// waves of a problem hold bit-identical scalars and take the same branch.  Each
// barrier wait has a spin limit: past it the kernel records an error and every
// wave returns.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstddef>
#include <cstdint>
#include <new>
#include <type_traits>
#include <vector>

#include "q1_elem.hpp"
#include "q1_internal.hpp"

namespace q1 {

namespace {

constexpr int kW = 64;            // lanes of a wavefront
constexpr int kRmax = 4;
constexpr uint32_t kFixedBitB = 0x40000000u;
constexpr uint32_t kIdMaskB = 0x3fffffffu;
// In the copy of the tile node lists the search-direction phase reads, bit 29
// (kOwnEntry) marks the one entry (in the first tile holding the node) that
// writes the node's new direction; ids are then below 2^29.
constexpr uint32_t kIdMaskOwnB = kOwnEntry - 1;
constexpr unsigned kSpinLimit = 1u << 26;  // barrier polls before giving up
// In the staging, the write-back and the vector phases a lane takes one right-hand side of a
// node: 64 / R nodes per instruction, so that the R values of a node (32 bytes for R = 4) and
// its neighbours' leave in whole lines.  (One node with all its R values per lane fetched every
// line R times, since these accesses bypass the caches.)
// Rounds issue all their loads before their stores: gfx9 waits for loads and stores on one
// counter, so a round costs one load and one store latency whatever its length is.
// A workgroup is NW wavefronts: four on parallelepiped tiles, which then stage, compute and
// write one tile together (one step of 64 elements each, the right-hand sides in turn, so that
// three fit a SIMD), and one otherwise (general elements keep their geometry for all sides at
// once, in 256 and more registers).  Twelve problems of 16^3 to 40^3 with four right-hand sides:
// 74 us per iteration with one wave per workgroup, 57 with four.  Three waves per SIMD are asked
// for: that spills 2 registers with four FP64 sides and 2 to 8 in the mixed form with two to
// four; two waves per SIMD would spill none, and run two thirds of the workgroups.
template <int R, int NW>
struct Lanes {
  static constexpr int NLW = kW / R;    // nodes per instruction of a wave
  static constexpr int NL = NLW * NW;   // and of the workgroup
  // nodes per lane per round: of the vector phases, of a tile's staging and of its node words
  static constexpr int kU = NW > 1 || R == 1 ? 4 : 6;
  static constexpr int kStage = NW > 1 ? 2 * R : R == 1 ? 8 : 12;
  static constexpr int kIds = NW > 1 ? 2 : 8;
  int c, sub;                           // right-hand side and node of this lane
  bool act;                             // R = 3 leaves one lane of a wave idle
  __device__ Lanes() {
    const int lane = threadIdx.x & (kW - 1), wave = threadIdx.x / kW;
    c = lane % R;
    sub = wave * NLW + lane / R;
    act = lane < NLW * R;
  }
};

// partial-sum slots per problem: [slot][rhs][nwg]
enum { kPQ = 0, kRho = 1, kRR = 2, kBB = 3, kRho0 = 4, kSlots = 5 };

struct BProb {
  int64_t nn;
  int n_tiles, max_nodes;
  const int32_t *node_ptr;
  const uint32_t *nodes;
  const uint32_t *onodes;     // the node lists with the writer bit
  const int32_t *tile_step;
  const uint4 *lconn;
  const double *coef_t;
  const double *xyz;
  const uint32_t *nptr;       // [nn + 1]: first slot of a node (bit 31: Dirichlet, no slots)
  const int32_t *pos;         // [entries]: slot of a tile entry (-1 on Dirichlet nodes)
  int64_t n_slots;
  double *b, *x, *r;          // [nn][R]
  double *q;                  // [n_slots][R]
  double *p[2];               // [nn][R]: directions of odd and even iterations
  const double *w;            // inverse diagonal [nn]
  // mixed precision: FP32 geometry, coefficients and directions; FP64 refresh output
  const float *xyz32, *coef32;
  float *p32[2];              // [nn][R]
  float *q32;                 // [n_slots][R]
  double *t;                  // [n_slots][R]
  double *part;               // [kSlots][R][nwg]
  double *tot;                // [2][kSub][2R] sub-group totals, two buffers
  unsigned *bar;              // [kBarWords]: sub-group counters and flags
  int wg0, nwg;
  int *iters, *status, *nref; // [R]
  double *rr, *bb;            // [R]
};

// The problem records are read from memory, so the compiler cannot tell that
// their pointers address global memory and would access them with flat
// instructions, which also count on the LDS counter: every LDS wait of the
// apply (node ids, accumulator atomics) would then wait for all outstanding
// memory loads.  The kernel therefore reads each record through a twin whose
// pointers are typed as global-address-space pointers; converting those to
// ordinary pointers keeps the fact that they address global memory, and the
// compiler emits global instructions for every access made through them.
#define Q1_GLB __attribute__((address_space(1)))
struct BProbG {
  int64_t nn;
  int n_tiles, max_nodes;
  const Q1_GLB int32_t *node_ptr;
  const Q1_GLB uint32_t *nodes;
  const Q1_GLB uint32_t *onodes;
  const Q1_GLB int32_t *tile_step;
  const Q1_GLB uint4 *lconn;
  const Q1_GLB double *coef_t;
  const Q1_GLB double *xyz;
  const Q1_GLB uint32_t *nptr;
  const Q1_GLB int32_t *pos;
  int64_t n_slots;
  Q1_GLB double *b, *x, *r;
  Q1_GLB double *q;
  Q1_GLB double *p[2];
  const Q1_GLB double *w;
  const Q1_GLB float *xyz32, *coef32;
  Q1_GLB float *p32[2];
  Q1_GLB float *q32;
  Q1_GLB double *t;
  Q1_GLB double *part;
  Q1_GLB double *tot;
  Q1_GLB unsigned *bar;
  int wg0, nwg;
  Q1_GLB int *iters, *status, *nref;
  Q1_GLB double *rr, *bb;
};
static_assert(sizeof(BProbG) == sizeof(BProb) && offsetof(BProbG, bb) == offsetof(BProb, bb) &&
                  offsetof(BProbG, n_slots) == offsetof(BProb, n_slots) &&
                  offsetof(BProbG, wg0) == offsetof(BProb, wg0),
              "BProbG must mirror BProb");

__device__ __forceinline__ BProb load_problem(const BProb *src) {
  BProbG G;
  __builtin_memcpy(&G, src, sizeof(G));
  BProb P;
  P.nn = G.nn;
  P.n_tiles = G.n_tiles;
  P.max_nodes = G.max_nodes;
  P.node_ptr = (const int32_t *)G.node_ptr;
  P.nodes = (const uint32_t *)G.nodes;
  P.onodes = (const uint32_t *)G.onodes;
  P.tile_step = (const int32_t *)G.tile_step;
  P.lconn = (const uint4 *)G.lconn;
  P.coef_t = (const double *)G.coef_t;
  P.xyz = (const double *)G.xyz;
  P.nptr = (const uint32_t *)G.nptr;
  P.pos = (const int32_t *)G.pos;
  P.n_slots = G.n_slots;
  P.b = (double *)G.b;
  P.x = (double *)G.x;
  P.r = (double *)G.r;
  P.p[0] = (double *)G.p[0];
  P.p[1] = (double *)G.p[1];
  P.q = (double *)G.q;
  P.w = (const double *)G.w;
  P.xyz32 = (const float *)G.xyz32;
  P.coef32 = (const float *)G.coef32;
  P.p32[0] = (float *)G.p32[0];
  P.p32[1] = (float *)G.p32[1];
  P.q32 = (float *)G.q32;
  P.t = (double *)G.t;
  P.part = (double *)G.part;
  P.tot = (double *)G.tot;
  P.bar = (unsigned *)G.bar;
  P.wg0 = G.wg0;
  P.nwg = G.nwg;
  P.iters = (int *)G.iters;
  P.status = (int *)G.status;
  P.nref = (int *)G.nref;
  P.rr = (double *)G.rr;
  P.bb = (double *)G.bb;
  return P;
}
#undef Q1_GLB

// Every value that one wave writes and another reads within the launch (r, p, q, the partial
// sums and totals; x and t of the mixed form) is read and written with these: relaxed atomics
// at agent scope, which go past the caches of the accelerator dies to the point where all
// dies see the same memory.  settle() waits until this wave's earlier accesses have been
// performed there, so what it then announces (a counter, a generation) can only be seen
// after them.
template <typename E>
__device__ __forceinline__ E get(const E *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename E>
__device__ __forceinline__ void put(E *p, E v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void settle() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

__device__ __forceinline__ double wave_sum64(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// Sum of v over the lanes of this lane's right-hand side (lane % R), in every such lane.
template <int R>
__device__ __forceinline__ double rhs_sum(double v, int lane) {
  if constexpr (R == 3) {
    double t = 0.0;
#pragma unroll
    for (int c = 0; c < R; ++c) {
      const double w = wave_sum64(lane % R == c && lane < kW - 1 ? v : 0.0);
      if (lane % R == c) t = w;
    }
    return t;
  } else {
#pragma unroll
    for (int off = 32; off >= R; off >>= 1) v += __shfl_xor(v, off);
    return v;
  }
}

// The same over the NW waves of the workgroup, in wave order.
template <int R, int NW>
__device__ __forceinline__ double group_sum(double v, int lane) {
  v = rhs_sum<R>(v, lane);
  if constexpr (NW > 1) {
    __shared__ double sh[NW][R];
    const int wave = threadIdx.x / kW;
    if (lane < R) sh[wave][lane] = v;
    __syncthreads();
    v = sh[0][lane % R];
#pragma unroll
    for (int w = 1; w < NW; ++w) v += sh[w][lane % R];
    __syncthreads();
  }
  return v;
}

// Barrier of the nwg workgroups of one problem (one wave of each), optionally fused with the
// sum of two partial-sum slots (sa, sb; either < 0 for none) over the workgroups; false when
// the spin limit was hit.  Workgroup me belongs to sub-group me % kSub, whose counter and flag
// share a cache line of their own.  The last arrival of a sub-group sums its members' partials
// (in member order) into the sub-group's totals, resets the counter and raises the flag to
// this barrier's number.  Every workgroup polls all the flags (a lane each) and then adds the
// sub-groups' totals in order, so every lane holds bit-identical totals of its right-hand side
// (a, b) and all take the same branch.  The totals alternate between two buffers: a sub-group
// can only come to the barrier after the next once everyone has left this one (it needs their arrival at the next).
// Ordering: every exchanged value is accessed past the caches (get, put) and each arrival and
// flag is preceded by settle(), so no wave writes back or invalidates an L2.  Agent-scope
// fences at each arrival did so for the die's whole L2, one wave after another: an iteration of
// twelve problems (16^3 to 40^3, one right-hand side) took 151 us, 47 without them and 34 now.
// A further counter over the sub-groups, whose last arrival makes the totals and releases
// everyone, costs four more memory round trips: 16^3 with four right-hand sides 20.1 us per
// iteration against 18.4.  Sub-groups: arrivals on one counter are served one by one, while each
// workgroup polls all the flags; 40^3 with four right-hand sides (400 workgroups): 4
// sub-groups 43 us per iteration, 8 37, 16 33, 32 36.
// bar: [32 k] counter of sub-group k, [32 k + 1] its flag.  tot: [2][kSub][2R].
constexpr unsigned kSub = 16;
constexpr unsigned kBarWords = 32 * kSub;
template <int R>
__device__ __forceinline__ bool problem_sync(const BProb &P, unsigned me, unsigned nwg,
                                             int *error, unsigned &gen, int sa, int sb, double &a,
                                             double &b) {
  const int lane = threadIdx.x;
  const unsigned nsub = nwg < kSub ? nwg : kSub;  // sub-groups in use
  const unsigned sub = me % nsub;
  const unsigned members = (nwg - sub + nsub - 1) / nsub;
  unsigned *sc = P.bar + 32 * sub;
  double *tot = P.tot + (gen & 1) * (kSub * 2 * R);
  ++gen;
  int last = 0;
  settle();  // this wave's writes
  if (lane == 0)
    last = __hip_atomic_fetch_add(sc, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
           members - 1;
  if (__shfl(last, 0)) {
    if (sa >= 0) {
      double va[R], vb[R];
#pragma unroll
      for (int c = 0; c < R; ++c) va[c] = vb[c] = 0.0;
      for (unsigned k = lane; k < members; k += kW) {
        const int64_t w = sub + int64_t(k) * nsub;
#pragma unroll
        for (int c = 0; c < R; ++c) {
          va[c] += get(&P.part[(int64_t(sa) * R + c) * nwg + w]);
          if (sb >= 0) vb[c] += get(&P.part[(int64_t(sb) * R + c) * nwg + w]);
        }
      }
#pragma unroll
      for (int c = 0; c < R; ++c) {
        va[c] = wave_sum64(va[c]);
        if (sb >= 0) vb[c] = wave_sum64(vb[c]);
      }
      if (lane == 0) {
#pragma unroll
        for (int c = 0; c < R; ++c) {
          put(&tot[sub * 2 * R + c], va[c]);
          put(&tot[sub * 2 * R + R + c], vb[c]);
        }
      }
    }
    // every member has arrived: the counter is reset before settle(), so the reset is
    // complete before anyone can pass this barrier
    if (lane == 0) put(sc, 0u);
    settle();
    if (lane == 0) put(sc + 1, gen);
  }
  // wait until every sub-group's flag has come to this barrier (the faster ones may show the
  // next one already, but no further: that needs this workgroup)
  bool ok = true;
  unsigned spins = 0;
  const unsigned *flag = P.bar + 32 * (unsigned(lane) < nsub ? unsigned(lane) : 0u) + 1;
  while (__any(int(get(flag) - gen) < 0)) {
    __builtin_amdgcn_s_sleep(1);
    if (++spins > kSpinLimit || __any(get(error))) {
      if (lane == 0) put(error, 1);
      ok = false;
      break;
    }
  }
  settle();  // nothing below is requested before the flags were seen
  if (ok && sa >= 0) {
    const int c = lane % R;
    double va[kSub], vb[kSub];
#pragma unroll
    for (unsigned k = 0; k < kSub; ++k) {
      const unsigned o = min(k, nsub - 1) * 2 * R;
      va[k] = get(&tot[o + c]);
      vb[k] = get(&tot[o + R + c]);
    }
    a = b = 0.0;
#pragma unroll
    for (unsigned k = 0; k < kSub; ++k)
      if (k < nsub) {
        a += va[k];
        b += vb[k];
      }
  }
  return ok;
}

// problem_sync of workgroups: the first wave meets the other workgroups' once every wave of
// this one has settled, and hands on what it brings back.
template <int R, int NW>
__device__ __forceinline__ bool group_sync(const BProb &P, unsigned me, unsigned nwg, int *error,
                                           unsigned &gen, int sa, int sb, double &a,
                                           double &b) {
  if constexpr (NW == 1) {
    return problem_sync<R>(P, me, nwg, error, gen, sa, sb, a, b);
  } else {
    __shared__ double sh[2 * R];
    __shared__ int sh_ok;
    settle();
    __syncthreads();
    if (threadIdx.x < kW) {
      const bool ok = problem_sync<R>(P, me, nwg, error, gen, sa, sb, a, b);
      if (threadIdx.x == 0) sh_ok = ok ? 1 : 0;
      if (threadIdx.x < R) {
        sh[threadIdx.x] = a;
        sh[R + threadIdx.x] = b;
      }
    }
    __syncthreads();
    const int c = (threadIdx.x & (kW - 1)) % R;
    a = sh[c];
    b = sh[R + c];
    const bool ok = sh_ok != 0;
    __syncthreads();
    return ok;
  }
}

// plain barrier
template <int R, int NW>
__device__ __forceinline__ bool problem_barrier(const BProb &P, unsigned me, unsigned nwg,
                                                int *error, unsigned &gen) {
  double a = 0.0, b = 0.0;
  return group_sync<R, NW>(P, me, nwg, error, gen, -1, -1, a, b);
}

// dst = A src over this workgroup's tiles (src [nn][R], dst [n_slots][R] of type T; LDS accumulation
// in FP64), used by the FP64 refresh of the mixed form.  The R right-hand sides are the components of one element product, so the geometry
// is evaluated once per element; PAR: every tile of every problem is a
// parallelepiped tile (flagged at set-up), so only corners 0, 1, 2, 4 are read
// and the closed-form parallelepiped action is used.  Dirichlet corners read
// zero; dst is by slot, as q; right-hand sides marked skip are neither read nor
// written.
template <typename T, int R, bool PAR, int NW>
__device__ __forceinline__ void apply_phase(const BProb &P, int me, int nwg, int lane, int wave,
                                            double *acc, uint32_t *sId, const T *xyz,
                                            const T *coef_t, const T *src, T *dst,
                                            int skip_m) {
  constexpr int kIds = Lanes<R, NW>::kIds;
  for (int t = me; t < P.n_tiles; t += nwg) {
    const int n0 = P.node_ptr[t], nm = P.node_ptr[t + 1] - n0;
    const int s0 = P.tile_step[t], s1 = P.tile_step[t + 1];
    // the first step's corner words and coefficient are requested with the staging
    // loads, and each later step's one step ahead, so a step waits for one memory
    // latency (its gathers) instead of two
    uint4 pk_next = make_uint4(0xffffffffu, 0, 0, 0);
    T k_next = T(0);
    if (s0 + wave < s1) {
      pk_next = P.lconn[int64_t(s0 + wave) * kW + lane];
      k_next = coef_t[int64_t(s0 + wave) * kW + lane];
    }
    // node ids staged kIds per lane per round, all loads of a round issued first
    for (int ib = threadIdx.x; ib < nm; ib += kIds * NW * kW) {
      uint32_t id[kIds];
#pragma unroll
      for (int u = 0; u < kIds; ++u) id[u] = P.nodes[n0 + min(ib + u * NW * kW, nm - 1)];
#pragma unroll
      for (int u = 0; u < kIds; ++u) {
        const int i = ib + u * NW * kW;
        if (i >= nm) continue;
        sId[i] = id[u];
#pragma unroll
        for (int c = 0; c < R; ++c) acc[c * P.max_nodes + i] = 0.0;
      }
    }
    __syncthreads();
    for (int s = s0 + wave; s < s1; s += NW) {
      const int64_t slot = int64_t(s) * kW + lane;
      const uint4 pk = pk_next;
      const T k = k_next;
      if (s + NW < s1) {
        pk_next = P.lconn[slot + NW * kW];
        k_next = coef_t[slot + NW * kW];
      }
      if (pk.x == 0xffffffffu) continue;
      const int lc[8] = {int(pk.x & 0xffff), int(pk.x >> 16), int(pk.y & 0xffff),
                         int(pk.y >> 16),    int(pk.z & 0xffff), int(pk.z >> 16),
                         int(pk.w & 0xffff), int(pk.w >> 16)};
      int64_t g[8];
      bool fx[8];
#pragma unroll
      for (int a = 0; a < 8; ++a) {
        const uint32_t raw = sId[lc[a]];
        g[a] = raw & kIdMaskB;
        fx[a] = (raw & kFixedBitB) != 0;
      }
      T X[3][8];
#pragma unroll
      for (int a = 0; a < 8; ++a)
        if (!PAR || a == 0 || a == 1 || a == 2 || a == 4)
#pragma unroll
          for (int d = 0; d < 3; ++d) X[d][a] = xyz[d * P.nn + g[a]];
      if constexpr (NW > 1) {  // one right-hand side at a time: a quarter of the registers
#pragma unroll 1
        for (int c = 0; c < R; ++c) {
          if ((skip_m >> c) & 1) continue;
          T u[1][8], v[1][8];
#pragma unroll
          for (int a = 0; a < 8; ++a) u[0][a] = fx[a] ? T(0) : get(&src[g[a] * R + c]);
          laplace_element_parallelepiped_n<T, 1>(X, u, k, v);
#pragma unroll
          for (int a = 0; a < 8; ++a)
            __hip_atomic_fetch_add(&acc[c * P.max_nodes + lc[a]], double(v[0][a]),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
      } else {
        T u[R][8], v[R][8];
#pragma unroll
        for (int a = 0; a < 8; ++a)
#pragma unroll
          for (int c = 0; c < R; ++c) u[c][a] = (fx[a] || ((skip_m >> c) & 1)) ? T(0) : get(&src[g[a] * R + c]);
        if constexpr (PAR)
          laplace_element_parallelepiped_n<T, R>(X, u, k, v);
        else
          laplace_element_n<T, R>(X, u, k, v);
#pragma unroll
        for (int c = 0; c < R; ++c) {
          if (((skip_m >> c) & 1)) continue;
#pragma unroll
          for (int a = 0; a < 8; ++a) {
            __hip_atomic_fetch_add(&acc[c * P.max_nodes + lc[a]], double(v[c][a]),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          }
        }
      }
    }
    __syncthreads();
    const Lanes<R, NW> L;
    const bool put_c = L.act && !((skip_m >> L.c) & 1);
    for (int i = put_c ? L.sub : nm; i < nm; i += L.NL) {
      const int32_t sl = P.pos[n0 + i];
      if (sl >= 0) put(&dst[int64_t(sl) * R + L.c], T(acc[L.c * P.max_nodes + i]));
    }
    __syncthreads();
  }
}

// The direction update and q = A p in one pass over this workgroup's tiles.  For
// each tile node the new direction p = D^-1 r + beta p_old (p = D^-1 r on the
// first iteration) is computed into LDS, where the element loop reads it (zero
// on Dirichlet corners and for finished right-hand sides); the node's writer
// entry also stores it to pnew and, on a Dirichlet node (whose row of A p is p
// itself), adds p^2 to pq.  A node held by several tiles is computed by each
// from the same values, so every copy agrees.  Reading p_old from one buffer
// and writing pnew to the other lets the update run without a barrier before
// the apply.  The tile's sums go to its slots of the nodes, and p times them to
// pq, this lane's share of p^T A p for its right-hand side.  T is the precision
// of p, q and the element arithmetic.
template <typename T, int R, bool PAR, int NW>
__device__ __forceinline__ void update_apply_phase(const BProb &P, int me, int nwg, int lane, int wave,
                                                   double *acc, uint32_t *sId, T *sP,
                                                   const T *xyz, const T *coef_t, const T *pold,
                                                   T *pnew, T *q, int done_m, double beta,
                                                   bool first, double &pq) {
  const int M = P.max_nodes;
  const Lanes<R, NW> L;
  const bool on = L.act && !((done_m >> L.c) & 1);
  constexpr int kStage = Lanes<R, NW>::kStage, kIds = Lanes<R, NW>::kIds;
  for (int t = me; t < P.n_tiles; t += nwg) {
    const int n0 = P.node_ptr[t], nm = P.node_ptr[t + 1] - n0;
    const int s0 = P.tile_step[t], s1 = P.tile_step[t + 1];
    uint4 pk_next = make_uint4(0xffffffffu, 0, 0, 0);
    T k_next = T(0);
    if (s0 + wave < s1) {
      pk_next = P.lconn[int64_t(s0 + wave) * kW + lane];
      k_next = coef_t[int64_t(s0 + wave) * kW + lane];
    }
    for (int ib = threadIdx.x; ib < nm; ib += kIds * NW * kW) {
      uint32_t id[kIds];
#pragma unroll
      for (int u = 0; u < kIds; ++u) id[u] = P.onodes[n0 + min(ib + u * NW * kW, nm - 1)];
#pragma unroll
      for (int u = 0; u < kIds; ++u)
        if (ib + u * NW * kW < nm) sId[ib + u * NW * kW] = id[u];
    }
    __syncthreads();
    for (int ib = L.act ? L.sub : nm; ib < nm; ib += kStage * L.NL) {
      uint32_t id[kStage];
      double wv[kStage], rv[kStage], pv[kStage];
#pragma unroll
      for (int u = 0; u < kStage; ++u) {
        id[u] = sId[min(ib + u * L.NL, nm - 1)];
        const int64_t g = id[u] & kIdMaskOwnB;
        wv[u] = rv[u] = pv[u] = 0.0;
        if (on) {
          wv[u] = P.w[g];
          rv[u] = get(&P.r[g * R + L.c]);
          if (!first) pv[u] = double(get(&pold[g * R + L.c]));
        }
      }
#pragma unroll
      for (int u = 0; u < kStage; ++u) {
        const int i = ib + u * L.NL;
        if (i >= nm) continue;
        const bool fixed = (id[u] & kFixedBitB) != 0;
        const T pn = on ? T(wv[u] * rv[u] + beta * pv[u]) : T(0);
        acc[L.c * M + i] = 0.0;
        sP[L.c * M + i] = fixed ? T(0) : pn;
        if (on && (id[u] & kOwnEntry)) {
          put(&pnew[int64_t(id[u] & kIdMaskOwnB) * R + L.c], pn);
          if (fixed) pq += double(pn) * double(pn);
        }
      }
    }
    __syncthreads();
    for (int s = s0 + wave; s < s1; s += NW) {
      const int64_t slot = int64_t(s) * kW + lane;
      const uint4 pk = pk_next;
      const T k = k_next;
      if (s + NW < s1) {
        pk_next = P.lconn[slot + NW * kW];
        k_next = coef_t[slot + NW * kW];
      }
      if (pk.x == 0xffffffffu) continue;
      const int lc[8] = {int(pk.x & 0xffff), int(pk.x >> 16), int(pk.y & 0xffff),
                         int(pk.y >> 16),    int(pk.z & 0xffff), int(pk.z >> 16),
                         int(pk.w & 0xffff), int(pk.w >> 16)};
      T X[3][8];
#pragma unroll
      for (int a = 0; a < 8; ++a)
        if (!PAR || a == 0 || a == 1 || a == 2 || a == 4) {
          const int64_t g = sId[lc[a]] & kIdMaskOwnB;
#pragma unroll
          for (int d = 0; d < 3; ++d) X[d][a] = xyz[d * P.nn + g];
        }
      if constexpr (NW > 1) {  // one right-hand side at a time: a quarter of the registers
#pragma unroll 1
        for (int c = 0; c < R; ++c) {
          if ((done_m >> c) & 1) continue;
          T u[1][8], v[1][8];
#pragma unroll
          for (int a = 0; a < 8; ++a) u[0][a] = sP[c * M + lc[a]];
          laplace_element_parallelepiped_n<T, 1>(X, u, k, v);
#pragma unroll
          for (int a = 0; a < 8; ++a)
            __hip_atomic_fetch_add(&acc[c * M + lc[a]], double(v[0][a]), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
        }
      } else {
        T u[R][8], v[R][8];
#pragma unroll
        for (int a = 0; a < 8; ++a)
#pragma unroll
          for (int c = 0; c < R; ++c) u[c][a] = sP[c * M + lc[a]];
        if constexpr (PAR)
          laplace_element_parallelepiped_n<T, R>(X, u, k, v);
        else
          laplace_element_n<T, R>(X, u, k, v);
#pragma unroll
        for (int c = 0; c < R; ++c) {
          if ((done_m >> c) & 1) continue;
#pragma unroll
          for (int a = 0; a < 8; ++a)
            __hip_atomic_fetch_add(&acc[c * M + lc[a]], double(v[c][a]), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
        }
      }
    }
    __syncthreads();
    for (int ib = on ? L.sub : nm; ib < nm; ib += kStage * L.NL) {
      int32_t sl[kStage];
#pragma unroll
      for (int u = 0; u < kStage; ++u) sl[u] = P.pos[n0 + min(ib + u * L.NL, nm - 1)];
#pragma unroll
      for (int u = 0; u < kStage; ++u) {
        const int i = ib + u * L.NL;
        if (i >= nm || sl[u] < 0) continue;
        const double vv = acc[L.c * M + i];
        put(&q[int64_t(sl[u]) * R + L.c], T(vv));
        pq += double(sP[L.c * M + i]) * vv;
      }
    }
    __syncthreads();
  }
}

// The sums of the slots of U nodes (slots [e0, e1) of each, in order) for one right-hand
// side; the first two slots of every node are requested together, then two at a time.
template <int R, int U, typename T>
__device__ __forceinline__ void slot_sums(const BProb &P, const T *q, int c,
                                          const uint32_t (&e0)[U], const uint32_t (&e1)[U],
                                          double (&sum)[U]) {
  int m = 0;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    m = max(m, int(e1[u] - e0[u]));
    sum[u] = 0.0;
  }
  const int64_t last = P.n_slots - 1;
  for (int k = 0; k < m; k += 2) {
    T v[U][2];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int d = 0; d < 2; ++d) {
        v[u][d] = T(0);
        if (e0[u] + k + d < e1[u]) v[u][d] = get(&q[min(int64_t(e0[u]) + k + d, last) * R + c]);
      }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int d = 0; d < 2; ++d)
        if (e0[u] + k + d < e1[u]) sum[u] += double(v[u][d]);
  }
}

template <int R, bool MIXED, bool PAR, int NW>
__global__ __launch_bounds__(kW * NW, NW > 1 ? 3 : 1) void k_batched_pcg(
    const BProb *__restrict__ probs, int nprob, const int *__restrict__ wg_prob, double tol2,
    int maxit, double delta2, int *error) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int lane = threadIdx.x & (kW - 1), wave = threadIdx.x / kW;
  const BProb P = load_problem(probs + wg_prob[blockIdx.x]);
  const int me = int(blockIdx.x) - P.wg0;
  const int nwg = P.nwg;
  using TP = typename std::conditional<MIXED, float, double>::type;  // precision of p, q
  double *acc = reinterpret_cast<double *>(smem_raw);                  // [R][max_nodes]
  TP *sP = reinterpret_cast<TP *>(acc + R * P.max_nodes);              // [R][max_nodes]
  uint32_t *sId = reinterpret_cast<uint32_t *>(sP + R * P.max_nodes);  // [max_nodes]
  auto part = [&](int slot, int r) { return P.part + (int64_t(slot) * R + r) * nwg; };
  // node range of this workgroup for the vector phases
  const int64_t chunk = (P.nn + nwg - 1) / nwg;
  const int64_t i0 = min(P.nn, int64_t(me) * chunk), i1 = min(P.nn, i0 + chunk);
  static_assert(NW == 1 || PAR, "several waves per workgroup: parallelepiped tiles");
  const Lanes<R, NW> L;
  constexpr int kU = Lanes<R, NW>::kU;

  // ---- init: x = 0, r = b, both direction buffers 0 (nodes in no tile keep p = 0);
  // partials rho_0 = b^T D^-1 b, b.b
  {
    double v_rho = 0.0, v_bb = 0.0;
    for (int64_t i = L.act ? i0 + L.sub : i1; i < i1; i += L.NL) {
      const int64_t o = i * R + L.c;
      const double wi = P.w[i], bi = P.b[o];
      if constexpr (MIXED)
        put(&P.x[o], 0.0);
      else
        P.x[o] = 0.0;
      put(&P.r[o], bi);
      if constexpr (MIXED) {
        put(&P.p32[0][o], 0.0f);
        put(&P.p32[1][o], 0.0f);
      } else {
        put(&P.p[0][o], 0.0);
        put(&P.p[1][o], 0.0);
      }
      v_rho += bi * (wi * bi);
      v_bb += bi * bi;
    }
    v_rho = group_sum<R, NW>(v_rho, lane);
    v_bb = group_sum<R, NW>(v_bb, lane);
    if (threadIdx.x < R) {
      put(&part(kRho0, lane)[me], v_rho);
      put(&part(kBB, lane)[me], v_bb);
    }
  }
  // Each lane keeps the scalars of its right-hand side (the lanes of one side hold the same
  // bits); done_m has a bit for each finished side.
  double rho = 0.0, bb = 0.0;
  unsigned gen = 0;  // barriers so far
  if (!group_sync<R, NW>(P, unsigned(me), unsigned(nwg), error, gen, kRho0, kBB, rho, bb)) return;
  constexpr int kAll = (1 << R) - 1;
  bool done = !(bb > 0.0);
  int it_done = 0, st = Q1_OK, nref = 0;
  double rr_last = bb, rr_ref = bb, beta = 0.0;
  int done_m = int(__ballot(done)) & kAll;  // lane c < R holds side c

  for (int it = 1; it <= maxit && done_m != kAll; ++it) {
    // ---- P1: p = D^-1 r + beta p_old and q = A p over this wave's tiles, with the
    // partials of p^T A p (element energies, Dirichlet p^2).  The direction
    // buffers of this iteration and the previous one are selected, not indexed,
    // so that the problem record stays in registers.
    const bool odd = (it & 1) != 0;
    double *const p64 = odd ? P.p[1] : P.p[0];
    double *const p64_old = odd ? P.p[0] : P.p[1];
    float *const p32 = odd ? P.p32[1] : P.p32[0];
    float *const p32_old = odd ? P.p32[0] : P.p32[1];
    double v_pq = 0.0;
    if constexpr (MIXED)
      update_apply_phase<float, R, PAR, NW>(P, me, nwg, lane, wave, acc, sId, sP, P.xyz32, P.coef32,
                                        p32_old, p32, P.q32, done_m, beta, it == 1, v_pq);
    else
      update_apply_phase<double, R, PAR, NW>(P, me, nwg, lane, wave, acc, sId, sP, P.xyz, P.coef_t,
                                         p64_old, p64, P.q, done_m, beta, it == 1, v_pq);
    v_pq = group_sum<R, NW>(v_pq, lane);
    if (threadIdx.x < R) put(&part(kPQ, lane)[me], v_pq);
    double pq = 0.0, none = 0.0;
    if (!group_sync<R, NW>(P, unsigned(me), unsigned(nwg), error, gen, kPQ, -1, pq, none)) return;

    // ---- P2: alpha, x, r; partials rho', r.r
    double alpha = 0.0;
    if (!done) {
      if (!(pq > 0.0) || !isfinite(pq) || !isfinite(rho)) {
        done = true;
        st = Q1_EBREAKDOWN;
        it_done = it - 1;
      } else {
        alpha = rho / pq;
      }
    }
    {
      double v_rho = 0.0, v_rr = 0.0;
      const bool on = L.act && !done;
      for (int64_t ib = on ? i0 + L.sub : i1; ib < i1; ib += kU * L.NL) {
        uint32_t e0[kU], e1[kU];
        bool fx[kU];
        double wv[kU], po[kU], qo[kU], xo[kU], ro[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          const int64_t i = min(ib + u * L.NL, i1 - 1);
          e0[u] = P.nptr[i];
          e1[u] = P.nptr[i + 1];
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          const int64_t i = min(ib + u * L.NL, i1 - 1), o = i * R + L.c;
          wv[u] = P.w[i];
          if constexpr (MIXED) {
            po[u] = double(get(&p32[o]));
            xo[u] = get(&P.x[o]);
          } else {
            po[u] = get(&p64[o]);
            xo[u] = P.x[o];
          }
          ro[u] = get(&P.r[o]);
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          fx[u] = (e0[u] >> 31) != 0;
          e0[u] &= 0x7fffffffu;
          e1[u] &= 0x7fffffffu;
        }
        if constexpr (MIXED)
          slot_sums<R>(P, P.q32, L.c, e0, e1, qo);
        else
          slot_sums<R>(P, P.q, L.c, e0, e1, qo);
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          const int64_t i = ib + u * L.NL, o = i * R + L.c;
          if (i >= i1) continue;
          if (fx[u]) qo[u] = po[u];
          const double xn = xo[u] + alpha * po[u], rn = ro[u] - alpha * qo[u];
          if constexpr (MIXED)
            put(&P.x[o], xn);
          else
            P.x[o] = xn;
          put(&P.r[o], rn);
          v_rho += rn * wv[u] * rn;
          v_rr += rn * rn;
        }
      }
      v_rho = group_sum<R, NW>(v_rho, lane);
      v_rr = group_sum<R, NW>(v_rr, lane);
      if (threadIdx.x < R) {
        put(&part(kRho, lane)[me], v_rho);
        put(&part(kRR, lane)[me], v_rr);
      }
    }
    double rho_n = 0.0, rr_n = 0.0;
    if (!group_sync<R, NW>(P, unsigned(me), unsigned(nwg), error, gen, kRho, kRR, rho_n, rr_n)) return;

    // ---- convergence and beta (the direction update runs with the next apply)
    bool refresh = false;
    beta = 0.0;
    if (!done) {
      rr_last = rr_n;
      if constexpr (MIXED) {
        // the recurrence only triggers a refresh; convergence is decided on b - A64 x
        if (!isfinite(rr_n)) {
          done = true;
          st = Q1_EBREAKDOWN;
          it_done = it;
        } else if (rr_n <= fmax(delta2 * rr_ref, 0.5 * tol2 * bb) || it >= maxit) {
          refresh = true;
        } else {
          beta = rho_n / rho;
          rho = rho_n;
        }
      } else {
        if (rr_n <= tol2 * bb || !isfinite(rr_n) || it >= maxit) {
          done = true;
          st = rr_n <= tol2 * bb ? Q1_OK : (!isfinite(rr_n) ? Q1_EBREAKDOWN : Q1_ENOCONV);
          it_done = it;
        } else {
          beta = rho_n / rho;
          rho = rho_n;
        }
      }
    }
    if constexpr (MIXED) {
      const int refresh_m = int(__ballot(refresh)) & kAll;
      if (refresh_m) {
        // R1: t = A64 x for the refreshed right-hand sides (FP64 geometry and coefficients)
        apply_phase<double, R, PAR, NW>(P, me, nwg, lane, wave, acc, sId, P.xyz, P.coef_t, P.x, P.t, ~refresh_m);
        if (!problem_barrier<R, NW>(P, unsigned(me), unsigned(nwg), error, gen)) return;
        // R2: r = b - A64 x (Dirichlet rows are the identity); partials rho', r.r
        double v_rho = 0.0, v_rr = 0.0;
        for (int64_t i = L.act && refresh ? i0 + L.sub : i1; i < i1; i += L.NL) {
          const int64_t o = i * R + L.c;
          const uint32_t f = P.nptr[i];
          const uint32_t e0[1] = {f & 0x7fffffffu}, e1[1] = {P.nptr[i + 1] & 0x7fffffffu};
          double t[1];
          slot_sums<R>(P, P.t, L.c, e0, e1, t);
          const double rn = P.b[o] - (f >> 31 ? get(&P.x[o]) : t[0]);
          put(&P.r[o], rn);
          v_rho += rn * P.w[i] * rn;
          v_rr += rn * rn;
        }
        v_rho = group_sum<R, NW>(v_rho, lane);
        v_rr = group_sum<R, NW>(v_rr, lane);
        if (threadIdx.x < R) {
          put(&part(kRho, lane)[me], v_rho);
          put(&part(kRR, lane)[me], v_rr);
        }
        if (!group_sync<R, NW>(P, unsigned(me), unsigned(nwg), error, gen, kRho, kRR, rho_n, rr_n))
          return;
        // R3: decide on the true residual; otherwise continue from it with p kept
        if (refresh) {
          rr_last = rr_n;
          ++nref;
          if (rr_n <= tol2 * bb || !isfinite(rr_n) || it >= maxit) {
            done = true;
            st = rr_n <= tol2 * bb ? Q1_OK : (!isfinite(rr_n) ? Q1_EBREAKDOWN : Q1_ENOCONV);
            it_done = it;
          } else {
            rr_ref = rr_n;
            beta = rho_n / rho;
            rho = rho_n;
          }
        }
      }
    }
    done_m = int(__ballot(done)) & kAll;
  }
  if (me == 0 && threadIdx.x < R) {
    const int c = threadIdx.x;
    P.iters[c] = it_done;
    P.status[c] = done ? st : Q1_ENOCONV;
    P.rr[c] = rr_last;
    P.bb[c] = bb;
    P.nref[c] = nref;
  }
}

// interleave: dst[i*R + c] = src_c[i]; and back
__global__ void k_interleave(int64_t n, int R, int c, const double *__restrict__ src,
                             double *__restrict__ dst) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) dst[i * R + c] = src[i];
}
__global__ void k_deinterleave(int64_t n, int R, int c, const double *__restrict__ src,
                               double *__restrict__ dst) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src[i * R + c];
}
__global__ void k_invert(int64_t n, double *__restrict__ d) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) d[i] = d[i] != 0.0 ? 1.0 / d[i] : 0.0;  // 0 on zero rows (unreferenced nodes)
}

__global__ void k_to_f32(int64_t n, const double *__restrict__ src, float *__restrict__ dst) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = float(src[i]);
}

template <int R, bool MIXED, bool PAR, int NW>
int run_batched(const std::vector<BProb> &hp, const std::vector<int> &wg_prob, double tol2,
                int maxit, double delta2, size_t lds, hipStream_t s, int *d_error) {
  BProb *dp = nullptr;
  int *dwg = nullptr;
  Q1_HIP(hipMalloc(&dp, hp.size() * sizeof(BProb)));
  Q1_HIP(hipMalloc(&dwg, wg_prob.size() * sizeof(int)));
  Q1_HIP(hipMemcpy(dp, hp.data(), hp.size() * sizeof(BProb), hipMemcpyHostToDevice));
  Q1_HIP(hipMemcpy(dwg, wg_prob.data(), wg_prob.size() * sizeof(int), hipMemcpyHostToDevice));
  int nprob = int(hp.size());
  void *args[] = {&dp, &nprob, &dwg, &tol2, &maxit, &delta2, &d_error};
  hipError_t e = hipLaunchCooperativeKernel(
      reinterpret_cast<const void *>(k_batched_pcg<R, MIXED, PAR, NW>),
      dim3(unsigned(wg_prob.size())), dim3(kW * NW), args, unsigned(lds), s);
  hipError_t e2 = hipStreamSynchronize(s);
  (void)hipFree(dp);
  (void)hipFree(dwg);
  if (e != hipSuccess) return fail(Q1_EHIP, "cooperative launch failed: %s", hipGetErrorString(e));
  if (e2 != hipSuccess) return fail(Q1_EHIP, "batched PCG: %s", hipGetErrorString(e2));
  return Q1_OK;
}

template <int R, bool MIXED, bool PAR, int NW>
int max_coresident(size_t lds) {
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
          &per_cu, reinterpret_cast<const void *>(k_batched_pcg<R, MIXED, PAR, NW>), kW * NW, lds) !=
      hipSuccess)
    return 0;
  int dev = 0, cus = 0;
  (void)hipGetDevice(&dev);
  (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  return per_cu * cus;
}

template <bool MIXED, bool PAR, int NW>
int coresident_for(int nrhs, size_t lds) {
  switch (nrhs) {
    case 1: return max_coresident<1, MIXED, PAR, NW>(lds);
    case 2: return max_coresident<2, MIXED, PAR, NW>(lds);
    case 3: return max_coresident<3, MIXED, PAR, NW>(lds);
    default: return max_coresident<4, MIXED, PAR, NW>(lds);
  }
}

template <bool MIXED, bool PAR, int NW>
int run_for(int nrhs, const std::vector<BProb> &hp, const std::vector<int> &wg_prob, double tol2,
            int maxit, double delta2, size_t lds, hipStream_t s, int *d_error) {
  switch (nrhs) {
    case 1: return run_batched<1, MIXED, PAR, NW>(hp, wg_prob, tol2, maxit, delta2, lds, s, d_error);
    case 2: return run_batched<2, MIXED, PAR, NW>(hp, wg_prob, tol2, maxit, delta2, lds, s, d_error);
    case 3: return run_batched<3, MIXED, PAR, NW>(hp, wg_prob, tol2, maxit, delta2, lds, s, d_error);
    default: return run_batched<4, MIXED, PAR, NW>(hp, wg_prob, tol2, maxit, delta2, lds, s, d_error);
  }
}

// f(MIXED, PAR, NW as integral constants) of the form to run
template <class F>
auto with_form(bool mixed, bool par, int nw, F f) {
  using t = std::true_type;
  using n = std::false_type;
  using one = std::integral_constant<int, 1>;
  using four = std::integral_constant<int, 4>;
  if (par && nw == 4) return mixed ? f(t{}, t{}, four{}) : f(n{}, t{}, four{});
  if (par) return mixed ? f(t{}, t{}, one{}) : f(n{}, t{}, one{});
  return mixed ? f(t{}, n{}, one{}) : f(n{}, n{}, one{});
}

// Shared host side of the FP64 and mixed-precision batched solvers.
int batched_impl(const char *name, bool mixed, int nprob, q1_op *const *ops, int nrhs,
                 const double *const *b_d, double *const *x_d, double rtol, double delta,
                 int maxit, q1_stats *st, hipStream_t s) {
  Q1_CHECK(nprob > 0 && ops && b_d && x_d, Q1_EINVAL, "%s: bad arguments", name);
  Q1_CHECK(nrhs >= 1 && nrhs <= kRmax, Q1_EINVAL, "%s: 1 <= nrhs <= %d", name, kRmax);
  Q1_CHECK(rtol >= 0 && maxit >= 0, Q1_EINVAL, "%s: bad tolerance or limit", name);
  Q1_CHECK(!mixed || (delta > 0 && delta < 1), Q1_EINVAL, "%s: need 0 < delta < 1", name);
  int max_nodes = 0;
  for (int p = 0; p < nprob; ++p) {
    const Op *o = reinterpret_cast<const Op *>(ops[p]);
    Q1_CHECK(o, Q1_EINVAL, "%s: NULL operator %d", name, p);
    Q1_CHECK(o->physics == Q1_LAPLACE && o->dtype == Q1_F64 && o->variant == Q1_V_LDS_TILE,
             Q1_EUNSUPPORTED, "%s: operator %d must be an FP64 scalar-Laplace LDS-tile operator",
             name, p);
    for (int c = 0; c < nrhs; ++c)
      Q1_CHECK(b_d[p * nrhs + c] && x_d[p * nrhs + c], Q1_EINVAL, "%s: NULL vector", name);
    max_nodes = std::max(max_nodes, o->tiles.max_nodes);
  }
  // LDS per wave: FP64 accumulators, the staged directions (FP32 in the mixed form)
  // and the node words
  const size_t lds = size_t(max_nodes) * (size_t(nrhs) * sizeof(double) +
                                          size_t(nrhs) * (mixed ? sizeof(float) : sizeof(double)) +
                                          sizeof(uint32_t));
  bool par = true;  // every tile of every problem a parallelepiped tile
  for (int p = 0; p < nprob; ++p) par = par && reinterpret_cast<const Op *>(ops[p])->tiles.all_affine;
  // four waves per workgroup on parallelepiped tiles, where one workgroup per problem fits so
  auto cap_of = [&](int nw) {
    return with_form(mixed, par, nw, [&](auto m, auto p, auto w) {
      return coresident_for<decltype(m)::value, decltype(p)::value, decltype(w)::value>(nrhs, lds);
    });
  };
  int nw = par ? 4 : 1, cap = cap_of(nw);
  if (cap < nprob) cap = cap_of(nw = 1);
  Q1_CHECK(cap >= nprob, Q1_EUNSUPPORTED,
           "%s: %d problems need one co-resident wave each, but only %d fit", name, nprob, cap);
  // waves per problem in proportion to its expected work, at least one each:
  // elements times iterations, and Jacobi-PCG iterations on an n^3 grid grow
  // like n, so the weight is n_elems^(4/3)
  std::vector<int> nwg(nprob, 1);
  int spare = cap - nprob;
  double wsum = 0.0;
  for (int p = 0; p < nprob; ++p)
    wsum += std::pow(double(reinterpret_cast<const Op *>(ops[p])->n_elems), 4.0 / 3.0);
  for (int p = 0; p < nprob; ++p) {
    const Op *o = reinterpret_cast<const Op *>(ops[p]);
    const double wp = std::pow(double(o->n_elems), 4.0 / 3.0);
    const int extra = int(double(spare) * wp / std::max(1.0, wsum));
    nwg[p] += std::min(extra, std::max(0, o->tiles.n_tiles - 1));
  }
  // device workspace per problem
  std::vector<void *> allocs;
  struct Guard {
    std::vector<void *> &a;
    ~Guard() {
      for (void *p : a) (void)hipFree(p);
    }
  } guard{allocs};
  auto dalloc = [&](void **ptr, size_t bytes) -> int {
    Q1_HIP(hipMalloc(ptr, std::max<size_t>(bytes, 8)));
    allocs.push_back(*ptr);
    return Q1_OK;
  };
  int *d_error = nullptr;
  int rc;
  if ((rc = dalloc(reinterpret_cast<void **>(&d_error), sizeof(int)))) return rc;
  Q1_HIP(hipMemsetAsync(d_error, 0, sizeof(int), s));
  std::vector<BProb> hp(nprob);
  std::vector<int> wg_prob;
  int *d_iters = nullptr, *d_status = nullptr, *d_nref = nullptr;
  double *d_rr = nullptr, *d_bb = nullptr;
  const size_t nres = size_t(nprob) * nrhs;
  if ((rc = dalloc(reinterpret_cast<void **>(&d_iters), nres * sizeof(int))) ||
      (rc = dalloc(reinterpret_cast<void **>(&d_status), nres * sizeof(int))) ||
      (rc = dalloc(reinterpret_cast<void **>(&d_nref), nres * sizeof(int))) ||
      (rc = dalloc(reinterpret_cast<void **>(&d_rr), nres * sizeof(double))) ||
      (rc = dalloc(reinterpret_cast<void **>(&d_bb), nres * sizeof(double))))
    return rc;
  auto grid = [](int64_t n) { return dim3(unsigned((n + 255) / 256)); };
  for (int p = 0; p < nprob; ++p) {
    Op &o = *reinterpret_cast<Op *>(ops[p]);
    const TileMap &tm = o.tiles;
    BProb &B = hp[p];
    B = BProb{};
    const int64_t n = o.n_nodes;
    B.nn = n;
    B.n_tiles = tm.n_tiles;
    B.max_nodes = max_nodes;
    B.node_ptr = tm.node_ptr;
    B.nodes = tm.nodes;
    B.tile_step = tm.tile_step;
    B.lconn = reinterpret_cast<const uint4 *>(tm.lconn);
    B.coef_t = static_cast<const double *>(tm.coef_t);
    B.xyz = static_cast<const double *>(o.xyz);
    Q1_CHECK(n < int64_t(kIdMaskOwnB) && tm.onodes, Q1_EUNSUPPORTED, "%s: operator %d has %lld nodes (at most %u)",
             name, p, (long long)n, kIdMaskOwnB);
    B.onodes = tm.onodes;
    B.nptr = tm.nptr;
    B.pos = tm.pos;
    B.n_slots = tm.n_node_slots;
    const size_t ns = size_t(tm.n_node_slots) * nrhs;
    const size_t nv = size_t(n) * nrhs;
    double *vec[6] = {nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};
    for (int v = 0; v < 6; ++v) {
      if (mixed && v >= 3) continue;  // p, q are FP32 in the mixed form
      if ((rc = dalloc(reinterpret_cast<void **>(&vec[v]), (v == 3 ? ns : nv) * sizeof(double))))
        return rc;
    }
    B.b = vec[0]; B.x = vec[1]; B.r = vec[2]; B.q = vec[3]; B.p[0] = vec[4]; B.p[1] = vec[5];
    if (mixed) {
      // FP32 copies of the geometry and of the lane-ordered coefficients: the FP32 operator
      float *xyz32 = nullptr, *coef32 = nullptr;
      const int64_t ncoef = tm.n_steps * kW;
      if ((rc = dalloc(reinterpret_cast<void **>(&B.p32[0]), nv * sizeof(float))) ||
          (rc = dalloc(reinterpret_cast<void **>(&B.p32[1]), nv * sizeof(float))) ||
          (rc = dalloc(reinterpret_cast<void **>(&B.q32), ns * sizeof(float))) ||
          (rc = dalloc(reinterpret_cast<void **>(&B.t), ns * sizeof(double))) ||
          (rc = dalloc(reinterpret_cast<void **>(&xyz32), size_t(3 * n) * sizeof(float))) ||
          (rc = dalloc(reinterpret_cast<void **>(&coef32), size_t(ncoef) * sizeof(float))))
        return rc;
      hipLaunchKernelGGL(k_to_f32, grid(3 * n), dim3(256), 0, s, 3 * n, B.xyz, xyz32);
      hipLaunchKernelGGL(k_to_f32, grid(ncoef), dim3(256), 0, s, ncoef, B.coef_t, coef32);
      B.xyz32 = xyz32;
      B.coef32 = coef32;
    }
    double *w = nullptr;
    if ((rc = dalloc(reinterpret_cast<void **>(&w), size_t(n) * sizeof(double)))) return rc;
    if ((rc = launch_diag(o, w, s))) return rc;
    hipLaunchKernelGGL(k_invert, grid(n), dim3(256), 0, s, n, w);
    B.w = w;
    for (int c = 0; c < nrhs; ++c)
      hipLaunchKernelGGL(k_interleave, grid(n), dim3(256), 0, s, n, nrhs, c, b_d[p * nrhs + c],
                         B.b);
    if ((rc = dalloc(reinterpret_cast<void **>(&B.part), size_t(kSlots) * nrhs * nwg[p] *
                                                             sizeof(double))))
      return rc;
    if ((rc = dalloc(reinterpret_cast<void **>(&B.bar), kBarWords * sizeof(unsigned)))) return rc;
    if ((rc = dalloc(reinterpret_cast<void **>(&B.tot), 2 * kSub * 2 * nrhs * sizeof(double))))
      return rc;
    Q1_HIP(hipMemsetAsync(B.bar, 0, kBarWords * sizeof(unsigned), s));
    B.wg0 = int(wg_prob.size());
    B.nwg = nwg[p];
    for (int k = 0; k < nwg[p]; ++k) wg_prob.push_back(p);
    B.iters = d_iters + p * nrhs;
    B.status = d_status + p * nrhs;
    B.nref = d_nref + p * nrhs;
    B.rr = d_rr + p * nrhs;
    B.bb = d_bb + p * nrhs;
  }
  Q1_HIP(hipGetLastError());
  Q1_HIP(hipStreamSynchronize(s));
  const auto t_setup = std::chrono::steady_clock::now();
  const double tol2 = rtol * rtol, delta2 = delta * delta;
  rc = with_form(mixed, par, nw, [&](auto m, auto p, auto w) {
    return run_for<decltype(m)::value, decltype(p)::value, decltype(w)::value>(
        nrhs, hp, wg_prob, tol2, maxit, delta2, lds, s, d_error);
  });
  if (rc) return rc;
  const auto t_solve = std::chrono::steady_clock::now();
  int h_error = 0;
  Q1_HIP(hipMemcpy(&h_error, d_error, sizeof(int), hipMemcpyDeviceToHost));
  Q1_CHECK(h_error == 0, Q1_EHIP, "%s: a problem barrier timed out", name);
  for (int p = 0; p < nprob; ++p)
    for (int c = 0; c < nrhs; ++c)
      hipLaunchKernelGGL(k_deinterleave, grid(hp[p].nn), dim3(256), 0, s, hp[p].nn, nrhs, c,
                         hp[p].x, x_d[p * nrhs + c]);
  Q1_HIP(hipGetLastError());
  std::vector<int> h_it(nres), h_st(nres), h_nref(nres);
  std::vector<double> h_rr(nres), h_bb(nres);
  Q1_HIP(hipMemcpy(h_it.data(), d_iters, nres * sizeof(int), hipMemcpyDeviceToHost));
  Q1_HIP(hipMemcpy(h_st.data(), d_status, nres * sizeof(int), hipMemcpyDeviceToHost));
  Q1_HIP(hipMemcpy(h_nref.data(), d_nref, nres * sizeof(int), hipMemcpyDeviceToHost));
  Q1_HIP(hipMemcpy(h_rr.data(), d_rr, nres * sizeof(double), hipMemcpyDeviceToHost));
  Q1_HIP(hipMemcpy(h_bb.data(), d_bb, nres * sizeof(double), hipMemcpyDeviceToHost));
  const double secs = std::chrono::duration<double>(t_solve - t_setup).count();
  int worst = Q1_OK;
  for (size_t k = 0; k < nres; ++k) {
    if (st) {
      st[k].iters = h_it[k];
      st[k].status = h_st[k];
      st[k].rel_res = h_bb[k] > 0 ? std::sqrt(h_rr[k] / h_bb[k]) : 0.0;
      st[k].true_rel_res = st[k].rel_res;
      st[k].seconds = secs;       // one launch for all solves
      st[k].fallback_at = -1;
      st[k].outer_iters = h_nref[k];
    }
    if (h_st[k] == Q1_EBREAKDOWN) worst = Q1_EBREAKDOWN;
    else if (h_st[k] == Q1_ENOCONV && worst == Q1_OK) worst = Q1_ENOCONV;
  }
  return worst;
}

}  // namespace
}  // namespace q1

using namespace q1;

extern "C" int q1_batched_pcg(int nprob, q1_op *const *ops, int nrhs,
                              const double *const *b_d, double *const *x_d, double rtol,
                              int maxit, q1_stats *st, void *stream) {
  return batched_impl("q1_batched_pcg", false, nprob, ops, nrhs, b_d, x_d, rtol, 0.0, maxit, st,
                      static_cast<hipStream_t>(stream));
}

extern "C" int q1_batched_mpcg(int nprob, q1_op *const *ops, int nrhs,
                               const double *const *b_d, double *const *x_d, double rtol,
                               double delta, int maxit, q1_stats *st, void *stream) {
  return batched_impl("q1_batched_mpcg", true, nprob, ops, nrhs, b_d, x_d, rtol, delta, maxit, st,
                      static_cast<hipStream_t>(stream));
}
