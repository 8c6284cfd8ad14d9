// Docking kernels for gfx950: restart placement, rigid rotation / translation
// scans, greedy torsion scans with the intramolecular clash check, nearest-voxel
// scan scores, trilinear final score, per-ligand top-k.
//
// Mapping.  One wavefront docks one restart (ligand, r).  A scan first bounds the
// score of every group of neighbouring samples (one group per lane) from above,
// then scores the samples of the groups whose bound exceeds the current pose's
// score, one sample per lane: the selected sample is that of a scan over every
// sample, at about half the lookups.  Where no bound pass pays or is possible, scans
// score every sample, several per lane.  Each lane loops over the atoms of the scan,
// reading per-atom scan data that the wavefront staged in LDS (broadcast reads), and
// accumulates nearest-voxel values gathered from the L2-resident grid.  The pose lives in registers, atom a = 64 s + lane in slot s < NSLOT.
// The best sample comes from a DPP/readlane reduction (lowest index among equal
// scores).  Torsion samples are tested for intramolecular clashes against a
// pruned list of the pairs that can clash at some angle.
//
// What bounds it: each scan's fixed part and the latency of its gathers.  Vector
// issue runs at 0.53 of its limit, the address unit is busy 84 % of the time (about
// 27 cache accesses for 64 scattered lookups), L2 hits 99.1 % (mixed library).
// Against scoring every sample, four per lane: 20 000 mixed ligands of 256
// restarts and 256 samples, two restarts per item, 457 -> 417 ms; 4 000 ligands of
// up to 160 atoms in the default tuning 160 -> 91 ms, one ligand 2.17 -> 0.28 ms (with
// shorter items for small launches).
//
// Outputs.  Each restart records its final score and the selected sample of
// every scan (a few bytes per scan); the per-ligand top-k then rebuilds the k
// kept poses by replaying their moves with the same apply functions the scans
// use, so the poses are bit-identical to the docked ones without storing every
// restart's coordinates.
//
// Arithmetic contract (matches the CPU oracle bit for bit): FP32, explicit
// fmaf, no contraction; sums of quantised grid values are exact in any order,
// the final trilinear sum runs in atom order.
#include "lg_device.h"

#include <algorithm>
#include <climits>
#include <type_traits>

namespace lg {

template <int NSLOT>
struct PoseReg {
  float x[3][NSLOT];
  float piv[3];
};

// ---- moves: the selected sample of a scan applied to the pose ----------------
// Rotation by sample j, (cos, sin) = cs, about lab axis E through the pivot.
template <int NSLOT, int E>
__device__ __forceinline__ void apply_rot(float2 cs, PoseReg<NSLOT>& p, int j) {
  constexpr int P = (E + 1) % 3, Q = (E + 2) % 3;
  if (j == 0) return;
  const float pP = p.piv[P], pQ = p.piv[Q];
  const float c = cs.x, sn = cs.y;
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) {
    float vp = p.x[P][s] - pP, vq = p.x[Q][s] - pQ;
    float np = fmaf(c, vp, -(sn * vq));
    float nq = fmaf(sn, vp, c * vq);
    p.x[P][s] = pP + np;
    p.x[Q][s] = pQ + nq;
  }
}

// Translation by sample j along lab axis E (the pivot moves along).
template <int NSLOT, int E>
__device__ __forceinline__ void apply_trans(const DockDev& D, PoseReg<NSLOT>& p, int j) {
  if (j == 0) return;
  const int m = j < D.T / 2 ? j : j - D.T;
  const float dd = D.delta * (float)m;
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) p.x[E][s] = p.x[E][s] + dd;
  p.piv[E] = p.piv[E] + dd;
  // update the pivot here: left to itself the compiler sinks this add past the
  // torsion scans and keeps dd alive (in scratch) until then
  asm volatile("" : "+v"(p.piv[E]));
}

// Bond k's axis at the current pose: pivot atom a, unit direction u.
struct BondAxis {
  int a, b;
  float xa, ya, za, ux, uy, uz;
};

template <int NSLOT>
__device__ __forceinline__ BondAxis bond_axis(uint32_t ab, float inv_len, const PoseReg<NSLOT>& p, int k) {
  BondAxis A;
  const uint32_t v = (uint32_t)__builtin_amdgcn_readlane((int)ab, k);
  A.a = (int)(v & 0xFFFFu);
  A.b = (int)(v >> 16);
  const float il = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(inv_len), k));
  A.xa = atom_value(p.x[0], A.a);
  A.ya = atom_value(p.x[1], A.a);
  A.za = atom_value(p.x[2], A.a);
  const float xb = atom_value(p.x[0], A.b), yb = atom_value(p.x[1], A.b), zb = atom_value(p.x[2], A.b);
  A.ux = (xb - A.xa) * il;
  A.uy = (yb - A.ya) * il;
  A.uz = (zb - A.za) * il;
  return A;
}

// Rotation of the moving fragment of bond k (its atoms other than b) by the
// matrix Mj about the axis through a.
template <int NSLOT>
__device__ __forceinline__ void apply_tors(PoseReg<NSLOT>& p, const BondAxis& A, const float (&Mj)[9],
                                           const bool (&mv)[NSLOT]) {
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) {
    if (mv[s]) {
      float y0, y1, y2;
      mat_apply(Mj, p.x[0][s] - A.xa, p.x[1][s] - A.ya, p.x[2][s] - A.za, y0, y1, y2);
      p.x[0][s] = A.xa + y0;
      p.x[1][s] = A.ya + y1;
      p.x[2][s] = A.za + y2;
    }
  }
}

// Moving atoms of bond k held by this lane: in F_k, not the axis atom b.
template <int NSLOT>
__device__ __forceinline__ void moving_atoms(const uint32_t (&mk)[NSLOT], int N, int k, int b, bool (&mv)[NSLOT]) {
  const int lane = lane_id();
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) {
    const int at = s * 64 + lane;
    mv[s] = at < N && ((mk[s] >> k) & 1u) && at != b;
  }
}

// Square root for radii that only bound something: the hardware's one-ulp root.
// The margins around them (0.05 A of the pair prune, thousandths of a node of
// the windows) are orders of magnitude above an ulp of a radius; no exact test
// uses a root.
__device__ __forceinline__ float prune_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }

// ---- samples of a launch -------------------------------------------------------
// A scan's samples are taken in groups of neighbours, at most 64 groups, one per
// lane.  What every scan of a launch needs to know of them; uniform but for the
// lane's group centre.
struct Samples {
  int A;              // angle samples
  int GA, nga;        // rotations and torsions: samples per group, groups
  int GT, ngt;        // translations, in order of displacement
  int tsub;           // lanes that share a translation group in the bound pass (log2): 0, 1, 2
  int gt0;            // translation group of sample 0
  bool bound_a, bound_t;   // rotations and torsions, translations: a bound pass pays (and is possible)
  float dlow;         // least displacement of the lane's translation group
  float radius;       // largest |(cos, sin)| of a sample (1 up to rounding)
  float chord;        // every sample of a group lies within chord of its centre, in (cos, sin)
  float cc, cs;       // centre of the lane's group: the mean of its two middle samples
  const float2* ang;  // (cos, sin) of every sample, in LDS
};

// How far apart two FP32 sums of the same n grid values can be, whatever their
// orders of addition (zero on grids whose sums are exact; the bound holds for all).
// Infinite wherever n values can add up past the largest float, since n * n * vmax
// does so first: a sum that ran to infinity on the way is above any finite bound.
__device__ __forceinline__ float sum_slack(const GridDev& G, int n) { return G.vmax * (float)(n * n) * 4.8e-7f; }

// Whether translation samples, GT to a group, have bounds in a grid.  A group spans less
// than one node, also after the rounding of x + d and of the displacements (T / 2 steps
// at most): |x| / h inside the grid is at most |c0| + n.  And no sum overflows: the
// current pose's could be infinite in one order of addition, across the lanes, and not
// in the other, its score as a sample.
__device__ __forceinline__ bool translation_bounds(const GridDev& G, const DockDev& D, int GT) {
  const float far = fmaxf(fmaxf(fabsf(G.c0[0]) + G.fn[0], fabsf(G.c0[1]) + G.fn[1]), fabsf(G.c0[2]) + G.fn[2]);
  const float steps = fmaf(1.2e-7f, (float)D.T, (float)(GT - 1));
  return fmaf(fabsf(D.delta) * G.inv_h, steps, 2.4e-7f * far) <= 0.998f &&
         sum_slack(G, LG_MAX_ATOMS) < __builtin_inff();
}

__device__ __forceinline__ void load_samples(const GridDev& G, const DockDev& D, const float2* ang, Samples& sm) {
  const int lane = lane_id();
  sm.ang = ang;
  sm.A = D.A;
  sm.GA = (D.A + 63) >> 6;
  sm.nga = (D.A + sm.GA - 1) / sm.GA;
  // the bound pass costs most of a scoring pass and can save all but one of GA: with
  // two it does not pay (100 samples, 1 000 mixed ligands: 18.5 ms without, 20.5
  // with); 130 to 1024 samples have three passes and more
  sm.bound_a = sm.GA > 2;
  const int j0 = lane * sm.GA, cnt = min(sm.GA, D.A - j0);
  float far2 = 0.f, len2 = 0.f;
  bool odd = false;
  sm.cc = 1.f;
  sm.cs = 0.f;
  if (cnt > 0) {
    const float2 a = ang[j0 + ((cnt - 1) >> 1)], b = ang[j0 + (cnt >> 1)];
    sm.cc = 0.5f * (a.x + b.x);
    sm.cs = 0.5f * (a.y + b.y);
    for (int q = 0; q < cnt; ++q) {
      const float2 s = ang[j0 + q];
      const float dc = s.x - sm.cc, ds = s.y - sm.cs, d2 = fmaf(dc, dc, ds * ds);
      len2 = fmaxf(len2, fmaf(s.x, s.x, s.y * s.y));
      odd = odd || !(d2 < 1e30f) || !(len2 < 1e30f);
      far2 = fmaxf(far2, d2);
    }
  }
  // non-negative floats order as ints; a table with NaN or huge entries has no
  // bound (every test against these fails)
  const float w2 = __int_as_float(wave_reduce_i32(__float_as_int(far2), OpMax()));
  const float r2 = __int_as_float(wave_reduce_i32(__float_as_int(len2), OpMax()));
  const bool none = wave_any(odd);
  sm.chord = none ? __builtin_inff() : prune_sqrt(w2) * 1.0001f + 1e-6f;
  sm.radius = none ? __builtin_inff() : prune_sqrt(r2) * 1.0001f;
  // a group may not span a whole node: 16 groups where that holds, else 32 or 64
  sm.tsub = 2;
  for (;; --sm.tsub) {
    sm.GT = (D.T + (64 >> sm.tsub) - 1) >> (6 - sm.tsub);
    sm.bound_t = translation_bounds(G, D, sm.GT);
    if (sm.bound_t || sm.tsub == 0) break;
  }
  if (D.T <= 64) {   // one pass scores every sample
    sm.GT = 1;
    sm.bound_t = false;
  }
  sm.ngt = (D.T + sm.GT - 1) / sm.GT;
  const int mlo = D.T >= 2 ? D.T / 2 - D.T : 0;
  sm.gt0 = -mlo / sm.GT;
  const int g = lane & ((64 >> sm.tsub) - 1);
  const int m0 = min(g * sm.GT, D.T - 1) + mlo, m1 = min(g * sm.GT + sm.GT - 1, D.T - 1) + mlo;
  sm.dlow = fminf(D.delta * (float)m0, D.delta * (float)m1);
}

// n / d of small whole numbers, 0 <= n < 2^13, 1 <= d <= 64, from r = 1 / d (a few
// ulps off): n + 1/2 over d is at least 1/128 from any whole number.
__device__ __forceinline__ int small_div(int n, float r) { return (int)(((float)n + 0.5f) * r); }

// A uniform value in a vector register: arithmetic with a scalar operand issues
// at half rate.
__device__ __forceinline__ float in_vgpr(float x) {
  asm volatile("" : "+v"(x));
  return x;
}

// The selected sample of a scan: the largest score of an admissible sample, the
// lowest index among equal ones; sample 0, the current pose with score s0, is
// always admissible (ZERO: its group is among `alive` and it is scored with the
// others).  `alive` holds the groups (bit g: samples g G .. g G + G - 1
// in the scan's own order) that may beat s0, `bound` the lane's group's upper
// bound.  Each pass scores the samples of the next 64 / G groups, one per lane,
// in order of the groups; groups whose bound falls below the best score since
// found drop out.  index(pos) is the sample at a position of the scan's order,
// score(j) its exact score, refuse(j, better) the lanes whose sample is not
// admissible (asked only for samples that beat the best so far).  Dropping a
// group changes no result: a bound is at least the score of every sample of
// its group, rounding included (upper_bound).
template <bool ZERO, class Index, class Score, class Refuse>
__device__ __forceinline__ int select_sample(uint64_t alive, float bound, int G, int n, float s0, Index index,
                                             Score score, Refuse refuse) {
  const int lane = lane_id();
  const float rG = __builtin_amdgcn_rcpf((float)G);
  const int per = __builtin_amdgcn_readfirstlane(small_div(64, rG));
  const int idx = small_div(lane, rG), sub = lane - idx * G;
  int best = ZERO ? INT_MIN : orderable(s0), bj = ZERO ? INT_MAX : 0;
  while (alive) {
    // the next groups: the lane that holds the r-th of them passes its number to lane r
    const bool in = (alive >> lane) & 1u;
    const int before =
        __builtin_amdgcn_mbcnt_hi((uint32_t)(alive >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)alive, 0u));
    const bool now = in && before < per;
    const uint64_t taken = __ballot(now);
    const int cnt = __popcll(taken);
    const int rest = lane - (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(taken >> 32),
                                                           __builtin_amdgcn_mbcnt_lo((uint32_t)taken, 0u));
    const int held = __builtin_amdgcn_ds_permute((now ? before : cnt + rest) << 2, lane);
    const int g = __builtin_amdgcn_ds_bpermute(idx << 2, held);
    const int pos = g * G + sub;
    const bool valid = idx < cnt && idx < per && pos < n;
    const int j = index(valid ? pos : 0);
    const int key = orderable(score(j));
    bool better = valid && (ZERO || j != 0) && (key > best || (key == best && j < bj));
    if (wave_any(better)) {
      const bool no = refuse(j, better);   // every lane takes part
      better = better && !no;
      const int wmax = wave_reduce_i32(better ? key : INT_MIN, OpMax());
      const int wj = wave_reduce_i32(better && key == wmax ? j : INT_MAX, OpMin());
      if (wj != INT_MAX) {
        best = wmax;
        bj = wj;
      }
    }
    alive &= ~taken;
    if (alive && bj != INT_MAX) alive &= __ballot(!(bound < __int_as_float(best ^ ((best >> 31) & 0x7FFFFFFF))));
  }
  return bj;
}

// A bound on the FP32 sum of n grid values from the sum of their dilated copies
// (whole numbers below 2^24).
__device__ __forceinline__ float upper_bound(const GridDev& G, int n, int sum) {
  return fmaf((float)sum, G.bound_scale, sum_slack(G, n));
}

// Groups that may hold a sample better than s0 (a NaN bound or score keeps them all).
__device__ __forceinline__ uint64_t groups_above(float bound, float s0, int groups) {
  return __ballot(lane_id() < groups && !(bound <= s0));
}

// acc + value(0) + value(1) + ... + value(n - 1), added in that order; U values are
// fetched ahead of the U being added (two register buffers, no copies).
template <int U, class V, class F>
__device__ __forceinline__ V ordered_sum(V acc, int n, F value) {
  V v0[U], v1[U];
  int t = 0;
  const int full = n - n % U;
  if (full > 0) {
#pragma unroll
    for (int u = 0; u < U; ++u) v0[u] = value(u);
    t = U;
    for (; t + U < full; t += 2 * U) {
#pragma unroll
      for (int u = 0; u < U; ++u) v1[u] = value(t + u);
      __builtin_amdgcn_sched_barrier(0);   // keep these fetches ahead of the sums before them
#pragma unroll
      for (int u = 0; u < U; ++u) acc += v0[u];
#pragma unroll
      for (int u = 0; u < U; ++u) v0[u] = value(t + U + u);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < U; ++u) acc += v1[u];
    }
    if (t < full) {
#pragma unroll
      for (int u = 0; u < U; ++u) v1[u] = value(t + u);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < U; ++u) acc += v0[u];
#pragma unroll
      for (int u = 0; u < U; ++u) acc += v1[u];
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u) acc += v0[u];
    }
  }
  for (int k = full; k < n; ++k) acc += value(k);
  return acc;
}

// The sum over n atoms of value(in, t): `in` says whether every node index is
// known to lie inside the padded grid, so that none needs its clamp (two clamps of
// an eighth of a rotation sample's vector cycles each).
template <int U, class V, class F>
__device__ __forceinline__ V scan_sum(bool inside, V acc, int n, F value) {
  if (inside) return ordered_sum<U>(acc, n, [&](int t) { return value(std::true_type{}, t); });
  return ordered_sum<U>(acc, n, [&](int t) { return value(std::false_type{}, t); });
}

template <class In>
__device__ __forceinline__ int node_index(In, float f, float fn) {
  return In::value ? floor_node(f) : clamp_node(f, fn);
}

// ---- rigid rotation scan about lab axis E through the pivot ------------------
// Bound pass: an atom at distance r from the axis stays within chord * r of its
// place at the group's centre, so every node a group's samples read lies in a
// window of w x w nodes of the rotation plane, w - 1 >= 2 chord r / h; the grid
// copies dilated over such windows (GridDev::dil) give the largest value in one
// lookup of 16 bits, in bricks of the rotation plane.  About a third of the groups
// survive (240 k scans of mixed ligands: 0.67, 0.34, 0.23 in sweeps 1, 2, 3),
// 2.6, 1.8 and 1.4 passes of 64 samples instead of 4.
template <int NSLOT, int E, int U>
__device__ __forceinline__ int rot_scan(ArgsPtr S, PoseReg<NSLOT>& p, int N, float4* scr, float4* aux,
                                        const Samples& sm, const int* tab) {
  const GridDev G = grid_of(S);
  constexpr int P = (E + 1) % 3, Q = (E + 2) % 3;
  const int lane = lane_id();
  const float pP = in_vgpr(p.piv[P]), pQ = in_vgpr(p.piv[Q]);
  const float cP = in_vgpr(G.c0[P]), cQ = in_vgpr(G.c0[Q]), ih = in_vgpr(G.inv_h), fnP = G.fn[P], fnQ = G.fn[Q];
  const int* tP = tab + G.tab_base[P] + 1;
  const int* tQ = tab + G.tab_base[Q] + 1;
  const char* gk = G.gk;
  float s0 = 0.f;
  // An atom stays within its distance from the axis, and the node map is
  // monotone: when both ends of every atom's range, widened by four nodes (the
  // windows) and the rounding of positions far from the origin (ferr), map inside
  // [-1, n], no sample and no window needs the clamp of the node index.
  bool inside = true, level = sm.bound_a && G.dil != nullptr;
  const float fp = fmaf(pP, ih, cP), fq = fmaf(pQ, ih, cQ);
  const float ferr = fmaf(1e-6f * ih, fabsf(pP) + fabsf(pQ), 2e-3f);
  const float reach = fminf(fminf(fp + 1.f, fnP - fp), fminf(fq + 1.f, fnQ - fq)) - 4.f - ferr;
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) {
    const int a = s * 64 + lane;
    if (a < N) {
      const float vp = p.x[P][s] - pP, vq = p.x[Q][s] - pQ;
      const int ie = clamp_node(fmaf(p.x[E][s], ih, G.c0[E]), G.fn[E]);
      const int part = boff(tab + G.tab_base[E] + 1, ie);
      scr[a] = make_float4(vp, vq, __int_as_float(part), 0.f);
      s0 += grid_at(gk, part + boff(tP, clamp_node(fmaf(p.x[P][s], ih, cP), fnP)) +
                            boff(tQ, clamp_node(fmaf(p.x[Q][s], ih, cQ), fnQ)));
      const float r = prune_sqrt(fmaf(vp, vp, vq * vq)) * (1.0001f * ih);
      inside = inside && sm.radius * r <= reach;
      const float del = fmaf(sm.chord, r, ferr);
      const int l = del <= 0.5f ? 0 : del <= 1.f ? 1 : del <= 1.5f ? 2 : 3;
      level = level && del <= 2.5f;
      aux[2 * a] = make_float4(vp * ih, vq * ih, fp - del, fq - del);
      reinterpret_cast<uint32_t*>(aux + 2 * a + 1)[0] =
          (uint32_t)__mul24(ie + 1, 128 * G.nb8[P] * G.nb8[Q]) + (uint32_t)(4 * E + l) * G.dil_stride;
    }
  }
  inside = !wave_any(!inside);
  level = !wave_any(!level);
  s0 = wave_sum(s0);
  wave_sync();
  float bound = __builtin_inff();
  if (level) {
    const float c = sm.cc, sn = sm.cs;
    const char* dil = G.dil;
    const int* dP = tab + G.tab_p + 1;
    const int* dQ = tab + G.tab_q[Q] + 1;
    bound = upper_bound(G, N, scan_sum<U>(inside, 0, N, [&](auto in, int t) {
      const float4 k = aux[2 * t];
      const uint32_t part = reinterpret_cast<const uint32_t*>(aux + 2 * t + 1)[0];
      const int ip = node_index(in, fmaf(c, k.x, fmaf(-sn, k.y, k.z)), fnP);
      const int iq = node_index(in, fmaf(sn, k.x, fmaf(c, k.y, k.w)), fnQ);
      return bound_at(dil, part + boff(dP, ip) + boff(dQ, iq));
    }));
  }
  const int j = select_sample<false>(
      groups_above(bound, s0, sm.nga), bound, sm.GA, sm.A, s0, [](int pos) { return pos; },
      [&](int js) {
        const float2 cs = sm.ang[js];
        return scan_sum<U>(inside, 0.f, N, [&](auto in, int t) {
          const float4 d = scr[t];
          const float np = fmaf(cs.x, d.x, -(cs.y * d.y));
          const float nq = fmaf(cs.y, d.x, cs.x * d.y);
          const int ip = node_index(in, fmaf(pP + np, ih, cP), fnP);
          const int iq = node_index(in, fmaf(pQ + nq, ih, cQ), fnQ);
          return grid_at(gk, __float_as_int(d.z) + boff(tP, ip) + boff(tQ, iq));
        });
      },
      [](int, bool) { return false; });
  apply_rot<NSLOT, E>(sm.ang[j], p, j);
  wave_sync();
  return j;
}

// 32-bit LDS address of a shared-memory pointer, and a float load from one.
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)p;
}
__device__ __forceinline__ float lds_load(uint32_t addr) {
  return *(const __attribute__((address_space(3))) float*)(uintptr_t)addr;
}

// Maximum of two floats as one v_max_f32 (fmaxf quiets signalling NaNs first).
__device__ __forceinline__ float larger(float a, float b) {
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// ---- rigid translation scan along lab axis E ---------------------------------
// A translation moves an atom along E only, so its T samples read nodes of one
// grid line: those between the nodes of the smallest and the largest
// displacement (the node index is monotone in the displacement), span nodes at
// most.  The wavefront reads each atom's run of nodes once -- 64 / (span + 1)
// atoms per gather instruction -- into an LDS stage, which holds every run of
// a ligand of average size, and takes all further values from there: the same
// value, node and sum order as a direct gather per sample.
// Bound pass: the samples of a group (in order of displacement) span less than
// one node, so the larger of two neighbouring nodes of the run bounds each.
// 16 groups and four lanes per group, which share the atoms: their partial sums
// are added in another order than the scores', so the bound is widened by what
// rounding can make of that (none on grids whose sums are exact).  About 0.25 of
// the groups survive; 1.6, 1.25, 1.14 passes (sweeps 1, 2, 3) instead of 4.
// Runs longer than a wavefront (very wide translation ranges) fall back to
// direct gathers of every sample, and so does STAGE = false (the plain launch,
// where a lone wavefront per SIMD would wait on every group's nodes) unless the
// bound saves it passes.
template <int NSLOT, int E, bool STAGE, int U>
__device__ __forceinline__ int trans_scan(ArgsPtr S, PoseReg<NSLOT>& p, int N, float4* scr, float* stage,
                                          const Samples& sm, const int* tab) {
  const GridDev G = grid_of(S);
  const DockDev D = dock_of(S);
  constexpr int P = (E + 1) % 3, Q = (E + 2) % 3;
  const int lane = lane_id();
  const float cE = in_vgpr(G.c0[E]), ih = in_vgpr(G.inv_h), fnE = G.fn[E];
  const int* tE = tab + G.tab_base[E] + 1;
  const char* gk = G.gk;
  // displacement delta * m of sample j (m = j, or j - T past T / 2) is monotone in
  // m, so every sample's lies between those of the two extreme m
  const int mlo = D.T >= 2 ? D.T / 2 - D.T : 0, mhi = D.T >= 2 ? D.T / 2 - 1 : 0;
  const float da = D.delta * (float)mlo, db = D.delta * (float)mhi;
  const float dmin = fminf(da, db), dmax = fmaxf(da, db);
  int span = 0;
  bool inside = true;
  float s0 = 0.f;
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) {
    const int a = s * 64 + lane;
    if (a < N) {
      const int ip = clamp_node(fmaf(p.x[P][s], ih, G.c0[P]), G.fn[P]);
      const int iq = clamp_node(fmaf(p.x[Q][s], ih, G.c0[Q]), G.fn[Q]);
      const int part = boff(tab + G.tab_base[P] + 1, ip) + boff(tab + G.tab_base[Q] + 1, iq);
      const int lo = clamp_node(fmaf(p.x[E][s] + dmin, ih, cE), fnE);
      const int hi = clamp_node(fmaf(p.x[E][s] + dmax, ih, cE), fnE);
      span = max(span, hi - lo + 1);
      inside = inside && lo >= 0 && hi < G.n[E];   // every sample's f in [0, n): no clamp needed
      scr[a] = make_float4(p.x[E][s], __int_as_float(part), __int_as_float(lo), 0.f);
      s0 += grid_at(gk, part + boff(tE, clamp_node(fmaf(p.x[E][s], ih, cE), fnE)));
    }
  }
  span = wave_reduce_i32(span, OpMax());
  inside = !wave_any(!inside);
  wave_sync();
  const uint64_t all = sm.ngt < 64 ? (1ull << sm.ngt) - 1u : ~0ull;
  // (one sample: no displacement, whose range `inside` and the runs were taken for)
  auto displacement = [&](int j) { return D.delta * (float)(j < max(D.T / 2, 1) ? j : j - D.T); };
  auto index = [&](int pos) { return pos + mlo < 0 ? pos + mlo + D.T : pos + mlo; };   // position: order of displacement
  auto none = [](int, bool) { return false; };
  int j;
  if ((!STAGE && !(sm.bound_t && D.T > 128)) || span > 63) {
    j = select_sample<true>(
        all, __builtin_inff(), sm.GT, D.T, 0.f, index,
        [&](int js) {
          const float d = displacement(js);
          return scan_sum<U>(inside, 0.f, N, [&](auto in, int t) {
            const float4 k = scr[t];
            return grid_at(gk, __float_as_int(k.y) + boff(tE, node_index(in, fmaf(k.x + d, ih, cE), fnE)));
          });
        },
        none);
  } else {
    const int run = span + 1;                          // nodes staged per atom: its run and one more
    const float rrun = __builtin_amdgcn_rcpf((float)run);
    const int room = __builtin_amdgcn_readfirstlane(small_div(stage_floats(NSLOT), rrun));   // atoms whose runs the stage holds
    const int per = __builtin_amdgcn_readfirstlane(small_div(64, rrun));                     // atoms read by one gather instruction
    const int tt = small_div(lane, rrun), ii = lane - tt * run;
    const int imax = (int)fnE;
    // runs of atoms t0 .. t1 - 1: atom t's node lo + i (clamped into the grid) at
    // stage[(t - t0) * run + i]; scr[t].w becomes the LDS byte address of its node 0
    auto fill = [&](int t0, int t1) {
      wave_sync();
      const int first = tt < per ? t0 + tt : t1;
      for (int t = first; t < t1; t += 4 * per) {
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float4 k = scr[min(t + u * per, t1 - 1)];
          v[u] = grid_at(gk, __float_as_int(k.y) + boff(tE, min(__float_as_int(k.z) + ii, imax)));
          if (ii == 0 && t + u * per < t1)
            reinterpret_cast<uint32_t*>(scr + t + u * per)[3] =
                lds_addr(stage) + 4u * (uint32_t)((t + u * per - t0) * run - __float_as_int(k.z));
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (t + u * per < t1) stage[(t + u * per - t0) * run + ii] = v[u];
      }
      wave_sync();
    };
    const bool once = room >= N;
    if (once) fill(0, N);
    auto place = [&](auto in, const float4& k, float d) {
      return __float_as_uint(k.w) + 4u * (uint32_t)node_index(in, fmaf(k.x + d, ih, cE), fnE);
    };
    float bound = __builtin_inff();
    uint64_t alive = all;
    if (sm.bound_t) {
      const int part = lane >> (6 - sm.tsub), step = 1 << sm.tsub;
      const float d = sm.dlow;
      float acc = 0.f;
      for (int t0 = 0; t0 < N; t0 += room) {
        const int t1 = min(N, t0 + room);
        if (!once) fill(t0, t1);
        auto windows = [&](auto in) {
#pragma unroll 2
          for (int t = t0 + part; t < t1; t += step) {
            const uint32_t at = place(in, scr[t], d);
            acc += larger(lds_load(at), lds_load(at + 4u));
          }
        };
        if (inside)
          windows(std::true_type{});
        else
          windows(std::false_type{});
      }
      if (sm.tsub == 2) acc += __shfl_xor(acc, 16);
      if (sm.tsub >= 1) acc += __shfl_xor(acc, 32);
      bound = acc + sum_slack(G, N);
      // sample 0's group stays: its own score decides between equal samples
      alive = groups_above(bound, wave_sum(s0), sm.ngt) | 1ull << sm.gt0;
    }
    j = select_sample<true>(
        alive, bound, sm.GT, D.T, 0.f, index,
        [&](int js) {
          const float d = displacement(js);
          float acc = 0.f;
          for (int t0 = 0; t0 < N; t0 += room) {
            const int t1 = min(N, t0 + room);
            if (!once) fill(t0, t1);
            acc = scan_sum<U>(inside, acc, t1 - t0, [&](auto in, int t) { return lds_load(place(in, scr[t0 + t], d)); });
          }
          return acc;
        },
        none);
  }
  apply_trans<NSLOT, E>(D, p, j);
  wave_sync();
  return j;
}

// Minimum of two floats as one v_min_f32: fminf's quieting of signalling NaNs
// costs two more instructions per call on a loop-carried value.  A NaN operand
// yields the other one, so a NaN distance never counts as a clash, as with the
// comparison d^2 < clash^2.
__device__ __forceinline__ float vmin(float a, float b) {
  float r;
  asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// ---- greedy torsion scan of bond k with the clash check ----------------------
// A moving atom sweeps a circle about the bond axis; a (moving, static) pair whose
// circle never comes within clash distance + margin of the static atom cannot
// clash at any angle (the margin is far above the FP32 deviation of the computed
// rotation from the exact circle), so only the remaining "risky" pairs are
// tested.  They are listed in LDS grouped by moving atom; a scan with more pairs
// than the list holds takes them in several lists of whole moving atoms.
// Bound pass, at the groups' centres: as in the rotation scan with cubic windows;
// and a group all of whose samples clash is dropped: a pair closer than the clash
// distance less chord * r (r: the moving atom's distance from the axis) at the
// centre clashes at every sample.  Better scores are mostly found where the
// fragment runs into the rest, so that test matters: 0.26, 0.13, 0.10 of the
// groups survive (sweeps 1, 2, 3) against 0.65, 0.46, 0.40 without it; 1.3, 1.1,
// 1.03 passes of 64 samples instead of 4.  The exact pair tests then run only
// for samples that beat the best so far.
template <int NSLOT, int U>
__device__ __forceinline__ int tors_scan(ArgsPtr S, PoseReg<NSLOT>& p, int N, uint32_t ab, float inv_len, int k, const uint32_t* mkl,
                                         float4* scr, float4* pairs, const Samples& sm, const int* tab) {
  const GridDev G = grid_of(S);
  const DockDev D = dock_of(S);
  constexpr int PAIR_CAP = pair_cap(NSLOT);
  float4* aux = pairs + PAIR_CAP;   // per moving atom: axial position, radius, squared distance of the group clash test, level
  const int lane = lane_id();
  uint32_t mk[NSLOT];   // fragment masks of this lane's atoms, kept in LDS between scans
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) mk[s] = mkl[s * 64 + lane];
  const BondAxis A = bond_axis(ab, inv_len, p, k);
  const int a = A.a, b = A.b;
  const float xa = in_vgpr(A.xa), ya = in_vgpr(A.ya), za = in_vgpr(A.za), ux = A.ux, uy = A.uy, uz = A.uz;
  const float ih = in_vgpr(G.inv_h), clash2 = D.clash2;
  const float cx = in_vgpr(G.c0[0]), cy = in_vgpr(G.c0[1]), cz = in_vgpr(G.c0[2]);

  // moving atoms of F_k other than b, compacted into scr and aux; their current score
  bool mv[NSLOT];
  int m = 0;
  float s0 = 0.f;
  // every place of a moving atom lies within |h u| + radius rho of a: when that
  // cube, widened by four nodes and the rounding of positions far from the origin
  // (ferr), is inside the padded grid, no node index needs its clamp
  bool inside = true, level = sm.bound_a && G.dil != nullptr;
  const float ulen = prune_sqrt(fmaf(ux, ux, fmaf(uy, uy, uz * uz))) * 1.0001f;
  const float f0 = fmaf(xa, ih, cx), f1 = fmaf(ya, ih, cy), f2 = fmaf(za, ih, cz);
  const float ferr = 1e-6f * (fabsf(xa) + fabsf(ya) + fabsf(za));
  const float reach = fminf(fminf(fminf(f0 + 1.f, G.fn[0] - f0), fminf(f1 + 1.f, G.fn[1] - f1)),
                            fminf(f2 + 1.f, G.fn[2] - f2)) - 4.f - ferr * ih;
  moving_atoms(mk, N, k, b, mv);
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) {
    const float vx = p.x[0][s] - xa, vy = p.x[1][s] - ya, vz = p.x[2][s] - za;
    const uint64_t bal = __ballot(mv[s]);
    const int at = m + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
    if (mv[s]) {
      s0 += nearest(G, p.x[0][s], p.x[1][s], p.x[2][s]);
      const float h = vx * ux + vy * uy + vz * uz, v2 = vx * vx + vy * vy + vz * vz;
      const float r = prune_sqrt(fmaxf(v2 - h * h, 0.f));
      // M v = c (v - h u) + s (u x v) + h u: the circle's radius is the length of
      // the parts that cos and sin multiply (equal for a unit axis)
      const float ax = vx - ux * h, ay = vy - uy * h, az = vz - uz * h;
      const float bx = uy * vz - uz * vy, by = uz * vx - ux * vz, bz = ux * vy - uy * vx;
      const float rho = prune_sqrt(fmaxf(ax * ax + ay * ay + az * az, bx * bx + by * by + bz * bz)) * 1.0001f;
      inside = inside && fmaf(sm.radius, rho, ulen * fabsf(h)) * ih <= reach;
      const float arc = sm.chord * rho;
      const float del = fmaf(arc + ferr, ih, 4e-3f);
      const int l = del <= 0.5f ? 0 : del <= 1.5f ? 1 : 2;
      level = level && del <= 2.5f;
      const float gap = D.clash - arc - ferr - 2e-3f;
      scr[at] = make_float4(vx, vy, vz, 0.f);
      aux[at] = make_float4(h, r, gap > 0.f ? gap * gap : 0.f, __int_as_float(l << 24));
    }
    m += __popcll(bal);
  }
  if (m == 0) return 0;
  s0 = wave_sum(s0);
  inside = !wave_any(!inside);
  level = !wave_any(!level);
  wave_sync();

  // risky pairs of the moving atoms t0 .. t1 - 1, with the atom's group clash
  // distance; scr[t].w = first pair | count << 16 | level << 24.  Returns t1:
  // whole atoms until the next one's pairs would not fit (one atom's always do).
  auto list_pairs = [&](int t0) {
    float hs[NSLOT], rs[NSLOT];   // of the static atoms
    bool st[NSLOT];
#pragma unroll
    for (int s = 0; s < NSLOT; ++s) {
      const int at = s * 64 + lane;
      st[s] = at < N && !((mkl[at] >> k) & 1u) && at != a;
      const float vx = p.x[0][s] - xa, vy = p.x[1][s] - ya, vz = p.x[2][s] - za;
      hs[s] = vx * ux + vy * uy + vz * uz;
      rs[s] = prune_sqrt(fmaxf(vx * vx + vy * vy + vz * vz - hs[s] * hs[s], 0.f));
    }
    wave_sync();   // reads of an earlier list are done
    int npairs = 0, t = t0;
    for (; t < m; ++t) {
      const float4 x = aux[t];
      uint64_t bal[NSLOT];
      int count = 0;
#pragma unroll
      for (int s = 0; s < NSLOT; ++s) {
        const float dh = x.x - hs[s], dr = x.y - rs[s];
        bal[s] = __ballot(st[s] && fmaf(dr, dr, dh * dh) < D.clash_r2);
        count += __popcll(bal[s]);
      }
      if (npairs + count > PAIR_CAP) break;
      if (lane == 0) reinterpret_cast<int*>(scr + t)[3] = npairs | (count << 16) | __float_as_int(x.w);
#pragma unroll
      for (int s = 0; s < NSLOT; ++s) {
        const int pre =
            __builtin_amdgcn_mbcnt_hi((uint32_t)(bal[s] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal[s], 0u));
        if ((bal[s] >> lane) & 1u) pairs[npairs + pre] = make_float4(p.x[0][s], p.x[1][s], p.x[2][s], x.z);
        npairs += __popcll(bal[s]);
      }
    }
    wave_sync();
    return t;
  };

  const char* gk = G.gk;
  const int* tX = tab + G.tab_base[0] + 1;
  const int* tY = tab + G.tab_base[1] + 1;
  const int* tZ = tab + G.tab_base[2] + 1;
  float bound = __builtin_inff();
  int listed = 0;   // atoms of the list in LDS, when it holds every pair
  uint64_t dead = 0u;
  if (level) {
    float M[9];
    torsion_matrix(ux, uy, uz, sm.cc, sm.cs, M);
    const char* dil = G.dil + 12 * (size_t)G.dil_stride;
    const int* cX = tab + G.tab_c[0] + 1;
    const int* cY = tab + G.tab_c[1] + 1;
    const int* cZ = tab + G.tab_c[2] + 1;
    const float k0 = cx - 0.5f, k1 = cy - 0.5f, k2 = cz - 0.5f;   // windows reach from half a node below
    bool hit = false;
    auto window = [&](auto in, int t) {
      const float4 v = scr[t];
      const float X = fmaf(M[0], v.x, fmaf(M[1], v.y, fmaf(M[2], v.z, xa)));
      const float Y = fmaf(M[3], v.x, fmaf(M[4], v.y, fmaf(M[5], v.z, ya)));
      const float Z = fmaf(M[6], v.x, fmaf(M[7], v.y, fmaf(M[8], v.z, za)));
      const int ix = node_index(in, fmaf(X, ih, k0), G.fn[0]);
      const int iy = node_index(in, fmaf(Y, ih, k1), G.fn[1]);
      const int iz = node_index(in, fmaf(Z, ih, k2), G.fn[2]);
      const int seg = __builtin_amdgcn_readfirstlane(__float_as_int(v.w));
      const int w = bound_at(dil + (uint32_t)(seg >> 24) * G.dil_stride, boff(cX, ix) + boff(cY, iy) + boff(cZ, iz));
      const int p0 = seg & 0xFFFF, p1 = p0 + ((seg >> 16) & 0xFF);
      if (p1 > p0 && !D.lazy_clash) {
        float dmin = __builtin_inff(), gap2 = 0.f;
        for (int pi = p0; pi < p1; ++pi) {
          const float4 c = pairs[pi];
          const float dx = X - c.x, dy = Y - c.y, dz = Z - c.z;
          dmin = vmin(dmin, fmaf(dz, dz, fmaf(dy, dy, dx * dx)));
          gap2 = c.w;
        }
        hit = hit || dmin < gap2;
      }
      return w;
    };
    int sum = 0, late = 0;
    for (int t0 = 0; t0 < m;) {
      const int t1 = list_pairs(t0);
      if (t0 == 0 && t1 == m) listed = m;
      // each value is added an atom later: its fetch runs under the pair tests
      if (inside) {
        for (int t = t0; t < t1; ++t) {
          sum += late;
          late = window(std::true_type{}, t);
        }
      } else {
        for (int t = t0; t < t1; ++t) {
          sum += late;
          late = window(std::false_type{}, t);
        }
      }
      t0 = t1;
    }
    bound = upper_bound(G, m, sum + late);
    dead = __ballot(hit);
  }
  float Mj[9];
  const int j = select_sample<false>(
      groups_above(bound, s0, sm.nga) & ~dead, bound, sm.GA, sm.A, s0, [](int pos) { return pos; },
      [&](int js) {
        const float2 cs = sm.ang[js];
        float M[9];
        torsion_matrix(ux, uy, uz, cs.x, cs.y, M);
        return scan_sum<U>(inside, 0.f, m, [&](auto in, int t) {
          const float4 v = scr[t];
          float y0, y1, y2;
          mat_apply(M, v.x, v.y, v.z, y0, y1, y2);
          const int ix = node_index(in, fmaf(xa + y0, ih, cx), G.fn[0]);
          const int iy = node_index(in, fmaf(ya + y1, ih, cy), G.fn[1]);
          const int iz = node_index(in, fmaf(za + y2, ih, cz), G.fn[2]);
          return grid_at(gk, boff(tX, ix) + boff(tY, iy) + boff(tZ, iz));
        });
      },
      [&](int js, bool better) {
        const float2 cs = sm.ang[js];
        float M[9];
        torsion_matrix(ux, uy, uz, cs.x, cs.y, M);
        bool hit = false;
        for (int t0 = 0; t0 < m;) {
          const int t1 = listed ? m : list_pairs(t0);
          if (t0 == 0 && t1 == m) listed = m;
          for (int t = t0; t < t1; ++t) {
            const float4 v = scr[t];
            // the segment is the same on every lane: a scalar loop; the least d^2
            // over the atom's pairs decides (min is exact)
            const int seg = __builtin_amdgcn_readfirstlane(__float_as_int(v.w));
            const int p0 = seg & 0xFFFF, p1 = p0 + ((seg >> 16) & 0xFF);
            if (p1 == p0) continue;
            float y0, y1, y2;
            mat_apply(M, v.x, v.y, v.z, y0, y1, y2);
            const float X = xa + y0, Y = ya + y1, Z = za + y2;
            float dmin = __builtin_inff();
            for (int pi = p0; pi < p1; ++pi) {
              const float4 c = pairs[pi];
              const float dx = X - c.x, dy = Y - c.y, dz = Z - c.z;
              dmin = vmin(dmin, fmaf(dz, dz, fmaf(dy, dy, dx * dx)));
            }
            hit = hit || dmin < clash2;
            if (!wave_any(better && !hit)) return hit;
          }
          t0 = t1;
        }
        return hit;
      });
  if (j != 0) {
    torsion_matrix(ux, uy, uz, sm.ang[j].x, sm.ang[j].y, Mj);
    apply_tors(p, A, Mj, mv);
  }
  wave_sync();
  return j;
}

// ---- scans of every sample ------------------------------------------------------
// Where no bound pass pays or is possible a scan scores every sample, SPL per lane
// (lane + 64 q) in one pass over the atoms: the atom's data is read and its fixed part
// done once for all of them, and the pass ends in one reduction.  Bounded scans without
// their bound pass score one sample per lane and pass: 4 000 mixed ligands of 128
// samples took 49.6 ms that way, 10 000 fragments of up to 20 atoms 37.5 ms, 2 000
// ligands in a grid of 0.1 A nodes and 256 samples 191 ms; these take 41.5, 24.3 and 144.
// What a launch's scans need to know of them, uniform but for `valid`; the (cos, sin)
// of the lane's samples are read from LDS in each scan.
template <int SPL>
struct SampleReg {
  uint32_t valid;      // bit q: sample lane + 64 q exists
  bool half_turn;      // A = 64 SPL and sample j + A/2 is sample j turned by pi:
                       // (cos, sin) of the two are exact negatives
  bool quarter_turn;   // A = 64 SPL and samples j + A/4, j + A/2, j + 3A/4 are j turned
                       // by pi/2, pi, 3pi/2: (-s, c), (-c, -s), (s, -c) exactly
  bool unit;           // every sample has |cos| <= 1 and |sin| <= 1
};

// (cos, sin) of sample lane + 64 q, the last one past the end.
__device__ __forceinline__ float2 lane_sample(const float2* ang, int A, int q) {
  return ang[min(lane_id() + 64 * q, A - 1)];
}

template <int SPL>
__device__ __forceinline__ void load_every_sample(const DockDev& D, const float2* ang, SampleReg<SPL>& sm) {
  const int lane = lane_id();
  sm.valid = 0u;
  bool unit = true;
  float c[SPL], s[SPL];
#pragma unroll
  for (int q = 0; q < SPL; ++q) {
    const int j = lane + 64 * q;
    const float2 cs = lane_sample(ang, D.A, q);
    c[q] = cs.x;
    s[q] = cs.y;
    if (j < D.A) sm.valid |= 1u << q;
    unit = unit && fabsf(cs.x) <= 1.f && fabsf(cs.y) <= 1.f;
  }
  sm.unit = !wave_any(!unit);
  sm.half_turn = sm.quarter_turn = false;
  if (SPL % 2 == 0 && D.A == 64 * SPL) {
    bool pair = true;
#pragma unroll
    for (int q = 0; q < SPL / 2; ++q) pair = pair && c[q + SPL / 2] == -c[q] && s[q + SPL / 2] == -s[q];
    sm.half_turn = !wave_any(!pair);
  }
  if (SPL % 4 == 0 && D.A == 64 * SPL) {
    constexpr int Q4 = SPL / 4;
    bool quad = sm.half_turn;
#pragma unroll
    for (int q = 0; q < Q4; ++q) quad = quad && c[q + Q4] == -s[q] && s[q + Q4] == c[q];
    sm.quarter_turn = !wave_any(!quad);
  }
}

// The sample of the largest score, the lowest index among equal ones.
template <int SPL>
__device__ __forceinline__ int wave_argmax(const float (&acc)[SPL], uint32_t alive) {
  const int lane = lane_id();
  int best = INT_MIN, bj = INT_MAX;
#pragma unroll
  for (int q = 0; q < SPL; ++q) {
    const int k = orderable(acc[q]);
    if (((alive >> q) & 1u) && k > best) {
      best = k;
      bj = lane + 64 * q;
    }
  }
  const int wmax = wave_reduce_i32(best, OpMax());
  return wave_reduce_i32(best == wmax ? bj : INT_MAX, OpMin());
}

// acc[q] += gather(t)[q] over t < n, with the gathers of atom t + 1 issued before the
// values of atom t are added (two register buffers, no copies).
template <int Q, int NA, class F>
__device__ __forceinline__ void pipelined_sum(int n, F gather, float (&acc)[NA], int qoff = 0) {
  float v0[Q], v1[Q];
  auto add = [&](const float (&v)[Q]) {
#pragma unroll
    for (int q = 0; q < Q; ++q) acc[q + qoff] += v[q];
  };
  gather(0, v0);
  int t = 1;
  for (; t + 1 < n; t += 2) {
    gather(t, v1);
    __builtin_amdgcn_sched_barrier(0);   // keep the loads of atom t ahead of the sums of atom t - 1
    add(v0);
    gather(t + 1, v0);
    __builtin_amdgcn_sched_barrier(0);
    add(v1);
  }
  if (t < n) {
    gather(t, v1);
    add(v0);
    add(v1);
  } else {
    add(v0);
  }
}

// The rotation scan over every sample.  A 2-D rotation serves the two or four samples
// of a lane that are turned by pi or pi/2: the rotated offsets are exact negatives or
// exchanged (fma and products are sign-symmetric), and a zero's sign cannot change the
// node.  With |cos|, |sin| <= 1 a rotated offset is at most |vp| + |vq| per axis (B
// covers the rounding), and the node map is monotone: when both ends of every atom's
// range map inside [-1, n], no sample needs the clamp of the node index.
template <int NSLOT, int E, int SPL>
__device__ __forceinline__ int rot_scan_all(ArgsPtr S, PoseReg<NSLOT>& p, int N, float4* scr,
                                            const SampleReg<SPL>& sm, const float2* ang, const int* tab) {
  const GridDev G = grid_of(S);
  const int A = S->D.A;
  constexpr int P = (E + 1) % 3, Q = (E + 2) % 3;
  const int lane = lane_id();
  const float pP = p.piv[P], pQ = p.piv[Q];
  const float cP = G.c0[P], cQ = G.c0[Q], ih = G.inv_h, fnP = G.fn[P], fnQ = G.fn[Q];
  const int* tP = tab + G.tab_base[P] + 1;
  const int* tQ = tab + G.tab_base[Q] + 1;
  const char* gk = G.gk;
  float s0 = 0.f;
  bool inside = sm.unit;
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) {
    const int a = s * 64 + lane;
    if (a < N) {
      const float vp = p.x[P][s] - pP, vq = p.x[Q][s] - pQ;
      const int part = boff(tab + G.tab_base[E] + 1, clamp_node(fmaf(p.x[E][s], ih, G.c0[E]), G.fn[E]));
      scr[a] = make_float4(vp, vq, __int_as_float(part), 0.f);
      s0 += grid_at(gk, part + boff(tP, clamp_node(fmaf(p.x[P][s], ih, cP), fnP)) +
                            boff(tQ, clamp_node(fmaf(p.x[Q][s], ih, cQ), fnQ)));
      const float B = (fabsf(vp) + fabsf(vq)) * (1.f + 0x1p-20f);
      inside = inside && fmaf(pP - B, ih, cP) >= -1.f && fmaf(pP + B, ih, cP) <= fnP &&
               fmaf(pQ - B, ih, cQ) >= -1.f && fmaf(pQ + B, ih, cQ) <= fnQ;
    }
  }
  inside = !wave_any(!inside);
  s0 = wave_sum(s0);
  wave_sync();
  float acc[SPL];
#pragma unroll
  for (int q = 0; q < SPL; ++q) acc[q] = 0.f;
  // TURNS samples of a lane from one rotation, sample q + SPL / TURNS a turn of 1 / TURNS on
  auto sums = [&](auto turns, auto in) {
    constexpr int TURNS = decltype(turns)::value, STEP = SPL / TURNS;
    float2 cs[STEP];
#pragma unroll
    for (int q = 0; q < STEP; ++q) cs[q] = lane_sample(ang, A, q);
    pipelined_sum<SPL>(N, [&](int t, float (&out)[SPL]) {
      const float4 d = scr[t];
      const int part = __float_as_int(d.z);
#pragma unroll
      for (int q = 0; q < STEP; ++q) {
        const float np = fmaf(cs[q].x, d.x, -(cs[q].y * d.y));
        const float nq = fmaf(cs[q].y, d.x, cs[q].x * d.y);
        auto at = [&](float xp, float xq) {
          return grid_at(gk, part + boff(tP, node_index(in, fmaf(xp, ih, cP), fnP)) +
                                 boff(tQ, node_index(in, fmaf(xq, ih, cQ), fnQ)));
        };
        out[q] = at(pP + np, pQ + nq);
        if (TURNS == 4) out[q + STEP] = at(pP - nq, pQ + np);
        if (TURNS >= 2) out[q + SPL / 2] = at(pP - np, pQ - nq);
        if (TURNS == 4) out[q + 3 * STEP] = at(pP + nq, pQ - np);
      }
    }, acc);
  };
  constexpr std::integral_constant<int, 1> one{};
  constexpr std::integral_constant<int, SPL % 2 == 0 ? 2 : 1> two{};
  constexpr std::integral_constant<int, SPL % 4 == 0 ? 4 : 1> four{};
  auto by_turns = [&](auto in) {
    if (SPL % 4 == 0 && sm.quarter_turn)
      sums(four, in);
    else if (SPL % 2 == 0 && sm.half_turn)
      sums(two, in);
    else
      sums(one, in);
  };
  if (inside)
    by_turns(std::true_type{});
  else
    by_turns(std::false_type{});
  if (lane == 0) acc[0] = s0;   // sample 0 is the current pose
  const int j = wave_argmax(acc, sm.valid);
  apply_rot<NSLOT, E>(ang[j], p, j);
  wave_sync();
  return j;
}

// The torsion scan over every sample.  The clash tests run in the scoring pass, on the
// list of risky pairs; a scan with more pairs than the list holds takes them in
// several lists of whole moving atoms, as the bounded scan does.
template <int NSLOT, int SPL>
__device__ __forceinline__ int tors_scan_all(ArgsPtr S, PoseReg<NSLOT>& p, int N, uint32_t ab, float inv_len, int k,
                                             const uint32_t* mkl, float4* scr, float4* pairs, const SampleReg<SPL>& sm,
                                             const float2* ang, const int* tab) {
  const GridDev G = grid_of(S);
  const DockDev D = dock_of(S);
  constexpr int PAIR_CAP = pair_cap(NSLOT) + 64 * NSLOT;
  const int lane = lane_id();
  uint32_t mk[NSLOT];
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) mk[s] = mkl[s * 64 + lane];
  const BondAxis A = bond_axis(ab, inv_len, p, k);
  const int a = A.a, b = A.b;
  const float xa = A.xa, ya = A.ya, za = A.za, ux = A.ux, uy = A.uy, uz = A.uz;

  // moving atoms of F_k other than b, compacted into scr; their current score; axial
  // position and radius of every static atom about the bond axis
  bool mv[NSLOT], st[NSLOT];
  float hs[NSLOT], rs[NSLOT];
  int m = 0;
  float s0 = 0.f;
  moving_atoms(mk, N, k, b, mv);
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) {
    const int at = s * 64 + lane;
    st[s] = at < N && !((mk[s] >> k) & 1u) && at != a;
    const float vx = p.x[0][s] - xa, vy = p.x[1][s] - ya, vz = p.x[2][s] - za;
    hs[s] = vx * ux + vy * uy + vz * uz;
    rs[s] = prune_sqrt(fmaxf(vx * vx + vy * vy + vz * vz - hs[s] * hs[s], 0.f));
    const uint64_t bal = __ballot(mv[s]);
    const int pre = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
    if (mv[s]) {
      scr[m + pre] = make_float4(vx, vy, vz, 0.f);
      s0 += nearest(G, p.x[0][s], p.x[1][s], p.x[2][s]);
    }
    m += __popcll(bal);
  }
  if (m == 0) return 0;
  s0 = wave_sum(s0);
  wave_sync();

  // risky pairs of the moving atoms t0 .. t1 - 1; scr[t].w = first pair | count << 16.
  // Returns t1: whole atoms until the next one's pairs would not fit (one atom's do).
  auto list_pairs = [&](int t0) {
    wave_sync();   // reads of an earlier list are done
    int npairs = 0, t = t0;
    for (; t < m; ++t) {
      const float4 v = scr[t];
      const float ht = v.x * ux + v.y * uy + v.z * uz;
      const float rt = prune_sqrt(fmaxf(v.x * v.x + v.y * v.y + v.z * v.z - ht * ht, 0.f));
      uint64_t bal[NSLOT];
      int count = 0;
#pragma unroll
      for (int s = 0; s < NSLOT; ++s) {
        const float dh = ht - hs[s], dr = rt - rs[s];
        bal[s] = __ballot(st[s] && fmaf(dr, dr, dh * dh) < D.clash_r2);
        count += __popcll(bal[s]);
      }
      if (npairs + count > PAIR_CAP) break;
      if (lane == 0) reinterpret_cast<int*>(scr + t)[3] = npairs | (count << 16);
#pragma unroll
      for (int s = 0; s < NSLOT; ++s) {
        const int pre =
            __builtin_amdgcn_mbcnt_hi((uint32_t)(bal[s] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal[s], 0u));
        if ((bal[s] >> lane) & 1u) pairs[npairs + pre] = make_float4(p.x[0][s], p.x[1][s], p.x[2][s], 0.f);
        npairs += __popcll(bal[s]);
      }
    }
    wave_sync();
    return t;
  };

  float acc[SPL];
#pragma unroll
  for (int q = 0; q < SPL; ++q) acc[q] = 0.f;
  uint32_t clash = 0u;   // bit q: sample lane + 64 q clashes
  constexpr int QG = SPL < 2 ? SPL : 2;   // samples whose matrices are held at once
  const float ih = G.inv_h, clash2 = D.clash2;
  const char* gk = G.gk;
  const int* tX = tab + G.tab_base[0] + 1;
  const int* tY = tab + G.tab_base[1] + 1;
  const int* tZ = tab + G.tab_base[2] + 1;
  for (int t0 = 0; t0 < m;) {
    const int t1 = list_pairs(t0);
#pragma unroll
    for (int g = 0; g < SPL; g += QG) {
      float M[QG][9];
#pragma unroll
      for (int q = 0; q < QG; ++q) {
        const float2 cs = lane_sample(ang, D.A, g + q);
        torsion_matrix(ux, uy, uz, cs.x, cs.y, M[q]);
      }
      pipelined_sum<QG>(t1 - t0, [&](int t, float (&out)[QG]) {
        const float4 v = scr[t0 + t];
        float X[QG], Y[QG], Z[QG];
#pragma unroll
        for (int q = 0; q < QG; ++q) {
          float y0, y1, y2;
          mat_apply(M[q], v.x, v.y, v.z, y0, y1, y2);
          X[q] = xa + y0;
          Y[q] = ya + y1;
          Z[q] = za + y2;
          const int ix = clamp_node(fmaf(X[q], ih, G.c0[0]), G.fn[0]);
          const int iy = clamp_node(fmaf(Y[q], ih, G.c0[1]), G.fn[1]);
          const int iz = clamp_node(fmaf(Z[q], ih, G.c0[2]), G.fn[2]);
          out[q] = grid_at(gk, boff(tX, ix) + boff(tY, iy) + boff(tZ, iz));
        }
        // the segment is the same on every lane: a scalar loop; the least d^2 over the
        // atom's pairs decides its clash bits (min is exact)
        const int seg = __builtin_amdgcn_readfirstlane(__float_as_int(v.w));
        const int p0 = seg & 0xFFFF, p1 = p0 + (seg >> 16);
        if (p1 == p0) return;
        float dmin[QG];
#pragma unroll
        for (int q = 0; q < QG; ++q) dmin[q] = __builtin_inff();
        for (int pi = p0; pi < p1; ++pi) {
          const float4 c = pairs[pi];
#pragma unroll
          for (int q = 0; q < QG; ++q) {
            const float dx = X[q] - c.x, dy = Y[q] - c.y, dz = Z[q] - c.z;
            dmin[q] = vmin(dmin[q], fmaf(dz, dz, fmaf(dy, dy, dx * dx)));
          }
        }
#pragma unroll
        for (int q = 0; q < QG; ++q)
          if (dmin[q] < clash2) clash |= 1u << (g + q);
      }, acc, g);
    }
    t0 = t1;
  }
  if (lane == 0) {
    acc[0] = s0;        // sample 0 is the current pose,
    clash &= ~1u;       // always admissible
  }
  const int j = wave_argmax(acc, sm.valid & ~clash);
  if (j != 0) {
    float Mj[9];
    torsion_matrix(ux, uy, uz, ang[j].x, ang[j].y, Mj);
    apply_tors(p, A, Mj, mv);
  }
  wave_sync();
  return j;
}

// The translation scan over every sample: as in the bounded scan the wavefront reads
// each atom's run of nodes once, here 64 / span atoms at a time into one of two
// buffers (a group's stage is written while the previous one's reads are retired), and
// every sample then takes its value from there.  At most 64 SPL samples.
template <int NSLOT, int E, int SPL>
__device__ __forceinline__ int trans_scan_all(ArgsPtr S, PoseReg<NSLOT>& p, int N, float4* scr, float* stage,
                                              const int* tab) {
  const GridDev G = grid_of(S);
  const DockDev D = dock_of(S);
  constexpr int P = (E + 1) % 3, Q = (E + 2) % 3;
  const int lane = lane_id();
  const float cE = G.c0[E], ih = G.inv_h, fnE = G.fn[E];
  float shift[SPL];
  uint32_t valid = 0u;
#pragma unroll
  for (int q = 0; q < SPL; ++q) {
    const int j = lane + 64 * q;
    shift[q] = j < D.T ? D.delta * (float)(j < max(D.T / 2, 1) ? j : j - D.T) : 0.f;
    if (j < D.T) valid |= 1u << q;
  }
  const int mlo = D.T >= 2 ? D.T / 2 - D.T : 0, mhi = D.T >= 2 ? D.T / 2 - 1 : 0;
  const float da = D.delta * (float)mlo, db = D.delta * (float)mhi;
  const float dmin = fminf(da, db), dmax = fmaxf(da, db);
  int span = 0;
  bool inside = true;
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) {
    const int a = s * 64 + lane;
    if (a < N) {
      const int ip = clamp_node(fmaf(p.x[P][s], ih, G.c0[P]), G.fn[P]);
      const int iq = clamp_node(fmaf(p.x[Q][s], ih, G.c0[Q]), G.fn[Q]);
      const int part = boff(tab + G.tab_base[P] + 1, ip) + boff(tab + G.tab_base[Q] + 1, iq);
      const int lo = clamp_node(fmaf(p.x[E][s] + dmin, ih, cE), fnE);
      const int hi = clamp_node(fmaf(p.x[E][s] + dmax, ih, cE), fnE);
      span = max(span, hi - lo + 1);
      inside = inside && lo >= 0 && hi < G.n[E];   // every sample's f in [0, n): no clamp needed
      scr[a] = make_float4(p.x[E][s], __int_as_float(part), __int_as_float(lo), 0.f);
    }
  }
  span = wave_reduce_i32(span, OpMax());
  inside = !wave_any(!inside);
  wave_sync();
  float acc[SPL];
#pragma unroll
  for (int q = 0; q < SPL; ++q) acc[q] = 0.f;
  const int* tE = tab + G.tab_base[E] + 1;
  const char* gk = G.gk;
  if (span > 64) {   // runs longer than a wavefront: direct gathers
    pipelined_sum<SPL>(N, [&](int t, float (&out)[SPL]) {
      const float4 d = scr[t];
#pragma unroll
      for (int q = 0; q < SPL; ++q)
        out[q] = grid_at(gk, __float_as_int(d.y) + boff(tE, clamp_node(fmaf(d.x + shift[q], ih, cE), fnE)));
    }, acc);
  } else {
    const float rspan = __builtin_amdgcn_rcpf((float)span);
    const int per = __builtin_amdgcn_readfirstlane(small_div(64, rspan));   // atoms whose runs one gather reads
    const int tt = small_div(lane, rspan), ii = lane - tt * span;
    const int imax = (int)fnE;
    // lane (tt, ii): node lo + ii of atom t0 + tt (clamped into the grid; positions past
    // an atom's own run are never read)
    auto stage_load = [&](int t0) {
      const int t = t0 + tt;
      if (tt >= per || t >= N) return 0.f;
      const float4 d = scr[t];
      return grid_at(gk, __float_as_int(d.y) + boff(tE, min(__float_as_int(d.z) + ii, imax)));
    };
    auto staged = [&](auto in) {
      float next = stage_load(0);
      int b = 0;
      for (int t0 = 0; t0 < N; t0 += per, b ^= 1) {
        float* buf = stage + b * 64;
        buf[lane] = next;
        wave_sync();
        const int t1 = min(N, t0 + per);
        if (t1 < N) next = stage_load(t1);
        for (int t = t0; t < t1; ++t) {
          const float4 d = scr[t];
          // LDS byte address of the atom's run, shifted so that node ie (in [lo, lo +
          // span)) is at run + 4 ie: one base per atom, one shift-add per sample
          uint32_t run = lds_addr(buf) + 4u * (uint32_t)((t - t0) * span - __float_as_int(d.z));
          asm volatile("" : "+v"(run));
          int ie[SPL];
          float v[SPL];
#pragma unroll
          for (int q = 0; q < SPL; ++q) ie[q] = node_index(in, fmaf(d.x + shift[q], ih, cE), fnE);
#pragma unroll
          for (int q = 0; q < SPL; ++q) v[q] = lds_load(run + 4u * (uint32_t)ie[q]);
#pragma unroll
          for (int q = 0; q < SPL; ++q) acc[q] += v[q];
        }
      }
    };
    if (inside)
      staged(std::true_type{});
    else
      staged(std::false_type{});
  }
  const int j = wave_argmax(acc, valid);
  apply_trans<NSLOT, E>(D, p, j);
  wave_sync();
  return j;
}

template <int NSLOT>
struct LigReg {
  int N, K, abase, toff;
  uint32_t mk[NSLOT];
  float P0[3];
  uint32_t ab;   // lane k: bond k's atoms, a | b << 16, and its inverse length (read
  float il;      // back with readlane: a load per torsion scan would wait on the L2)
};

template <int NSLOT>
__device__ void load_ligand(const LigDev& Lg, int lig, LigReg<NSLOT>& L) {
  const int lane = lane_id();
  L.abase = __builtin_amdgcn_readfirstlane(Lg.atom_offset[lig]);
  L.N = __builtin_amdgcn_readfirstlane(Lg.atom_offset[lig + 1]) - L.abase;
  L.toff = __builtin_amdgcn_readfirstlane(Lg.tors_offset[lig]);
  L.K = __builtin_amdgcn_readfirstlane(Lg.tors_offset[lig + 1]) - L.toff;
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) {
    const int a = s * 64 + lane;
    const bool in = a < L.N;
    L.mk[s] = in ? Lg.mask[L.abase + a] : 0u;
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) L.P0[c] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(Lg.ref[3 * lig + c])));
  L.ab = lane < L.K ? (uint32_t)Lg.tors_atoms[2 * (L.toff + lane)] | (uint32_t)Lg.tors_atoms[2 * (L.toff + lane) + 1] << 16 : 0u;
  L.il = lane < L.K ? Lg.inv_len[L.toff + lane] : 0.f;
}

// The fragment masks of the ligand's atoms into the wavefront's LDS: read by
// every torsion scan, they would otherwise be held in registers through the
// restart loop (and spilled to scratch at the register budget of the persistent
// instances, a store per work item).  Each lane reads back only its own words.
template <int NSLOT>
__device__ __forceinline__ void store_masks(const LigReg<NSLOT>& L, uint32_t* mkl) {
  const int lane = lane_id();
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) mkl[s * 64 + lane] = L.mk[s];
}

// Restart placement: x = M_r (x0 - P0) + (c + t_r), pivot c + t_r.
template <int NSLOT>
__device__ __forceinline__ void place_pose(const LigDev& Lg, const DockDev& D, const LigReg<NSLOT>& L, int r,
                                           PoseReg<NSLOT>& p) {
  const int lane = lane_id();
  const float* row = D.restarts + 12 * r;
  float m[12];
#pragma unroll
  for (int i = 0; i < 12; ++i) m[i] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(row[i])));
  float q[3] = {D.c[0] + m[9], D.c[1] + m[10], D.c[2] + m[11]};
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) {
    // the input coordinates are re-read (L2-resident) rather than held in
    // registers, through one 32-bit byte offset on the scalar bases: 64-bit
    // per-lane addresses would be hoisted out of the restart loop and spilled
    const int a = s * 64 + lane;
    const bool in = a < L.N;
    uint32_t off = (uint32_t)(L.abase + a) * 4u;
    asm volatile("" : "+v"(off));   // computed here, per restart
    const float x0 = in ? *reinterpret_cast<const float*>(reinterpret_cast<const char*>(Lg.x) + off) : 0.f;
    const float y0 = in ? *reinterpret_cast<const float*>(reinterpret_cast<const char*>(Lg.y) + off) : 0.f;
    const float z0 = in ? *reinterpret_cast<const float*>(reinterpret_cast<const char*>(Lg.z) + off) : 0.f;
    float vx = x0 - L.P0[0], vy = y0 - L.P0[1], vz = z0 - L.P0[2];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      float y = fmaf(m[3 * c + 2], vz, fmaf(m[3 * c + 1], vy, m[3 * c] * vx));
      p.x[c][s] = y + q[c];
    }
  }
  p.piv[0] = q[0]; p.piv[1] = q[1]; p.piv[2] = q[2];
}

// Selected samples of restart r of a ligand: S rows of 6 + K entries.
__device__ __forceinline__ uint16_t* move_record(const DockDev& D, int lig, int toff, int K, int r) {
  return D.moves + (size_t)D.R * D.S * (6 * (size_t)lig + toff) + (size_t)r * D.S * (6 + K);
}

// LDS of a block: the brick offset tables, the samples' (cos, sin), then per
// wavefront the scan data of 64*NSLOT atoms, the regions of the scans (risky
// torsion pairs and moving atoms, staged grid values, bound-pass data) and the
// fragment masks.
struct BlockLds {
  int* tab;
  float2* ang;
  float4* scr;
  float4* cand;
  uint32_t* mkl;
};

// One restart: placement, S sweeps, final trilinear score, outputs.
// U: values in flight per buffer of the scans' sums (and half of it in the torsion
// scans, whose fragments are small).
// SPL: 0, scans that bound groups of samples; else scans of every sample, SPL per lane.
template <int NSLOT, bool STAGE, int U, int SPL>
__device__ __forceinline__ void dock_restart(ArgsPtr S, const Samples& sm, const SampleReg<SPL ? SPL : 1>& every,
                                             const LigReg<NSLOT>& L, int lig, int r, const BlockLds& B) {
  const int lane = lane_id();
  const int N = L.N;
  PoseReg<NSLOT> p;
  place_pose(ligands_of(S), dock_of(S), L, r, p);
  const int sweeps = S->D.S;
  float* stage = reinterpret_cast<float*>(B.cand);
  for (int sw = 0; sw < sweeps; ++sw) {
    int j[6];
    if constexpr (SPL > 0) {
      j[0] = rot_scan_all<NSLOT, 0, SPL>(S, p, N, B.scr, every, B.ang, B.tab);
      j[1] = rot_scan_all<NSLOT, 1, SPL>(S, p, N, B.scr, every, B.ang, B.tab);
      j[2] = rot_scan_all<NSLOT, 2, SPL>(S, p, N, B.scr, every, B.ang, B.tab);
      j[3] = trans_scan_all<NSLOT, 0, SPL>(S, p, N, B.scr, stage, B.tab);
      j[4] = trans_scan_all<NSLOT, 1, SPL>(S, p, N, B.scr, stage, B.tab);
      j[5] = trans_scan_all<NSLOT, 2, SPL>(S, p, N, B.scr, stage, B.tab);
    } else {
      j[0] = rot_scan<NSLOT, 0, U>(S, p, N, B.scr, B.cand, sm, B.tab);
      j[1] = rot_scan<NSLOT, 1, U>(S, p, N, B.scr, B.cand, sm, B.tab);
      j[2] = rot_scan<NSLOT, 2, U>(S, p, N, B.scr, B.cand, sm, B.tab);
      j[3] = trans_scan<NSLOT, 0, STAGE, U>(S, p, N, B.scr, stage, sm, B.tab);
      j[4] = trans_scan<NSLOT, 1, STAGE, U>(S, p, N, B.scr, stage, sm, B.tab);
      j[5] = trans_scan<NSLOT, 2, STAGE, U>(S, p, N, B.scr, stage, sm, B.tab);
    }
    const DockDev D = dock_of(S);
    uint16_t* mrow = move_record(D, lig, L.toff, L.K, r) + (size_t)sw * (6 + L.K);
    int16_t* trow = D.trace ? D.trace + (((size_t)lig * D.R + r) * (size_t)sweeps + sw) * D.trace_w : nullptr;
    if (lane == 0) {
#pragma unroll
      for (int q = 0; q < 6; ++q) mrow[q] = (uint16_t)j[q];
      if (trow) {
#pragma unroll
        for (int q = 0; q < 6; ++q) trow[q] = (int16_t)j[q];
      }
    }
    for (int k = 0; k < L.K; ++k) {
      int jk;
      if constexpr (SPL > 0)
        jk = tors_scan_all<NSLOT, SPL>(S, p, N, L.ab, L.il, k, B.mkl, B.scr, B.cand, every, B.ang, B.tab);
      else
        jk = tors_scan<NSLOT, U / 2>(S, p, N, L.ab, L.il, k, B.mkl, B.scr, B.cand, sm, B.tab);
      if (lane == 0) {
        mrow[6 + k] = (uint16_t)jk;
        if (trow) trow[6 + k] = (int16_t)jk;
      }
    }
  }
  const GridDev G = grid_of(S);
  const DockDev D = dock_of(S);

  // final trilinear score, summed in atom order
  float v[NSLOT];
#pragma unroll
  for (int s = 0; s < NSLOT; ++s)
    v[s] = (s * 64 + lane < N) ? trilinear(G, p.x[0][s], p.x[1][s], p.x[2][s], nullptr) : 0.f;
  float total = 0.f;
#pragma unroll
  for (int s = 0; s < NSLOT; ++s) {
    const int cnt = min(64, N - s * 64);
    for (int l = 0; l < cnt; ++l) total = total + __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v[s]), l));
  }
  if (lane == 0) D.final_scores[(size_t)lig * D.R + r] = total;
}

// The pose of restart r after its recorded moves: placement, then every
// sweep's rotations, translations and torsions with the selected samples.  A
// sweep's record is one load (lane q: entry q) and one more for the (cos, sin)
// of its samples; the moves themselves touch no memory.
template <int NSLOT>
__device__ void replay_restart(const LigDev& Lg, const DockDev& D, const LigReg<NSLOT>& L, int lig, int r,
                               PoseReg<NSLOT>& p) {
  place_pose(Lg, D, L, r, p);
  const int lane = lane_id();
  const uint16_t* mrec = move_record(D, lig, L.toff, L.K, r);
  for (int sw = 0; sw < D.S; ++sw) {
    const uint16_t* mrow = mrec + (size_t)sw * (6 + L.K);
    // recorded indices are below A (rotations, torsions) and T (translations); the
    // clamps only keep table reads in range
    const bool shift = lane >= 3 && lane < 6;
    const int mine = lane < 6 + L.K ? min((int)mrow[lane], (shift ? D.T : D.A) - 1) : 0;
    const int jt = shift ? 0 : mine;
    const float c = D.angles[2 * jt], sn = D.angles[2 * jt + 1];
    auto entry = [&](int q) { return __builtin_amdgcn_readlane(mine, q); };
    auto turn = [&](int q) {
      return make_float2(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(c), q)),
                         __int_as_float(__builtin_amdgcn_readlane(__float_as_int(sn), q)));
    };
    apply_rot<NSLOT, 0>(turn(0), p, entry(0));
    apply_rot<NSLOT, 1>(turn(1), p, entry(1));
    apply_rot<NSLOT, 2>(turn(2), p, entry(2));
    apply_trans<NSLOT, 0>(D, p, entry(3));
    apply_trans<NSLOT, 1>(D, p, entry(4));
    apply_trans<NSLOT, 2>(D, p, entry(5));
    for (int k = 0; k < L.K; ++k) {
      if (entry(6 + k) == 0) continue;
      const BondAxis A = bond_axis(L.ab, L.il, p, k);
      const float2 cs = turn(6 + k);
      float Mj[9];
      torsion_matrix(A.ux, A.uy, A.uz, cs.x, cs.y, Mj);
      bool mv[NSLOT];
      moving_atoms(L.mk, L.N, k, A.b, mv);
      apply_tors(p, A, Mj, mv);
    }
  }
}

// The running kernel's first argument.
__device__ __forceinline__ ArgsPtr kernel_args() { return (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr(); }

// Plain method: one launch per ligand; wavefront w of the grid docks restart w.
template <int NSLOT, bool BOUNDS>
__device__ __forceinline__ BlockLds block_lds(const GridDev& G, const DockDev& D, float4* lds) {
  BlockLds b;
  b.tab = reinterpret_cast<int*>(lds);
  const int head = (G.table_entries(BOUNDS) + 3) / 4;
  b.ang = reinterpret_cast<float2*>(lds + head);
  b.scr = lds + head + (D.A + 1) / 2 + (size_t)(threadIdx.x >> 6) * dock_wave_float4(NSLOT);
  b.cand = b.scr + 64 * NSLOT;
  b.mkl = reinterpret_cast<uint32_t*>(b.scr + dock_wave_float4(NSLOT) - 16 * NSLOT);
  fill_brick_tables(G, b.tab, BOUNDS && G.tab_bounds);
  for (int j = threadIdx.x; j < D.A; j += blockDim.x) b.ang[j] = make_float2(D.angles[2 * j], D.angles[2 * j + 1]);
  __syncthreads();
  return b;
}

template <int NSLOT, int SPL>
__global__ __launch_bounds__(256) void dock_plain_kernel(DockArgs X, int lig) {
  extern __shared__ float4 lds[];
  const BlockLds B = block_lds<NSLOT, SPL == 0>(X.G, X.D, lds);
  const int wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6;
  const int r = blockIdx.x * nwaves + wave;
  if (r >= X.D.R) return;
  Samples sm;
  SampleReg<SPL ? SPL : 1> every;
  if constexpr (SPL > 0)
    load_every_sample(X.D, B.ang, every);
  else
    load_samples(X.G, X.D, B.ang, sm);
  LigReg<NSLOT> L;
  load_ligand(X.Lg, lig, L);
  if (L.N > 64 * NSLOT) {   // the host's sizes are not the device's: as in the bucket kernel
    if (lane_id() == 0) X.D.final_scores[(size_t)lig * X.D.R + r] = __builtin_nanf("");
    return;
  }
  store_masks(L, B.mkl);
  // One wavefront per SIMD or less: latency, so more fetches in flight (400 mixed
  // ligands of 256 restarts and 256 samples: 133 ms, 137 with four).  The staged
  // translation scan's read-then-use of each group's nodes pays only where its
  // bound saves passes (129 ms); with two passes or fewer the gathers stay direct
  // (100 samples, 64 restarts: 95 ms, 99 staged).
  dock_restart<NSLOT, false, 8, SPL>(kernel_args(), sm, every, L, lig, r, B);
}

// Bucketed method: persistent; wavefronts pull (ligand, restart chunk) items of
// one size bucket from an atomic cursor until the bucket is drained.  Occupancy
// target per instance (wavefronts per SIMD), chosen by measurement.  Bounded scans: 8 000
// mixed ligands take 163 ms at 5 per SIMD (96 VGPRs), 166 at 6, 174 at 7.  Scans of every
// sample (without the clamp-free variants and lists): 4 000 of them, 256 and 128 samples,
// 68.8 and 44.9 ms at 5, 66.6 and 43.9 at 6, 70.7 and 44.9 at 7; 1 200 ligands of 65 to
// 128 atoms 76.9 and 47.5 ms at 4, 74.7 and 44.2 at 5, 74.1 and 46.3 at 6.
constexpr int bucket_waves_per_simd(int nslot, int spl) {
  return spl > 0 ? (nslot == 1 ? 6 : 5) : nslot == 1 ? 5 : 4;
}

// LONE: the instance for launches of at most two wavefronts per SIMD, where a
// wavefront waits for each of its fetches alone: more of them in flight, in the
// registers that nobody else needs.
template <bool LONE>
constexpr int in_flight() { return LONE ? 8 : 4; }

// Restarts per work item: the tuning's chunk, or fewer when the launch would
// have less than 16 items per wavefront.  A longer chunk saves ligand loads (a
// chunk of one costs under 1 % against eight); a shorter one keeps every
// wavefront of a small launch at work and its last items short.
__device__ __forceinline__ int restart_chunk(int chunk, long long restarts, int waves_per_block) {
  const long long share = restarts / (16LL * gridDim.x * waves_per_block);
  return share < 1 ? 1 : share < chunk ? (int)share : chunk;
}

template <int NSLOT, bool LONE, int SPL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(LONE ? 2 : bucket_waves_per_simd(NSLOT, SPL))))
void dock_bucket_kernel(DockArgs X, QueueDev Q) {
  extern __shared__ float4 lds[];
  const int b0 = __builtin_amdgcn_readfirstlane(Q.bucket_start[Q.bucket]);
  const int b1 = __builtin_amdgcn_readfirstlane(Q.bucket_start[Q.bucket + 1]);
  if (b0 == b1) return;   // no ligand of this class in the batch
  const BlockLds B = block_lds<NSLOT, SPL == 0>(X.G, X.D, lds);
  const int lane = lane_id();
  const int chunk = restart_chunk(Q.chunk, (long long)(b1 - b0) * X.D.R, blockDim.x >> 6);
  const int nch = (X.D.R + chunk - 1) / chunk;
  const long long n_items = (long long)(b1 - b0) * nch;
  Samples sm;
  SampleReg<SPL ? SPL : 1> every;
  if constexpr (SPL > 0)
    load_every_sample(X.D, B.ang, every);
  else
    load_samples(X.G, X.D, B.ang, sm);
  int cur_lig = -1;
  LigReg<NSLOT> L;
  for (;;) {
    int item = 0;
    if (lane == 0) item = atomicAdd(Q.cursor + Q.bucket, 1);
    item = __builtin_amdgcn_readlane(item, 0);
    if ((long long)item >= n_items) break;
    const int li = item / nch, ch = item - li * nch;
    const int lig = __builtin_amdgcn_readfirstlane(Q.perm[b0 + li]);
    if (lig != cur_lig) {
      load_ligand(X.Lg, lig, L);
      store_masks(L, B.mkl);
      cur_lig = lig;
    }
    const int r0 = ch * chunk, r1 = min(X.D.R, r0 + chunk);
    if (L.N > 64 * NSLOT) {
      // cannot happen with the host's plan (instances sized for the largest
      // ligand); marks the restarts instead of touching memory out of range
      for (int r = r0 + lane; r < r1; r += 64) X.D.final_scores[(size_t)lig * X.D.R + r] = __builtin_nanf("");
      continue;
    }
    for (int r = r0; r < r1; ++r) dock_restart<NSLOT, true, in_flight<LONE>(), SPL>(kernel_args(), sm, every, L, lig, r, B);
  }
}

// Several docking sites: the bucket kernel's loop over items (site, ligand of
// the bucket, restart chunk); each item works on its site's entry of the table.  The brick tables depend on the
// grid dimensions only, shared by every site.
template <int NSLOT, int SPL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(bucket_waves_per_simd(NSLOT, SPL))))
void dock_sites_kernel(DockArgs X, QueueDev Q, SitesDev Sd) {
  extern __shared__ float4 lds[];
  const int b0 = __builtin_amdgcn_readfirstlane(Q.bucket_start[Q.bucket]);
  const int b1 = __builtin_amdgcn_readfirstlane(Q.bucket_start[Q.bucket + 1]);
  if (b0 == b1) return;   // no ligand of this class in the batch
  const BlockLds B = block_lds<NSLOT, SPL == 0>(X.G, X.D, lds);
  const int lane = lane_id();
  const int nlig = b1 - b0;
  const int chunk = restart_chunk(Q.chunk, (long long)nlig * X.D.R * Sd.n_sites, blockDim.x >> 6);
  const int nch = (X.D.R + chunk - 1) / chunk;
  const long long per_site = (long long)nlig * nch;
  const long long n_items = per_site * Sd.n_sites;
  Samples sm;
  SampleReg<SPL ? SPL : 1> every;
  if constexpr (SPL > 0)
    load_every_sample(X.D, B.ang, every);
  else
    load_samples(X.G, X.D, B.ang, sm);
  int cur_lig = -1;
  LigReg<NSLOT> L;
  for (;;) {
    int item = 0;
    if (lane == 0) item = atomicAdd(Q.cursor + Q.bucket, 1);
    item = __builtin_amdgcn_readlane(item, 0);
    if ((long long)item >= n_items) break;
    int site, li, ch;
    if (Sd.site_major) {
      site = (int)(item / per_site);
      const int rem = (int)(item - site * per_site);
      li = rem / nch;
      ch = rem - li * nch;
    } else {
      li = item / (nch * Sd.n_sites);
      const int rem = item - li * nch * Sd.n_sites;
      site = rem / nch;
      ch = rem - site * nch;
    }
    const int lig = __builtin_amdgcn_readfirstlane(Q.perm[b0 + li]);
    if (lig != cur_lig) {
      load_ligand(X.Lg, lig, L);
      store_masks(L, B.mkl);
      cur_lig = lig;
    }
    const ArgsPtr S = (ArgsPtr)(Sd.sites + __builtin_amdgcn_readfirstlane(site));
    if constexpr (SPL == 0) sm.bound_t = X.D.T > 64 && translation_bounds(grid_of(S), X.D, sm.GT);   // the site's
    const int r0 = ch * chunk, r1 = min(X.D.R, r0 + chunk);
    if (L.N > 64 * NSLOT) {
      for (int r = r0 + lane; r < r1; r += 64) S->D.final_scores[(size_t)lig * X.D.R + r] = __builtin_nanf("");
      continue;
    }
    for (int r = r0; r < r1; ++r) dock_restart<NSLOT, true, 4, SPL>(S, sm, every, L, lig, r, B);
  }
}

// Per-ligand top-k over restarts (score descending, equal scores: lower r).  One
// wavefront per ligand.
__global__ __launch_bounds__(256) void topk_kernel(DockDev D, int n, int k, float* score, int32_t* rid,
                                                   float* all_scores) {
  const int wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6, lane = lane_id();
  const int lig = blockIdx.x * nwaves + wave;
  if (lig >= n) return;
  const float* fs = D.final_scores + (size_t)lig * D.R;
  if (all_scores)
    for (int r = lane; r < D.R; r += 64) all_scores[(size_t)lig * D.R + r] = fs[r];
  int pk = INT_MAX, pr = -1;   // previous selection (key, r)
  for (int qi = 0; qi < k; ++qi) {
    int best = INT_MIN, br = INT_MAX;
    for (int r = lane; r < D.R; r += 64) {
      const int key = orderable(fs[r] + 0.0f);
      const bool after = key < pk || (key == pk && r > pr);
      if (after && (key > best || (key == best && r < br))) { best = key; br = r; }
    }
    const int wmax = wave_reduce_i32(best, OpMax());
    const int rs = wave_reduce_i32(best == wmax ? br : INT_MAX, OpMin());
    pk = wmax;
    pr = rs;
    if (lane == 0) {
      score[(size_t)lig * k + qi] = fs[rs];
      rid[(size_t)lig * k + qi] = rs;
    }
  }
}

// The kept poses and pivots rebuilt from their recorded moves.  One wavefront per
// pose: a replay is a chain of dependent moves, so the poses of a ligand side by
// side take the time of one (64 ligands, 32 kept poses: 175 us one after another).
template <int NSLOT>
__global__ __launch_bounds__(256) void replay_kernel(LigDev Lg, DockDev D, int n, int k, const int32_t* rid, float* ox,
                                                     float* oy, float* oz, float* opiv) {
  const int wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6, lane = lane_id();
  for (long long w = (long long)blockIdx.x * nwaves + wave; w < (long long)n * k; w += (long long)gridDim.x * nwaves) {
    const int lig = __builtin_amdgcn_readfirstlane((int)(w / k));
    const int qi = __builtin_amdgcn_readfirstlane((int)(w - (long long)lig * k));
    LigReg<NSLOT> L;
    load_ligand(Lg, lig, L);
    if (L.N > 64 * NSLOT) continue;   // cannot happen: the instance is sized for the largest ligand
    const int r = min(max(__builtin_amdgcn_readfirstlane(rid[w]), 0), D.R - 1);
    PoseReg<NSLOT> p;
    replay_restart(Lg, D, L, lig, r, p);
    const size_t dst = (size_t)k * L.abase + (size_t)qi * L.N;
#pragma unroll
    for (int s = 0; s < NSLOT; ++s) {
      const int a = s * 64 + lane;
      if (a < L.N) {
        ox[dst + a] = p.x[0][s];
        oy[dst + a] = p.x[1][s];
        oz[dst + a] = p.x[2][s];
      }
    }
    const float pv = lane == 0 ? p.piv[0] : lane == 1 ? p.piv[1] : p.piv[2];
    if (opiv && lane < 3) opiv[(size_t)w * 3 + lane] = pv;
  }
}

// ---------------------------------------------------------------- dispatch
size_t dock_lds_bytes(int nslot, int wpb, int tab_len, int angles) {
  return ((size_t)(tab_len + 3) / 4 + (size_t)(angles + 1) / 2 + (size_t)wpb * dock_wave_float4(nslot)) * sizeof(float4);
}

// Instances: NSLOT atom slots per lane; bounded scans (SPL 0; in kernels of their own for
// LONE launches), or scans of every sample, SPL per lane.
#define LG_INSTANCES(nslot, spl, CALL)                                                     \
  switch ((nslot) * 10 + (spl)) {                                                          \
    case 10: CALL(1, 0); case 20: CALL(2, 0); case 30: CALL(3, 0); case 40: CALL(4, 0);    \
    case 11: CALL(1, 1); case 12: CALL(1, 2); case 14: CALL(1, 4);                         \
    case 22: CALL(2, 2); case 24: CALL(2, 4);                                              \
    default: return hipErrorInvalidValue;                                                  \
  }

template <int NS, int SP>
hipError_t plain_launch(int wpb, const DockArgs& X, int lig, hipStream_t st) {
  if constexpr (SP == 1) {
    return hipErrorInvalidValue;   // never the better one here: no such instance
  } else {
    hipLaunchKernelGGL((dock_plain_kernel<NS, SP>), dim3((X.D.R + wpb - 1) / wpb), dim3(64 * wpb),
                       dock_lds_bytes(NS, wpb, X.G.table_entries(SP == 0), X.D.A), st, X, lig);
    return hipGetLastError();
  }
}

hipError_t launch_dock_plain(int nslot, int spl, int wpb, const GridDev& G, const LigDev& Lg, const DockDev& D, int lig,
                             hipStream_t st) {
#define CALL(NS, SP) return plain_launch<NS, SP>(wpb, DockArgs{G, Lg, D}, lig, st)
  LG_INSTANCES(nslot, spl, CALL)
#undef CALL
}

template <int NS, int SP>
constexpr auto bucket_kernel(bool lone) {
  return SP == 0 && lone ? dock_bucket_kernel<NS, true, 0> : dock_bucket_kernel<NS, false, SP>;
}

hipError_t launch_dock_bucket(int nslot, int spl, bool lone, int wpb, int blocks, const GridDev& G, const LigDev& Lg,
                              const DockDev& D, const QueueDev& Q, hipStream_t st) {
#define CALL(NS, SP)                                                                                 \
  {                                                                                                  \
    hipLaunchKernelGGL((bucket_kernel<NS, SP>(lone)), dim3(blocks), dim3(64 * wpb),                  \
                       dock_lds_bytes(NS, wpb, G.table_entries(SP == 0), D.A), st, DockArgs{G, Lg, D}, Q);          \
    return hipGetLastError();                                                                        \
  }
  LG_INSTANCES(nslot, spl, CALL)
#undef CALL
}

hipError_t launch_dock_sites(int nslot, int spl, int wpb, int blocks, const GridDev& G, const LigDev& Lg, const DockDev& D,
                             const QueueDev& Q, const SitesDev& Sd, hipStream_t st) {
#define CALL(NS, SP)                                                                                 \
  {                                                                                                  \
    hipLaunchKernelGGL((dock_sites_kernel<NS, SP>), dim3(blocks), dim3(64 * wpb),                    \
                       dock_lds_bytes(NS, wpb, G.table_entries(SP == 0), D.A), st, DockArgs{G, Lg, D}, Q, Sd);      \
    return hipGetLastError();                                                                        \
  }
  LG_INSTANCES(nslot, spl, CALL)
#undef CALL
}

// Resident blocks per compute unit of a bucket kernel instance (the b of Eq. 1).
hipError_t occupancy_dock_bucket(int nslot, int spl, bool lone, int wpb, int tab_len, int angles, int* blocks_per_cu) {
#define CALL(NS, SP)                                                                                           \
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, bucket_kernel<NS, SP>(lone), 64 * wpb,    \
                                                      dock_lds_bytes(NS, wpb, tab_len, angles))
  LG_INSTANCES(nslot, spl, CALL)
#undef CALL
}

hipError_t attributes_dock_bucket(int nslot, int spl, bool lone, hipFuncAttributes* attr) {
#define CALL(NS, SP) return hipFuncGetAttributes(attr, reinterpret_cast<const void*>(bucket_kernel<NS, SP>(lone)))
  LG_INSTANCES(nslot, spl, CALL)
#undef CALL
}

#define LG_DISPATCH(nslot, CALL)              \
  switch (nslot) {                            \
    case 1: CALL(1); case 2: CALL(2);         \
    case 3: CALL(3); case 4: CALL(4);         \
    default: return hipErrorInvalidValue;     \
  }

hipError_t launch_topk(int nslot, const LigDev& Lg, const DockDev& D, int n, int k, float* score, int32_t* rid,
                       float* ox, float* oy, float* oz, float* all_scores, float* pivot, hipStream_t st) {
  if (n == 0) return hipSuccess;
  const int wpb = 4;
  hipLaunchKernelGGL(topk_kernel, dim3((n + wpb - 1) / wpb), dim3(64 * wpb), 0, st, D, n, k, score, rid, all_scores);
  const long long poses = (long long)n * k;
  const dim3 grid((unsigned)std::min<long long>((poses + wpb - 1) / wpb, 1 << 22)), block(64 * wpb);
#define CALL(NS)                                                                                         \
  {                                                                                                      \
    hipLaunchKernelGGL(replay_kernel<NS>, grid, block, 0, st, Lg, D, n, k, rid, ox, oy, oz, pivot);      \
    return hipGetLastError();                                                                            \
  }
  LG_DISPATCH(nslot, CALL)
#undef CALL
}

}  // namespace lg
