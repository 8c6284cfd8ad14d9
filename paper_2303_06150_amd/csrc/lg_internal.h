// Internal device-side types and wavefront primitives of the docking library.
// gfx950 only: 64-lane wavefronts, DPP row operations, readlane.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

#include "lg.h"

namespace lg {

// Grid as the kernels see it: the library stores the pocket with a one-node
// border of out_value on every side, so a clamp of the node index to [-1, n]
// replaces the per-axis range test of the nearest-voxel rule.  g0 points at
// padded node (1,1,1) = logical node (0,0,0); strides are the padded ones.
struct GridDev {
  const float* g0;
  const char* gb;   // padded grid, byte addressed: node (ix,iy,iz) in [-1,n]^3 sits at
  int bs[3];        //   gb + b0 + ix*bs[0] + iy*bs[1] + iz*bs[2] (bs = byte strides 4, 4(nx+2), ...)
  int b0;           //   b0 = byte offset of logical node (0,0,0); every offset is >= 0 and < 2^31
  // The scans read a second copy in 4x4x2-node bricks, one 128-byte cache line
  // each, so the samples of one lookup instruction (an arc or a short segment)
  // touch few lines.  Byte offset of padded node (px,py,pz) = Tx[px]+Ty[py]+Tz[pz]
  // with per-axis tables built in LDS by every block (brick_tables).
  const char* gk;
  int nb[3];        // bricks per axis
  int tab_base[3];  // first entry of each axis table in the LDS table array
  int tab_len;      // entries of all the LDS tables
  float c0[3];      // nearest-node map: f = fma(x, inv_h, c0), c0 = fma(-o, inv_h, 0.5)
  int n[3];
  int stride[3];    // 1, nx+2, (nx+2)(ny+2)
  float o[3];
  float fn[3];      // (float)n per axis
  float fn1[3];     // (float)(n-1) per axis, trilinear range
  float inv_h;
  float out;
  // Upper bounds for the scans: 16-bit copies of the padded grid, dilated (node i
  // holds the largest value of a window) and rounded up to whole multiples of
  // bound_scale.  Copy 4 e + l: w x w nodes i .. i + w - 1 of the plane across
  // axis e, w = 2, 3, 4, 6, in bricks of 8 x 8 nodes of that plane.  Copy 12 + l:
  // w^3 nodes i - w/2 + 1 .. i + w/2, w = 2, 4, 6, in bricks of 4 x 4 x 4.  A
  // brick is a 128-byte line.  nullptr where there are none (very large grids,
  // non-finite values).
  const char* dil;
  uint32_t dil_stride;   // bytes per copy
  float bound_scale;
  float vmax;            // largest |value| of the grid, infinite if one is not finite
  int nb8[3], nb4[3];    // bricks of 8 and of 4 nodes per axis
  int tab_p, tab_q[3], tab_c[3];   // first entries of their offset tables (see fill_brick_tables)
  int tab_bounds;                  // the tables hold them
  // entries of the LDS tables, with or without those of the bounds (which come last)
  __host__ __device__ int table_entries(bool bounds) const { return bounds ? tab_len : tab_base[2] + n[2] + 2; }
};

constexpr int kDilated = 15;   // dilated copies

struct LigDev {
  const int32_t* atom_offset;
  const int32_t* tors_offset;
  const float* x;
  const float* y;
  const float* z;
  const uint32_t* mask;
  const int32_t* tors_atoms;
  const float* inv_len;
  const float* ref;
};

struct DockDev {
  int R, A, T, S;
  float delta, clash2;
  float clash_r2;          // (sqrt(clash2) + margin)^2: pairs farther apart on their circles never clash
  float clash;             // sqrt(clash2), 0 if that is not positive
  int lazy_clash;          // 1: no clash tests of whole groups, only of samples that beat the best so far
  float c[3];
  const float* restarts;   // [R][12]
  const float* angles;     // [A][2]
  float* final_scores;     // [n*R]
  uint16_t* moves;         // [R*S*(6n + total_torsions)]: selected sample of every scan;
                           // ligand i restart r sweep s at R*S*(6i + tors_offset[i]) + (r*S + s)*(6 + K_i)
  int16_t* trace;          // optional [n][R][S][trace_w]
  int trace_w;
};

// Refinement parameters and outputs.  kpl poses per ligand: pose i is member
// i % kpl of ligand i / kpl, its coordinates at kpl*atom_offset[lig] + member*N.
struct RefineDev {
  int steps, kpl;
  const int32_t* lig_ids;  // ligands of this launch (a size class), or nullptr: 0..n-1
  float eta_t, eta_w, eta_th, clip_t, clip_w, clip_th, clash2;
  float* xo;
  float* yo;
  float* zo;
  float* score;
};

// What a docking wavefront works on: the first kernel argument, or a site's entry
// in device memory.  The scans read it through this pointer, anew in each scan
// (uniform scalar loads): held in scalar registers over the whole restart loop,
// its 80 words would spill into vector lanes and come back through the vector
// ALU at every use.
struct DockArgs {
  GridDev G;
  LigDev Lg;
  DockDev D;
};
typedef const __attribute__((address_space(4))) DockArgs* ArgsPtr;

template <class T>
__device__ __forceinline__ T fresh_copy(const __attribute__((address_space(4))) T* p) {
  asm volatile("" : "+s"(p));   // loaded here
  T v;
  __builtin_memcpy(&v, (const T*)p, sizeof v);
  return v;
}
__device__ __forceinline__ GridDev grid_of(ArgsPtr S) { return fresh_copy(&S->G); }
__device__ __forceinline__ LigDev ligands_of(ArgsPtr S) { return fresh_copy(&S->Lg); }
__device__ __forceinline__ DockDev dock_of(ArgsPtr S) { return fresh_copy(&S->D); }

// Several docking sites in one launch: grids of identical dimensions and
// spacing (so one set of brick tables serves all); per site its own grid copies,
// origin, centre, final scores and move records.  Items are (site, ligand,
// chunk), site by site or with the sites interleaved per ligand.
struct SitesDev {
  const DockArgs* sites;    // device [n_sites]
  int n_sites;
  int site_major;           // 1: site by site; 0: every site of a ligand in turn
};

// LDS of a docking wavefront, in float4: scan data of 64*nslot atoms, risky
// torsion pairs, data of the moving atoms, the ligand's fragment masks (one
// 32-bit word per atom).  The two middle regions together hold the bound-pass
// data of a rotation scan (two float4 per atom) or the staged nodes of a
// translation scan; in scans of every sample the pair list takes both.  The bounded
// scans' list takes what leaves the instances their occupancy (a list holds at least
// every pair of one atom).
constexpr int pair_cap(int nslot) { return nslot == 1 ? 128 : 64 * nslot; }
constexpr int dock_wave_float4(int nslot) { return 2 * 64 * nslot + pair_cap(nslot) + 16 * nslot; }
constexpr int stage_floats(int nslot) { return 4 * (pair_cap(nslot) + 64 * nslot); }

// Persistent work source of one bucket: items are (ligand of the bucket,
// chunk of `chunk` restarts), pulled from `cursor` by whole wavefronts.
struct QueueDev {
  const int32_t* perm;          // ligand ids grouped by bucket
  const int32_t* bucket_start;  // [B+1]
  int32_t* cursor;              // one counter per bucket
  int bucket;
  int chunk;
};

// Cluster bounds of the device-side input preparation: atom cluster c holds
// ligands with atoms <= atom[c] (first match), rotamer cluster c bonds <= rot[c].
struct ClusterBounds {
  int na, nr;
  int atom[16];
  int rot[32];
};

// Radix-select state of the global ranking: the selected key prefix and its
// mask, how many keys of that prefix are still to take, whether the threshold is
// fixed, and the compaction counter.
struct RankState {
  uint64_t prefix, mask;
  uint32_t need, done, count, pad;
};

// ------------------------------------------------------------ wave helpers
__device__ __forceinline__ int lane_id() { return (int)__lane_id(); }

// Orders a wavefront's LDS writes before its later LDS reads by other lanes:
// waits for outstanding LDS operations and stops the compiler from moving
// memory operations across this point.
__device__ __forceinline__ void wave_sync() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_wave_barrier();
}

// Row-of-16 all-reduce with DPP, then the four row results through readlane.
// Needs all 64 lanes active.
template <class Op>
__device__ __forceinline__ int wave_reduce_i32(int v, Op op) {
  v = op(v, __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true));   // quad_perm [1,0,3,2]
  v = op(v, __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true));   // quad_perm [2,3,0,1]
  v = op(v, __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, true));  // row_half_mirror
  v = op(v, __builtin_amdgcn_mov_dpp(v, 0x140, 0xF, 0xF, true));  // row_mirror
  int a = __builtin_amdgcn_readlane(v, 0), b = __builtin_amdgcn_readlane(v, 16);
  int c = __builtin_amdgcn_readlane(v, 32), d = __builtin_amdgcn_readlane(v, 48);
  return op(op(a, b), op(c, d));
}

struct OpMax { __device__ int operator()(int a, int b) const { return a > b ? a : b; } };
struct OpMin { __device__ int operator()(int a, int b) const { return a < b ? a : b; } };
struct OpAdd { __device__ int operator()(int a, int b) const { return a + b; } };
struct OpAddF {
  __device__ int operator()(int a, int b) const { return __float_as_int(__int_as_float(a) + __int_as_float(b)); }
};

__device__ __forceinline__ float wave_sum(float v) { return __int_as_float(wave_reduce_i32(__float_as_int(v), OpAddF())); }

// Per-axis byte-offset tables of the brick layouts, indexed by padded node
// coordinate p in [0, n+1]; filled by all threads of a block.
//   grid (4 x 4 x 2 floats), axes x, y, z at tab_base:
//     (p>>2)*128 + (p&3)*4, (p>>2)*128*nbx + (p&3)*16, (p>>1)*128*nbx*nby + (p&1)*64
//   dilated planes (8 x 8 of 16 bits): the plane across axis e has first axis
//     e + 1 and second axis e + 2 (mod 3); first: (p>>3)*128 + (p&7)*2 at tab_p, for
//     every axis; second: (p>>3)*128*nb8[first] + (p&7)*16 at tab_q[axis]
//   dilated cubes (4 x 4 x 4 of 16 bits) at tab_c:
//     (p>>2)*128 + (p&3)*2, (p>>2)*128*nb4x + (p&3)*8, (p>>2)*128*nb4x*nb4y + (p&3)*32
__device__ __forceinline__ void fill_brick_tables(const GridDev& G, int* tab, bool bounds) {
  const int longest = max(G.n[0], max(G.n[1], G.n[2])) + 2;
  for (int p = threadIdx.x; p < longest; p += blockDim.x) {
    if (bounds) tab[G.tab_p + p] = (p >> 3) * 128 + (p & 7) * 2;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      if (p >= G.n[a] + 2) continue;
      tab[G.tab_base[a] + p] = a == 0   ? (p >> 2) * 128 + (p & 3) * 4
                               : a == 1 ? (p >> 2) * 128 * G.nb[0] + (p & 3) * 16
                                        : (p >> 1) * 128 * G.nb[0] * G.nb[1] + (p & 1) * 64;
      if (!bounds) continue;
      tab[G.tab_q[a] + p] = (p >> 3) * 128 * G.nb8[(a + 2) % 3] + (p & 7) * 16;
      tab[G.tab_c[a] + p] = a == 0   ? (p >> 2) * 128 + (p & 3) * 2
                            : a == 1 ? (p >> 2) * 128 * G.nb4[0] + (p & 3) * 8
                                     : (p >> 2) * 128 * G.nb4[0] * G.nb4[1] + (p & 3) * 32;
    }
  }
}

// 24-bit signed multiply-add (full-rate v_mad_i32_i24); |a| <= 1025, |b| < 2^23.
__device__ __forceinline__ int mad24(int a, int b, int c) { return __mul24(a, b) + c; }

// Grid value at a non-negative byte offset from the padded base (32-bit offset,
// scalar base address).
__device__ __forceinline__ float grid_at(const char* gb, int off) {
  return *reinterpret_cast<const float*>(gb + (uint32_t)off);
}

// Bound of a dilated copy at a byte offset, in units of bound_scale.
__device__ __forceinline__ int bound_at(const char* dil, uint32_t off) {
  return *reinterpret_cast<const int16_t*>(dil + off);
}

// Order-preserving map of a float to a signed int (total order on non-NaN).
__device__ __forceinline__ int orderable(float f) {
  int b = __float_as_int(f);
  return b ^ ((b >> 31) & 0x7FFFFFFF);
}

__device__ __forceinline__ bool wave_any(bool p) { return __ballot(p) != 0ull; }

// Floor of f for a node map value already known to lie in [-1, n].
__device__ __forceinline__ int floor_node(float f) {
  int i;
  asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(i) : "v"(f));
  return i;
}

// Node index on the padded grid for coordinate offset f (already scaled):
// floor of f clamped to [-1, n] -- -1 and n land on the out_value border.
__device__ __forceinline__ int clamp_node(float f, float fn) {
  f = __builtin_amdgcn_fmed3f(f, -1.0f, fn);
  int i;
  asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(i) : "v"(f));
  return i;
}

}  // namespace lg
