// Pose scoring (nearest / trilinear + force-torque adjoint), pocket padding,
// device-side input preparation (classify / scan / scatter into size buckets)
// and validation kernels.
#include "lg_device.h"

#include <algorithm>
#include <climits>

namespace lg {

__global__ void zero_kernel(int32_t* p, int n) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0;
}

// Sum over the W lanes (16 or 64) of a row, on every lane of it.
template <int W>
__device__ __forceinline__ float row_sum(float v) {
  if (W == 64) return wave_sum(v);
  auto add = [&](int moved) { v += __int_as_float(moved); };
  add(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, true));    // quad_perm [1,0,3,2]
  add(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x4E, 0xF, 0xF, true));    // quad_perm [2,3,0,1]
  add(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x141, 0xF, 0xF, true));   // row_half_mirror
  add(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x140, 0xF, 0xF, true));   // row_mirror
  return v;
}

// Score of every pose = sum over its atoms in atom order; optional gradient with
// respect to (t, omega, theta) at zero (force / torque form).
// A pose takes a row of W lanes, atom W s + lane in slot s < S.  With rows of 16 a
// wavefront works on four poses, its lanes are filled to a sixteenth of a pose, and a
// sum over a pose is four DPP steps.  Bounded by vector issue: per bond 16 operations
// a slot and 12 to add up.  A wavefront per pose spent three quarters of its time on
// atom-by-atom broadcasts and on 64-lane reductions of 41 atoms: 200 000 poses of
// 41 atoms 520 us, as it is 231 us.
template <int S, int W>
__global__ __launch_bounds__(256) void score_kernel(GridDev G, LigDev P, int n, int interp, float* score,
                                                     float* grad) {
  extern __shared__ float4 lds[];
  const int wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6, lane = lane_id(), row = lane / W, l = lane % W;
  float4* pos = lds + (size_t)(wave * (64 / W) + row) * (W * S);   // the pose's atoms: coordinates and value
  const int i = (blockIdx.x * nwaves + wave) * (64 / W) + row;
  const bool live = i < n;
  const int abase = live ? P.atom_offset[i] : 0, N = live ? P.atom_offset[i + 1] - abase : 0;
  const int most = wave_reduce_i32(N, OpMax());
  const bool want = grad && interp == LG_TRILINEAR;
  float x[3][S], g[3][S];
  uint32_t mk[S];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    x[0][s] = x[1][s] = x[2][s] = g[0][s] = g[1][s] = g[2][s] = 0.f;
    mk[s] = 0u;
    if (W * s >= most) continue;
    const int a = W * s + l;
    if (a < N) {
      const float px = P.x[abase + a], py = P.y[abase + a], pz = P.z[abase + a];
      x[0][s] = px;
      x[1][s] = py;
      x[2][s] = pz;
      if (want) mk[s] = P.mask[abase + a];
      float gg[3] = {0.f, 0.f, 0.f};
      const float v = interp == LG_TRILINEAR ? trilinear(G, px, py, pz, gg) : nearest(G, px, py, pz);
      g[0][s] = gg[0];
      g[1][s] = gg[1];
      g[2][s] = gg[2];
      pos[a] = make_float4(px, py, pz, v);
    }
  }
  wave_sync();
  // the score by the row's first lane, atom after atom
  if (l == 0 && live) {
    float total = 0.f;
    int a = 0;
    for (; a + 4 <= N; a += 4) {
      const float v0 = pos[a].w, v1 = pos[a + 1].w, v2 = pos[a + 2].w, v3 = pos[a + 3].w;
      total = total + v0;
      total = total + v1;
      total = total + v2;
      total = total + v3;
    }
    for (; a < N; ++a) total = total + pos[a].w;
    score[i] = total;
  }
  if (!want) return;
  const int toff = live ? P.tors_offset[i] : 0, K = live ? P.tors_offset[i + 1] - toff : 0;
  float* out = grad + 6 * (size_t)(live ? i : 0) + toff;
  {
    float Pv[3], f[3] = {0.f, 0.f, 0.f}, tq[3] = {0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < 3; ++c) Pv[c] = live ? P.ref[3 * (size_t)i + c] : 0.f;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      if (W * s >= most) continue;
      const float rx = x[0][s] - Pv[0], ry = x[1][s] - Pv[1], rz = x[2][s] - Pv[2];
      f[0] += g[0][s];
      f[1] += g[1][s];
      f[2] += g[2][s];
      tq[0] += ry * g[2][s] - rz * g[1][s];
      tq[1] += rz * g[0][s] - rx * g[2][s];
      tq[2] += rx * g[1][s] - ry * g[0][s];
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      f[c] = row_sum<W>(f[c]);
      tq[c] = row_sum<W>(tq[c]);
    }
    const float mine = l == 0 ? f[0] : l == 1 ? f[1] : l == 2 ? f[2] : l == 3 ? tq[0] : l == 4 ? tq[1] : tq[2];
    if (l < 6 && live) out[l] = mine;
  }
  // bonds W b .. W b + W - 1 of the poses: lane l holds bond W b + l's axis and takes its
  // sums
  const int bonds = wave_reduce_i32(K, OpMax());
  for (int b = 0; W * b < bonds; ++b) {
    const int mine = W * b + l;
    int pa = 0, pb = 0;
    if (mine < K) {
      pa = P.tors_atoms[2 * (toff + mine)];
      pb = P.tors_atoms[2 * (toff + mine) + 1];
    }
    float own[3] = {0.f, 0.f, 0.f};
    const int last = min(W, bonds - W * b);
    for (int q = 0; q < last; ++q) {
      const int k = W * b + q;
      const float4 at = pos[__builtin_amdgcn_ds_bpermute((row * W | q) << 2, pa)];   // bond k's pivot atom, of the row's pose
      float t[3] = {0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < S; ++s) {
        if (W * s >= most) continue;
        const bool in = (mk[s] >> k) & 1u;
        const float rx = x[0][s] - at.x, ry = x[1][s] - at.y, rz = x[2][s] - at.z;
        const float t0 = ry * g[2][s] - rz * g[1][s], t1 = rz * g[0][s] - rx * g[2][s], t2 = rx * g[1][s] - ry * g[0][s];
        t[0] += in ? t0 : 0.f;
        t[1] += in ? t1 : 0.f;
        t[2] += in ? t2 : 0.f;
      }
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const float sum = row_sum<W>(t[c]);
        own[c] = l == q ? sum : own[c];
      }
    }
    if (mine < K) {
      const float4 A = pos[pa], B = pos[pb];
      float ux = B.x - A.x, uy = B.y - A.y, uz = B.z - A.z;
      const float inv = 1.0f / sqrtf(ux * ux + uy * uy + uz * uz);
      ux *= inv;
      uy *= inv;
      uz *= inv;
      out[6 + mine] = ux * own[0] + uy * own[1] + uz * own[2];
    }
  }
}

// Instances by the batch's largest pose.  Above 128 atoms the 16 slots of a row of 16 take
// a pose's chain four times as long as a wavefront of its own, which shows while few
// poses leave the chip idle: wavefronts of their own up to 2 048 poses (64 poses of 180 to
// 256 atoms 66 us by rows, 44 so; 1 000 75, 53), or 8 192 where they are small on average
// (5 000 of 41 atoms with one of 200 among them 81, 66).  Many poses are faster by rows
// (200 000 of 41 atoms 231 us against 520 by a wavefront each).
hipError_t launch_score(int max_atoms, int total_atoms, const GridDev& G, const LigDev& P, int n, int interp, float* score,
                        float* grad, hipStream_t st) {
  if (n == 0) return hipSuccess;
  const bool own = max_atoms > 128 && n <= (total_atoms / n <= 64 ? 8192 : 2048);
  const int slots = own ? 4 : max_atoms <= 64 ? 4 : max_atoms <= 128 ? 8 : 16;
  const int wpb = slots == 16 ? 2 : 4;   // 32 KB of LDS a block at most
  const int rows = own ? 1 : 4, width = 64 / rows;
  const dim3 grid((unsigned)(((long long)n + rows * wpb - 1) / (rows * wpb))), block(64 * wpb);
  const size_t bytes = (size_t)wpb * rows * width * slots * sizeof(float4);
  if (own)
    hipLaunchKernelGGL((score_kernel<4, 64>), grid, block, bytes, st, G, P, n, interp, score, grad);
  else if (slots == 4)
    hipLaunchKernelGGL((score_kernel<4, 16>), grid, block, bytes, st, G, P, n, interp, score, grad);
  else if (slots == 8)
    hipLaunchKernelGGL((score_kernel<8, 16>), grid, block, bytes, st, G, P, n, interp, score, grad);
  else
    hipLaunchKernelGGL((score_kernel<16, 16>), grid, block, bytes, st, G, P, n, interp, score, grad);
  return hipGetLastError();
}

// Local parameters of every pose packed into the layout of lg_score's moves (6 i +
// tors_offset[i]: t, w, theta), and where each went.  One thread per pose and
// entry; a pose whose offsets do not fit the sizes is left out (lg_score reports it).
__global__ __launch_bounds__(256) void pack_moves_kernel(const int32_t* tors_offset, int n, int total_torsions,
                                                         const float* t, const float* w, const float* theta,
                                                         float* moves, int64_t* idx_t, int64_t* idx_w, int64_t* idx_th,
                                                         int64_t* pose_of_bond) {
  constexpr int kEntries = 6 + LG_MAX_TORSIONS;
  const long long e = blockIdx.x * 256LL + threadIdx.x;
  const int i = (int)(e / kEntries), q = (int)(e - (long long)i * kEntries);
  if (i >= n) return;
  const int t0 = tors_offset[i], t1 = tors_offset[i + 1];
  if (t0 < 0 || t1 < t0 || t1 > total_torsions) return;
  const long long base = 6LL * i + t0;
  if (q < 3) {
    moves[base + q] = t[3LL * i + q];
    idx_t[3LL * i + q] = base + q;
  } else if (q < 6) {
    moves[base + q] = w[3LL * i + q - 3];
    idx_w[3LL * i + q - 3] = base + q;
  } else if (q - 6 < t1 - t0) {
    const int b = t0 + q - 6;
    moves[base + q] = theta[b];
    idx_th[b] = base + q;
    pose_of_bond[b] = i;
  }
}

hipError_t launch_pack_moves(const int32_t* tors_offset, int n, int total_torsions, const float* t, const float* w,
                             const float* theta, float* moves, int64_t* idx_t, int64_t* idx_w, int64_t* idx_th,
                             int64_t* pose_of_bond, hipStream_t st) {
  const long long entries = (long long)n * (6 + LG_MAX_TORSIONS);
  hipLaunchKernelGGL(pack_moves_kernel, dim3((unsigned)((entries + 255) / 256)), dim3(256), 0, st, tors_offset, n,
                     total_torsions, t, w, theta, moves, idx_t, idx_w, idx_th, pose_of_bond);
  return hipGetLastError();
}

// Copy the grid into the padded layout with an out_value border.
__global__ void pad_kernel(const float* src, int nx, int ny, int nz, float out, float* dst) {
  const long long px = nx + 2, py = ny + 2, pz = nz + 2;
  const long long total = px * py * pz;
  for (long long idx = blockIdx.x * (long long)blockDim.x + threadIdx.x; idx < total;
       idx += (long long)gridDim.x * blockDim.x) {
    const long long ix = idx % px, iy = (idx / px) % py, iz = idx / (px * py);
    const bool in = ix >= 1 && ix <= nx && iy >= 1 && iy <= ny && iz >= 1 && iz <= nz;
    dst[idx] = in ? src[((iz - 1) * ny + (iy - 1)) * nx + (ix - 1)] : out;
  }
}

// Copy of the padded grid in 4x4x2 bricks (see GridDev); nodes past the padded
// extent (brick round-up) hold out_value and are never addressed.
__global__ void brick_kernel(const float* padded, int px, int py, int pz, int nbx, int nby, int nbz, float out,
                             float* brick) {
  const long long total = (long long)nbx * nby * nbz * 32;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
       e += (long long)gridDim.x * blockDim.x) {
    const long long b = e >> 5;
    const int w = (int)(e & 31);
    const int bx = (int)(b % nbx), by = (int)((b / nbx) % nby), bz = (int)(b / ((long long)nbx * nby));
    const int X = 4 * bx + (w & 3), Y = 4 * by + ((w >> 2) & 3), Z = 2 * bz + (w >> 4);
    brick[e] = (X < px && Y < py && Z < pz) ? padded[((long long)Z * py + Y) * px + X] : out;
  }
}

hipError_t launch_brick(const float* padded, int px, int py, int pz, int nbx, int nby, int nbz, float out,
                        float* brick, hipStream_t st) {
  hipLaunchKernelGGL(brick_kernel, dim3(1024), dim3(256), 0, st, padded, px, py, pz, nbx, nby, nbz, out, brick);
  return hipGetLastError();
}

// Whole multiple of scale at or above v.
__device__ __forceinline__ int round_up_to(float v, float scale) {
  int q = (int)ceilf(v / scale);
  if ((float)q * scale < v) ++q;
  return q;
}

// One step of a dilated copy of kind E (planes across axis E, or cubes: 3) from another
// one or from the grid's own values (src nullptr): the largest of the source's nodes at
// offsets lo and hi along the copy's axes (two of a plane, all three of a cube), clamped
// to the padded extent.  A wavefront writes whole bricks, 64 nodes in one line, eight of
// them one behind another along the third axis, so that the source's lines stay in the
// cache: all copies of 256^3 nodes with their allocation 1.2 ms, of 96^3 0.2 (a thread a
// node in the grid's own order, with divisions and a line a lane, 5.5 and 0.26).
template <int E>
__device__ __forceinline__ void dilate(const GridDev& G, const float* padded, const char* src, char* dst, int lo, int hi) {
  constexpr bool CUBE = E == 3;
  constexpr int P = CUBE ? 0 : (E + 1) % 3, Q = CUBE ? 1 : (E + 2) % 3, R = CUBE ? 2 : E;   // R: the third axis
  constexpr int BITS = CUBE ? 2 : 3, RUN = 8;
  const int np = G.n[P] + 2, nq = G.n[Q] + 2, nr = G.n[R] + 2;
  const int bp = CUBE ? G.nb4[P] : G.nb8[P], bq = CUBE ? G.nb4[Q] : G.nb8[Q], slices = CUBE ? G.nb4[R] : nr;
  const int step[3] = {1, G.n[0] + 2, (G.n[0] + 2) * (G.n[1] + 2)};
  auto offset = [&](int p, int q, int r) {   // as in fill_brick_tables
    return CUBE ? (uint32_t)(128 * (((r >> 2) * bq + (q >> 2)) * bp + (p >> 2)) + 2 * (((r & 3) * 4 + (q & 3)) * 4 + (p & 3)))
                : (uint32_t)(128 * ((r * bq + (q >> 3)) * bp + (p >> 3)) + 2 * ((q & 7) * 8 + (p & 7)));
  };
  auto value = [&](int p, int q, int r) {
    p = min(max(p, 0), np - 1);
    q = min(max(q, 0), nq - 1);
    r = min(max(r, 0), nr - 1);
    return src ? (int)*reinterpret_cast<const int16_t*>(src + offset(p, q, r))
               : round_up_to(padded[p * step[P] + q * step[Q] + r * step[R]], G.bound_scale);
  };
  const int lane = lane_id(), waves = blockDim.x >> 6;
  const int dp = lane & ((1 << BITS) - 1), dq = (lane >> BITS) & ((1 << BITS) - 1), dr = CUBE ? lane >> 4 : 0;
  const int runs = (slices + RUN - 1) / RUN, total = bp * bq * runs;
  for (int w = __builtin_amdgcn_readfirstlane(blockIdx.x * waves + (threadIdx.x >> 6)); w < total; w += gridDim.x * waves) {
    const int run = w / (bp * bq), b = w - run * (bp * bq), qb = b / bp, pb = b - qb * bp;
    const int p = (pb << BITS) + dp, q = (qb << BITS) + dq;
    for (int t = run * RUN; t < min(slices, run * RUN + RUN); ++t) {
      const int r = CUBE ? 4 * t + dr : t;
      if (p >= np || q >= nq || r >= nr) continue;
      int best = max(max(value(p + lo, q + lo, CUBE ? r + lo : r), value(p + hi, q + lo, CUBE ? r + lo : r)),
                     max(value(p + lo, q + hi, CUBE ? r + lo : r), value(p + hi, q + hi, CUBE ? r + lo : r)));
      if (CUBE)
        best = max(best, max(max(value(p + lo, q + lo, r + hi), value(p + hi, q + lo, r + hi)),
                             max(value(p + lo, q + hi, r + hi), value(p + hi, q + hi, r + hi))));
      *reinterpret_cast<int16_t*>(dst + offset(p, q, r)) = (int16_t)best;
    }
  }
}

// One step of the copies of kind e0 + blockIdx.y: level `to` from level `from` (-1: the
// grid's own values).  Windows of 2, 3, 4 and 6 nodes are built from those before (2 of
// the grid's own values, 3 and 4 of twos, 6 of fours).
__global__ __launch_bounds__(256) void dilate_kernel(GridDev G, const float* padded, int e0, int from, int to, int lo, int hi) {
  const int e = e0 + (int)blockIdx.y;
  char* copies = const_cast<char*>(G.dil) + (size_t)(4 * e) * G.dil_stride;
  const char* src = from < 0 ? nullptr : copies + (size_t)from * G.dil_stride;
  char* dst = copies + (size_t)to * G.dil_stride;
  switch (e) {
    case 0: dilate<0>(G, padded, src, dst, lo, hi); break;
    case 1: dilate<1>(G, padded, src, dst, lo, hi); break;
    case 2: dilate<2>(G, padded, src, dst, lo, hi); break;
    default: dilate<3>(G, padded, src, dst, lo, hi); break;
  }
}

// G: the finished description of the grid, dil included.  Planes (e = 0, 1, 2) and cubes
// (e = 3) that take the same step share a launch.
hipError_t launch_dilate(const GridDev& G, const float* padded, hipStream_t st) {
  const long long total = (long long)(G.n[0] + 2) * (G.n[1] + 2) * (G.n[2] + 2);
  const int blocks = (int)std::min<long long>(total / 2048 + 1, 8192);   // a wavefront of a block writes 512 nodes
  auto step = [&](int e0, int kinds, int from, int to, int lo, int hi) {
    hipLaunchKernelGGL(dilate_kernel, dim3(blocks, kinds), dim3(256), 0, st, G, padded, e0, from, to, lo, hi);
  };
  step(0, 4, -1, 0, 0, 1);   // planes 2 x 2, cubes i .. i + 1
  step(0, 3, 0, 1, 0, 1);    // 3 x 3
  step(0, 3, 0, 2, 0, 2);    // 4 x 4
  step(0, 3, 2, 3, 0, 2);    // 6 x 6
  step(3, 1, 0, 1, -1, 1);   // i - 1 .. i + 2
  step(3, 1, 1, 2, -1, 1);   // i - 2 .. i + 3
  return hipGetLastError();
}

// Bits of the largest |value|: NaN above infinity above every finite value.
__global__ void grid_max_kernel(const float* v, long long n, uint32_t* out) {
  uint32_t best = 0;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
    const uint32_t b = __float_as_uint(v[i]) & 0x7FFFFFFFu;
    best = b > best ? b : best;
  }
  const int wave = wave_reduce_i32((int)best, OpMax());
  if (lane_id() == 0) atomicMax(out, (uint32_t)wave);
}

hipError_t launch_grid_max(const float* padded, long long n, uint32_t* out, hipStream_t st) {
  hipLaunchKernelGGL(zero_kernel, dim3(1), dim3(64), 0, st, reinterpret_cast<int32_t*>(out), 1);
  hipLaunchKernelGGL(grid_max_kernel, dim3(256), dim3(256), 0, st, padded, n, out);
  return hipGetLastError();
}

hipError_t launch_pad(const float* src, int nx, int ny, int nz, float out, float* dst, hipStream_t st) {
  hipLaunchKernelGGL(pad_kernel, dim3(1024), dim3(256), 0, st, src, nx, ny, nz, out, dst);
  return hipGetLastError();
}

// ---------------------------------------------------- input preparation (buckets)
constexpr int kMaxBuckets = 16 * 32;   // ClusterBounds: atom x rotamer clusters

__device__ __forceinline__ int bucket_of(const int32_t* atom_offset, const int32_t* tors_offset, int i,
                                         const ClusterBounds& cb) {
  const int N = atom_offset[i + 1] - atom_offset[i];
  const int K = tors_offset[i + 1] - tors_offset[i];
  int ca = cb.na - 1, cr = cb.nr - 1;
  for (int c = cb.na - 1; c >= 0; --c)
    if (N <= cb.atom[c]) ca = c;
  for (int c = cb.nr - 1; c >= 0; --c)
    if (K <= cb.rot[c]) cr = c;
  return ca * cb.nr + cr;
}

// start[b] = counts[0] + .. + counts[b - 1] for b <= B, by the threads of a block
// (at least kMaxBuckets of them); run: kMaxBuckets ints of LDS, left holding start.
__device__ __forceinline__ void bucket_starts(int32_t* run, int count, int B, int32_t* start) {
  const int t = threadIdx.x;
  if (t < kMaxBuckets) run[t] = t < B ? count : 0;
  __syncthreads();
  for (int o = 1; o < B; o *= 2) {
    const int v = t < B && t >= o ? run[t - o] : 0;
    __syncthreads();
    if (t < B) run[t] += v;
    __syncthreads();
  }
  const int incl = t < B ? run[t] : 0;
  __syncthreads();
  if (t < B) {
    run[t] = incl - count;
    start[t] = incl - count;
    if (t == B - 1) start[B] = incl;
  }
  __syncthreads();
}

// The whole preparation of at most kSmallBatch ligands in one launch of one
// block: launches, not work, are what it costs there (five launches 23 us, this one 6).
constexpr int kSmallBatch = 8192;
__global__ __launch_bounds__(1024) void bucket_small_kernel(const int32_t* atom_offset, const int32_t* tors_offset,
                                                            int n, ClusterBounds cb, int32_t* counts, int32_t* start,
                                                            int32_t* perm, int32_t* cursors) {
  __shared__ int32_t cnt[kMaxBuckets], run[kMaxBuckets];
  __shared__ uint16_t cls[kSmallBatch];
  const int B = cb.na * cb.nr, t = threadIdx.x;
  if (t < B) {
    cnt[t] = 0;
    cursors[t] = 0;
  }
  __syncthreads();
  for (int i = t; i < n; i += 1024) {
    const int b = bucket_of(atom_offset, tors_offset, i, cb);
    cls[i] = (uint16_t)b;
    atomicAdd(&cnt[b], 1);
  }
  __syncthreads();
  const int mine = t < B ? cnt[t] : 0;
  if (t < B) counts[t] = mine;
  bucket_starts(run, mine, B, start);
  for (int i = t; i < n; i += 1024) perm[atomicAdd(&run[cls[i]], 1)] = i;
}

__global__ void bucket_init_kernel(int32_t* counts, int32_t* cursors, int B) {
  for (int b = threadIdx.x; b < B; b += blockDim.x) counts[b] = cursors[b] = 0;
}

// Counts and places per block in LDS, one addition per block and bucket to the
// global counters: one addition per ligand queues at the few counters (100 000
// ligands: 1.7 ms).
__global__ __launch_bounds__(256) void classify_kernel(const int32_t* atom_offset, const int32_t* tors_offset, int n,
                                                       ClusterBounds cb, int32_t* cls, int32_t* counts) {
  __shared__ int32_t cnt[kMaxBuckets];
  const int B = cb.na * cb.nr;
  for (int b = threadIdx.x; b < B; b += 256) cnt[b] = 0;
  __syncthreads();
  const int i0 = blockIdx.x * 1024, i1 = min(n, i0 + 1024);
  for (int i = i0 + threadIdx.x; i < i1; i += 256) {
    const int b = bucket_of(atom_offset, tors_offset, i, cb);
    cls[i] = b;
    atomicAdd(&cnt[b], 1);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < B; b += 256)
    if (cnt[b]) atomicAdd(&counts[b], cnt[b]);
}

__global__ __launch_bounds__(kMaxBuckets) void bucket_scan_kernel(const int32_t* counts, int B, int32_t* start,
                                                                  int32_t* fill) {
  __shared__ int32_t run[kMaxBuckets];
  const int t = threadIdx.x;
  bucket_starts(run, t < B ? counts[t] : 0, B, start);
  if (t < B) fill[t] = run[t];
}

__global__ __launch_bounds__(256) void scatter_kernel(const int32_t* cls, int n, int B, int32_t* fill, int32_t* perm) {
  __shared__ int32_t cnt[kMaxBuckets];
  for (int b = threadIdx.x; b < B; b += 256) cnt[b] = 0;
  __syncthreads();
  const int i0 = blockIdx.x * 1024;
  int place[4], b[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int i = i0 + u * 256 + (int)threadIdx.x;
    b[u] = i < n ? cls[i] : 0;
    place[u] = i < n ? atomicAdd(&cnt[b[u]], 1) : 0;
  }
  __syncthreads();
  for (int q = threadIdx.x; q < B; q += 256)
    if (cnt[q]) cnt[q] = atomicAdd(&fill[q], cnt[q]);   // now the block's first place in the bucket
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int i = i0 + u * 256 + (int)threadIdx.x;
    if (i < n) perm[cnt[b[u]] + place[u]] = i;
  }
}

// counts, start, perm and cursors of a batch; fill: B ints of scratch.
hipError_t launch_bucketing(const int32_t* atom_offset, const int32_t* tors_offset, int n, const ClusterBounds& cb,
                            int32_t* cls, int32_t* counts, int32_t* start, int32_t* fill, int32_t* perm,
                            int32_t* cursors, hipStream_t st) {
  const int B = cb.na * cb.nr;
  if (n <= kSmallBatch) {
    hipLaunchKernelGGL(bucket_small_kernel, dim3(1), dim3(1024), 0, st, atom_offset, tors_offset, n, cb, counts, start,
                       perm, cursors);
    return hipGetLastError();
  }
  const dim3 grid((n + 1023) / 1024);
  hipLaunchKernelGGL(bucket_init_kernel, dim3(1), dim3(kMaxBuckets), 0, st, counts, cursors, B);
  hipLaunchKernelGGL(classify_kernel, grid, dim3(256), 0, st, atom_offset, tors_offset, n, cb, cls, counts);
  hipLaunchKernelGGL(bucket_scan_kernel, dim3(1), dim3(kMaxBuckets), 0, st, counts, B, start, fill);
  hipLaunchKernelGGL(scatter_kernel, grid, dim3(256), 0, st, cls, n, B, fill, perm);
  return hipGetLastError();
}

// ---------------------------------------------------- device validation
// stats: [0] min atoms, [1] max atoms, [2] min bonds, [3] max bonds,
//        [4] count of bad bond ids, [5] count of inconsistent offsets
__global__ void check_kernel(const int32_t* atom_offset, const int32_t* tors_offset, const int32_t* tors_atoms,
                             int n, int total_atoms, int total_tors, int32_t* stats) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int a0 = atom_offset[i], a1 = atom_offset[i + 1];
  const int t0 = tors_offset[i], t1 = tors_offset[i + 1];
  const int N = a1 - a0, K = t1 - t0;
  atomicMin(&stats[0], N);
  atomicMax(&stats[1], N);
  atomicMin(&stats[2], K);
  atomicMax(&stats[3], K);
  bool offsets_ok = a0 >= 0 && a1 <= total_atoms && t0 >= 0 && t1 <= total_tors && N >= 0 && K >= 0;
  if (i == 0 && (a0 != 0 || t0 != 0)) offsets_ok = false;
  if (i == n - 1 && (a1 != total_atoms || t1 != total_tors)) offsets_ok = false;
  if (!offsets_ok) {
    atomicAdd(&stats[5], 1);
    return;
  }
  if (tors_atoms)
    for (int k = t0; k < t1; ++k) {
      const int a = tors_atoms[2 * k], b = tors_atoms[2 * k + 1];
      if (a < 0 || a >= N || b < 0 || b >= N || a == b) atomicAdd(&stats[4], 1);
    }
}

__global__ void check_init_kernel(int32_t* stats) {
  if (threadIdx.x == 0) {
    stats[0] = INT_MAX; stats[1] = INT_MIN; stats[2] = INT_MAX; stats[3] = INT_MIN;
    stats[4] = 0; stats[5] = 0;
  }
}

hipError_t launch_check(const int32_t* atom_offset, const int32_t* tors_offset, const int32_t* tors_atoms, int n,
                        int total_atoms, int total_tors, int32_t* stats, hipStream_t st) {
  hipLaunchKernelGGL(check_init_kernel, dim3(1), dim3(64), 0, st, stats);
  if (n > 0)
    hipLaunchKernelGGL(check_kernel, dim3((n + 255) / 256), dim3(256), 0, st, atom_offset, tors_offset, tors_atoms,
                       n, total_atoms, total_tors, stats);
  return hipGetLastError();
}

// ---------------------------------------------------------------- VALU rate probe
// Eight independent chains of non-packed VALU operations per lane, no memory
// traffic but one store per lane: the sustained issue rate of one operation
// (kinds 0-4), of two operations from different chains interleaved (5: v_fma_f32
// and v_add_u32), and of the nearest-node index sequence of a scan sample (6:
// v_add_f32, v_fma_f32, v_med3_f32, v_cvt_flr_i32_f32, v_lshl_add_u32,
// v_add3_u32, v_add_f32; seven VALU operations per step of a chain).
template <int KIND>
__global__ __launch_bounds__(256) void valu_probe_kernel(float* out, int iters, float a, float b) {
  float x[8];
  int y[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    x[i] = threadIdx.x * 0.001f + i;
    y[i] = threadIdx.x + i;
  }
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (KIND == 0) x[i] = fmaf(x[i], a, b);                      // v_fma_f32
      if (KIND == 1) x[i] = x[i] + a;                              // v_add_f32
      if (KIND == 2) y[i] = y[i] + it;                             // v_add_u32
      if (KIND == 3) x[i] = __builtin_amdgcn_fmed3f(x[i], a, b);   // v_med3_f32
      if (KIND == 4) y[i] = __mul24(y[i], 3) + it;                 // v_mad_i32_i24
      if (KIND == 5) {
        if (i < 4) x[i] = fmaf(x[i], a, b);
        else y[i] = y[i] + it;
      }
      if (KIND == 6) {
        const float f = __builtin_amdgcn_fmed3f(fmaf(x[i] + a, b, 0.5f), -1.0f, 90.0f);
        int n;
        asm volatile("v_cvt_flr_i32_f32 %0, %1" : "=v"(n) : "v"(f));
        y[i] = (n << 2) + y[i];
        y[i] = y[i] + n + it;
        x[i] = x[i] + (float)(y[i] & 1);
      }
    }
  }
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) s += x[i] + (float)y[i];
  out[(size_t)blockIdx.x * blockDim.x + threadIdx.x] = s;
}

hipError_t launch_valu_probe(int kind, int blocks, int iters, float* out, hipStream_t st) {
  const dim3 grid(blocks), block(256);
  switch (kind) {
    case 0: hipLaunchKernelGGL(valu_probe_kernel<0>, grid, block, 0, st, out, iters, 1.0001f, 0.5f); break;
    case 1: hipLaunchKernelGGL(valu_probe_kernel<1>, grid, block, 0, st, out, iters, 1.0001f, 0.5f); break;
    case 2: hipLaunchKernelGGL(valu_probe_kernel<2>, grid, block, 0, st, out, iters, 1.0001f, 0.5f); break;
    case 3: hipLaunchKernelGGL(valu_probe_kernel<3>, grid, block, 0, st, out, iters, 0.1f, 0.5f); break;
    case 4: hipLaunchKernelGGL(valu_probe_kernel<4>, grid, block, 0, st, out, iters, 0.1f, 0.5f); break;
    case 5: hipLaunchKernelGGL(valu_probe_kernel<5>, grid, block, 0, st, out, iters, 1.0001f, 0.5f); break;
    case 6: hipLaunchKernelGGL(valu_probe_kernel<6>, grid, block, 0, st, out, iters, 1e-7f, 1.0f); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace lg
