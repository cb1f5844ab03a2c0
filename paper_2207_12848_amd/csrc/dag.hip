// Dependency-graph construction for the transport sweep (gfx950).
//
// Compiled with -ffp-contract=off: the face orientation s = (Ox nx + Oy ny) + Oz nz
// must round exactly as written so that every kernel here (and any FP64
// implementation of the same expression) classifies each face identically.
//
//   k_count   per task (unit, cell): upwind/downwind counts, Aperp, boundary outflow
//   k_kahn    per unit, one workgroup: levels by Kahn's algorithm (algorithm 2's
//             counters, in LDS or a hash table there), ready cells compacted with
//             wavefront ballots
//   k_slices  the sweep's slices: every level in runs of at most 64 tasks
//   k_gather_tasks, k_fill  row lengths and rows of the upwind/downwind lists,
//             stored slice by slice in schedule order (and Aperp and the volumes in
//             schedule order, for the per-call preparation)
#include <hipcub/hipcub.hpp>

#include <type_traits>

#include "device.h"
#include "internal.h"
#include "sweep.h"

namespace sweep {

namespace {

constexpr int kCountBlock = 256;
// k_count_aligned and k_count_in: 512 threads, 16 directions of a 32-cell tile at a time
constexpr int kCountThreads = 512;
constexpr int kTileCells = 32;  // cells per tile of the cell-order kernels
__device__ __forceinline__ double orient(double ox, double oy, double oz, const double* n) {
  const double a = ox * n[0];
  const double b = oy * n[1];
  const double c = oz * n[2];
  return (a + b) + c;
}

// Face weight w = A |Omega . n| from the FP64 orientation s, rounded once to
// FP32: within one rounding of the FP64 weight however grazing the face is (a
// weight formed from FP32 normals would carry an absolute error of ~1e-7 A,
// large against A |s| for nearly parallel faces).  Twin half-faces have equal
// areas and exactly negated normals, so their s differ only in sign and both
// sides of a face get the same weight: what a cell sends through a face is
// exactly what its neighbour receives.
__device__ __forceinline__ float face_w(double A, double s) { return (float)(A * fabs(s)); }

// Signed weight of a face: its class, by the orientation, in the sign (outflow +, inflow -,
// also of a zero weight); NaN for neither.  A negative or undefined area (meshes that were
// not checked) gives an infinite weight of that class: the face still orders its cells, and
// makes its cell's Aperp infinite, which the sweep reports.
__device__ __forceinline__ float signed_w(double A, double s, double eps) {
  if (!(s > eps || s < -eps)) return __int_as_float(0x7fc00000);
  return copysignf(A >= 0.0 ? face_w(A, s) : INFINITY, (float)s);
}

// The cell-order kernel stages a tile of kTileCells consecutive cells' faces
// in LDS with coalesced loads (room for kTileFaces faces per cell on average,
// above the ~15.5 of a Voronoi cell and small enough for several workgroups per CU;
// a tile with more faces is read from global memory instead); the workgroup
// then covers every direction, 32 consecutive lanes handling the tile's cells
// for one direction.
constexpr int kTileFaces = 17;

struct FaceTile {
  int c0, cend;       // cells [c0, cend) of mesh m
  int64_t f0;         // first face of the tile
  bool in_lds;        // the tile's faces are in LDS
  const int64_t* fp;  // LDS copy of face_ptr[c0 .. cend] (relative to f0)
};

__host__ __device__ inline size_t tile_lds_bytes() {
  const size_t cap = (size_t)kTileCells * kTileFaces;
  return (8 * (kTileCells + 1) + cap * (24 + 8 + 4 + 1) + 15) / 16 * 16;
}

__device__ __forceinline__ FaceTile stage_tile(const MeshDev& M, int c0, unsigned char* smem) {
  FaceTile T;
  T.c0 = c0;
  T.cend = min(c0 + kTileCells, M.n_cells);
  const int nc = T.cend - c0;
  T.f0 = M.face_ptr[c0];
  const int nf = (int)(M.face_ptr[T.cend] - T.f0);
  constexpr int cap = kTileCells * kTileFaces;
  T.in_lds = nf <= cap;
  int64_t* fp = reinterpret_cast<int64_t*>(smem);
  for (int i = threadIdx.x; i <= nc; i += blockDim.x) fp[i] = M.face_ptr[c0 + i] - T.f0;
  if (T.in_lds) {
    double* nrm = reinterpret_cast<double*>(fp + kTileCells + 1);
    double* area = nrm + 3 * cap;
    int32_t* nbr = reinterpret_cast<int32_t*>(area + cap);
    int8_t* shift = reinterpret_cast<int8_t*>(nbr + cap);
    for (int i = threadIdx.x; i < 3 * nf; i += blockDim.x) nrm[i] = M.face_normal[3 * T.f0 + i];
    for (int i = threadIdx.x; i < nf; i += blockDim.x) {
      area[i] = M.face_area[T.f0 + i];
      nbr[i] = M.face_nbr[T.f0 + i];
      shift[i] = M.face_shift != nullptr ? M.face_shift[T.f0 + i] : (int8_t)0;
    }
  }
  T.fp = fp;
  return T;
}

// Per task: upwind/downwind counts, Aperp = sum of outflow w, boundary outflow
// weights, the signed weight of every face (NaN: neither inflow nor outflow) and
// the fixed-width row of downwind cells.  A row holds dn_width entries padded
// with -1; a task with more downwind cells keeps dn_width - 1 of them and stores
// -(o + 2) in the last slot, o being the offset in dn_ovf of [count, rest of the
// list].
//
// A workgroup takes a tile of kTileCells cells through the directions, kTileDirs at
// a time: first a thread per face works out its FP64 orientation and signed weight
// for those directions, then a thread per (cell, direction) goes over its faces'
// weights.  The weights of a tile lie in LDS in between (from memory when it has more
// than kTileFaces faces per cell).  The rows are assembled in LDS and written out as
// contiguous blocks (STAGE), or written straight to global memory.
//
// Bound by its writes, in runs of 128 bytes to 2 KB (3.2 GB at 64^3 cells and 84
// directions, 2.4 TB/s; a third of the issue slots are used).  64^3 cells, 84 directions:
// 1.29 ms, and 1.45 with the orientations taken in the cells' loop from normals in LDS and
// again for the weights; 2 M cells: 11.5 ms, and 13.3.  With few directions a tile's fixed
// part counts, its totals above all (CountTotals).
constexpr int kTileDirs = 8;
constexpr int kTileThreads = kTileDirs * kTileCells;
constexpr int kTileCap = kTileCells * kTileFaces;

size_t count_tile_bytes() {
  return sizeof(int64_t) * (kTileCells + 2) + sizeof(int32_t) * kTileCap + sizeof(float) * kTileDirs * kTileCap;
}

template <bool STAGE>
__global__ __launch_bounds__(kTileThreads) void k_count(DagBuildArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int s_max[2];
  __shared__ unsigned long long s_ent[2];
  if (threadIdx.x < 2) {
    s_max[threadIdx.x] = 0;
    s_ent[threadIdx.x] = 0ull;
  }
  const int tile = xcd_block(blockIdx.x, gridDim.x);
  const int m = a.cblk_mesh[tile];
  const MeshDev M = a.meshes[m];
  const int W = a.dn_width;
  const int c0 = a.cblk_c0[tile];
  const int nc = min(kTileCells, M.n_cells - c0);
  const int64_t f0 = M.face_ptr[c0];
  const int nf = (int)(M.face_ptr[c0 + nc] - f0);
  int64_t* s_fp = reinterpret_cast<int64_t*>(smem);
  int32_t* s_code = reinterpret_cast<int32_t*>(s_fp + kTileCells + 2);
  int32_t* srow = s_code + (kTileDirs + 1) * kTileCap;
  // directions at a time: fewer for a tile of many faces (its cells may have none at all)
  const int kd = nf > 0 ? min(kTileDirs, (kTileDirs + 1) * kTileCap / nf - 1) : kTileDirs;
  const bool in_lds = kd > 0;
  const int nd = in_lds ? kd : kTileDirs;
  float* s_w = reinterpret_cast<float*>(s_code + nf);  // [direction][face]
  for (int i = threadIdx.x; i <= nc; i += kTileThreads) s_fp[i] = M.face_ptr[c0 + i] - f0;
  if (in_lds)
    for (int f = threadIdx.x; f < nf; f += kTileThreads) s_code[f] = M.fcode[f0 + f];
  const int ci = threadIdx.x % kTileCells;
  const int dj = threadIdx.x / kTileCells;
  const int c = c0 + ci;
  const bool cell = ci < nc;
  float* const wface = a.wface + (int64_t)a.D * M.face_off + f0;
  int mi = 0, mo = 0;
  unsigned long long eu = 0, ed = 0;  // row entries of the thread's tasks
  for (int d0 = 0; d0 < a.D; d0 += nd) {
    for (int f = threadIdx.x; f < nf; f += kTileThreads) {
      const double n[3] = {M.face_normal[3 * (f0 + f)], M.face_normal[3 * (f0 + f) + 1], M.face_normal[3 * (f0 + f) + 2]};
      const double A = M.face_area[f0 + f];
#pragma unroll
      for (int j = 0; j < kTileDirs; ++j) {
        const int d = d0 + j;
        if (d >= a.D || j >= nd) break;
        const double sv = orient(a.dirs[3 * d], a.dirs[3 * d + 1], a.dirs[3 * d + 2], n);
        const float x = signed_w(A, sv, a.eps);
        wface[(int64_t)d * M.n_faces + f] = x;
        if (in_lds) s_w[j * nf + f] = x;
      }
    }
    __syncthreads();
    const int d = d0 + dj;
    const bool mine = dj < nd && d < a.D;
    if (cell && mine) {
      const int fb = (int)s_fp[ci], fe = (int)s_fp[ci + 1];
      const int64_t t = a.units[m * a.D + d].task_base + c;
      int32_t* row = STAGE ? srow + threadIdx.x * W : a.dnw + t * W;  // LDS: [dj][ci][W]
      int32_t* ovf = nullptr;
      int nup = 0, ndn = 0;
      double ap = 0.0, wall = 0.0, per = 0.0;
      auto run = [&](auto* weights, auto* codes) {
        for (int f = fb; f < fe; ++f) {
          const float w = weights[f];
          const int code = codes[f];
          if (isnan(w)) continue;
          if (signbit(w)) {
            nup += code >= 0 ? 1 : 0;
            if (isinf(w)) ap = -w;
            continue;
          }
          ap += w;
          if (code == -1) {
            wall += w;
          } else if (code < -1) {
            per += w;
          } else {
            if (ndn < W) {
              row[ndn] = code;
            } else {
              if (ndn == W) {  // the row is full: continue in an overflow list
                const int need = (fe - fb) + 2;
                const int o = atomicAdd(a.dn_ovf_top, need);
                // a pool that has run out gets the list in its spare end (the
                // host sees the count past the capacity and redoes the counts)
                ovf = a.dn_ovf + (o + need <= a.dn_ovf_cap ? o : a.dn_ovf_cap);
                ovf[1] = row[W - 1];
                row[W - 1] = -(o + 2);
              }
              ovf[1 + ndn - (W - 1)] = code;
            }
            ++ndn;
          }
        }
      };
      if (in_lds) run(s_w + dj * nf, s_code);
      else run(wface + (int64_t)d * M.n_faces, M.fcode + f0);
      if (ovf != nullptr) ovf[0] = ndn - (W - 1);
      if (nup >= a.big_min && a.big != nullptr) a.big[atomicAdd(a.big_top, 1)] = t;  // count too large for its place
      for (int q = ndn; q < W; ++q) row[q] = -1;
      a.indeg[t] = nup;
      a.rowlen_dn[t] = ndn;
      a.aperp[t] = (float)ap;
      a.bnd[t] = make_float2((float)wall, (float)per);
      mi = max(mi, nup);
      mo = max(mo, ndn);
      eu += (unsigned long long)nup;
      ed += (unsigned long long)ndn;
    }
    __syncthreads();
    if (STAGE) {
      // the tile's rows of direction d0 + j are nc * W consecutive ints of dnw; 32
      // threads write one direction's
      if (mine) {
        int4* out = reinterpret_cast<int4*>(a.dnw + (a.units[m * a.D + d].task_base + c0) * W);
        const int4* in = reinterpret_cast<const int4*>(srow + dj * kTileCells * W);
        for (int r = ci; r < nc * W / 4; r += kTileCells) out[r] = in[r];
      }
      // (the next rows are written behind the next barrier)
    }
  }
  atomicMax(&s_max[0], mi);
  atomicMax(&s_max[1], mo);
  atomicAdd(&s_ent[0], eu);
  atomicAdd(&s_ent[1], ed);
  __syncthreads();
  if (threadIdx.x < 2) {
    CountTotals& t = a.totals[blockIdx.x % kCountTotals];
    atomicMax(&t.longest[threadIdx.x], s_max[threadIdx.x]);
    atomicAdd(&t.entries[threadIdx.x], s_ent[threadIdx.x]);
  }
}

// Transport scheme (b) (direction-conserving transport, sec. 2.6), per task:
// the cell's outflow Aperp phi is shared equally by its n = min(n_aligned,
// outflow faces) outflow faces with the largest s (ties: the lower face
// index), each carrying w_b = Aperp / n.  Those faces get the signed weight
// +w_b, every other face NaN (nothing leaves through it); they are the task's
// only downwind edges (rows of at most n entries), and the boundary sums count
// only them.  Upwind counts depend on the neighbours' choices and are made by
// k_count_in once every choice is written.
__device__ __forceinline__ void top_insert(double (&bs)[kMaxAligned], int (&bf)[kMaxAligned],
                                           double v, int f) {
  // bs descending; an equal value already present stays first (lower face index)
  const double os[kMaxAligned] = {bs[0], bs[1], bs[2], bs[3]};
  const int of[kMaxAligned] = {bf[0], bf[1], bf[2], bf[3]};
#pragma unroll
  for (int k = 0; k < kMaxAligned; ++k) {
    const bool keep = os[k] >= v;
    const bool from_above = !keep && k > 0 && os[k > 0 ? k - 1 : 0] < v;
    bs[k] = keep ? os[k] : (from_above ? os[k > 0 ? k - 1 : 0] : v);
    bf[k] = keep ? of[k] : (from_above ? of[k > 0 ? k - 1 : 0] : f);
  }
}

__global__ __launch_bounds__(kCountThreads) void k_count_aligned(DagBuildArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int s_max;
  __shared__ unsigned long long s_ent;
  if (threadIdx.x == 0) {
    s_max = 0;
    s_ent = 0ull;
  }
  const int m = a.cblk_mesh[blockIdx.x];
  const MeshDev M = a.meshes[m];
  const FaceTile T = stage_tile(M, a.cblk_c0[blockIdx.x], smem);
  const int W = a.dn_width;
  __syncthreads();
  const int ci = threadIdx.x % kTileCells;
  const int dj = threadIdx.x / kTileCells;
  constexpr int kDirs = kCountThreads / kTileCells;
  const int c = T.c0 + ci;
  const bool cell = c < T.cend;
  const int fb = cell ? (int)T.fp[ci] : 0, fe = cell ? (int)T.fp[ci + 1] : 0;
  int mo = 0;
  unsigned long long ed = 0;
  auto run = [&](const double* nrm, const double* area, const int32_t* nbr, const int8_t* shift) {
    for (int d0 = 0; d0 < a.D; d0 += kDirs) {
      const int d = d0 + dj;
      if (!(cell && d < a.D)) continue;
      const double ox = a.dirs[3 * d], oy = a.dirs[3 * d + 1], oz = a.dirs[3 * d + 2];
      const int64_t t = a.units[m * a.D + d].task_base + c;
      float* wf = a.wface + (int64_t)a.D * M.face_off + (int64_t)d * M.n_faces + T.f0;
      double ap = 0.0;
      int nout = 0;
      double bs[kMaxAligned];
      int bf[kMaxAligned];
#pragma unroll
      for (int k = 0; k < kMaxAligned; ++k) {
        bs[k] = -__builtin_huge_val();
        bf[k] = -1;
      }
      for (int f = fb; f < fe; ++f) {
        const double sv = orient(ox, oy, oz, nrm + 3 * f);
        if (sv > a.eps) {
          ap += face_w(area[f], sv);
          ++nout;
          top_insert(bs, bf, sv, f);
        }
      }
      // (an undefined Aperp, which the sweep reports, leaves no shares to carry)
      const int n = isnan(ap) ? 0 : min(nout, a.n_aligned);
      const float wb = n > 0 ? (float)(ap / n) : 0.0f;
      int32_t* row = a.dnw + t * W;
      int ndn = 0;
      double wall = 0.0, per = 0.0;
      for (int f = fb; f < fe; ++f) {
        bool chosen = false;
#pragma unroll
        for (int k = 0; k < kMaxAligned; ++k) chosen |= k < n && bf[k] == f;
        wf[f] = chosen ? wb : __int_as_float(0x7fc00000);
        if (!chosen) continue;
        const int nb = nbr[f];
        if (nb < 0) wall += wb;
        else if (shift != nullptr && shift[f] != 0) {
          per += wb;
        } else {
          row[ndn++] = nb;
        }
      }
      for (int q = ndn; q < W; ++q) row[q] = -1;
      a.aperp[t] = (float)ap;
      a.bnd[t] = make_float2((float)wall, (float)per);
      a.rowlen_dn[t] = ndn;
      mo = max(mo, ndn);
      ed += (unsigned long long)ndn;
    }
  };
  if (T.in_lds) {
    constexpr int cap = kTileCells * kTileFaces;
    const double* nrm = reinterpret_cast<const double*>(T.fp + kTileCells + 1);
    const double* area = nrm + 3 * cap;
    const int32_t* nbr = reinterpret_cast<const int32_t*>(area + cap);
    const int8_t* shift = reinterpret_cast<const int8_t*>(nbr + cap);
    run(nrm, area, nbr, shift);
  } else {
    run(M.face_normal + 3 * T.f0, M.face_area + T.f0, M.face_nbr + T.f0,
        M.face_shift != nullptr ? M.face_shift + T.f0 : nullptr);
  }
  atomicMax(&s_max, mo);
  atomicAdd(&s_ent, ed);
  __syncthreads();
  if (threadIdx.x == 0) {
    CountTotals& t = a.totals[blockIdx.x % kCountTotals];
    atomicMax(&t.longest[1], s_max);
    atomicAdd(&t.entries[1], s_ent);
  }
}

// Scheme (b), per task: the upwind dependencies are the faces whose twin the
// neighbour chose (its signed weight is not NaN); counts, row lengths and the
// tasks with 15 or more dependencies, as k_count does for scheme (a).
__global__ __launch_bounds__(kCountThreads) void k_count_in(DagBuildArgs a) {
  __shared__ int s_max;
  __shared__ unsigned long long s_ent;
  if (threadIdx.x == 0) {
    s_max = 0;
    s_ent = 0ull;
  }
  __syncthreads();
  const int m = a.cblk_mesh[blockIdx.x];
  const MeshDev M = a.meshes[m];
  const int ci = threadIdx.x % kTileCells;
  const int dj = threadIdx.x / kTileCells;
  constexpr int kDirs = kCountThreads / kTileCells;
  const int c = a.cblk_c0[blockIdx.x] + ci;
  int mi = 0;
  unsigned long long eu = 0;
  if (c < M.n_cells) {
    const int64_t fb = M.face_ptr[c], fe = M.face_ptr[c + 1];
    for (int d = dj; d < a.D; d += kDirs) {
      const float* wf = a.wface + (int64_t)a.D * M.face_off + (int64_t)d * M.n_faces;
      int nup = 0;
      for (int64_t f = fb; f < fe; ++f) {
        if (M.face_nbr[f] < 0) continue;
        if (isnan(wf[M.face_twin[f]])) continue;
        if (M.face_shift == nullptr || M.face_shift[f] == 0) ++nup;
      }
      const int64_t t = a.units[m * a.D + d].task_base + c;
      if (nup >= a.big_min && a.big != nullptr) a.big[atomicAdd(a.big_top, 1)] = t;  // count too large for its place
      a.indeg[t] = nup;
      mi = max(mi, nup);
      eu += (unsigned long long)nup;
    }
  }
  atomicMax(&s_max, mi);
  atomicAdd(&s_ent, eu);
  __syncthreads();
  if (threadIdx.x == 0) {
    CountTotals& t = a.totals[blockIdx.x % kCountTotals];
    atomicMax(&t.longest[0], s_max);
    atomicAdd(&t.entries[0], s_ent);
  }
}

// Tasks with more upwind dependencies than their counter's place holds (15 with 4-bit
// fields) keep it in global memory; the entries that point at them in their upwind cells' downwind rows
// get bit 30 set, so that Kahn's algorithm sends those decrements there without
// first reading the LDS counter.  One wavefront per such task, one face per lane.
constexpr int32_t kBigFlag = 0x40000000;

__global__ __launch_bounds__(256) void k_mark(DagBuildArgs a, int32_t n_big) {
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= n_big) return;
  const int64_t t = a.big[i];
  int lo = 0, hi = a.n_units - 1;  // unit of task t (task bases ascend)
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (a.units[mid].task_base <= t) lo = mid; else hi = mid - 1;
  }
  const Unit U = a.units[lo];
  const int c = (int)(t - U.task_base);
  const MeshDev M = a.meshes[U.mesh];
  const double ox = a.dirs[3 * U.dir], oy = a.dirs[3 * U.dir + 1], oz = a.dirs[3 * U.dir + 2];
  const int W = a.dn_width;
  const float* wf = a.wface + (int64_t)a.D * M.face_off + (int64_t)U.dir * M.n_faces;
  for (int64_t f = M.face_ptr[c] + (threadIdx.x & 63); f < M.face_ptr[c + 1]; f += 64) {
    const int nb = M.face_nbr[f];
    if (nb < 0 || (M.face_shift != nullptr && M.face_shift[f] != 0)) continue;
    const bool upwind = a.scheme == SWEEP_SCHEME_ALIGNED ? !isnan(wf[M.face_twin[f]])
                                                         : orient(ox, oy, oz, M.face_normal + 3 * f) < -a.eps;
    if (!upwind) continue;
    // nb is upwind of c: flag c in nb's row (or in its overflow list)
    int32_t* row = a.dnw + (U.task_base + nb) * W;
    for (int q = 0; q < W; q += 4) {
      const int4 e = *reinterpret_cast<const int4*>(row + q);
      if (e.x == c) row[q] = c | kBigFlag;
      if (e.y == c) row[q + 1] = c | kBigFlag;
      if (e.z == c) row[q + 2] = c | kBigFlag;
      if (e.w == c) row[q + 3] = c | kBigFlag;
      if (q == W - 4 && e.w < -1) {
        int32_t* ov = a.dn_ovf + (-(e.w + 2));
        for (int r = 1; r <= ov[0]; ++r)
          if (ov[r] == c) ov[r] = c | kBigFlag;
      }
    }
  }
}

constexpr int kFrontierCap = 2048;  // frontier entries kept in LDS per level

// Where Kahn's counters live (k_kahn).
enum KahnMode { kKahnLds4 = 0, kKahnLds8 = 1, kKahnGlobal = 2, kKahnHash = 3, kKahnHashBig = 4 };

// The hash table of counters: a bucket is two words, four tag bytes and four
// counts.  Cell c belongs to one bucket, and its tag c / buckets + 1 (0: free way)
// tells it from the others there: consecutive cells (neighbours on the
// space-filling curve) lie in different buckets.  A free way's count is kHashBias.
constexpr int kHashBits = 14;  // at most 2^14 buckets (128 KB)
constexpr uint32_t kHashBias = 128;
static_assert(kHashMaxDeps < (int)kHashBias - 4, "counts stay above 0 while they count down from the bias");
constexpr int kMissCap = 2048;  // a level's decrements that did not find their cell, listed in LDS

using lds_int = int __attribute__((address_space(3)));

// First byte of w that is 0, as its bit offset (0, 8, 16, 24); -1 if there is none.
// (The bytes above a zero byte may be marked wrongly, the lowest mark is exact.)
__device__ __forceinline__ int zero_byte(uint32_t w) {
  const uint32_t t = (w - 0x01010101u) & ~w & 0x80808080u;
  return t != 0u ? (__ffs((int)t) - 1) & 24 : -1;
}

// Kahn's algorithm for one (mesh, direction) unit per workgroup: tasks without
// upwind dependencies form level 0; solving a level decrements the counters of
// its tasks' downwind cells and those reaching zero form the next level.  The
// schedule lists every level's cells in the order they were appended (slots
// [lp[l], lp[l+1]) hold level l); k_sort_levels brings it into canonical order.
//
// Each lane takes four entries of a downwind row (the lanes of a row read it with
// one line request, and a level of a few hundred tasks keeps every wavefront
// busy); ready cells are compacted with ballots and one LDS atomic per wavefront.
// The last wavefront makes every global store of the level loop (the schedule and
// the level pointers) and never waits for a load, so the others' waits for row
// loads never include a store.
//
// Counters:
//  kKahnLds8    bytes in LDS, when the largest mesh fits (and no task has more than
//               254 dependencies).
//  kKahnLds4    4-bit fields in LDS, when those fit; the value 15 marks a cell whose
//               count (>= 15) is kept in global memory instead (it is never changed,
//               so reading the field to pick the counter is race-free; the entries that
//               point at such cells are flagged beforehand, k_mark).  A decrement in
//               global memory costs its level a round trip, which on meshes of a few
//               thousand cells was most of the level.
//  kKahnHash    larger meshes: only cells between their first and last decrement need
//               a counter on chip (about 20,000 of 2M clustered cells at a time).  They
//               live in an LDS hash table.  A level's decrements that find their cell
//               in the table are made at once; the others are listed and, after a
//               barrier, made by full wavefronts: the first of a cell inserts it and
//               loads its remaining count (a byte in global memory).  A ready cell is
//               removed while the next level's rows are loaded, so that while cells
//               are inserted full buckets stay full and every lane of a cell comes to
//               the same decision.  A cell whose bucket is full is decremented in
//               global memory, where a later insertion finds its remaining count.
//  kKahnHashBig the same for meshes with a few cells of more dependencies than the
//               table's counts hold (kHashMaxDeps): their entries are flagged beforehand
//               (k_mark), and they are always counted in global memory.
//  kKahnGlobal  bytes in global memory, four to a word: meshes too large for the
//               table's keys, and few graphs at a time (the rule stands where the host
//               chooses).
//
// What bounds it: narrow levels, the chain from a level's barrier to the next (the
// rows come from HBM); wider ones, the instructions of 16 wavefronts (about 90 per
// row's lane and batch).  Per launch, against one lane per row of 16 entries and
// counters of larger meshes decremented in global memory (1.1 G atomics there at 2M
// cells): 4,096 cells x 8 directions 0.63 -> 0.21 ms, 64^3 jittered cells x 84
// directions 4.0 -> 2.3 ms, 2M clustered cells x 84 directions 69 -> 41 ms (43 with a few
// cells of more than 123 dependencies).  Loading a word of each newly ready cell's row at
// once, so that the next level finds it in L2, made it 7 to 9 % slower.
template <int MODE>
__global__ __launch_bounds__(1024) void k_kahn(DagBuildArgs a) {
  constexpr bool HASH = MODE == kKahnHash || MODE == kKahnHashBig;
  extern __shared__ __align__(16) uint32_t tab[];  // counters or hash table
  constexpr bool LDS = MODE == kKahnLds4 || MODE == kKahnLds8;
  constexpr int B = MODE == kKahnLds4 ? 4 : 8;  // bits of a counter in LDS, 32 / B to a word
  constexpr int PW = 32 / B;
  constexpr int LPW = MODE == kKahnLds4 ? 3 : 2;
  constexpr uint32_t M = (1u << B) - 1u;
  __shared__ int fr[2][kFrontierCap + 64];  // and 64 dummy words
  __shared__ int s_cnt[3];
  __shared__ int misses[HASH ? kMissCap + 64 : 1];
  __shared__ int s_nmiss[2];
  const Unit U = a.units[blockIdx.x];
  const int C = U.n_cells;
  const int64_t tb = U.task_base;
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int lane = tid & 63;
  const int wfirst = __builtin_amdgcn_readfirstlane(tid & ~63);  // the wavefront's first thread
  int32_t* cnt = a.cnt + tb;
  // counters in global memory: one byte per cell, four to a word, so that the
  // counters of a whole unit (C bytes) stay in the last-level caches
  uint8_t* cnt8 = reinterpret_cast<uint8_t*>(cnt);
  uint32_t* cntw = reinterpret_cast<uint32_t*>(cnt);
  int32_t* sched = a.sched + tb;
  int32_t* spill = sched;  // frontier entries beyond the LDS copy (rewritten in place)
  int32_t* lp = a.lp + U.lp_base;
  const int W = a.dn_width;          // 4, 8, 16 or 32
  const int sh = 31 - __clz(W >> 2); // lanes per row: 1 << sh
  if (tid < 3) s_cnt[tid] = 0;
  if (tid < 2) s_nmiss[tid] = 0;
  const int nwords = (C + PW - 1) / PW;  // counter words; 64 dummy words follow
  const int hbits = a.hash_bits;
  if (LDS) {
    if (tid < 64) tab[nwords + tid] = 0u;
    for (int wi = tid; wi < nwords; wi += nthr) {
      int n[PW];
#pragma unroll
      for (int j = 0; j < PW; ++j) n[j] = a.indeg[tb + min(PW * wi + j, C - 1)];
      uint32_t v = 0;
#pragma unroll
      for (int j = 0; j < PW; ++j) {
        const int c = PW * wi + j;
        if (c < C) {
          if (MODE == kKahnLds4 && n[j] >= 15) cnt[c] = n[j];
          v |= (uint32_t)min(n[j], (int)M) << (B * j);
        }
      }
      tab[wi] = v;
    }
  }
  if (HASH) {
    for (uint32_t i = tid; i < 2u << hbits; i += nthr) tab[i] = (i & 1u) ? kHashBias * 0x01010101u : 0u;
    if (tid < 64) tab[(2u << hbits) + tid] = 0u;  // dummy words
  }
  __syncthreads();
  // level 0: cells without upwind dependencies (global counters: the in-degrees
  // of kInitBatch cells per thread are loaded together, then stored as bytes)
  constexpr int kInitBatch = LDS ? 1 : 8;
  for (int c0 = 0; c0 < C; c0 += kInitBatch * nthr) {
    int n[kInitBatch];
    if (!LDS) {
#pragma unroll
      for (int j = 0; j < kInitBatch; ++j) {
        const int c = c0 + j * nthr + tid;
        n[j] = c < C ? a.indeg[tb + c] : -1;
      }
    }
#pragma unroll
    for (int j = 0; j < kInitBatch; ++j) {
      const int c = c0 + j * nthr + tid;
      bool ready = false;
      if (c < C) {
        if (LDS) {
          ready = ((tab[c >> LPW] >> (B * (c & (PW - 1)))) & M) == 0u;
        } else {
          cnt8[c] = (uint8_t)n[j];  // below 256 (the host checks the largest in-degree)
          ready = n[j] == 0;
        }
      }
      const unsigned long long m = __ballot(ready);
      if (m != 0ull) {
        const int leader = __ffsll((long long)m) - 1;
        int base = 0;
        if (lane == leader) base = atomicAdd(&s_cnt[0], __popcll(m));
        base = __shfl(base, leader);
        if (ready) {
          const int slot = base + __popcll(m & ((1ull << lane) - 1ull));
          if (slot < kFrontierCap) fr[0][slot] = c;
          else spill[slot] = c;
        }
      }
    }
  }
  __syncthreads();
  int head = 0;
  int tail = s_cnt[0];
  int l = 0;
  __syncthreads();
  if (tid == 0) {
    s_cnt[0] = 0;
    lp[0] = 0;
    lp[1] = tail;
  }
  __syncthreads();
  const int nwork = nthr - 64;
  const bool writer = wfirst >= nwork;
  const int4* rows = reinterpret_cast<const int4*>(a.dnw + tb * W);  // (at most 2^31 chunks: T < 2^31)

  // Decrement of a counter in global memory; true if the cell became ready.
  auto dec_global = [&](int nb) -> bool {
    if (MODE == kKahnLds4) {  // whole words (cells with 15 or more dependencies)
      const int old = __hip_atomic_fetch_add(cnt + nb, -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      return old == 1;
    }
    const uint32_t s8 = (uint32_t)(nb & 3) * 8u;
    const uint32_t old = __hip_atomic_fetch_add(cntw + (nb >> 2), 0u - (1u << s8), __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_WORKGROUP);
    return ((old >> s8) & 255u) == 1u;
  };
  // Hash table: a cell's bucket (index of its tag word) and tag.
  auto bucket_of = [&](int c) -> uint32_t {
    return 2u * (((uint32_t)c ^ __umul24((uint32_t)c >> hbits, 2897u)) & ((1u << hbits) - 1u));
  };
  auto tags_of = [&](int c) -> uint32_t {
    return __builtin_amdgcn_perm(0u, ((uint32_t)c >> hbits) + 1u, 0u);  // in all four bytes
  };
  // the remaining count past any cached copy (it may have been lowered in memory)
  auto remaining = [&](int c) -> uint32_t {
    const uint32_t w = __hip_atomic_load(cntw + (c >> 2), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return (w >> ((c & 3) * 8)) & 255u;
  };
  // One decrement of a cell that was not in the table (or may be by now); true if
  // the cell became ready.
  auto dec_new = [&](int c) -> bool {
    const uint32_t b = bucket_of(c), tg = tags_of(c);
    int at;
    bool fresh = false;
    for (;;) {  // (a lost race means that another lane filled a way: at most 4 times)
      const uint32_t w = __hip_atomic_load(&tab[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      at = zero_byte(w ^ tg);
      if (at >= 0) break;
      at = zero_byte(w);
      if (at < 0) break;
      if (atomicCAS(&tab[b], w, w | ((tg & 255u) << at)) == w) {
        fresh = true;
        break;
      }
    }
    if (at < 0) return dec_global(c);
    // a new cell counts down from the bias until its remaining count is known
    uint32_t by = 1u;
    if (fresh) by += kHashBias - remaining(c);
    const uint32_t old = atomicSub(&tab[b + 1], by << at);
    return ((old >> at) & 255u) == by;
  };
  auto remove = [&](int c) {
    const uint32_t b = bucket_of(c);
    const int at = zero_byte(tab[b] ^ tags_of(c));
    if (at < 0) return;
    atomicAnd(&tab[b], ~(255u << at));
    atomicAdd(&tab[b + 1], kHashBias << at);  // (a ready cell's count is 0)
  };
  auto dec_one = [&](int e) -> bool {  // one entry, any mode (overflow lists)
    const int nb = e & ~kBigFlag;
    if (LDS) {
      if ((e & kBigFlag) != 0) return dec_global(nb);
      const uint32_t sb = (uint32_t)(nb & (PW - 1)) * B;
      return ((atomicSub(&tab[nb >> LPW], 1u << sb) >> sb) & M) == 1u;
    }
    if (MODE == kKahnGlobal || (MODE == kKahnHashBig && (e & kBigFlag) != 0)) return dec_global(nb);
    return dec_new(nb);
  };

  // Level l: the frontier is [head, tail); its pushes count in s_cnt[l % 3].
  // s_cnt[(l + 1) % 3] was last read right after the barrier that ended level
  // l - 2, so it can be cleared now for level l + 1.
  while (head < tail) {
    if (tid == 0) {
      s_cnt[(l + 1) % 3] = 0;
      s_nmiss[(l + 1) & 1] = 0;
    }
    int* s_push = &s_cnt[l % 3];
    int* s_miss = &s_nmiss[l & 1];
    // (LDS pointers by type: mixed with the spill's pointer they became flat accesses)
    lds_int* const frc = (lds_int*)fr[l & 1];
    lds_int* const frn = (lds_int*)fr[(l + 1) & 1];
    const int dummy = kFrontierCap + lane;
    const int n = tail - head;
    const bool fr_lds = n <= kFrontierCap;  // the whole frontier is in LDS
    if (writer) {
      // the level's cells in slot order form the schedule (entries past the LDS
      // copy are in place already; each store is issued without waiting)
      const int ns = min(n, kFrontierCap);
      for (int i = lane; i < ns; i += 64) sched[head + i] = frc[i];
      if (lane == 0) lp[l + 1] = tail;
    }
    auto cell_at = [&](int kk) -> int {
      if (fr_lds) return frc[kk];
      int c;
      if (kk < kFrontierCap) {
        c = frc[kk];
      } else {
        c = spill[head + kk];
      }
      // no load of this path stays in flight: the common path's waits for the
      // loads of earlier levels are then counted exactly
      __builtin_amdgcn_s_waitcnt(0);
      return c;
    };
    // four entries of the row of frontier cell idx >> sh (none: -1)
    auto load = [&](int idx) -> int4 {
      if (idx >= n << sh) return make_int4(-1, -1, -1, -1);
      const int c = cell_at(idx >> sh);
      return rows[(uint32_t)((c << sh) | (idx & ((1 << sh) - 1)))];
    };
    // cells that became ready, appended to the next frontier: ballots and one LDS
    // atomic per wavefront
    auto push = [&](const bool (&ready)[4], const int (&xs)[4], auto n_c) {
      constexpr int N = decltype(n_c)::value;
      unsigned long long m[N];
      int total = 0;
#pragma unroll
      for (int i = 0; i < N; ++i) {
        m[i] = __ballot(ready[i]);
        total += __popcll(m[i]);
      }
      if (total == 0) return;
      int base = 0;
      if (lane == 0) base = atomicAdd(s_push, total);
      base = __builtin_amdgcn_readfirstlane(base);
      if (base + total <= kFrontierCap) {
        // (lanes without a ready cell write their dummy word: no branches)
#pragma unroll
        for (int i = 0; i < N; ++i) {
          frn[ready[i] ? base + rank_in(m[i]) : dummy] = xs[i] & ~kBigFlag;
          base += __popcll(m[i]);
        }
      } else {
#pragma unroll
        for (int i = 0; i < N; ++i) {
          const int q = base + rank_in(m[i]);
          if (ready[i] && q < kFrontierCap) frn[q] = xs[i] & ~kBigFlag;
          if (ready[i] && q >= kFrontierCap) spill[tail + q] = xs[i] & ~kBigFlag;
          base += __popcll(m[i]);
        }
      }
    };
    auto process = [&](const int4& v, bool last_chunk) {
      const int xs[4] = {v.x, v.y, v.z, v.w};
      bool ready[4];
      if (LDS) {
        // every entry issues one LDS decrement without a branch (padding: a zero from
        // the lane's private dummy word); flagged entries are decremented in global
        // memory instead
        uint32_t old[4];
        const bool big = max(max(v.x, v.y), max(v.z, v.w)) >= kBigFlag;
        const bool any_big = MODE == kKahnLds4 && __ballot(big) != 0ull;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int e = xs[i];
          const bool lds = e >= 0 && !(any_big && e >= kBigFlag);
          old[i] = atomicSub(&tab[lds ? e >> LPW : nwords + lane], lds ? 1u << ((e * B) & 31) : 0u);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) ready[i] = ((old[i] >> ((xs[i] * B) & 31)) & M) == 1u;  // (padding: 0)
        if (any_big) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (xs[i] >= kBigFlag) ready[i] = dec_global(xs[i] & ~kBigFlag);
        }
      } else if (MODE == kKahnGlobal) {
        uint32_t old[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t s8 = (uint32_t)(xs[i] & 3) * 8u;
          old[i] = xs[i] >= 0 ? __hip_atomic_fetch_add(cntw + (xs[i] >> 2), 0u - (1u << s8), __ATOMIC_RELAXED,
                                                       __HIP_MEMORY_SCOPE_WORKGROUP)
                              : 0u;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
          ready[i] = xs[i] >= 0 && ((old[i] >> ((uint32_t)(xs[i] & 3) * 8u)) & 255u) == 1u;
      } else {
        // entries in the table are decremented, the others listed (flagged ones: at once)
        int x[4];
        bool any_big = false;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const bool big = MODE == kKahnHashBig && xs[i] >= kBigFlag;
          x[i] = big ? -1 : xs[i];
          any_big |= big;
        }
        uint32_t bk[4];
        uint2 w[4];
        int at[4];
        bool miss[4];
        uint32_t old[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          bk[i] = bucket_of(max(x[i], 0));
          w[i] = *reinterpret_cast<const uint2*>(tab + bk[i]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          at[i] = zero_byte(w[i].x ^ tags_of(max(x[i], 0)));
          const bool hit = x[i] >= 0 && at[i] >= 0;
          miss[i] = x[i] >= 0 && at[i] < 0;
          // (lanes without a hit: their own dummy word; one address would serialise them)
          old[i] = atomicSub(&tab[hit ? bk[i] + 1 : (2u << hbits) + lane], hit ? 1u << (at[i] & 31) : 0u);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) ready[i] = ((old[i] >> (at[i] & 31)) & 255u) == 1u;  // (no hit: 0)
        if (MODE == kKahnHashBig && __ballot(any_big) != 0ull) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (xs[i] >= kBigFlag) ready[i] = dec_global(xs[i] & ~kBigFlag);
        }
        unsigned long long m[4];
        int total = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          m[i] = __ballot(miss[i]);
          total += __popcll(m[i]);
        }
        if (total > 0) {
          int base = 0;
          if (lane == 0) base = atomicAdd(s_miss, total);
          base = __builtin_amdgcn_readfirstlane(base);
          const bool fits = base + total <= kMissCap;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int q = base + rank_in(m[i]);
            misses[miss[i] && q < kMissCap ? q : kMissCap + lane] = x[i];
            base += __popcll(m[i]);
          }
          if (!fits) {  // past the list: at once
            base -= total;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              if (miss[i] && base + rank_in(m[i]) >= kMissCap) ready[i] = dec_new(x[i]);
              base += __popcll(m[i]);
            }
          }
        }
      }
      // a full row may end in a pointer to its overflow list (rare): one
      // wavefront push per extra entry
      const int ptr = last_chunk ? v.w : -1;
      if (__ballot(ptr < -1) != 0ull) {
        const int o = ptr < -1 ? -(ptr + 2) : 0;
        const int no = ptr < -1 ? a.dn_ovf[o] : 0;
        int mx = no;
#pragma unroll
        for (int s = 1; s < 64; s <<= 1) mx = max(mx, __shfl_xor(mx, s));
        for (int i = 0; i < mx; ++i) {
          const int e = i < no ? a.dn_ovf[o + 1 + i] : -1;
          const int one[4] = {e, -1, -1, -1};
          const bool rdy[4] = {e >= 0 && dec_one(e), false, false, false};
          push(rdy, one, std::integral_constant<int, 1>{});
        }
      }
      push(ready, xs, std::integral_constant<int, 4>{});
    };
    // two rows' worth of lanes in flight at a time
    constexpr int kBatch = 2;
    const int lanes = n << sh;
    int4 v[kBatch];
    if (!writer) {
#pragma unroll
      for (int b = 0; b < kBatch; ++b) v[b] = load(tid + b * nwork);
    }
    if (HASH) {
      // the frontier's cells leave the table (while the rows arrive)
      if (!writer)
        for (int i = tid; i < n; i += nwork) remove(cell_at(i));
      __syncthreads();
    }
    if (!writer) {
      const bool lc = (tid & ((1 << sh) - 1)) == (1 << sh) - 1;  // (nwork is a multiple of the lanes per row)
      for (int i0 = 0; i0 < lanes; i0 += kBatch * nwork) {
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
          // a wavefront without a row in this batch has nothing to do
          if (i0 + b * nwork + wfirst < lanes) process(v[b], lc);
        }
        if (i0 + kBatch * nwork < lanes) {
#pragma unroll
          for (int b = 0; b < kBatch; ++b) v[b] = load(i0 + (kBatch + b) * nwork + tid);
        }
      }
    }
    __syncthreads();
    if (HASH) {
      const int nm = min(*s_miss, kMissCap);
      if (!writer)
        for (int i = tid, iw = wfirst; iw < nm; i += nwork, iw += nwork) {  // (whole wavefronts)
          const int e = i < nm ? misses[i] : -1;
          const int one[4] = {e, -1, -1, -1};
          const bool rdy[4] = {e >= 0 && dec_new(e), false, false, false};
          push(rdy, one, std::integral_constant<int, 1>{});
        }
      __syncthreads();
    }
    head = tail;
    tail += s_cnt[l % 3];
    ++l;
  }
  if (tid == 0) lp[l + 1] = tail;
  if (tid == 0) {
    a.depth[blockIdx.x] = l;
    if (tail != C) atomicOr(a.err, 1);
  }
}

// Every level's cells in ascending cell id (the canonical order, so the
// schedule no longer depends on the order Kahn's wavefronts appended them),
// and the inverse schedule.  Consecutive tasks of a level then lie close in the
// spatially numbered cells, so the per-task gathers and the cell-order result
// stores of the later kernels share cache lines.  Workgroup b of a unit takes the
// unit's levels b, b + kSortPerUnit, ...
//
// Levels of up to kSortWave cells: a wavefront each, which counts for every cell the
// smaller ones (LDS broadcasts of four, no barrier).  Wider levels: by the
// workgroup in LDS (bitonic, padded to a power of two, a barrier per step); a
// level wider than kSortCap keeps its order.  64^3 cells x 84 directions (levels of
// about 230, up to 500): 641 us, and 708 with the bitonic sort alone; 50 K cells x 48 directions
// (57): 47 and 257; 4096 cells x 8 directions (18): 6.7 and 43.
constexpr int kSortBlock = 256;
constexpr int kSortPerUnit = 16;  // workgroups per unit
constexpr int kSortWave = 256;
static_assert(kSortBlock / 64 * kSortWave <= kSortCap, "the wavefronts' cells share the keys' LDS");

__global__ __launch_bounds__(kSortBlock) void k_sort_levels(DagBuildArgs a) {
  __shared__ __align__(16) int key[kSortCap];
  __shared__ int s_wide;
  const int u = blockIdx.x / kSortPerUnit;
  const Unit U = a.units[u];
  const int depth = a.depth[u];
  int32_t* sched = a.sched + U.task_base;
  int32_t* inv = a.inv + U.task_base;
  const int32_t* lp = a.lp + U.lp_base;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (threadIdx.x == 0) s_wide = 0;
  __syncthreads();
  int* const mine = key + wave * kSortWave;
  for (int l = blockIdx.x % kSortPerUnit + wave * kSortPerUnit; l < depth; l += kSortPerUnit * (kSortBlock / 64)) {
    const int k0 = lp[l], n = lp[l + 1] - k0;
    if (n > kSortWave) {
      if (lane == 0) atomicOr(&s_wide, 1);
      continue;
    }
    auto sort = [&](auto k_c) {
      constexpr int K = decltype(k_c)::value;  // cells per lane
      int x[K], rank[K];
#pragma unroll
      for (int q = 0; q < K; ++q) {
        const int i = 64 * q + lane;
        mine[i] = x[q] = i < n ? sched[k0 + i] : INT_MAX;
        rank[q] = 0;
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // the cells, to the wavefront's other lanes
      for (int i = 0; i < n; i += 4) {
        const int4 y = *reinterpret_cast<const int4*>(mine + i);
#pragma unroll
        for (int q = 0; q < K; ++q)
          rank[q] += (y.x < x[q] ? 1 : 0) + (y.y < x[q] ? 1 : 0) + (y.z < x[q] ? 1 : 0) + (y.w < x[q] ? 1 : 0);
      }
#pragma unroll
      for (int q = 0; q < K; ++q)
        if (64 * q + lane < n) {
          sched[k0 + rank[q]] = x[q];
          inv[x[q]] = k0 + rank[q];
        }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // read before the next level's
    };
    if (n <= 64) sort(std::integral_constant<int, 1>{});
    else if (n <= 128) sort(std::integral_constant<int, 2>{});
    else sort(std::integral_constant<int, 4>{});
  }
  __syncthreads();
  if (s_wide == 0) return;
  for (int l = blockIdx.x % kSortPerUnit; l < depth; l += kSortPerUnit) {
    const int k0 = lp[l], n = lp[l + 1] - k0;
    if (n <= kSortWave) continue;
    if (n > kSortCap) {
      for (int i = threadIdx.x; i < n; i += kSortBlock) inv[sched[k0 + i]] = k0 + i;
      continue;
    }
    int P = 2;
    while (P < n) P <<= 1;
    for (int i = threadIdx.x; i < P; i += kSortBlock) key[i] = i < n ? sched[k0 + i] : INT_MAX;
    __syncthreads();
    for (int size = 2; size <= P; size <<= 1)
      for (int stride = size >> 1; stride > 0; stride >>= 1) {
        for (int i = threadIdx.x; i < P / 2; i += kSortBlock) {
          const int lo = 2 * i - (i & (stride - 1));  // pair (lo, lo + stride)
          const int hi = lo + stride;
          const bool up = (lo & size) == 0;
          const int x = key[lo], y = key[hi];
          if ((x > y) == up) {
            key[lo] = y;
            key[hi] = x;
          }
        }
        __syncthreads();
      }
    for (int i = threadIdx.x; i < n; i += kSortBlock) {
      const int c = key[i];
      sched[k0 + i] = c;
      inv[c] = k0 + i;
    }
    __syncthreads();  // the next level reuses the keys
  }
}

// Per mesh: the largest face count of a cell, and the overflow room the wide
// rows need ((faces + 2) ints per direction for every cell with more than
// row_cap faces), accumulated into out[0] (max) and out[1] (sum).
__global__ __launch_bounds__(256) void k_face_stats(const int64_t* face_ptr, int n_cells, int row_cap, int n_dirs,
                             unsigned long long* out) {
  unsigned long long mx = 0, sum = 0;
  for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < n_cells; c += gridDim.x * blockDim.x) {
    const unsigned long long nf = (unsigned long long)(face_ptr[c + 1] - face_ptr[c]);
    mx = nf > mx ? nf : mx;
    if (nf > (unsigned long long)row_cap) sum += (nf + 2) * (unsigned long long)n_dirs;
  }
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned long long m2 = __shfl_xor(mx, o);
    mx = m2 > mx ? m2 : mx;
    sum += __shfl_xor(sum, o);
  }
  // one atomic pair per block: same-address atomics from every wave serialise
  __shared__ unsigned long long part[2][4];
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    part[0][w] = mx;
    part[1][w] = sum;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < (int)(blockDim.x >> 6); ++i) {
      mx = part[0][i] > mx ? part[0][i] : mx;
      sum += part[1][i];
    }
    atomicMax(out, mx);
    atomicAdd(out + 1, sum);
  }
}

// The mesh check: every condition the host's check of a mesh reports (api.cpp),
// face_twin and face_shift when given; *bad is set if one may be violated (the host then
// looks for the first and words the message).  16 lanes per cell, one face each;
// nothing is read through an index before it has been found in range.  Bound by
// memory, the twins' gathers above all: 64^3 cells 0.14 ms, 2 M 1.09.  (With the mesh
// copied to the host and checked there, a build of 50 K cells took 13.7 ms; a build and a
// sweep take 2.2.)
__global__ __launch_bounds__(256) void k_check_mesh(MeshDev M, int32_t* bad) {
  const int c = blockIdx.x * 16 + (threadIdx.x >> 4);
  if (c >= M.n_cells) return;
  const int64_t F = M.n_faces;
  const int64_t a = M.face_ptr[c], b = M.face_ptr[c + 1];
  bool wrong = b < a || a < 0 || b > F || (c == 0 && a != 0) || (c == M.n_cells - 1 && b != F);
  const double V = M.cell_volume[c];
  wrong |= !(V > 0.0) || !isfinite(V);
  if (!wrong) {
    for (int64_t f = a + (threadIdx.x & 15); f < b; f += 16) {
      const int nb = M.face_nbr[f];
      const double A = M.face_area[f];
      const double x = M.face_normal[3 * f], y = M.face_normal[3 * f + 1], z = M.face_normal[3 * f + 2];
      const int sh = M.face_shift != nullptr ? M.face_shift[f] : 0;
      // (a little inside the host's 1e-9, which decides)
      wrong |= nb < -1 || nb >= M.n_cells || !(A >= 0.0) || !isfinite(A) ||
               !(fabs(sqrt(x * x + y * y + z * z) - 1.0) <= 0.9e-9) || (sh != 0 && nb < 0);
      if (wrong || nb < 0 || M.face_twin == nullptr) continue;
      const int64_t t = M.face_twin[f];
      // the twin lies among the neighbour's faces and points back at this one
      if (t < 0 || t >= F || t < M.face_ptr[nb] || t >= M.face_ptr[nb + 1]) {
        wrong = true;
        continue;
      }
      wrong |= M.face_twin[t] != f || M.face_nbr[t] != c || M.face_area[t] != A || M.face_normal[3 * t] != -x ||
               M.face_normal[3 * t + 1] != -y || M.face_normal[3 * t + 2] != -z ||
               (M.face_shift != nullptr && M.face_shift[t] != -sh);
    }
  }
  if (wrong) atomicOr(bad, 1);
}

// Per face: the neighbour code (>= 0: interior neighbour, -1: vacuum wall,
// -(nb + 2): periodic image of cell nb), which the row fill reads next to the
// face's signed weight instead of the FP64 geometry; per cell: whether one is
// negative.  16 lanes per cell.
__global__ __launch_bounds__(256) void k_face_codes(MeshDev M, int32_t* fcode, uint8_t* edge) {
  const int c = blockIdx.x * 16 + (threadIdx.x >> 4);
  bool e = false;
  if (c < M.n_cells) {
    for (int64_t f = M.face_ptr[c] + (threadIdx.x & 15); f < M.face_ptr[c + 1]; f += 16) {
      const int nb = M.face_nbr[f];
      const bool periodic = M.face_shift != nullptr && M.face_shift[f] != 0;
      fcode[f] = nb < 0 ? -1 : (periodic ? -(nb + 2) : nb);
      e |= nb < 0 || periodic;
    }
  }
  const unsigned long long any = __ballot(e);
  if (c < M.n_cells && (threadIdx.x & 15) == 0)
    edge[M.cell_off + c] = ((any >> (threadIdx.x & 48)) & 0xffffull) != 0ull ? 1 : 0;
}

// Unit of a slice.
__device__ __forceinline__ int unit_of_slice(const int64_t* slice_base, int n_units, int64_t i) {
  int lo = 0, hi = n_units - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (slice_base[mid] <= i) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Slices of the sweep: every level's tasks in ceil(w / 64) runs of consecutive
// schedule positions with (nearly) equal task counts.
__device__ __forceinline__ int level_slices(int w) { return (w + 63) >> 6; }

__global__ __launch_bounds__(256) void k_count_slices(DagBuildArgs a) {
  __shared__ int s_n;
  const Unit U = a.units[blockIdx.x];
  const int depth = a.depth[blockIdx.x];
  const int32_t* lp = a.lp + U.lp_base;
  if (threadIdx.x == 0) s_n = 0;
  __syncthreads();
  int n = 0;
  for (int l = threadIdx.x; l < depth; l += blockDim.x) n += level_slices(lp[l + 1] - lp[l]);
  for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o);
  if ((threadIdx.x & 63) == 0) atomicAdd(&s_n, n);
  __syncthreads();
  if (threadIdx.x == 0) a.n_unit_slices[blockIdx.x] = s_n;
}

// The slice tables of both walks (SliceRec but for the entries' place, which
// k_fill adds), one workgroup per unit: a scan over the levels gives each its
// first slice.  A chain of scans over 256 levels at a time: 23 us at 64^3 cells x 84
// directions (about 1,000 levels).
constexpr int kSlicesBlock = 256;
__global__ __launch_bounds__(kSlicesBlock) void k_slices(DagBuildArgs a) {
  __shared__ int s_scan[kSlicesBlock];
  __shared__ int s_carry;
  const Unit U = a.units[blockIdx.x];
  const int depth = a.depth[blockIdx.x];
  const int tid = threadIdx.x;
  const int32_t* lp = a.lp + U.lp_base;
  const int64_t base = a.slice_base[blockIdx.x];
  const int ns = (int)(a.slice_base[blockIdx.x + 1] - base);
  const int C = U.n_cells;
  if (tid == 0) s_carry = 0;
  __syncthreads();
  for (int l0 = 0; l0 < depth; l0 += kSlicesBlock) {
    const int l = l0 + tid;
    const int k0 = l < depth ? lp[l] : 0;
    const int w = l < depth ? lp[l + 1] - k0 : 0;
    const int n = level_slices(w);
    s_scan[tid] = n;
    __syncthreads();
    for (int o = 1; o < kSlicesBlock; o <<= 1) {  // inclusive scan over the block
      const int x = tid >= o ? s_scan[tid - o] : 0;
      __syncthreads();
      s_scan[tid] += x;
      __syncthreads();
    }
    const int off = s_carry + s_scan[tid] - n;
    for (int c = 0; c < n; ++c) {
      const int ka = k0 + (int)(((int64_t)c * w) / n), kb = k0 + (int)(((int64_t)(c + 1) * w) / n);
      SliceRec f{ka, kb - ka, off, k0 + w, k0, 0u, 0u, 0};
      SliceRec r{ka, kb - ka, ns - (off + n), C - k0, C - (k0 + w), 0u, 0u, 0};
      a.sl_up[base + off + c] = f;
      a.sl_dn[base + off + c] = r;
    }
    __syncthreads();
    if (tid == kSlicesBlock - 1) s_carry += s_scan[tid];
    __syncthreads();
  }
}

// Per task in schedule order: row lengths, Aperp and the cell's volume; per
// slice: its rows' entry pairs (the input of the scan that places them).  One
// wavefront per slice.  Bound by four gathers per task, a line request each: 64^3 cells
// x 84 directions 0.55 ms (22 M tasks), 2 M cells 4.8 ms.
__global__ __launch_bounds__(kCountBlock) void k_gather_tasks(DagBuildArgs a) {
  const int64_t i = (int64_t)xcd_block(blockIdx.x, gridDim.x) * (kCountBlock / 64) + (threadIdx.x >> 6);
  if (i >= a.n_slices) return;
  const int lane = threadIdx.x & 63;
  const Unit U = a.units[unit_of_slice(a.slice_base, a.n_units, i)];
  const int k0 = a.sl_up[i].k0, cnt = a.sl_up[i].cnt;
  int pu = 0, pd = 0;
  if (lane < cnt) {
    const int64_t t = U.task_base + k0 + lane;
    const int c = a.sched[t];
    const int nu = a.indeg[U.task_base + c], nd = a.rowlen_dn[U.task_base + c];
    a.len_up[t] = nu;
    a.len_dn[t] = nd;
    a.aperp_s[t] = a.aperp[U.task_base + c];
    a.vol_s[t] = (float)a.meshes[U.mesh].cell_volume[c];
    pu = (nu + 1) >> 1;
    pd = (nd + 1) >> 1;
  }
  for (int o = 32; o > 0; o >>= 1) {
    pu += __shfl_xor(pu, o);
    pd += __shfl_xor(pd, o);
  }
  if (lane == 0) {
    a.np_up[i] = pu;
    a.np_dn[i] = pd;
  }
}

// Row entries of the units for the check of their number (meshes with very many
// faces only), one workgroup per unit.
__global__ __launch_bounds__(256) void k_unit_entries(const Unit* units, const int32_t* len_up,
                                                      const int32_t* len_dn, unsigned long long* out) {
  const Unit U = units[blockIdx.x];
  unsigned long long u = 0, d = 0;
  for (int k = threadIdx.x; k < U.n_cells; k += blockDim.x) {
    u += (unsigned long long)len_up[U.task_base + k];
    d += (unsigned long long)len_dn[U.task_base + k];
  }
  for (int o = 32; o > 0; o >>= 1) {
    u += __shfl_xor(u, o);
    d += __shfl_xor(d, o);
  }
  if ((threadIdx.x & 63) == 0) {
    atomicAdd(out + 2 * blockIdx.x, u);
    atomicAdd(out + 2 * blockIdx.x + 1, d);
  }
}

// Rows of the upwind and downwind lists.  The rows of a slice (up to 64 tasks)
// lie together as entry pairs, column by column: pair j of the rows longer than
// 2 j, in task order, then pair j + 1 of those longer than 2 j + 2, and so on,
// so that a wavefront with one task per lane reads each column with one
// coalesced 128-bit load and no padding but the second half of an odd row's
// last pair (no entry).  An entry is (position code, w): 4 (p + 1), p the
// neighbour's position in the walk that reads the row (upwind rows: its
// schedule position; downwind rows, walked backwards: the unit's last position
// minus it), so 0 means no entry and the code with the low bits masked is the
// byte offset of a ring slot.  Rows keep the cell's face order.
//
// One wavefront per slice.  Every lane first loads one task (cell, row lengths,
// face range); then four lanes share one task, four faces per lane and 16 tasks
// at a time, and the wavefront assembles the rows of 32 tasks in LDS: entry e of
// the upwind row of task t at [e][t], entry e of its downwind row at [K - 1 - e][t]
// (slices with a cell of more faces than that holds: 16 tasks at a time).  Each
// face's neighbour code and signed weight (from k_count) give its class, a sum over
// the four lanes its entry number.  The columns are then read from LDS with one task
// and side per lane and stored in whole cache lines; entries stored one by one from
// where their face was looked at cost a line request each.
//
// Bound by the requests that the L1 keeps in flight: about 28 per task, of which 15
// find the neighbours' positions (2.2 TB/s).  64^3 cells, 84 directions: 2.18 ms, and
// 3.25 with 16 lanes per task and stores of single entries; 2 M cells: 20.6 ms, and
// 29.1.
constexpr int kFillBlock = 256;
constexpr int kFillTasks = 32;  // tasks assembled in LDS at a time
constexpr int kFillFaces = 96;  // entries per task in LDS at most

// Value of lane L of the lane's group of four.
template <int L>
__device__ __forceinline__ int quad_lane(int v) {
  return __builtin_amdgcn_update_dpp(0, v, L * 0x55, 0xf, 0xf, true);  // quad_perm [L, L, L, L]
}

template <bool ALIGNED>
__global__ __launch_bounds__(kFillBlock) __attribute__((amdgpu_waves_per_eu(5))) void k_fill(DagBuildArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int wv = threadIdx.x >> 6;
  const int lane = threadIdx.x & 63;
  const int room = a.fill_faces * (kFillTasks + 1);  // entries of a wavefront's LDS
  int2* const s_ent = reinterpret_cast<int2*>(smem) + wv * room;
  const int64_t sl = (int64_t)xcd_block(blockIdx.x, gridDim.x) * (kFillBlock / 64) + wv;
  if (sl >= a.n_slices) return;  // (wavefronts share nothing here: no barrier below)
  const Unit U = a.units[unit_of_slice(a.slice_base, a.n_units, sl)];
  const MeshDev M = a.meshes[U.mesh];
  const int64_t tb = U.task_base;
  const int C = U.n_cells;
  const int32_t* inv = a.inv + tb;
  const float* wf = a.wface + (int64_t)a.D * M.face_off + (int64_t)U.dir * M.n_faces;
  const int k0 = a.sl_up[sl].k0, cnt = a.sl_up[sl].cnt;
  const int64_t bu = a.pb_up[sl], bd = a.pb_dn[sl];
  const bool act = lane < cnt;
  const int c = act ? a.sched[tb + k0 + lane] : 0;
  const int nu = act ? a.len_up[tb + k0 + lane] : 0;
  const int nd = act ? a.len_dn[tb + k0 + lane] : 0;
  const int64_t f0 = M.face_ptr[c];
  const int nf = act ? (int)(M.face_ptr[c + 1] - f0) : 0;
  if (lane == 0) {
    SliceRec& ru = a.sl_up[sl];
    ru.base_lo = (uint32_t)bu;
    ru.base_hi = (uint32_t)((uint64_t)bu >> 32);
    ru.np = (int)(a.pb_up[sl + 1] - bu);
    SliceRec& rd = a.sl_dn[sl];
    rd.base_lo = (uint32_t)bd;
    rd.base_hi = (uint32_t)((uint64_t)bd >> 32);
    rd.np = (int)(a.pb_dn[sl + 1] - bd);
  }
  // class and weight of a face with neighbour code `code` (>= 0: an interior neighbour)
  // and signed weight ws
  auto classify = [&](int64_t f, bool has, int code, float ws, bool& up, bool& dn, float& w) {
    has = has && code >= 0;
    if (ALIGNED) {
      // radiation leaves through the faces the cell chose and enters through the
      // faces whose twin the neighbour chose
      const float wi = wf[has ? M.face_twin[f] : 0];
      up = has && !isnan(wi);
      dn = has && !isnan(ws);
      w = up ? wi : ws;
    } else {
      has = has && !isnan(ws);
      up = has && signbit(ws);   // interior inflow
      dn = has && !signbit(ws);  // interior outflow
      w = fabsf(ws);
    }
  };
  // faces f..f + 3, of which the first m are the cell's (what lies behind them is readable)
  auto faces = [&](int64_t f, int m, int (&code)[4], bool (&up)[4], bool (&dn)[4], float (&w)[4]) {
    struct __attribute__((packed, aligned(4))) Four {
      int x[4];
    };
    const Four c4 = *reinterpret_cast<const Four*>(M.fcode + f);
    const Four w4 = *reinterpret_cast<const Four*>(wf + f);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      code[k] = c4.x[k];
      classify(f + k, k < m, code[k], __int_as_float(w4.x[k]), up[k], dn[k], w[k]);
    }
  };
  // entry of a neighbour at schedule position p, upwind or downwind
  auto code_of = [&](bool up, int p) { return up ? 4 * p + 4 : 4 * C - 4 * p; };
  // tasks at a time, the stride of the entry numbers (odd: 16 lanes of one task fall on
  // 16 banks) and the entries per task
  const int tasks = __any(nf > a.fill_faces) ? kFillTasks / 2 : kFillTasks;
  const int stride = tasks + 1;
  const int K = tasks == kFillTasks ? a.fill_faces : room / stride;
  if (__any(nf > K)) {
    // each lane looks through its own task's faces, two entries per column
    for (int side = 0; side < 2; ++side) {
      const int n = side == 0 ? nu : nd;
      int4* out = side == 0 ? a.up + bu : a.dn + bd;
      int q = 0;
      for (int j = 0;; ++j) {
        const unsigned long long m = __ballot(n > 2 * j);
        if (m == 0ull) break;
        if (n > 2 * j) {
          int4 pair = make_int4(0, 0, 0, 0);
          for (int k = 0; q < nf && k < 2; ++q) {
            const int code = M.fcode[f0 + q];
            bool up, dn;
            float w;
            classify(f0 + q, true, code, wf[f0 + q], up, dn, w);
            if (!(side == 0 ? up : dn)) continue;
            const int at = code_of(up, inv[code]);
            if (k++ == 0) {
              pair.x = at;
              pair.y = __float_as_int(w);
            } else {
              pair.z = at;
              pair.w = __float_as_int(w);
            }
          }
          out[__popcll(m & ((1ull << lane) - 1ull))] = pair;
        }
        out += __popcll(m);
      }
    }
    return;
  }
  const int q = lane & 3;
  const int before[3] = {q > 0 ? -1 : 0, q > 1 ? -1 : 0, q > 2 ? -1 : 0};  // masks of the task's lanes below this one
  for (int t0 = 0; t0 < cnt; t0 += tasks) {
#pragma unroll 1
    for (int tl = lane >> 2; tl < tasks; tl += 16) {
      const int64_t fb = __shfl(f0, t0 + tl);
      const int nft = __shfl(nf, t0 + tl);
      int mx = nft;
      for (int o = 4; o < 64; o <<= 1) mx = max(mx, __shfl_xor(mx, o));
      mx = __builtin_amdgcn_readfirstlane(mx);
      int eu = tl, ed = (K - 1) * stride + tl;  // places of the rows' next entries
      for (int h = 0; h < mx; h += 16) {
        const int64_t f = fb + h + 4 * q;
        const int m = nft - h - 4 * q;  // faces of this lane
        int code[4], pos[4];
        bool up[4], dn[4];
        float w[4];
        int n = 0;  // upwind entries, downwind entries << 16
        if (m > 0) {
          faces(f, m, code, up, dn, w);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            pos[k] = inv[up[k] || dn[k] ? code[k] : 0];
            n += (up[k] ? 1 : 0) + (dn[k] ? 1 << 16 : 0);
          }
        }
        const int n0 = quad_lane<0>(n), n1 = quad_lane<1>(n), n2 = quad_lane<2>(n), n3 = quad_lane<3>(n);
        const int p = (n0 & before[0]) + (n1 & before[1]) + (n2 & before[2]);
        if (m > 0) {
          int xu = eu + stride * (p & 0xffff), xd = ed - stride * (p >> 16);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            if (up[k] || dn[k])
              s_ent[up[k] ? xu : xd] = make_int2(code_of(up[k], pos[k]), __float_as_int(w[k]));
            xu += up[k] ? stride : 0;
            xd -= dn[k] ? stride : 0;
          }
        }
        const int all = n0 + n1 + n2 + n3;
        eu += stride * (all & 0xffff);
        ed -= stride * (all >> 16);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // the entries, to the wavefront's other lanes
    // lanes 0..31: the upwind rows' columns, lanes 32..63: the downwind rows'
    const bool mine = (lane & 31) < tasks;
    const int t = mine ? t0 + (lane & 31) : 0;
    const bool dside = lane >= 32;
    const int xu = __shfl(nu, t), xd = __shfl(nd, t);
    const int n = mine ? (dside ? xd : xu) : 0;
    const unsigned long long low = (1ull << t) - 1ull;
    int4* out = dside ? a.dn + bd : a.up + bu;
    const int2* row = s_ent + (dside ? (K - 1) * stride : 0) + (lane & 31);
    const int step = dside ? -stride : stride;
    for (int j = 0;; ++j) {
      const unsigned long long mu = __ballot(nu > 2 * j), md = __ballot(nd > 2 * j);
      if ((mu | md) == 0ull) break;
      if (n > 2 * j) {
        const int2 x = row[2 * j * step];
        const bool odd = n == 2 * j + 1;
        const int2 y = row[(odd ? 2 * j : 2 * j + 1) * step];
        typedef int v4 __attribute__((ext_vector_type(4)));
        const v4 pair = {x.x, x.y, odd ? 0 : y.x, odd ? 0 : y.y};  // (no entry: 0 times it is 0)
        __builtin_nontemporal_store(pair, reinterpret_cast<v4*>(out) + __popcll((dside ? md : mu) & low));
      }
      out += dside ? __popcll(md) : __popcll(mu);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // read before the next tasks' entries
  }
}

// Periodic half-faces of every cell of mesh M (neighbour code -(nb + 2)).
__global__ void k_pcount(DagBuildArgs a, MeshDev M) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= M.n_cells) return;
  int n = 0;
  for (int64_t f = M.face_ptr[c]; f < M.face_ptr[c + 1]; ++f) n += M.fcode[f] < -1 ? 1 : 0;
  a.npf[M.cell_off + c] = n;
  a.pflag[M.cell_off + c] = n > 0 ? 1 : 0;
}

// The periodic cells of mesh M in cell order with their periodic half-faces in
// face order (the face and its partner).
__global__ void k_plist(DagBuildArgs a, MeshDev M) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= M.n_cells) return;
  const int gc = M.cell_off + c;
  const int64_t pc = a.pc_off[gc];
  const bool per = a.pc_off[gc + 1] > pc;
  a.pc_map[gc] = per ? (int)pc : -1;
  if (!per) return;
  a.pcell[pc] = gc;
  a.pf_ptr[pc] = (int32_t)a.pf_off[gc];
  int64_t j = a.pf_off[gc];
  for (int64_t f = M.face_ptr[c]; f < M.face_ptr[c + 1]; ++f) {
    const int code = M.fcode[f];
    if (code >= -1) continue;
    a.pface[j] = (int32_t)f;
    a.pnb[j] = M.cell_off + (-(code + 2));
    ++j;
  }
}

// Per (direction, periodic cell of mesh M): the inflow and outflow weight of
// each periodic half-face (the classes and weights k_fill gives the row
// entries, 0 where the half-face carries nothing that way) and the cell's task.
__global__ void k_pdir(DagBuildArgs a, MeshDev M, int mesh) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)a.D * a.n_pc) return;
  const int pc = (int)(i % a.n_pc);
  const int d = (int)(i / a.n_pc);
  const int c = a.pcell[pc] - M.cell_off;
  if (c < 0 || c >= M.n_cells) return;  // a cell of another mesh
  const float* wf = a.wface + (int64_t)a.D * M.face_off + (int64_t)d * M.n_faces;
  for (int j = a.pf_ptr[pc]; j < a.pf_ptr[pc + 1]; ++j) {
    const int f = a.pface[j];
    float fw, aw;
    if (a.scheme == SWEEP_SCHEME_ALIGNED) {
      // inflow: the neighbour's share through the twin; outflow: the cell's own
      const float wi = wf[M.face_twin[f]];
      const float ws = wf[f];
      fw = isnan(wi) ? 0.0f : wi;
      aw = isnan(ws) ? 0.0f : ws;
    } else {
      const float ws = wf[f];
      const bool has = !isnan(ws);
      const bool in = has && signbit(ws);
      fw = in ? fabsf(ws) : 0.0f;
      aw = has && !in ? fabsf(ws) : 0.0f;
    }
    a.pwf[(int64_t)d * a.n_pf + j] = fw;
    a.pwa[(int64_t)d * a.n_pf + j] = aw;
  }
  const Unit U = a.units[mesh * a.D + d];
  a.ptask[i] = (int32_t)(U.task_base + a.inv[U.task_base + c]);
}

// Tasks per level, one workgroup per unit.
__global__ void k_level_widths(const Unit* units, const int32_t* lp, int32_t mesh,
                               unsigned long long* width, int32_t n_levels) {
  const Unit U = units[blockIdx.x];
  if (mesh >= 0 && U.mesh != mesh) return;
  const int32_t* l = lp + U.lp_base;
  for (int k = threadIdx.x; k < min(U.depth, n_levels); k += blockDim.x)
    atomicAdd(width + k, (unsigned long long)(l[k + 1] - l[k]));
}

__global__ void k_d2f(const double* in, float* out, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = (float)in[i];
}

__global__ void k_fill_i32(int32_t* p, int64_t n, int32_t v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__global__ void k_fill_f32(float* p, int64_t n, float v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

inline unsigned grid1d(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

}  // namespace

hipError_t launch_count(const DagBuildArgs& a, int32_t n_cblocks, int32_t lds_limit, hipStream_t s) {
  if (n_cblocks <= 0) return hipSuccess;
  if (a.scheme == SWEEP_SCHEME_ALIGNED) {
    const size_t tile = tile_lds_bytes();
    hipError_t e = hipFuncSetAttribute((const void*)k_count_aligned,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)tile);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_count_aligned, dim3(n_cblocks), dim3(kCountThreads), tile, s, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    // upwind counts once every cell's choice is written
    hipLaunchKernelGGL(k_count_in, dim3(n_cblocks), dim3(kCountThreads), 0, s, a);
    return hipGetLastError();
  }
  const size_t tile = count_tile_bytes();
  const size_t staged = tile + (size_t)kTileThreads * a.dn_width * 4;
  const bool stage = staged <= (size_t)lds_limit - 64;
  const size_t lds = stage ? staged : tile;
  auto kernel = stage ? k_count<true> : k_count<false>;
  hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kernel, dim3(n_cblocks), dim3(kTileThreads), lds, s, a);
  return hipGetLastError();
}

hipError_t launch_kahn(const DagBuildArgs& a, int32_t lds_bits, int32_t max_cells, hipStream_t s) {
  auto launch = [&](auto kernel, size_t lds) {
    if (lds > 0) {
      const hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                               (int)lds);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kernel, dim3(a.n_units), dim3(1024), lds, s, a);
    return hipGetLastError();
  };
  if (lds_bits == 8) return launch(k_kahn<kKahnLds8>, kahn_lds_bytes(8, max_cells));
  if (lds_bits == 4) return launch(k_kahn<kKahnLds4>, kahn_lds_bytes(4, max_cells));
  if (a.hash_bits > 0) {
    const size_t lds = sizeof(uint32_t) * (((size_t)2 << a.hash_bits) + 64);
    return a.hash_big ? launch(k_kahn<kKahnHashBig>, lds) : launch(k_kahn<kKahnHash>, lds);
  }
  return launch(k_kahn<kKahnGlobal>, 0);
}

// log2 of k_kahn's hash buckets for meshes of up to max_cells cells: at least a bucket
// (four ways) per 128 cells, at most 2^kHashBits.  0: the table cannot hold them (tags of
// one byte).
int kahn_hash_bits(int32_t max_cells) {
  int bits = 3;
  while (bits < kHashBits && (max_cells >> bits) >= 128) ++bits;
  return (max_cells >> bits) < 254 ? bits : 0;
}

hipError_t launch_mark(const DagBuildArgs& a, int32_t n_big, hipStream_t s) {
  if (n_big <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_mark, dim3((n_big + 3) / 4), dim3(256), 0, s, a, n_big);
  return hipGetLastError();
}

hipError_t launch_sort_levels(const DagBuildArgs& a, hipStream_t s) {
  if (a.n_units <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_sort_levels, dim3(a.n_units * kSortPerUnit), dim3(kSortBlock), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_count_slices(const DagBuildArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_count_slices, dim3(a.n_units), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_slices(const DagBuildArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_slices, dim3(a.n_units), dim3(kSlicesBlock), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_gather_tasks(const DagBuildArgs& a, hipStream_t s) {
  if (a.n_slices <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_gather_tasks, dim3(grid1d(a.n_slices, kCountBlock / 64)), dim3(kCountBlock), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_fill(const DagBuildArgs& a, hipStream_t s) {
  if (a.n_slices <= 0) return hipSuccess;
  const dim3 grid(grid1d(a.n_slices, kFillBlock / 64));
  const size_t lds = kFillBlock / 64 * sizeof(int2) * (size_t)a.fill_faces * (kFillTasks + 1);
  auto kernel = a.scheme == SWEEP_SCHEME_ALIGNED ? k_fill<true> : k_fill<false>;
  const hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kernel, grid, dim3(kFillBlock), lds, s, a);
  return hipGetLastError();
}

// Entries per task that k_fill holds in LDS (one per face) for meshes of mean_faces faces
// per cell on average and max_faces at most.
int fill_faces(double mean_faces, int64_t max_faces) {
  return (int)std::max(1.0, std::min({std::ceil(1.9 * mean_faces), (double)max_faces, (double)kFillFaces}));
}

hipError_t launch_pcount(const DagBuildArgs& a, const MeshDev& m, hipStream_t s) {
  if (m.n_cells <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_pcount, dim3(grid1d(m.n_cells, 256)), dim3(256), 0, s, a, m);
  return hipGetLastError();
}

hipError_t launch_plist(const DagBuildArgs& a, const MeshDev& m, hipStream_t s) {
  if (m.n_cells <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_plist, dim3(grid1d(m.n_cells, 256)), dim3(256), 0, s, a, m);
  return hipGetLastError();
}

hipError_t launch_pdir(const DagBuildArgs& a, const MeshDev& m, int32_t mesh, hipStream_t s) {
  const int64_t n = (int64_t)a.D * a.n_pc;
  if (m.n_cells <= 0 || n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_pdir, dim3(grid1d(n, 256)), dim3(256), 0, s, a, m, mesh);
  return hipGetLastError();
}

hipError_t launch_face_stats(const int64_t* face_ptr, int32_t n_cells, int32_t row_cap, int32_t n_dirs,
                             unsigned long long* out, hipStream_t s) {
  if (n_cells <= 0) return hipSuccess;
  const unsigned grid = (unsigned)std::min<int64_t>(256, grid1d(n_cells, 256));
  hipLaunchKernelGGL(k_face_stats, dim3(grid), dim3(256), 0, s, face_ptr, n_cells, row_cap, n_dirs, out);
  return hipGetLastError();
}

hipError_t launch_check_mesh(const MeshDev& m, int32_t* bad, hipStream_t s) {
  hipLaunchKernelGGL(k_check_mesh, dim3(grid1d(m.n_cells, 16)), dim3(256), 0, s, m, bad);
  return hipGetLastError();
}

hipError_t launch_face_codes(const MeshDev& m, int32_t* fcode, uint8_t* edge, hipStream_t s) {
  if (m.n_cells <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_face_codes, dim3(grid1d(m.n_cells, 16)), dim3(256), 0, s, m, fcode, edge);
  return hipGetLastError();
}

struct WidenToI64 {
  __host__ __device__ int64_t operator()(int32_t v) const { return (int64_t)v; }
};

hipError_t launch_scan_len(const int32_t* in, int64_t* out, int64_t n, void* tmp, size_t* tmp_bytes,
                           hipStream_t s) {
  // exclusive prefix sum of int32 row lengths into int64 row pointers (the
  // lengths are widened as they are read, so the sums never overflow);
  // tmp == nullptr queries the temporary storage size
  hipcub::TransformInputIterator<int64_t, WidenToI64, const int32_t*> it(in, WidenToI64());
  return hipcub::DeviceScan::ExclusiveSum(tmp, *tmp_bytes, it, out, (int)n, s);
}

hipError_t launch_unit_entries(const Unit* units, int32_t n_units, const int32_t* len_up,
                               const int32_t* len_dn, int64_t* out, hipStream_t s) {
  if (n_units <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_unit_entries, dim3(n_units), dim3(256), 0, s, units, len_up, len_dn,
                     reinterpret_cast<unsigned long long*>(out));
  return hipGetLastError();
}

hipError_t launch_level_widths(const Unit* units, int32_t n_units, const int32_t* lp, int32_t mesh,
                               int64_t* width, int32_t n_levels, hipStream_t s) {
  if (n_units <= 0 || n_levels <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_level_widths, dim3(n_units), dim3(256), 0, s, units, lp, mesh,
                     reinterpret_cast<unsigned long long*>(width), n_levels);
  return hipGetLastError();
}

hipError_t launch_d2f(const double* in, float* out, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_d2f, dim3(grid1d(n, 256)), dim3(256), 0, s, in, out, n);
  return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t* p, int64_t n, int32_t v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_i32, dim3(grid1d(n, 256)), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

hipError_t launch_fill_f32(float* p, int64_t n, float v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_f32, dim3(grid1d(n, 256)), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

}  // namespace sweep
