// Forward and adjoint sweep kernels and the per-cell reductions (gfx950).
//
// Schedule: one workgroup owns one (mesh, direction) sweep at a time and works
// through its levels in order (reverse order for the adjoint).  The tasks of a
// level are independent (their upwind tasks sit on earlier levels), so the
// workgroup's wavefronts solve them in parallel, ordered by counters in LDS instead
// of barriers; every task pulls its inflow from its upwind tasks' results in a fixed
// row order, so results do not depend on which lane runs which task.  Persistent
// form: a grid sized to the resident capacity takes (mesh, direction) units from an
// atomic counter, longest first.
//
// LDS ring: the results of the last `ring` tasks of the schedule are kept in LDS,
// indexed by schedule position modulo `ring`, so most upwind reads are LDS reads; an
// older upwind result is loaded from global memory before the task's turn.
#include <float.h>
#include <limits.h>

#include <algorithm>
#include <type_traits>

#include "device.h"
#include "internal.h"
#include "sweep.h"

namespace sweep {

namespace {

constexpr float kInv4Pi = 0.0795774715459476678f;  // 1 / (4 pi)

// Buffer loads: every per-unit array is addressed through a buffer resource
// (base in scalar registers, 32-bit offsets); offsets past the end read 0.
constexpr int32_t kBufFlags = 0x00020000;  // raw buffer, 32-bit data (gfx9 family)
constexpr uint32_t kOob = 0x7ffffff0u;     // an offset past the end of any buffer here

template <class T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const T* p, int64_t bytes) {
  // the arguments are uniform; read from the first lane so that the descriptor
  // is built in scalar registers (a descriptor in vector registers costs a
  // loop over the distinct values at every access)
  const uint64_t a = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
  const int n = __builtin_amdgcn_readfirstlane((int)(p == nullptr ? 0 : bytes));
  return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(((uint64_t)hi << 32) | lo), (short)0, n,
                                           kBufFlags);
}

// Cache policy of the accesses the sweep makes once per step and never again
// (row entries, task records, results in cell order): non-temporal, so the L2
// keeps the schedule-order results that later steps read back.
constexpr int kStream = 2;

template <int POL = 0>
__device__ __forceinline__ int4 ld_b128(__amdgpu_buffer_rsrc_t r, uint32_t vo, uint32_t so) {
  return __builtin_bit_cast(int4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)vo, (int)so, POL));
}
template <int POL = 0>
__device__ __forceinline__ void st_f32(float v, __amdgpu_buffer_rsrc_t r, uint32_t vo) {
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(v), r, (int)vo, 0, POL);
}

// GN consecutive FP32 values at byte offset vo + so of a buffer (one access for
// GN = 2 or 4; offsets past the buffer's end read zeros and drop stores).
template <int GN, int POL = 0>
__device__ __forceinline__ void ld_gn(__amdgpu_buffer_rsrc_t r, uint32_t vo, uint32_t so, float* v) {
  if constexpr (GN == 4) {
    const int4 x = __builtin_bit_cast(int4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)vo, (int)so, POL));
    v[0] = __int_as_float(x.x);
    v[1] = __int_as_float(x.y);
    v[2] = __int_as_float(x.z);
    v[3] = __int_as_float(x.w);
  } else if constexpr (GN == 2) {
    const int2 x = __builtin_bit_cast(int2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)vo, (int)so, POL));
    v[0] = __int_as_float(x.x);
    v[1] = __int_as_float(x.y);
  } else {
#pragma unroll
    for (int g = 0; g < GN; ++g) v[g] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)(vo + 4u * g), (int)so, POL));
  }
}

template <int GN, int POL = 0>
__device__ __forceinline__ void st_gn(const float* v, __amdgpu_buffer_rsrc_t r, uint32_t vo) {
  if constexpr (GN == 4) {
    const int4 x = make_int4(__float_as_int(v[0]), __float_as_int(v[1]), __float_as_int(v[2]),
                             __float_as_int(v[3]));
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(__attribute__((ext_vector_type(4))) int, x), r, (int)vo, 0, POL);
  } else if constexpr (GN == 2) {
    const int2 x = make_int2(__float_as_int(v[0]), __float_as_int(v[1]));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(__attribute__((ext_vector_type(2))) int, x), r, (int)vo, 0, POL);
  } else {
#pragma unroll
    for (int g = 0; g < GN; ++g) st_f32<POL>(v[g], r, vo + 4u * g);
  }
}

__device__ __forceinline__ int64_t uniform64(int64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// A uniform pointer to global memory in scalar registers (its loads take a 32-bit
// offset per lane).
template <class T>
using global_ptr = const T __attribute__((address_space(1)))*;

template <class T>
__device__ __forceinline__ global_ptr<T> uniform_ptr(const T* p) {
  return (global_ptr<T>)(uint64_t)uniform64((int64_t)(uint64_t)p);
}

// Values of other lanes: lane `from` mod 64 (__shfl without its width, which takes
// registers), lane `from` for a uniform `from`, the lane below.
__device__ __forceinline__ float lane_value(float v, int from) {
  return __int_as_float(__builtin_amdgcn_ds_bpermute(4 * from, __float_as_int(v)));
}
__device__ __forceinline__ float lane_scalar(float v, int from) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), from));
}
__device__ __forceinline__ float lane_below(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, true));  // wave_shr:1
}

// Entry pairs of a row held in registers, the kernel's P: kPairs (16 entries), or 2 where no
// row of the walk is longer (regular grids, tetrahedra), which leaves out the loads and the
// work for columns that nobody has.  128^3 lattice cells x 84 directions: 2.70 ms with 2
// pairs, 4.14 with 8; 32^3: 57 and 86 us.  One longer row is enough for 8, although the
// pairs past the registers have a path of their own: a choice by how many rows are that long
// would also serve scheme (b), with 2.7 entries per row on average and 10 at most.
constexpr int kPairs = 8;

// The unit's arrays (uniform over the workgroup).
struct UnitBufs {
  global_ptr<int32_t> len;       // row lengths of the unit, schedule order
  global_ptr<float> den;         // [slot][G] at group g0 of the unit's first task
  global_ptr<float> src;
  __amdgpu_buffer_rsrc_t outs;   // out_s at group g0 of the unit's first task: [slot][G]
  int C;                         // tasks of the unit
  int ns;                        // slices of the unit
};

// GN consecutive values at 32-bit word offset `off` of a uniform pointer.
template <int GN>
__device__ __forceinline__ void ld_stream(global_ptr<float> p, uint32_t off, float* v) {
#pragma unroll
  for (int g = 0; g < GN; ++g) v[g] = __builtin_nontemporal_load(p + off + g);
}

// One slice: its uniform part and one task per lane.
template <int GN>
struct Slice {
  int k0, cnt, dep, lim, ks;  // uniform: SliceRec
  int64_t base;               // uniform: first entry pair
  int np;                     // uniform: entry pairs
  int n4 = 0, n6 = 0, nt;     // uniform: pairs in columns 4 and 6; pairs past the columns in registers
  int len;                    // per lane: row length
  float den[GN], src[GN];
};

// Row entries of a slice in registers: P pairs of this lane's row, and one
// pair of the slice's entries past those columns.  Loaded as (position code,
// factor) twice; resolving turns the codes into LDS byte offsets.
template <int P>
struct Entries {
  int4 e[P];
  int4 t;
};

// LDS byte offset of the ring slot of position code x (see k_fill).
template <int GN>
__device__ __forceinline__ int slot_of(int x, int mask4) { return (x & mask4) * GN; }

// The sweep's LDS is dynamic only (sweep_static_lds), so it starts at LDS address 0 and
// slot offsets are addresses: GN consecutive floats read or written there in one access.
template <int GN>
struct LdsVec {
  using type = float __attribute__((ext_vector_type(GN)));
};
template <class T>
__device__ __forceinline__ T __attribute__((address_space(3)))* lds_at(int addr) {
  return (T __attribute__((address_space(3)))*)(uint32_t)addr;
}

template <int GN>
__device__ __forceinline__ void lds_read(int addr, float* v) {
  if constexpr (GN == 1) {
    v[0] = *lds_at<float>(addr);
  } else if constexpr (GN == 3) {
#pragma unroll
    for (int g = 0; g < 3; ++g) v[g] = *lds_at<float>(addr + 4 * g);
  } else {
    const typename LdsVec<GN>::type x = *lds_at<typename LdsVec<GN>::type>(addr);
#pragma unroll
    for (int g = 0; g < GN; ++g) v[g] = x[g];
  }
}

template <int GN>
__device__ __forceinline__ void lds_write(int addr, const float* v) {
  if constexpr (GN == 1 || GN == 3) {
#pragma unroll
    for (int g = 0; g < GN; ++g) *lds_at<float>(addr + 4 * g) = v[g];
  } else {
    typename LdsVec<GN>::type x;
#pragma unroll
    for (int g = 0; g < GN; ++g) x[g] = v[g];
    *lds_at<typename LdsVec<GN>::type>(addr) = x;
  }
}

using lds_int = int __attribute__((address_space(3)));

// Waits until the workgroup's counter has reached `need` (it is only ever
// raised by wavefronts that never wait for this one, see k_sweep; a counter that
// stands still for millions of reads raises the error flag instead of hanging).
__device__ __forceinline__ void wait_count(lds_int* counter, int need, int& seen, int32_t* flag) {
  if (seen >= need) return;
  // (five reads in a row: with a loop's branches behind every read, each link of the chain
  // of levels is longer, 4,096 cells x 8 directions 82.8 instead of 75.7 us)
  for (int it = 0; it < kSpinLimit; it += 5) {
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      seen = uni(__hip_atomic_load(counter, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP));
      if (seen >= need) return;
    }
  }
  atomicOr(flag, kErrStall);
  seen = INT_MAX;
}

// Waits until every wavefront has stored its slices before `need`: last[w] is the slice
// that wavefront w (of nw) stored last.  All of these slices are counted by then, and a
// counted slice waits for nothing before its store.
__device__ __forceinline__ void wait_stored(lds_int* last, int nw, int lane, int need, int32_t* flag) {
  int w = lane;
  asm volatile("" : "+v"(w));  // (nothing of it is kept in registers of the common path)
  w = min(w, nw - 1);          // (no branch: the turn's control flow stays uniform)
  for (int it = 0;; ++it) {
    const int next = __hip_atomic_load(last + w, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) + nw;
    if (__ballot(next < need) == 0ull) return;
    if (it >= kSpinLimit) {
      atomicOr(flag, kErrStall);
      return;
    }
  }
}

// One workgroup sweeps one (mesh, direction, group chunk) work item at a time.
// The tasks of every level are cut into slices of at most 64 (k_slices), one
// task per lane, and slice i belongs to wavefront i mod (wavefronts).  A slice
// may run once every slice of the earlier levels has finished: each finishing
// slice adds one to an LDS counter, and a wavefront waits until the counter has
// reached the number of slices before its level (SliceRec.dep; slices of the
// level itself or later ones cannot be among those counted, as they wait for
// the same number).  There is no barrier: a wavefront has everything of its next
// slice but the recent upwind results in registers before its turn comes, and
// between two turns of a wavefront the others' levels pass.  The wavefront with
// the lowest unfinished slice never waits for anything unfinished, so every wait
// ends.
//
// Per slice and lane: the row's entries (position code, factor), loaded a turn
// ahead from a layout in which pair j of the rows that have one is contiguous
// over the lanes (k_fill), so each load is coalesced; upwind results older than
// the LDS ring's window, loaded a turn ahead into registers; then, in turn, one
// LDS read per entry, the fused multiply-adds in row order, the division, the
// ring slot and the count.  The store to out_s (schedule order, coalesced) follows
// the count; k_to_cells brings the results into cell order afterwards (a store in
// cell order here would touch a line per lane, more than all the loads together).
//
// LDS ring: the results of the last R positions of the schedule.  Position p is
// read from the ring by a slice of a level that ends at `lim` only if p >= lim - R:
// while a slice runs, no later level writes, so the slot has not been reused (and
// of a level wider than the ring, whose slices run in any order, only the last R
// positions write at all).
// An older result is read from out_s.  It is visible there to a slice's early
// loads if it lies before the level of the wavefront's previous slice by more than
// the positions whose slices may have been counted but not yet stored (one slice
// per wavefront: 64 x wavefronts).  A slice with an older result that is neither
// (very wide levels, tiny rings), or with more row entries than the registers
// hold, loads such results after its wait, once every wavefront has
// stored its slices of the earlier levels (each keeps the slice that it stored last
// in LDS.  The number of stored slices would not do: other slices of the
// same level, which do not wait for stores, may be among them while one of an earlier
// level is counted but not yet stored); same terms in the same order, so every path
// gives the same bits.
//
// The adjoint walks the slices backwards; its rows name reversed positions, so
// the same code serves both.
//
// What bounds it: narrow levels, the chain from one level's count to the next (about
// 0.31 us: LDS reads, multiply-adds, division, ring write, count, poll); all that does not
// wait for the level before is kept out of it, against the compiler where need be (the
// slots' addresses, the reads of the row's tail).  Wide levels, the line requests of one
// compute unit's L1 (a unit runs on one) and its instruction issue.  Against steps of a
// level with one barrier each, whose wavefronts loaded, staged through LDS and solved by
// turns (forward sweep per launch): 64^3 cells x 84 directions 2.27 -> 0.71 ms; 4,096 cells
// x 8 directions 0.288 -> 0.075 ms; 2M clustered cells x 84 directions x 4 groups 27.0 ->
// 12.0 ms (+ 1.5 ms for k_to_cells; with the results stored in cell order from here, 26.4).
// A division with the reciprocal taken before the wait, and a test whether that is exact,
// was slower: the test's branch costs more than the divide's dependent steps.
template <int GN, bool REVERSE, int P>
__global__ __launch_bounds__(kSweepMaxBlock(GN)) void k_sweep(SweepArgs a) {
  constexpr int P4 = P < 4 ? P : 4, P6 = P < 6 ? P : 6;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = uni(tid >> 6);
  const int nw = blockDim.x >> 6;
  const int R = a.ring_mask + 1;
  const int mask4 = a.ring_mask * 4;
  const int lag = 64 * nw;
  const uint32_t lane4G = 4u * (uint32_t)(lane * a.G);
  const int zero = R * GN * 4;  // the zero slot's address
  if (tid < GN) *lds_at<float>(zero + 4 * tid) = 0.0f;
  // behind the ring, the zero slot and the sink: the count of finished slices, the next
  // work item, the slice that every wavefront stored last
  lds_int* s_done = lds_at<int>(zero + 2 * GN * 4);
  lds_int* s_last = s_done + 2;
  const int my_last = zero + 2 * GN * 4 + 8 + 4 * wave;  // (its address)
  for (int it = 0;; ++it) {
    __syncthreads();  // the previous item's counters and ring are no longer read
    int mine = wave, z = zero;
    asm volatile("" : "+s"(mine), "+s"(z));  // (or addresses made of them are kept in vector registers)
    lds_int* const s_unit = lds_at<int>(z + 2 * GN * 4) + 1;
    if (lane == 0) s_last[mine] = mine - nw;
    if (lane + mine == 0) {
      *s_done = 0;
      if (a.work_counter != nullptr) *s_unit = atomicAdd(a.work_counter, 1);
    }
    __syncthreads();
    const int ui = a.work_counter != nullptr ? uni(*s_unit) : (it == 0 ? (int)blockIdx.x : INT_MAX);
    if (ui >= a.n_units * a.n_chunks) break;
    const int u = a.unit_order[ui / a.n_chunks];
    const int g0 = a.g0 + (ui % a.n_chunks) * GN;
    const Unit U = a.units[u];
    const int64_t tb = U.task_base;
    UnitBufs B;
    B.C = uni(U.n_cells);
    const int64_t s0 = a.slice_base[u];
    B.ns = uni((int)(a.slice_base[u + 1] - s0));
    if (B.ns <= 0) continue;
    const int64_t C = B.C;
    B.len = uniform_ptr(a.len + tb);
    B.den = uniform_ptr(a.tden + tb * a.G + g0);
    B.src = uniform_ptr(a.tsrc + tb * a.G + g0);
    B.outs = rsrc(a.out_s + tb * a.G + g0, 4 * (C * a.G - g0));

    // a slice record, one word per lane (lanes 0 to 7); past the unit's last slice
    // it is empty
    const global_ptr<int32_t> recs = uniform_ptr(reinterpret_cast<const int32_t*>(a.slices + s0));
    auto load_info = [&](int i) -> int {
      const int at = min(i, B.ns - 1);
      return recs[8u * (uint32_t)(REVERSE ? B.ns - 1 - at : at) + (uint32_t)(lane & 7)];
    };
    auto take_info = [&](int i, int info, Slice<GN>& S) {
      const bool in = i < B.ns;
      S.k0 = __builtin_amdgcn_readlane(info, 0);
      S.cnt = in ? __builtin_amdgcn_readlane(info, 1) : 0;
      S.dep = in ? __builtin_amdgcn_readlane(info, 2) : 0;
      S.lim = __builtin_amdgcn_readlane(info, 3);
      S.ks = __builtin_amdgcn_readlane(info, 4);
      S.base = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readlane(info, 6) << 32) |
                         (uint32_t)__builtin_amdgcn_readlane(info, 5));
      S.np = in ? __builtin_amdgcn_readlane(info, 7) : 0;
    };
    // (lanes without a task read the slice's first one)
    auto load_tasks = [&](Slice<GN>& S) {
      const uint32_t k = (uint32_t)(S.k0 + (lane < S.cnt ? lane : 0));
      S.len = __builtin_nontemporal_load(B.len + k);
      ld_stream<GN>(B.den, k * (uint32_t)a.G, S.den);
      ld_stream<GN>(B.src, k * (uint32_t)a.G, S.src);
    };
    // Pair j of the rows that have one is stored for those lanes in lane order.
    auto load_entries = [&](Slice<GN>& S, Entries<P>& E) {
      const __amdgpu_buffer_rsrc_t ent = rsrc(a.ent + S.base, 16 * (int64_t)S.np);
      const int len = S.len = lane < S.cnt ? S.len : 0;
      int off = 0;
#pragma unroll
      for (int j = 0; j < P; ++j) {
        const bool has = len > 2 * j;
        const uint64_t m = __ballot(has);
        uint32_t at = 16u * (uint32_t)rank_in(m);
        asm volatile("" : "+v"(at));  // (a select, not a branch around its computation)
        E.e[j] = ld_b128<kStream>(ent, has ? at : kOob, 16u * (uint32_t)off);
        const int n = __popcll(m);
        off += n;
        if (j == 4) S.n4 = n;
        if (j == 6) S.n6 = n;
      }
      S.nt = S.np - off;
      E.t = ld_b128<kStream>(ent, lane < S.nt ? 16u * (uint32_t)lane : kOob, 16u * (uint32_t)off);
    };

    int i = wave;  // slice S0
    Slice<GN> S0, S1, S2;
    int info;                  // record of the slice after S2
    Entries<P> EA, EB;
    float f[2 * P][GN], ft[2][GN];  // results from outside the window (else 0), of the slice resolved last
    // how the slice resolved last is summed: its rows have up to P4, P6 or P pairs, all in
    // the window; kOlder: some entry lies outside it, or rows go past the registers; kSlow:
    // one of those is not visible yet, or rows go on still longer (not resolved: codes)
    enum { kUpTo4, kUpTo6, kUpTo8, kOlder, kSlow };
    int mode = kUpTo4;
    int seen = 0;                        // the count as last read
    int vis = 0;                         // results before this position are in out_s

    // LDS address of the entry with position code x (outside the window: the zero slot).
    auto slot = [&](int& x, uint32_t lo4) {
      x = (uint32_t)x < lo4 ? zero : slot_of<GN>(x, mask4);
      asm volatile("" : "+v"(x));
    };
    // Window test, early loads of the older results and LDS offsets of a slice
    // (entries outside the window, and lanes without an entry, name the zero slot).
    auto resolve = [&](const Slice<GN>& S, Entries<P>& E, auto&& between) {
      // codes below lo4 lie outside the window; real ones (not 0) are tested after
      // subtracting 4, which sends 0 to the top
      const uint32_t lo4 = 4u * (uint32_t)(max(S.lim - R, 0) + 1);
      const uint32_t vis4 = 4u * (uint32_t)max(vis, 0);
      uint32_t low = 0xffffffffu;  // the smallest real code
      auto lowest = [&](int j0, int j1) {
#pragma unroll
        for (int j = j0; j < j1; ++j) low = min(min(low, (uint32_t)E.e[j].x - 4u), (uint32_t)E.e[j].z - 4u);
      };
      const bool past4 = P > 4 && S.n4 > 0, past6 = P > 6 && S.n6 > 0;
      lowest(0, P4);
      if (past4) lowest(P4, P6);
      if (past6) lowest(P6, P);
      if (S.nt > 0) low = min(min(low, (uint32_t)E.t.x - 4u), (uint32_t)E.t.z - 4u);
      const bool any = __ballot(low < lo4 - 4u) != 0ull;
      bool bad = S.nt > 64;
      // the older results of the slice before are dead (their registers are free until here)
#pragma unroll
      for (int q = 0; q < 2 * P; ++q)
#pragma unroll
        for (int g = 0; g < GN; ++g) asm volatile("" : "=v"(f[q][g]));
#pragma unroll
      for (int g = 0; g < GN; ++g) asm volatile("" : "=v"(ft[0][g]), "=v"(ft[1][g]));
      between();
      if (any) {
        bool b = false;
        // the early load of one entry: out of range (0) for lanes without one
        auto old = [&](int x, float* v) {
          const uint32_t y = (uint32_t)x - 4u;
          const bool need = y < lo4 - 4u;
          const uint32_t d = REVERSE ? 4u * (uint32_t)B.C - (uint32_t)x : y;
          b |= need && y >= vis4;
          ld_gn<GN>(B.outs, need ? d * (uint32_t)a.G : kOob, 0, v);
        };
#pragma unroll
        for (int j = 0; j < P; ++j) {
          old(E.e[j].x, f[2 * j]);
          old(E.e[j].z, f[2 * j + 1]);
        }
        old(E.t.x, ft[0]);
        old(E.t.z, ft[1]);
        bad |= __ballot(b) != 0ull;
      } else if (S.nt > 0) {  // (summed as kOlder)
#pragma unroll
        for (int q = 0; q < 2 * P; ++q)
#pragma unroll
          for (int g = 0; g < GN; ++g) f[q][g] = 0.0f;
#pragma unroll
        for (int g = 0; g < GN; ++g) ft[0][g] = ft[1][g] = 0.0f;
      }
      mode = bad ? kSlow : any || S.nt > 0 ? kOlder : past6 ? kUpTo8 : past4 ? kUpTo6 : kUpTo4;
      if (bad) return;  // (its codes are resolved after the wait)
      // (computed now, not after the wait for the slice's turn, where they are used)
      auto slots = [&](int j0, int j1) {
#pragma unroll
        for (int j = j0; j < j1; ++j) {
          slot(E.e[j].x, lo4);
          slot(E.e[j].z, lo4);
        }
      };
      slots(0, P4);
      if (past4 || any) slots(P4, P6);
      if (past6 || any) slots(P6, P);
      if (any || S.nt > 0) {
        slot(E.t.x, lo4);
        slot(E.t.z, lo4);
      }
    };

    // Inflow of a resolved slice, the terms of each row in order: its first J1 pairs, every
    // read issued before the first is used.  OLD: a value is the ring's or the early-loaded
    // one; the other of the two is +0, so their bits are joined.
    auto join = [&](auto old_c, float x, float y) {
      return decltype(old_c)::value ? __int_as_float(__float_as_int(x) | __float_as_int(y)) : x;
    };
    auto gather = [&](const Entries<P>& E, auto old_c, auto j0_c, auto j1_c, float* acc) {
      constexpr int J0 = decltype(j0_c)::value, J1 = decltype(j1_c)::value;
      float v[2 * (J1 - J0)][GN];
#pragma unroll
      for (int j = J0; j < J1; ++j) {
        lds_read<GN>(E.e[j].x, v[2 * (j - J0)]);
        lds_read<GN>(E.e[j].z, v[2 * (j - J0) + 1]);
      }
#pragma unroll
      for (int q = 2 * J0; q < 2 * J1; ++q) {
        const float w = __int_as_float(q & 1 ? E.e[q / 2].w : E.e[q / 2].y);
#pragma unroll
        for (int g = 0; g < GN; ++g) acc[g] = __builtin_fmaf(w, join(old_c, v[q - 2 * J0][g], f[q][g]), acc[g]);
      }
    };
    constexpr std::integral_constant<int, 0> c0{};
    constexpr std::integral_constant<int, P4> c4{};
    constexpr std::integral_constant<int, P6> c6{};
    constexpr std::integral_constant<int, P> c8{};
    constexpr std::false_type ring{};
    constexpr std::true_type older{};
    // kOlder: in two halves (the registers do not hold all values at once)
    auto gather_older = [&](const Slice<GN>& S, const Entries<P>& E, float* acc) {
      gather(E, older, c0, c4, acc);
      if constexpr (P > 4) gather(E, older, c4, c8, acc);
      if (S.nt > 0) {
        // pairs past the registers: lane i holds pair i of them; each column's rows
        // take theirs in turn
        float x0[GN], x1[GN];
        lds_read<GN>(E.t.x, x0);
        lds_read<GN>(E.t.z, x1);
#pragma unroll
        for (int g = 0; g < GN; ++g) {
          x0[g] = join(older, x0[g], ft[0][g]);
          x1[g] = join(older, x1[g], ft[1][g]);
        }
        for (int j = P, at = 0; at < S.nt; ++j) {
          const bool has = S.len > 2 * j;
          const uint64_t m = __ballot(has);
          const int from = at + rank_in(m);
          const float w0 = lane_value(__int_as_float(E.t.y), from), w1 = lane_value(__int_as_float(E.t.w), from);
#pragma unroll
          for (int g = 0; g < GN; ++g) {
            const float y0 = lane_value(x0[g], from), y1 = lane_value(x1[g], from);
            const float s = __builtin_fmaf(w1, y1, __builtin_fmaf(w0, y0, acc[g]));
            acc[g] = has ? s : acc[g];
          }
          at += __popcll(m);
        }
      }
    };

    // The same sum after the wait for the stores of the earlier levels, when every older
    // result can be loaded, of slice `at`: the columns in registers by halves, then the pairs
    // past them 64 at a time, the next ones on their way meanwhile.  (All pairs one after the
    // other, from memory, took three to six times as long: 400 cells that all border each other x 8
    // directions 8.9 ms, now 1.5; 8,000 cells x 24 directions with a ring of 64 results 0.93
    // and 0.34.)
    auto gather_slow = [&](int at, const Slice<GN>& S, Entries<P>& E, float* acc) {
      wait_stored(s_last, nw, lane, S.dep, a.flag);
      const uint32_t lo4 = 4u * (uint32_t)(max(S.lim - R, 0) + 1);
      auto old = [&](int x, float* v) {
        const uint32_t y = (uint32_t)x - 4u;
        const uint32_t d = REVERSE ? 4u * (uint32_t)B.C - (uint32_t)x : y;
        ld_gn<GN>(B.outs, y < lo4 - 4u ? d * (uint32_t)a.G : kOob, 0, v);
      };
      auto columns = [&](auto j0_c, auto j1_c) {
        constexpr int J0 = decltype(j0_c)::value, N = 2 * (decltype(j1_c)::value - J0);
        float o[N][GN], v[N][GN];
#pragma unroll
        for (int q = 0; q < N; ++q) {
          int& x = q & 1 ? E.e[J0 + q / 2].z : E.e[J0 + q / 2].x;
          old(x, o[q]);
          slot(x, lo4);
        }
#pragma unroll
        for (int q = 0; q < N; ++q) lds_read<GN>(q & 1 ? E.e[J0 + q / 2].z : E.e[J0 + q / 2].x, v[q]);
#pragma unroll
        for (int q = 0; q < N; ++q) {
          const float w = __int_as_float(q & 1 ? E.e[J0 + q / 2].w : E.e[J0 + q / 2].y);
#pragma unroll
          for (int g = 0; g < GN; ++g) acc[g] = __builtin_fmaf(w, join(older, v[q][g], o[q][g]), acc[g]);
        }
        __builtin_amdgcn_sched_barrier(0);  // (or both halves' values take registers at once)
      };
      columns(c0, c4);
      if constexpr (P > 4) columns(c4, c8);
      if (S.nt > 0) {
        const int rec = load_info(at);  // (the place of the entries is not kept up to here)
        int4& t = E.t;
        int j = P, first = 0;  // the column, and its first pair of the S.nt
        for (int b = 0; b < S.nt; b += 64) {
          float x0[GN], x1[GN], o0[GN], o1[GN];
          old(t.x, o0);
          old(t.z, o1);
          slot(t.x, lo4);
          slot(t.z, lo4);
          lds_read<GN>(t.x, x0);
          lds_read<GN>(t.z, x1);
          Slice<GN> R0;
          take_info(at, rec, R0);
          const __amdgpu_buffer_rsrc_t ent = rsrc(a.ent + R0.base, 16 * (int64_t)R0.np);
          int l = lane;
          asm volatile("" : "+v"(l));  // (nothing of it is kept in registers of the common path)
          const int at64 = R0.np - S.nt + b + 64;
          const int4 next = ld_b128(ent, at64 + l < R0.np ? 16u * (uint32_t)(at64 + l) : kOob, 0);
#pragma unroll
          for (int g = 0; g < GN; ++g) {
            x0[g] = join(older, x0[g], o0[g]);
            x1[g] = join(older, x1[g], o1[g]);
          }
          // lane i holds pair b + i; kCols columns at a time, whose values are under way
          // together; one that goes on behind the pairs at hand is taken up again there
          constexpr int kCols = GN > 2 ? 2 : 4;
          const int end = min(b + 64, S.nt);
          int rows = __popcll(__ballot(S.len > 2 * j));
          for (bool more = true; more && first < end && rows > 1;) {
            float w0[kCols], w1[kCols], y0[kCols][GN], y1[kCols][GN];
            bool in[kCols];
#pragma unroll
            for (int u = 0; u < kCols; ++u) {
              const bool has = S.len > 2 * j;
              const uint64_t m = __ballot(has);
              const int n = __popcll(m), from = first + rank_in(m) - b;
              in[u] = has && more && (uint32_t)from < 64u;
              w0[u] = lane_value(__int_as_float(t.y), from);
              w1[u] = lane_value(__int_as_float(t.w), from);
#pragma unroll
              for (int g = 0; g < GN; ++g) {
                y0[u][g] = lane_value(x0[g], from);
                y1[u][g] = lane_value(x1[g], from);
              }
              more = more && first + n <= end;
              first += more ? n : 0;
              j += more ? 1 : 0;
            }
#pragma unroll
            for (int u = 0; u < kCols; ++u)
#pragma unroll
              for (int g = 0; g < GN; ++g) {
                const float s = __builtin_fmaf(w1[u], y1[u][g], __builtin_fmaf(w0[u], y0[u][g], acc[g]));
                acc[g] = in[u] ? s : acc[g];
              }
            rows = __popcll(__ballot(S.len > 2 * j));
          }
          if (rows == 1 && first < end) {
            // the longest row alone: its sum goes from lane to lane
            const uint64_t m = __ballot(S.len > 2 * j);
            const int owner = __ffsll((long long)m) - 1;
            float r[GN];
#pragma unroll
            for (int g = 0; g < GN; ++g) {
              r[g] = lane_scalar(acc[g], owner);
              r[g] = __builtin_fmaf(__int_as_float(t.w), x1[g], __builtin_fmaf(__int_as_float(t.y), x0[g], r[g]));
            }
            for (int q = first + 1; q < end; ++q) {
#pragma unroll
              for (int g = 0; g < GN; ++g)
                r[g] = __builtin_fmaf(__int_as_float(t.w), x1[g], __builtin_fmaf(__int_as_float(t.y), x0[g], lane_below(r[g])));
            }
#pragma unroll
            for (int g = 0; g < GN; ++g) acc[g] = lane == owner ? lane_scalar(r[g], end - 1 - b) : acc[g];
            j += end - first;
            first = end;
          }
          t = next;
        }
      }
      // no memory operation of this path stays in flight, so the waits of the
      // common path are counted exactly
      __builtin_amdgcn_s_waitcnt(0);
    };

    // The early-loaded results are consumed whether any were loaded or not (the loads
    // issued after them are counted exactly, and nothing later waits for them).
    auto consume_old = [&]() {
#pragma unroll
      for (int q = 0; q < 2 * P; ++q)
#pragma unroll
        for (int g = 0; g < GN; ++g) asm volatile("" : "+v"(f[q][g]));
#pragma unroll
      for (int g = 0; g < GN; ++g) asm volatile("" : "+v"(ft[0][g]), "+v"(ft[1][g]));
    };

    // One turn: slice S0 (entries E resolved) is solved, S1 (entries N in flight)
    // is resolved, S2's entries are loaded into E, and the loads of the
    // following slices are issued.

    auto turn = [&](Entries<P>& E, Entries<P>& N) {
      consume_old();
      // ring slot of the lane's result: the sink for lanes without a task and for
      // positions of a level wider than the ring that a later one of the level reuses
      const bool act = lane < S0.cnt;
      const int code = 4 * (REVERSE ? B.C - (S0.k0 + lane) : S0.k0 + lane + 1);
      const int at = act && code > 4 * (S0.lim - R) ? slot_of<GN>(code, mask4) : zero + 4 * GN;
      wait_count(s_done, S0.dep, seen, a.flag);
      __builtin_amdgcn_s_setprio(3);
      float acc[GN], v[GN];
#pragma unroll
      for (int g = 0; g < GN; ++g) acc[g] = 0.0f;
      // (The same choice three times, as the branches' order and nesting decide how the
      // compiler lays the ways out, and with them the sweep's time.  Eight pairs, one group:
      // 4,096 cells x 8 directions 74.5 us, 78.7 in one chain with the slow path.  Packed
      // groups: 64^3 cells x 84 directions x 2 groups 843 us in one chain, 902 with the slow
      // path behind it.  Two pairs: 64^3 lattice cells along an axis 262 us, 272 and 276.)
      if constexpr (P <= 4) {
        if (__builtin_expect(mode < kOlder, 1)) gather(E, ring, c0, c4, acc);
        else if (__builtin_expect(mode == kOlder, 1)) gather_older(S0, E, acc);
        else gather_slow(i, S0, E, acc);
      } else if constexpr (GN > 1) {
        if (mode == kUpTo6) gather(E, ring, c0, c6, acc);
        else if (mode == kUpTo4) gather(E, ring, c0, c4, acc);
        else if (mode == kUpTo8) gather(E, ring, c0, c8, acc);
        else if (mode == kOlder) gather_older(S0, E, acc);
        else gather_slow(i, S0, E, acc);
      } else {
        if (mode == kUpTo6) gather(E, ring, c0, c6, acc);
        else if (mode == kUpTo4) gather(E, ring, c0, c4, acc);
        else if (mode == kUpTo8) gather(E, ring, c0, c8, acc);
        else if (mode == kOlder) gather_older(S0, E, acc);
        if (__builtin_expect(mode == kSlow, 0)) gather_slow(i, S0, E, acc);
      }
      const int n0 = S0.cnt > 0 ? 1 : 0;  // (past the wavefront's last slice a turn has no task)
#pragma unroll
      for (int g = 0; g < GN; ++g) v[g] = __fdiv_rn(__fadd_rn(acc[g], S0.src[g]), S0.den[g]);
      lds_write<GN>(at, v);
      // (LDS operations of a wavefront are performed in order: no wait between the two)
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      if (lane < n0) __hip_atomic_fetch_add(s_done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      __builtin_amdgcn_s_setprio(0);
      st_gn<GN>(v, B.outs, act ? 4u * (uint32_t)(S0.k0 * a.G) + lane4G : kOob);
      int n1 = n0;
      asm volatile("" : "+v"(n1));  // (its own condition, or the compiler splits the code between the two)
      int mine = my_last;
      asm volatile("" : "+s"(mine));  // (not kept in a vector register)
      if (lane < n1) __hip_atomic_store(lds_at<int>(mine), i, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
      vis = S0.ks - lag;
      Slice<GN> next = S2;
      resolve(S1, N, [&]() {
        // S2's tasks are consumed, by copies, before the early loads, whose number
        // varies, are issued: their wait is counted exactly, and the registers they
        // were loaded into take the next tasks' loads without a move behind those
#pragma unroll
        for (int g = 0; g < GN; ++g) {
          asm volatile("v_mov_b32 %0, %1" : "=v"(next.den[g]) : "v"(S2.den[g]));
          asm volatile("v_mov_b32 %0, %1" : "=v"(next.src[g]) : "v"(S2.src[g]));
        }
        asm volatile("v_mov_b32 %0, %1" : "=v"(next.len) : "v"(S2.len));
        asm volatile("" : "+v"(info));
      });
      load_entries(next, E);
      S0 = S1;
      S1 = next;
      take_info(i + 3 * nw, info, S2);
      load_tasks(S2);
      info = load_info(i + 4 * nw);
      i += nw;
    };
    // prologue: slices i, i + nw, i + 2 nw of this wavefront
    {
      const int i0 = load_info(i), i1 = load_info(i + nw), i2 = load_info(i + 2 * nw);
      info = load_info(i + 3 * nw);
      take_info(i, i0, S0);
      take_info(i + nw, i1, S1);
      take_info(i + 2 * nw, i2, S2);
    }
    load_tasks(S0);
    load_tasks(S1);
    load_tasks(S2);
#pragma unroll
    for (int q = 0; q < 2 * P; ++q)
#pragma unroll
      for (int g = 0; g < GN; ++g) f[q][g] = 0.0f;
#pragma unroll
    for (int g = 0; g < GN; ++g) ft[0][g] = ft[1][g] = 0.0f;
    load_entries(S0, EA);
    load_entries(S1, EB);
    resolve(S0, EA, []() {});
    consume_old();
    __builtin_amdgcn_s_waitcnt(0);
    while (i < B.ns) {
      turn(EA, EB);
      turn(EB, EA);  // (a turn past the last slice has nothing to wait for and counts nothing)
    }
  }
}

template <int GN, bool REVERSE>
hipError_t launch_sweep_g(const SweepArgs& a, int32_t grid, int32_t block, size_t lds,
                          hipStream_t s) {
  if (block < 64 || block % 64 != 0 || block > kSweepMaxBlock(GN)) return hipErrorInvalidValue;
  auto kernel = a.max_row <= 4 ? k_sweep<GN, REVERSE, 2> : k_sweep<GN, REVERSE, kPairs>;
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(block), lds, s, a);
  return hipGetLastError();
}

__device__ __forceinline__ int unit_of_block(const int32_t* blk_base, int n_units, int b) {
  int lo = 0, hi = n_units - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (blk_base[mid] <= b) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Results in schedule order -> cell order, [D][C][G]: one thread per (cell, VEC
// consecutive groups), the workgroups of a unit together on one XCD so that its
// gathers find the unit's lines in that L2.  Memory-bound: 2M cells x 84 directions x 4
// groups (5.6 GB of results in and out, 0.7 GB of positions) in 1.5 ms.
template <int VEC>
__global__ __launch_bounds__(256) void k_to_cells(const Unit* units, int n_units, const int32_t* blk_base,
                                                  const int32_t* inv, const float* out_s, float* out,
                                                  int64_t C_total, int G) {
  const int blk = xcd_block(blockIdx.x, gridDim.x);
  const int u = unit_of_block(blk_base, n_units, blk);
  const Unit U = units[u];
  const int c0 = (blk - blk_base[u]) * 256;
  const int n = min(256, U.n_cells - c0);
  const int64_t ob = (((int64_t)U.dir * C_total + U.cell_off) + c0) * G;
  const int32_t* iv = inv + U.task_base + c0;
  const float* os = out_s + U.task_base * G;
  const int GV = G / VEC;
  for (int i = threadIdx.x; i < n * GV; i += 256) {
    const int c = i / GV, g = i - c * GV;
    struct __attribute__((aligned(4 * VEC))) Vec {
      float x[VEC];
    };
    reinterpret_cast<Vec*>(out + ob)[i] = reinterpret_cast<const Vec*>(os + (int64_t)iv[c] * G)[g];
  }
}

template <bool REVERSE>
hipError_t launch_sweep_t(const SweepArgs& a, int32_t gn, int32_t grid, int32_t block,
                          size_t lds, hipStream_t s) {
  switch (gn) {
    case 1: return launch_sweep_g<1, REVERSE>(a, grid, block, lds, s);
    case 2: return launch_sweep_g<2, REVERSE>(a, grid, block, lds, s);
    case 3: return launch_sweep_g<3, REVERSE>(a, grid, block, lds, s);
    case 4: return launch_sweep_g<4, REVERSE>(a, grid, block, lds, s);
    default: return hipErrorInvalidValue;
  }
}

// Exponential cell law: with the optical depth tau = kappa V / Aperp (capped at
// 40 for the transmission), the entering power T of a task becomes the exit
// flux density x = T / den, den = Aperp e^{min(tau, 40)}, and the cell average
// is r x, r = Aperp (e^{min(tau, 40)} - 1) / (kappa V) (1 at kappa = 0).
constexpr double kTauCap = 40.0;

__device__ __forceinline__ double exp_den(double ap, double kV) {
  return ap * exp(fmin(kV / ap, kTauCap));
}

__device__ __forceinline__ double exp_r(double ap, double kV) {
  return kV > 0.0 ? ap * expm1(fmin(kV / ap, kTauCap)) / kV : 1.0;
}

// h'(t) for h(t) = (e^t - 1) / t: below 0.5 the power series
// sum_{k>=1} k t^{k-1} / (k+1)! to 18 terms (remainder below 1e-18, Horner
// with the coefficients folded at compile time), above it
// ((t - 1)(e^t - 1) + t) / t^2.
struct DhSeries {
  double c[18];
};

constexpr DhSeries dh_series() {
  DhSeries r{};
  double f = 2.0;  // (k+1)!
  for (int k = 1; k <= 18; ++k) {
    r.c[k - 1] = (double)k / f;
    f *= (double)(k + 2);
  }
  return r;
}

__device__ __forceinline__ double dh_dt(double t) {
  if (t < 0.5) {
    constexpr DhSeries S = dh_series();
    double s = S.c[17];
#pragma unroll
    for (int k = 16; k >= 0; --k) s = s * t + S.c[k];
    return s;
  }
  return ((t - 1.0) * expm1(t) + t) / (t * t);
}

// Per-task denominators (Aperp + kappa V, or the exponential law's den) and
// sources, in schedule order (what the sweep streams).  The sources do not
// depend on the direction: a first pass over the cells packs each cell's
// (kappa, source) per group into one record, so that the pass over the tasks
// reads its Aperp (schedule order) and writes its outputs coalesced, and
// gathers one record and the cell's volume from arrays every direction shares
// (which stay cache resident).  The adjoint source of the exponential law is
// r g, g being the derivative with respect to the cell average.
__global__ __launch_bounds__(256) void k_prep_cells(PrepArgs a) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= a.C_total * a.G) return;
  const int64_t ci = i / a.G;
  const double kap = (double)a.kappa[i];
  double s;
  if (a.emission != nullptr) {
    s = (double)a.emission[i];
    if (a.jsum_prev != nullptr) s += (double)a.albedo * kap * (double)a.vol[ci] * (double)a.jsum_prev[i];
    s *= (double)a.inv_D;
  } else {
    s = (double)a.gsrc[i];
  }
  // invalid inputs raise the DAG's error flag (reported by the next call that
  // synchronises); the kernels run on regardless
  int32_t bad = 0;
  if (!(kap >= 0.0 && kap <= DBL_MAX)) bad |= kErrKappa;
  if (a.emission != nullptr && !((double)a.emission[i] >= 0.0 && (double)a.emission[i] <= DBL_MAX))
    bad |= kErrEmission;
  if (bad != 0) atomicOr(a.flag, bad);
  a.crec[i] = make_float2(a.kappa[i], (float)s);
}

// Tasks of a workgroup whose G values per task are staged in LDS, so that the
// workgroup's [tasks][G] block of denominators and sources is written with
// consecutive threads on consecutive words (G up to kPrepStageG; larger G is
// written per task).
constexpr int kPrepStageG = 8;

// A line request per task, for its cell's record; the workgroups of a unit's consecutive
// tasks run on one XCD, so that neighbouring levels find the records' lines in its L2.
// 128^3 cells x 84 directions, exponential law: 1.48 ms, dealt round-robin 1.80; 64^3 x
// 84: 165 us either way.
template <bool EXP_LAW>
__global__ __launch_bounds__(256) void k_prep(PrepArgs a) {
  __shared__ float sden[256 * kPrepStageG], ssrc[256 * kPrepStageG];
  const int blk = xcd_block(blockIdx.x, gridDim.x);
  const int u = unit_of_block(a.blk_base, a.n_units, blk);
  const Unit U = a.units[u];
  const int k0 = (blk - a.blk_base[u]) * 256;
  const int k = k0 + threadIdx.x;
  const int G = a.G;
  const bool stage = G <= kPrepStageG;
  int32_t bad = 0;
  if (k < U.n_cells) {
    const int64_t t = U.task_base + k;  // schedule position
    const int64_t ci = (int64_t)U.cell_off + a.sched[t];
    const double V = (double)a.vol_s[t];
    const double ap = (double)a.aperp_s[t];
    // denominator and source of one group from the cell's (kappa, source) record
    auto task = [&](float2 r, float& den_out, float& src_out) {
      const double kap = (double)r.x;
      const double den = EXP_LAW ? exp_den(ap, kap * V) : ap + kap * V;
      double s = (double)r.y;
      if (EXP_LAW && a.emission == nullptr) s *= exp_r(ap, kap * V);
      if (!(den > 0.0 && den <= DBL_MAX)) bad |= kErrCell;
      den_out = (float)den;
      src_out = (float)s;
    };
    if (G == 1) {
      task(a.crec[ci], a.tden[t], a.tsrc[t]);
    } else if (stage) {
      // every group's record is loaded before the first is used: unconditional
      // loads (groups past G reread the last one), and the staged results go to
      // LDS, so no store orders them
      float2 r[kPrepStageG];
#pragma unroll
      for (int g = 0; g < kPrepStageG; ++g) r[g] = a.crec[ci * G + min(g, G - 1)];
#pragma unroll
      for (int g = 0; g < kPrepStageG; ++g)
        if (g < G) task(r[g], sden[threadIdx.x * G + g], ssrc[threadIdx.x * G + g]);
    } else {
      for (int g = 0; g < G; ++g) task(a.crec[ci * G + g], a.tden[t * G + g], a.tsrc[t * G + g]);
    }
  }
  if (stage && G > 1) {
    __syncthreads();
    const int n = min(256, U.n_cells - k0) * G;
    const int64_t base = (U.task_base + k0) * G;
    for (int i = threadIdx.x; i < n; i += 256) {
      a.tden[base + i] = sden[i];
      a.tsrc[base + i] = ssrc[i];
    }
  }
  if (bad != 0) atomicOr(a.flag, bad);
}

// Periodic coupling folded into the sources (PinArgs): one thread per
// (direction, periodic cell, group).
__global__ __launch_bounds__(256) void k_pin(PinArgs a) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (int64_t)a.D * a.n_pc * a.G) return;
  const int g = (int)(i % a.G);
  const int64_t dp = i / a.G;
  const int pc = (int)(dp % a.n_pc);
  const int d = (int)(dp / a.n_pc);
  const int f0 = a.pf_ptr[pc], f1 = a.pf_ptr[pc + 1];
  const float* w = a.pw + (int64_t)d * a.n_pf;
  const float* o = a.other + (int64_t)d * a.C_total * a.G + g;
  float s = 0.0f;
  for (int f = f0; f < f1; ++f) {
    const float wf = w[f];
    if (wf != 0.0f) s = __builtin_fmaf(wf, o[(int64_t)a.pnb[f] * a.G], s);
  }
  const int64_t t = a.ptask[dp];
  float base;
  if (a.capture) {
    base = a.tsrc[t * a.G + g];
    a.pbase[i] = base;
  } else {
    base = a.pbase[i];
  }
  a.tsrc[t * a.G + g] = base + s;
  if (a.pval != nullptr) a.pval[i] = s;
}

// The folded inflow of every (periodic cell, group) summed over directions in
// order, in FP64.
__global__ __launch_bounds__(256) void k_psum(PinArgs a) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t n = (int64_t)a.n_pc * a.G;
  if (i >= n) return;
  double pn = 0.0;
  for (int d = 0; d < a.D; ++d) pn += (double)a.pval[(int64_t)d * n + i];
  a.psum[i] = pn;
}

// ----------------------------------------------------------------------- reductions
constexpr int kRedItems = 256;  // (cell, group) items of a workgroup
constexpr int kRedBatch = 4;    // directions whose loads a thread has in flight
constexpr int kNPart = 9;

// Threads per item, among which its directions go round.
constexpr int red_teams(bool sched) { return sched ? 4 : 1; }

// The direction sums of a pass.  SCHED: straight from the sweep's results in schedule
// order (STORE: with their copy in cell order on the way), else from that copy.  Bound
// by the gathers (SCHED, a line request per task; the workgroups of consecutive cells
// run on one XCD, whose L2 then serves the other cells of a line) or by memory.  Four
// threads share an item (SCHED), since one per item leaves small meshes waiting for a
// chain of loads, and the boundary weights are read for cells that have boundary faces
// only (8 bytes per task, all zero elsewhere).  Copy and sums of 4096 cells x 8
// directions: 6.4 us, before 32; 32^3 x 84, exponential law: 32 us, before 96; 64^3 x 84:
// 122 us, before 197; 12 meshes of 512 to 8192 cells x 24 directions: 41 us, before 97.
// From the copy: 128^3 x 84, exponential law: 0.67 ms, before 0.80; 2 M cells x 84 x 4
// groups: 0.79 ms (3.6 TB/s), before 1.31.
template <bool EXP_LAW, bool SCHED, bool STORE>
__global__ __launch_bounds__(kRedItems* red_teams(SCHED)) void k_reduce(ReduceArgs a) {
  constexpr int kTeams = red_teams(SCHED);
  __shared__ double part[kNPart][kRedItems];
  __shared__ double sums[kTeams][3][kRedItems];
  const int i = threadIdx.x % kRedItems;
  const int team = __builtin_amdgcn_readfirstlane(threadIdx.x / kRedItems);
  const int blk = xcd_block(blockIdx.x, gridDim.x);
  const int m = a.blk_mesh[blk];
  const int G = a.G;
  const int c = a.blk_cell0[blk] + i / G;
  const int g = i % G;
  const int C = a.mesh_cells[m];
  const int lc = c - a.mesh_off[m];
  const bool active = i < a.cells_per_block * G && lc < C;
  const int64_t cg = (int64_t)c * G + g;
  double V = 0.0, kap = 0.0, js = 0.0, esc = 0.0, pout = 0.0;
  if (active) {
    const int64_t stride = a.C_total * G;
    const int64_t t0 = (int64_t)a.D * a.mesh_off[m];  // tasks of the mesh: [direction][cell]
    V = (double)a.vol[c];
    kap = (double)a.kappa[cg];
    const bool edge = a.edge[c] != 0;
    float zero = 0.0f;  // 0 x every value, as the sums of zero weights would be
    for (int d0 = team; d0 < a.D; d0 += kTeams * kRedBatch) {
      int64_t t[kRedBatch];
      int p[kRedBatch];
      float ph[kRedBatch];
#pragma unroll
      for (int k = 0; k < kRedBatch; ++k) {  // (past the last direction: read again)
        const int d = min(d0 + kTeams * k, a.D - 1);
        t[k] = t0 + (int64_t)d * C;
        if (SCHED) p[k] = a.inv[t[k] + lc];
        else ph[k] = a.phi[d * stride + cg];
      }
      if (SCHED) {
#pragma unroll
        for (int k = 0; k < kRedBatch; ++k) ph[k] = a.out_s[(t[k] + p[k]) * G + g];
      }
#pragma unroll
      for (int k = 0; k < kRedBatch; ++k) {
        const int d = d0 + kTeams * k;
        if (d >= a.D) break;
        // (the exit flux density x: phi itself under the upwind law)
        const double x = (double)ph[k];
        if (STORE) a.phi[d * stride + cg] = ph[k];
        js += EXP_LAW ? x * exp_r((double)a.aperp[t[k] + lc], kap * V) : x;
        zero = __builtin_fmaf(0.0f, ph[k], zero);
        if (edge) {
          const float2 b = a.bnd[t[k] + lc];
          esc += (double)b.x * x;
          pout += (double)b.y * x;
        }
      }
    }
    if (!edge) esc = pout = (double)zero;
  }
  if (team > 0) {
    sums[team][0][i] = js;
    sums[team][1][i] = esc;
    sums[team][2][i] = pout;
  }
  __syncthreads();
  if (team == 0) {
    double v[kNPart] = {};
    if (active) {
#pragma unroll
      for (int k = 1; k < kTeams; ++k) {
        js += sums[k][0][i];
        esc += sums[k][1][i];
        pout += sums[k][2][i];
      }
      // the periodic inflow of the pass (and of the pass before), summed over
      // directions when the pass's sources were folded
      const int pc = a.pc_map != nullptr ? a.pc_map[c] : -1;
      const double pn = pc >= 0 && a.psum != nullptr ? a.psum[(int64_t)pc * G + g] : 0.0;
      const double ka = (1.0 - (double)a.albedo) * kap;
      const double ks = (double)a.albedo * kap;
      const double ab = ka * V * js;
      a.jsum[cg] = (float)js;
      a.J[cg] = (float)(js * (double)kInv4Pi);
      a.absorbed[cg] = (float)ab;
      const double jp = a.jsum_prev != nullptr ? (double)a.jsum_prev[cg] : 0.0;
      v[0] = (double)a.emission[cg];
      v[1] = ab;
      v[2] = esc;
      v[3] = pn;
      v[4] = pout;
      v[5] = ks * V * (jp - js);
      if (a.with_e) {
        const double po = pc >= 0 && a.psum_prev != nullptr ? a.psum_prev[(int64_t)pc * G + g] : 0.0;
        const double den = pn + po;
        v[6] = den > 0.0 ? fabs(pn - po) / den : 0.0;
        v[7] = fabs(pn - po);
        v[8] = den;
      }
    }
#pragma unroll
    for (int k = 0; k < kNPart; ++k) part[k][i] = v[k];
  }
  __syncthreads();
  // the workgroup's sums, a wavefront per (quantity, group), in a fixed order
  const int lane = threadIdx.x & 63;
  for (int q = threadIdx.x >> 6; q < kNPart * G; q += kRedItems * kTeams / 64) {
    const int k = q / G, gq = q % G;
    double r = 0.0;
    for (int j = lane * G + gq; j < a.cells_per_block * G; j += 64 * G) r = k == 6 ? fmax(r, part[k][j]) : r + part[k][j];
    for (int o = 32; o > 0; o >>= 1) {
      const double x = __shfl_xor(r, o);
      r = k == 6 ? fmax(r, x) : r + x;
    }
    if (lane == 0) a.partial[((int64_t)blk * G + gq) * kNPart + k] = r;
  }
}

// One workgroup per (mesh, group): strided partial sums then a fixed-order
// tree, so the FP64 totals are reproducible.
__global__ __launch_bounds__(256) void k_totals(const double* partial, const int32_t* mesh_blk_base,
                                                int32_t n_meshes, int32_t G, double* totals) {
  __shared__ double sh[256][kNPart];
  const int t = blockIdx.x;
  const int m = t / G, g = t % G;
  double s[kNPart];
  for (int k = 0; k < kNPart; ++k) s[k] = 0.0;
  for (int b = mesh_blk_base[m] + threadIdx.x; b < mesh_blk_base[m + 1]; b += 256)
    for (int k = 0; k < kNPart; ++k) {
      const double x = partial[((int64_t)b * G + g) * kNPart + k];
      if (k == 6) s[k] = fmax(s[k], x); else s[k] += x;
    }
  for (int k = 0; k < kNPart; ++k) sh[threadIdx.x][k] = s[k];
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w)
      for (int k = 0; k < kNPart; ++k) {
        const double x = sh[threadIdx.x + w][k];
        sh[threadIdx.x][k] = k == 6 ? fmax(sh[threadIdx.x][k], x) : sh[threadIdx.x][k] + x;
      }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    double* o = totals + (int64_t)t * 8;
    for (int k = 0; k < 7; ++k) o[k] = sh[0][k];
    o[7] = sh[0][8] > 0.0 ? sh[0][7] / sh[0][8] : 0.0;
  }
}

__global__ void k_adj_init(const float* dJ, const float* dA, const float* kappa, const float* vol,
                           const float* jsum_last, float albedo, int32_t G, int64_t n,
                           float* gsrc, double* dk, double* de, int32_t* flag) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double V = (double)vol[i / G];
  const double ga = (double)dA[i];
  if (!(fabs(ga) <= DBL_MAX && fabs((double)dJ[i]) <= DBL_MAX)) atomicOr(flag, kErrGrad);
  const double ka = (1.0 - (double)albedo) * (double)kappa[i];
  gsrc[i] = (float)((double)dJ[i] * (double)kInv4Pi + ga * ka * V);
  dk[i] = ga * (1.0 - (double)albedo) * V * (double)jsum_last[i];
  de[i] = 0.0;
}

// The adjoint's direction sums.  SCHED: lambda straight from the sweep's results in schedule
// order (STORE: with its copy in cell order on the way), else from that copy.
constexpr int kAdjBatch = 8;  // directions whose loads a thread has in flight

template <bool EXP_LAW, bool SCHED, bool STORE>
__global__ __launch_bounds__(256) void k_adj_reduce(AdjReduceArgs a, double* dk, double* de) {
  const int64_t n = a.C_total * a.G;
  const int64_t i = (int64_t)(SCHED ? xcd_block(blockIdx.x, gridDim.x) : blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int c = (int)(i / a.G);
  const int g = (int)(i - (int64_t)c * a.G);
  const double V = (double)a.vol[c];
  int lo = 0, hi = a.n_meshes - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (a.mesh_off[mid] <= c) lo = mid; else hi = mid - 1;
  }
  // tasks of mesh m: [direction][local cell] from D * (first cell of m)
  const int64_t Cm = a.mesh_off[lo + 1] - a.mesh_off[lo];
  const int64_t t0 = (int64_t)a.D * a.mesh_off[lo];
  const int lc = c - a.mesh_off[lo];
  const double kap = (double)a.kappa[i];
  const double kV = kap * V;
  const double gs = EXP_LAW && a.use_g ? (double)a.gsrc[i] : 0.0;
  double ls = 0.0, dks = 0.0;
  for (int d0 = 0; d0 < a.D; d0 += kAdjBatch) {
    int p[kAdjBatch];
    float lam[kAdjBatch], phi[kAdjBatch];
#pragma unroll
    for (int k = 0; k < kAdjBatch; ++k) {  // (past the last direction: read again)
      const int d = min(d0 + k, a.D - 1);
      if (SCHED) p[k] = a.inv[t0 + d * Cm + lc];
      else lam[k] = a.lam[d * n + i];
      phi[k] = a.phi[d * n + i];
    }
    if (SCHED) {
#pragma unroll
      for (int k = 0; k < kAdjBatch; ++k)
        lam[k] = a.out_s[(t0 + min(d0 + k, a.D - 1) * Cm + p[k]) * a.G + g];
    }
#pragma unroll
    for (int k = 0; k < kAdjBatch; ++k) {
      const int d = d0 + k;
      if (d >= a.D) break;
      const double l = (double)lam[k];
      const double x = (double)phi[k];
      if (STORE) a.lam[d * n + i] = lam[k];
      ls += l;
      if (EXP_LAW) {
        // per direction: -lambda x d(den)/dkappa + g x dr/dkappa, with
        // tau < 40: d(den)/dkappa = V e^tau, dr/dkappa = h'(tau) V / Aperp;
        // tau >= 40: d(den)/dkappa = 0, dr/dkappa = -r / kappa
        const double ap = (double)a.aperp[t0 + d * Cm + lc];
        const double tau = kV / ap;
        double dden, dr;
        if (tau < kTauCap) {
          dden = V * exp(tau);
          dr = dh_dt(tau) * V / ap;
        } else {
          dden = 0.0;
          dr = -(ap * expm1(kTauCap) / kV) / kap;
        }
        dks += -l * x * dden + gs * x * dr;
      } else {
        dks += l * x;
      }
    }
  }
  if (!EXP_LAW) dks = -V * dks;
  const double prev = a.jsum_prev != nullptr ? (double)a.jsum_prev[i] : 0.0;
  const double alb = (double)a.albedo;
  const double invD = (double)a.inv_D;
  dk[i] += dks + alb * V * ls * prev * invD;
  de[i] += ls * invD;
  const double gn = alb * (double)a.kappa[i] * V * ls * invD;
  a.gsrc_next[i] = (float)(a.accumulate ? (double)a.gsrc_next[i] + gn : gn);
}

__global__ void k_d2f_pair(const double* a, const double* b, float* oa, float* ob, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) {
    oa[i] = (float)a[i];
    ob[i] = (float)b[i];
  }
}

inline unsigned grid1d(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

}  // namespace

hipError_t launch_sweep_fwd(const SweepArgs& a, int32_t gn, int32_t grid, int32_t block,
                            size_t lds, hipStream_t s) {
  return launch_sweep_t<false>(a, gn, grid, block, lds, s);
}

hipError_t launch_sweep_adj(const SweepArgs& a, int32_t gn, int32_t grid, int32_t block,
                            size_t lds, hipStream_t s) {
  return launch_sweep_t<true>(a, gn, grid, block, lds, s);
}

hipError_t launch_to_cells(const Unit* units, int32_t n_units, const int32_t* blk_base, int32_t n_blocks,
                           const int32_t* inv, const float* out_s, float* out, int64_t C_total,
                           int32_t G, hipStream_t s) {
  if (n_blocks <= 0) return hipSuccess;
  // several groups in one access where every address is a multiple of it
  const uintptr_t al = reinterpret_cast<uintptr_t>(out) | reinterpret_cast<uintptr_t>(out_s);
  auto launch = [&](auto fn) {
    hipLaunchKernelGGL(fn, dim3(n_blocks), dim3(256), 0, s, units, n_units, blk_base, inv, out_s, out,
                       C_total, G);
  };
  if (G % 4 == 0 && al % 16 == 0) launch(k_to_cells<4>);
  else if (G % 2 == 0 && al % 8 == 0) launch(k_to_cells<2>);
  else launch(k_to_cells<1>);
  return hipGetLastError();
}

hipError_t launch_prep(const PrepArgs& a, int32_t n_blocks, hipStream_t s) {
  if (n_blocks <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_prep_cells, dim3(grid1d(a.C_total * a.G, 256)), dim3(256), 0, s, a);
  if (a.law == SWEEP_LAW_EXP) hipLaunchKernelGGL(k_prep<true>, dim3(n_blocks), dim3(256), 0, s, a);
  else hipLaunchKernelGGL(k_prep<false>, dim3(n_blocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

// Calls f(kernel) for the sweep kernels of GN groups until one fails.
template <int GN, class F>
hipError_t each_sweep_g(F&& f) {
  for (auto kernel : {k_sweep<GN, false, 2>, k_sweep<GN, false, kPairs>, k_sweep<GN, true, 2>, k_sweep<GN, true, kPairs>}) {
    const hipError_t e = f((const void*)kernel);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <class F>
hipError_t each_sweep(F&& f) {
  hipError_t e;
  if ((e = each_sweep_g<1>(f)) != hipSuccess) return e;
  if ((e = each_sweep_g<2>(f)) != hipSuccess) return e;
  if ((e = each_sweep_g<3>(f)) != hipSuccess) return e;
  return each_sweep_g<4>(f);
}

hipError_t set_sweep_lds_limit(int32_t bytes) {
  return each_sweep([&](const void* kernel) {
    return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  });
}

hipError_t sweep_static_lds(size_t* bytes) {
  *bytes = 0;
  return each_sweep([&](const void* kernel) {
    hipFuncAttributes at;
    const hipError_t e = hipFuncGetAttributes(&at, kernel);
    if (e == hipSuccess) *bytes = std::max(*bytes, at.sharedSizeBytes);
    return e;
  });
}

hipError_t launch_pin(const PinArgs& a, hipStream_t s) {
  const int64_t n = (int64_t)a.n_pc * a.G;
  if (n <= 0) return hipSuccess;
  if (a.psum != nullptr && a.pval == nullptr) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_pin, dim3(grid1d(n * a.D, 256)), dim3(256), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.psum == nullptr) return e;
  hipLaunchKernelGGL(k_psum, dim3(grid1d(n, 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_reduce(const ReduceArgs& a, hipStream_t s) {
  if (a.n_blocks <= 0) return hipSuccess;
  auto pick = [&](auto e) {
    constexpr bool E = decltype(e)::value;
    return a.out_s == nullptr ? k_reduce<E, false, false> : a.phi != nullptr ? k_reduce<E, true, true> : k_reduce<E, true, false>;
  };
  auto kernel = a.law == SWEEP_LAW_EXP ? pick(std::true_type()) : pick(std::false_type());
  hipLaunchKernelGGL(kernel, dim3(a.n_blocks), dim3(kRedItems * red_teams(a.out_s != nullptr)), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_totals(const double* partial, const int32_t* mesh_blk_base, int32_t n_meshes,
                         int32_t G, double* totals, hipStream_t s) {
  hipLaunchKernelGGL(k_totals, dim3(n_meshes * G), dim3(256), 0, s, partial, mesh_blk_base,
                     n_meshes, G, totals);
  return hipGetLastError();
}

hipError_t launch_adj_init(const float* dJ, const float* dA, const float* kappa, const float* vol,
                           const float* jsum_last, float albedo, int32_t G, int64_t C,
                           float* gsrc, double* dk, double* de, int32_t* flag, hipStream_t s) {
  const int64_t n = C * G;
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_adj_init, dim3(grid1d(n, 256)), dim3(256), 0, s, dJ, dA, kappa, vol,
                     jsum_last, albedo, G, n, gsrc, dk, de, flag);
  return hipGetLastError();
}

hipError_t launch_adj_reduce(const AdjReduceArgs& a, double* dk, double* de, hipStream_t s) {
  const int64_t n = a.C_total * a.G;
  if (n <= 0) return hipSuccess;
  auto pick = [&](auto e) {
    constexpr bool E = decltype(e)::value;
    return a.out_s == nullptr ? k_adj_reduce<E, false, false>
           : a.lam != nullptr ? k_adj_reduce<E, true, true> : k_adj_reduce<E, true, false>;
  };
  auto kernel = a.law == SWEEP_LAW_EXP ? pick(std::true_type()) : pick(std::false_type());
  hipLaunchKernelGGL(kernel, dim3(grid1d(n, 256)), dim3(256), 0, s, a, dk, de);
  return hipGetLastError();
}

hipError_t launch_d2f_pair(const double* a, const double* b, float* oa, float* ob, int64_t n,
                           hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_d2f_pair, dim3(grid1d(n, 256)), dim3(256), 0, s, a, b, oa, ob, n);
  return hipGetLastError();
}

}  // namespace sweep
