// The resident-value solve kernel: dense MDPs whose value vector fits in the
// LDS of a compute unit.
//
// Every workgroup keeps a full copy of V (W = V - R in a solve) in LDS for the
// whole call, and streams the rows of its share of each batch from memory, a
// wavefront per row (or per segment of a row).  The workgroups exchange only
// the b new values of a batch, as 64-bit words that carry the value, its
// state and the number of the batch: a reader polls the words themselves, so
// a batch costs one trip through memory instead of a grid barrier (arrival,
// release, fences that write back and invalidate every L2) followed by the
// read of the new values.  Words are written and read with agent-coherent
// accesses; nothing else is shared between workgroups inside a sweep.
//
// Why it pays: the fenced grid barrier took ~5 us per batch with the stream
// of rows stopped on both sides of it, and a row was reduced over a whole
// workgroup with two workgroup barriers.  Here a wavefront issues the loads
// of its first row of the next batch before it waits for the exchange, so
// the stream goes on across batches.
//
// What bounds it: the row stream from HBM for large tables (and there the
// slower odd XCDs: 80 us of rows per batch at 8192 x 16 FP32, b = 1024, against
// 71 us on the even ones); for small ones the exchange (a store to and a load
// from the memory side, ~1.5 us) and the instructions around it (~3 us).
//
// Measured per batch against the workgroup-per-state engine with a grid
// barrier per batch: 8192 x 16, b = 1024 in FP32 96.3 -> 85.3 us (5.6 -> 6.3 TB/s
// of rows), in FP8 44.9 -> 25.2 us (3.0 -> 5.3 TB/s); 500 x 6, b = 100 26.4 ->
// 5.3 us.  Modified policy iteration of 6166 x 4 (b = 512, rows of 4-byte
// alignment) 104 -> 37.5 ms; one sweep of 64 x 4 108 -> 26 us a call; the
// FP64 correction of 4096 x 8 (b = 512) 19.2 -> 8.6 ms.

#pragma once

#include "mbdp_engines.h"

#define MBDP_GLOBAL __attribute__((address_space(1)))

namespace mbdp {

constexpr int kResQ = 1024;          // rows (state, action) of one round of a workgroup
constexpr int kResSolo = 1024;       // words of a batch of a lone workgroup (in LDS)

// LDS-only workgroup barrier: waits for this wavefront's LDS operations but
// leaves its global loads in flight (a prefetched row stays in flight).
__device__ __forceinline__ void lds_barrier() {
  __asm__ volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Sum over the wavefront by data-parallel-primitive moves inside each row of
// 16 lanes, then across the four rows; every lane gets the result.
#define MBDP_DPP_ADD(v, ctrl) \
  ((v) + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), (ctrl), 0xF, 0xF, true)))
#define MBDP_DPP_ADD_D(v, ctrl)                                                              \
  ((v) + __hiloint2double(                                                                   \
             __builtin_amdgcn_mov_dpp(__double2hiint(v), (ctrl), 0xF, 0xF, true),            \
             __builtin_amdgcn_mov_dpp(__double2loint(v), (ctrl), 0xF, 0xF, true)))
__device__ __forceinline__ double wave_sum_dpp(double v) {
  v = MBDP_DPP_ADD_D(v, 0xB1);
  v = MBDP_DPP_ADD_D(v, 0x4E);
  v = MBDP_DPP_ADD_D(v, 0x141);
  v = MBDP_DPP_ADD_D(v, 0x140);
  const int h = __double2hiint(v), l = __double2loint(v);
  double r[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    r[i] = __hiloint2double(__builtin_amdgcn_readlane(h, 16 * i), __builtin_amdgcn_readlane(l, 16 * i));
  return (r[0] + r[1]) + (r[2] + r[3]);
}
__device__ __forceinline__ float wave_sum_dpp(float v) {
  v = MBDP_DPP_ADD(v, 0xB1);   // quad_perm [1,0,3,2]
  v = MBDP_DPP_ADD(v, 0x4E);   // quad_perm [2,3,0,1]
  v = MBDP_DPP_ADD(v, 0x141);  // row_half_mirror
  v = MBDP_DPP_ADD(v, 0x140);  // row_mirror
  const int i = __float_as_int(v);
  return (__int_as_float(__builtin_amdgcn_readlane(i, 0)) +
          __int_as_float(__builtin_amdgcn_readlane(i, 16))) +
         (__int_as_float(__builtin_amdgcn_readlane(i, 32)) +
          __int_as_float(__builtin_amdgcn_readlane(i, 48)));
}

// What a workgroup computes in one batch: units (position, part) u = g, g + G,
// ... < bk << lgp; a part is a run of rpp of the state's rows.
struct alignas(16) ResBatch {
  int mode;
  int bk;                // positions of the batch
  int lgp, rpp;          // parts per position (log2), rows per unit
  int rinv;              // ceil(2^20 / rpp): r / rpp = r * rinv >> 20 for r * rpp < 2^20
  int cnt, per;          // this workgroup's units; units per workgroup of a full batch
  int round;             // units per round (their Q values share LDS)
  int lgs, sps, nc;      // segments per row (log2), steps per segment, chunks per segment
  int kb;                // first position
  int list;              // entry of the first unit in the sweep's list; -1: states are positions
  int buf;               // list buffer
  int pad[2];
};

// VT: float for the solvers (W = V - R), double for the FP64 correction (V
// itself, up to half as many states).
template <class VT>
struct ResShared {
  static constexpr int kStates = kResMaxStates * 4 / (int)sizeof(VT);
  VT V[kStates];                       // W of every state (layout ResRows::at), zero beyond n
  uint16_t pol[kResMaxStates];         // the policy (policy sweeps, MPI)
  uint16_t list[2][kResList];          // states of this workgroup's units, by sweep parity
  double q[kResQ];                     // Q of the rows of a round (their cost while segments are open)
  double seg[64];                      // segment sums of rows split over wavefronts
  unsigned cnt[kResQ];                 // finished tasks per unit of the round
  unsigned long long x[sizeof(VT) / 4 * kResSolo];  // the batch's words of a lone workgroup
  unsigned long long resid;            // max |TW - W| of an improvement pass (FP64 bits)
  double s_dv[4], s_err[4], s_resid;   // sweep statistics by communicating wavefront
  unsigned s_wabs[4];
  unsigned s_changes[4];
  int abort;
  ResBatch desc[3];                    // a full batch, the sweep's last, an improvement pass
};

template <class VT>
__device__ __forceinline__ ResShared<VT>& res_shared() {
  __shared__ ResShared<VT> sh;
  return sh;
}

template <int TASK>
struct ResValue {
  typedef float type;
};
template <>
struct ResValue<kTaskRefine> {
  typedef double type;
};

// Whether the sweeps of a call apply a policy (else the minimum).
__host__ __device__ __forceinline__ bool res_policy_sweeps(int task, int policy_sweep, int K) {
  return task == kTaskMPI || (task == kTaskSweep && policy_sweep) || (task == kTaskRefine && K > 0);
}

// A row of P as 16-byte loads.  One step of a wavefront covers kStep
// consecutive columns, kEpl per lane.  V is laid out so that the quads of V
// that a lane needs for one load sit 256 floats apart, lane by lane: 16-byte
// LDS reads without bank conflicts.
template <class T>
struct ResRows {
  static constexpr int kEpl = 16 / T::kBytes;
  static constexpr int kStep = kWave * kEpl;
  static constexpr int kQuads = kEpl / 4;
  __device__ __forceinline__ static int at(int j) {
    if constexpr (kQuads == 1) return j;
    constexpr int lg = kQuads == 2 ? 3 : 4;  // log2(kEpl)
    return (j & ~(kStep - 1)) | (((j >> 2) & (kQuads - 1)) << 8) | (((j >> lg) & 63) << 2) |
           (j & 3);
  }
};

// 16 bytes from an address that is a multiple of 4 (rows of a table whose n
// is not a multiple of 4 values start at any value).
typedef unsigned int u4a4 __attribute__((ext_vector_type(4), aligned(4)));

template <bool NT>
__device__ __forceinline__ u4 res_load(const uint8_t* p0) {
  const MBDP_GLOBAL uint8_t* p = (const MBDP_GLOBAL uint8_t*)p0;
  if constexpr (NT)
    return __builtin_nontemporal_load(reinterpret_cast<const MBDP_GLOBAL u4a4*>(p));
  else
    return *reinterpret_cast<const MBDP_GLOBAL u4a4*>(p);
}

#define MBDP_CONST __attribute__((address_space(4)))

// The arguments, read through a pointer that is made opaque once per phase:
// the compiler then loads a field where it is used instead of keeping them
// all in scalar registers across the loop (it spilled ~300 of them).
//
// A chunk of a wavefront is RC rows of U steps: RC = 1 for long rows (the
// whole wavefront streams one row at a time), several rows side by side
// where a row is only a step or two, so that one chunk's latency serves them.
template <class T, bool NT, bool TAIL, int RC, int U, class VT>
struct ResEngine {
  using Rows = ResRows<T>;
  using Shared = ResShared<VT>;
  static constexpr bool k64 = sizeof(VT) == 8;
  // 64-bit words of a value: (tag, state, FP32 value), or the two halves of
  // an FP64 value, each with the tag
  static constexpr int kWords = k64 ? 2 : 1;
  typedef VT v4 __attribute__((ext_vector_type(4)));

  struct Buf {
    u4 x[RC * U];
    int c0, c1;           // of row `lane`: the shifted cost (two halves), or the stored one (c0)
    float scale;          // BF16, FP8
    float tail[RC];       // the row's last n % 4 values (TAIL)
  };

  const MBDP_CONST KParams* p;
  Shared& sh;
  int g, G, lane, wave, nw, lgnw, ncw;  // lgnw: log2 of the wavefronts
  int n, m, bs, nsteps;   // bs: the batch size
  bool shifted;           // costs are c' (after the first re-centring)
  // (held in registers: a scalar load from the arguments where it is used
  // would add its latency to every row)
  const uint8_t* table;
  const float* rscale;
  const int* cost;        // c, or c' as pairs
  double gamma;
  unsigned long long* xch;
  unsigned phase;
  double dv, err;         // of the sweep, this lane (communicating wavefronts)
  unsigned wabs;
  Buf A, B;
  bool have;              // A and B hold the first two chunks of the next batch

  __device__ __forceinline__ void refresh() { __asm__ volatile("" : "+s"(p)); }

  __device__ __forceinline__ ResEngine(const MBDP_CONST KParams* kp, Shared& s) : p(kp), sh(s) {
    g = (int)blockIdx.x;
    G = (int)gridDim.x;
    lane = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    nw = (int)(blockDim.x >> 6);
    lgnw = 31 - __clz(nw);
    n = (int)p->n;
    m = p->m;
    bs = (int)p->b;
    if constexpr (T::kType == kF32)
      table = reinterpret_cast<const uint8_t*>(p->P);
    else
      table = static_cast<const uint8_t*>(p->pq);
    rscale = p->rscale;
    cost = reinterpret_cast<const int*>(p->c32);
    gamma = p->gamma;
    xch = p->xch;
    nsteps = (n + Rows::kStep - 1) / Rows::kStep;
    shifted = false;
    phase = 1;
    dv = err = 0.0;
    wabs = 0;
    drop_prefetch();
  }

  __device__ __forceinline__ void drop_prefetch() {
    have = false;
#pragma unroll
    for (int u = 0; u < RC * U; ++u) A.x[u] = B.x[u] = u4{0u, 0u, 0u, 0u};
    A.c0 = A.c1 = B.c0 = B.c1 = 0;
    A.scale = B.scale = 0.f;
#pragma unroll
    for (int r = 0; r < RC; ++r) A.tail[r] = B.tail[r] = 0.f;
    nta = ntb = Task{};
  }

  // ---- tasks

  // The batch shapes of the call (kind 0: full, 1: a sweep's last, 2:
  // improvement), computed once by one thread.
  __device__ __forceinline__ void describe(int kind, int smode) {
    ResBatch b{};
    const bool imp = kind == 2;
    const int nb = (n + bs - 1) / bs;
    b.mode = imp ? kModeImproveCount : smode;
    b.bk = imp ? n : (kind == 1 ? n - (nb - 1) * bs : bs);
    const int mr = b.mode == kModePolicy ? 1 : m;
    b.lgp = b.mode == kModeMin ? p->res_lgp : 0;
    b.rpp = (mr + (1 << b.lgp) - 1) >> b.lgp;
    b.rinv = ((1 << 20) + b.rpp - 1) / b.rpp;
    const int units = b.bk << b.lgp;
    b.cnt = g < units ? (units - g + G - 1) / G : 0;
    b.per = ((bs << b.lgp) + G - 1) / G;
    b.round = max(1, kResQ / b.rpp);
    // fewer row groups than wavefronts: rows are cut into segments of whole steps
    const int groups = (min(b.round, b.cnt) * b.rpp + RC - 1) / RC;
    b.lgs = 0;
    while ((groups << (b.lgs + 1)) <= nw && (2 << b.lgs) <= nsteps) ++b.lgs;
    b.sps = (nsteps + (1 << b.lgs) - 1) >> b.lgs;
    b.nc = (b.sps + U - 1) / U;
    sh.desc[kind] = b;
  }

  // Batch k of a sweep (its list from entry `first` of buffer buf), or kind 2.
  __device__ __forceinline__ ResBatch get(int kind, int k, int buf, int first) const {
    const i4* src = reinterpret_cast<const i4*>(&sh.desc[kind]);
    const i4 w[3] = {src[0], src[1], src[2]};
    ResBatch b;
    int* dst = reinterpret_cast<int*>(&b);
#pragma unroll
    for (int i = 0; i < 11; ++i) dst[i] = __builtin_amdgcn_readfirstlane(w[i / 4][i % 4]);
    const bool imp = kind == 2;
    b.kb = imp ? 0 : k * bs;
    b.list = imp || bs >= n ? -1 : first + k * b.per;
    b.buf = buf;
    return b;
  }

  __device__ __forceinline__ int tasks_of(const ResBatch& b, int units) const {
    return ((units * b.rpp + RC - 1) / RC) << b.lgs;
  }

  // This wavefront's chunks of a round of `all` tasks.
  __device__ __forceinline__ int chunks_of(const ResBatch& b, int all) const {
    const int r0 = nw - 1 - wave;
    return (all > r0 ? (all - r0 + nw - 1) >> lgnw : 0) * b.nc;
  }

  // Task t of a round: segment seg of the rows rs0 .. rs0 + RC - 1 of the
  // round's units.  Lane r % RC describes row rs0 + r.
  struct Task {
    int seg;
    int unit, row;        // of the round, of the unit
    int state, action;
    int at;               // row of the table
    bool valid, on;       // within the round; an action of the state
  };

  Task nta, ntb;          // the tasks of the chunks in A and B, while `have`

  __device__ __forceinline__ Task task(const ResBatch& b, int u0, int units, int t) const {
    Task k;
    const int grp = t >> b.lgs;
    k.seg = t - (grp << b.lgs);
    const int rows = units * b.rpp;
    const int rs0 = grp * RC + (RC > 1 ? lane & (RC - 1) : 0);
    k.valid = rs0 < rows;
    const int rs = min(rs0, rows - 1);
    k.unit = (rs * b.rinv) >> 20;
    k.row = rs - k.unit * b.rpp;
    const int u = g + (u0 + k.unit) * G;
    const int pos = u >> b.lgp;
    const int part = u - (pos << b.lgp);
    int s = b.list < 0 ? b.kb + pos : (int)sh.list[b.buf][b.list + u0 + k.unit];
    if (RC == 1) s = __builtin_amdgcn_readfirstlane(s);
    k.state = s;
    int a = b.mode == kModePolicy ? (int)sh.pol[s] : part * b.rpp + k.row;
    if (RC == 1) a = __builtin_amdgcn_readfirstlane(a);
    k.action = a;
    k.on = k.valid && a < m;
    k.at = s * m + (a < m ? a : 0);
    return k;
  }

  __device__ __forceinline__ bool whole(const ResBatch& b, int seg, int c) const {
    const int st0 = seg * b.sps + c * U;
    return st0 + U <= min(seg * b.sps + b.sps, nsteps) && (st0 + U) * 1024 <= n * T::kBytes;
  }

  // Every chunk issues the same number of loads, so that the wait for a chunk
  // leaves the next one in flight.  One address per four steps where the
  // chunk is whole (the rest in the instruction's offset field; opaque, so
  // that no address is kept across the loop); otherwise addresses past the
  // row are moved to its last 16 bytes (those past the segment but inside the
  // row bring the next segment's steps), and consume() drops the values.
  __device__ __forceinline__ void load(const ResBatch& b, const Task& t, int c, Buf& f) const {
    const int st0 = t.seg * b.sps + c * U;
    const size_t rbytes = (size_t)n * T::kBytes;
    const int off = st0 * 1024 + lane * 16;  // a step is 1024 bytes of the row
    const uint8_t* base[RC];
#pragma unroll
    for (int r = 0; r < RC; ++r)
      base[r] = table + (size_t)(RC == 1 ? t.at : __builtin_amdgcn_readlane(t.at, r)) * rbytes;
    if (U >= 4 && whole(b, t.seg, c)) {
#pragma unroll
      for (int r = 0; r < RC; ++r) {
        const uint8_t* at[(U + 3) / 4];
#pragma unroll
        for (int u = 0; u < U / 4; ++u) {
          at[u] = base[r] + off + u * 4096;
          __asm__ volatile("" : "+v"(at[u]));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) f.x[r * U + u] = res_load<NT>(at[u / 4] + (u % 4) * 1024);
      }
    } else {
      const int end = n * T::kBytes - 16;  // n * kBytes >= 16
#pragma unroll
      for (int r = 0; r < RC; ++r)
#pragma unroll
        for (int u = 0; u < U; ++u) {
          f.x[r * U + u] = res_load<NT>(base[r] + min(off + u * 1024, end));
          if ((r * U + u) % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
    }
    if constexpr (TAIL) {
#pragma unroll
      for (int r = 0; r < RC; ++r)
        f.tail[r] = reinterpret_cast<const float*>(base[r])[min((n & ~3) + lane, n - 1)];
    }
    const int* ca = cost + (shifted ? 2 * (size_t)t.at : (size_t)t.at);
    f.c0 = ca[0];
    f.c1 = ca[shifted ? 1 : 0];
    if constexpr (T::kType != kF32) f.scale = rscale[t.at];
  }

  // Sums of a task: four per row where one row is streamed (their order
  // is that of the columns of a lane mod 4), one per row otherwise.
  static constexpr int kAcc = RC == 1 ? 4 : RC;

  __device__ __forceinline__ static void step(const u4& x, const v4* v, VT (&acc)[kAcc], int r) {
    if constexpr (k64) {  // FP32 rows
      acc[RC == 1 ? 0 : r] = fma((double)__uint_as_float(x.x), v[0].x, acc[RC == 1 ? 0 : r]);
      acc[RC == 1 ? 1 : r] = fma((double)__uint_as_float(x.y), v[0].y, acc[RC == 1 ? 1 : r]);
      acc[RC == 1 ? 2 : r] = fma((double)__uint_as_float(x.z), v[0].z, acc[RC == 1 ? 2 : r]);
      acc[RC == 1 ? 3 : r] = fma((double)__uint_as_float(x.w), v[0].w, acc[RC == 1 ? 3 : r]);
    } else if constexpr (T::kType == kF32) {
      acc[RC == 1 ? 0 : r] = fmaf(__uint_as_float(x.x), v[0].x, acc[RC == 1 ? 0 : r]);
      acc[RC == 1 ? 1 : r] = fmaf(__uint_as_float(x.y), v[0].y, acc[RC == 1 ? 1 : r]);
      acc[RC == 1 ? 2 : r] = fmaf(__uint_as_float(x.z), v[0].z, acc[RC == 1 ? 2 : r]);
      acc[RC == 1 ? 3 : r] = fmaf(__uint_as_float(x.w), v[0].w, acc[RC == 1 ? 3 : r]);
    } else {
#pragma unroll
      for (int w = 0; w < 4; ++w) T::fma_word(x[w], w, v, acc[RC == 1 ? w : r]);
    }
  }

  // acc += chunk c of the task's segment times V
  __device__ __forceinline__ void consume(const ResBatch& b, const Task& t, int c, const Buf& f,
                                          VT (&acc)[kAcc]) const {
    const int st0 = t.seg * b.sps + c * U;
    if (U >= 4 && whole(b, t.seg, c)) {
      const VT* vb = sh.V + st0 * Rows::kStep + lane * 4;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        v4 v[Rows::kQuads];
#pragma unroll
        for (int q = 0; q < Rows::kQuads; ++q)
          v[q] = *reinterpret_cast<const v4*>(vb + u * Rows::kStep + q * 256);
#pragma unroll
        for (int r = 0; r < RC; ++r) step(f.x[r * U + u], v, acc, r);
        if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // four steps' V at a time in registers
      }
    } else {
      const int st1 = min(t.seg * b.sps + b.sps, nsteps);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int st = min(st0 + u, nsteps - 1);
        const bool ok = st0 + u < st1 && st * 1024 + lane * 16 <= n * T::kBytes - 16;
        v4 v[Rows::kQuads];
#pragma unroll
        for (int q = 0; q < Rows::kQuads; ++q)
          v[q] = *reinterpret_cast<const v4*>(sh.V + st * Rows::kStep + lane * 4 + q * 256);
        // What a lane drops must not meet V: 0 times an infinite value is not 0.
        // One FP32 row: zeros all the same, and finish_task() takes a sum that
        // is NaN again; otherwise the lane skips the step.  (Each the faster
        // one: 6166 x 4, b = 512, 37.4 ms with zeros, 37.8 with the skip, 37.5
        // with zeros in the place of V; 500 x 6 2.96 ms with the skip, 3.03 with
        // zeros, the FP64 correction of 4096 x 8 8.6 and 8.7.)
        if constexpr (kRetake) {
          step(ok ? f.x[u] : u4{0u, 0u, 0u, 0u}, v, acc, 0);
        } else if (ok) {
#pragma unroll
          for (int r = 0; r < RC; ++r) step(f.x[r * U + u], v, acc, r);
        }
        if (u % 4 == 3) __builtin_amdgcn_sched_barrier(0);
      }
    }
    if constexpr (TAIL) {
      const int s0 = t.seg * b.sps;  // (a segment past the row's end has none of it)
      if (c == b.nc - 1 && s0 < nsteps && s0 + b.sps >= nsteps) {
        const int jt = (n & ~3) + lane;
        const VT v = jt < n ? sh.V[jt] : (VT)0;
#pragma unroll
        for (int r = 0; r < RC; ++r)
          acc[RC == 1 ? 0 : r] = fma(jt < n ? (VT)f.tail[r] : (VT)0, v, acc[RC == 1 ? 0 : r]);
      }
    }
  }

  // Where consume() multiplies what it drops by 0, NaN where V is infinite.
  static constexpr bool kRetake = RC == 1 && Rows::kQuads == 1 && !k64;

  // The task's segment times V, without products of columns that are not its own.
  __device__ __forceinline__ VT retake(const ResBatch& b, const Task& t) const {
    const uint8_t* base = table + (size_t)t.at * (size_t)n * T::kBytes;
    const int s0 = t.seg * b.sps, s1 = min(s0 + b.sps, nsteps);
    VT acc[kAcc];
#pragma unroll
    for (int i = 0; i < kAcc; ++i) acc[i] = 0;
#pragma unroll 1
    for (int st = s0; st < s1; ++st) {
      if (st * 1024 + lane * 16 > n * T::kBytes - 16) continue;
      const v4 v[1] = {*reinterpret_cast<const v4*>(sh.V + st * Rows::kStep + lane * 4)};
      step(res_load<NT>(base + st * 1024 + lane * 16), v, acc, 0);
    }
    const int jt = (n & ~3) + lane;
    if (TAIL && s0 < nsteps && s0 + b.sps >= nsteps && jt < n)
      acc[0] = fma((VT)reinterpret_cast<const float*>(base)[jt], sh.V[jt], acc[0]);
    return wave_sum_dpp((acc[0] + acc[1 % kAcc]) + (acc[2 % kAcc] + acc[3 % kAcc]));
  }

  // The segment's sums are complete: their share of Q goes to LDS, and the
  // wavefront that completes a unit finds the unit's minimum and publishes it.
  __device__ __forceinline__ void finish_task(const ResBatch& b, int u0, const Task& t,
                                              const Buf& f, const VT (&acc)[kAcc]) {
    VT sum;
    if constexpr (RC == 1) {
      sum = wave_sum_dpp((acc[0] + acc[1]) + (acc[2] + acc[3]));
    } else {
      sum = (VT)0;
#pragma unroll
      for (int r = 0; r < RC; ++r) {
        const VT x = wave_sum_dpp(acc[r]);
        sum = lane == r ? x : sum;
      }
    }
    if constexpr (kRetake) {
      if (__builtin_expect(__builtin_isnan(sum), 0)) sum = retake(b, t);
    }
    const double part = T::kType == kF32 ? (double)sum : (double)sum * (double)f.scale;
    const double c = shifted ? __hiloint2double(f.c1, f.c0) : (double)__int_as_float(f.c0);
    const double q1 = t.on ? c + gamma * part : (double)INFINITY;  // of an unsplit row
    const int S = 1 << b.lgs, tasks = b.rpp * S;
    const bool pol = b.mode == kModePolicy;
    const bool mine = lane < RC && t.valid;  // this lane's row is one of the task's
    if (tasks == 1) {
      if (mine) publish(b, u0 + t.unit, t.state, pol || q1 < INFINITY ? q1 : (double)INFINITY, t.action);
      return;
    }
    unsigned prev = 0;
    if (mine) {
      const int qi = t.unit * b.rpp + t.row;
      if (S == 1) {
        sh.q[qi] = q1;
      } else {
        sh.seg[qi * S + t.seg] = part;
        if (t.seg == 0) sh.q[qi] = t.on ? c : (double)INFINITY;
      }
      __asm__ volatile("" ::: "memory");
      prev = atomicAdd(&sh.cnt[t.unit], 1u);  // LDS operations of a wavefront stay in order
    }
    unsigned long long done = __ballot(mine && prev == (unsigned)(tasks - 1));
    while (done) {  // the units this task completed
      const int l = __ffsll((unsigned long long)done) - 1;
      done &= done - 1;
      const int unit = __builtin_amdgcn_readlane(t.unit, l);
      const int state = __builtin_amdgcn_readlane(t.state, l);
      const int act = __builtin_amdgcn_readlane(t.action, l);
      const int a0 = act - __builtin_amdgcn_readlane(t.row, l);
      __asm__ volatile("" ::: "memory");
      if (lane == 0) sh.cnt[unit] = 0u;
      double qb = INFINITY;
      int ab = 0x7fffffff;
      for (int r = lane; r < b.rpp; r += kWave) {
        double q = sh.q[unit * b.rpp + r];
        if (S > 1) {
          double sum2 = 0.0;
          for (int s = 0; s < S; ++s) sum2 += sh.seg[(unit * b.rpp + r) * S + s];
          q += gamma * sum2;
        }
        if (pol || q < qb) {  // ascending actions: strictly smaller keeps the lowest
          qb = q;
          ab = pol ? act : a0 + r;
        }
      }
      for (int o = 1; o < b.rpp && o < kWave; o <<= 1) {
        const double q2 = __shfl_xor(qb, o);
        const int a2 = __shfl_xor(ab, o);
        if (q2 < qb || (q2 == qb && a2 < ab)) {
          qb = q2;
          ab = a2;
        }
      }
      if (ab == 0x7fffffff) ab = 0;
      if (lane == 0) publish(b, u0 + unit, state, qb, ab);
    }
  }

  // The unit's result to the workgroups (and to the caller's arrays), by one lane.
  __device__ __forceinline__ void publish(const ResBatch& b, int i, int s, double q, int a) {
    const int u = g + i * G;
    unsigned long long w, w2 = 0;
    if (b.mode >= kModeImprove) {
      const double old = (double)sh.V[Rows::at(s)];
      const double d = fabs(q - old);
      if (d == d) atomicMax(&sh.resid, (unsigned long long)__double_as_longlong(d));
      if (p->policy) p->policy[s] = a;
      w = ((unsigned long long)(phase & 0x7FFFFFFFu) << 32) | (unsigned)a;
    } else {
      if (p->argmin_out && b.lgp == 0) p->argmin_out[s] = a;
      const unsigned long long head =
          (unsigned long long)(0x80000000u | ((phase & 0x7FFu) << 20) | (unsigned)s) << 32;
      if constexpr (k64) {
        w = head | (unsigned)__double2loint(q);
        w2 = head | (unsigned)__double2hiint(q);
      } else {
        w = head | __float_as_uint((float)q);
      }
    }
    if (G == 1) {
      sh.x[u] = w;
      if (k64) sh.x[kResSolo + u] = w2;
    } else {
      unsigned long long* to = words_of(phase);
      atomic_store_agent(&to[u], w);
      if (k64 && b.mode < kModeImprove) atomic_store_agent(&to[n + u], w2);
    }
  }

  // The phase's words: [kWords][n], by phase parity.
  __device__ __forceinline__ unsigned long long* words_of(unsigned ph) const {
    return xch + (size_t)(ph & 1) * kWords * n;
  }

  // Streams this workgroup's units of the batch, then requests the first two
  // chunks of the batch that ahead(next) finds, if it says so (not the
  // communicating wavefronts, whose polling would wait for them).  Finding it
  // here keeps its LDS reads and arguments off the path from one exchange to
  // the next.
  template <class Ahead>
  __device__ __forceinline__ void compute(const ResBatch& b, const Ahead& ahead, ResBatch& next) {
    const int r0 = nw - 1 - wave;  // the communicating wavefronts get the last tasks
    for (int u0 = 0; u0 < b.cnt; u0 += b.round) {
      const int units = min(b.round, b.cnt - u0);
      const int all = tasks_of(b, units);
      const int C = chunks_of(b, all);
      const bool loaded = have && u0 == 0;
      if (C > 0) {
        VT acc[kAcc];
#pragma unroll
        for (int i = 0; i < kAcc; ++i) acc[i] = 0.f;
        // (the tasks of requested chunks were found with them)
        Task ta = loaded ? nta : task(b, u0, units, r0), tb = ntb;
        int i = 0, c = 0;  // task and chunk that were requested last
        int x = 0;         // their number
        const auto advance = [&](Task& to, const Task& from) {
          to = from;
          if (++x >= C) return;  // nothing is left: the last chunk again
          if (++c == b.nc) {
            c = 0;
            ++i;
            to = task(b, u0, units, r0 + i * nw);
          }
        };
        const auto use = [&](const Task& t, int ct, const Buf& f) {
          consume(b, t, ct, f, acc);
          if (ct == b.nc - 1) {
            finish_task(b, u0, t, f, acc);
#pragma unroll
            for (int i2 = 0; i2 < kAcc; ++i2) acc[i2] = 0.f;
          }
        };
        // A and B in turn, each requested again as soon as it is used: the
        // loads of one or two chunks are in flight all the time.  No load
        // here is conditional: the compiler could not count past it and
        // would wait for both.
        int ca = 0, cb;
        if (loaded) {
          if (++x < C && ++c == b.nc) {
            c = 0;
            ++i;
          }
          cb = c;
        } else {
          advance(tb, ta);
          cb = c;
          load(b, ta, 0, A);
          load(b, tb, cb, B);
        }
        int left = C;
        while (left > 2) {
          use(ta, ca, A);
          advance(ta, tb);
          ca = c;
          load(b, ta, ca, A);
          use(tb, cb, B);
          advance(tb, ta);
          cb = c;
          load(b, tb, cb, B);
          left -= 2;
        }
        use(ta, ca, A);
        if (left == 2) use(tb, cb, B);
      }
      if (u0 + b.round < b.cnt) lds_barrier();  // the round's LDS is reused
    }
    have = false;
    refresh();
    const bool has_next = ahead(next);
    if (has_next && wave >= ncw) {
      const int units = min(next.round, next.cnt);
      const int all = tasks_of(next, units);
      if (r0 < all) {
        nta = task(next, 0, units, r0);
        load(next, nta, 0, A);
        ntb = nta;
        const bool second = next.nc == 1 && r0 + nw < all;  // the second chunk is the next task's
        if (second) ntb = task(next, 0, units, r0 + nw);
        load(next, ntb, next.nc > 1 ? 1 : 0, B);
        have = true;
      }
    }
    // The words a short last batch (or a batch of fewer units than workgroups)
    // leaves unused are written all the same: every workgroup is waited for
    // in every phase, so none overwrites a word that another still reads, and
    // a word is at most two phases old.
    if (G > 1 && b.mode < kModeImprove && wave == nw - 1) {
      const int all = sweep_words(b.lgp);
      const unsigned long long w =
          (unsigned long long)(0x80000000u | ((phase & 0x7FFu) << 20)) << 32;
      for (int u = g + b.cnt * G + lane * G; u < all; u += kWave * G) {
        atomic_store_agent(&words_of(phase)[u], w);
        if (k64) atomic_store_agent(&words_of(phase)[n + u], w);
      }
    }
  }

  // Words of a sweep phase, read and written whatever the batch uses of them.
  __device__ __forceinline__ int sweep_words(int lgp) const { return max(bs << lgp, G); }

  // ---- exchange

  // Words base + j * stride, j < J, of the first H planes of the phase; false
  // on abort.  (Polls back to back: a pause of 128 cycles between them cost 2%
  // at 500 x 6, b = 100; a second poll in flight, half a round trip behind,
  // 4%.)
  template <int J, int H>
  __device__ __forceinline__ bool fetch(const ResBatch& b, int base, int stride, int limit,
                                        unsigned long long (&w)[H][J]) {
    const bool imp = b.mode >= kModeImprove;
    const unsigned want = imp ? (phase & 0x7FFFFFFFu) : (0x800u | (phase & 0x7FFu));
    if (G == 1) {
#pragma unroll
      for (int h = 0; h < H; ++h)
#pragma unroll
        for (int j = 0; j < J; ++j) {
          const int i = base + j * stride;
          w[h][j] = sh.x[h * kResSolo + (i < limit ? i : 0)];
        }
      return true;
    }
    const unsigned long long* src = words_of(phase);
    const auto request = [&](unsigned long long (&x)[H][J]) {
#pragma unroll
      for (int h = 0; h < H; ++h)
#pragma unroll
        for (int j = 0; j < J; ++j) {
          const int i = base + j * stride;
          x[h][j] = atomic_load_agent(src + (size_t)h * n + (i < limit ? i : 0));
        }
    };
    const auto complete = [&](const unsigned long long (&x)[H][J]) {
      bool ok = true;
#pragma unroll
      for (int h = 0; h < H; ++h)
#pragma unroll
        for (int j = 0; j < J; ++j) {
          const int i = base + j * stride;
          const unsigned hi = (unsigned)(x[h][j] >> 32);
          ok = ok && (i >= limit || (imp ? hi : hi >> 20) == want);
        }
      return (bool)__all(ok);
    };
    unsigned long long t0 = 0;
    for (int spin = 0;; ++spin) {
      request(w);
      if (complete(w)) return true;
      if (!keep_waiting(spin, t0)) return false;
    }
  }

  __device__ __forceinline__ bool keep_waiting(int spin, unsigned long long& t0) {
    if ((spin & 15) == 15) {
      if (__hip_atomic_load(&p->ctl->abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return false;
      const unsigned long long now = wall_clock64();
      if (t0 == 0) t0 = now;
      if (now - t0 > p->timeout_ticks) {
        if (lane == 0) raise_abort(p->ctl, kDevBarrierTimeout);
        return false;
      }
    }
    return true;
  }

  // J words of each lane from i0 on, to this workgroup's V (or policy).
  template <int J>
  __device__ __forceinline__ bool take(const ResBatch& b, int i0, int stride, int used, int words,
                                       unsigned& changes) {
    unsigned long long v0[kWords][J];
    unsigned long long (&w)[J] = v0[0];
    unsigned long long (&w2)[J] = v0[kWords - 1];
    if (k64 && b.mode >= kModeImprove) {  // one plane only
      unsigned long long x[1][J];
      if (!fetch<J, 1>(b, i0 + lane, stride, words, x)) return false;
#pragma unroll
      for (int j = 0; j < J; ++j) w[j] = x[0][j];
    } else if (!fetch<J, kWords>(b, i0 + lane, stride, words, v0)) {
      return false;
    }
    if (b.mode >= kModeImprove) {
#pragma unroll
      for (int j = 0; j < J; ++j) {
        const int i = i0 + j * stride + lane;
        if (i < used) {
          if (k64 && p->vref) err = fmax(err, fabs((double)sh.V[i] - p->vref[i]));
          const uint16_t a = (uint16_t)(unsigned)w[j];
          changes += sh.pol[i] != a;
          sh.pol[i] = a;
        }
      }
      return true;
    }
    const int part = (1 << b.lgp) - 1;
    if (b.lgp) {
      for (int off = 1; off <= part; off <<= 1)
#pragma unroll
        for (int j = 0; j < J; ++j) {
          if constexpr (k64) {
            const double v = __hiloint2double((int)w2[j], (int)w[j]);
            const double q = fmin(v, __shfl_xor(v, off));
            w[j] = (w[j] & 0xFFFFFFFF00000000ull) | (unsigned)__double2loint(q);
            w2[j] = (unsigned)__double2hiint(q);
          } else {
            const float v = __uint_as_float((unsigned)w[j]);
            const float o = __shfl_xor(v, off);
            w[j] = (w[j] & 0xFFFFFFFF00000000ull) | __float_as_uint(fminf(v, o));
          }
        }
    }
    VT old[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {  // (an unused word's state is read too, and dropped)
      const int s = (int)((unsigned)(w[j] >> 32) & 0xFFFFFu);
      old[j] = sh.V[Rows::at(min(s, n - 1))];
    }
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int i = i0 + j * stride + lane;
      if (i < used && (i & part) == 0) {
        const int s = (int)((unsigned)(w[j] >> 32) & 0xFFFFFu);
        VT v;
        if constexpr (k64)
          v = __hiloint2double((int)w2[j], (int)w[j]);
        else
          v = __uint_as_float((unsigned)w[j]);
        sh.V[Rows::at(s)] = v;
        dv = fmax(dv, fabs((double)v - (double)old[j]));
        if (p->vref) err = fmax(err, fabs((double)v - (shifted ? p->tgt[s] : p->vref[s])));
        if constexpr (!k64) wabs = max(wabs, __float_as_uint(v) & 0x7FFFFFFFu);
      }
    }
    return true;
  }

  // Communicating wavefronts of a phase of `words` words: they prefetch no
  // rows (a poll would wait for them), so no more than read the words in one
  // round trip.
  __device__ __forceinline__ int comm_waves(int words) const {
    return nw < 8 ? 1 : (words <= 512 ? 1 : (words <= 1024 ? 2 : 4));
  }

  // Commits the batch's words.
  __device__ __forceinline__ bool receive(const ResBatch& b) {
    const int used = b.bk << b.lgp;
    const int words = G == 1 || b.mode >= kModeImprove ? used : sweep_words(b.lgp);
    const int stride = ncw * kWave;
    unsigned changes = 0;
    if (words <= 4 * stride) {
      if (!take<4>(b, wave * kWave, stride, used, words, changes)) return false;
    } else {
      for (int i0 = wave * kWave; i0 < words; i0 += 8 * stride)
        if (!take<8>(b, i0, stride, used, words, changes)) return false;
    }
    if (b.mode >= kModeImprove) {
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) changes += __shfl_xor(changes, off);
      if (lane == 0) sh.s_changes[wave] = changes;
      if (wave == 0) return exchange_resid();
    }
    return true;
  }

  // max over the workgroups of sh.resid (FP64), by wavefront 0.
  __device__ __forceinline__ bool exchange_resid() {
    unsigned long long mine = sh.resid;
    if (lane == 0) sh.resid = 0ull;
    if (G > 1) {
      unsigned long long* rec = p->ctl->bar_slots + kMaxBlocks / 2 + (size_t)(phase & 1) * 2 * G;
      if (lane < 2)
        atomic_store_agent(&rec[2 * g + lane], ((unsigned long long)phase << 32) |
                                                   (lane ? mine >> 32 : mine & 0xFFFFFFFFull));
      unsigned long long best = mine;
      for (int i0 = 0; i0 < G; i0 += kWave) {
        const int i = min(i0 + lane, G - 1);
        unsigned long long lo, hi, t0 = 0;
        for (int spin = 0;; ++spin) {
          lo = atomic_load_agent(&rec[2 * i]);
          hi = atomic_load_agent(&rec[2 * i + 1]);
          if (__all((unsigned)(lo >> 32) == phase && (unsigned)(hi >> 32) == phase)) break;
          if (!keep_waiting(spin, t0)) return false;
        }
        const unsigned long long v = ((hi & 0xFFFFFFFFull) << 32) | (lo & 0xFFFFFFFFull);
        best = v > best ? v : best;
      }
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) {
        const unsigned long long o = __shfl_xor(best, off);
        best = o > best ? o : best;
      }
      mine = best;
    }
    if (lane == 0) sh.s_resid = __longlong_as_double((long long)mine);
    return true;
  }

  // ---- the sweep order

  // feistel() of mbdp_device.h with the outer loop kept (fewer registers), one
  // 64-bit product where a round needs both halves, and the sweep per lane.
  __device__ __forceinline__ static uint32_t feistel_at(uint32_t x, const OrderKey& k, uint64_t t) {
    uint32_t left = x >> k.h, right = x & k.mask;
#pragma unroll 1
    for (uint32_t j = 0; j < 4; ++j) {
      uint32_t x0 = right, x1 = j, x2 = (uint32_t)t, x3 = (uint32_t)(t >> 32);
      uint32_t k0 = k.s_lo, k1 = k.s_hi;
#pragma unroll
      for (int r = 0; r < 10; ++r) {
        const uint64_t a = (uint64_t)0xD2511F53u * x0, b = (uint64_t)0xCD9E8D57u * x2;
        x0 = (uint32_t)(b >> 32) ^ x1 ^ k0;
        x1 = (uint32_t)b;
        x2 = (uint32_t)(a >> 32) ^ x3 ^ k1;
        x3 = (uint32_t)a;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
      }
      const uint32_t nr = left ^ (x0 & k.mask);
      left = right;
      right = nr;
    }
    return (left << k.h) | right;
  }

  // The order is drawn for `span` sweeps at a time, into one of two list
  // buffers: with few units per sweep a lane per entry would leave most lanes
  // idle, and an evaluation of the network takes ~1 us whatever the number of
  // lanes.  Entry e of a sweep's list is unit (e % per) of batch e / per; lanes
  // walk the network for one entry at a time, `passes` evaluations per phase
  // (all that is left when `rest`), so the work hides behind the exchanges of
  // the span before.
  int span, entries;  // sweeps per span, entries per sweep
  int ord_e;
  uint32_t ord_y;
  __device__ __forceinline__ int ord_entries() const {
    const int per = (((int)p->b << list_lgp()) + G - 1) / G;
    return (int)((n + p->b - 1) / p->b) * per;
  }
  __device__ __forceinline__ int list_lgp() const {
    return res_policy_sweeps(p->task, p->policy_sweep, p->K) ? 0 : p->res_lgp;
  }
  __device__ __forceinline__ int ord_position(int e) const {  // -1: no such unit
    const int lgp = list_lgp();
    const int per = (((int)p->b << lgp) + G - 1) / G;
    const int k = e / per, i = e - k * per;
    const int kb = k * (int)p->b, bk = min((int)p->b, n - kb);
    const int u = g + i * G;
    return u < (bk << lgp) ? kb + (u >> lgp) : -1;
  }
  __device__ __forceinline__ void ord_skip(int all, int lanes) {
    while (ord_e < all) {
      const int pos = ord_position(ord_e % entries);
      if (pos >= 0) {
        ord_y = (uint32_t)pos;
        return;
      }
      ord_e += lanes;
    }
  }
  // lanes of the order work: the workgroup's last wavefronts first
  __device__ __forceinline__ int ord_lanes(int all, int waves) const {
    const int w = min(waves, (all + kWave - 1) / kWave);
    return w * kWave;
  }
  __device__ __forceinline__ void ord_start(int lanes) {
    const int all = span * entries;
    ord_e = (nw - 1 - wave) * kWave + lane;
    if (ord_e >= lanes) ord_e = all;
    ord_skip(all, lanes);
  }
  // t: the span's first sweep
  __device__ __forceinline__ void ord_run(uint64_t t, int buf, int passes, bool rest, int lanes) {
    const int all = span * entries;
    if (!__any(ord_e < all)) return;
    const OrderKey key = make_order_key(n, p->seed, 0);
    for (int i = 0; (rest || i < passes) && __any(ord_e < all); ++i) {
      if (ord_e < all) {
        ord_y = feistel_at(ord_y, key, t + (uint64_t)(ord_e / entries));
        if (ord_y < key.n) {
          sh.list[buf][ord_e] = (uint16_t)ord_y;
          ord_e += lanes;
          ord_skip(all, lanes);
        }
      }
    }
  }

  // ---- a phase

  // One batch or improvement pass: compute, exchange, commit.  ahead(next)
  // finds the batch that follows; true if its first rows may be requested early.
  // order_for: list buffer the order from sweep order_t on is written to, `passes`
  // evaluations of it now or (passes < 0) all that is left; -1: none.
  template <class Ahead>
  __device__ __forceinline__ bool run(const ResBatch& b, const Ahead& ahead, ResBatch& next,
                                      bool last, uint64_t order_t, int order_for, int passes,
                                      int lanes) {
    compute(b, ahead, next);
    lds_barrier();  // every unit of this workgroup is published, V is no longer read
    if (wave < ncw) {
      const bool ok = receive(b);
      if (last) {
        const double d = wave_max_d(dv);
        const double e = p->vref ? wave_max_d(err) : 0.0;
        unsigned w = wabs;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) w = max(w, (unsigned)__shfl_xor((int)w, off));
        if (lane == 0) {
          sh.s_dv[wave] = d;
          sh.s_err[wave] = e;
          sh.s_wabs[wave] = w;
        }
      }
      if (!ok && lane == 0) sh.abort = 1;
    } else if (order_for >= 0) {
      ord_run(order_t, order_for, passes, passes < 0, lanes);
    }
    lds_barrier();
    if (sh.abort) return false;
    ++phase;
    return true;
  }

  __device__ __forceinline__ double sweep_dv() const {
    double d = sh.s_dv[0];
    for (int i = 1; i < ncw; ++i) d = fmax(d, sh.s_dv[i]);
    return d;
  }
  __device__ __forceinline__ double sweep_err() const {
    double d = sh.s_err[0];
    for (int i = 1; i < ncw; ++i) d = fmax(d, sh.s_err[i]);
    return d;
  }
  __device__ __forceinline__ float sweep_wabs() const {
    unsigned d = sh.s_wabs[0];
    for (int i = 1; i < ncw; ++i) d = max(d, sh.s_wabs[i]);
    return __uint_as_float(d);
  }

  // c'(s,a) = c(s,a) - R(s) + gamma (P R)(s,a) in FP64, a wavefront per row; R
  // (FP64) in LDS in the place of V where it fits.
  __device__ __forceinline__ void shift_rows() {
    constexpr int F = 4;  // steps in flight
    const double* R = p->shift;
    const bool staged = 2 * n <= kResMaxStates;
    double* lr = reinterpret_cast<double*>(sh.V);
    if (staged)
      for (int j = (int)threadIdx.x; j < n; j += (int)blockDim.x) lr[j] = R[j];
    __syncthreads();
    const int rows = n * m, end = n * T::kBytes - 16;
#pragma unroll 1
    for (int r = g * nw + wave; r < rows; r += G * nw) {
      const uint8_t* base = table + (size_t)r * (size_t)n * T::kBytes;
      double acc = 0.0;
      if (TAIL && (n & ~3) + lane < n) {
        const int j = (n & ~3) + lane;
        acc = (double)reinterpret_cast<const float*>(base)[j] * (staged ? lr[j] : R[j]);
      }
#pragma unroll 1
      for (int st = 0; st < nsteps; st += F) {
        u4 x[F];
#pragma unroll
        for (int u = 0; u < F; ++u) x[u] = res_load<NT>(base + min((st + u) * 1024 + lane * 16, end));
#pragma unroll
        for (int u = 0; u < F; ++u) {
          const int off = (st + u) * 1024 + lane * 16;
          if (off > end) continue;
          const int j = off / T::kBytes;
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            f4 d;  // the values of word w
            constexpr int per = 4 / T::kBytes;
            if constexpr (T::kType == kF32) d.x = __uint_as_float(x[u][w]);
            if constexpr (T::kType == kBF16) {
              d.x = bf16_lo(x[u][w]);
              d.y = bf16_hi(x[u][w]);
            }
            if constexpr (T::kType == kFP8) d = fp8x4(x[u][w]);
#pragma unroll
            for (int e = 0; e < per; ++e)
              acc = fma((double)d[e], staged ? lr[j + w * per + e] : R[j + w * per + e], acc);
          }
        }
      }
      acc = wave_sum_d(acc);
      if (lane == 0) {
        float scale = 1.f;
        if constexpr (T::kType != kF32) scale = rscale[r];
        p->ceff[r] = (double)p->c32[r] - R[r / m] + p->gamma * (acc * (double)scale);
      }
    }
    __syncthreads();
  }

  // Folds W into the anchor and rebuilds the shifted costs (two grid barriers).
  __device__ __forceinline__ bool recentre(GridBarrier& gb) {
    for (int s = (int)(blockIdx.x * blockDim.x + threadIdx.x); s < n; s += (int)(gridDim.x * blockDim.x)) {
      const double r = (shifted ? p->shift[s] : 0.0) + (double)sh.V[Rows::at(s)];
      p->shift[s] = r;
      if (p->vref) p->tgt[s] = p->vref[s] - r;
    }
    if (!grid_sync(gb)) return false;
    shift_rows();
    for (int i = (int)threadIdx.x; i < nsteps * Rows::kStep; i += (int)blockDim.x) sh.V[i] = 0.f;
    shifted = true;
    cost = reinterpret_cast<const int*>(p->ceff);
    drop_prefetch();  // its costs are the old ones
    return grid_sync(gb);
  }
};

// Task of the kernel: a solver's, or the FP64 correction.
template <class T, bool NT, bool TAIL, int RC, int U, int TASK>
__global__ void __launch_bounds__(kResThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
resident_kernel(KParams kp) {
  using VT = typename ResValue<TASK>::type;
  ResShared<VT>& sh = res_shared<VT>();
  using Eng = ResEngine<T, NT, TAIL, RC, U, VT>;
  using Rows = typename Eng::Rows;
  Eng e((const MBDP_CONST KParams*)__builtin_amdgcn_kernarg_segment_ptr(), sh);
  const MBDP_CONST KParams*& p = e.p;
  const int n = e.n, tid = (int)threadIdx.x, nt = (int)blockDim.x;
  GridBarrier gb{p->ctl, 0, gridDim.x, p->timeout_ticks};
  uint64_t t = p->first_sweep;

  // prologue: V, the policy, the first sweep's order.  A workgroup that finds a
  // bad entry of the caller's order or policy leaves before its first batch:
  // the others wait for its words there and leave too, V untouched.
  bool bad_entry = false;
  if (blockIdx.x == 0 && tid == 0 && p->dv_out) *p->dv_out = 0.f;  // what a failed call leaves
  if (gridDim.x == 1 && tid == 0) {  // a lone workgroup clears its own status words
    store_shared(&p->ctl->abort, 0u);
    store_shared(&p->ctl->error, 0u);
    // performed before any error is raised (after the workgroup barrier below)
    __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  for (int i = tid; i < kResQ; i += nt) sh.cnt[i] = 0u;
  if (tid == 0) {
    sh.resid = 0ull;
    sh.abort = 0;
  }
  for (int j = tid; j < e.nsteps * Rows::kStep; j += nt) {
    if constexpr (TASK == kTaskRefine)
      sh.V[Rows::at(j)] = j < n ? p->vd0[j] : 0.0;
    else
      sh.V[Rows::at(j)] = j < n ? p->vbuf0[j] : 0.f;
  }
  const bool policy_mode = TASK == kTaskMPI ? p->policy_is_init != 0
                                            : (TASK == kTaskSweep && p->policy_sweep);
  if (gridDim.x == 1) __syncthreads();  // the status words are clear before an error is raised
  if (policy_mode || TASK == kTaskMPI || TASK == kTaskRefine)
    for (int s = tid; s < n; s += nt) {
      int a = policy_mode ? p->policy[s] : 0;
      if (a < 0 || a >= p->m) {
        raise_abort(p->ctl, kDevBadPolicy);
        bad_entry = true;
        a = 0;
      }
      sh.pol[s] = (uint16_t)a;
    }
  const int smode = res_policy_sweeps(TASK, p->policy_sweep, p->K) ? kModePolicy : kModeMin;
  if (tid < 3) e.describe(tid, smode);
  const int nb = (int)((n + p->b - 1) / p->b);
  e.entries = nb > 1 ? e.ord_entries() : 0;
  e.span = 1;
  if (TASK != kTaskSweep && e.entries) e.span = max(1, min(16, min(64, kResList) / e.entries));
  if (e.entries) {
    if (p->perm) {
      for (int i = tid; i < e.entries; i += nt) {
        const int pos = e.ord_position(i);
        if (pos < 0) continue;
        int v = p->perm[pos];
        if (v < 0 || v >= n) {
          raise_abort(p->ctl, kDevBadPerm);
          bad_entry = true;
          v = 0;
        }
        sh.list[0][i] = (uint16_t)v;
      }
    } else {
      const int lanes = e.ord_lanes(e.span * e.entries, e.nw);
      e.ord_start(lanes);
      e.ord_run(t, 0, 0, true, lanes);
    }
  } else if (p->perm) {
    // one batch: the order inside it is free, its entries are checked
    for (int i = tid; i < n; i += nt)
      if (p->perm[i] < 0 || p->perm[i] >= n) {
        raise_abort(p->ctl, kDevBadPerm);
        bad_entry = true;
      }
  }
  if (TASK == kTaskSweep || TASK == kTaskMPI) {  // (the others read neither)
    if (__syncthreads_or(bad_entry)) return;
  } else {
    __syncthreads();
  }

  long long sweeps = 0, outer = 0, changes_last = -1, recentrings = 0, since = 0;
  double last_dv = NAN, last_err = NAN;
  int converged = 0;
  const auto want_recentre = [&](double d) {
    ++since;
    if (p->recentre_every <= 0 || since < p->recentre_every) return false;
    const double w = (double)e.sweep_wabs();
    if (!isfinite(w) || w <= 0.0) return false;
    return p->recentre_force || w > 16384.0 * d;
  };

  // One phase per turn: batch k of a sweep, or an improvement pass (imp).
  const bool ordered = e.entries > 0 && TASK != kTaskSweep;
  const int ncw_sweep = e.comm_waves(e.sweep_words(e.list_lgp()));
  const int ncw_imp = e.comm_waves(n);
  const int lanes = e.ord_lanes(e.span * e.entries, e.nw - ncw_sweep);
  // evaluations per entry: 4^h / n < 4, 2.5 on average over n
  const int passes = lanes ? (e.span * e.entries / lanes * 3 + 6) / (e.span * nb) + 1 : 0;
  int in_span = 0, buf = 0;  // the sweep's place in its span, the span's list buffer
  bool imp = (TASK == kTaskMPI && !p->policy_is_init) || TASK == kTaskRefine;
  bool first_imp = imp;  // Algorithm 1's initial policy, not an outer iteration
  bool ending = false;   // VI, correction: the pass that writes the greedy policy
  // the correction's certificate
  double residual = NAN, residual_in = NAN, bound = INFINITY;
  bool fresh = false, done = false;
  int k = 0, kk = 0;     // batch of the sweep, sweep of the evaluation
  if (ordered) e.ord_start(lanes);
  const int kind0 = nb > 1 ? 0 : 1;  // of a sweep's first batch
  ResBatch b = e.get(imp ? 2 : kind0, 0, 0, 0);
  while (true) {
    const bool last = imp || k == nb - 1;
    e.ncw = imp ? ncw_imp : ncw_sweep;
    const bool span_end = in_span == e.span - 1;
    ResBatch nx;
    // what follows in the same mode: the next batch, or the first of the next sweep
    const auto ahead = [&](ResBatch& to) {
      bool more = !imp;
      if (last) {
        if (TASK == kTaskSweep) more = false;
        if (TASK == kTaskVI) more = more && sweeps + 1 < p->max_sweeps;
        if (TASK == kTaskMPI) more = more && kk + 1 < p->K;
        if (TASK == kTaskRefine) more = more && (p->K ? kk + 1 < p->K : sweeps + 1 < p->max_sweeps);
      }
      // the sweep's list, and the next one's
      const int nx_buf = span_end ? buf ^ 1 : buf, nx_first = span_end ? 0 : (in_span + 1) * e.entries;
      const bool over = last && !imp;  // the next batch is the next sweep's first
      to = e.get(last ? kind0 : (k + 1 == nb - 1 ? 1 : 0), last ? 0 : k + 1,
                 over ? nx_buf : buf, over ? nx_first : in_span * e.entries);
      return more;
    };
    // the next span's order is complete before the last batch of this one
    const bool rest = span_end && k == nb - 2;
    const bool order = ordered && !imp && !(span_end && k == nb - 1);
    if (!e.run(b, ahead, nx, last, t + (uint64_t)(e.span - in_span), order ? buf ^ 1 : -1,
               rest ? -1 : passes, lanes))
      return;
    b = nx;
    if (!last) {
      ++k;
      continue;
    }
    k = 0;
    if constexpr (TASK == kTaskRefine) {
      // max|V - J*| <= max|TV - V| / (1 - gamma), and a sweep contracts by gamma
      const double g = p->gamma, inv = 1.0 / (1.0 - g);
      const bool ref = p->vref != nullptr;
      bool stop = false;
      if (imp) {
        residual = sh.s_resid;
        fresh = true;
        if (ending) break;
        if (first_imp) {
          residual_in = residual;
          bound = residual * inv;
          if (ref) last_err = e.sweep_err();
          done = ref ? last_err <= p->eps : bound <= p->eps;
        } else {
          ++outer;
          bound = residual * inv;
          if (!ref) done = bound <= p->eps;
        }
        first_imp = false;
        if (done || (p->K ? outer >= p->max_outer : p->max_sweeps <= 0)) break;
        imp = false;
        kk = 0;
      } else {
        ++t;
        ++sweeps;
        if (++in_span == e.span) {
          in_span = 0;
          buf ^= 1;
          if (ordered) e.ord_start(lanes);
        }
        fresh = false;
        last_dv = e.sweep_dv();
        if (ref) last_err = e.sweep_err();
        if (p->K == 0) {
          bound = fmin(g * last_dv * inv, g * bound);
          done = ref ? last_err <= p->eps : bound <= p->eps;
          stop = done || sweeps >= p->max_sweeps;
        } else if (ref && last_err <= p->eps) {
          done = stop = true;
        }
        if (stop) {
          // the output's residual and greedy policy, when wanted
          if (!p->policy && p->K == 0) break;
          ending = true;
        }
        if (ending || (p->K && ++kk == p->K)) {
          imp = true;
          e.drop_prefetch();
          b = e.get(2, 0, 0, 0);
        }
      }
      e.dv = e.err = 0.0;
      __syncthreads();
      continue;
    }
    if (TASK == kTaskSweep) {
      sweeps = 1;
      last_dv = e.sweep_dv();
      converged = 1;
      break;
    }
    if (imp) {
      if (TASK == kTaskVI) break;
      imp = false;
      if (!first_imp) {
        ++outer;
        changes_last = 0;
        for (int i = 0; i < e.ncw; ++i) changes_last += sh.s_changes[i];
        last_dv = sh.s_resid;
        if (changes_last == 0 && p->tol_dv >= 0.0 && last_dv <= p->tol_dv) {
          converged = 1;
          break;
        }
        if (outer >= p->max_outer) break;
      }
      first_imp = false;
      kk = 0;
      __syncthreads();  // the statistics are read before they are written again
      continue;
    }
    // the end of a sweep
    ++t;
    ++sweeps;
    if (++in_span == e.span) {
      in_span = 0;
      buf ^= 1;
      if (ordered) e.ord_start(lanes);
    }
    const double d = e.sweep_dv();
    bool stop = false;
    if (TASK == kTaskVI) {
      last_dv = d;
      stop = p->tol_dv >= 0.0 && d <= p->tol_dv;
    }
    if (p->vref) {
      last_err = e.sweep_err();
      stop = stop || last_err <= p->eps;
    }
    if (stop) converged = 1;
    if (stop || (TASK == kTaskVI && sweeps >= p->max_sweeps)) {
      if (TASK == kTaskMPI || !p->want_policy_out) break;
      ending = true;
    }
    if constexpr (TASK != kTaskRefine) {
      if (!ending && want_recentre(d)) {
        if (!e.recentre(gb)) return;
        ++recentrings;
        since = 0;
      }
    }
    if (ending || (TASK == kTaskMPI && ++kk == p->K)) {
      imp = true;
      e.drop_prefetch();
      b = e.get(2, 0, 0, 0);
    }
    e.dv = e.err = 0.0;
    e.wabs = 0;
    __syncthreads();
  }
  __syncthreads();
  if constexpr (TASK == kTaskRefine) {
    for (int s = (int)(blockIdx.x * blockDim.x) + tid; s < n; s += (int)(gridDim.x * blockDim.x))
      p->vd0[s] = sh.V[s];
    if (blockIdx.x == 0 && tid == 0) {
      const double residual_out = fresh ? residual : (double)NAN;
      Control* ctl = p->ctl;
      ctl->sweeps = sweeps;
      ctl->outer_iters = outer;
      ctl->final_dv_inf = last_dv;
      ctl->final_err_ref = last_err;
      ctl->converged = done ? 1 : 0;
      ctl->residual_in = residual_in;
      ctl->residual_out = residual_out;
      ctl->bound_out = p->K > 0 ? residual_out / (1.0 - p->gamma) : bound;
    }
    return;
  }
  // V = W + R into the caller's buffers
  for (int s = (int)(blockIdx.x * blockDim.x) + tid; s < n; s += (int)(gridDim.x * blockDim.x)) {
    const double v = (double)sh.V[Rows::at(s)] + (e.shifted ? p->shift[s] : 0.0);
    p->vbuf0[s] = (float)v;
    if (p->v64_out) p->v64_out[s] = v;
  }
  if (blockIdx.x == 0 && tid == 0) {
    Control* ctl = p->ctl;
    ctl->sweeps = sweeps;
    ctl->outer_iters = outer;
    ctl->policy_changes_last = changes_last;
    ctl->recentrings = recentrings;
    ctl->final_dv_inf = last_dv;
    ctl->final_err_ref = last_err;
    ctl->converged = converged;
    ctl->dv_last = (float)last_dv;
    if (p->dv_out) *p->dv_out = (float)last_dv;
  }
}

// The instantiation for a chunk shape and task.
template <class T, bool TAIL, int RC, int U, bool NT>
inline SolveFn resident_task(int task) {
  if constexpr (T::kType == kF32)
    if (task == kTaskRefine) return &resident_kernel<T, NT, TAIL, RC, U, kTaskRefine>;
  if (task == kTaskSweep) return &resident_kernel<T, NT, TAIL, RC, U, kTaskSweep>;
  if (task == kTaskVI) return &resident_kernel<T, NT, TAIL, RC, U, kTaskVI>;
  return &resident_kernel<T, NT, TAIL, RC, U, kTaskMPI>;
}

template <class T, bool TAIL>
inline SolveFn resident_fn(ResShape shape, int task) {
  switch (shape) {
    case kResShort: return resident_task<T, TAIL, 4, 2, false>(task);
    case kResCached: return resident_task<T, TAIL, 1, 4, false>(task);
    default: return resident_task<T, TAIL, 1, 8, true>(task);
  }
}

}  // namespace mbdp
