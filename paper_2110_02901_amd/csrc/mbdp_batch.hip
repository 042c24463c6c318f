// Many independent dense MDPs of uneven size in one launch.
//
// A workgroup takes the next MDP from a queue and runs MB-VI on it alone:
// the sweep order sigma_t of its own n and seed, batches of its own b, and
// between batches only a workgroup barrier, since no other workgroup
// touches the MDP.  V (FP64, up to 8192 states) lives in LDS for the whole
// solve; the rows stream from HBM, FP32 / BF16 / FP8 values decoded exactly
// and accumulated in FP64, so no re-centring is needed.  The launch is an
// ordinary one (no cooperative launch) and can be captured in a hipGraph.
//
// Heavy MDPs are served by a team of workgroups instead, so that one long
// solve does not hold the whole launch on one compute unit: the members
// split each batch's states, store the new values through to memory, meet
// at an arrival counter, and each copies the batch into its own LDS V.  The
// queue hands out the teams' tickets first and the host keeps the members of
// all teams within the compute units of the device, so every member of every
// team is resident from the start and no member waits for a workgroup that
// is busy with another MDP.
//
// Bound: the rows (a compute unit alone reads 35 to 47 GB/s of BF16 / FP32
// rows, above its 25 GB/s share of HBM), for FP8 the conversions to FP64
// (9 GB/s), in teams the meeting of each batch (4 to 9 us where the members
// arrive together: 1024 x 8 BF16, b = 128, takes 55.5 us a batch alone, 11.4
// with 8 members; ~10 us of 36 at 13 members of a large MDP among others).
// 96 BF16 MDPs of 256 to 2048 states, m = 8: 546 -> 194 ms against one state
// after the other per lane group, each waiting for its own order, rows, costs
// and sums.

#include <hip/hip_runtime.h>

#include <math.h>

#include "mbdp_engines.h"

namespace mbdp {

// rows of a state taken together: FP8 holds 16 values of V per step, so 4
template <int VT>
constexpr int batch_rows() {
  return VT == kFP8 ? 4 : 8;
}

template <int VT>
struct BatchVals;

template <>
struct BatchVals<kF32> {
  static constexpr int kEpl = 4;  // values per 16-byte load
  static constexpr int kBytes = 4;
  __device__ __forceinline__ static void decode(const u4& x, double (&out)[kEpl]) {
    out[0] = (double)__uint_as_float(x.x);
    out[1] = (double)__uint_as_float(x.y);
    out[2] = (double)__uint_as_float(x.z);
    out[3] = (double)__uint_as_float(x.w);
  }
};

template <>
struct BatchVals<kBF16> {
  static constexpr int kEpl = 8;
  static constexpr int kBytes = 2;
  __device__ __forceinline__ static void decode(const u4& x, double (&out)[kEpl]) {
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      out[2 * w] = (double)bf16_lo(x[w]);
      out[2 * w + 1] = (double)bf16_hi(x[w]);
    }
  }
};

template <>
struct BatchVals<kFP8> {
  static constexpr int kEpl = 16;
  static constexpr int kBytes = 1;
  __device__ __forceinline__ static void decode(const u4& x, double (&out)[kEpl]) {
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const f4 d = fp8x4(x[w]);
      out[4 * w] = (double)d.x;
      out[4 * w + 1] = (double)d.y;
      out[4 * w + 2] = (double)d.z;
      out[4 * w + 3] = (double)d.w;
    }
  }
};

// The item table holds generic pointers; these views make the compiler use
// global (not flat) memory instructions for them.
#define MBDP_GLOBAL __attribute__((address_space(1)))
template <class T>
__device__ __forceinline__ const MBDP_GLOBAL T* gview(const void* p) {
  return (const MBDP_GLOBAL T*)p;
}
template <class T>
__device__ __forceinline__ MBDP_GLOBAL T* gview_mut(void* p) {
  return (MBDP_GLOBAL T*)p;
}

struct BatchShared {
  double V[kBatchMaxN];
  double newv[kBatchMaxB];            // a lone workgroup's new values of the batch
  uint16_t order[2][kBatchMaxN];      // sigma_t, by sweep parity
  double zero[16];                    // V of the columns past a row's end
  double red[16];
  int item, rank, ok;
};

__device__ __forceinline__ BatchShared& batch_shared() {
  __shared__ BatchShared sh;
  return sh;
}

// LDS-only workgroup barrier: row loads in flight stay in flight.
__device__ __forceinline__ void batch_lds_barrier() {
  __asm__ volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// MB-VI on one MDP by a team of K >= 1 workgroups; `rank` is this one's.
//
// A lane group of LANES lanes serves one state at a time.  Its work is a
// sequence of chunks: R rows of the state by one step of LANES * 16 bytes of
// each row.  Two chunk buffers are in flight in turn, across states and, since
// rows do not depend on V, across batches: the first two chunks of the next
// batch are requested before the batch is committed.  Every chunk issues the
// same loads (rows past m and columns past ld are moved to valid ones and
// dropped), so that the wait for one chunk leaves the other in flight.
// The order of a sweep is drawn once, by all threads, into LDS; drawing it
// per state on every lane cost ~2 us per state, and waiting for each state's
// rows, costs and reductions in turn held a workgroup to 12-20 GB/s.
template <int VT, int LANES>
struct BatchSolver {
  using B = BatchVals<VT>;
  static constexpr int EPL = B::kEpl;
  static constexpr int R = batch_rows<VT>();
  static constexpr int GPW = kWave / LANES;  // lane groups per wavefront

  struct Buf {
    u4 x[R];
    float cost, scale;  // of row row_of_lane()
  };

  const BatchItem* it;
  BatchShared& sh;
  const BatchArgs& A;
  const MBDP_GLOBAL uint8_t* P;
  const MBDP_GLOBAL float* C;
  const MBDP_GLOBAL float* RS;
  double gamma;
  int lane, wave, nw, sl, gid, gstride;
  int n, m, ld, nsteps, nc, K;   // steps per row, chunks per state, workgroups
  Buf a, b;
  bool have;

  __device__ __forceinline__ BatchSolver(const BatchItem* item, int rank, BatchShared& s,
                                         const BatchArgs& args)
      : it(item), sh(s), A(args) {
    const BatchItem& I = *item;
    P = gview<uint8_t>(I.P);
    C = gview<float>(I.c);
    RS = gview<float>(I.rscale);
    gamma = I.gamma;
    K = I.team;
    lane = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    nw = (int)(blockDim.x >> 6);
    sl = lane % LANES;
    gid = (rank * nw + wave) * GPW + lane / LANES;
    gstride = K * nw * GPW;
    n = (int)I.n;
    m = I.m;
    ld = (int)I.ld;
    nsteps = (ld + LANES * EPL - 1) / (LANES * EPL);
    nc = nsteps * ((m + R - 1) / R);
    have = false;
    for (int r = 0; r < R; ++r) a.x[r] = b.x[r] = u4{0u, 0u, 0u, 0u};
    a.cost = a.scale = b.cost = b.scale = 0.f;
  }

  // After the halving reduction lane sl holds row row_of_lane() of the chunk.
  __device__ __forceinline__ int row_of_lane() const {
    return sl / (LANES / R);
  }

  // Chunk c of the t-th state of this lane group's positions kb + gid + t gstride < kb + bk.
  __device__ __forceinline__ int state_at(const uint16_t* ord, int kb, int bk, int t) const {
    const int pos = min(gid + t * gstride, bk - 1);
    return ord ? (int)ord[kb + pos] : kb + pos;
  }

  __device__ __forceinline__ void load(int s, int pass, int st, Buf& f) const {
    const int j = min((st * LANES + sl) * EPL, ld - EPL);
    const MBDP_GLOBAL uint8_t* p0 = P + ((size_t)s * m * (size_t)ld + (size_t)j) * B::kBytes;
    const size_t rb = (size_t)ld * B::kBytes;
#pragma unroll
    for (int r = 0; r < R; ++r)
      f.x[r] = __builtin_nontemporal_load(
          (const MBDP_GLOBAL u4*)(p0 + (size_t)min(pass * R + r, m - 1) * rb));
    const size_t row = (size_t)s * m + min(pass * R + row_of_lane(), m - 1);
    f.cost = C[row];
    if constexpr (VT != kF32) f.scale = RS[row];
  }

  __device__ __forceinline__ void consume(int st, const Buf& f, double (&acc)[R]) const {
    const int j = (st * LANES + sl) * EPL;
    const bool in = j < ld;
    const double* vp = in ? sh.V + j : sh.zero;
    double v[EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) v[e] = vp[e];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      double d[EPL];
      B::decode(in ? f.x[r] : u4{0u, 0u, 0u, 0u}, d);
#pragma unroll
      for (int e = 0; e < EPL; ++e) acc[r] = fma(d[e], v[e], acc[r]);
    }
  }

  // Sums over the lane group of the R accumulators, one row per lane: each
  // step halves the rows a lane keeps, then the lanes of a row are summed.
  __device__ __forceinline__ double reduce(double (&acc)[R]) const {
    int off = LANES / 2;
#pragma unroll
    for (int k = R / 2; k >= 1; k >>= 1) {
      const bool hi = (sl & off) != 0;
#pragma unroll
      for (int r = 0; r < k; ++r) {
        const double give = hi ? acc[r] : acc[r + k], keep = hi ? acc[r + k] : acc[r];
        acc[r] = keep + __shfl_xor(give, off);
      }
      off >>= 1;
    }
    double x = acc[0];
#pragma unroll
    for (int o = LANES / R / 2; o >= 1; o >>= 1) x += __shfl_xor(x, o);
    return x;
  }

  // Streams this workgroup's states of positions [kb, kb + bk) and hands every
  // state's minimum (q, lowest action) to `commit` on lane 0 of its group;
  // then requests the first chunks of the next positions (nbk > 0).
  template <class F>
  __device__ __forceinline__ void run(const uint16_t* ord, int kb, int bk, const uint16_t* nord,
                                      int nkb, int nbk, bool prefetch, F commit) {
    // the states of the wavefront's first lane group bound the others'
    const int g0 = __builtin_amdgcn_readfirstlane(gid);
    const int cnt = g0 < bk ? (bk - g0 + gstride - 1) / gstride : 0;
    const int C = cnt * nc;
    if (C > 0) {
      // chunk requested last: state t (of this lane group), pass, step
      int t = 0, pass = 0, st = 0, x = 0;
      int s = state_at(ord, kb, bk, 0);
      const auto next = [&]() {
        if (++x >= C) return;  // nothing is left: the last chunk again
        if (++st == nsteps) {
          st = 0;
          if (++pass * R >= m) {
            pass = 0;
            ++t;
            s = state_at(ord, kb, bk, t);
          }
        }
      };
      double acc[R], qb = INFINITY;
      int ab = 0;
#pragma unroll
      for (int r = 0; r < R; ++r) acc[r] = 0.0;
      int ct = 0, cpass = 0, cst = 0;  // chunk being used
      const auto use = [&](const Buf& f) {
        consume(cst, f, acc);
        if (++cst < nsteps) return;
        cst = 0;
        const double sum = reduce(acc);
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r] = 0.0;
        const int act = cpass * R + row_of_lane();
        const double sc = VT == kF32 ? 1.0 : (double)f.scale;
        const double q0 = (double)f.cost + gamma * (sc * sum);
        double q = act < m && q0 < INFINITY ? q0 : (double)INFINITY;
        int aq = q < INFINITY ? act : 0x7fffffff;
#pragma unroll
        for (int o = LANES / R; o < LANES; o <<= 1) {
          const double q2 = __shfl_xor(q, o);
          const int a2 = __shfl_xor(aq, o);
          if (q2 < q || (q2 == q && a2 < aq)) {
            q = q2;
            aq = a2;
          }
        }
        if (q < qb) {  // strictly smaller keeps the lowest action on ties
          qb = q;
          ab = aq;
        }
        if (++cpass * R < m) return;
        cpass = 0;
        const int i = gid + ct * gstride;
        if (sl == 0 && i < bk) commit(i, ord ? (int)ord[kb + i] : kb + i, qb, ab);
        ++ct;
        qb = INFINITY;
        ab = 0;
      };
      if (have) {
        next();
      } else {
        load(s, pass, st, a);
        next();
        load(s, pass, st, b);
      }
      int left = C;
      while (left > 2) {
        use(a);
        next();
        load(s, pass, st, a);
        use(b);
        next();
        load(s, pass, st, b);
        left -= 2;
      }
      use(a);
      if (left == 2) use(b);
    }
    have = false;
    if (prefetch && g0 < nbk) {
      int s = state_at(nord, nkb, nbk, 0);
      load(s, 0, 0, a);
      int pass = 0, st = 0;
      if (nsteps > 1) {
        st = 1;
      } else if (R < m) {
        pass = 1;
      } else if (g0 + gstride < nbk) {
        s = state_at(nord, nkb, nbk, 1);
      }
      load(s, pass, st, b);
      have = true;
    }
  }

  __device__ __forceinline__ void draw_order(uint64_t t) {
    const OrderKey key = make_order_key(n, it->seed, t);
    for (int i = (int)threadIdx.x; i < n; i += (int)blockDim.x)
      sh.order[t & 1][i] = (uint16_t)sweep_order_at((uint32_t)i, key);
  }

  // Arrival of this workgroup at the team's p-th meeting (p = 0, 1, ...) and
  // the wait for the others, by thread 0 (the counter only grows).  The new
  // values are written and read with agent-coherent accesses, so no cache is
  // written back or invalidated.  Gives up (false, and raises the launch's
  // abort flag) after `timeout` ticks or when another team gave up.
  __device__ __forceinline__ bool meet(unsigned long long p) const {
    unsigned long long* arrive = &A.ctl->arrive[it->slot];
    const unsigned long long target = (p + 1) * (unsigned long long)K;
    __hip_atomic_fetch_add(arrive, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long t0 = wall_clock64();
    while (atomic_load_agent(arrive) < target) {
      if (__hip_atomic_load(&A.ctl->abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return false;
      if (wall_clock64() - t0 > A.timeout_ticks) {
        __hip_atomic_store(&A.ctl->abort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return false;
      }
      __builtin_amdgcn_s_sleep(1);
    }
    return true;
  }

  __device__ __forceinline__ void solve(int rank) {
    const BatchItem& I = *it;
    const int bs = (int)I.b, nb = (n + bs - 1) / bs;
    const bool team = K > 1;
    double* dvm = A.team_dv + (size_t)I.slot * 2 * kBatchMaxTeam;   // [2][kBatchMaxTeam]
    double* gnew = A.team_new + (size_t)I.slot * 2 * kBatchMaxB;    // [2][kBatchMaxB]
    const MBDP_GLOBAL double* V0 = gview<double>(I.V);
    for (int j = (int)threadIdx.x; j < ld; j += (int)blockDim.x) sh.V[j] = j < n ? V0[j] : 0.0;
    if (threadIdx.x < 16) sh.zero[threadIdx.x] = 0.0;
    draw_order(0);
    __syncthreads();
    const unsigned long long t_start = wall_clock64();
    long long sweeps = 0;
    double dv = INFINITY;
    int converged = 0;
    unsigned long long phase = 0;
    bool ok = true;
    for (uint64_t t = 0; ok && (long long)t < A.max_sweeps; ++t) {
      const uint16_t* ord = sh.order[t & 1];
      draw_order(t + 1);  // visible after this sweep's barriers
      double dvl = 0.0;
      for (int k = 0; k < nb; ++k) {
        const int kb = k * bs, bk = min(bs, n - kb);
        const bool last = k == nb - 1;
        // (with one batch the next order is not yet visible to every thread)
        const bool pre = !(last && nb == 1) && !(team && wave == 0);
        double* buf = gnew + (phase & 1) * kBatchMaxB;
        const auto commit = [&](int i, int s, double q, int) {
          if (team)
            store_shared(&buf[i], q);
          else
            sh.newv[i] = q;
          dvl = fmax(dvl, fabs(q - sh.V[s]));
        };
        run(ord, kb, bk, last ? sh.order[(t + 1) & 1] : ord, last ? 0 : kb + bs,
            last ? min(bs, n) : min(bs, n - kb - bs), pre && !team, commit);
        if (last) {
          const double d = wave_max_d(dvl);
          if (lane == 0) sh.red[wave] = d;
        }
        if (team) {
          // this wavefront's values are performed; then the workgroup's
          __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
          batch_lds_barrier();
          if (wave == 0) {
            if (threadIdx.x == 0) {
              if (last) {  // this member's max |dV| of the sweep, by sweep parity
                double d = 0.0;
                for (int w = 0; w < nw; ++w) d = fmax(d, sh.red[w]);
                store_shared(&dvm[(t & 1) * kBatchMaxTeam + rank], d);
                __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
              }
              // buffers of parity p are rewritten at phase p + 2, after meeting
              // p + 1, which every member reaches only once it has read them
              sh.ok = meet(phase);
            }
          } else if (pre) {
            const int nbk = last ? min(bs, n) : min(bs, n - kb - bs);
            run(nullptr, 0, 0, last ? sh.order[(t + 1) & 1] : ord, last ? 0 : kb + bs, nbk, true,
                commit);
          }
          batch_lds_barrier();
          ok = sh.ok != 0;
          if (!ok) break;
          for (int i = (int)threadIdx.x; i < bk; i += (int)blockDim.x)
            sh.V[ord[kb + i]] = load_shared(&buf[i]);
          ++phase;
        } else {
          batch_lds_barrier();  // every state of the batch read the values before it
          for (int i = (int)threadIdx.x; i < bk; i += (int)blockDim.x) sh.V[ord[kb + i]] = sh.newv[i];
        }
        batch_lds_barrier();  // committed before the next batch reads
      }
      if (!ok) break;
      ++sweeps;
      dv = 0.0;
      if (team)
        for (int r = 0; r < K; ++r) dv = fmax(dv, load_shared(&dvm[(t & 1) * kBatchMaxTeam + r]));
      else
        for (int w = 0; w < nw; ++w) dv = fmax(dv, sh.red[w]);
      if (dv <= A.tol) {
        converged = 1;
        break;
      }
      batch_lds_barrier();  // sh.red and the order of sweep t - 1 are written again
    }
    have = false;
    __syncthreads();
    if (ok) {
      // results: V, and the greedy policy at the final V
      if (rank == 0) {
        MBDP_GLOBAL double* Vout = gview_mut<double>(I.V);
        for (int j = (int)threadIdx.x; j < n; j += (int)blockDim.x) Vout[j] = sh.V[j];
      }
      if (I.policy) {
        MBDP_GLOBAL int32_t* pol = gview_mut<int32_t>(I.policy);
        run(nullptr, 0, n, nullptr, 0, 0, false,
            [&](int, int s, double, int act) { pol[s] = act; });
      }
    }
    if (rank == 0 && threadIdx.x == 0) {
      BatchStat st;
      st.sweeps = sweeps;
      st.dv = dv;
      st.converged = ok ? converged : 0;
      st.pad = ok ? 0 : 1;
      st.t_start = t_start;  // member 0's: the team starts together
      st.t_end = wall_clock64();
      A.stats[I.index] = st;
    }
    __syncthreads();
  }
};

// Out of line: each value type and width has its own register allocation.
template <int VT, int LANES>
__device__ __noinline__ void batch_solve(const BatchItem* it, int rank, BatchArgs A) {
  BatchSolver<VT, LANES>(it, rank, batch_shared(), A).solve(rank);
}

template <int VT>
__device__ __forceinline__ void batch_dispatch_lanes(const BatchItem* it, int rank,
                                                     const BatchArgs& A) {
  if (it->lanes == 16)
    batch_solve<VT, 16>(it, rank, A);
  else if (it->lanes == 32)
    batch_solve<VT, 32>(it, rank, A);
  else
    batch_solve<VT, 64>(it, rank, A);
}

// Tickets 0, 1, ... are handed out in order; item i owns the tickets
// [ticket0, ticket0 + team), the items ordered by ticket0.
__global__ void __launch_bounds__(kBatchThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
batch_kernel(BatchArgs A) {
  BatchShared& sh = batch_shared();
  const BatchItem& last = A.items[A.count - 1];
  const long long tickets = last.ticket0 + last.team;
  while (true) {
    if (threadIdx.x == 0) {
      const long long u = (long long)atomicAdd(&A.ctl->queue, 1u);
      int it = A.count;
      if (u < tickets) {  // the last item whose first ticket is <= u
        int lo = 0, hi = A.count - 1;
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (A.items[mid].ticket0 <= u) lo = mid; else hi = mid - 1;
        }
        it = lo;
        sh.rank = (int)(u - A.items[lo].ticket0);
      }
      sh.item = it;
    }
    __syncthreads();
    const int it = sh.item, rank = sh.rank;
    __syncthreads();
    if (it >= A.count) break;
    const BatchItem* item = A.items + it;
    if (item->dtype == kBF16)
      batch_dispatch_lanes<kBF16>(item, rank, A);
    else if (item->dtype == kFP8)
      batch_dispatch_lanes<kFP8>(item, rank, A);
    else
      batch_dispatch_lanes<kF32>(item, rank, A);
    if (__hip_atomic_load(&A.ctl->abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) break;
  }
}

int launch_batch(const BatchArgs& a, int blocks, void* stream) {
  hipLaunchKernelGGL(batch_kernel, dim3(blocks), dim3(kBatchThreads), 0,
                     reinterpret_cast<hipStream_t>(stream), a);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace mbdp
