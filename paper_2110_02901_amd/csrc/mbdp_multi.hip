// Several value vectors against one dense P on the matrix cores.
//
// r value vectors V[:, j], one per cost vector C[:, :, j], share P (BF16
// codes with one FP32 scale per row), gamma, the batch size b and the sweep
// order sigma_t; each follows MB-VI (Sec. III-B) of its own MDP.  For one
// batch the expected values of all vectors are a matrix product: the batch's
// rows (s, a) of P against V [n x r], which these kernels run on MFMA
// (v_mfma_f32_16x16x32_bf16).
//
// Precision.  MFMA multiplies BF16 operands and accumulates in FP32.  The
// codes of P are BF16 already; V is held as V = R + W with an FP64 anchor R
// and a small difference W, and only W goes through the matrix cores, split
// into two BF16 terms (hi + lo carry 16 significant bits): the anchor's share
// P R is computed once per re-centring in FP64.  The error of a backup is
// then a small multiple of 2^-16 max|W|, which the host keeps below a
// fraction of the current change per sweep by folding W into R (the same
// idea as the single-vector anchor).
//
// A sweep starts with `multi_order_kernel`, which writes sigma_t into a table
// of the workspace.  One batch is two launches: `multi_gemm_kernel` writes the partial products
// of a K-range of P per (row, vector) (split over K so that a batch of a few
// thousand rows still fills the device), `multi_commit_kernel` adds the
// partials in FP64 with the cost, the anchor share and the row scale, takes
// the minimum over actions and commits the batch.  `multi_end_kernel` closes
// a sweep (its max |dV| from the commits' per-position maxima, the stop flag).  Every kernel returns at once when
// the stop flag is set, so the host can enqueue several sweeps and read the
// control block once.

#include <hip/hip_runtime.h>

#include <math.h>

#include <algorithm>

#include "mbdp_device.h"
#include "mbdp_internal.h"

namespace mbdp {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

#define MBDP_GLOBAL __attribute__((address_space(1)))

// round-to-nearest-even FP32 -> BF16 bits (NaN is not produced here: W is finite)
__device__ __forceinline__ unsigned multi_bf16_rne(float x) {
  const unsigned u = __float_as_uint(x);
  return ((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16) & 0xFFFFu;
}

__device__ __forceinline__ bool multi_done(const MultiControl* ctl) {
  return __hip_atomic_load(&ctl->done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
}

// Row `row` of a launch over positions kb, kb + 1, ... : its state and
// action.  Positions are those of sweep order sigma_t (the table the sweep's
// order kernel wrote), or (full) the states themselves, for the greedy policy.
__device__ __forceinline__ void multi_row_state(int64_t row, int32_t m, int full, int64_t kb,
                                                const int32_t* order, int64_t& s, int32_t& a) {
  const int64_t p = row / m;
  a = (int32_t)(row - p * m);
  s = full ? kb + p : (int64_t)order[kb + p];
}

// sigma_t of a whole sweep, once per sweep: every product and commit launch
// of the sweep reads its states from this table instead of evaluating the
// Feistel network per row (40 Philox rounds of 32-bit multiplies each).
// A wavefront runs its cycle walk until its slowest lane is done, so only
// kMultiOrderLanes lanes of each take a position (the expected longest of 16
// walks is about 5 Feistel passes, of 64 about 7) and the positions spread
// over four times as many wavefronts.
constexpr int kMultiOrderLanes = 16;
__global__ void __launch_bounds__(256) multi_order_kernel(MultiArgs A, uint64_t t) {
  if (multi_done(A.ctl)) return;  // uniform over the launch
  if ((threadIdx.x & 63) >= kMultiOrderLanes) return;
  const OrderKey key = make_order_key(A.n, A.seed, t);
  const int64_t lane_id = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / 64 * kMultiOrderLanes +
                          (threadIdx.x & 63);
  const int64_t lanes = (int64_t)gridDim.x * (blockDim.x / 64) * kMultiOrderLanes;
  for (int64_t p = lane_id; p < A.n; p += lanes)
    A.order[p] = (int32_t)sweep_order_at((uint32_t)p, key);
}

// LDS-only workgroup barrier: global loads stay in flight across it.
__device__ __forceinline__ void multi_lds_barrier() {
  __asm__ volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Partial products of one K-range: part[split][row][j] = sum over k in the
// range of code(row, k) * (hi + lo)(k, j).  A wavefront owns 16 RT rows and
// all NCT * 16 vectors; lane l feeds rows l % 16 of each row tile and vectors
// l % 16 of each column tile, 8 consecutive k from 8 (l / 16) (the same k map
// for both operands).  K runs in rounds: the rows come straight from HBM into
// one of two register buffers, requested a round before their products, while
// the W terms, shared by the workgroup's wavefronts, go through LDS (double
// buffered) by way of registers, requested two rounds before.  So nothing is
// waited for in the round that requests it, and the workgroup's barriers wait
// for LDS only.  Reading W per wavefront from L2 in 64-byte pieces cost more
// than the row stream itself.
// A row load brings 64 bytes of each of 16 rows (the MFMA operand layout),
// so each 128-byte line is asked for by two loads of the same wavefront;
// plain loads, which L1 keeps, serve the second half from the first
// (non-temporal ones were 1-7% slower).
// Bound by the row stream: 8192 x 16, b = 1024, r = 32 (268 MB of rows) took
// 63.1 us a batch with rows and W requested and used in the same round (4.3
// TB/s), 53.7 with the next round's requested ahead, 52.4 with W two ahead
// (5.1 TB/s).  Starting the workgroups at different rounds gave 2.5% more but
// changes the order of the sums.  Wider rounds for 48 and 64 vectors spill.
template <int RT, int NCT, int ROUND, int NW>  // ROUND: K per round; NW: wavefronts
__global__ void __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2, 2)))
multi_gemm_kernel(MultiArgs A, uint64_t t, int64_t k, int full) {
  constexpr int U = ROUND / 32;
  constexpr int PITCH = ROUND + 8;                     // staged W row, 16-byte pad
  constexpr int PPR = ROUND / 8;                       // 16-byte pieces per staged row
  constexpr int WROWS = 2 * NCT * 16;                  // staged W rows: 2 terms x r vectors
  constexpr int WPER = WROWS * PPR / (64 * NW);        // pieces per thread and round
  static_assert(WPER * 64 * NW == WROWS * PPR, "");
  __shared__ __attribute__((aligned(16))) uint16_t Wl[2][WROWS][PITCH];
  if (!full && multi_done(A.ctl)) return;  // uniform over the launch
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t kb = k * A.b;
  const int64_t rows = min(A.b, A.n - kb) * A.m;
  const int64_t wg0 = (int64_t)blockIdx.x * NW * (16 * RT);
  if (wg0 >= rows) return;  // whole workgroup: no barrier is skipped by part of it
  const int64_t tile0 = wg0 + wave * (16 * RT);
  const int i = lane & 15, g = lane >> 4;
  const int64_t n = A.n;
  const MBDP_GLOBAL uint16_t* P = (const MBDP_GLOBAL uint16_t*)A.P;
  const MBDP_GLOBAL uint16_t* Ws = (const MBDP_GLOBAL uint16_t*)A.Ws;
  const MBDP_GLOBAL uint16_t* arow[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    int64_t row = tile0 + rt * 16 + i;
    row = row < rows ? row : rows - 1;  // ragged tile: a valid row, result dropped
    int64_t s;
    int32_t a;
    multi_row_state(row, A.m, full, kb, A.order, s, a);
    arow[rt] = P + ((size_t)s * A.m + a) * (size_t)n + 8 * g;
  }
  f32x4 acc[RT][NCT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int c = 0; c < NCT; ++c) acc[rt][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int k0 = (int)(blockIdx.y * A.kchunk);
  const int k1 = (int)min(n, (int64_t)k0 + A.kchunk);
  // staged W row w = h * r + j holds W term h of vector j; piece q of a round
  // is row q / PPR, values 8 (q % PPR) .. +7.  The last round may be short:
  // addresses stay inside the range, what they bring is not used.
  auto fetch_w = [&](int kk, u32x4 (&wr)[WPER]) {
#pragma unroll
    for (int e = 0; e < WPER; ++e) {
      const int q = threadIdx.x + 64 * NW * e;
      const int w = q / PPR, c8 = (q % PPR) * 8;  // (Ws is [2][r][n]: w counts its rows)
      wr[e] = *(const MBDP_GLOBAL u32x4*)(Ws + (size_t)w * (size_t)n + min(kk + c8, k1 - 8));
    }
  };
  auto store_w = [&](int buf, const u32x4 (&wr)[WPER]) {
#pragma unroll
    for (int e = 0; e < WPER; ++e) {
      const int q = threadIdx.x + 64 * NW * e;
      *(u32x4*)&Wl[buf][q / PPR][(q % PPR) * 8] = wr[e];
    }
  };
  auto load_a = [&](int kk, u32x4 (&av)[U][RT]) {
    if (kk + ROUND <= k1) {
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
          av[u][rt] = *(const MBDP_GLOBAL u32x4*)(arow[rt] + kk + 32 * u);
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
          av[u][rt] = *(const MBDP_GLOBAL u32x4*)(arow[rt] + min(kk + 32 * u, k1 - 32));
    }
  };
  auto products = [&](const u32x4 (&av)[U][RT], int buf, int steps) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (u >= steps) break;
#pragma unroll
      for (int c = 0; c < NCT; ++c)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const u32x4 bv = *(const u32x4*)&Wl[buf][h * NCT * 16 + c * 16 + i][32 * u + 8 * g];
#pragma unroll
          for (int rt = 0; rt < RT; ++rt)
            acc[rt][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                __builtin_bit_cast(bf16x8, av[u][rt]), __builtin_bit_cast(bf16x8, bv), acc[rt][c],
                0, 0, 0);
        }
    }
  };
  u32x4 A0[U][RT], A1[U][RT], wr[WPER];
  // One round, with its W in LDS, its rows in `cur` and the next one's W in
  // wr (both requested a round ago): the next W goes to the other buffer (last
  // read in the previous round, before its barrier), the W after it and the
  // next rows are requested, then the products.
  auto round = [&](int kk, const u32x4 (&cur)[U][RT], u32x4 (&nxt)[U][RT], int buf) {
    store_w(buf ^ 1, wr);
    fetch_w(kk + 2 * ROUND, wr);
    load_a(kk + ROUND, nxt);
    __builtin_amdgcn_sched_barrier(0);
    products(cur, buf, U);
    multi_lds_barrier();
  };
  fetch_w(k0, wr);
  load_a(k0, A0);
  __builtin_amdgcn_sched_barrier(0);
  store_w(0, wr);
  fetch_w(k0 + ROUND, wr);
  multi_lds_barrier();
  for (int kk = k0;; kk += 2 * ROUND) {
    if (kk + ROUND >= k1) {
      products(A0, 0, (k1 - kk) / 32);
      break;
    }
    round(kk, A0, A1, 0);
    if (kk + 2 * ROUND >= k1) {
      products(A1, 1, (k1 - kk - ROUND) / 32);
      break;
    }
    round(kk + ROUND, A1, A0, 1);
  }
  if (tile0 >= rows) return;  // after the last barrier
  // lane l holds rows 4 (l / 16) + v of each 16-row tile, vector l % 16 of each column tile
  MBDP_GLOBAL float* part = (MBDP_GLOBAL float*)A.part + (size_t)blockIdx.y * A.part_rows * A.r;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t row = tile0 + rt * 16 + 4 * g + v;
      if (row < rows) {
#pragma unroll
        for (int c = 0; c < NCT; ++c) part[(size_t)row * A.r + c * 16 + i] = acc[rt][c][v];
      }
    }
}

// Commit of batch k (mode 0), or the greedy action of states kb .. kb + b - 1
// (mode 1): a workgroup per state.  Thread (al, j) serves vector j and the
// actions a = al, al + AL, ... (AL = 256 / r action lanes); the lanes' minima
// meet in LDS, lowest action on ties.
__global__ void __launch_bounds__(256) multi_commit_kernel(MultiArgs A, uint64_t t, int64_t k,
                                                           int mode) {
  __shared__ double qs[256];
  __shared__ int32_t as[256];
  const int64_t kb = k * A.b;
  const int64_t p = blockIdx.x;                // position in the launch (< min(b, n - kb))
  const int AL = 256 / A.r;
  const int al = threadIdx.x / A.r, j = threadIdx.x - al * A.r;
  // The stop flag is requested with the state (the table is read in either
  // mode, so neither load waits behind a branch) and tested only before the
  // first store; the state's old W and R are requested with its costs.
  const unsigned done = __hip_atomic_load(&A.ctl->done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int64_t o = A.order[kb + p];
  const bool stop = mode == 0 && done != 0u;
  const int64_t s = mode ? kb + p : o;
  const size_t e = (size_t)s * A.r + j;
  const bool commit = mode == 0 && al == 0;
  const double w_old = commit ? A.W[e] : 0.0, r_old = commit ? A.R[e] : 0.0;
  double best = INFINITY;
  int32_t besta = 0;
  if (al < AL) {
    for (int32_t a = al; a < A.m; a += AL) {
      const int64_t lrow = p * A.m + a;      // row of the launch
      const int64_t grow = s * A.m + a;      // row of P
      double acc = 0.0;
#pragma unroll 4
      for (int sp = 0; sp < A.splits; ++sp)
        acc += (double)A.part[((size_t)sp * A.part_rows + lrow) * A.r + j];
      const double q = (double)A.C[(size_t)grow * A.r + j] +
                       A.gamma * ((double)A.rscale[grow] * acc + A.PR[(size_t)grow * A.r + j]);
      if (q < best) {  // ascending actions: strictly smaller keeps the lowest
        best = q;
        besta = a;
      }
    }
  }
  qs[threadIdx.x] = best;
  as[threadIdx.x] = besta;
  __syncthreads();
  if (stop) return;  // uniform over the launch; nothing was stored
  double dv = 0.0;
  if (al == 0) {
    for (int l = 1; l < AL; ++l) {
      const double q2 = qs[l * A.r + j];
      const int32_t a2 = as[l * A.r + j];
      if (q2 < best || (q2 == best && a2 < besta)) {
        best = q2;
        besta = a2;
      }
    }
    if (mode == 1) {
      A.policy[e] = besta;
    } else {
      const double wnew = best - r_old;
      dv = fabs(wnew - w_old);
      A.W[e] = wnew;
      const unsigned hi = multi_bf16_rne((float)wnew);
      const unsigned lo = multi_bf16_rne((float)(wnew - (double)__uint_as_float(hi << 16)));
      A.Ws[(size_t)j * A.n + s] = (uint16_t)hi;
      A.Ws[((size_t)A.r + j) * A.n + s] = (uint16_t)lo;
    }
  }
  if (mode == 0 && threadIdx.x < 64) {  // the r <= 64 threads with al == 0 are in wavefront 0
    dv = wave_max_d(dv);
    // one slot per position of the sweep (every sweep writes all n), reduced
    // by the end-of-sweep kernel: no contended atomic per workgroup
    if (threadIdx.x == 0) A.dvs[kb + p] = dv;
  }
}

// End of sweep t: its max |dV| (over the per-position maxima the commits
// wrote), the bound on max |W|, the stop flag.  One workgroup.
__global__ void __launch_bounds__(256) multi_end_kernel(MultiArgs A) {
  __shared__ double red[4];
  if (multi_done(A.ctl)) return;  // uniform over the workgroup
  double dv = 0.0;
#pragma unroll 8  // independent loads, so several are in flight
  for (int64_t e = threadIdx.x; e < A.n; e += blockDim.x) dv = fmax(dv, A.dvs[e]);
  dv = wave_max_d(dv);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = dv;
  __syncthreads();
  if (threadIdx.x != 0) return;
  dv = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
  MultiControl* c = A.ctl;
  c->dv_last = dv;
  c->w_bound += dv;
  c->sweeps += 1;
  if (A.tol >= 0.0 && dv <= A.tol)
    __hip_atomic_store(&c->done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// mode 0: R = V, W = 0 (start); mode 1: R += W, W = 0 (re-centring);
// mode 2: V = R + W (result).  Clears the split copy of W in modes 0 and 1.
__global__ void __launch_bounds__(256) multi_anchor_kernel(MultiArgs A, double* V, int mode) {
  const int64_t total = A.n * A.r;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    if (mode == 2) {
      V[e] = A.R[e] + A.W[e];
      continue;
    }
    A.R[e] = mode == 0 ? V[e] : A.R[e] + A.W[e];
    A.W[e] = 0.0;
    const int64_t s = e / A.r, j = e - s * A.r;
    A.Ws[(size_t)j * A.n + s] = 0;
    A.Ws[((size_t)A.r + j) * A.n + s] = 0;
  }
  if (mode != 2 && blockIdx.x == 0 && threadIdx.x == 0) A.ctl->w_bound = 0.0;
}

// PR[row][j] = scale(row) * sum_k code(row, k) R[k][j] in FP64 on the matrix
// cores (v_mfma_f64_16x16x4_f64).  A wavefront owns 32 rows and all r vectors;
// K runs in rounds of 32: lane l feeds codes 8 (l / 16) .. +7 of row l % 16 of
// each row tile, one 16-byte load for the eight products of the round (product
// s multiplies the k = 8 (l / 16) + s of either operand), and reads R from the
// round's copy in LDS (padded so that the two lane groups of a read phase
// fall on different banks).  Rows, and R two rounds ahead, are requested a
// round before their use.  Bound by the FP64 rate (r = 32: 69 GFLOP at 8192 x
// 16, 0.9 ms at the card's nominal 78 TFLOP/s).  4.21 ms with 4 x 4 blocks of
// vector FMAs of 64 columns whatever r; 1.14 ms here.
template <int NCT>
__global__ void __launch_bounds__(256) multi_pr_kernel(MultiArgs A) {
  constexpr int RT = 2, r = NCT * 16;
  constexpr int GP = 8 * r + 16;        // doubles per group of 8 staged R rows
  constexpr int RPER = 32 * r / 2 / 256;  // 16-byte pieces of R per thread and round
  __shared__ __attribute__((aligned(16))) double Rt[2][4 * GP];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = lane & 15, g = lane >> 4;
  const int64_t rows = A.n * A.m;
  const int n = (int)A.n;
  const int64_t tile0 = ((int64_t)blockIdx.x * 4 + wave) * (16 * RT);
  const MBDP_GLOBAL uint16_t* arow[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
    arow[rt] = (const MBDP_GLOBAL uint16_t*)A.P +
               (size_t)min(tile0 + rt * 16 + i, rows - 1) * (size_t)n + 8 * g;
  const MBDP_GLOBAL double* R = (const MBDP_GLOBAL double*)A.R;
  f64x4 acc[RT][NCT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int c = 0; c < NCT; ++c) acc[rt][c] = f64x4{0.0, 0.0, 0.0, 0.0};
  // rounds past the last: addresses stay inside, what they bring is not used
  auto fetch_r = [&](int k0, f64x2 (&x)[RPER]) {
    const MBDP_GLOBAL f64x2* src = (const MBDP_GLOBAL f64x2*)(R + (size_t)min(k0, n - 32) * r);
#pragma unroll
    for (int e = 0; e < RPER; ++e) x[e] = src[threadIdx.x + 256 * e];
  };
  auto store_r = [&](int buf, const f64x2 (&x)[RPER]) {
#pragma unroll
    for (int e = 0; e < RPER; ++e) {
      const int q = 2 * (threadIdx.x + 256 * e);  // of the round's [32][r]
      *(f64x2*)&Rt[buf][q + 16 * (q / (8 * r))] = x[e];
    }
  };
  auto load_a = [&](int k0, u32x4 (&x)[RT]) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
      x[rt] = *(const MBDP_GLOBAL u32x4*)(arow[rt] + min(k0, n - 32));
  };
  f64x2 rr[RPER];
  u32x4 x[RT], y[RT];
  fetch_r(0, rr);
  load_a(0, x);
  store_r(0, rr);
  fetch_r(32, rr);
  multi_lds_barrier();
  int buf = 0;
  for (int k0 = 0; k0 < n; k0 += 32, buf ^= 1) {
    store_r(buf ^ 1, rr);
    fetch_r(k0 + 64, rr);
    load_a(k0 + 32, y);
    __builtin_amdgcn_sched_barrier(0);
    const double* b0 = &Rt[buf][g * GP + i];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      double bv[NCT];
#pragma unroll
      for (int c = 0; c < NCT; ++c) bv[c] = b0[s * r + c * 16];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const unsigned w = x[rt][s / 2];
        const double av = (double)__uint_as_float(s % 2 ? w & 0xFFFF0000u : w << 16);
#pragma unroll
        for (int c = 0; c < NCT; ++c)
          acc[rt][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv[c], acc[rt][c], 0, 0, 0);
      }
    }
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) x[rt] = y[rt];
    multi_lds_barrier();
  }
  // lane l holds rows 4 v + l / 16 of each 16-row tile, vector l % 16 of each column tile
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t row = tile0 + rt * 16 + 4 * v + g;
      if (row >= rows) continue;
      const double sc = (double)A.rscale[row];
#pragma unroll
      for (int c = 0; c < NCT; ++c) A.PR[(size_t)row * r + c * 16 + i] = sc * acc[rt][c][v];
    }
}

// ------------------------------------------------------------------ launches

typedef void (*MultiGemmFn)(MultiArgs, uint64_t, int64_t, int);

// The product's instantiation and its wavefronts per workgroup.  Eight share
// one copy of W where the launch's wavefronts fill the device that way (2048,
// what the split over K aims at): half the W traffic of four.  Below, four
// keep more compute units busy.  Per sweep, eight against four (us): 8192 x
// 16, b = 1024, r = 16 498 / 525, r = 32 555 / 573, r = 64 729 / 782; 2048 x
// 5, b = 200, r = 16 148 / 141, r = 32 163 / 150, r = 64 243 / 203.  48
// vectors need more registers than eight wavefronts leave: 906 / 885.
static MultiGemmFn multi_gemm_fn(int32_t r, int64_t waves, int* nw) {
  const bool full = waves >= 2048 && r != 48;
  *nw = full ? 8 : 4;
  switch (r) {
    case 16: return full ? multi_gemm_kernel<1, 1, 256, 8> : multi_gemm_kernel<1, 1, 128, 4>;
    case 32: return full ? multi_gemm_kernel<2, 2, 128, 8> : multi_gemm_kernel<2, 2, 128, 4>;
    case 48: return multi_gemm_kernel<3, 3, 64, 4>;
    case 64: return full ? multi_gemm_kernel<4, 4, 64, 8> : multi_gemm_kernel<4, 4, 32, 4>;
    default: return nullptr;
  }
}

int launch_multi_gemm(const MultiArgs& a, uint64_t t, int64_t k, int full, void* stream) {
  const int64_t rows = std::min<int64_t>(a.b, a.n - k * a.b) * a.m;
  const int64_t by = (a.n + a.kchunk - 1) / a.kchunk;
  const int64_t tile = multi_rows_per_wave(a.r);
  int nw = 0;
  MultiGemmFn f = multi_gemm_fn(a.r, (rows + tile - 1) / tile * by, &nw);
  if (!f) return -1;
  const int64_t bx = (rows + nw * tile - 1) / (nw * tile);
  hipLaunchKernelGGL(f, dim3((unsigned)bx, (unsigned)by), dim3(64 * nw), 0,
                     reinterpret_cast<hipStream_t>(stream), a, t, k, full);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_multi_commit(const MultiArgs& a, uint64_t t, int64_t k, int mode, void* stream) {
  const int64_t blocks = std::min<int64_t>(a.b, a.n - k * a.b);  // a workgroup per state
  hipLaunchKernelGGL(multi_commit_kernel, dim3((unsigned)blocks), dim3(256), 0,
                     reinterpret_cast<hipStream_t>(stream), a, t, k, mode);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_multi_end(const MultiArgs& a, void* stream) {
  hipLaunchKernelGGL(multi_end_kernel, dim3(1), dim3(256), 0,
                     reinterpret_cast<hipStream_t>(stream), a);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_multi_order(const MultiArgs& a, uint64_t t, void* stream) {
  const int64_t per_block = 4 * kMultiOrderLanes;  // positions per 256-thread workgroup and pass
  int64_t blocks = (a.n + per_block - 1) / per_block;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(multi_order_kernel, dim3((unsigned)blocks), dim3(256), 0,
                     reinterpret_cast<hipStream_t>(stream), a, t);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_multi_anchor(const MultiArgs& a, double* V, int mode, void* stream) {
  int64_t blocks = (a.n * a.r + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(multi_anchor_kernel, dim3((unsigned)blocks), dim3(256), 0,
                     reinterpret_cast<hipStream_t>(stream), a, V, mode);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_multi_pr(const MultiArgs& a, void* stream) {
  void (*f)(MultiArgs) = a.r == 16   ? multi_pr_kernel<1>
                         : a.r == 32 ? multi_pr_kernel<2>
                         : a.r == 48 ? multi_pr_kernel<3>
                                     : multi_pr_kernel<4>;
  const int64_t blocks = (a.n * a.m + 127) / 128;  // 32 rows per wavefront
  hipLaunchKernelGGL(f, dim3((unsigned)blocks), dim3(256), 0, reinterpret_cast<hipStream_t>(stream), a);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace mbdp
