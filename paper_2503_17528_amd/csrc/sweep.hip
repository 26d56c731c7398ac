// The backward sweep of POBTASI as one persistent launch, for blocks whose
// products are too small to fill the chip one launch at a time.
//
// Per block i (from the last one down), with P_B = L_{i+1,i} W_i, P_R = L_{n,i}
// W_i and V_i = W_i^T W_i already formed:
//   R(i)  X_{n,i}   = -(X_{n,i+1} P_B + X_nn P_R)
//   A(i)  X_{i+1,i} = -(X_{i+1,i+1} P_B + X_{n,i+1}^T P_R)
//   B(i)  X_{i,i}   = V_i - X_{i+1,i}^T P_B - X_{n,i}^T P_R   (lower, mirrored)
// each cut into 32 x 32 output tiles (64 x 64 for larger b), one task per tile and
// workgroup: at b = 512 a phase A is 256 tasks, one per CU, where 64 x 64 tiles
// would be 64.  Launched product by product, a step of b = 512 took 68 us (four
// launches on the chain besides the copy and the arrow row); here it is two
// waits, 30 us (both without W, P and V: 9 us a block), bound by reading the
// operands (64 MB of tiles a phase A).  Taking
// the next ticket while a task runs left ready tasks with busy workgroups (n=256,
// b=512: 17.1 ms against 10.0).
//
// Tasks are taken from an atomic counter in the order R(i), A(i), B(i), i
// descending, so a task only waits for tasks of smaller tickets, which running
// workgroups own.  Tiles that the launch itself produces are stored and loaded
// device-coherently (a flag per tile behind the stores); P_B and P_R, final
// before the launch, come through the caches.
#include <algorithm>
#include <vector>

#include "bta_device.hpp"
#include "bta_internal.hpp"
#include "bta_testing.h"
#include "gemm_stage.hpp"

namespace bta {

namespace {

struct SweepArgs {
  const double* PB; const double* PR; const double* XT;
  double* XD; double* XB; double* XR;
  int* flags;  // per block: T*T of A, T*T of B, TA*T of R
  int* ctl;    // ticket counter (64 bits), abort flag at ctl[2]
  int n, b, a, T, TA;  // T, TA: tiles per edge of a block and of the tip
  int SW;              // tile edge
  long long per_step, ntasks;  // tasks of a step with an A phase; all
};

enum : int { SW_R = 0, SW_A = 1, SW_B = 2 };

struct SweepTask {
  int kind, i, m, n;
};

__host__ __device__ inline SweepTask sweep_decode(const SweepArgs& p, long long t) {
  SweepTask k;
  const int nr = p.TA * p.T, nb = p.T * (p.T + 1) / 2, na = p.T * p.T;
  const long long first = nr + nb;  // the last block has no A phase
  int rem;
  if (t < first) {
    k.i = p.n - 1;
    rem = (int)t;
  } else {
    const long long q = (t - first) / p.per_step;
    k.i = p.n - 2 - (int)q;
    rem = (int)(t - first - q * p.per_step);
  }
  const int nar = k.i < p.n - 1 ? na : 0;
  if (rem < nr) {
    k.kind = SW_R;
    k.m = rem / p.T;
    k.n = rem - k.m * p.T;
  } else if (rem < nr + nar) {
    rem -= nr;
    k.kind = SW_A;
    k.m = rem / p.T;
    k.n = rem - k.m * p.T;
  } else {
    rem -= nr + nar;
    k.kind = SW_B;
    k.m = 0;
    while (rem > k.m) rem -= ++k.m;
    k.n = rem;
  }
  return k;
}

__host__ __device__ inline int64_t sweep_flag(const SweepArgs& p, int kind, int i, int m, int n) {
  const int64_t base = (int64_t)i * (2 * p.T * p.T + p.TA * p.T);
  return base + (kind == SW_A ? 0 : kind == SW_B ? p.T * p.T : 2 * p.T * p.T) + (int64_t)m * p.T + n;
}

// One product term: A(m, k) at A[k*lda + m] (at) or A[m*lda + k], B(k, n) at B[k*ldb + n].
struct SweepSeg {
  const double* A; const double* B;
  int64_t lda, ldb;
  int at, K;
};

__device__ __forceinline__ bool sweep_aborted(const SweepArgs& p) {
  return __hip_atomic_load(p.ctl + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
}

// Lanes of one wave: wait for flag f0 + lane * step, lane < count.  A wait that
// gives up makes its own tile and those of every later wait NaN, so the last
// block's tiles hold NaN after any of them.  (The limit is a constant and the tiles
// that were done stay: the limit as an argument cost 0.5 and 1.6% at b = 512 and 640;
// NaN for all of X cost 0.5% at b = 512 by the last workgroup, 1.5% at n = 16, b = 64
// by a launch of its own.)
__device__ __forceinline__ void sweep_wait(const SweepArgs& p, int64_t f0, int64_t step, int count, int lane) {
  long long polls = 0;
  for (int e = lane; e < count; e += 64)
    while (!flag_set(p.flags + f0 + e * step)) {
      if (++polls > WAIT_LIMIT || ((polls & 63) == 0 && sweep_aborted(p))) {
        __hip_atomic_store(p.ctl + 2, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
}

// SW: tile edge (wave w takes the quadrant (w / 2, w % 2)).  An LDS stage of 32 KB
// holds 64 k of a 32-tile, or 32 k of a 64-tile, in sub-stages of 16 k.  BYTES:
// operand loads (16, or 4 for operands off 16-byte lines); NS: LDS stages, NS - 1
// of them in flight (two with the 4-byte loads: more would outrun the load counter).
template <int SW, int BYTES, int NS>
__global__ __launch_bounds__(256, 1) void selinv_sweep_kernel(SweepArgs p) {
  constexpr int WB = SW / 32, SUBS = 4 / WB, SWK = 16 * SUBS, SUB = SW * 16;  // doubles per operand and sub-stage
  constexpr int NI = WB * (BYTES == 16 ? 4 : 16), LPS = NI * 2 / WB;  // loads per sub-stage operand; per wave and stage
  __shared__ __align__(16) double lds[NS * 2 * SUBS * SUB];
  __shared__ long long ticket;
  __shared__ int good;
  const int tid0 = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid0 >> 6);
  const int b = p.b, a = p.a, T = p.T;
  const int64_t bb = (int64_t)b * b, ab = (int64_t)a * b;
  for (;;) {
    __syncthreads();  // the last task's reads of ticket and lds
    if (tid0 == 0) ticket = (long long)atomicAdd((unsigned long long*)p.ctl, 1ULL);
    __syncthreads();
    const long long tv = ticket;
    const long long tk = ((long long)__builtin_amdgcn_readfirstlane((int)(tv >> 32)) << 32) |
                         (unsigned)__builtin_amdgcn_readfirstlane((int)tv);
    if (tk >= p.ntasks) break;
    int tid = tid0;
    asm volatile("" : "+v"(tid));  // lane offsets formed per task
    const int lane = tid & 63;
    const SweepTask q = sweep_decode(p, tk);
    const int i = q.i, m0 = SW * q.m, n0 = SW * q.n;
    const bool sub = i < p.n - 1;
    const int rows = q.kind == SW_R ? a : b;
    const int mext = min(SW, rows - m0), next = min(SW, b - n0);

    // ---- operands and waits
    SweepSeg sg[2];
    const double* PBi = p.PB + (sub ? i : 0) * bb + n0;
    const double* PRi = p.PR + i * ab + n0;
    sg[0] = SweepSeg{nullptr, PBi, b, b, 0, sub ? b : 0};
    sg[1] = SweepSeg{nullptr, PRi, b, b, 0, a};
    if (w == 0) {
      if (q.kind == SW_R) {
        if (sub) sweep_wait(p, sweep_flag(p, SW_R, i + 1, q.m, 0), 1, T, lane);
      } else if (q.kind == SW_A) {
        // row block m of X_{i+1,i+1}: tiles (m, k), k <= m, and (k, m) below
        sweep_wait(p, sweep_flag(p, SW_B, i + 1, q.m, 0), 1, q.m + 1, lane);
        sweep_wait(p, sweep_flag(p, SW_B, i + 1, q.m, q.m), T, T - q.m, lane);
        sweep_wait(p, sweep_flag(p, SW_R, i + 1, 0, q.m), T, p.TA, lane);
      } else {
        if (sub) sweep_wait(p, sweep_flag(p, SW_A, i, 0, q.m), T, T, lane);
        sweep_wait(p, sweep_flag(p, SW_R, i, 0, q.m), T, p.TA, lane);
      }
      if (tid == 0) good = sweep_aborted(p) ? 0 : 1;
    }
    if (q.kind == SW_R) {
      sg[0].A = p.XR + (sub ? i + 1 : i) * ab + (int64_t)m0 * b;
      sg[1].A = p.XT + (int64_t)m0 * a;
      sg[1].lda = a;
    } else if (q.kind == SW_A) {
      sg[0].A = p.XD + (i + 1) * bb + (int64_t)m0 * b;
      sg[1].A = p.XR + (i + 1) * ab + m0;
      sg[1].at = 1;
    } else {
      sg[0].A = p.XB + (sub ? i : 0) * bb + m0;
      sg[0].at = 1;
      sg[1].A = p.XR + i * ab + m0;
      sg[1].at = 1;
    }
    const int nk0 = (sg[0].K + SWK - 1) / SWK, total = nk0 + (sg[1].K + SWK - 1) / SWK;

    // V's elements of this tile (B), in flight during the wait's barrier
    double* const out = q.kind == SW_R ? p.XR + i * ab : q.kind == SW_A ? p.XB + i * bb : p.XD + i * bb;
    const int r0 = 16 * WB * (w >> 1), c0 = 16 * WB * (w & 1);
    d4 v[WB][WB];
#pragma unroll
    for (int x = 0; x < WB; ++x)
#pragma unroll
      for (int y = 0; y < WB; ++y) {
        v[x][y] = d4{0.0, 0.0, 0.0, 0.0};
        if (q.kind == SW_B) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int r = r0 + 16 * x + acc_row(lane, j), c = c0 + 16 * y + acc_col(lane);
            if (r < mext && c < next && n0 + c <= m0 + r) v[x][y][j] = ld_dev(out + (int64_t)(m0 + r) * b + n0 + c);
          }
        }
      }
    __syncthreads();
    const bool ok = good != 0;

    // wave w moves both operands of sub-stage w (32-tiles), or operand w % 2 of
    // sub-stage w / 2 (64-tiles)
    const int us = w / WB;
    auto issue = [&](int kk) {
      const bool first = kk < nk0;
      const SweepSeg& g = first ? sg[0] : sg[1];
      const int k = (first ? kk : kk - nk0) * SWK + 16 * us, kext = g.K - k;
      double* st = lds + ((kk % NS) * SUBS + us) * 2 * SUB;
      if (WB == 1 || w % 2 == 0) stage_pieces<SW, NI, BYTES, true>(g.A, g.lda, g.at, 0, mext, k, kext, st, 0, lane);
      if (WB == 1 || w % 2 == 1) stage_pieces<SW, NI, BYTES, false>(g.B, g.ldb, 1, 0, next, k, kext, st + SUB, 0, lane);
    };
    // one sum per element, in k order (two, even and odd sub-stages, would cost a
    // rounding: X_{i+1,i} 1.65e-15 against 1.56e-15 off at b = 512)
    d4 acc[WB][WB] = {};
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // V has landed: the counts below are the stages' alone
    for (int kk = 0; kk < NS - 1 && kk < total; ++kk) issue(kk);
    for (int kk = 0; kk < total; ++kk) {
      if (NS > 2 && kk + 2 < total) wait_vm_barrier<(NS > 2 ? 2 * LPS : 0)>();
      else if (NS > 2 && kk + 1 < total) wait_vm_barrier<(NS > 2 ? LPS : 0)>();
      else wait_vm_barrier<0>();
      if (kk + NS - 1 < total) issue(kk + NS - 1);
      const double* st = lds + (kk % NS) * SUBS * 2 * SUB;
      const int at = kk < nk0 ? sg[0].at : sg[1].at;
#pragma unroll
      for (int u = 0; u < SUBS; ++u) {
        double x[WB][4], y[WB][4];
        stage_read<SW, WB>(x, st + u * 2 * SUB, at, r0, lane);
        stage_read<SW, WB>(y, st + u * 2 * SUB + SUB, 1, c0, lane);
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int e = 0; e < WB; ++e)
#pragma unroll
            for (int f = 0; f < WB; ++f) acc[e][f] = mfma16(x[e][s], y[f][s], acc[e][f]);
      }
    }
    wait_vm_barrier<0>();  // the stages are read: the tile's image takes their place

    // ---- the tile, through LDS for whole rows (and, mirrored, whole columns)
    constexpr int LDI = SW + 1;
#pragma unroll
    for (int x = 0; x < WB; ++x)
#pragma unroll
      for (int y = 0; y < WB; ++y)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const double val = v[x][y][j] - acc[x][y][j];
          lds[(r0 + 16 * x + acc_row(lane, j)) * LDI + c0 + 16 * y + acc_col(lane)] = ok ? val : __builtin_nan("");
        }
    __syncthreads();
    const int c = tid % SW;
    for (int r = tid / SW; r < SW; r += 256 / SW) {
      if (q.kind != SW_B) {
        if (r < mext && c < next) st_dev(out + (int64_t)(m0 + r) * b + n0 + c, lds[r * LDI + c]);
      } else if (q.m == q.n) {
        if (r < mext && c < next) st_dev(out + (int64_t)(m0 + r) * b + n0 + c, lds[max(r, c) * LDI + min(r, c)]);
      } else {
        if (r < mext && c < next) st_dev(out + (int64_t)(m0 + r) * b + n0 + c, lds[r * LDI + c]);
        if (r < next && c < mext) st_dev(out + (int64_t)(n0 + r) * b + m0 + c, lds[c * LDI + r]);
      }
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (tid == 0)
      __hip_atomic_store(p.flags + sweep_flag(p, q.kind, i, q.m, q.n), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Control words and flags to zero; give_up: the abort flag set from the start.
__global__ __launch_bounds__(256) void sweep_reset_kernel(int* p, int64_t count, int give_up) {
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < count; e += (int64_t)gridDim.x * 256)
    p[e] = e == 2 ? give_up : 0;
}

// Tile edge 64 from this b on: at 32 a phase reads its operands twice as often and,
// at b = 768, needs three rounds of the CUs (us per block with 32 / 64: b = 512
// 40 / 72, 640 71 / 96, 768 124 / 119, 1024 210 / 169).
constexpr int64_t SWEEP_WIDE_B = 768;

SweepArgs sweep_args(int64_t n, int64_t b, int64_t a) {
  SweepArgs p{};
  p.n = (int)n; p.b = (int)b; p.a = (int)a;
  p.SW = b >= SWEEP_WIDE_B ? 64 : 32;
  p.T = (int)((b + p.SW - 1) / p.SW);
  p.TA = (int)((a + p.SW - 1) / p.SW);
  const long long nr = (long long)p.TA * p.T, nb = (long long)p.T * (p.T + 1) / 2;
  p.per_step = nr + (long long)p.T * p.T + nb;
  p.ntasks = nr + nb + (n - 1) * p.per_step;
  return p;
}

}  // namespace

// ints: a 256-byte line of control words, then the flags
size_t sweep_work_bytes(int64_t n, int64_t b, int64_t a) {
  const SweepArgs p = sweep_args(n, b, a);
  return 256 + 4 * (size_t)(n * (2 * (int64_t)p.T * p.T + (int64_t)p.TA * p.T));
}

hipError_t sweep_launch(int64_t n, int64_t b, int64_t a, const double* PB, const double* PR, const double* XT, double* XD,
                        double* XB, double* XR, void* work, hipStream_t s) {
  SweepArgs p = sweep_args(n, b, a);
  if (g_dry) {
    ++g_dry->op;
    g_dry->add(PB, (n - 1) * b, b, b, false);
    if (a > 0) {
      g_dry->add(PR, n * a, b, b, false);
      g_dry->add(XT, a, a, a, false);
      g_dry->add(XR, n * a, b, b, true);
    }
    g_dry->add(XD, n * b, b, b, true);
    g_dry->add(XB, (n - 1) * b, b, b, true);
    return hipSuccess;
  }
  p.PB = PB; p.PR = PR; p.XT = XT; p.XD = XD; p.XB = XB; p.XR = XR;
  p.ctl = static_cast<int*>(work);
  p.flags = p.ctl + 64;
  const int64_t ints = (int64_t)(sweep_work_bytes(n, b, a) / 4);
  hipLaunchKernelGGL(sweep_reset_kernel, dim3((unsigned)std::min<int64_t>(1024, (ints + 255) / 256)), dim3(256), 0, s, p.ctl,
                     ints, g_wait_limit == 0 ? 1 : 0);
  auto al = [](const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15) == 0; };
  const bool pairs = b % 2 == 0 && a % 2 == 0 && al(PB) && al(PR) && al(XT) && al(XD) && al(XB) && al(XR);
  const long long grid = std::min<long long>(p.ntasks, std::max(1, device_cu_count()));
  timing_mark(KT_GEMM, true, s);
  auto kernel = p.SW == 64 ? (pairs ? selinv_sweep_kernel<64, 16, 4> : selinv_sweep_kernel<64, 4, 2>)
                           : (pairs ? selinv_sweep_kernel<32, 16, 4> : selinv_sweep_kernel<32, 4, 2>);
  hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(256), 0, s, p);
  timing_mark(KT_GEMM, false, s);
  return hipGetLastError();
}

}  // namespace bta

namespace bta {
thread_local long long g_wait_limit = WAIT_LIMIT;
}

BTA_TESTING_API long long bta_internal_wait_limit(long long polls) {
  const long long prev = bta::g_wait_limit;
  if (polls >= 0) bta::g_wait_limit = polls;
  return prev;
}

// Host replay of the sweep's tickets: every flag index in bounds and set once,
// and every awaited flag set by a smaller ticket.  Returns 0 when all hold.
BTA_TESTING_API int bta_internal_sweep_check(int64_t n, int64_t b, int64_t a) {
  using namespace bta;
  const SweepArgs p = sweep_args(n, b, a);
  std::vector<char> set((sweep_work_bytes(n, b, a) - 256) / 4, 0);
  for (long long t = 0; t < p.ntasks; ++t) {
    const SweepTask q = sweep_decode(p, t);
    if (q.i < 0 || q.i >= n || q.m < 0 || q.n < 0 || q.n >= p.T || q.m >= (q.kind == SW_R ? p.TA : p.T)) return 1;
    const bool sub = q.i < n - 1;
    bool ok = true;
    auto need = [&](int kind, int i, int m, int c) { ok = ok && set[sweep_flag(p, kind, i, m, c)]; };
    for (int k = 0; k < p.T; ++k) {
      if (q.kind == SW_R && sub) need(SW_R, q.i + 1, q.m, k);
      if (q.kind == SW_A) need(SW_B, q.i + 1, std::max(q.m, k), std::min(q.m, k));
      if (q.kind == SW_B && sub) need(SW_A, q.i, k, q.m);
    }
    for (int r = 0; r < p.TA; ++r) {
      if (q.kind == SW_A) need(SW_R, q.i + 1, r, q.m);
      if (q.kind == SW_B) need(SW_R, q.i, r, q.m);
    }
    if (!ok) return 2;
    const int64_t f = sweep_flag(p, q.kind, q.i, q.m, q.n);
    if (f < 0 || f >= (int64_t)set.size() || set[f]) return 3;
    set[f] = 1;
  }
  return 0;
}
