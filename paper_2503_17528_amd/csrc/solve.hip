// Triangular solves with the BTA factor (A x = y via L z = y, L^T x = z) and
// the log-determinant 2 * sum log diag(L).  Neither is in the paper; both are
// needed for f(A) = log det A + y^T A^{-1} y and its gradient.
//
// The solve is memory bound (O(n b^2) reads of L per sweep) and sequential in
// the block index.  The diagonal blocks are inverted up front in batched MFMA
// launches (W_i = L_ii^{-1}, the same inverse-factor form as the selected
// inversion), so that every step of both sweeps is a pair of dense products,
// and each sweep is one persistent launch whose tasks (16 rows of a product)
// hand their rows on without leaving the chip.  Every sum runs in a fixed order
// (deterministic).
#include <algorithm>

#include "bta_device.hpp"
#include "bta_internal.hpp"
#include "bta_testing.h"

namespace bta {

#define BTA_TRY_E(x)                    \
  do {                                  \
    hipError_t e_ = (x);                \
    if (e_ != hipSuccess) return e_;    \
  } while (0)

// ---------------------------------------------------------------- logdet
__global__ __launch_bounds__(256) void logdet_partial_kernel(const double* LD, const double* LT, int64_t n, int64_t b,
                                                             int64_t a, double* partial) {
  __shared__ double red[256];
  const int64_t blk = blockIdx.x;
  const double* L;
  int64_t m;
  if (blk < n) { L = LD + blk * b * b; m = b; } else { L = LT; m = a; }
  double s = 0.0;
  for (int64_t k = threadIdx.x; k < m; k += 256) s += log(L[k * m + k]);
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blk] = red[0];
}

__global__ __launch_bounds__(256) void logdet_final_kernel(const double* partial, int64_t count, double* out) {
  __shared__ double red[256];
  double s = 0.0;
  for (int64_t k = threadIdx.x; k < count; k += 256) s += partial[k];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = 2.0 * red[0];
}

size_t logdet_work_bytes(int64_t n, int64_t b, int64_t a) { return 8 * (size_t)(n + 1 + 1024) + 256; }

// ---------------------------------------------------------------- quadratic term and gradient

// partial[blk] = sum over a fixed slice of the elementwise product y * x
__global__ __launch_bounds__(256) void dot_partial_kernel(const double* y, const double* x, int64_t count, int nslices,
                                                          double* partial) {
  __shared__ double red[256];
  const int64_t per = (count + nslices - 1) / nslices;
  const int64_t lo = (int64_t)blockIdx.x * per, hi = std::min<int64_t>(count, lo + per);
  double s = 0.0;
  for (int64_t k = lo + threadIdx.x; k < hi; k += 256) s += y[k] * x[k];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

// out = 2 * sum(logs) + sum(dots), every partial summed in a fixed order
__global__ __launch_bounds__(256) void logdet_quad_final_kernel(const double* plog, int64_t nlog, const double* pdot,
                                                                int ndot, double* out) {
  __shared__ double red[256];
  double s = 0.0, t = 0.0;
  for (int64_t k = threadIdx.x; k < nlog; k += 256) s += plog[k];
  for (int64_t k = threadIdx.x; k < ndot; k += 256) t += pdot[k];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  const double ls = red[0];
  __syncthreads();
  red[threadIdx.x] = t;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = 2.0 * ls + red[0];
}

hipError_t logdet_quad_launch(int64_t n, int64_t b, int64_t a, const double* LD, const double* LT, const double* y,
                              const double* x, int64_t nrhs, double* out, void* work, hipStream_t stream) {
  double* plog = static_cast<double*>(work);
  double* pdot = plog + (n + 1);
  const int64_t nb = n + (a > 0 ? 1 : 0);
  hipLaunchKernelGGL(logdet_partial_kernel, dim3((unsigned)nb), dim3(256), 0, stream, LD, LT, n, b, a, plog);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t count = (n * b + a) * nrhs;
  const int nslices = (int)std::min<int64_t>(1024, (count + 4095) / 4096);
  hipLaunchKernelGGL(dot_partial_kernel, dim3((unsigned)nslices), dim3(256), 0, stream, y, x, count, nslices, pdot);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(logdet_quad_final_kernel, dim3(1), dim3(256), 0, stream, plog, nb, pdot, nslices, out);
  return hipGetLastError();
}

// G = s * f * (X - sum_j x_j x_j^T) on the pattern (f = 1 for the diagonal and
// tip blocks, 2 for the lower and arrow blocks, which also stand at their
// mirrored positions), gy = 2 s x.  Elementwise: G may alias X.
struct GradParams {
  int64_t n, b, a, nrhs;
  const double* XD; const double* XB; const double* XR; const double* XT;
  const double* x;
  const double* scale;
  double* GD; double* GB; double* GR; double* GT;
  double* gy;
};

__global__ __launch_bounds__(256) void grad_pattern_kernel(GradParams p) {
  const int64_t n = p.n, b = p.b, a = p.a, nr = p.nrhs;
  const int64_t bb = b * b, ab = a * b;
  const int64_t nD = n * bb, nB = (n - 1) * bb, nR = n * ab, nT = a * a, N = n * b + a;
  const int64_t total = nD + nB + nR + nT + (p.gy ? N * nr : 0);
  const double s = p.scale ? *p.scale : 1.0;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    int64_t k = e;
    int64_t row, col;  // global row / column indices into x
    const double* X;
    double* G;
    double f;
    if (k < nD) {
      const int64_t i = k / bb, rc = k - i * bb, r = rc / b, c = rc - r * b;
      row = i * b + r; col = i * b + c; X = p.XD; G = p.GD; f = 1.0;
    } else if ((k -= nD) < nB) {
      const int64_t i = k / bb, rc = k - i * bb, r = rc / b, c = rc - r * b;
      row = (i + 1) * b + r; col = i * b + c; X = p.XB; G = p.GB; f = 2.0;
    } else if ((k -= nB) < nR) {
      const int64_t i = k / ab, rc = k - i * ab, r = rc / b, c = rc - r * b;
      row = n * b + r; col = i * b + c; X = p.XR; G = p.GR; f = 2.0;
    } else if ((k -= nR) < nT) {
      const int64_t r = k / a, c = k - r * a;
      row = n * b + r; col = n * b + c; X = p.XT; G = p.GT; f = 1.0;
    } else {
      k -= nT;
      p.gy[k] = 2.0 * s * p.x[k];
      continue;
    }
    double o = 0.0;
    for (int64_t j = 0; j < nr; ++j) o += p.x[row * nr + j] * p.x[col * nr + j];
    G[k] = s * f * (X[k] - o);
  }
}

hipError_t grad_launch(int64_t n, int64_t b, int64_t a, const double* XD, const double* XB, const double* XR,
                       const double* XT, const double* x, int64_t nrhs, const double* scale, double* GD, double* GB,
                       double* GR, double* GT, double* gy, hipStream_t stream) {
  GradParams p{n, b, a, nrhs, XD, XB, XR, XT, x, scale, GD, GB, GR, GT, gy};
  const int64_t total = n * b * b + (n - 1) * b * b + n * a * b + a * a + (gy ? (n * b + a) * nrhs : 0);
  const unsigned grid = (unsigned)std::min<int64_t>(16384, (total + 255) / 256);
  hipLaunchKernelGGL(grad_pattern_kernel, dim3(grid), dim3(256), 0, stream, p);
  return hipGetLastError();
}

hipError_t logdet_launch(int64_t n, int64_t b, int64_t a, const double* LD, const double* LT, double* out, void* work,
                         hipStream_t stream) {
  double* partial = static_cast<double*>(work);
  const int64_t nb = n + (a > 0 ? 1 : 0);
  hipLaunchKernelGGL(logdet_partial_kernel, dim3((unsigned)nb), dim3(256), 0, stream, LD, LT, n, b, a, partial);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(logdet_final_kernel, dim3(1), dim3(256), 0, stream, partial, nb, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------- solve

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// out[r] = sum_k M[r*ld + k] x[k] for the rows of this workgroup, batched over
// blockIdx.y (right-hand sides) and blockIdx.z (independent blocks).  tri = 0:
// k < K; tri = 1 (lower triangular M): only k < r0 + rows of the workgroup are
// read; tri = 2 (upper): only k >= r0.  Elements of a triangular M outside its
// triangle must be zero.
struct MvArgs {
  const double* M; int64_t ld, sMz;
  const double* x; int64_t sxy, sxz;
  double* out; int64_t soy, soz;
  int64_t rows, K;
  int tri;
};

// Wave w takes RPW consecutive rows; its lanes run along k in 64-wide chunks,
// CH chunks per trip, so RPW * CH loads per lane are in flight at once.  Rows
// past the end read the last row and columns past the end read column 0 (both
// inside the matrix) and contribute zero: no per-load branch.
template <int RPW, int CH>
__global__ __launch_bounds__(256) void matvec_rows_kernel(MvArgs p) {
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t y = blockIdx.y, z = blockIdx.z;
  const int64_t r0 = (int64_t)blockIdx.x * (4 * RPW);
  const int64_t rw = r0 + (int64_t)w * RPW;
  int64_t k0 = 0, k1 = p.K;
  if (p.tri == 1) k1 = std::min<int64_t>(p.K, r0 + 4 * RPW);
  if (p.tri == 2) k0 = r0;
  double s[RPW];
#pragma unroll
  for (int j = 0; j < RPW; ++j) s[j] = 0.0;
  if (k1 > k0) {
    const double* M = p.M + z * p.sMz;
    const double* x = p.x + y * p.sxy + z * p.sxz;
    int64_t roff[RPW];
#pragma unroll
    for (int j = 0; j < RPW; ++j) roff[j] = std::min<int64_t>(rw + j, p.rows - 1) * p.ld;
    for (int64_t kb = k0; kb < k1; kb += 64 * CH) {
      double xv[CH];
      int64_t kk[CH];
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        const int64_t k = kb + 64 * c + lane;
        const bool in = k < k1;
        kk[c] = in ? k : 0;
        xv[c] = in ? x[kk[c]] : 0.0;
      }
      double mv[RPW][CH];
#pragma unroll
      for (int j = 0; j < RPW; ++j)
#pragma unroll
        for (int c = 0; c < CH; ++c) mv[j][c] = M[roff[j] + kk[c]];
#pragma unroll
      for (int j = 0; j < RPW; ++j)
#pragma unroll
        for (int c = 0; c < CH; ++c) s[j] = __builtin_fma(mv[j][c], xv[c], s[j]);
    }
  }
#pragma unroll
  for (int j = 0; j < RPW; ++j) {
    const double t = wave_sum(s[j]);
    const int64_t r = rw + j;
    if (lane == 0 && r < p.rows) p.out[y * p.soy + z * p.soz + r] = t;
  }
}

static hipError_t matvec_rows(const MvArgs& a, int nrhs, int nz, hipStream_t s) {
  if (a.rows <= 0 || nrhs <= 0 || nz <= 0) return hipSuccess;
  // short rows: one row per wave and many workgroups; long rows: two per wave
  if (a.K <= 1024) {
    const unsigned gx = (unsigned)((a.rows + 3) / 4);
    hipLaunchKernelGGL((matvec_rows_kernel<1, 8>), dim3(gx, (unsigned)nrhs, (unsigned)nz), dim3(256), 0, s, a);
  } else {
    const unsigned gx = (unsigned)((a.rows + 7) / 8);
    hipLaunchKernelGGL((matvec_rows_kernel<2, 8>), dim3(gx, (unsigned)nrhs, (unsigned)nz), dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

// dst[z](c, r) = src[z](r, c) for rows x cols matrices (64 x 64 tiles through
// LDS; grid (tiles, 1, nz)).
__global__ __launch_bounds__(256) void transpose_kernel(const double* src, int64_t lds, int64_t ss, double* dst,
                                                        int64_t ldd, int64_t sd, int64_t rows, int64_t cols) {
  __shared__ double tile[64][65];
  const int64_t tc = (cols + 63) / 64;
  const int64_t tr = blockIdx.x / tc, tcol = blockIdx.x - tr * tc;
  const double* S = src + (int64_t)blockIdx.z * ss;
  double* Dm = dst + (int64_t)blockIdx.z * sd;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int rr = w; rr < 64; rr += 4) {
    const int64_t r = tr * 64 + rr, c = tcol * 64 + lane;
    if (r < rows && c < cols) tile[rr][lane] = S[r * lds + c];
  }
  __syncthreads();
  for (int cc = w; cc < 64; cc += 4) {
    const int64_t c = tcol * 64 + cc, r = tr * 64 + lane;
    if (r < rows && c < cols) Dm[c * ldd + r] = tile[lane][cc];
  }
}

static hipError_t transpose_launch(const double* src, int64_t lds, int64_t ss, double* dst, int64_t ldd, int64_t sd,
                                   int64_t rows, int64_t cols, int nz, hipStream_t s) {
  if (rows <= 0 || cols <= 0 || nz <= 0) return hipSuccess;
  const unsigned g = (unsigned)(((rows + 63) / 64) * ((cols + 63) / 64));
  hipLaunchKernelGGL(transpose_kernel, dim3(g, 1, (unsigned)nz), dim3(256), 0, s, src, lds, ss, dst, ldd, sd, rows,
                     cols);
  return hipGetLastError();
}

// ---------------------------------------------------------------- the chain of blocks
// Right-hand sides travel in groups of NR: 1 (vector FMAs) or 16 (one MFMA column
// block).  Element e of right-hand side j is at ((j / NR) N + e) NR + j % NR, so a
// group is one array of rows.  A phase of single groups is shorter (its tasks hand
// elements on, not flags) until their tasks, ceil(b / 16) per right-hand side,
// outnumber the CUs.  Solves with single / sixteen-wide groups (ms): 400 blocks of
// b = 64, 32 right-hand sides (128 tasks a phase) 4.2 / 6.2, 64 (256) 7.2 / 6.2; 256
// of b = 256, 8 (128) 3.1 / 4.3, 12 (192) 4.3 / 4.3, 16 (256) 5.1 / 4.3; 128 of b =
// 512, 5 (160) 2.5 / 2.7, 8 (256) 3.1 / 2.7; 64 of b = 1024, 4 (256) 2.6 / 3.3, 8
// (512) 4.0 / 3.3; 32 of b = 2048, 2 (256) 4.2 / 5.2, 4 (512) 5.3 / 5.2.  Single
// groups keep several copies of the vectors, so above SOLVE_SINGLE of them only
// where a copy is small.
constexpr int64_t SOLVE_SINGLE = 4;           // right-hand sides that always go singly
constexpr int64_t SOLVE_SINGLE_TASKS = 192;   // tasks of a phase up to which more of them do
constexpr int64_t SOLVE_SINGLE_SIZE = int64_t(1) << 25;  // and elements of all of them
constexpr int SOLVE_ROWS = 16;                // rows of a block's vector per task
static int solve_group(int64_t b, int64_t N, int64_t nrhs) {
  const bool few = nrhs * ((b + SOLVE_ROWS - 1) / SOLVE_ROWS) <= SOLVE_SINGLE_TASKS && nrhs * N <= SOLVE_SINGLE_SIZE;
  return nrhs <= SOLVE_SINGLE || few ? 1 : 16;
}
__host__ __device__ inline int64_t rhs_at(int64_t j, int64_t e, int64_t N, int NR) { return (j / NR * N + e) * NR + j % NR; }

// A vector element that no task has written yet (one NaN; a result with the
// same bits is stored as its neighbour).
constexpr unsigned long long SOLVE_PENDING = 0x7ff8b17ab17ab17aULL;

// One sweep over blocks [i0, i1) as one launch: per block two phases,
//   forward   t_i = y_i - L_{i,i-1} z_{i-1},    z_i = W_i t_i
//   backward  t_i = y_i - L_{i+1,i}^T x_{i+1},  x_i = W_i^T t_i
// each cut into tasks of SOLVE_ROWS rows of one group.  Tasks are taken from an
// atomic counter in phase order, so a task only waits for tasks of smaller
// tickets, which running workgroups own: no wait depends on how many workgroups
// are resident.  A task's matrix elements do not depend on the chain and are
// loaded before its wait; the transposed products read the matrix as it lies,
// SOLVE_ROWS columns (a cache line) per task.
//
// Groups of 16 work in place: z (x) takes the place of y's rows, which only the
// same rows' task of phase 0 reads, before them, and t is one block's, as every
// task of the next block's phase 0 waits for all of phase 1.  Single vectors
// carry their readiness, so y, t and z are arrays of their own.
struct ChainArgs {
  const double* LB; const double* W;  // W of block i0 on
  const double* y; double* t; double* z;  // phase 0 input, phase 0 and 1 outputs (groups of N, Nt, N rows)
  int* flags;                         // NR = 16: [block][phase][group][task]
  int* ctl;                           // ticket counter (64 bits), abort flag at ctl[2]
  int64_t n, b, N, Nt, i0, i1;           // Nt: N, or b (groups of 16: one block's t)
  int S, NG;                          // tasks per phase and group, groups
  long long ntasks, spin;             // spin: polls before a wait gives up (its outputs are then NaN)
};

struct ChainTask {
  int64_t i, r0, k0, k1;  // block, first row, k range
  const double* M;        // matrix (nullptr: empty k range)
  const double* x; const double* base; double* out;  // the group's rows of x's, y's (or null) and the output's block
  int s, g, ph;
};

template <bool BWD, int NR>
__device__ __forceinline__ ChainTask chain_task(const ChainArgs& p, long long t) {
  ChainTask k;
  const long long per = (long long)p.S * p.NG, q = t / per;
  const int rem = (int)(t - q * per);
  k.s = rem / p.NG;
  k.g = rem - k.s * p.NG;
  k.ph = (int)(q & 1);
  k.i = BWD ? p.i1 - 1 - (q >> 1) : p.i0 + (q >> 1);
  k.r0 = (int64_t)SOLVE_ROWS * k.s;
  const int64_t bb = p.b * p.b;
  const int64_t at = (k.g * p.N + k.i * p.b) * NR;
  double* const tb = p.t + (k.g * p.Nt + (NR == 1 ? k.i * p.b : 0)) * NR;
  if (k.ph == 0) {
    const bool has = BWD ? k.i < p.n - 1 : k.i > 0;
    k.M = has ? p.LB + (BWD ? k.i : k.i - 1) * bb : nullptr;
    k.x = p.z + at + (has ? (BWD ? p.b : -p.b) * NR : 0);
    k.k0 = 0;
    k.k1 = has ? p.b : 0;
    k.base = p.y + at;
    k.out = tb;
  } else {
    k.M = p.W + (k.i - p.i0) * bb;
    k.x = tb;
    k.k0 = BWD ? k.r0 : 0;
    k.k1 = BWD ? p.b : std::min<int64_t>(p.b, k.r0 + SOLVE_ROWS);
    k.base = nullptr;
    k.out = p.z + at;
  }
  return k;
}

__device__ __forceinline__ long long chain_ticket(const ChainArgs& p, long long* sh, int tid) {
  __syncthreads();  // the last task's reads of *sh and of the shared arrays
  if (tid == 0) *sh = (long long)atomicAdd((unsigned long long*)p.ctl, 1ULL);
  __syncthreads();
  const long long t = *sh;
  const int lo = __builtin_amdgcn_readfirstlane((int)t), hi = __builtin_amdgcn_readfirstlane((int)(t >> 32));
  return ((long long)hi << 32) | (unsigned)lo;
}

// p[0] + p[step] + ... + p[7 step], pairwise
__device__ __forceinline__ double sum8(const double* p, int step) {
  return ((p[0] + p[step]) + (p[2 * step] + p[3 * step])) + ((p[4 * step] + p[5 * step]) + (p[6 * step] + p[7 * step]));
}

__device__ __forceinline__ bool chain_aborted(const ChainArgs& p) {
  return __hip_atomic_load(p.ctl + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
}

// One right-hand side per group.  The vectors carry their own readiness: every
// element starts as SOLVE_PENDING, and a reader polls the elements it needs.
// That leaves one store and one load of latency between phases, where a flag
// behind the stores would add the wait for them and its own round trip.
template <bool BWD>
__global__ __launch_bounds__(512, 2) void solve_chain_kernel(ChainArgs p) {
  constexpr int KC = 1024;
  __shared__ double xs[KC];
  __shared__ double red[8 * SOLVE_ROWS];
  __shared__ long long ticket;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (;;) {
    const long long tk = chain_ticket(p, &ticket, tid);
    if (tk >= p.ntasks) break;
    const ChainTask q = chain_task<BWD, 1>(p, tk);
    const double* x = q.x;
    // forward: rows 2w, 2w + 1 of the task, lanes along k; backward: column
    // tid % 16, rows tid / 16 + 32 j
    const int64_t ra = std::min<int64_t>(q.r0 + 2 * w, p.b - 1), rb = std::min<int64_t>(q.r0 + 2 * w + 1, p.b - 1);
    const int64_t cc = std::min<int64_t>(q.r0 + (tid & 15), p.b - 1);
    const int rg = tid >> 4;
    double m[32], sum[4] = {0.0, 0.0, 0.0, 0.0};  // four short sums per thread, then trees
    for (int64_t kc = q.k0; kc < q.k1; kc += KC) {
      const int64_t left = q.k1 - kc;
      if constexpr (!BWD) {
#pragma unroll
        for (int c = 0; c < 16; ++c) {
          const int64_t k = kc + std::min<int64_t>(64 * c + lane, left - 1);
          m[c] = q.M[ra * p.b + k];
          m[16 + c] = q.M[rb * p.b + k];
        }
      } else {
#pragma unroll
        for (int j = 0; j < 32; ++j) m[j] = q.M[(kc + std::min<int64_t>(rg + 32 * j, left - 1)) * p.b + cc];
      }
      if (kc > q.k0) __syncthreads();  // xs is read
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int e = tid + 512 * h;
        double v = 0.0;
        if (e < left) {
          v = ld_dev(x + kc + e);
          long long polls = 0;
          while (__builtin_bit_cast(unsigned long long, v) == SOLVE_PENDING) {
            if (++polls > p.spin || ((polls & 63) == 0 && chain_aborted(p))) {
              __hip_atomic_store(p.ctl + 2, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              break;
            }
            __builtin_amdgcn_s_sleep(1);
            v = ld_dev(x + kc + e);
          }
        }
        xs[e] = v;
      }
      __syncthreads();
      // elements past the range were read from its last one: they count as zero
      if constexpr (!BWD) {
#pragma unroll
        for (int c = 0; c < 16; ++c) {
          const bool in = 64 * c + lane < left;
          sum[c & 1] = __builtin_fma(in ? m[c] : 0.0, xs[64 * c + lane], sum[c & 1]);
          sum[2 + (c & 1)] = __builtin_fma(in ? m[16 + c] : 0.0, xs[64 * c + lane], sum[2 + (c & 1)]);
        }
      } else {
#pragma unroll
        for (int j = 0; j < 32; ++j)
          sum[j & 3] = __builtin_fma(rg + 32 * j < left ? m[j] : 0.0, xs[rg + 32 * j], sum[j & 3]);
      }
    }
    if constexpr (!BWD) {
      const double s0 = wave_sum(sum[0] + sum[1]), s1 = wave_sum(sum[2] + sum[3]);
      if (lane < 2) red[2 * w + lane] = lane ? s1 : s0;
    } else {
      double s0 = (sum[0] + sum[1]) + (sum[2] + sum[3]);
      s0 += __shfl_xor(s0, 16, 64);
      s0 += __shfl_xor(s0, 32, 64);
      if (lane < 16) red[16 * w + lane] = s0;
    }
    __syncthreads();
    if (tid < SOLVE_ROWS && q.r0 + tid < p.b) {
      double v = BWD ? sum8(red + tid, 16) : red[tid];
      if (q.base) v = q.base[q.r0 + tid] - v;
      if (__builtin_bit_cast(unsigned long long, v) == SOLVE_PENDING)
        v = __builtin_bit_cast(double, SOLVE_PENDING ^ 1ULL);
      st_dev(q.out + q.r0 + tid, v);
    }
  }
}

// Sixteen right-hand sides per group on MFMA: a task's 16 x 16 output is
// accumulated by eight waves, each a share of the k range, and summed pairwise.
// Readiness is a flag per task: a poll of every element, as for one right-hand
// side, would repeat 128 bytes per row.
template <bool BWD>
__global__ __launch_bounds__(512, 2) void solve_chain16_kernel(ChainArgs p) {
  constexpr int KC = 512, Q = KC / 128;  // k per chunk, groups of 16 k per wave
  __shared__ double red[8 * 256];
  __shared__ long long ticket;
  __shared__ int good;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int mn = lane & 15, g4 = 4 * (lane >> 4);
  for (;;) {
    const long long tk = chain_ticket(p, &ticket, tid);
    if (tk >= p.ntasks) break;
    const ChainTask q = chain_task<BWD, 16>(p, tk);
    const double* x = q.x;
    const int64_t rm = std::min<int64_t>(q.r0 + mn, p.b - 1);
    const double* M = q.M + (BWD ? rm : rm * p.b);
    struct __attribute__((packed, aligned(8))) Row4 { d4 v; };  // four k of a row, any 8-byte alignment
    const bool live = tid < 256 && q.r0 + (tid >> 4) < p.b;
    const double base = live && q.base ? ld_dev(q.base + q.r0 * 16 + tid) : 0.0;
    bool ok = true;
    d4 acc[2 * Q] = {};  // two chains per group of k: short sums, added pairwise at the end
    for (int64_t kc = q.k0; kc < q.k1; kc += KC) {
      double a[Q][4], v[Q][4];
#pragma unroll
      for (int u = 0; u < Q; ++u) {
        const int64_t k = kc + 16 * (w + 8 * u);
        if (!BWD && k + 16 <= q.k1) {
          const d4 r = reinterpret_cast<const Row4*>(M + k + g4)->v;
#pragma unroll
          for (int j = 0; j < 4; ++j) a[u][j] = r[j];
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) a[u][j] = M[std::min<int64_t>(k + g4 + j, q.k1 - 1) * (BWD ? p.b : 1)];
        }
      }
      if (kc == q.k0) {
        // the slices of the previous phase that this task reads
        const int64_t ib = q.ph ? q.i : BWD ? q.i + 1 : q.i - 1;
        const int* f = p.flags + ((ib * 2 + (1 - q.ph)) * p.NG + q.g) * p.S;
        const int f0 = (BWD && q.ph) ? q.s : 0, f1 = (!BWD && q.ph) ? q.s + 1 : p.S;
        if (w == 0) {
          long long polls = 0;
          for (int e = f0 + lane; e < f1; e += 64)
            while (!flag_set(f + e)) {
              if (++polls > p.spin || ((polls & 63) == 0 && chain_aborted(p))) {
                __hip_atomic_store(p.ctl + 2, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
              }
              __builtin_amdgcn_s_sleep(1);
            }
          if (tid == 0) good = chain_aborted(p) ? 0 : 1;
        }
        __syncthreads();
        ok = good != 0;
      }
#pragma unroll
      for (int u = 0; u < Q; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int64_t k = kc + 16 * (w + 8 * u) + g4 + j;
          v[u][j] = ld_dev(x + std::min<int64_t>(k, q.k1 - 1) * 16 + mn);
        }
#pragma unroll
      for (int u = 0; u < Q; ++u)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const bool in = kc + 16 * (w + 8 * u) + g4 + j < q.k1;
          acc[2 * u + (j & 1)] = mfma16(in ? a[u][j] : 0.0, in ? v[u][j] : 0.0, acc[2 * u + (j & 1)]);
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      red[w * 256 + acc_row(lane, j) * 16 + acc_col(lane)] = ((acc[0][j] + acc[1][j]) + (acc[2][j] + acc[3][j])) +
                                                             ((acc[4][j] + acc[5][j]) + (acc[6][j] + acc[7][j]));
    __syncthreads();
    if (live) {
      double v = sum8(red + tid, 256);
      if (q.base) v = base - v;
      st_dev(q.out + q.r0 * 16 + tid, ok ? v : __builtin_nan(""));
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    // every wave's stores are complete at device scope: the flag needs no
    // release of its own (which would write the L2 back), nor its readers an
    // acquire (which would invalidate it), as x is read at device scope too
    if (tid == 0)
      __hip_atomic_store(p.flags + ((q.i * 2 + q.ph) * p.NG + q.g) * p.S + q.s, 1, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
  }
}

// The right-hand sides into groups (padded with zero columns), the forward
// sweep's vectors to pending (single groups), and the flags and ticket counters
// to zero.
__global__ __launch_bounds__(256) void solve_gather_kernel(const double* rhs, int64_t nrhs, int64_t N, int NR, int64_t NG,
                                                           double* y, unsigned long long* t, unsigned long long* z, int64_t npend,
                                                           int* zero, int64_t nzero) {
  const int64_t t0 = (int64_t)blockIdx.x * 256 + threadIdx.x, step = (int64_t)gridDim.x * 256;
  for (int64_t e = t0; e < NG * N * NR; e += step) {
    const int64_t row = e / NR, j = row / N * NR + e % NR;
    y[e] = j < nrhs ? rhs[row % N * nrhs + j] : 0.0;
  }
  for (int64_t e = t0; e < npend; e += step) t[e] = z[e] = SOLVE_PENDING;
  for (int64_t e = t0; e < nzero; e += step) zero[e] = 0;
}
// x in the caller's layout; NaN throughout if a wait of any sweep gave up (part of
// x may then be right, and nothing else would tell).
__global__ __launch_bounds__(256) void solve_scatter_kernel(double* rhs, int64_t nrhs, int64_t N, int64_t nb, int NR,
                                                            const double* x, const double* xn, const int* ctl,
                                                            int64_t nsweeps) {
  int gave_up = 0;
  for (int64_t c = 0; c < nsweeps; ++c) gave_up |= ctl[4 * c + 2];
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < N * nrhs; e += (int64_t)gridDim.x * 256) {
    const int64_t r = e / nrhs, j = e - r * nrhs;
    const double v = r < nb ? x[rhs_at(j, r, N, NR)] : xn[j * (N - nb) + r - nb];
    rhs[e] = gave_up ? __builtin_nan("") : v;
  }
}

// ptip(j, i, r) = sum_k L_{n,i}[r][k] z_i(j)[k] for one group of 16 and TIP_ROWS
// rows per workgroup: thread (k residue, right-hand side), residues summed in
// order.  Bound by reading z_i from the L2, once per TIP_ROWS rows (once per row:
// n=16, b=512, a=2048, 64 right-hand sides 4.25 ms a solve against 3.89).
constexpr int TIP_ROWS = 4;
__global__ __launch_bounds__(256) void solve_tip16_kernel(const double* LR, int64_t b, int64_t a, int64_t n, int64_t N,
                                                          const double* z, double* ptip) {
  __shared__ double red[TIP_ROWS * 256];
  const int64_t r0 = (int64_t)TIP_ROWS * blockIdx.x, i = blockIdx.y, g = blockIdx.z;
  const double* zi = z + (g * N + i * b) * 16;
  const double* M[TIP_ROWS];  // rows past the end read the last one; they are not stored
  double s[TIP_ROWS] = {};
#pragma unroll
  for (int q = 0; q < TIP_ROWS; ++q) M[q] = LR + (i * a + std::min<int64_t>(r0 + q, a - 1)) * b;
  for (int64_t k = threadIdx.x >> 4; k < b; k += 16) {
    const double zk = zi[k * 16 + (threadIdx.x & 15)];
#pragma unroll
    for (int q = 0; q < TIP_ROWS; ++q) s[q] = __builtin_fma(M[q][k], zk, s[q]);
  }
#pragma unroll
  for (int q = 0; q < TIP_ROWS; ++q) red[256 * q + threadIdx.x] = s[q];
  __syncthreads();
  const int q = threadIdx.x >> 4, j = threadIdx.x & 15;
  if (q < TIP_ROWS && r0 + q < a) {
    double t = red[256 * q + j];
    for (int u = 1; u < 16; ++u) t += red[256 * q + 16 * u + j];
    ptip[((g * n + i) * a + r0 + q) * 16 + j] = t;
  }
}

// t[j][r] = y(j)[n*b + r] - sum_i ptip(j, i, r), the blocks summed in order.
__global__ __launch_bounds__(256) void solve_tip_rhs_kernel(const double* y, int64_t N, int64_t nb, const double* ptip,
                                                            int64_t n, int64_t a, int NR, double* t) {
  const int64_t j = blockIdx.y;
  for (int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x; r < a; r += (int64_t)gridDim.x * 256) {
    double acc = 0.0;
    for (int64_t i = 0; i < n; ++i) acc += ptip[rhs_at(j, i * a + r, n * a, NR)];
    t[j * a + r] = y[rhs_at(j, nb + r, N, NR)] - acc;
  }
}

// z(j)[i*b + c] -= sum_{r<a} L_{n,i}[r][c] x_n(j)[r] for every block i < n
// (the arrow terms of the backward sweep: x_n is final before it starts), and
// that sweep's vectors to pending where they carry their readiness (t and x, not
// null: the same places as the forward sweep's t and y, which it is done with).
__global__ __launch_bounds__(256) void solve_arrow_terms_kernel(const double* LR, int64_t n, int64_t b, int64_t a,
                                                                const double* xn, int64_t nrhs, int64_t N, int NR, double* z,
                                                                unsigned long long* t, unsigned long long* x) {
  const int64_t g = blockIdx.y;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n * b * NR; e += (int64_t)gridDim.x * 256) {
    const int64_t row = e / NR, j = g * NR + e % NR, i = row / b, c = row - i * b;
    if (t) t[g * N + row] = x[g * N + row] = SOLVE_PENDING;
    if (j >= nrhs || a == 0) continue;
    const double* M = LR + i * a * b + c;
    const double* xt = xn + j * a;
    double acc = 0.0;
    for (int64_t r = 0; r < a; ++r) acc = __builtin_fma(M[r * b], xt[r], acc);
    z[g * N * NR + e] -= acc;
  }
}

// Workspace layout of one solve.  C blocks per chunk of inverses: the whole
// matrix when its inverses fit in the budget beside the scratch that forms them
// (C1 blocks at a time), else chunks; the backward sweep then forms all but the
// last one again.
struct SolvePlan {
  int64_t C, C1, nchunks, NG, Nt, npend, nzero;
  int NR, S;
  size_t off_W, off_T1, off_WT, off_WTt, off_y, off_t, off_z, off_zero, off_tb, off_t2, off_xn, off_ptip, bytes;
};

static SolvePlan solve_plan(int64_t n, int64_t b, int64_t a, int64_t nrhs) {
  SolvePlan sp{};
  const size_t per_block = 8 * (size_t)b * (size_t)b;
  const size_t budget = size_t(2) << 30;
  sp.C1 = std::max<int64_t>(1, std::min<int64_t>(n, (int64_t)((budget >> 2) / per_block)));
  sp.C = std::max<int64_t>(1, std::min<int64_t>(n, (int64_t)(budget / per_block) - sp.C1));
  sp.C1 = std::min(sp.C1, sp.C);
  sp.nchunks = (n + sp.C - 1) / sp.C;
  const int64_t N = n * b + a;
  sp.NR = solve_group(b, N, nrhs);
  sp.NG = (nrhs + sp.NR - 1) / sp.NR;
  sp.S = (int)((b + SOLVE_ROWS - 1) / SOLVE_ROWS);
  const int64_t nv = sp.NG * N * sp.NR;
  sp.Nt = sp.NR > 1 ? b : N;
  sp.npend = sp.NR > 1 ? 0 : nv;  // elements of t and of z that start as pending
  // per sweep and chunk a ticket counter and an abort flag (4 ints), then the flags of both sweeps
  sp.nzero = 8 * sp.nchunks + (sp.NR > 1 ? 4 * n * sp.NG * sp.S : 0);
  size_t off = 0;
  auto take = [&](size_t x) { size_t o = off; off += (std::max<size_t>(x, 8) + 255) & ~size_t(255); return o; };
  sp.off_W = take(per_block * (size_t)sp.C);
  sp.off_T1 = take(per_block * (size_t)sp.C1);
  sp.off_WT = take(8 * (size_t)(a * a));
  sp.off_WTt = take(8 * (size_t)(a * a));
  sp.off_y = take(8 * (size_t)nv);
  sp.off_t = take(8 * (size_t)(sp.NG * sp.Nt * sp.NR));
  sp.off_z = sp.NR > 1 ? sp.off_y : take(8 * (size_t)nv);
  sp.off_zero = take(4 * (size_t)sp.nzero);
  sp.off_tb = take(8 * (size_t)(a * nrhs));
  sp.off_t2 = take(8 * (size_t)(a * nrhs));
  sp.off_xn = take(8 * (size_t)(a * nrhs));
  sp.off_ptip = take(8 * (size_t)(n * a * sp.NG * sp.NR));
  sp.bytes = off;
  return sp;
}

size_t solve_work_bytes(int64_t n, int64_t b, int64_t a, int64_t nrhs) { return solve_plan(n, b, a, nrhs).bytes; }

hipError_t solve_launch(int64_t n, int64_t b, int64_t a, const double* LD, const double* LB, const double* LR,
                        const double* LT, double* rhs, int64_t nrhs, void* work, hipStream_t stream) {
  const SolvePlan sp = solve_plan(n, b, a, nrhs);
  char* w = static_cast<char*>(work);
  auto at = [&](size_t off) { return reinterpret_cast<double*>(w + off); };
  double *W = at(sp.off_W), *T1 = at(sp.off_T1), *WT = at(sp.off_WT), *WTt = at(sp.off_WTt), *y = at(sp.off_y);
  double *tb = at(sp.off_tb), *t2 = at(sp.off_t2), *xn = at(sp.off_xn), *ptip = at(sp.off_ptip);
  const int64_t N = n * b + a, bb = b * b, ab = a * b, nv = sp.NG * N * sp.NR;
  double *t = at(sp.off_t), *z = at(sp.off_z);
  using Bits = unsigned long long;
  int* ctl = reinterpret_cast<int*>(w + sp.off_zero);
  int* flags = ctl + 8 * sp.nchunks;
  const int nr = (int)nrhs;
  auto ok = [&]() { return hipGetLastError(); };
  auto blocks = [](int64_t count) { return dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>(4096, (count + 255) / 256))); };

  hipLaunchKernelGGL(solve_gather_kernel, blocks(nv), dim3(256), 0, stream, rhs, nrhs, N, sp.NR, sp.NG, y,
                     reinterpret_cast<Bits*>(t), reinterpret_cast<Bits*>(z), sp.npend, ctl, sp.nzero);
  if (hipError_t e = ok()) return e;

  auto invert_chunk = [&](int64_t i0, int64_t cnt) -> hipError_t {
    BTA_TRY_E(fill_zero_launch(W, (size_t)(cnt * bb), stream));
    for (int64_t q = 0; q < cnt; q += sp.C1)
      BTA_TRY_E(trtri_batched(LD + (i0 + q) * bb, b, bb, W + q * bb, T1, b, bb, (int)b, (int)std::min(sp.C1, cnt - q), stream,
                              0, 0));
    return hipSuccess;
  };
  // one sweep over a chunk: enough workgroups for two phases in flight (the
  // second has its matrix elements loaded when the first ends), at most one a CU
  auto chain = [&](bool bwd, int64_t c) -> hipError_t {
    ChainArgs p{};
    p.LB = LB; p.W = W; p.y = bwd ? z : y; p.t = t; p.z = bwd ? y : z;
    p.flags = flags + (bwd ? 2 * n * sp.NG * sp.S : 0);
    p.ctl = ctl + 4 * (2 * c + (bwd ? 1 : 0));
    p.n = n; p.b = b; p.N = N; p.Nt = sp.Nt; p.i0 = c * sp.C; p.i1 = std::min(n, p.i0 + sp.C);
    p.S = sp.S; p.NG = (int)sp.NG;
    p.ntasks = 2 * (p.i1 - p.i0) * sp.NG * sp.S;
    p.spin = g_wait_limit;
    const long long grid = std::min<long long>(std::max(1, device_cu_count()), 2 * sp.NG * sp.S);
    auto kernel = sp.NR == 1 ? (bwd ? solve_chain_kernel<true> : solve_chain_kernel<false>)
                             : (bwd ? solve_chain16_kernel<true> : solve_chain16_kernel<false>);
    hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(512), 0, stream, p);
    return ok();
  };

  for (int64_t c = 0; c < sp.nchunks; ++c) {
    BTA_TRY_E(invert_chunk(c * sp.C, std::min<int64_t>(sp.C, n - c * sp.C)));
    BTA_TRY_E(chain(false, c));
  }

  // ---- the tip: z_n = W_T (y_n - sum_i L_{n,i} z_i), x_n = W_T^T z_n, then
  // the arrow terms of every block's backward right-hand side
  if (a > 0) {
    if (sp.NR == 1) {
      MvArgs pp{};
      pp.M = LR; pp.ld = b; pp.sMz = ab;
      pp.x = z; pp.sxy = N; pp.sxz = b;
      pp.out = ptip; pp.soy = n * a; pp.soz = a;
      pp.rows = a; pp.K = b; pp.tri = 0;
      BTA_TRY_E(matvec_rows(pp, nr, (int)n, stream));
    } else {
      const dim3 g((unsigned)((a + TIP_ROWS - 1) / TIP_ROWS), (unsigned)n, (unsigned)sp.NG);
      hipLaunchKernelGGL(solve_tip16_kernel, g, dim3(256), 0, stream, LR, b, a, n, N, z, ptip);
      if (hipError_t e = ok()) return e;
    }
    hipLaunchKernelGGL(solve_tip_rhs_kernel, dim3((unsigned)((a + 255) / 256), (unsigned)nrhs), dim3(256), 0, stream, y, N,
                       n * b, ptip, n, a, sp.NR, t2);
    if (hipError_t e = ok()) return e;
    BTA_TRY_E(fill_zero_launch(WT, (size_t)(a * a), stream));
    BTA_TRY_E(trtri_batched(LT, a, 0, WT, WTt, a, 0, (int)a, 1, stream, 0, 0));
    BTA_TRY_E(transpose_launch(WT, a, 0, WTt, a, 0, a, a, 1, stream));
    MvArgs fz{};
    fz.M = WT; fz.ld = a;
    fz.x = t2; fz.sxy = a;
    fz.out = tb; fz.soy = a;
    fz.rows = a; fz.K = a; fz.tri = 1;
    BTA_TRY_E(matvec_rows(fz, nr, 1, stream));
    MvArgs bx{};
    bx.M = WTt; bx.ld = a;
    bx.x = tb; bx.sxy = a;
    bx.out = xn; bx.soy = a;
    bx.rows = a; bx.K = a; bx.tri = 2;
    BTA_TRY_E(matvec_rows(bx, nr, 1, stream));
  }
  if (a > 0 || sp.npend > 0) {
    dim3 g = blocks(n * b * sp.NR);
    g.y = (unsigned)sp.NG;
    hipLaunchKernelGGL(solve_arrow_terms_kernel, g, dim3(256), 0, stream, LR, n, b, a, xn, nrhs, N, sp.NR, z,
                       sp.npend ? reinterpret_cast<Bits*>(t) : nullptr, sp.npend ? reinterpret_cast<Bits*>(y) : nullptr);
    if (hipError_t e = ok()) return e;
  }

  for (int64_t c = sp.nchunks - 1; c >= 0; --c) {
    if (c < sp.nchunks - 1) BTA_TRY_E(invert_chunk(c * sp.C, sp.C));
    BTA_TRY_E(chain(true, c));
  }
  hipLaunchKernelGGL(solve_scatter_kernel, blocks(N * nrhs), dim3(256), 0, stream, rhs, nrhs, N, n * b, sp.NR, y, xn, ctl,
                     2 * sp.nchunks);
  return ok();
}

}  // namespace bta

// Right-hand sides per group of a solve (1 or 16).
BTA_TESTING_API int bta_internal_solve_group(int64_t n, int64_t b, int64_t a, int64_t nrhs) {
  return bta::solve_group(b, n * b + a, nrhs);
}
