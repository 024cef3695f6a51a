// FP64 dense kernels for the projected (subspace) problems of at most 512 vectors.  All of
// them are chains of dependent steps: what counts is the latency of a step, so short vectors
// and small matrices sit in registers or LDS and the work of a step is spread over just the
// waves that shorten it.
//
// Symmetric eigensolver (syev_kernel): Householder reduction to tridiagonal form with explicit
// accumulation of the orthogonal factor, then the implicit QL iteration with
// Wilkinson-type shifts (the textbook tred2/tql2 pair), with the scalar
// recurrence run by one thread and each rotation sequence applied to all rows of
// the eigenvector matrix in parallel.  Eigenvalues are returned ascending.
#include <algorithm>
#include <cfloat>
#include <vector>

#include "solver.h"

namespace ppw {
namespace {

constexpr int kT = 1024;
constexpr int kMaxN = 512;

__device__ double block_reduce_sum(double v, double* red) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) red[wave] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0) {
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) s += red[w];
    red[32] = s;
  }
  __syncthreads();
  s = red[32];
  __syncthreads();
  return s;
}

// Sum over the wave, in every lane: row shifts and row broadcasts (about 150 cycles, a quarter
// of the time of lane permutes through LDS).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_get(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, true);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_total(double v) {
  v += dpp_get<0x111, 0xf>(v);  // row_shr 1, 2, 4, 8: lane 15 of each row of 16 holds its sum
  v += dpp_get<0x112, 0xf>(v);
  v += dpp_get<0x114, 0xf>(v);
  v += dpp_get<0x118, 0xf>(v);
  v += dpp_get<0x142, 0xa>(v);  // row_bcast 15 into rows 1 and 3
  v += dpp_get<0x143, 0xc>(v);  // row_bcast 31 into rows 2 and 3
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), 63);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), 63);
  return __hiloint2double(hi, lo);
}

// Largest of non-negative values over the wave, in every lane.
__device__ __forceinline__ double wave_max(double v) {
  v = fmax(v, dpp_get<0x111, 0xf>(v));
  v = fmax(v, dpp_get<0x112, 0xf>(v));
  v = fmax(v, dpp_get<0x114, 0xf>(v));
  v = fmax(v, dpp_get<0x118, 0xf>(v));
  v = fmax(v, dpp_get<0x142, 0xa>(v));
  v = fmax(v, dpp_get<0x143, 0xc>(v));
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63),
                          __builtin_amdgcn_readlane(__double2loint(v), 63));
}
__device__ __forceinline__ double lane_value(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// W: n x n working copy (row-major, symmetric), Zc: n x n, column-major eigenvectors.
// NT threads (1024 for the large projected problems; one wave for n <= 64, where the
// block-wide barriers of the rotation sweeps cost more than the arithmetic).  INLDS
// (n <= 64): W and Zr live in LDS instead of the scratch arrays passed in, so the
// sweeps run at LDS latency rather than at that of an L2 shared with concurrent GEMMs.
template <int NT, bool INLDS>
__global__ __launch_bounds__(NT) void syev_kernel(int n, const double* __restrict__ A, double* __restrict__ w,
                                                  double* __restrict__ Z, double* __restrict__ W,
                                                  double* __restrict__ Zr) {
  __shared__ double lds_w[INLDS ? 64 * 64 : 1], lds_z[INLDS ? 64 * 64 : 1];
  if (INLDS) {
    W = lds_w;
    Zr = lds_z;
  }
  __shared__ double u[kMaxN];
  __shared__ double q[kMaxN];
  __shared__ double d[kMaxN];
  __shared__ double e[kMaxN];
  __shared__ double cs[kMaxN];
  __shared__ double sn[kMaxN];
  __shared__ double red[40];
  __shared__ int ctl[4];
  const int tid = threadIdx.x;
  const long nn = (long)n * n;
  for (long i = tid; i < nn; i += NT) W[i] = A[i];
  __syncthreads();

  // ---- Householder tridiagonalization (W <- H W H, u_k stored in column k) ----
  for (int k = 0; k + 2 < n; ++k) {
    const int m = n - k - 1;  // length of the reflected part (rows k+1..n-1)
    double part = 0.0;
    for (int r = tid; r < m; r += NT) {
      const double x = W[(long)(k + 1 + r) * n + k];
      part += x * x;
    }
    const double xx = block_reduce_sum(part, red);
    const double x0 = W[(long)(k + 1) * n + k];
    const double xnorm = sqrt(xx);
    if (xnorm == 0.0) {
      if (tid == 0) {
        d[k] = W[(long)k * n + k];
        e[k] = 0.0;
      }
      for (int r = tid; r < m; r += NT) u[r] = 0.0;
      __syncthreads();
      for (int r = tid; r < m; r += NT) W[(long)(k + 1 + r) * n + k] = 0.0;
      __syncthreads();
      continue;
    }
    const double alpha = x0 > 0 ? -xnorm : xnorm;
    // v = x - alpha e1, |v|^2 = 2 xnorm^2 - 2 x0 alpha
    const double vnorm = sqrt(2.0 * xx - 2.0 * x0 * alpha);
    for (int r = tid; r < m; r += NT) {
      const double x = W[(long)(k + 1 + r) * n + k];
      u[r] = (r == 0 ? x - alpha : x) / vnorm;
    }
    __syncthreads();
    // p = A22 u (column form, symmetric)
    for (int r = tid; r < m; r += NT) q[r] = 0.0;
    __syncthreads();
    for (int r = tid; r < m; r += NT) {
      double acc = 0.0;
      for (int cc = 0; cc < m; ++cc) acc += W[(long)(k + 1 + cc) * n + (k + 1 + r)] * u[cc];
      q[r] = acc;
    }
    __syncthreads();
    double kp = 0.0;
    for (int r = tid; r < m; r += NT) kp += u[r] * q[r];
    const double K = block_reduce_sum(kp, red);
    for (int r = tid; r < m; r += NT) q[r] = q[r] - K * u[r];
    __syncthreads();
    // A22 <- A22 - 2 (u q^T + q u^T)
    const long mm = (long)m * m;
    for (long idx = tid; idx < mm; idx += NT) {
      const int r = (int)(idx / m), cc = (int)(idx % m);
      W[(long)(k + 1 + r) * n + (k + 1 + cc)] -= 2.0 * (u[r] * q[cc] + q[r] * u[cc]);
    }
    if (tid == 0) {
      d[k] = W[(long)k * n + k];
      e[k] = alpha;
    }
    __syncthreads();
    for (int r = tid; r < m; r += NT) W[(long)(k + 1 + r) * n + k] = u[r];
    __syncthreads();
  }
  if (tid == 0) {
    if (n >= 2) {
      d[n - 2] = W[(long)(n - 2) * n + (n - 2)];
      e[n - 2] = W[(long)(n - 1) * n + (n - 2)];
    }
    d[n - 1] = W[(long)(n - 1) * n + (n - 1)];
    e[n - 1] = 0.0;
  }
  // ---- Q = H_0 H_1 ... H_{n-3}, accumulated backwards into Zr (row-major) ----
  for (long i = tid; i < nn; i += NT) Zr[i] = ((i / n) == (i % n)) ? 1.0 : 0.0;
  __syncthreads();
  for (int k = n - 3; k >= 0; --k) {
    const int m = n - k - 1;
    for (int r = tid; r < m; r += NT) u[r] = W[(long)(k + 1 + r) * n + k];
    __syncthreads();
    // t_c = sum_r u_r Z[k+1+r][k+1+c]
    for (int cc = tid; cc < m; cc += NT) {
      double acc = 0.0;
      for (int r = 0; r < m; ++r) acc += u[r] * Zr[(long)(k + 1 + r) * n + (k + 1 + cc)];
      q[cc] = acc;
    }
    __syncthreads();
    const long mm = (long)m * m;
    for (long idx = tid; idx < mm; idx += NT) {
      const int r = (int)(idx / m), cc = (int)(idx % m);
      Zr[(long)(k + 1 + r) * n + (k + 1 + cc)] -= 2.0 * u[r] * q[cc];
    }
    __syncthreads();
  }
  // column-major copy for the rotation phase: W[c*n + r] = Zr[r*n + c]
  for (long idx = tid; idx < nn; idx += NT) {
    const long r = idx / n, cc = idx % n;
    W[cc * n + r] = Zr[idx];
  }
  __syncthreads();
  double* Zc = W;

  // ---- implicit QL on (d, e) ----
  for (int l = 0; l < n; ++l) {
    int iter = 0;
    while (true) {
      if (tid == 0) {
        int mm = l;
        for (; mm < n - 1; ++mm) {
          const double dd = fabs(d[mm]) + fabs(d[mm + 1]);
          if (fabs(e[mm]) <= DBL_EPSILON * dd) break;
        }
        ctl[0] = mm;
        int nrot = 0;
        if (mm != l && iter < 100) {
          double g = (d[l + 1] - d[l]) / (2.0 * e[l]);
          double r = hypot(g, 1.0);
          g = d[mm] - d[l] + e[l] / (g + copysign(r, g));
          double s = 1.0, c = 1.0, p = 0.0;
          int i = mm - 1;
          bool early = false;
          for (; i >= l; --i) {
            const double f = s * e[i];
            const double b = c * e[i];
            r = hypot(f, g);
            e[i + 1] = r;
            if (r == 0.0) {
              d[i + 1] -= p;
              e[mm] = 0.0;
              early = true;
              break;
            }
            s = f / r;
            c = g / r;
            g = d[i + 1] - p;
            r = (d[i] - g) * s + 2.0 * c * b;
            p = s * r;
            d[i + 1] = g + p;
            g = c * r - b;
            cs[nrot] = c;
            sn[nrot] = s;
            ++nrot;
          }
          if (!early) {
            d[l] -= p;
            e[l] = g;
            e[mm] = 0.0;
          }
        }
        ctl[1] = nrot;
        ctl[2] = (mm != l && iter >= 100) ? 1 : 0;
      }
      __syncthreads();
      const int mm = ctl[0], nrot = ctl[1];
      const bool done = mm == l || ctl[2];
      // every thread holds its copy of ctl before thread 0 may rewrite it (for the
      // next sweep or the next l); without this barrier a late wave can read the
      // next values, miss the break and spin on a ctl that no thread updates
      __syncthreads();
      if (done) break;
      // apply rotations i = mm-1, mm-2, ... to columns (i, i+1) of Z, one row per thread
      for (int row = tid; row < n; row += NT) {
        for (int t = 0; t < nrot; ++t) {
          const int i = mm - 1 - t;
          const double c = cs[t], s = sn[t];
          double* zi = Zc + (long)i * n + row;
          double* zj = Zc + (long)(i + 1) * n + row;
          const double f = *zj;
          *zj = s * (*zi) + c * f;
          *zi = c * (*zi) - s * f;
        }
      }
      __syncthreads();
      ++iter;
    }
  }
  __syncthreads();
  // ---- sort ascending (selection order by one thread), write outputs ----
  __shared__ int perm[kMaxN];
  if (tid == 0) {
    for (int i = 0; i < n; ++i) perm[i] = i;
    for (int i = 0; i < n; ++i) {
      int best = i;
      for (int j = i + 1; j < n; ++j)
        if (d[perm[j]] < d[perm[best]]) best = j;
      const int t = perm[i];
      perm[i] = perm[best];
      perm[best] = t;
    }
  }
  __syncthreads();
  for (int i = tid; i < n; i += NT) w[i] = d[perm[i]];
  for (long idx = tid; idx < nn; idx += NT) {
    const long r = idx / n, cc = idx % n;
    Z[idx] = Zc[(long)perm[cc] * n + r];
  }
}

// Panel of the blocked Cholesky: columns j0..j0+jb-1 (jb <= 64) of the lower factor, read from
// W and written to L (row-major n x n, zeros above the diagonal); the update of the trailing
// columns is a GEMM issued by the host.  info (nullable): 0 on success, j+1 for the first
// non-positive pivot j (later panels then stop).
//
// The panel is a chain of jb columns, so its time is the latency of one column.  Every
// workgroup factors the 64-row diagonal block itself (wave 0, a row per lane) and then owns 128
// of the rows below it (waves 1 and 2), which removes all exchange between workgroups.  Columns
// go in blocks of 16 held in registers: the earlier columns' part is subtracted first, from LDS
// (column-major: lanes read consecutive words, the pivot rows' entries are broadcasts), then wave
// 0 factors the block with lane reads alone and the other waves follow behind the one barrier
// per block, so that they solve a block while wave 0 is at the next.  Measured at n = 480: 8
// panels of 0.30 ms in one workgroup that updated the panel in global memory, 0.08 ms with a
// barrier per column, now 0.04 ms (0.055 beside three other windows).
constexpr int kCholNB = 64, kCholRows = 128, kCholC = 16;
__global__ __launch_bounds__(kCholNB + kCholRows) void chol_panel_kernel(int n, int j0, int jb,
                                                                         const double* __restrict__ W,
                                                                         double* __restrict__ L,
                                                                         int* __restrict__ info) {
  __shared__ double Ds[kCholNB][kCholNB];    // [column][row] of the diagonal block
  __shared__ double Os[kCholNB][kCholRows];  // [column][row] of this workgroup's rows below it
  __shared__ int bad, failed;
  const int tid = threadIdx.x, nt = kCholNB + kCholRows;
  const int j1 = j0 + jb, r0 = j1 + (int)blockIdx.x * kCholRows;
  const int nown = max(0, min(kCholRows, n - r0));
  for (int i = tid; i < jb * jb; i += nt) {
    const int r = i / jb, k = i % jb;
    Ds[k][r] = W[(long)(j0 + r) * n + j0 + k];
  }
  for (int i = tid; i < nown * jb; i += nt) {
    const int r = i / jb, k = i % jb;
    Os[k][r] = W[(long)(r0 + r) * n + j0 + k];
  }
  if (tid == 0) {
    bad = 0;
    // (read once: workgroup 0 may be writing its own failure while another starts)
    failed = info && j0 > 0 && *info != 0;
  }
  __syncthreads();
  if (failed) return;
  const bool diag = tid < kCholNB;
  const int row = diag ? tid : tid - kCholNB;
  const bool live = diag ? row < jb : row < nown;
  double* mine = diag ? &Ds[0][row] : &Os[0][row];
  const int ld = diag ? kCholNB : kCholRows;
  for (int c0 = 0; c0 < jb; c0 += kCholC) {
    const int cn = min(kCholC, jb - c0);
    double a[kCholC];
#pragma unroll
    for (int c = 0; c < kCholC; ++c) a[c] = live && c < cn ? mine[(c0 + c) * ld] : 0.0;
#pragma unroll 2
    for (int k = 0; k < c0; ++k) {
      const double m = live ? mine[k * ld] : 0.0;
#pragma unroll
      for (int c = 0; c < kCholC; ++c) a[c] = fma(-m, Ds[k][c0 + c], a[c]);
    }
    if (diag) {
      // (rows above the diagonal of the block hold what is never read)
      bool ok = true;
#pragma unroll
      for (int c = 0; c < kCholC; ++c) {
        if (c < cn && ok) {
          const double piv = lane_value(a[c], c0 + c);
          if (!(piv > 0.0)) {
            ok = false;
            if (tid == 0) bad = j0 + c0 + c + 1;
          } else {
            const double ljj = sqrt(piv);
            a[c] = row == c0 + c ? ljj : a[c] / ljj;
#pragma unroll
            for (int d = c + 1; d < kCholC; ++d) a[d] = fma(-a[c], lane_value(a[c], (c0 + d) & 63), a[d]);
            Ds[c0 + c][row] = a[c];
          }
        }
      }
    }
    __syncthreads();
    // (wave 0 may be a block ahead by now: a failure there is this loop's next turn)
    if (bad && bad <= j0 + c0 + cn) break;
    if (!diag) {
#pragma unroll
      for (int c = 0; c < kCholC; ++c) {
        if (c < cn) {
          a[c] = a[c] / Ds[c0 + c][c0 + c];
#pragma unroll
          for (int d = c + 1; d < kCholC; ++d) a[d] = fma(-a[c], Ds[c0 + c][(c0 + d) & 63], a[d]);
          Os[c0 + c][row] = a[c];
        }
      }
    }
  }
  __syncthreads();
  if (bad) {
    if (info && blockIdx.x == 0 && tid == 0) *info = bad;
    return;
  }
  if (info && j0 == 0 && blockIdx.x == 0 && tid == 0) *info = 0;
  if (blockIdx.x == 0)
    for (int i = tid; i < jb * jb; i += nt) {
      const int r = i / jb, k = i % jb;
      L[(long)(j0 + r) * n + j0 + k] = k <= r ? Ds[k][r] : 0.0;
    }
  for (int i = tid; i < nown * jb; i += nt) {
    const int r = i / jb, k = i % jb;
    L[(long)(r0 + r) * n + j0 + k] = Os[k][r];
  }
  for (int i = (int)blockIdx.x * nt + tid; i < j0 * jb; i += (int)gridDim.x * nt)
    L[(long)(i / jb) * n + j0 + i % jb] = 0.0;
}

__global__ __launch_bounds__(kT) void trinv_kernel(int n, const double* __restrict__ L, double* __restrict__ X) {
  // thread j solves L x = e_j by forward substitution, column j of X
  for (int j = threadIdx.x; j < n; j += kT) {
    for (int i = 0; i < j; ++i) X[(long)i * n + j] = 0.0;
    for (int i = j; i < n; ++i) {
      double acc = (i == j) ? 1.0 : 0.0;
      for (int k = j; k < i; ++k) acc -= L[(long)i * n + k] * X[(long)k * n + j];
      X[(long)i * n + j] = acc / L[(long)i * n + i];
    }
  }
}


// ---------------------------------------------------------------------------
// Spectrum slicing for the projected problem (only the eigenpairs near a target)
// ---------------------------------------------------------------------------

// Householder tridiagonalization: d[n], e[n] (e[i] couples i, i+1); Hh[k][n] holds the unit
// reflector u_k of step k (zero in entries <= k).
//
// Step k reflects column k of the trailing block B (rows and columns k+1..n-1): u from that
// column, q = B u - (u.B u) u, then B -= 2 (u q^T + q u^T).  The n - 2 steps depend on each
// other, and one CU cannot hold the matrix (1.8 MB at n = 480), so one workgroup spends 7 us
// (n = 100) to 12 us (n = 400) a step in sweeps through the L2 and block-wide reductions.
// Here the matrix stays in registers: 64 waves (16 workgroups of 4, one SIMD each), wave w
// holding the columns 64 t + w, lane l the rows 64 s + l.  Every wave keeps u, q and the next
// column whole (row r in lane r % 64) and computes all scalars itself, from the same values in
// the same order, so a step needs one exchange and no barrier: each wave publishes q_c of its
// columns, the owner of column k+1 that column as it was before the update, and each wave
// reads both back.  A value is its own flag: the exchange (2 n doubles per step, a fresh row
// for every step) starts filled with kUnset, a NaN that no published value equals, and is
// written and read with relaxed device-scope atomics, so it holds whichever XCDs the
// workgroups run on.  Which lanes and register slots a step touches depends on k / 64 alone:
// phase P handles the steps with k + 1 in slot P.  Measured in window solves: 0.27 ms at
// n = 128, 0.58 ms at n = 240 and 1.13 ms at n = 400 (2.4-2.8 us a step, mostly the exchange),
// against 0.78 ms at n = 100 and 3.0 ms on average over n = 40..430 in one workgroup.
//
// Every wait ends: the waves take 16 slots of one workgroup each, all waves that a wait depends
// on are in the same grid, other kernels' workgroups end by themselves, and a wave that has
// polled kPolls times in one step (half a microsecond or more each, the time of a load that passes
// the L2: 17 s at least) reports in *err and leaves; the solve then ends with the device error that
// partial_syev raises (PP_EDEVICE).  (The device's clock in this loop instead of a count costs the
// compiler half as many registers again, and spills at n > 448.)
constexpr unsigned long long kUnset = ~0ull;
constexpr int kPolls = 1 << 25;
constexpr int kTriWaves = 64;

__global__ void exchange_fill_kernel(long n, unsigned long long* __restrict__ x, int* __restrict__ err) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) x[i] = kUnset;
  if (blockIdx.x == 0 && threadIdx.x == 0) *err = 0;
}

__device__ __forceinline__ void publish(unsigned long long* p, double v) {
  unsigned long long b = v == v ? (unsigned long long)__double_as_longlong(v) : 0x7ff8000000000000ull;
  __hip_atomic_store(p, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int S>
struct TriState {
  double a[S][S];  // [t][s]: rows 64 s + lane of column 64 t + w
  double col[S];   // column k of the updated matrix
};

// Steps k with k + 1 in [64 P, 64 P + 63]; false when a wait gave up.
template <int P, int S>
__device__ __forceinline__ bool tri_phase(TriState<S>& st, int n, int w, int lane, unsigned long long* ex,
                                          double* __restrict__ dout, double* __restrict__ eout,
                                          double* __restrict__ Hh, int* err) {
  const int k1 = min(64 * P + 62, n - 3);
  for (int k = P ? 64 * P - 1 : 0; k <= k1; ++k) {
    const int nl = (k + 1) & 63;
    // reflector of column k
    double u[S], q[S], cn[S], qc[S];
    double part = 0.0;
#pragma unroll
    for (int t = P; t < S; ++t) {
      u[t] = 64 * t + lane > k ? st.col[t] : 0.0;
      part = fma(u[t], u[t], part);
    }
    const double xx = wave_total(part);
    const double x0 = lane_value(u[P], nl);
    double alpha = 0.0, rv = 0.0;
    if (xx != 0.0) {
      alpha = x0 > 0.0 ? -sqrt(xx) : sqrt(xx);
      rv = 1.0 / sqrt(2.0 * xx - 2.0 * x0 * alpha);
    }
    if (lane == nl) u[P] -= alpha;
#pragma unroll
    for (int t = P; t < S; ++t) u[t] *= rv;
    // q of the own columns, published as they come
    unsigned long long* eq = ex + (long)k * 2 * n;
    unsigned long long* ec = eq + n;
    if (w == nl) {
#pragma unroll
      for (int s = P; s < S; ++s) {
        const int r = 64 * s + lane;
        if (r > k && r < n) publish(ec + r, st.a[P][s]);
      }
    }
#pragma unroll
    for (int t = P; t < S; ++t) {
      double acc = 0.0;
#pragma unroll
      for (int s = P; s < S; ++s) acc = fma(st.a[t][s], u[s], acc);
      qc[t] = wave_total(acc);
      const int c = 64 * t + w;
      if (lane == 0 && c > k && c < n) publish(eq + c, qc[t]);
    }
    if (w == (k & (kTriWaves - 1))) {
#pragma unroll
      for (int t = 0; t < S; ++t) {
        const int r = 64 * t + lane;
        if (r < n) Hh[(long)k * n + r] = t >= P ? u[t] : 0.0;
      }
      if (lane == 0) eout[k] = alpha;
    }
    // all of q and the next column
    for (int it = 0;; ++it) {
      bool ok = true;
      unsigned long long bq[S], bc[S];
#pragma unroll
      for (int t = P; t < S; ++t) {
        const int r = 64 * t + lane;
        const bool act = r > k && r < n;
        bq[t] = act ? __hip_atomic_load(eq + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull;
        bc[t] = act ? __hip_atomic_load(ec + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull;
      }
#pragma unroll
      for (int t = P; t < S; ++t) {
        ok = ok && bq[t] != kUnset && bc[t] != kUnset;
        q[t] = __longlong_as_double((long long)bq[t]);
        cn[t] = __longlong_as_double((long long)bc[t]);
      }
      if (__all(ok)) break;
      if (it >= kPolls) {
        if (lane == 0) *err = 1;
        return false;
      }
    }
    part = 0.0;
#pragma unroll
    for (int t = P; t < S; ++t) part = fma(u[t], q[t], part);
    const double K = wave_total(part);
#pragma unroll
    for (int t = P; t < S; ++t) q[t] = fma(-K, u[t], q[t]);
    const double u2 = -2.0 * lane_value(u[P], nl), q2 = -2.0 * lane_value(q[P], nl);
#pragma unroll
    for (int t = P; t < S; ++t) st.col[t] = fma(u[t], q2, fma(q[t], u2, cn[t]));
    if (w == nl && lane == nl) dout[k + 1] = st.col[P];
#pragma unroll
    for (int t = P; t < S; ++t) {
      const double uc = lane_value(u[t], w);
      const double uc2 = -2.0 * uc, qc2 = -2.0 * fma(-K, uc, qc[t]);
#pragma unroll
      for (int s = P; s < S; ++s) st.a[t][s] = fma(u[s], qc2, fma(q[s], uc2, st.a[t][s]));
    }
  }
  if constexpr (P + 1 < S)
    return tri_phase<P + 1, S>(st, n, w, lane, ex, dout, eout, Hh, err);
  else
    return true;
}

template <int S>
__global__ __launch_bounds__(256, 2) void tridiag_kernel(int n, const double* __restrict__ A,
                                                         unsigned long long* ex, double* __restrict__ dout,
                                                         double* __restrict__ eout, double* __restrict__ Hh,
                                                         int* err) {
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
  if (w >= n) return;
  TriState<S> st;
#pragma unroll
  for (int t = 0; t < S; ++t) {
    const int c = 64 * t + w;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int r = 64 * s + lane;
      st.a[t][s] = r < n && c < n ? A[(long)c * n + r] : 0.0;  // A is symmetric
    }
    st.col[t] = 64 * t + lane < n ? A[64 * t + lane] : 0.0;
  }
  if (w == 0 && lane == 0) dout[0] = st.col[0];
  if (!tri_phase<0, S>(st, n, w, lane, ex, dout, eout, Hh, err)) return;
  // the last 2 x 2 block: column n-2 is in col, d[n-1] in the owner of column n-1
#pragma unroll
  for (int t = 0; t < S; ++t) {
    const int r = 64 * t + lane;
    if (r == n - 1 && w == 0) {
      if (n >= 2) eout[n - 2] = st.col[t];
      eout[n - 1] = 0.0;
    }
    if (r == n - 1 && 64 * t + w == n - 1) dout[n - 1] = st.a[t][t];
  }
}

template <int S>
void launch_tridiag(int n, const double* A, double* ex, double* d, double* e, double* Hh, int* err, hipStream_t s) {
  unsigned long long* x = reinterpret_cast<unsigned long long*>(ex);
  const long cells = 2L * n * std::max(0, n - 2);
  exchange_fill_kernel<<<(int)std::max(1L, std::min(256L, (cells + 255) / 256)), 256, 0, s>>>(cells, x, err);
  PPW_LAUNCH_CHECK();
  const int waves = std::min(n, kTriWaves);
  tridiag_kernel<S><<<(waves + 3) / 4, 256, 0, s>>>(n, A, x, d, e, Hh, err);
  PPW_LAUNCH_CHECK();
}

void tridiagonalize(int n, const double* A, double* ex, double* d, double* e, double* Hh, int* err, hipStream_t s) {
  switch ((n + 63) / 64) {
    case 1: return launch_tridiag<1>(n, A, ex, d, e, Hh, err, s);
    case 2: return launch_tridiag<2>(n, A, ex, d, e, Hh, err, s);
    case 3: return launch_tridiag<3>(n, A, ex, d, e, Hh, err, s);
    case 4: return launch_tridiag<4>(n, A, ex, d, e, Hh, err, s);
    case 5: return launch_tridiag<5>(n, A, ex, d, e, Hh, err, s);
    case 6: return launch_tridiag<6>(n, A, ex, d, e, Hh, err, s);
    case 7: return launch_tridiag<7>(n, A, ex, d, e, Hh, err, s);
    default: return launch_tridiag<8>(n, A, ex, d, e, Hh, err, s);
  }
}

// Spectrum slicing of the tridiagonal (d, e) is a chain of n dependent steps per Sturm count
// and per triangular solve, so its time is (steps in sequence) x (latency of a step), and the
// two kernels below shorten both.  Measured on MI355X at n = 240..480, p = 28: 1.4 ms in one
// workgroup (one thread per eigenvalue bisecting with a division per Sturm step, then one
// thread per vector with its arrays in global memory); now both kernels together 0.16 ms.

// Scale of the tridiagonal: a power of two that brings its Gershgorin interval [gl, gu]
// into [-1, 1], so that a Sturm sequence grows by at most a factor 4 per step.
__device__ __forceinline__ void tridiag_bounds(int n, const double* d, const double* e, int lane, double& gl,
                                               double& gu) {
  double lo = DBL_MAX, hi = -DBL_MAX;
  for (int i = lane; i < n; i += 64) {
    const double r = (i > 0 ? fabs(e[i - 1]) : 0.0) + (i + 1 < n ? fabs(e[i]) : 0.0);
    lo = fmin(lo, d[i] - r);
    hi = fmax(hi, d[i] + r);
  }
  for (int off = 32; off > 0; off >>= 1) {
    lo = fmin(lo, __shfl_xor(lo, off, 64));
    hi = fmax(hi, __shfl_xor(hi, off, 64));
  }
  const double span = fmax(hi - lo, 1e-300);
  gl = lo - 1e-14 * span;
  gu = hi + 1e-14 * span;
}

// Number of eigenvalues of the scaled tridiagonal below x: the sign changes of the Sturm
// sequence p_i = (d_i - x) p_(i-1) - e_(i-1)^2 p_(i-2).  One dependent fused multiply-add per
// step (the quotient form needs a division); the pair is rescaled by a power of two every 8
// steps (a step shrinks it by 2^-100 at most: a zero is replaced by that much of its
// predecessor, of the sign that counts it as below x).  de[i] = {d_i, e_(i-1)^2}.
__device__ __forceinline__ int sturm_below(int n, const double2* de, double x) {
  double prev = 1.0, p = de[0].x - x;
  if (p == 0.0) p = -0x1p-100;
  int c = p < 0.0 ? 1 : 0;
  int i = 1;
  auto step = [&](const double2& q) {
    double t = fma(q.x - x, p, -q.y * prev);
    t = t == 0.0 ? -0x1p-100 * p : t;
    c += (t < 0.0) != (p < 0.0) ? 1 : 0;
    prev = p;
    p = t;
  };
  for (; i + 8 <= n; i += 8) {
    double2 q[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) q[t] = de[i + t];
#pragma unroll
    for (int t = 0; t < 8; ++t) step(q[t]);
    const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(p), fabs(prev)));
    p = __builtin_amdgcn_ldexp(p, ex);
    prev = __builtin_amdgcn_ldexp(prev, ex);
  }
  for (; i < n; ++i) step(de[i]);
  return c;
}

// The eigenvalues of the tridiagonal around 'target': the p below and the p above it, one wave
// each (the p nearest lie among them), by multisection: the 64 lanes count at 64 points of the
// interval, which shrinks 65-fold per round (10 rounds instead of 53 bisections, each as long).
// cand[c]: ascending; *nc: how many there are.
__global__ __launch_bounds__(64) void multisect_kernel(int n, const double* __restrict__ d,
                                                       const double* __restrict__ e, double target, int p,
                                                       double* __restrict__ cand, int* __restrict__ nc) {
  __shared__ double2 de[kMaxN];
  const int lane = threadIdx.x;
  double gl, gu;
  tridiag_bounds(n, d, e, lane, gl, gu);
  const double big = fmax(fabs(gl), fabs(gu));
  const int ex = (big > 0.0 && big < 1e300) ? __builtin_amdgcn_frexp_exp(big) : 0;
  for (int i = lane; i < n; i += 64) {
    const double ei = i > 0 ? __builtin_amdgcn_ldexp(e[i - 1], -ex) : 0.0;
    de[i] = double2{__builtin_amdgcn_ldexp(d[i], -ex), ei * ei};
  }
  __syncthreads();
  // (a target beyond the spectrum counts none or all, at the interval's ends as well)
  const double ts = fmin(fmax(__builtin_amdgcn_ldexp(target, -ex), -1.5), 1.5);
  const int j0 = sturm_below(n, de, ts);
  const int lo = max(0, j0 - p), count = min(n, j0 + p) - lo;
  if (blockIdx.x == 0 && lane == 0) *nc = count;
  if ((int)blockIdx.x >= count) return;
  const int idx = lo + blockIdx.x;
  double a = __builtin_amdgcn_ldexp(gl, -ex), b = __builtin_amdgcn_ldexp(gu, -ex);
  for (int it = 0; it < 32 && (b - a) > 4.0 * DBL_EPSILON * fmax(fabs(a), fabs(b)) + DBL_MIN; ++it) {
    const double w = (b - a) * (1.0 / 65.0);
    const double x = fma((double)(lane + 1), w, a);
    const unsigned long long above = __ballot(sturm_below(n, de, x) > idx);
    const int f = above ? __ffsll((long long)above) - 1 : 64;  // first point with more than idx below it
    const double a0 = a;
    if (f < 64) b = fma((double)(f + 1), w, a0);
    if (f > 0) a = fma((double)f, w, a0);
  }
  if (lane == 0) cand[blockIdx.x] = __builtin_amdgcn_ldexp(0.5 * (a + b), ex);
}

// Partially pivoted LU of T - lmb I (a vanishing pivot is replaced by pert) and three inverse
// iterations from a fixed start vector, each normalised (the eigenvalue is exact to rounding, so
// the second already reaches that level).  One wave per vector: lane 0 runs the recurrences with
// every array in LDS and the pivots stored as reciprocals, the lanes share the rest.
__global__ __launch_bounds__(64) void inverse_iteration_kernel(int n, const double* __restrict__ d,
                                                               const double* __restrict__ e, double target, int p,
                                                               const double* __restrict__ cand,
                                                               const int* __restrict__ ncp, double* __restrict__ lam,
                                                               double* __restrict__ V) {
  __shared__ double sd[kMaxN], se[kMaxN], dl[kMaxN], di[kMaxN], du[kMaxN], du2[kMaxN], x[kMaxN], y[kMaxN];
  __shared__ int piv[kMaxN];
  const int lane = threadIdx.x, t = blockIdx.x;
  const int nc = *ncp;
  // the p candidates nearest the target (ties: the lower) are the contiguous run whose start is
  // the first candidate not farther than the one p places above it
  const bool farther = lane + p < nc && fabs(cand[lane] - target) > fabs(cand[lane + p] - target);
  const unsigned long long m = ~__ballot(farther);
  const int i0 = m ? __ffsll((long long)m) - 1 : 64;
  const double lmb = cand[i0 + t];
  double gl, gu;
  tridiag_bounds(n, d, e, lane, gl, gu);
  const double pert = 1e-15 * fmax(fmax(fabs(gl), fabs(gu)), 1e-300);
  for (int i = lane; i < n; i += 64) {
    sd[i] = d[i];
    se[i] = i + 1 < n ? e[i] : 0.0;
    x[i] = 1.0 + 0.5 * sin(0.7 * i + 1.3 * t + 0.1);  // deterministic start vector
  }
  if (lane == 0) lam[t] = lmb;
  __syncthreads();
  if (lane == 0) {
    double dc = sd[0] - lmb, uc = se[0];
    for (int i = 0; i + 1 < n; ++i) {
      const double sub = se[i], dn = sd[i + 1] - lmb, un = se[i + 1];
      const bool keep = fabs(dc) >= fabs(sub);
      double pv = keep ? dc : sub;
      if (fabs(pv) < 1e-290) pv = pert;
      const double inv = 1.0 / pv;
      const double f = (keep ? sub : dc) * inv;
      dl[i] = f;
      di[i] = inv;
      du[i] = keep ? uc : dn;
      du2[i] = keep ? 0.0 : un;
      piv[i] = keep ? 0 : 1;
      dc = keep ? dn - f * uc : uc - f * dn;
      uc = keep ? un : -f * un;
    }
    if (fabs(dc) < 1e-290) dc = pert;
    di[n - 1] = 1.0 / dc;
  }
  for (int iter = 0; iter < 3; ++iter) {
    __syncthreads();
    if (lane == 0) {
      double xi = x[0];
#pragma unroll 8
      for (int i = 0; i + 1 < n; ++i) {
        const double xn = x[i + 1];
        const bool sw = piv[i] != 0;
        const double top = sw ? xn : xi;
        y[i] = top;
        xi = (sw ? xi : xn) - dl[i] * top;
      }
      double x1 = xi * di[n - 1], x2 = 0.0;
      x[n - 1] = x1;
      if (n >= 2) {
        x2 = x1;
        x1 = (y[n - 2] - du[n - 2] * x2) * di[n - 2];
        x[n - 2] = x1;
      }
#pragma unroll 8
      for (int i = n - 3; i >= 0; --i) {
        const double xi0 = (y[i] - du2[i] * x2 - du[i] * x1) * di[i];
        x[i] = xi0;
        x2 = x1;
        x1 = xi0;
      }
    }
    __syncthreads();
    double big = 0.0;
    for (int i = lane; i < n; i += 64) big = fmax(big, fabs(x[i]));
    for (int off = 32; off > 0; off >>= 1) big = fmax(big, __shfl_xor(big, off, 64));
    const double r = 1.0 / big;
    double s2 = 0.0;
    for (int i = lane; i < n; i += 64) s2 += (x[i] * r) * (x[i] * r);
    for (int off = 32; off > 0; off >>= 1) s2 += __shfl_xor(s2, off, 64);
    const double sc = 1.0 / sqrt(s2);
    for (int i = lane; i < n; i += 64) x[i] = (x[i] * r) * sc;
  }
  __syncthreads();
  for (int i = lane; i < n; i += 64) V[(long)t * n + i] = x[i];
}

// Factors that orthonormalise k <= 64 vectors from their Gram matrix G: pivoted Cholesky
// G = R^T R in pivot order, stopped at the first pivot not above thresh (the rest lies within
// sqrt(thresh) of the span found).  T[k][q] (ld q): X T is orthonormal; R[q][k]: X = (X T) R
// (both in the original order of the columns); *q_out = q.
//
// The vectors only have to be orthonormal and to span the same space, so a triangular factor
// does for the symmetric one (eigenvectors of G): k dependent steps of one wave in LDS, 18 us at
// k = 40, where the eigensolver below took 260 us (its rotations are a scalar recurrence of
// about k^2 steps).
//
// KM (32 or 64, k at most) sizes its LDS: beside the products of other windows the kernel has to find
// a compute unit with room for it, and 16 or 64 KiB fit where the 96 KiB of three arrays of 64 x 64
// did not: 18 us alone, and in two windows at 40/160/600 in split BF16 330 us on average with 96 KiB,
// 87 us with 16 (the Cholesky panel below 64 KiB, with 64 rows a workgroup, gained nothing).
template <int KM>
__global__ __launch_bounds__(64) void orth_factors_kernel(int k, const double* __restrict__ G, double thresh,
                                                          double* __restrict__ T, double* __restrict__ R,
                                                          int* __restrict__ q_out) {
  __shared__ double Gs[KM][KM], Rs[KM][KM];
  __shared__ int perm[KM], rank[KM];
  const int lane = threadIdx.x, col = min(lane, KM - 1);
  for (int i = lane; i < k * k; i += 64) Gs[i / k][i % k] = G[i];
  if (lane < KM) rank[lane] = -1;
  __syncthreads();
  double dj = lane < k ? Gs[col][col] : -1.0;
  bool done = lane >= k;
  int q = 0;
  for (; q < k; ++q) {
    const double best = wave_max(done ? 0.0 : fmax(dj, 0.0));  // (a NaN counts as 0)
    const int at = __ffsll((long long)__ballot(!done && dj == best)) - 1;
    if (!(best > thresh)) break;
    const double piv = sqrt(best);
    double acc = Gs[at][col];
#pragma unroll 8
    for (int t = 0; t < q; ++t) acc = fma(-Rs[t][at], Rs[t][col], acc);
    const double r = done ? 0.0 : (lane == at ? piv : acc / piv);
    if (lane < KM) Rs[q][lane] = r;
    dj = fma(-r, r, dj);
    if (lane == at) {
      done = true;
      perm[q] = lane;
      rank[lane] = q;
    }
    __syncthreads();
  }
  // upper triangle in pivot order, then column c of its inverse by lane c, row by row from the last in
  // the rows' own places
  for (int i = 0; i < q; ++i)
    if (lane < q) Gs[i][lane] = Rs[i][perm[lane]];
  __syncthreads();
  for (int i = q - 1; i >= 0; --i) {
    const double gii = Gs[i][i];
    double acc = lane == i ? 1.0 : 0.0;
#pragma unroll 4
    for (int t = i + 1; t < q; ++t) acc = fma(-Gs[i][t], Gs[t][col], acc);
    __syncthreads();
    if (lane < q) Gs[i][lane] = lane >= i ? acc / gii : 0.0;
    __syncthreads();
  }
  for (int i = lane; i < k * q; i += 64) {
    const int j = i / q, c = i % q;
    T[i] = rank[j] >= 0 ? Gs[rank[j]][c] : 0.0;
    R[i] = Rs[i / k][i % k];
  }
  if (lane == 0) *q_out = q;
}

void launch_orth_factors(int k, const double* G, double thresh, double* T, double* R, int* count, hipStream_t s) {
  if (k <= 32)
    orth_factors_kernel<32><<<1, 64, 0, s>>>(k, G, thresh, T, R, count);
  else
    orth_factors_kernel<64><<<1, 64, 0, s>>>(k, G, thresh, T, R, count);
  PPW_LAUNCH_CHECK();
}

// Eigenpairs of a symmetric n x n matrix (n <= 64) that is diagonal but for a few elements, by
// cyclic Jacobi: w ascending, Z[r * n + c] component r of vector c.  Pairs of the round-robin
// order whose element is below a tenth of a rounding unit of the largest diagonal element are
// left alone, and a round without a rotation costs one barrier, so the matrices it is for (the
// tridiagonal in the span of its own eigenvectors, off-diagonal only in clusters) take 10-60 us.
__global__ __launch_bounds__(256) void jacobi_kernel(int n, const double* __restrict__ A, double* __restrict__ w,
                                                     double* __restrict__ Z) {
  __shared__ double H[64][65], U[64][65];
  __shared__ double cs[32], sn[32];
  __shared__ int pp[32], qq[32], pos[64];
  __shared__ double diag[64];
  const int tid = threadIdx.x;
  for (int i = tid; i < 64 * 64; i += 256) {
    const int r = i / 64, c = i % 64;
    H[r][c] = r < n && c < n ? 0.5 * (A[r * n + c] + A[c * n + r]) : 0.0;
    U[r][c] = r == c ? 1.0 : 0.0;
  }
  __syncthreads();
  double big = 0.0;
  for (int i = 0; i < n; ++i) big = fmax(big, fabs(H[i][i]));
  const double tol = 0.1 * DBL_EPSILON * big;
  const int m = n + (n & 1), half = m / 2;
  for (int sweep = 0; sweep < 40 && n > 1; ++sweep) {
    int rotated = 0;
    for (int rd = 0; rd < m - 1; ++rd) {
      int rot = 0;
      if (tid < half) {
        int p = tid == 0 ? m - 1 : (rd + tid) % (m - 1), q = tid == 0 ? rd : (rd - tid + m - 1) % (m - 1);
        if (p > q) {
          const int t = p;
          p = q;
          q = t;
        }
        const double apq = H[p][q];
        double c = 1.0, s = 0.0;
        if (q < n && fabs(apq) > tol) {
          const double th = (H[q][q] - H[p][p]) / (2.0 * apq);
          const double t = copysign(1.0, th) / (fabs(th) + sqrt(th * th + 1.0));
          c = 1.0 / sqrt(t * t + 1.0);
          s = t * c;
          rot = 1;
        }
        cs[tid] = c;
        sn[tid] = s;
        pp[tid] = p;
        qq[tid] = q;
      }
      if (!__syncthreads_or(rot)) continue;
      rotated = 1;
      for (int i = tid; i < half * n; i += 256) {
        const int t = i / n, r = i % n, p = pp[t], q = qq[t];
        if (q >= n) continue;
        const double c = cs[t], s = sn[t];
        const double hp = H[r][p], hq = H[r][q], up = U[r][p], uq = U[r][q];
        H[r][p] = c * hp - s * hq;
        H[r][q] = s * hp + c * hq;
        U[r][p] = c * up - s * uq;
        U[r][q] = s * up + c * uq;
      }
      __syncthreads();
      for (int i = tid; i < half * n; i += 256) {
        const int t = i / n, k = i % n, p = pp[t], q = qq[t];
        if (q >= n) continue;
        const double c = cs[t], s = sn[t];
        const double hp = H[p][k], hq = H[q][k];
        H[p][k] = c * hp - s * hq;
        H[q][k] = s * hp + c * hq;
      }
      __syncthreads();
    }
    if (!rotated) break;  // the same in every thread
  }
  if (tid < n) diag[tid] = H[tid][tid];
  __syncthreads();
  if (tid < n) {
    int k = 0;
    for (int j = 0; j < n; ++j) k += diag[j] < diag[tid] || (diag[j] == diag[tid] && j < tid) ? 1 : 0;
    pos[tid] = k;
    w[k] = diag[tid];
  }
  __syncthreads();
  for (int i = tid; i < n * n; i += 256) {
    const int r = i / n, c = i % n;
    Z[r * n + pos[c]] = U[r][c];
  }
}

// Y[t][i] = (T V)[t][i] for the tridiagonal (d, e) and p row vectors of length n
__global__ void tridiag_apply_kernel(int n, int p, const double* __restrict__ d, const double* __restrict__ e,
                                     const double* __restrict__ V, double* __restrict__ Y) {
  const long tot = (long)n * p;
  for (long idx = blockIdx.x * (long)blockDim.x + threadIdx.x; idx < tot; idx += (long)gridDim.x * blockDim.x) {
    const int t = (int)(idx / n), i = (int)(idx % n);
    const double* v = V + (long)t * n;
    double y = d[i] * v[i];
    if (i > 0) y += e[i - 1] * v[i - 1];
    if (i + 1 < n) y += e[i] * v[i + 1];
    Y[idx] = y;
  }
}

// Z[r][j] = (H_0 ... H_{n-3} v_j)[r], one wave per vector with the vector in registers (8 per
// lane up to n = 512): a reflector costs one wave sum and no barrier, and the next one's
// elements are loaded meanwhile.  In four windows with bases up to
// 430: 74 us on average, 150 us with a workgroup per vector.
__global__ __launch_bounds__(64) void backtransform_kernel(int n, int p, const double* __restrict__ Hh,
                                                           const double* __restrict__ V, double* __restrict__ Z) {
  constexpr int S = kMaxN / 64;
  const int j = blockIdx.x, lane = threadIdx.x;
  double v[S], u[S], un[S];
#pragma unroll
  for (int t = 0; t < S; ++t) {
    const int i = lane + 64 * t;
    v[t] = i < n ? V[(long)j * n + i] : 0.0;
    un[t] = (n >= 3 && i < n) ? Hh[(long)(n - 3) * n + i] : 0.0;
  }
  for (int k = n - 3; k >= 0; --k) {
#pragma unroll
    for (int t = 0; t < S; ++t) u[t] = un[t];
    if (k > 0) {
#pragma unroll
      for (int t = 0; t < S; ++t) {
        const int i = lane + 64 * t;
        un[t] = i < n ? Hh[(long)(k - 1) * n + i] : 0.0;  // zero in entries <= k - 1
      }
    }
    double part = 0.0;
#pragma unroll
    for (int t = 0; t < S; ++t) part = fma(u[t], v[t], part);
    const double f = -2.0 * wave_total(part);
#pragma unroll
    for (int t = 0; t < S; ++t) v[t] = fma(f, u[t], v[t]);
  }
#pragma unroll
  for (int t = 0; t < S; ++t) {
    const int i = lane + 64 * t;
    if (i < n) Z[(long)i * p + j] = v[t];
  }
}

// X[:, j] = scale_j L^-T B[:, j] with scale_j = sqrt(th[j]), one wave per right-hand side with
// the column in registers: an unknown costs one broadcast (a lane read) and no barrier.
__global__ __launch_bounds__(64) void trsm_lt_kernel(int n, const double* __restrict__ L, const double* __restrict__ B,
                                                     long ldb, const double* __restrict__ th, double* __restrict__ X,
                                                     long ldx) {
  constexpr int S = kMaxN / 64;
  __shared__ double rdiag[kMaxN];
  const int j = blockIdx.x, lane = threadIdx.x;
  double b[S], ln[S];
#pragma unroll
  for (int t = 0; t < S; ++t) {
    const int i = lane + 64 * t;
    b[t] = i < n ? B[(long)i * ldb + j] : 0.0;
    if (i < n) rdiag[i] = 1.0 / L[(long)i * n + i];
    ln[t] = i < n ? L[(long)(n - 1) * n + i] : 0.0;
  }
  __syncthreads();
  const double sc = sqrt(th[j]);
  // unknown i = 64 blk + src, from the last; row i of L feeds the unknowns below it
#pragma unroll
  for (int blk = S - 1; blk >= 0; --blk) {
    if (64 * blk >= n) continue;
    for (int src = min(63, n - 1 - 64 * blk); src >= 0; --src) {
      const int i = 64 * blk + src;
      const int lo = __builtin_amdgcn_readlane(__double2loint(b[blk]), src);
      const int hi = __builtin_amdgcn_readlane(__double2hiint(b[blk]), src);
      const double x = __hiloint2double(hi, lo) * rdiag[i];
      double l[S];
#pragma unroll
      for (int t = 0; t <= blk; ++t) l[t] = ln[t];
      if (i > 0) {
#pragma unroll
        for (int t = 0; t <= blk; ++t) {
          const int c = lane + 64 * t;
          ln[t] = c < n ? L[(long)(i - 1) * n + c] : 0.0;
        }
      }
#pragma unroll
      for (int t = 0; t <= blk; ++t) {
        const int c = lane + 64 * t;
        b[t] = c < i ? fma(-l[t], x, b[t]) : b[t];
      }
      if (lane == src) b[blk] = x;
    }
  }
#pragma unroll
  for (int t = 0; t < S; ++t) {
    const int i = lane + 64 * t;
    if (i < n) X[(long)i * ldx + j] = sc * b[t];
  }
}

}  // namespace

void small_syev(int n, const double* A, double* w, double* Z, hipStream_t s, double* scratch) {
  if (n < 1 || n > kMaxN) throw InvalidArg("small_syev: n out of range");
  double* ws = scratch;
  if (!ws) PPW_HIP(hipMalloc(&ws, sizeof(double) * 2 * (size_t)n * n));
  if (n <= 64)
    syev_kernel<64, true><<<1, 64, 0, s>>>(n, A, w, Z, ws, ws + (size_t)n * n);
  else
    syev_kernel<kT, false><<<1, kT, 0, s>>>(n, A, w, Z, ws, ws + (size_t)n * n);
  hipError_t e = hipGetLastError();
  if (!scratch) {
    (void)hipStreamSynchronize(s);
    (void)hipFree(ws);
  }
  if (e != hipSuccess) throw DeviceError(std::string("syev launch: ") + hipGetErrorString(e));
}

size_t partial_syev_scratch(int n, int p) {
  return (size_t)3 * n * n + 2 * (size_t)n + 4 * (size_t)p * n + 5 * (size_t)p * p + 2 * (size_t)p + 64;
}

int partial_syev(int n, const double* A, double target, int p, double* lam, double* Z, double* scratch, int* flags,
                 hipStream_t s) {
  if (n < 1 || n > kMaxN || p < 1 || p > 64 || p > n) throw InvalidArg("partial_syev: size out of range");
  double* ex = scratch;  // the tridiagonalization's exchange
  double* Hh = ex + (size_t)2 * n * n;
  double* d = Hh + (size_t)n * n;
  double* e = d + n;
  double* V = e + n;
  double* V1 = V + (size_t)p * n;
  double* Y = V1 + (size_t)p * n;
  double* V2 = Y + (size_t)p * n;
  double* work = V2 + (size_t)p * n;
  double* G = work + (size_t)2 * p;
  double* UG = G + (size_t)p * p;
  double* T1 = UG + (size_t)p * p;
  double* H = T1 + (size_t)p * p;
  double* UH = H + (size_t)p * p;
  double* cand = work;
  int* nc = flags + 2;  // a count, and whether the tridiagonalization gave up
  tridiagonalize(n, A, ex, d, e, Hh, flags + 3, s);
  multisect_kernel<<<2 * p, 64, 0, s>>>(n, d, e, target, p, cand, nc);
  PPW_LAUNCH_CHECK();
  inverse_iteration_kernel<<<p, 64, 0, s>>>(n, d, e, target, p, cand, nc, lam, V);
  PPW_LAUNCH_CHECK();
  // Rayleigh-Ritz inside span(V): G = V V^T, orthonormalization, H = V1 T V1^T
  GemmDesc g;
  g.M = p; g.N = p; g.K = n; g.transA = 0; g.lda = n; g.transB = 1; g.ldb = n; g.ldc = p;
  gemm_f64(g, 1.0, V, V, 0.0, G, s);
  // (T1 is p x q, ld q; R goes to UG)
  launch_orth_factors(p, G, 1e-12, T1, UG, nc, s);
  int got[4] = {0, 0, 0, 0};
  PPW_HIP(hipMemcpyAsync(got, flags, sizeof(got), hipMemcpyDeviceToHost, s));
  PPW_HIP(hipStreamSynchronize(s));
  if (got[0]) return 0;
  if (got[3]) throw DeviceError("tridiagonalization: a workgroup waited in vain for the others");
  const int q = got[2];
  if (q == 0) throw Unstable("partial_syev: inverse iteration produced no independent vectors");
  // V1[j][r] = sum_t T1[t][j] V[t][r]
  GemmDesc a;
  a.M = q; a.N = n; a.K = p; a.transA = 1; a.lda = q; a.transB = 0; a.ldb = n; a.ldc = n;
  gemm_f64(a, 1.0, T1, V, 0.0, V1, s);
  tridiag_apply_kernel<<<(n * q + 255) / 256, 256, 0, s>>>(n, q, d, e, V1, Y);
  PPW_LAUNCH_CHECK();
  GemmDesc h;
  h.M = q; h.N = q; h.K = n; h.transA = 0; h.lda = n; h.transB = 1; h.ldb = n; h.ldc = q;
  gemm_f64(h, 1.0, V1, Y, 0.0, H, s);
  jacobi_kernel<<<1, 256, 0, s>>>(q, H, lam, UH);
  PPW_LAUNCH_CHECK();
  // V2[j][r] = sum_t UH[t][j] V1[t][r]
  GemmDesc b;
  b.M = q; b.N = n; b.K = q; b.transA = 1; b.lda = q; b.transB = 0; b.ldb = n; b.ldc = n;
  gemm_f64(b, 1.0, UH, V1, 0.0, V2, s);
  backtransform_kernel<<<q, 64, 0, s>>>(n, p, Hh, V2, Z);
  PPW_LAUNCH_CHECK();
  return q;
}

int orth_factors(int k, const double* G, double thresh, double* T, double* R, int* count, hipStream_t s) {
  if (k < 1 || k > 64) throw InvalidArg("orth_factors: k out of range");
  launch_orth_factors(k, G, thresh, T, R, count, s);
  int q = 0;
  PPW_HIP(hipMemcpyAsync(&q, count, sizeof(int), hipMemcpyDeviceToHost, s));
  PPW_HIP(hipStreamSynchronize(s));
  return q;
}

void small_trsm_lt(int n, const double* L, int p, const double* B, long ldb, const double* th, double* X, long ldx,
                   hipStream_t s) {
  if (n < 1 || n > kMaxN) throw InvalidArg("small_trsm_lt: n out of range");
  trsm_lt_kernel<<<p, 64, 0, s>>>(n, L, B, ldb, th, X, ldx);
  PPW_LAUNCH_CHECK();
}

void small_cholesky(int n, const double* A, double* L, int* info, double* work, hipStream_t s) {
  if (n < 1 || n > kMaxN) throw InvalidArg("small_cholesky: n out of range");
  // blocked right-looking: panels of 64 columns, trailing updates as GEMMs on a working copy
  // (the first panel reads A itself)
  const double* W = A;
  for (int j0 = 0; j0 < n; j0 += kCholNB) {
    const int jb = std::min(kCholNB, n - j0), j1 = j0 + jb, m2 = n - j1;
    if (j0 == 0 && m2 > 0) {
      PPW_HIP(hipMemcpyAsync(work, A, sizeof(double) * n * n, hipMemcpyDeviceToDevice, s));
      W = work;
    }
    const int blocks = std::max(1, (m2 + kCholRows - 1) / kCholRows);
    chol_panel_kernel<<<blocks, kCholNB + kCholRows, 0, s>>>(n, j0, jb, W, L, info);
    PPW_LAUNCH_CHECK();
    if (m2 > 0) {
      GemmDesc d;
      d.M = m2;
      d.N = m2;
      d.K = jb;
      d.transA = 0;
      d.lda = n;
      d.transB = 1;
      d.ldb = n;
      d.ldc = n;
      const double* panel = L + (size_t)j1 * n + j0;
      gemm_f64(d, -1.0, panel, panel, 1.0, work + (size_t)j1 * n + j1, s);
    }
  }
}

void small_trinv(int n, const double* L, double* X, hipStream_t s) {
  if (n < 1 || n > kMaxN) throw InvalidArg("small_trinv: n out of range");
  trinv_kernel<<<1, kT, 0, s>>>(n, L, X);
  PPW_LAUNCH_CHECK();
}

}  // namespace ppw
