// Bandwidth-bound kernels: layout permutations, amplitude-strip formation,
// diagonals, product assembly and vector reductions.  All loops are grid-stride
// with 64-bit indices; reductions use wavefront shuffles in a fixed order so every
// result is bitwise reproducible.
#include "kernels.h"

#include <algorithm>

namespace ppw {
namespace {

constexpr int kBlock = 256;

inline int grid_for(long n, int block = kBlock) {
  long g = (n + block - 1) / block;
  return (int)std::max<long>(1, std::min<long>(g, 65536));
}

__device__ __forceinline__ double wave_sum(double v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  return v;
}

// block-wide sum (blockDim.x == 256), result valid in thread 0
__device__ double block_sum(double v) {
  __shared__ double part[kBlock / 64];
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) part[wave] = v;
  __syncthreads();
  double s = 0;
  if (threadIdx.x == 0)
    for (int w = 0; w < kBlock / 64; ++w) s += part[w];
  __syncthreads();
  return s;
}

__global__ void permute3_kernel(const double* __restrict__ in, double* __restrict__ out, int d0, int d1, int d2,
                                int p0, int p1, int p2) {
  const int dims[3] = {d0, d1, d2};
  const int o0 = dims[p0], o1 = dims[p1], o2 = dims[p2];
  const long n = (long)d0 * d1 * d2;
  for (long idx = blockIdx.x * (long)blockDim.x + threadIdx.x; idx < n; idx += (long)gridDim.x * blockDim.x) {
    // idx enumerates the OUTPUT in row-major order (coalesced writes)
    const int c2 = (int)(idx % o2);
    const long r = idx / o2;
    const int c1 = (int)(r % o1);
    const int c0 = (int)(r / o1);
    int ii[3];
    ii[p0] = c0;
    ii[p1] = c1;
    ii[p2] = c2;
    out[idx] = in[((long)ii[0] * d1 + ii[1]) * d2 + ii[2]];
  }
}

// Amplitudes of a strip from its integrals S[(k, x)][(l, y)] (k in the strip, any l).  Bound by
// the bytes of S and tau.  The element (x, y) also needs S at (y, x), so a workgroup takes the
// 32 x 32 tiles (X, Y) and (Y, X) of a pair k, l together and S is read once; and where l lies in
// the strip too, S is read above its diagonal only (row (k, x), column (l, y) with (l, y) not
// before (k, x): the part the integral GEMM computes) and the pair l, k comes from the tiles of
// k, l.  SPLIT: tau goes out in the chunk layout of split_sbf16 (v a multiple of 8, so that no
// chunk crosses a pair).  Measured at 96/384/1152 in FP64, one strip: see tau_strip.
template <typename T, bool SPLIT>
__global__ __launch_bounds__(kBlock) void tau_strip_kernel(const T* __restrict__ S, int o, int v, int k0, int ib,
                                                           const double* __restrict__ eo,
                                                           const double* __restrict__ ev, T* __restrict__ tau, long ldt,
                                                           double* __restrict__ t, double* __restrict__ tEv,
                                                           double* __restrict__ tEo, double* __restrict__ partial) {
  __shared__ T Ta[32][33];  // S[(k, X)][(l, Y)]
  __shared__ T Tb[32][33];  // S[(k, Y)][(l, X)]
  __shared__ T Out[SPLIT ? 32 : 1][33];
  const int nt = (v + 31) / 32, pairs = nt * (nt + 1) / 2;
  const int kl = (int)(blockIdx.x / (unsigned)pairs), pr = (int)(blockIdx.x % (unsigned)pairs);
  const int kloc = kl / o, l = kl % o, k = k0 + kloc, lloc = l - k0;
  const int tid = threadIdx.x;
  const bool inside = lloc >= 0 && lloc < ib;
  if (inside && lloc < kloc) {
    if (partial && tid == 0) partial[blockIdx.x] = 0.0;
    return;
  }
  // tile pair (tx <= ty)
  int ty = (int)((sqrtf(8.0f * (float)pr + 1.0f) - 1.0f) * 0.5f);
  while ((ty + 1) * (ty + 2) / 2 <= pr) ++ty;
  while (ty * (ty + 1) / 2 > pr) --ty;
  const int tx = pr - ty * (ty + 1) / 2;
  const int x0 = tx * 32, y0 = ty * 32;
  const long N = (long)o * v;
  const bool diag = inside && lloc == kloc;
  for (int e = tid; e < 1024; e += kBlock) {
    const int r = e / 32, c = e % 32;
    const T a = x0 + r < v && y0 + c < v ? S[((long)kloc * v + x0 + r) * N + (long)l * v + y0 + c] : T(0);
    Ta[r][c] = a;
    if (diag) {
      if (tx != ty || c >= r) Tb[c][r] = a;  // S is symmetric
    } else if (tx != ty) {
      Tb[r][c] = y0 + r < v && x0 + c < v ? S[((long)kloc * v + y0 + r) * N + (long)l * v + x0 + c] : T(0);
    } else {
      Tb[r][c] = a;
    }
  }
  __syncthreads();
  if (diag && tx == ty) {  // above its diagonal only: Tb holds the lower half
    for (int e = tid; e < 1024; e += kBlock) {
      const int r = e / 32, c = e % 32;
      if (c < r)
        Ta[r][c] = Tb[r][c];
      else
        Tb[r][c] = Ta[r][c];
    }
    __syncthreads();
  }
  double acc = 0.0;
  // elements (xb + r, yb + c) of the pair p, q (p local row block ploc): s1 = S there, s2 = S at
  // the exchanged virtuals
  auto emit = [&](int p, int ploc, int q, int xb, int yb, auto s1f, auto s2f) {
    const double epq = eo[p] + eo[q];
    for (int e = tid; e < 1024; e += kBlock) {
      const int r = e / 32, c = e % 32;
      const int x = xb + r, y = yb + c;
      double tu = 0.0;
      if (x < v && y < v) {
        const double sxy = (double)s1f(r, c), syx = (double)s2f(r, c);
        const double D = epq - ev[x] - ev[y];
        tu = (2.0 * sxy - syx) / D;
        const long row = (long)ploc * v + x, col = (long)q * v + y;
        if (!SPLIT) tau[row * ldt + col] = (T)tu;
        if (t) {
          const double tt = sxy / D;
          const long idx = row * N + col;
          t[idx] = tt;
          tEv[idx] = tt * (epq - ev[y]);
          tEo[idx] = tt * (eo[p] - ev[x] - ev[y]);
        }
        acc += tu * sxy;
      }
      if (SPLIT) Out[r][c] = (T)tu;
    }
    if constexpr (SPLIT) {
      __syncthreads();
      if (tid < 128) {
        const int r = tid / 4, c = (tid % 4) * 8;
        if (xb + r < v && yb + c < v) {
          float w[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) w[i] = (float)Out[r][c + i];
          store_sbf16_chunk(w, (float*)tau + ((long)ploc * v + xb + r) * ldt + (long)q * v + yb + c);
        }
      }
      __syncthreads();
    }
  };
  auto a = [&](int r, int c) { return Ta[r][c]; };
  auto at = [&](int r, int c) { return Ta[c][r]; };
  auto b = [&](int r, int c) { return Tb[r][c]; };
  auto bt = [&](int r, int c) { return Tb[c][r]; };
  emit(k, kloc, l, x0, y0, a, bt);
  if (tx != ty) emit(k, kloc, l, y0, x0, b, at);
  if (inside && lloc > kloc) {  // S of the pair l, k is that of k, l transposed
    emit(l, lloc, k, x0, y0, bt, a);
    if (tx != ty) emit(l, lloc, k, y0, x0, at, b);
  }
  if (partial) {
    const double s = block_sum(acc);
    if (tid == 0) partial[blockIdx.x] = s;
  }
}

// one block per chunk of x; fixed order
__global__ void sum_reduce_kernel(const double* __restrict__ x, long n, long chunk, double* __restrict__ out) {
  const long i1 = min(n, (blockIdx.x + 1) * chunk);
  double acc = 0.0;
  for (long i = blockIdx.x * chunk + threadIdx.x; i < i1; i += blockDim.x) acc += x[i];
  const double s = block_sum(acc);
  if (threadIdx.x == 0) out[blockIdx.x] = s;
}

__global__ void diag_integrals_kernel(const double* __restrict__ Bov, const double* __restrict__ Boo,
                                      const double* __restrict__ Bvv, int o, int v, int naux,
                                      double* __restrict__ coul, double* __restrict__ exch) {
  const long N = (long)o * v;
  for (long ia = blockIdx.x * (long)blockDim.x + threadIdx.x; ia < N; ia += (long)gridDim.x * blockDim.x) {
    const int i = (int)(ia / v), a = (int)(ia % v);
    double c = 0.0, x = 0.0;
    for (int P = 0; P < naux; ++P) {
      const double b = Bov[(long)P * N + ia];
      c += b * b;
      x += Boo[((long)P * o + i) * o + i] * Bvv[((long)P * v + a) * v + a];
    }
    coul[ia] = c;
    exch[ia] = x;
  }
}

__global__ void diag_assemble_kernel(int o, int v, int order, const double* __restrict__ eo,
                                     const double* __restrict__ ev, const double* __restrict__ coul,
                                     const double* __restrict__ exch, const double* __restrict__ Gv,
                                     const double* __restrict__ Ev, const double* __restrict__ Go,
                                     const double* __restrict__ Eo, double* __restrict__ dA, double* __restrict__ dB,
                                     double* __restrict__ dS) {
  const long N = (long)o * v;
  for (long ia = blockIdx.x * (long)blockDim.x + threadIdx.x; ia < N; ia += (long)gridDim.x * blockDim.x) {
    const int i = (int)(ia / v), a = (int)(ia % v);
    double A = ev[a] - eo[i], B = 0.0, S = 1.0;
    if (order >= 1) {
      A += 2.0 * coul[ia] - exch[ia];
      B = coul[ia];
    }
    if (order >= 2) {
      const double gv = Gv[(long)a * v + a], ee = Ev[(long)a * v + a];
      const double go = Go[(long)i * o + i], eoo = Eo[(long)i * o + i];
      A += -(ee - eo[i] * gv) - (ev[a] * go + eoo);
      S -= go + gv;
    }
    dA[ia] = A;
    dB[ia] = B;
    dS[ia] = S;
  }
}

__global__ void sigma_assemble_kernel(int o, int v, int k, int order, const double* __restrict__ eo,
                                      const double* __restrict__ ev, const double* __restrict__ V,
                                      const double* __restrict__ J, const double* __restrict__ P1,
                                      const double* __restrict__ P2, const double* __restrict__ P3,
                                      const double* __restrict__ P4, double* __restrict__ AV, double* __restrict__ BV,
                                      double* __restrict__ SV) {
  const long N = (long)o * v;
  const long n = N * k;
  for (long idx = blockIdx.x * (long)blockDim.x + threadIdx.x; idx < n; idx += (long)gridDim.x * blockDim.x) {
    const long ia = idx % N;
    const int i = (int)(ia / v), a = (int)(ia % v);
    const double x = V[idx];
    double av = (ev[a] - eo[i]) * x;
    double bv = 0.0;
    double sv = x;
    if (order >= 1) {
      const double j2 = 2.0 * J[idx];
      av += j2 + AV[idx];
      bv = j2 + BV[idx];
    }
    if (order >= 2) {
      av += -P2[idx] + eo[i] * P1[idx] - ev[a] * P3[idx] - P4[idx];
      sv -= P3[idx] + P1[idx];
    }
    AV[idx] = av;
    BV[idx] = bv;
    if (SV) SV[idx] = sv;
  }
}

__global__ void ring_operand_kernel(const double* __restrict__ Bov, const double* __restrict__ Lam, int o, int v,
                                    int naux, double* __restrict__ R) {
  // output R[j][s][P][a] (s in {0,1} when Lam != null) enumerated row-major
  const int ns = Lam ? 2 : 1;
  const long n = (long)o * ns * naux * v;
  const long N = (long)o * v;
  for (long idx = blockIdx.x * (long)blockDim.x + threadIdx.x; idx < n; idx += (long)gridDim.x * blockDim.x) {
    const int a = (int)(idx % v);
    long r = idx / v;
    const int P = (int)(r % naux);
    r /= naux;
    const int s = (int)(r % ns);
    const int j = (int)(r / ns);
    const long src = (long)P * N + (long)j * v + a;
    double val = Bov[src];
    if (Lam && s == 0) val += Lam[src];
    R[idx] = val;
  }
}

__global__ void axpby_kernel(long n, double alpha, const double* __restrict__ x, double beta, double* __restrict__ y) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    y[i] = alpha * x[i] + (beta == 0.0 ? 0.0 : beta * y[i]);
}

__global__ void to_f32_kernel(long n, const double* __restrict__ x, float* __restrict__ y) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    y[i] = (float)x[i];
}

// one block per bin: pairs with eps_a - eps_i in [lo, hi); sums in a fixed order
__global__ void dos_kernel(int o, int v, const double* __restrict__ eo, const double* __restrict__ ev,
                           const double* __restrict__ dip, const double* __restrict__ edges, double* __restrict__ out) {
  const int b = blockIdx.x;
  const double lo = edges[b], hi = edges[b + 1];
  const long N = (long)o * v;
  double cnt = 0.0, m2 = 0.0;
  for (long ia = threadIdx.x; ia < N; ia += blockDim.x) {
    const int i = (int)(ia / v), a = (int)(ia % v);
    const double d = ev[a] - eo[i];
    if (d >= lo && d < hi) {
      cnt += 1.0;
      if (dip) m2 += dip[ia] * dip[ia] + dip[N + ia] * dip[N + ia] + dip[2 * N + ia] * dip[2 * N + ia];
    }
  }
  cnt = block_sum(cnt);
  m2 = block_sum(m2);
  if (threadIdx.x == 0) {
    out[2 * b] = cnt;
    out[2 * b + 1] = m2;
  }
}

__global__ void response_kernel(int n, const double* __restrict__ e, const double* __restrict__ f, int ng,
                                const double* __restrict__ om, double eta, double* __restrict__ re,
                                double* __restrict__ im, double* __restrict__ lor) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= ng) return;
  const double w = om[g];
  double sr = 0.0, si = 0.0, sl = 0.0;
  const double eta2 = eta * eta;
  for (int k = 0; k < n; ++k) {
    const double c = f[k] / (2.0 * e[k]);
    const double dm = w - e[k], dp = w + e[k];
    const double qm = 1.0 / (dm * dm + eta2), qp = 1.0 / (dp * dp + eta2);
    // 1 / (d + i eta) = (d - i eta) / (d^2 + eta^2)
    sr += c * (dm * qm - dp * qp);
    si += c * (-eta * qm + eta * qp);
    sl += f[k] * qm;
  }
  if (re) re[g] = sr;
  if (im) im[g] = si;
  if (lor) lor[g] = sl * eta * 0.31830988618379067154;  // eta / pi
}

__global__ void fill_zero_kernel(long n, double* __restrict__ y) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) y[i] = 0.0;
}

__global__ void to_f32_rows_kernel(long rows, long cols, const double* __restrict__ x, long ldx,
                                   float* __restrict__ y, long ldy) {
  const long n = rows * ldy;
  for (long idx = blockIdx.x * (long)blockDim.x + threadIdx.x; idx < n; idx += (long)gridDim.x * blockDim.x) {
    const long r = idx / ldy, c = idx % ldy;
    y[idx] = c < cols ? (float)x[r * ldx + c] : 0.0f;
  }
}

// 32 x 32 tiles through LDS: reads along x's rows, writes along y's rows.
__global__ void transpose_to_f32_kernel(long rows, long cols, const double* __restrict__ x, float* __restrict__ y,
                                        long ldy) {
  __shared__ float tile[32][33];
  const long r0 = (long)blockIdx.y * 32, c0 = (long)blockIdx.x * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 256 threads: 8 rows of 32
  for (int i = ty; i < 32; i += 8) {
    const long r = r0 + i, c = c0 + tx;
    tile[i][tx] = (r < rows && c < cols) ? (float)x[r * cols + c] : 0.0f;
  }
  __syncthreads();
  for (int i = ty; i < 32; i += 8) {
    const long c = c0 + i, r = r0 + tx;
    if (c < cols && r < ldy) y[c * ldy + r] = tile[tx][i];
  }
}

__global__ void to_f64_kernel(long n, const float* __restrict__ x, double* __restrict__ y) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    y[i] = (double)x[i];
}

__global__ void combine_pairs_kernel(long N, int m, const double* __restrict__ AV, const double* __restrict__ BV,
                                     const double* __restrict__ SV, int metric, double* __restrict__ out) {
  const long n = 2 * N * m;
  for (long idx = blockIdx.x * (long)blockDim.x + threadIdx.x; idx < n; idx += (long)gridDim.x * blockDim.x) {
    const long r = idx % N;
    const long qh = idx / N;
    const int q = (int)(qh / 2), h = (int)(qh % 2);
    const long a = (long)q * N + r, b = (long)(m + q) * N + r;
    double val;
    if (metric)
      val = h == 0 ? SV[a] : -SV[b];
    else
      val = h == 0 ? AV[a] + BV[b] : BV[a] + AV[b];
    out[idx] = val;
  }
}

}  // namespace

void combine_pairs(long N, int m, const double* AV, const double* BV, const double* SV, bool metric, double* out,
                   hipStream_t s) {
  const long n = 2 * N * m;
  combine_pairs_kernel<<<grid_for(n), kBlock, 0, s>>>(N, m, AV, BV, SV, metric ? 1 : 0, out);
  PPW_LAUNCH_CHECK();
}

void permute3(const double* in, double* out, int d0, int d1, int d2, const int perm[3], hipStream_t s) {
  const long n = (long)d0 * d1 * d2;
  permute3_kernel<<<grid_for(n), kBlock, 0, s>>>(in, out, d0, d1, d2, perm[0], perm[1], perm[2]);
  PPW_LAUNCH_CHECK();
}

long tau_blocks(int o, int v, int ib) {
  const long nt = (v + 31) / 32;
  return nt * (nt + 1) / 2 * (long)ib * o;
}

namespace {
dim3 tau_grid(int o, int v, int ib) {
  const long n = tau_blocks(o, v, ib);
  if (n > 2147483647L) throw InvalidArg("amplitude strip: too many workgroups");
  return dim3((unsigned)n);
}
}  // namespace

// One FP64 strip at 96/384/1152 (the whole 36864^2 matrix): 4.4 ms against 7.2 ms when every
// tile read its transpose as well and S was complete.
void tau_strip(const double* S, int o, int v, int k0, int ib, const double* eps_o, const double* eps_v, double* tau,
               long ld, double* t, double* tEv, double* tEo, double* partial, hipStream_t s) {
  tau_strip_kernel<double, false><<<tau_grid(o, v, ib), kBlock, 0, s>>>(S, o, v, k0, ib, eps_o, eps_v, tau, ld,
                                                                        t, tEv, tEo, partial);
  PPW_LAUNCH_CHECK();
}

// split: tau in the chunk layout of split_sbf16, written by this kernel where v is a multiple of
// 8 (the strip is then not read and written once more: 13 -> 6.6 ms a strip at 128/512/1536),
// else by a pass over the finished rows.
void tau_strip_f32(const float* S, int o, int v, int k0, int ib, const double* eps_o, const double* eps_v, float* tau,
                   long ld, bool split, hipStream_t s) {
  const dim3 g = tau_grid(o, v, ib);
  if (split && v % 8 == 0) {
    tau_strip_kernel<float, true><<<g, kBlock, 0, s>>>(S, o, v, k0, ib, eps_o, eps_v, tau, ld, nullptr, nullptr,
                                                       nullptr, nullptr);
    PPW_LAUNCH_CHECK();
    return;
  }
  tau_strip_kernel<float, false><<<g, kBlock, 0, s>>>(S, o, v, k0, ib, eps_o, eps_v, tau, ld, nullptr, nullptr, nullptr,
                                                      nullptr);
  PPW_LAUNCH_CHECK();
  if (split) split_sbf16((long)ib * v * ld, tau, s);
}

void sum_reduce(const double* x, long n, double* out, hipStream_t s) {
  const long blocks = std::max(1L, std::min<long>(kSumBlocks, n / 1024));
  if (blocks > 1) {
    const long chunk = (n + blocks - 1) / blocks;
    sum_reduce_kernel<<<(unsigned)blocks, kBlock, 0, s>>>(x, n, chunk, out + 1);
    PPW_LAUNCH_CHECK();
    x = out + 1;
    n = blocks;
  }
  sum_reduce_kernel<<<1, kBlock, 0, s>>>(x, n, n, out);
  PPW_LAUNCH_CHECK();
}

void diag_integrals(const double* Bov, const double* Boo, const double* Bvv, int o, int v, int naux, double* coul,
                    double* exch, hipStream_t s) {
  diag_integrals_kernel<<<grid_for((long)o * v), kBlock, 0, s>>>(Bov, Boo, Bvv, o, v, naux, coul, exch);
  PPW_LAUNCH_CHECK();
}

void diag_assemble(int o, int v, int order, const double* eps_o, const double* eps_v, const double* coul,
                   const double* exch, const double* Gv, const double* Ev, const double* Go, const double* Eo,
                   double* dA, double* dB, double* dS, hipStream_t s) {
  diag_assemble_kernel<<<grid_for((long)o * v), kBlock, 0, s>>>(o, v, order, eps_o, eps_v, coul, exch, Gv, Ev, Go,
                                                                 Eo, dA, dB, dS);
  PPW_LAUNCH_CHECK();
}

void sigma_assemble(int o, int v, int k, int order, const double* eps_o, const double* eps_v, const double* V,
                    const double* J, const double* P1, const double* P2, const double* P3, const double* P4,
                    double* AV, double* BV, double* SV, hipStream_t s) {
  const long n = (long)o * v * k;
  sigma_assemble_kernel<<<grid_for(n), kBlock, 0, s>>>(o, v, k, order, eps_o, eps_v, V, J, P1, P2, P3, P4, AV, BV,
                                                        SV);
  PPW_LAUNCH_CHECK();
}

void build_ring_operand(const double* Bov, const double* Lam, int o, int v, int naux, double* R, hipStream_t s) {
  const long n = (long)o * (Lam ? 2 : 1) * naux * v;
  ring_operand_kernel<<<grid_for(n), kBlock, 0, s>>>(Bov, Lam, o, v, naux, R);
  PPW_LAUNCH_CHECK();
}

void axpby(long n, double alpha, const double* x, double beta, double* y, hipStream_t s) {
  axpby_kernel<<<grid_for(n), kBlock, 0, s>>>(n, alpha, x, beta, y);
  PPW_LAUNCH_CHECK();
}

void to_f32(long n, const double* x, float* y, hipStream_t s) {
  to_f32_kernel<<<grid_for(n), kBlock, 0, s>>>(n, x, y);
  PPW_LAUNCH_CHECK();
}

void response_on_grid(int n, const double* e, const double* f, int n_omega, const double* omega, double eta,
                      double* re, double* im, double* lor, hipStream_t s) {
  if (n_omega <= 0) return;
  response_kernel<<<(n_omega + kBlock - 1) / kBlock, kBlock, 0, s>>>(n, e, f, n_omega, omega, eta, re, im, lor);
  PPW_LAUNCH_CHECK();
}

void fill_zero(long n, double* y, hipStream_t s) {
  if (n <= 0) return;
  fill_zero_kernel<<<grid_for(n), kBlock, 0, s>>>(n, y);
  PPW_LAUNCH_CHECK();
}

void to_f32_rows(long rows, long cols, const double* x, long ldx, float* y, long ldy, hipStream_t s) {
  to_f32_rows_kernel<<<grid_for(rows * ldy), kBlock, 0, s>>>(rows, cols, x, ldx, y, ldy);
  PPW_LAUNCH_CHECK();
}

void transpose_to_f32(long rows, long cols, const double* x, float* y, long ldy, hipStream_t s) {
  if (rows <= 0 || cols <= 0) return;
  // padded rows of y (r >= rows up to ldy) are covered by the tiles of the last block row
  const long brows = (std::max(rows, ldy) + 31) / 32, bcols = (cols + 31) / 32;
  if (brows > 65535) throw InvalidArg("transpose_to_f32: too many rows");
  transpose_to_f32_kernel<<<dim3((unsigned)bcols, (unsigned)brows), kBlock, 0, s>>>(rows, cols, x, y, ldy);
  PPW_LAUNCH_CHECK();
}

void exciton_dos(int o, int v, const double* eo, const double* ev, const double* dip, const double* edges,
                 int n_bins, double* out, hipStream_t s) {
  dos_kernel<<<n_bins, kBlock, 0, s>>>(o, v, eo, ev, dip, edges, out);
  PPW_LAUNCH_CHECK();
}

void to_f64(long n, const float* x, double* y, hipStream_t s) {
  to_f64_kernel<<<grid_for(n), kBlock, 0, s>>>(n, x, y);
  PPW_LAUNCH_CHECK();
}

}  // namespace ppw
