// HBS compression (paper Sec. 3.2), leaf factor (Alg. 1, leaf loop) and the
// leaf steps of the apply (Alg. 2) on gfx950.

#include <algorithm>
#include <cmath>
#include <cstdlib>

#include <functional>
#include <vector>

#include "cpqr.hpp"
#include "hbs.hpp"
#include "wave.hpp"
#include "ops.hpp"
#include "prof.hpp"

namespace lsh {

// ------------------------------------------------------------- gathers
__global__ void k_gather_table(const z64* __restrict__ T, int D, const I2* __restrict__ rows, int m,
                               const I2* __restrict__ cols, int np, z64* out, long ld) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  const int i = blockIdx.y;
  if (j >= np) return;
  int dx = rows[i].x - cols[j].x, dy = rows[i].y - cols[j].y;
  dx = dx < 0 ? -dx : dx;
  dy = dy < 0 ? -dy : dy;
  out[(long)i * ld + j] = T[(long)dy * (D + 1) + dx];
}

void gather_table(hipStream_t s, const z64* T, int D, const I2* rows, int m, const I2* cols, int np, z64* out,
                  long ld) {
  if (m <= 0 || np <= 0) return;
  LSH_REQUIRE(m <= 65535 * 16, -6, "gather: too many rows");
  for (int i0 = 0; i0 < m; i0 += 65535) {
    int mm = m - i0 < 65535 ? m - i0 : 65535;
    hipLaunchKernelGGL(k_gather_table, dim3(ceil_div(np, 256), mm), dim3(256), 0, s, T, D, rows + i0, mm, cols,
                       np, out + (long)i0 * ld, ld);
    LSH_LAUNCH_CHECK();
  }
}

// rows r in [r0, r1) of the parent's proxy matrix, interleaved (r = 2q + c:
// pivot q of this level in child c): out[r][j] = T(point - prox[j]) (and
// T2 at column np + j), point = cand[J[q]] + off[c]
__global__ void k_next_gram_rows(const z64* __restrict__ T, const z64* __restrict__ T2, int D,
                                 const I2* __restrict__ cand, const int* __restrict__ J, I2 off0, I2 off1,
                                 const I2* __restrict__ prox, int np, int r0, z64* out, long ld) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  const int r = r0 + blockIdx.y;
  if (j >= np) return;
  const I2 c = cand[J[r >> 1]], o = (r & 1) ? off1 : off0;
  int dx = c.x + o.x - prox[j].x, dy = c.y + o.y - prox[j].y;
  dx = dx < 0 ? -dx : dx;
  dy = dy < 0 ? -dy : dy;
  const long t = (long)dy * (D + 1) + dx;
  out[(long)r * ld + j] = T[t];
  if (T2) out[(long)r * ld + np + j] = T2[t];
}

// M[c k + q][c' k + q'] from the interleaved rows r = 2q + c, r' = 2q' + c'
// (entry (r, r') stored when r >= r'; else the conjugate of (r', r))
__global__ void k_next_gram_pack(const z64* __restrict__ G, long ldg, int k, z64* M) {
  const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long m = 2L * k;
  if (e >= m * m) return;
  const int i = (int)(e / m), jj = (int)(e - (long)i * m);
  const int ci = i >= k, qi = i - ci * k, cj = jj >= k, qj = jj - cj * k;
  const long r = 2L * qi + ci, rr = 2L * qj + cj;
  M[e] = r >= rr ? G[r * ldg + rr] : conjg(G[rr * ldg + r]);
}

void next_gram_rows(NextGram& g, const int* J, int j) {
  if (j > g.cap) j = g.cap;
  if (j <= g.done) return;
  const int r0 = 2 * g.done, nr = 2 * (j - g.done);
  for (int a = 0; a < nr; a += 65535) {
    const int rows = nr - a < 65535 ? nr - a : 65535;
    hipLaunchKernelGGL(k_next_gram_rows, dim3(ceil_div(g.np, 256), rows), dim3(256), 0, g.gs, g.T, g.T2, g.D,
                       g.cand, J, g.off[0], g.off[1], g.prox, g.np, r0 + a, g.A, (long)g.ncols);
    LSH_LAUNCH_CHECK();
  }
  // G rows [r0, 2 j), columns [0, 2 j): the new rows against every row so far
  cgemm<double>(g.gs, nr, 2 * j, g.ncols, mk(1.0, 0.0), g.A + (long)r0 * g.ncols, g.ncols, 0, OP_N, g.A, g.ncols, 0,
                OP_C, mk(0.0, 0.0), nullptr, 0, 0, g.G + (long)r0 * 2 * g.cap, 2L * g.cap, 0, 1);
  g.done = j;
}

void next_gram_pack(hipStream_t s, const NextGram& g, int k, z64* M) {
  const long mm = 4L * k * k;
  hipLaunchKernelGGL(k_next_gram_pack, dim3(ceil_div(mm, 256L)), dim3(256), 0, s, g.G, 2L * g.cap, k, M);
  LSH_LAUNCH_CHECK();
}

__device__ __forceinline__ void wave_argmax_d(double& v, int& idx) {
  for (int off = 32; off > 0; off >>= 1) {
    double ov = __shfl_xor(v, off);
    int oi = __shfl_xor(idx, off);
    if (ov > v || (ov == v && oi < idx)) { v = ov; idx = oi; }
  }
}
__device__ __forceinline__ double readlane_f64(double v, int lane) {
  const long long bits = __double_as_longlong(v);
  return __longlong_as_double(
      (long long)(((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(bits >> 32), lane) << 32) |
                  (unsigned)__builtin_amdgcn_readlane((int)bits, lane)));
}
// ----------------------------------------------------------- CPQR row ID
// Columns of A^T are the rows of W (contiguous); Householder reflectors act
// on the proxy index.  One launch per pivot, one workgroup per row.  A step
// is a rank-one update of the whole matrix, so its bytes (32 m np) bound it
// where the matrix is large; at the sizes of direct solves on small grids
// (m = 64 .. 500 rows) the step is bound by its chain of latencies: launch,
// norms, pivot search, pivot row, dot product, norm.  Every workgroup
// therefore repeats the pivot search from the rows' norms (m values from L2)
// instead of waiting for another launch or a grid barrier to do it, and
// starts its own row's loads before the search.  Rows are not moved: W[i][a]
// holds R[a][i] for the steps a that came before row i was chosen (all steps
// for a row never chosen), Rd[a] the diagonal.  The norms are double-buffered
// by the step's parity (a workgroup may finish before another has read
// them); a chosen row's norm is -1.
// Against one workgroup holding the whole loop, setup of a 64 x 64 grid at
// tol 1e-10 (order 10, m up to 892, np up to 1224) fell from 518 to 22 ms,
// that of 32 x 32 (order 4) from 17.4 to 6.0 ms.
constexpr int QR_NT = 1024, QR_NW = QR_NT / 64;
constexpr int QS_NT = 256, QS_NW = QS_NT / 64;

__device__ __forceinline__ double cpqr_block_sum(double v, double* sb, int lane, int wave) {
  v = group_sum<64>(v);
  if (lane == 0) sb[wave] = v;
  __syncthreads();
  return (sb[0] + sb[1]) + (sb[2] + sb[3]);
}

// squared norms of the rows
__global__ __launch_bounds__(QS_NT) void k_cpqr_norms(const z64* __restrict__ W, int np, double* nrm) {
  __shared__ double sb[QS_NW];
  const int tid = threadIdx.x;
  const z64* w = W + (long)blockIdx.x * np;
  double a = 0;
  for (int q = tid; q < np; q += QS_NT) a += abs2(w[q]);
  a = cpqr_block_sum(a, sb, tid & 63, tid >> 6);
  if (tid == 0) nrm[blockIdx.x] = a;
}

// the state: thr2 = tol^2 ||A||_F^2, summed in a fixed order
__global__ __launch_bounds__(QR_NT) void k_cpqr_init(const double* nrm, int m, double tol2, int kmax,
                                                      CpqrState* st) {
  __shared__ double part[QR_NT];
  double v = 0.0;
  for (int i = threadIdx.x; i < m; i += QR_NT) v += nrm[i];
  part[threadIdx.x] = v;
  __syncthreads();
  for (int w = QR_NT / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *st = CpqrState{kmax, 0, tol2 * part[0]};
}

// Step j: the pivot p (largest norm, ties to the lower row), its reflector,
// and row blockIdx.x less its reflection.  NE entries of the row per thread
// stay in registers between the dot product and the update (np - j <=
// NE * QS_NT); NE = 0 reads the row twice (any length).
template <int NE>
__global__ __launch_bounds__(QS_NT) void k_cpqr_step(z64* W, int m, int np, int j, const double* __restrict__ nin,
                                                      double* nout, int* J, z64* Rd, CpqrState* st) {
  __shared__ double sb[QS_NW], sx[QS_NW], sy[QS_NW];
  __shared__ int si[QS_NW];
  if (st->over(j)) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, i = blockIdx.x;
  z64* w = W + (long)i * np;
  z64 e[NE > 0 ? NE : 1];
#pragma unroll
  for (int u = 0; u < NE; ++u) {
    const int q = j + tid + u * QS_NT;
    e[u] = q < np ? w[q] : mk(0.0, 0.0);
  }
  // the pivot
  double best = -1;
  int p = m;
  for (int r = tid; r < m; r += QS_NT) {
    const double a = nin[r];
    if (a > best) { best = a; p = r; }
  }
  wave_argmax_d(best, p);
  if (lane == 0) { sb[wave] = best; si[wave] = p; }
  __syncthreads();
  best = sb[0];
  p = si[0];
#pragma unroll
  for (int v = 1; v < QS_NW; ++v)
    if (sb[v] > best || (sb[v] == best && si[v] < p)) { best = sb[v]; p = si[v]; }
  if (!(best > st->thr2)) {  // (the same in every workgroup)
    if (i == 0 && tid == 0) st->stop(j);
    return;
  }
  const z64* v = W + (long)p * np;
  // Householder vector: row p from entry j on, with v_j = x0 - alpha
  const z64 x0 = v[j];
  const double nx = sqrt(best), ax0 = sqrt(abs2(x0));
  const z64 ph = ax0 > 0 ? mk(x0.x / ax0, x0.y / ax0) : mk(1.0, 0.0);
  const z64 alpha = mk(-ph.x * nx, -ph.y * nx);
  const z64 v0 = x0 - alpha;
  const double vn2 = best - ax0 * ax0 + abs2(v0);
  const double beta = vn2 > 0 ? 2.0 / vn2 : 0.0;
  if (i == p) {
    if (tid == 0) {
      J[j] = p;
      Rd[j] = alpha;
      nout[i] = -1.0;
    }
    return;
  }
  if (nin[i] < 0) {  // chosen before
    if (tid == 0) nout[i] = -1.0;
    return;
  }
  z64 h[NE > 0 ? NE : 1];
  z64 acc = mk(0.0, 0.0);
  if (NE > 0) {
#pragma unroll
    for (int u = 0; u < NE; ++u) {
      const int q = j + tid + u * QS_NT;
      h[u] = q < np ? v[q] : mk(0.0, 0.0);
    }
    if (tid == 0) h[0] = v0;
#pragma unroll
    for (int u = 0; u < NE; ++u) fma_acc(acc, conjg(h[u]), e[u]);
  } else {
    for (int q = j + tid; q < np; q += QS_NT) fma_acc(acc, conjg(q == j ? v0 : v[q]), w[q]);
  }
  acc.x = group_sum<64>(acc.x);
  acc.y = group_sum<64>(acc.y);
  if (lane == 0) {
    sx[wave] = acc.x;
    sy[wave] = acc.y;
  }
  __syncthreads();
  const z64 f = beta * mk((sx[0] + sx[1]) + (sx[2] + sx[3]), (sy[0] + sy[1]) + (sy[2] + sy[3]));
  double nn = 0;
  if (NE > 0) {
#pragma unroll
    for (int u = 0; u < NE; ++u) {
      const int q = j + tid + u * QS_NT;
      if (q < np) {
        const z64 t = e[u] - f * h[u];
        w[q] = t;
        if (q > j) nn += abs2(t);
      }
    }
  } else {
    for (int q = j + tid; q < np; q += QS_NT) {
      const z64 t = w[q] - f * (q == j ? v0 : v[q]);
      w[q] = t;
      if (q > j) nn += abs2(t);
    }
  }
  // (sb was last read before the barrier above)
  nn = cpqr_block_sum(nn, sb, lane, wave);
  if (tid == 0) nout[i] = nn;
}

// U rows of the rows off the skeleton, (R11^{-1} R12)^T: row x of U solves
// x L = t with L[a][b] = W[J[a]][b] (b < a), L[a][a] = Rd[a], t = the row's
// entries of W, by substitution from the last column.  One wave per row, the
// row in registers (column lane + 64 u, u < NU; k <= 64 NU): step a
// broadcasts x_a and subtracts x_a L[a][:], row a - 1 in flight meanwhile.
// k_cpqr_units writes the skeleton's unit rows.
template <int NU>
__global__ __launch_bounds__(64) void k_cpqr_interp(const z64* __restrict__ W, int np, int k,
                                                    const int* __restrict__ J, const z64* __restrict__ Rd,
                                                    const int* __restrict__ rest, z64* __restrict__ U) {
  const int lane = threadIdx.x, row = rest[blockIdx.x];
  const z64* w = W + (long)row * np;
  z64 t[NU], nx[NU];
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int c = lane + 64 * u;
    t[u] = c < k ? w[c] : mk(0.0, 0.0);
    nx[u] = mk(0.0, 0.0);
  }
#pragma unroll
  for (int ub = NU - 1; ub >= 0; --ub) {
    if (64 * ub >= k) continue;
    const int top = (k - 64 * ub < 64 ? k - 64 * ub : 64) - 1;
    const int jl = 64 * ub + lane < k ? J[64 * ub + lane] : 0;  // this block's pivots and diagonal
    const z64 rl = 64 * ub + lane < k ? crecip(Rd[64 * ub + lane]) : mk(0.0, 0.0);
    {
      const z64* l = W + (long)__builtin_amdgcn_readlane(jl, top) * np;
#pragma unroll
      for (int u = 0; u <= ub; ++u)
        nx[u] = lane + 64 * u < 64 * ub + top ? l[lane + 64 * u] : mk(0.0, 0.0);
    }
    for (int al = top; al >= 0; --al) {
      const int a = 64 * ub + al;
      z64 cur[NU];
#pragma unroll
      for (int u = 0; u <= ub; ++u) cur[u] = nx[u];
      if (al > 0) {
        const z64* l = W + (long)__builtin_amdgcn_readlane(jl, al - 1) * np;
#pragma unroll
        for (int u = 0; u <= ub; ++u) nx[u] = lane + 64 * u < a - 1 ? l[lane + 64 * u] : mk(0.0, 0.0);
      }
      const z64 x = mk(readlane_f64(t[ub].x, al), readlane_f64(t[ub].y, al)) *
                    mk(readlane_f64(rl.x, al), readlane_f64(rl.y, al));
#pragma unroll
      for (int u = 0; u <= ub; ++u) t[u] = t[u] - x * cur[u];  // (cur is zero from column a on)
      if (lane == al) t[ub] = x;
    }
  }
#pragma unroll
  for (int u = 0; u < NU; ++u)
    if (lane + 64 * u < k) U[(long)row * k + lane + 64 * u] = t[u];
}

// the same for any k, the row in U itself, a workgroup per row
__global__ __launch_bounds__(QS_NT) void k_cpqr_interp_long(const z64* __restrict__ W, int np, int k,
                                                             const int* __restrict__ J, const z64* __restrict__ Rd,
                                                             const int* __restrict__ rest, z64* U) {
  const int tid = threadIdx.x, row = rest[blockIdx.x];
  const z64* w = W + (long)row * np;
  z64* u = U + (long)row * k;
  for (int c = tid; c < k; c += QS_NT) u[c] = w[c];
  __syncthreads();
  for (int a = k - 1; a >= 0; --a) {
    const z64 x = u[a] * crecip(Rd[a]);
    const z64* l = W + (long)J[a] * np;
    for (int c = tid; c < a; c += QS_NT) u[c] = u[c] - x * l[c];
    __syncthreads();  // (u[a] has been read by every thread)
    if (tid == 0) u[a] = x;
  }
}

__global__ void k_cpqr_units(z64* U, int k, const int* J) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= k * k) return;
  const int a = e / k, b = e % k;
  U[(long)J[a] * k + b] = mk(a == b ? 1.0 : 0.0, 0.0);
}

size_t rowid_cpqr_ws(int m) {
  return (size_t)m * (2 * sizeof(double) + sizeof(z64) + sizeof(int)) + sizeof(CpqrState) + 5 * 256;
}

int rowid_cpqr(hipStream_t s, z64* A, int m, int np, double tol, int* J, std::vector<int>& Jh, z64* U, void* ws,
               const std::function<void(int)>& on_skel) {
  ProfScope ps("cpqr", s, 16.0 * (double)m * np);
  char* wp = static_cast<char*>(ws);
  auto take = [&](size_t bytes) { char* r = wp; wp += ((bytes + 255) / 256) * 256; return (void*)r; };
  double* nrm[2];
  nrm[0] = static_cast<double*>(take(sizeof(double) * m));
  nrm[1] = static_cast<double*>(take(sizeof(double) * m));
  z64* Rd = static_cast<z64*>(take(sizeof(z64) * m));
  int* rest = static_cast<int*>(take(sizeof(int) * m));
  CpqrState* st = static_cast<CpqrState*>(take(sizeof(CpqrState)));
  const int kmax = m < np ? m : np;
  hipLaunchKernelGGL(k_cpqr_norms, dim3(m), dim3(QS_NT), 0, s, A, np, nrm[0]);
  LSH_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_cpqr_init, dim3(1), dim3(QR_NT), 0, s, nrm[0], m, tol * tol, kmax, st);
  LSH_LAUNCH_CHECK();
  // steps in batches, the done flag read once per batch: a step queued after
  // the end returns at entry
  constexpr int BATCH = 32;
  CpqrState h{kmax, 0, 0.0};
  for (int j = 0; j < kmax && !h.done;) {
    const int end = j + BATCH < kmax ? j + BATCH : kmax;
    for (; j < end; ++j) {
      const int ne = ceil_div(np - j, QS_NT);
      auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(m), dim3(QS_NT), 0, s, A, m, np, j, nrm[j & 1], nrm[1 - (j & 1)], J, Rd, st);
      };
      if (ne <= 1) go(k_cpqr_step<1>);
      else if (ne <= 2) go(k_cpqr_step<2>);
      else if (ne <= 4) go(k_cpqr_step<4>);
      else if (ne <= 8) go(k_cpqr_step<8>);
      else go(k_cpqr_step<0>);
      LSH_LAUNCH_CHECK();
    }
    LSH_HIP(hipMemcpyAsync(&h, st, sizeof(h), hipMemcpyDeviceToHost, s));
    LSH_HIP(hipStreamSynchronize(s));
  }
  int k = h.k;
  if (k < 1) {  // a zero block still gets one skeleton: row 0, U = e_0
    k = 1;
    const int zero = 0;
    const z64 one = mk(1.0, 0.0);
    LSH_HIP(hipMemcpyAsync(J, &zero, sizeof(int), hipMemcpyHostToDevice, s));
    fill_zero(s, U, sizeof(z64) * (size_t)m);
    LSH_HIP(hipMemcpyAsync(U, &one, sizeof(z64), hipMemcpyHostToDevice, s));
    LSH_HIP(hipStreamSynchronize(s));
    Jh.assign(1, 0);
    if (on_skel) on_skel(k);
    return k;
  }
  // the skeleton to the host: the other rows' list, and the caller's notice
  std::vector<int> rh;
  Jh.resize(k);
  LSH_HIP(hipMemcpyAsync(Jh.data(), J, sizeof(int) * k, hipMemcpyDeviceToHost, s));
  LSH_HIP(hipStreamSynchronize(s));
  std::vector<char> used(m, 0);
  for (int v : Jh) {
    LSH_REQUIRE(v >= 0 && v < m && !used[v], -4, "row ID: skeleton rows not distinct");
    used[v] = 1;
  }
  for (int i = 0; i < m; ++i)
    if (!used[i]) rh.push_back(i);
  const int nr = (int)rh.size();
  if (on_skel) on_skel(k);
  if (nr) {
    LSH_HIP(hipMemcpyAsync(rest, rh.data(), sizeof(int) * nr, hipMemcpyHostToDevice, s));
    auto go = [&](auto kern, int nt) {
      hipLaunchKernelGGL(kern, dim3(nr), dim3(nt), 0, s, A, np, k, J, Rd, rest, U);
    };
    if (k <= 64) go(k_cpqr_interp<1>, 64);
    else if (k <= 128) go(k_cpqr_interp<2>, 64);
    else if (k <= 256) go(k_cpqr_interp<4>, 64);
    else if (k <= 512) go(k_cpqr_interp<8>, 64);
    else go(k_cpqr_interp_long, QS_NT);
    LSH_LAUNCH_CHECK();
  }
  hipLaunchKernelGGL(k_cpqr_units, dim3(ceil_div((long)k * k, 256)), dim3(256), 0, s, U, k, J);
  LSH_LAUNCH_CHECK();
  LSH_HIP(hipStreamSynchronize(s));  // (rh goes)
  return k;
}

// ------------------------------------------- Gram / pivoted Cholesky row ID
__global__ void k_gram_init(const z64* M, int m, double* d, int* chosen, int* state) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < m) { d[i] = M[(long)i * m + i].x; chosen[i] = 0; }
  if (i == 0) { state[0] = 0; state[1] = 0; }
}

// One-workgroup panel of nb <= PCH_NB pivots.  Per pivot: block argmax of the
// Schur diagonal over unchosen rows, then the new column
//   l_i = (conj(M[p][i]) - sum_{t in panel} L[i][t] conj(L[p][t])) / sqrt(d_p)
// where each thread first issues all its panel loads (independent, in
// registers) and the pivot row's panel entries come from LDS.
constexpr int PCH_NB = 32, PCH_MAXM = 4096;

__global__ __launch_bounds__(QR_NT) void k_pchol_panel(const z64* __restrict__ M, int m, double* d, int* chosen,
                                                        z64* Lt, int* piv, int j0, int nb, double thr2,
                                                        int* state) {
  constexpr int RPT = PCH_MAXM / QR_NT;  // rows per thread
  extern __shared__ unsigned char smem_raw[];
  double* ds = reinterpret_cast<double*>(smem_raw);        // Schur diagonal (m)
  unsigned char* cs = smem_raw + sizeof(double) * m;        // chosen flags (m)
  __shared__ double sb[QR_NW];
  __shared__ int si[QR_NW];
  __shared__ int s_p;
  __shared__ double s_d;
  __shared__ z64 lpc[PCH_NB];  // conj(L[p][t]) for the panel columns so far
  if (state[1]) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int i = tid; i < m; i += QR_NT) {
    ds[i] = d[i];
    cs[i] = (unsigned char)chosen[i];
  }
  __syncthreads();
  int jj = 0;
  bool stop = false;
  for (; jj < nb; ++jj) {
    const int j = j0 + jj;
    if (j >= m) {
      if (tid == 0) { state[0] = m; state[1] = 1; }
      stop = true;
      break;
    }
    double best = -1;
    int bi = m;
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
      const int i = tid + r * QR_NT;
      if (i < m && !cs[i]) {
        const double a = ds[i];
        if (a > best || (a == best && i < bi)) { best = a; bi = i; }
      }
    }
    wave_argmax_d(best, bi);
    if (lane == 0) { sb[wave] = best; si[wave] = bi; }
    __syncthreads();
    if (tid < 64) {  // final reduction by one wave, then stage the pivot's panel row
      double bb = tid < QR_NW ? sb[tid] : -1.0;
      int ii = tid < QR_NW ? si[tid] : m;
      wave_argmax_d(bb, ii);
      if (tid == 0) { s_p = ii; s_d = bb; }
      if (tid < jj && ii < m) lpc[tid] = conjg(Lt[(long)(j0 + tid) * m + ii]);
    }
    __syncthreads();
    const int p = s_p;
    const double dp = s_d;
    if (!(dp > thr2)) {
      if (tid == 0) { state[0] = j; state[1] = 1; }
      stop = true;
      break;
    }
    const double sq = sqrt(dp), rs = 1.0 / sq;
    // issue every row's loads before any arithmetic
    z64 l[RPT];
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
      const int i = tid + r * QR_NT;
      l[r] = (i < m) ? conjg(M[(long)p * m + i]) : mk(0.0, 0.0);
    }
    for (int t0 = 0; t0 < jj; t0 += 4) {
      z64 v[RPT][4];
#pragma unroll
      for (int r = 0; r < RPT; ++r)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int i = tid + r * QR_NT;
          v[r][t] = (i < m && t0 + t < jj) ? Lt[(long)(j0 + t0 + t) * m + i] : mk(0.0, 0.0);
        }
#pragma unroll
      for (int r = 0; r < RPT; ++r)
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if (t0 + t < jj) l[r] = l[r] - v[r][t] * lpc[t0 + t];
    }
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
      const int i = tid + r * QR_NT;
      if (i >= m) continue;
      z64 li;
      if (i == p) li = mk(sq, 0.0);
      else if (cs[i]) li = mk(0.0, 0.0);
      else {
        li = rs * l[r];
        ds[i] -= abs2(li);
      }
      Lt[(long)j * m + i] = li;
    }
    __syncthreads();
    if (tid == 0) { cs[p] = 1; piv[j] = p; ds[p] = 0; }
    __syncthreads();
  }
  for (int i = tid; i < m; i += QR_NT) {
    d[i] = ds[i];
    chosen[i] = cs[i];
  }
  if (!stop && tid == 0) state[0] = j0 + nb;
}


__global__ void k_gather_L11(const z64* Lt, int m, const int* piv, int k, z64* L11) {
  const long e = blockIdx.x * (long)blockDim.x + threadIdx.x;
  if (e >= (long)k * k) return;
  const int a = (int)(e / k), b = (int)(e % k);
  L11[e] = Lt[(long)b * m + piv[a]];
}

// Lr[r][t] = L(rest[r], t)
__global__ void k_gather_rows(const z64* Lt, int m, const int* rest, int nr, int k, z64* Lr) {
  const long e = blockIdx.x * (long)blockDim.x + threadIdx.x;
  if (e >= (long)nr * k) return;
  const int r = (int)(e / k), t = (int)(e % k);
  Lr[e] = Lt[(long)t * m + rest[r]];
}

// Inverses of the 64 x 64 lower-triangular diagonal blocks of L11 (the last
// block padded with the identity), one workgroup per block, in LDS: the four
// 16 x 16 diagonal blocks by forward substitution, a thread per column with
// the column in registers, then joined by doubling (inv [[A, 0], [B, C]] =
// [[A^-1, 0], [-C^-1 B A^-1, C^-1]]).  Bound by its chain of LDS latencies:
// 16 dependent steps and four barriers, 32 us a launch at n = 256; 64 steps
// with a lane exchange each took 130.
constexpr int TRI_B = 64;
__global__ __launch_bounds__(256) void k_trinv_blocks(const z64* L11, int k, z64* Dinv) {
  constexpr int S = 16, LD = TRI_B + 1;
  __shared__ z64 X[TRI_B][LD];
  __shared__ z64 T[32][33];
  const int tid = threadIdx.x, base = blockIdx.x * TRI_B;
  for (int e = tid; e < TRI_B * TRI_B; e += 256) {
    const int r = e / TRI_B, c = e % TRI_B, gi = base + r, gj = base + c;
    z64 v = mk(0.0, 0.0);
    if (gi < k && gj < k) v = r >= c ? L11[(long)gi * k + gj] : v;
    else if (r == c) v = mk(1.0, 0.0);
    X[r][c] = v;
  }
  __syncthreads();
  if (tid < TRI_B) {  // column tid % 16 of diagonal block tid / 16
    const int o = tid & ~(S - 1), c = tid & (S - 1);
    z64 x[S];
#pragma unroll
    for (int q = 0; q < S; ++q) {
      z64 t = mk(q == c ? 1.0 : 0.0, 0.0);
#pragma unroll
      for (int r = 0; r < q; ++r) t = t - X[o + q][o + r] * x[r];
      x[q] = t * crecip(X[o + q][o + q]);
    }
    // (one wave: every column has been read before any is written)
#pragma unroll
    for (int q = 0; q < S; ++q) X[o + q][o + c] = x[q];
  }
  __syncthreads();
#pragma unroll
  for (int h = S; h < TRI_B; h *= 2) {
    // pairs (A at i0, C at i0 + h): T = B A^-1, then B <- -C^-1 T
    const int np = TRI_B / (2 * h), tot = np * h * h;
    for (int e = tid; e < tot; e += 256) {
      const int q = e / (h * h), r = e / h % h, c = e % h, i0 = q * 2 * h;
      z64 t = mk(0.0, 0.0);
      for (int u = c; u < h; ++u) fma_acc(t, X[i0 + h + r][i0 + u], X[i0 + u][i0 + c]);
      T[q * h + r][c] = t;
    }
    __syncthreads();
    for (int e = tid; e < tot; e += 256) {
      const int q = e / (h * h), r = e / h % h, c = e % h, i0 = q * 2 * h;
      z64 t = mk(0.0, 0.0);
      for (int u = 0; u <= r; ++u) fma_acc(t, X[i0 + h + r][i0 + h + u], T[q * h + u][c]);
      X[i0 + h + r][i0 + c] = mk(-t.x, -t.y);
    }
    __syncthreads();
  }
  z64* D = Dinv + (long)blockIdx.x * TRI_B * TRI_B;
  for (int e = tid; e < TRI_B * TRI_B; e += 256) D[e] = X[e / TRI_B][e % TRI_B];
}

// U[piv[a]] = e_a ; U[rest[r]] = X[r]
__global__ void k_scatter_U(z64* U, int k, const int* piv, const int* rest, int nr, const z64* X) {
  const long e = blockIdx.x * (long)blockDim.x + threadIdx.x;
  const long tot = (long)(k + nr) * k;
  if (e >= tot) return;
  const int row = (int)(e / k), b = (int)(e % k);
  if (row < k) U[(long)piv[row] * k + b] = mk(row == b ? 1.0 : 0.0, 0.0);
  else U[(long)rest[row - k] * k + b] = X[(long)(row - k) * k + b];
}

// ------------------------------------ block-pivoted left-looking Cholesky
// The panels above take one pivot per workgroup-wide step and keep the whole
// Schur complement M - L L^H up to date (a rank-nb update of all m x m
// entries per panel).  The block variant below takes up to BP_NP pivots per
// step and never forms the trailing Schur complement:
//  1. candidates C = the BP_B unchosen rows with the largest Schur diagonal
//     d_i (radix selection), and dout = the largest d_i outside C;
//  2. S_C = M[C,C] - L[C,:] L[C,:]^H;
//  3. greedy pivoted Cholesky of S_C in one workgroup: pivots P, factor L_PP
//     and its inverse;
//  4. the new columns L[:, P] = (M[:, P] - L L[P,:]^H) L_PP^{-H} and
//     d_i -= |L[i, P]|^2.
// Step 3 stops before a pivot whose Schur diagonal falls below alpha * dout.
// Diagonals only decrease, so every pivot taken has a Schur diagonal of at
// least alpha times the largest over all rows.  With alpha = 1 each pivot is
// the greedy pivot, and the pivot sequence, the stopping point and the rank
// are those of one-at-a-time greedy pivoting (up to ties); alpha < 1 takes
// more pivots per step (alpha-greedy pivoting: the same stopping rule, so the
// same error bound, with a rank that can differ by a few).  All step state (rank so far,
// pivot count, done flag) lives on the device: the host queues steps in
// batches and reads the done flag once per batch; a step queued after the
// end returns at entry.
constexpr int BP_B = 48, BP_NP = 32, BP_KCMAX = 128, BP_KCS = 64, BP_SEL = 16384;
// state words (int): 0 rank j, 1 done, 2 pivots of this step, 3 candidates,
// 4..5 dout (double), 6 error flag, 8..8+BP_B candidate rows, 120..121 the
// stopping threshold thr2 (double)
constexpr int BPS_J = 0, BPS_DONE = 1, BPS_NP = 2, BPS_NC = 3, BPS_DOUT = 4, BPS_ERR = 6, BPS_CAND = 8,
              BPS_THR = 120, BPS_WORDS = 128;
static_assert(BPS_CAND + BP_B <= BPS_THR && BPS_THR + 2 <= BPS_WORDS - 4, "step state layout");

// thr2 = tol^2 sum_i d_i (the squared Frobenius norm of the candidate
// matrix), in one workgroup with a fixed summation order
__global__ __launch_bounds__(1024) void k_bp_thr2(const double* d, int m, double tol2, int* st) {
  __shared__ double part[1024];
  double v = 0.0;
  for (int i = threadIdx.x; i < m; i += 1024) v += d[i];
  part[threadIdx.x] = v;
  __syncthreads();
  for (int w = 512; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) reinterpret_cast<double*>(st + BPS_THR)[0] = tol2 * part[0];
}

// selection key of candidate row i: the Schur diagonal's bits above the
// index field, then the complemented index (ties go to the lower row)
constexpr unsigned BP_IDX = 0x3FFF;  // index field: rows < BP_SEL
static_assert(BP_SEL <= BP_IDX + 1, "key index field");
__device__ __forceinline__ unsigned long long bp_key(double d, int i) {
  return d > 0.0 ? (((unsigned long long)__double_as_longlong(d) & ~(unsigned long long)BP_IDX) | (BP_IDX - i))
                 : 0ull;
}

// Candidates: the BP_B largest keys (unchosen rows, d > 0) by an 8-pass
// most-significant-digit radix selection of the BP_B-th largest key, then
// the <= BP_B keys at or above it, sorted descending.
// KPT keys per thread: m <= 1024 KPT
template <int KPT>
__global__ __launch_bounds__(1024) void k_bp_select(const double* d, const int* chosen, int m, int* st) {
  __shared__ unsigned int hist[256];
  __shared__ unsigned long long s_prefix, s_mask;
  __shared__ int s_rank, s_cnt, s_stop;
  __shared__ unsigned long long ck[64];
  __shared__ unsigned long long s_below;
  if (st[BPS_DONE]) return;
  const double thr2 = reinterpret_cast<const double*>(st + BPS_THR)[0];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // the previous step's pivots join the rank here (every later kernel of
  // this step reads the rank after this kernel has ended)
  {
    const int jn = st[BPS_J] + st[BPS_NP];
    __syncthreads();
    if (tid == 0) {
      st[BPS_J] = jn;
      st[BPS_NP] = 0;
      if (jn >= m) st[BPS_DONE] = 1;
    }
    if (jn >= m) return;
  }
  unsigned long long key[KPT];
  int nz = 0;
#pragma unroll
  for (int r = 0; r < KPT; ++r) {
    const int i = tid + r * 1024;
    key[r] = (i < m && !chosen[i]) ? bp_key(d[i], i) : 0ull;
    nz += key[r] != 0;
  }
  if (tid == 0) { s_prefix = 0; s_mask = 0; s_rank = BP_B; s_cnt = 0; s_below = 0; s_stop = 0; }
  // total nonzero keys: when at most BP_B, every one is a candidate
  for (int off = 32; off > 0; off >>= 1) nz += __shfl_xor(nz, off);
  __shared__ int wz[16];
  if (lane == 0) wz[wave] = nz;
  __syncthreads();
  int total = 0;
  for (int w = 0; w < 16; ++w) total += wz[w];
  unsigned long long thr = 1;  // keys >= thr are candidates
  if (total > BP_B) {
    for (int pass = 7; pass >= 0; --pass) {
      const int sh = 8 * pass;
      for (int b = tid; b < 256; b += 1024) hist[b] = 0;
      __syncthreads();
      const unsigned long long pre = s_prefix, msk = s_mask;
#pragma unroll
      for (int r = 0; r < KPT; ++r)
        if (key[r] && (key[r] & msk) == pre) atomicAdd(&hist[(key[r] >> sh) & 255], 1u);
      __syncthreads();
      if (wave == 0) {
        // bins from the top: lane l holds bins 255-4l .. 252-4l
        unsigned int c[4], sum = 0;
        for (int q = 0; q < 4; ++q) { c[q] = hist[255 - 4 * lane - q]; sum += c[q]; }
        unsigned int inc = sum;  // inclusive prefix over lanes
        for (int off = 1; off < 64; off <<= 1) {
          const unsigned int o = __shfl_up(inc, off);
          if (lane >= off) inc += o;
        }
        const unsigned int exc = inc - sum;
        const int rank = s_rank;
        if ((int)exc < rank && rank <= (int)inc) {
          unsigned int run = exc;
          for (int q = 0; q < 4; ++q) {
            if (rank <= (int)(run + c[q])) {
              const unsigned long long digit = 255 - 4 * lane - q;
              s_prefix = pre | (digit << sh);
              s_mask = msk | (255ull << sh);
              s_rank = rank - (int)run;
              // the whole bin is among the BP_B largest: keys >= the prefix
              // (lower digits zero) are exactly the candidates
              if (rank - (int)run == (int)c[q]) s_stop = 1;
              break;
            }
            run += c[q];
          }
        }
      }
      __syncthreads();
      if (s_stop) break;  // (uniform)
    }
    thr = s_prefix;
  }
  // gather the candidates and the largest key below them
  unsigned long long below = 0;
#pragma unroll
  for (int r = 0; r < KPT; ++r) {
    if (key[r] >= thr && key[r]) {
      const int slot = atomicAdd(&s_cnt, 1);
      if (slot < 64) ck[slot] = key[r];
    } else if (key[r] > below) {
      below = key[r];
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    const unsigned long long o = __shfl_xor(below, off);
    below = o > below ? o : below;
  }
  if (lane == 0) atomicMax(&s_below, below);
  __syncthreads();
  if (wave == 0) {
    const int cnt = s_cnt < BP_B ? s_cnt : BP_B;
    unsigned long long k = lane < cnt ? ck[lane] : 0ull;
    // bitonic sort of 64 keys across the wave, descending
    for (int size = 2; size <= 64; size <<= 1)
      for (int stride = size >> 1; stride > 0; stride >>= 1) {
        const unsigned long long o = __shfl_xor(k, stride);
        const bool up = (lane & size) == 0;  // descending blocks
        const bool lower = (lane & stride) == 0;
        const bool takeMax = (up == lower);
        k = takeMax ? (o > k ? o : k) : (o < k ? o : k);
      }
    const int row = k ? (int)(BP_IDX - (unsigned)(k & BP_IDX)) : -1;
    if (lane < BP_B) st[BPS_CAND + lane] = row;
    int valid = (lane < BP_B && row >= 0 && d[row] > thr2) ? 1 : 0;
    for (int off = 32; off > 0; off >>= 1) valid += __shfl_xor(valid, off);
    if (lane == 0) {
      st[BPS_NC] = valid;
      const unsigned long long kb = s_below;
      reinterpret_cast<double*>(st + BPS_DOUT)[0] = kb ? d[BP_IDX - (unsigned)(kb & BP_IDX)] : 0.0;
      if (valid == 0) st[BPS_DONE] = 1;
    }
  }
}

// S_C partial sums: blockIdx.x = depth chunk c (BP_KCS deep), blockIdx.y =
// output quadrant (rows a0.., columns b0.., each BP_B / 2 wide):
// part[c][a][b] = sum_{t in chunk, t < j} L(C_a, t) conj(L(C_b, t)).  The chunk
// is staged at once; a lane of each of the four waves takes 3 x 3 outputs (six
// LDS reads for nine products; LDS bandwidth bounds the kernel, after the
// staging's latency) over a quarter of the depth, and the waves' sums meet in
// LDS.  With one output at a time per thread and two stagings: 14 us a step at
// depth 700, this way 12.
__global__ __launch_bounds__(256) void k_bp_sc(const z64* Lt, int m, const int* st, z64* part) {
  constexpr int H = BP_B / 2, Q = BP_KCS / 4;
  static_assert(H == 24, "64 lanes of 3 x 3 outputs");
  __shared__ z64 stage[2][BP_KCS][H + 1];
  static_assert(2 * BP_KCS * (H + 1) >= 4 * H * H, "the waves' sums fit the staging");
  z64(*La)[H + 1] = stage[0];
  z64(*Lb2)[H + 1] = stage[1];
  if (st[BPS_DONE]) return;
  const int j = st[BPS_J], nc = st[BPS_NC];
  const int c = blockIdx.x, t0 = c * BP_KCS;
  if (t0 >= j) return;
  const int a0 = (blockIdx.y >> 1) * H, b0 = (blockIdx.y & 1) * H;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int* cand = st + BPS_CAND;
  for (int e = tid; e < 2 * BP_KCS * H; e += 256) {
    const int half = e / (BP_KCS * H), f = e % (BP_KCS * H), t = f / H, a = f % H;
    const int row = (half ? b0 : a0) + a;
    const z64 v = (row < nc && t0 + t < j) ? Lt[(long)(t0 + t) * m + cand[row]] : mk(0.0, 0.0);
    if (half) Lb2[t][a] = conjg(v);
    else La[t][a] = v;
  }
  __syncthreads();
  const int ta = lane >> 3, tb = lane & 7;  // outputs ta + 8 i, tb + 8 k
  z64 acc[3][3];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int k = 0; k < 3; ++k) acc[i][k] = mk(0.0, 0.0);
  for (int t = wave * Q; t < (wave + 1) * Q; ++t) {
    z64 x[3], y[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      x[i] = La[t][ta + 8 * i];
      y[i] = Lb2[t][tb + 8 * i];
    }
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int k = 0; k < 3; ++k) fma_acc(acc[i][k], x[i], y[k]);
  }
  __syncthreads();
  z64* red = &La[0][0];  // [wave][output]
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int k = 0; k < 3; ++k) red[wave * H * H + (ta + 8 * i) * H + tb + 8 * k] = acc[i][k];
  __syncthreads();
  for (int e = tid; e < H * H; e += 256)
    part[(long)c * BP_B * BP_B + (a0 + e / H) * BP_B + b0 + e % H] =
        (red[e] + red[H * H + e]) + (red[2 * H * H + e] + red[3 * H * H + e]);
}

// Greedy pivoted Cholesky of the candidate block S_C = M[C,C] - sum_c
// part[c] (formed first, in LDS; zero past the nc candidates) while the
// pivot exceeds thr2 and, after the first, is not below alpha * dout; at
// most BP_NP pivots.  Writes J[j + q], the pivot count, Lpp (np x np, lower,
// pivot order) and Linv = Lpp^{-1}, both with ld BP_NP; sets done when no
// pivot qualifies.
//
// Four waves: lane b of wave w holds rows 12w..12w+11 of column b of S in
// registers, and every wave keeps all the Schur diagonals d_b (lane b).  Per
// pivot p: the wave that holds row p writes column t of the factor (rl times
// the row's conjugate, an entry per lane, zero in picked rows) to LDS, one
// barrier, then every lane updates its rows, S[:, b] -= L[:, t] conj(L[b, t]),
// and d_b -= |L[b, t]|^2.  The next pivot's search (a DPP maximum of d) is
// independent of the row updates, so the two run interleaved.  Pivot keys hold
// the top 26 bits of d (sign, exponent, 14 mantissa bits): diagonals within a
// relative 2^-14 of the largest count as ties, won by the lower candidate.
// L_PP^{-1} follows by forward substitution inside each wave.  Bound by the
// pivots' chain of latencies: with the column written by the pivot's lane of
// each wave (twelve writes of one lane) a step of 24 pivots at depth 700 took
// 50 us, this way 33.  (Joining the partial sums above into this launch, and
// the selection into the new-columns one, by the workgroup that ends last was
// slower, n = 1024 111 against 103 ms a setup: each workgroup's device fence
// writes its L2 back, beside the factor's products.)
constexpr int BP_CW = 4, BP_CR = BP_B / BP_CW;  // waves, rows per wave
__global__ __launch_bounds__(64 * BP_CW) void k_bp_chol(const z64* M, const z64* part, int m, double alpha, int* J,
                                                        int* st, z64* Lpp, z64* Linv) {
  static_assert(BP_B <= 64 && BP_NP == 32 && BP_CR == 12 && BP_CW * 8 == BP_NP,
                "one lane per candidate; 8 columns of L_PP^{-1} per wave");
  __shared__ z64 Ss[BP_B][BP_B + 1];   // S_C
  __shared__ z64 Lb[BP_NP][BP_B + 1];  // factor columns for every candidate row: [column][row]
  __shared__ z64 xs[BP_NP][BP_NP + 1]; // L_PP^{-1}
  __shared__ double rlv[BP_NP];        // 1 / L[t][t]
  __shared__ int piv[BP_NP];
  if (st[BPS_DONE]) return;
  const int tid = threadIdx.x, b = tid & 63, w = tid >> 6, r0 = w * BP_CR;
  const int nc = st[BPS_NC], j = st[BPS_J];
  const double dout = alpha * reinterpret_cast<const double*>(st + BPS_DOUT)[0];
  const double thr2 = reinterpret_cast<const double*>(st + BPS_THR)[0];
  const int* cand = st + BPS_CAND;
  {  // S_C: the Gram entries less the depth chunks' partial products, in chunk order.  Each thread
     // holds PE entries and loads CB chunks of all of them at a time (PE * CB loads in flight).
    const int nch = (j + BP_KCS - 1) / BP_KCS;
    constexpr long CS = (long)BP_B * BP_B;
    constexpr int PE = BP_B * BP_B / (64 * BP_CW), CB = 4;
    static_assert(PE * 64 * BP_CW == BP_B * BP_B, "entries per thread");
    z64 v[PE];
    bool live[PE];
#pragma unroll
    for (int i = 0; i < PE; ++i) {
      const int e = tid + i * 64 * BP_CW, a = e / BP_B, c2 = e % BP_B;
      live[i] = a < nc && c2 < nc;
      v[i] = live[i] ? M[(long)cand[a] * m + cand[c2]] : mk(0.0, 0.0);
    }
    int c = 0;
    for (; c + CB <= nch; c += CB) {
      z64 pv[CB][PE];
#pragma unroll
      for (int q = 0; q < CB; ++q)
#pragma unroll
        for (int i = 0; i < PE; ++i)
          pv[q][i] = live[i] ? part[(c + q) * CS + tid + i * 64 * BP_CW] : mk(0.0, 0.0);
#pragma unroll
      for (int q = 0; q < CB; ++q)
#pragma unroll
        for (int i = 0; i < PE; ++i) v[i] = v[i] - pv[q][i];
    }
    for (; c < nch; ++c)
#pragma unroll
      for (int i = 0; i < PE; ++i)
        if (live[i]) v[i] = v[i] - part[c * CS + tid + i * 64 * BP_CW];
#pragma unroll
    for (int i = 0; i < PE; ++i) {
      const int e = tid + i * 64 * BP_CW;
      Ss[e / BP_B][e % BP_B] = v[i];
    }
    __syncthreads();
  }
  z64 col[BP_CR];
#pragma unroll
  for (int i = 0; i < BP_CR; ++i) col[i] = (r0 + i < nc && b < nc) ? Ss[r0 + i][b] : mk(0.0, 0.0);
  double d = b < nc ? Ss[b][b].x : 0.0;
  unsigned long long picked = 0;  // (the same in every lane)
  auto pick = [&]() -> int {      // largest unpicked diagonal, or -1
    unsigned key = 0;
    if (b < nc && !((picked >> b) & 1ull) && d > 0.0)
      key = ((unsigned)((unsigned long long)__double_as_longlong(d) >> 32) & ~63u) | (unsigned)(63 - b);
    key = wave_max_u32_uniform(key);
    return key ? 63 - (int)(key & 63u) : -1;
  };
  int p = pick();
  double dp = (p >= 0 && p < nc) ? readlane_f64(d, p) : 0.0;
  bool go = p >= 0 && p < nc && dp > thr2;
  int np = 0;
  for (int t = 0; t < BP_NP && go; ++t) {
    // rl = 1 / sqrt(dp): hardware estimate and two Newton steps
    double rl = __builtin_amdgcn_rsq(dp);
    rl = rl * (1.5 - 0.5 * dp * rl * rl);
    rl = rl * (1.5 - 0.5 * dp * rl * rl);
    const double lpp = dp * rl;
    // column t of the factor from row p of S (S is Hermitian), one entry per
    // lane of the wave that holds the row: one LDS write instead of twelve by
    // a single lane
    if (w == p / BP_CR) {
      z64 v = mk(0.0, 0.0);
      const int ip = __builtin_amdgcn_readfirstlane(p - r0);
      switch (ip) {
#define LSH_ROW(I) \
  case I:          \
    v = col[I];    \
    break;
        LSH_ROW(0) LSH_ROW(1) LSH_ROW(2) LSH_ROW(3) LSH_ROW(4) LSH_ROW(5) LSH_ROW(6) LSH_ROW(7) LSH_ROW(8)
        LSH_ROW(9) LSH_ROW(10) LSH_ROW(11)
#undef LSH_ROW
      }
      v = rl * conjg(v);
      const bool zero = (picked >> b) & 1ull;
      v.x = b == p ? lpp : (zero ? 0.0 : v.x);
      v.y = (b == p || zero) ? 0.0 : v.y;
      if (b < BP_B) Lb[t][b] = v;
      if (b == 0) {
        rlv[t] = rl;
        piv[t] = p;
      }
    }
    __syncthreads();
    const z64 clb = conjg(Lb[t][b < BP_B ? b : 0]);
    d -= abs2(clb);
    if (b == p) d = 0.0;
    picked |= 1ull << p;
    np = t + 1;
    // the next pivot (rows outside the block have Schur diagonal <= dout /
    // alpha, since diagonals only decrease: an accepted pivot is
    // alpha-greedy over all rows) and this pivot's row updates
    const int pn = pick();
#pragma unroll
    for (int i = 0; i < BP_CR; ++i) col[i] = col[i] - Lb[t][r0 + i] * clb;
    dp = (pn >= 0 && pn < nc) ? readlane_f64(d, pn) : 0.0;
    go = pn >= 0 && pn < nc && dp > thr2 && dp >= dout;
    p = pn;
  }
  __syncthreads();
  // X = L_PP^{-1}: wave w takes columns c = 8w + lane / 8; lane k = lane % 8
  // of a column holds rows r = k + 8i.  Step q: the owner of row q finishes
  // X[q][c] and passes it to the column's lanes, which subtract
  // L[r][q] X[q][c] from their later rows.
  {
    const int c = 8 * w + (b >> 3), k = b & 7;
    z64 acc[BP_NP / 8];
    int pr[BP_NP / 8];
#pragma unroll
    for (int i = 0; i < BP_NP / 8; ++i) {
      const int r = k + 8 * i;
      acc[i] = mk(r == c ? 1.0 : 0.0, 0.0);
      pr[i] = r < np ? piv[r] : 0;
    }
    for (int q = 0; q < np; ++q) {
      z64 xq = mk(0.0, 0.0);
#pragma unroll
      for (int i = 0; i < BP_NP / 8; ++i)
        if (i == (q >> 3)) xq = rlv[q] * acc[i];
      const int src = (b & ~7) | (q & 7);
      xq.x = __shfl(xq.x, src);
      xq.y = __shfl(xq.y, src);
      if (k == (q & 7)) xs[q][c] = xq;
#pragma unroll
      for (int i = 0; i < BP_NP / 8; ++i) {
        const int r = k + 8 * i;
        if (r > q && r < np) acc[i] = acc[i] - Lb[q][pr[i]] * xq;
      }
    }
  }
  __syncthreads();
  for (int e = tid; e < BP_NP * BP_NP; e += 64 * BP_CW) {
    const int q = e / BP_NP, r = e % BP_NP;
    const bool in = q < np && r <= q;
    Lpp[e] = in ? Lb[r][piv[q]] : mk(0.0, 0.0);
    Linv[e] = in ? xs[q][r] : mk(0.0, 0.0);
  }
  if (w == 0) {
    int bad = 0;
    if (b < np) {
      const int row = cand[piv[b]];
      bad = row < 0 || row >= m;  // (cannot happen: candidates are rows)
      J[j + b] = row;
    }
    bad = __any(bad);
    if (b == 0) {
      st[BPS_NP] = bad ? 0 : np;
      if (np == 0 || bad) st[BPS_DONE] = 1;
      if (bad) st[BPS_ERR] = 1;
    }
  }
}

// Wt partial sums over depth chunk c (BP_KC deep): part[c][q][i] =
// sum_{t in chunk, t < j} conj(L(P_q, t)) L(i, t) for q < np, as a product
// on the 16x16x4 FP64 matrix instruction: (pivots x depth) times (depth x
// rows).  The pivot rows' conjugated values for the chunk sit in LDS (real
// and imaginary planes); each wave owns 64 rows i and streams their factor
// entries from HBM (16 consecutive rows per instruction operand, the next
// four depths in flight).  Three real products per complex step (Gauss's
// form: t1 = ar br, t2 = ai bi, t3 = (ar + ai)(br + bi); Re = t1 - t2,
// Im = t3 - t1 - t2); the second pivot tile is skipped when np <= 16.  Rows
// already chosen are computed too (the new-columns kernel ignores them).
// rows per workgroup: four waves of 16 JT rows.  The MFMA work of a
// workgroup, not the memory, bounds a launch here (FP64 16x16x4 at 64 cycles
// a wave), and early steps have few depth chunks: small row blocks (JT = 1)
// keep every unit busy then.  (Two wavefronts per SIMD asked for: see k_cgemm;
// six matrix instructions stood beside 96 accumulator moves before.)
constexpr int BP_WT_JT = 1, BP_WT_ROWS = 64 * BP_WT_JT;
template <int BP_KC>
__global__ __launch_bounds__(256, 2) void k_bp_wt(const z64* Lt, const int* J, int m, const int* st, z64* part) {
  typedef double d4 __attribute__((ext_vector_type(4)));
  __shared__ double Apr[BP_NP][BP_KC + 1], Api[BP_NP][BP_KC + 1];
  if (st[BPS_DONE]) return;
  const int j = st[BPS_J], np = st[BPS_NP];
  const int c = blockIdx.y, t0 = c * BP_KC;
  if (t0 >= j) return;
  const int tn = (j - t0) < BP_KC ? (j - t0) : BP_KC;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int* Pq = J + j;
  for (int e = tid; e < BP_NP * BP_KC; e += 256) {
    const int q = e / BP_KC, t = e % BP_KC;
    const z64 v = (q < np && t < tn) ? Lt[(long)(t0 + t) * m + Pq[q]] : mk(0.0, 0.0);
    Apr[q][t] = v.x;
    Api[q][t] = -v.y;
  }
  __syncthreads();
  constexpr int JT = BP_WT_JT;
  const int i0 = blockIdx.x * BP_WT_ROWS + wave * 16 * JT, lr = lane & 15, lk = lane >> 4;
  const bool two = np > 16;
  d4 w1[2][JT], w2[2][JT], w3[2][JT];
#pragma unroll
  for (int qt = 0; qt < 2; ++qt)
#pragma unroll
    for (int jt = 0; jt < JT; ++jt) {
      w1[qt][jt] = d4{0.0, 0.0, 0.0, 0.0};
      w2[qt][jt] = d4{0.0, 0.0, 0.0, 0.0};
      w3[qt][jt] = d4{0.0, 0.0, 0.0, 0.0};
    }
  // B (the rows' factor entries) streams in stages of WT_DS depths: the next
  // stage's loads are issued before the current stage's MFMAs, so that a
  // stage of matrix work (WT_DS / 4 depth steps) covers the memory latency
  constexpr int WT_DS = 16, WT_SUB = WT_DS / 4;
  static_assert(BP_KC % WT_DS == 0, "stages tile the depth chunk");
  auto loadB = [&](int s0, double (&br)[WT_SUB][JT], double (&bi)[WT_SUB][JT]) {
#pragma unroll
    for (int u = 0; u < WT_SUB; ++u) {
      const int t = s0 + 4 * u + lk;
#pragma unroll
      for (int jt = 0; jt < JT; ++jt) {
        const int i = i0 + 16 * jt + lr;
        const z64 v = (t < tn && i < m) ? Lt[(long)(t0 + t) * m + i] : mk(0.0, 0.0);
        br[u][jt] = v.x;
        bi[u][jt] = v.y;
      }
    }
  };
  double br[WT_SUB][JT], bi[WT_SUB][JT];
  loadB(0, br, bi);
  for (int s0 = 0; s0 < tn; s0 += WT_DS) {
    double nbr[WT_SUB][JT], nbi[WT_SUB][JT];
    loadB(s0 + WT_DS, nbr, nbi);  // the next stage in flight meanwhile
#pragma unroll
    for (int u = 0; u < WT_SUB; ++u) {
      const int t = s0 + 4 * u + lk;  // (< BP_KC: s0 <= BP_KC - WT_DS, BP_KC % WT_DS == 0)
      double bs[JT];
#pragma unroll
      for (int jt = 0; jt < JT; ++jt) bs[jt] = br[u][jt] + bi[u][jt];
#pragma unroll
      for (int qt = 0; qt < 2; ++qt) {
        if (qt == 1 && !two) break;
        const double ar = Apr[16 * qt + lr][t], ai = Api[16 * qt + lr][t], as = ar + ai;
#pragma unroll
        for (int jt = 0; jt < JT; ++jt) {
          w1[qt][jt] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar, br[u][jt], w1[qt][jt], 0, 0, 0);
          w2[qt][jt] = __builtin_amdgcn_mfma_f64_16x16x4f64(ai, bi[u][jt], w2[qt][jt], 0, 0, 0);
          w3[qt][jt] = __builtin_amdgcn_mfma_f64_16x16x4f64(as, bs[jt], w3[qt][jt], 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < WT_SUB; ++u)
#pragma unroll
      for (int jt = 0; jt < JT; ++jt) {
        br[u][jt] = nbr[u][jt];
        bi[u][jt] = nbi[u][jt];
      }
  }
  // accumulator register r of lane l holds the pivot row lk + 4 r of its tile
  z64* pc = part + (long)c * BP_NP * m;
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
    if (qt == 1 && !two) break;
#pragma unroll
    for (int jt = 0; jt < JT; ++jt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int q = 16 * qt + lk + 4 * r, i = i0 + 16 * jt + lr;
        if (q < np && i < m) {
          const double t1 = w1[qt][jt][r], t2 = w2[qt][jt][r];
          pc[(long)q * m + i] = mk(t1 - t2, w3[qt][jt][r] - t1 - t2);
        }
      }
  }
}

// New factor rows Lt[j+q][i] = sum_q' conj(Linv[q][q']) W[q'][i] with
// W[q'][i] = conj(M[P_q'][i]) - sum_c part[c][q'][i]; then rows already
// chosen get exact zeros, the pivot rows get Lpp exactly, other rows have
// their Schur diagonal reduced, and the pivots are marked chosen.  A
// workgroup takes 32 rows i; thread (q, i) forms W[q][i] (its chunk sum
// spread over all threads), the products go through LDS.
constexpr int BP_NCR = 32;
static_assert(BP_NCR == BP_NP && BP_NCR * BP_NP == 1024, "one thread per (pivot, row) pair");
__global__ __launch_bounds__(1024) void k_bp_newcols(z64* Lt, const z64* M, int m, const int* J, const z64* part,
                                                     const z64* Lpp, const z64* Linv, int* chosen, double* d,
                                                     const int* st, int kc) {
  __shared__ z64 W[BP_NP][BP_NCR + 1];
  __shared__ z64 Li[BP_NP][BP_NP + 1];
  __shared__ double sd[BP_NP][BP_NCR + 1];
  if (st[BPS_DONE]) return;
  const int j = st[BPS_J], np = st[BPS_NP];
  const int nch = (j + kc - 1) / kc;
  const int tid = threadIdx.x, q = tid / BP_NCR, ii = tid % BP_NCR;
  const int i = blockIdx.x * BP_NCR + ii;
  const int* Pq = J + j;
  Li[q][ii] = conjg(Linv[q * BP_NP + ii]);  // (BP_NCR == BP_NP: one entry per thread)
  z64 w = mk(0.0, 0.0);
  if (i < m && q < np && !chosen[i]) {
    w = conjg(M[(long)Pq[q] * m + i]);
    int c = 0;
    for (; c + 4 <= nch; c += 4) {
      const z64 p0 = part[((long)(c + 0) * BP_NP + q) * m + i], p1 = part[((long)(c + 1) * BP_NP + q) * m + i];
      const z64 p2 = part[((long)(c + 2) * BP_NP + q) * m + i], p3 = part[((long)(c + 3) * BP_NP + q) * m + i];
      w = w - p0;
      w = w - p1;
      w = w - p2;
      w = w - p3;
    }
    for (; c < nch; ++c) w = w - part[((long)c * BP_NP + q) * m + i];
  }
  W[q][ii] = w;
  __syncthreads();
  const bool live = i < m;
  int q0 = -1;
  for (int r = 0; r < np; ++r)
    if (live && Pq[r] == i) q0 = r;
  const bool was_chosen = live && chosen[i] != 0;
  z64 v = mk(0.0, 0.0);
  if (live && q < np) {
    if (q0 >= 0) v = Lpp[q0 * BP_NP + q];
    else if (!was_chosen)
      for (int r = 0; r <= q; ++r) v = v + Li[q][r] * W[r][ii];
    Lt[(long)(j + q) * m + i] = v;
  }
  sd[q][ii] = abs2(v);
  __syncthreads();
  if (live && q == 0) {
    if (q0 >= 0) {
      chosen[i] = 1;
      d[i] = 0.0;
    } else if (!was_chosen) {
      double t = 0.0;
      for (int r = 0; r < np; ++r) t += sd[r][ii];
      d[i] -= t;
    }
  }
}

// depth of k_bp_wt's chunks: 64 up to 1536 candidates, where 128 would leave
// units idle (at depth 700 of 750 candidates: 22 us a step with 128, 14 with
// 64), 128 beyond, where the partial sums' bytes count (n = 1024: 98.5 ms a setup
// with this line at 1536, 99.8 with 128 everywhere, 100 with 64 everywhere)
constexpr int BP_SHALLOW = 1536;
static int bp_kc(int m) { return m <= BP_SHALLOW ? 64 : 128; }

// Enough for every row ID of at most m rows: a plan's memory is sized from
// bounds on m, and BP_SHALLOW rows have more partial sums than a few more.
size_t rowid_bp_ws(int m) {
  const size_t mm = (size_t)m * m, mp = (size_t)m + BP_KCMAX;
  auto wt = [](int r) { return ((size_t)(r + BP_KCMAX) / bp_kc(r) + 1) * BP_NP * r; };
  const size_t partw = m > BP_SHALLOW ? std::max(wt(m), wt(BP_SHALLOW)) : wt(m);
  return sizeof(z64) * (mm + mp * m + 2 * mm) + sizeof(double) * m + sizeof(int) * (3 * m + BPS_WORDS) +
         sizeof(z64) * (BP_B * BP_B + 2 * BP_NP * BP_NP + (mp / BP_KCS + 1) * BP_B * BP_B + partw) +
         inverse_ws_bytes<double>(64, m / 64 + 1) + sizeof(z64) * (size_t)(m / 64 + 1) * 64 * 64 + 32 * 256;
}

static int grid_of(long n) {
  const long g = (n + 255) / 256;
  return (int)(g < 2048 ? (g > 0 ? g : 1) : 2048);
}

// Linv[q] (diagonal block q of the k x k array, row-major, leading dimension
// k) = D[q] for the nb inverted 64 x 64 blocks (the last one cut at k)
__global__ void k_place_diag(const z64* D, int k, z64* Linv) {
  const int q = blockIdx.y, base = q * TRI_B;
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < TRI_B * TRI_B; e += gridDim.x * blockDim.x) {
    const int r = e / TRI_B, c = e % TRI_B;
    if (base + r < k && base + c < k) Linv[(long)(base + r) * k + base + c] = D[(long)q * TRI_B * TRI_B + e];
  }
}

// U = L(rest, 0:k) L11^{-1} with U(J) = I, from the column-major factor Lt
// (shared by both Gram paths).  L11^{-1} is formed explicitly from the
// inverted 64 x 64 diagonal blocks by doubling (inv [[A, 0], [B, C]] =
// [[A^-1, 0], [-C^-1 B A^-1, C^-1]], all pairs of one size in two batched
// products), then U(rest) = L(rest) L11^{-1} is one product: a dozen wide
// launches instead of a block-by-block substitution chain.  Linv (k x k) and
// the pairs' temporaries T (at most k^2 / 4 entries) are scratch.
// Jh: the skeleton on the host; rh receives the other rows (the upload's
// source: it has to stay until the work on s is done).
static void gram_interp(hipStream_t s, const z64* Lt, int m, int k, const int* Jh, std::vector<int>& rh, int* J,
                        z64* U, int* rest, z64* L11, z64* Lr, z64* Dinv, z64* Linv, z64* T) {
  const int DB = 64;
  {
    std::vector<char> used(m, 0);
    for (int q = 0; q < k; ++q) used[Jh[q]] = 1;
    rh.clear();
    for (int i = 0; i < m; ++i)
      if (!used[i]) rh.push_back(i);
  }
  const int nr = (int)rh.size();
  if (nr) LSH_HIP(hipMemcpyAsync(rest, rh.data(), sizeof(int) * nr, hipMemcpyHostToDevice, s));
  hipLaunchKernelGGL(k_gather_L11, dim3(ceil_div((long)k * k, 256)), dim3(256), 0, s, Lt, m, J, k, L11);
  LSH_LAUNCH_CHECK();
  if (nr) {
    hipLaunchKernelGGL(k_gather_rows, dim3(ceil_div((long)nr * k, 256)), dim3(256), 0, s, Lt, m, rest, nr, k, Lr);
    LSH_LAUNCH_CHECK();
    const int nblk = ceil_div(k, DB);
    static_assert(DB == TRI_B, "diagonal block size");
    hipLaunchKernelGGL(k_trinv_blocks, dim3(nblk), dim3(256), 0, s, L11, k, Dinv);
    LSH_LAUNCH_CHECK();
    fill_zero(s, Linv, sizeof(z64) * (size_t)k * k);
    hipLaunchKernelGGL(k_place_diag, dim3(16, nblk), dim3(256), 0, s, Dinv, k, Linv);
    LSH_LAUNCH_CHECK();
    const z64 one = mk(1.0, 0.0), mone = mk(-1.0, 0.0), zero = mk(0.0, 0.0);
    for (int b = DB; b < k; b *= 2) {
      // pairs (A at rows i0 .. i0+b, C at i0+b .. min(i0+2b, k)), i0 = p 2b
      const int full = k / (2 * b);                  // pairs with a whole C block
      const long st = 2L * b * (k + 1);              // stride between pairs' diagonal positions
      if (full > 0) {
        // T_p = B_p A_p^{-1}, then Linv(C rows, A cols) = -C_p^{-1} T_p
        cgemm<double>(s, b, b, b, one, L11 + (long)b * k, k, st, OP_N, Linv, k, st, OP_N, zero, nullptr, 0, 0, T,
                      b, (long)b * b, full);
        cgemm<double>(s, b, b, b, mone, Linv + (long)b * (k + 1), k, st, OP_N, T, b, (long)b * b, OP_N, zero,
                      nullptr, 0, 0, Linv + (long)b * k, k, st, full);
      }
      const int i0 = full * 2 * b, c2 = k - i0 - b;  // a last pair with a partial C block
      if (c2 > 0) {
        cgemm<double>(s, c2, b, b, one, L11 + (long)(i0 + b) * k + i0, k, 0, OP_N, Linv + (long)i0 * (k + 1), k, 0,
                      OP_N, zero, nullptr, 0, 0, T, b, 0, 1);
        cgemm<double>(s, c2, b, c2, mone, Linv + (long)(i0 + b) * (k + 1), k, 0, OP_N, T, b, 0, OP_N, zero,
                      nullptr, 0, 0, Linv + (long)(i0 + b) * k + i0, k, 0, 1);
      }
    }
    z64* X = L11 + (size_t)k * k;  // (nr x k) after L11 in the same buffer
    cgemm<double>(s, nr, k, k, one, Lr, k, 0, OP_N, Linv, k, 0, OP_N, zero, nullptr, 0, 0, X, k, 0, 1);
    hipLaunchKernelGGL(k_scatter_U, dim3(ceil_div((long)(k + nr) * k, 256)), dim3(256), 0, s, U, k, J, rest, nr, X);
  } else {
    hipLaunchKernelGGL(k_scatter_U, dim3(ceil_div((long)k * k, 256)), dim3(256), 0, s, U, k, J, rest, 0, L11);
  }
  LSH_LAUNCH_CHECK();
}

int rowid_bp(hipStream_t s, const z64* A, int m, int np, double tol, double alpha, int* J, z64* U, void* ws,
             bool gram_ready, NextGram* next, const std::function<void(int)>& on_skel, BpInterp* later) {
  LSH_REQUIRE(alpha > 0.0 && alpha <= 1.0, -1, "row ID: alpha must lie in (0, 1]");
  LSH_REQUIRE(m <= BP_SEL, -6, "row ID: more than 16384 candidate rows in one level");
  char* p = static_cast<char*>(ws);
  auto take = [&](size_t bytes) { char* r = p; p += ((bytes + 255) / 256) * 256; return (void*)r; };
  const size_t mp = (size_t)m + BP_KCMAX;
  const int kc = bp_kc(m), nch = (int)(mp / kc) + 1, nchS = (int)(mp / BP_KCS) + 1;
  z64* M = static_cast<z64*>(take(sizeof(z64) * (size_t)m * m));
  z64* Lt = static_cast<z64*>(take(sizeof(z64) * mp * m));
  z64* L11 = static_cast<z64*>(take(sizeof(z64) * (size_t)m * m));
  z64* Lr = static_cast<z64*>(take(sizeof(z64) * (size_t)m * m));
  double* d = static_cast<double*>(take(sizeof(double) * m));
  int* chosen = static_cast<int*>(take(sizeof(int) * m));
  int* rest = static_cast<int*>(take(sizeof(int) * m));
  int* st = static_cast<int*>(take(sizeof(int) * BPS_WORDS));
  z64* Lpp = static_cast<z64*>(take(sizeof(z64) * BP_NP * BP_NP));
  z64* Linv = static_cast<z64*>(take(sizeof(z64) * BP_NP * BP_NP));
  z64* partS = static_cast<z64*>(take(sizeof(z64) * (size_t)nchS * BP_B * BP_B));
  z64* partW = static_cast<z64*>(take(sizeof(z64) * (size_t)nch * BP_NP * m));
  const int DB = 64;
  z64* Dinv = static_cast<z64*>(take(sizeof(z64) * (size_t)(m / DB + 1) * DB * DB));
  void* invws = take(inverse_ws_bytes<double>(DB, m / DB + 1));
  // Gram matrix and its diagonal; the factor starts at zero
  if (!gram_ready) {
    cgemm<double>(s, m, m, np, mk(1.0, 0.0), A, np, 0, OP_N, A, np, 0, OP_C, mk(0.0, 0.0), nullptr, 0, 0, M, m, 0,
                  1, false, nullptr, true);  // Hermitian: lower tiles, then the mirror
    mirror_lower<double>(s, M, m, m);
  }
  fill_zero(s, Lt, sizeof(z64) * mp * m);
  fill_zero(s, st, sizeof(int) * BPS_WORDS);
  hipLaunchKernelGGL(k_gram_init, dim3(ceil_div(m, 256)), dim3(256), 0, s, M, m, d, chosen, st + BPS_WORDS - 4);
  LSH_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_bp_thr2, dim3(1), dim3(1024), 0, s, d, m, tol * tol, st);
  LSH_LAUNCH_CHECK();
  const int gm = ceil_div(m, 256);
  // steps in batches of four, then eight: a batch costs one read-back (about
  // 20 us with the queue empty), a step queued after the end about 10 us, and
  // the parent's Gram rows start after each batch (n = 1024: 100.3 ms a setup
  // with batches up to 8, 103.2 with 16 and, without a parent, 32)
  int batch = 4, host_st[4] = {0, 0, 0, 0};
  constexpr int max_batch = 8;
  while (true) {
    for (int b = 0; b < batch; ++b) {
      {
        ProfScope ps("bp_select", s, 16.0 * m);
        if (m <= 4096) hipLaunchKernelGGL(k_bp_select<4>, dim3(1), dim3(1024), 0, s, d, chosen, m, st);
        else if (m <= 8192) hipLaunchKernelGGL(k_bp_select<8>, dim3(1), dim3(1024), 0, s, d, chosen, m, st);
        else hipLaunchKernelGGL(k_bp_select<BP_SEL / 1024>, dim3(1), dim3(1024), 0, s, d, chosen, m, st);
      }
      LSH_LAUNCH_CHECK();
      hipLaunchKernelGGL(k_bp_sc, dim3(nchS, 4), dim3(256), 0, s, Lt, m, st, partS);
      LSH_LAUNCH_CHECK();
      {
        ProfScope ps("bp_chol", s, 16.0 * BP_B * BP_B);
        hipLaunchKernelGGL(k_bp_chol, dim3(1), dim3(64 * BP_CW), 0, s, M, partS, m, alpha, J, st, Lpp, Linv);
      }
      LSH_LAUNCH_CHECK();
      {
        ProfScope ps("bp_wt", s, 16.0 * m * m);
        hipLaunchKernelGGL(kc == 64 ? k_bp_wt<64> : k_bp_wt<128>, dim3(ceil_div(m, BP_WT_ROWS), nch), dim3(256), 0, s,
                           Lt, J, m, st, partW);
      }
      LSH_LAUNCH_CHECK();
      hipLaunchKernelGGL(k_bp_newcols, dim3(ceil_div(m, BP_NCR)), dim3(1024), 0, s, Lt, M, m, J, partW, Lpp, Linv,
                         chosen, d, st, kc);
      LSH_LAUNCH_CHECK();
    }
    LSH_HIP(hipMemcpyAsync(host_st, st, sizeof(int) * 4, hipMemcpyDeviceToHost, s));
    LSH_HIP(hipStreamSynchronize(s));
    if (host_st[BPS_DONE]) break;
    if (next) next_gram_rows(*next, J, host_st[BPS_J] + host_st[BPS_NP]);
    batch = batch < max_batch ? batch * 2 : max_batch;
  }
  int j = 0;
  {
    int hs[8];
    LSH_HIP(hipMemcpyAsync(hs, st, sizeof(int) * 8, hipMemcpyDeviceToHost, s));
    LSH_HIP(hipStreamSynchronize(s));
    LSH_REQUIRE(hs[BPS_ERR] == 0, -4, "row ID: pivot row out of range");
    j = hs[BPS_J] + hs[BPS_NP];  // (pivots of a step not yet advanced)
  }
  if (j < 1) {  // a zero block still gets one skeleton: row 0, U = e_0
    const int zero = 0;
    const z64 one = mk(1.0, 0.0);
    LSH_HIP(hipMemcpyAsync(J, &zero, sizeof(int), hipMemcpyHostToDevice, s));
    fill_zero(s, U, sizeof(z64) * (size_t)m);
    LSH_HIP(hipMemcpyAsync(U, &one, sizeof(z64), hipMemcpyHostToDevice, s));
    LSH_HIP(hipStreamSynchronize(s));
    if (next) next_gram_rows(*next, J, 1);
    if (on_skel) on_skel(1);
    if (later) later->m = 0;  // (U is complete)
    return 1;
  }
  if (next) next_gram_rows(*next, J, j);  // (J is final: the stream was synchronised)
  if (on_skel) on_skel(j);                // (before the interpolation matrix)
  // (the Gram is no longer needed: it holds L11^{-1}; the pairs' temporaries
  // follow the rest rows in Lr)
  const BpInterp I{Lt, m, j, J, rest, L11, Lr, Dinv, M, Lr + (size_t)(m - j) * j};
  (void)invws;
  if (later) {
    *later = I;
    return j;
  }
  std::vector<int> ph(j), rh;
  LSH_HIP(hipMemcpyAsync(ph.data(), J, sizeof(int) * j, hipMemcpyDeviceToHost, s));
  LSH_HIP(hipStreamSynchronize(s));
  bp_interp(s, I, ph.data(), rh, U);
  LSH_HIP(hipStreamSynchronize(s));
  return j;
}

void bp_interp(hipStream_t s, const BpInterp& I, const int* Jh, std::vector<int>& rh, z64* U) {
  gram_interp(s, I.Lt, I.m, I.k, Jh, rh, I.J, U, I.rest, I.L11, I.Lr, I.Dinv, I.Linv, I.T);
}

size_t rowid_gram_ws(int m) {
  const size_t mm = (size_t)m * m;
  return sizeof(z64) * mm * 4 + sizeof(double) * m + sizeof(int) * (3 * m + 16) +
         inverse_ws_bytes<double>(64, m / 64 + 1) + sizeof(z64) * (size_t)(m / 64 + 1) * 64 * 64 +
         (sizeof(double) + sizeof(int)) * 512 + 16384;
}

int rowid_gram(hipStream_t s, const z64* A, int m, int np, double tol, int* J, z64* U, void* ws) {
  LSH_REQUIRE(m <= PCH_MAXM, -6, "row ID: more than 4096 candidate rows in one level");
  char* p = static_cast<char*>(ws);
  auto take = [&](size_t bytes) { char* r = p; p += ((bytes + 255) / 256) * 256; return (void*)r; };
  z64* M = static_cast<z64*>(take(sizeof(z64) * (size_t)m * m));
  z64* Lt = static_cast<z64*>(take(sizeof(z64) * (size_t)m * m));
  z64* L11 = static_cast<z64*>(take(sizeof(z64) * (size_t)m * m));
  z64* Lr = static_cast<z64*>(take(sizeof(z64) * (size_t)m * m));
  double* d = static_cast<double*>(take(sizeof(double) * m));
  int* chosen = static_cast<int*>(take(sizeof(int) * m));
  int* rest = static_cast<int*>(take(sizeof(int) * m));
  int* state = static_cast<int*>(take(sizeof(int) * 16));
  const int DB = 64;
  z64* Dinv = static_cast<z64*>(take(sizeof(z64) * (size_t)(m / DB + 1) * DB * DB));
  void* invws = take(inverse_ws_bytes<double>(DB, m / DB + 1));
  cgemm<double>(s, m, m, np, mk(1.0, 0.0), A, np, 0, OP_N, A, np, 0, OP_C, mk(0.0, 0.0), nullptr, 0, 0, M, m, 0, 1,
                false, nullptr, true);  // Hermitian: lower tiles, then the mirror
  mirror_lower<double>(s, M, m, m);
  hipLaunchKernelGGL(k_gram_init, dim3(ceil_div(m, 256)), dim3(256), 0, s, M, m, d, chosen, state);
  LSH_LAUNCH_CHECK();
  // ||A||_F^2 = trace(M)
  std::vector<double> dh(m);
  LSH_HIP(hipMemcpyAsync(dh.data(), d, sizeof(double) * m, hipMemcpyDeviceToHost, s));
  LSH_HIP(hipStreamSynchronize(s));
  double fro2 = 0;
  for (double v : dh) fro2 += v;
  const double thr2 = tol * tol * fro2;
  static const int nb = [] {
    const char* e = std::getenv("LSH_PCHOL_NB");
    int v = e ? std::atoi(e) : 16;
    return (v >= 4 && v <= PCH_NB) ? v : 16;
  }();
  int rank = 0;
  // One workgroup per panel: the per-pivot cost is one workgroup's L2
  // stream of the panel, ~m * nb / 2 entries.  All panels and trailing updates are queued at once: each panel kernel
  // returns at entry once state[1] (done) is set, and each update is skipped
  // through the same flag, so the host reads the rank once per level.
  for (int j0 = 0; j0 < m; j0 += nb) {
    {
      ProfScope ps("pchol_panel", s, 16.0 * (double)m * nb);
      hipLaunchKernelGGL(k_pchol_panel, dim3(1), dim3(QR_NT), (size_t)m * (sizeof(double) + 1), s, M, m, d, chosen,
                         Lt, J, j0, nb, thr2, state);
    }
    LSH_LAUNCH_CHECK();
    if (j0 + nb < m)  // trailing update of the Schur complement: M -= Lp Lp^H
      cgemm<double>(s, m, m, nb, mk(-1.0, 0.0), Lt + (long)j0 * m, m, 0, OP_T, Lt + (long)j0 * m, m, 0, OP_R,
                    mk(1.0, 0.0), M, m, 0, M, m, 0, 1, false, state + 1);
  }
  {
    int st[2];
    LSH_HIP(hipMemcpyAsync(st, state, sizeof(int) * 2, hipMemcpyDeviceToHost, s));
    LSH_HIP(hipStreamSynchronize(s));
    rank = st[0];
  }
  const int k = rank < 1 ? 1 : rank;
  std::vector<int> ph(k), rh;
  LSH_HIP(hipMemcpyAsync(ph.data(), J, sizeof(int) * k, hipMemcpyDeviceToHost, s));
  LSH_HIP(hipStreamSynchronize(s));
  gram_interp(s, Lt, m, k, ph.data(), rh, J, U, rest, L11, Lr, Dinv, M, Lr + (size_t)(m - k) * k);
  LSH_HIP(hipStreamSynchronize(s));
  (void)invws;
  return k;
}

// ------------------------------------------------------------- leaf factor
template <typename R>
__global__ void k_leaf_build(cplx<R>* X, const cplx<R>* __restrict__ G, int mL, const double* __restrict__ b,
                             double kappa2, const I2* __restrict__ org, const I2* __restrict__ pts, int n) {
  const long t = blockIdx.y;
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= mL * mL) return;
  const int i = e / mL, j = e % mL;
  const I2 o = org[t], pi = pts[i];
  const double bi = kappa2 * b[(long)(o.y + pi.y) * n + (o.x + pi.x)];
  cplx<R> v = (R)bi * G[e];
  if (i == j) v.x += R(1);
  X[t * (long)mL * mL + e] = v;
}

template <typename R>
void leaf_build(hipStream_t s, cplx<R>* X, const cplx<R>* Gleaf, int mL, const double* b, double kappa2,
                const I2* leaf_origin, const I2* leaf_pts, int nleaf, int n) {
  LSH_REQUIRE(nleaf <= 65535 * 64, -6, "too many leaves");
  for (int t0 = 0; t0 < nleaf; t0 += 65535) {
    int nt = nleaf - t0 < 65535 ? nleaf - t0 : 65535;
    hipLaunchKernelGGL(k_leaf_build<R>, dim3(ceil_div(mL * mL, 256), nt), dim3(256), 0, s,
                       X + (long)t0 * mL * mL, Gleaf, mL, b, kappa2, leaf_origin + t0, leaf_pts, n);
    LSH_LAUNCH_CHECK();
  }
}

template <typename R>
__global__ void k_leaf_scale_U(cplx<R>* Y, const cplx<R>* __restrict__ U, int mL, int k,
                               const double* __restrict__ b, double kappa2, const I2* __restrict__ org,
                               const I2* __restrict__ pts, int n) {
  const long t = blockIdx.y;
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= mL * k) return;
  const int i = e / k;
  const I2 o = org[t], pi = pts[i];
  const double bi = kappa2 * b[(long)(o.y + pi.y) * n + (o.x + pi.x)];
  Y[t * (long)mL * k + e] = (R)bi * U[e];
}

template <typename R>
void leaf_scale_U(hipStream_t s, cplx<R>* Y, const cplx<R>* U, int mL, int k, const double* b, double kappa2,
                  const I2* leaf_origin, const I2* leaf_pts, int nleaf, int n) {
  for (int t0 = 0; t0 < nleaf; t0 += 65535) {
    int nt = nleaf - t0 < 65535 ? nleaf - t0 : 65535;
    hipLaunchKernelGGL(k_leaf_scale_U<R>, dim3(ceil_div(mL * k, 256), nt), dim3(256), 0, s,
                       Y + (long)t0 * mL * k, U, mL, k, b, kappa2, leaf_origin + t0, leaf_pts, n);
    LSH_LAUNCH_CHECK();
  }
}

// -------------------------------------------------------------- leaf apply
// One workgroup per leaf and group of up to NV right-hand sides: the leaf's
// X_tau and U_L are read once for the group. Each right-hand side gets the
// same arithmetic, in the same order, as in a one-vector launch.
constexpr int LEAF_MAX = 144;
constexpr int LEAF_NV = 4;

// Rows i < nrows of the row-major matrix A (nrows x ncols) times NV vectors
// in LDS (ins[v][0 .. ncols)); fn(i, v, sum) once per row and vector v < nv.
// Rows of at most 64 (the leaf matrices and U_L of leaves up to 8 x 8): 16
// lanes per row in four 16-wide chunks, four rows per wave at a time and
// four such row groups per wave with every load issued before the products
// (16 loads in flight per lane); a lane adds its chunks as (s0 + s1) +
// (s2 + s3), then a DPP butterfly over the row's 16 lanes.  Longer rows: one
// wave per row, LEAF_RU rows at a time, butterfly over the wave.  Each vector
// gets the same arithmetic in the same order for any NV.
constexpr int LEAF_RU = 4;
template <typename R, int NV, typename Fn>
__device__ __forceinline__ void leaf_rows(const cplx<R>* __restrict__ A, int nrows, int ncols,
                                          const cplx<R> (*ins)[LEAF_MAX], int nv, Fn fn) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (ncols <= 64) {
    constexpr int L = 16, NCH = 4, RW = 64 / L, P = 4;
    const int sub = lane & (L - 1), rs = lane / L;
    for (int base = wave * RW; base < nrows; base += 4 * RW * P) {
      cplx<R> a[P][NCH];
#pragma unroll
      for (int p = 0; p < P; ++p) {
        const int i = base + p * 4 * RW + rs;
#pragma unroll
        for (int u = 0; u < NCH; ++u) {
          const int c = sub + u * L;
          a[p][u] = (i < nrows && c < ncols) ? A[(long)i * ncols + c] : mk<R>(0, 0);
        }
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        if (v >= nv) break;  // (uniform)
        cplx<R> xin[NCH];
#pragma unroll
        for (int u = 0; u < NCH; ++u) {
          const int c = sub + u * L;
          xin[u] = c < ncols ? ins[v][c] : mk<R>(0, 0);
        }
#pragma unroll
        for (int p = 0; p < P; ++p) {
          cplx<R> a4[NCH];
#pragma unroll
          for (int u = 0; u < NCH; ++u) {
            a4[u] = mk<R>(0, 0);
            fma_acc(a4[u], a[p][u], xin[u]);
          }
          cplx<R> t = (a4[0] + a4[1]) + (a4[2] + a4[3]);
          t.x = group_sum<L>(t.x);
          t.y = group_sum<L>(t.y);
          const int i = base + p * 4 * RW + rs;
          if (sub == 0 && i < nrows) fn(i, v, t);
        }
      }
    }
    return;
  }
  for (int i0 = wave; i0 < nrows; i0 += 4 * LEAF_RU) {
    cplx<R> acc[LEAF_RU][NV];
#pragma unroll
    for (int u = 0; u < LEAF_RU; ++u)
#pragma unroll
      for (int v = 0; v < NV; ++v) acc[u][v] = mk<R>(0, 0);
    for (int j = lane; j < ncols; j += 64) {
      cplx<R> xv[LEAF_RU];
#pragma unroll
      for (int u = 0; u < LEAF_RU; ++u) {
        const int i = i0 + 4 * u;
        xv[u] = i < nrows ? A[(long)i * ncols + j] : mk<R>(0, 0);
      }
#pragma unroll
      for (int u = 0; u < LEAF_RU; ++u)
#pragma unroll
        for (int v = 0; v < NV; ++v) fma_acc(acc[u][v], xv[u], ins[v][j]);
    }
#pragma unroll
    for (int u = 0; u < LEAF_RU; ++u) {
      const int i = i0 + 4 * u;
      if (i >= nrows) break;  // (uniform across the wave)
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        if (v >= nv) break;
        cplx<R> a = acc[u][v];
        a.x = group_sum<64>(a.x);
        a.y = group_sum<64>(a.y);
        if (lane == 0) fn(i, v, a);
      }
    }
  }
}

// Up: r = X_tau f_tau ; rt = U_L^T r  (ULt: U_L transposed, k x mL)
template <typename R, int NV>
__global__ __launch_bounds__(256) void k_leaf_up(const cplx<R>* __restrict__ X, const cplx<R>* __restrict__ ULt,
                                                 int mL, int k, const z64* __restrict__ f, cplx<R>* r, cplx<R>* rt,
                                                 const I2* __restrict__ org, const I2* __restrict__ pts, int n,
                                                 int nleaf, int nrhs, const double* __restrict__ b, double sb) {
  __shared__ cplx<R> fs[NV][LEAF_MAX];
  __shared__ cplx<R> rs[NV][LEAF_MAX];
  const long t = blockIdx.x, r0 = (long)blockIdx.y * NV;
  const int nv = nrhs - r0 < NV ? (int)(nrhs - r0) : NV;
  const I2 o = org[t];
  for (int i = threadIdx.x; i < mL; i += blockDim.x) {
    const I2 pi = pts[i];
    const long at = (long)(o.y + pi.y) * n + (o.x + pi.x);
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      z64 val = mk(0.0, 0.0);
      if (v < nv) val = f[(r0 + v) * (long)n * n + at];
      fs[v][i] = mk<R>((R)val.x, (R)val.y);
    }
  }
  __syncthreads();
  leaf_rows<R, NV>(X + t * (long)mL * mL, mL, mL, fs, nv, [&](int i, int v, cplx<R> acc) { rs[v][i] = acc; });
  __syncthreads();
  for (int v = 0; v < nv; ++v) {
    if (r) {
      cplx<R>* rr = r + ((r0 + v) * nleaf + t) * (long)mL;
      for (int i = threadIdx.x; i < mL; i += blockDim.x) rr[i] = rs[v][i];
    }
    if (b) {  // transpose pass: rs <- sb * b .* rs before U_L^T
      for (int i = threadIdx.x; i < mL; i += blockDim.x) {
        const I2 pi = pts[i];
        rs[v][i] = (R)(sb * b[(long)(o.y + pi.y) * n + (o.x + pi.x)]) * rs[v][i];
      }
    }
  }
  if (b) __syncthreads();
  leaf_rows<R, NV>(ULt, k, mL, rs, nv,
                   [&](int a, int v, cplx<R> acc) { rt[((r0 + v) * nleaf + t) * (long)k + a] = acc; });
}

template <typename R>
void leaf_up(hipStream_t s, const cplx<R>* X, const cplx<R>* ULt, int mL, int k, const z64* f, cplx<R>* r,
             cplx<R>* rt, const I2* leaf_origin, const I2* leaf_pts, int nleaf, int n, int nrhs, const double* b,
             double sb) {
  LSH_REQUIRE(mL <= LEAF_MAX, -6, "leaf too large");
  const int ng = nrhs == 1 ? 1 : ceil_div(nrhs, LEAF_NV);
  ProfScope ps("leaf_up", s, (double)sizeof(cplx<R>) * nleaf * ((double)ng * mL * mL + (double)nrhs * (2.0 * mL + k)) +
                                 16.0 * nrhs * (double)nleaf * mL);
  if (nrhs == 1)
    hipLaunchKernelGGL((k_leaf_up<R, 1>), dim3(nleaf, 1), dim3(256), 0, s, X, ULt, mL, k, f, r, rt, leaf_origin,
                       leaf_pts, n, nleaf, nrhs, b, sb);
  else
    hipLaunchKernelGGL((k_leaf_up<R, LEAF_NV>), dim3(nleaf, ng), dim3(256), 0, s, X, ULt, mL, k, f, r, rt,
                       leaf_origin, leaf_pts, n, nleaf, nrhs, b, sb);
  LSH_LAUNCH_CHECK();
}

// Down: q_tau = r_tau - X_tau B_tau U_L wt_tau, written to the grid (FP64)
template <typename R, int NV>
__global__ __launch_bounds__(256) void k_leaf_down(const cplx<R>* __restrict__ X, const cplx<R>* __restrict__ UL,
                                                   int mL, int k, const cplx<R>* __restrict__ wt,
                                                   const cplx<R>* __restrict__ r, z64* q,
                                                   const double* __restrict__ b, double kappa2,
                                                   const I2* __restrict__ org, const I2* __restrict__ pts, int n,
                                                   int nleaf, int nrhs) {
  __shared__ cplx<R> us[NV][LEAF_MAX];
  __shared__ cplx<R> ws[NV][LEAF_MAX];
  __shared__ cplx<R> rl[NV][LEAF_MAX];  // r, then the result (stored to the grid together at the end)
  const long t = blockIdx.x, r0 = (long)blockIdx.y * NV;
  const int nv = nrhs - r0 < NV ? (int)(nrhs - r0) : NV;
  const I2 o = org[t];
  for (int a = threadIdx.x; a < k; a += blockDim.x)
#pragma unroll
    for (int v = 0; v < NV; ++v) ws[v][a] = v < nv ? wt[((r0 + v) * nleaf + t) * (long)k + a] : mk<R>(0, 0);
  for (int v = 0; v < nv; ++v)
    for (int i = threadIdx.x; i < mL; i += blockDim.x) rl[v][i] = r[((r0 + v) * nleaf + t) * (long)mL + i];
  __syncthreads();
  leaf_rows<R, NV>(UL, mL, k, ws, nv, [&](int i, int v, cplx<R> acc) {
    const I2 pi = pts[i];
    us[v][i] = (R)(kappa2 * b[(long)(o.y + pi.y) * n + (o.x + pi.x)]) * acc;
  });
  __syncthreads();
  leaf_rows<R, NV>(X + t * (long)mL * mL, mL, mL, us, nv,
                   [&](int i, int v, cplx<R> acc) { rl[v][i] = rl[v][i] - acc; });
  __syncthreads();
  for (int v = 0; v < nv; ++v)
    for (int i = threadIdx.x; i < mL; i += blockDim.x) {
      const I2 pi = pts[i];
      const cplx<R> val = rl[v][i];
      q[(r0 + v) * (long)n * n + (long)(o.y + pi.y) * n + (o.x + pi.x)] = mk((double)val.x, (double)val.y);
    }
}

template <typename R>
void leaf_down(hipStream_t s, const cplx<R>* X, const cplx<R>* UL, int mL, int k, const cplx<R>* wt,
               const cplx<R>* r, z64* q, const double* b, double kappa2, const I2* leaf_origin, const I2* leaf_pts,
               int nleaf, int n, int nrhs) {
  LSH_REQUIRE(mL <= LEAF_MAX, -6, "leaf too large");
  const int ng = nrhs == 1 ? 1 : ceil_div(nrhs, LEAF_NV);
  ProfScope ps("leaf_down", s, (double)sizeof(cplx<R>) * nleaf * ((double)ng * mL * mL + (double)nrhs * (mL + k)) +
                                   (16.0 + 8.0) * nrhs * (double)nleaf * mL);
  if (nrhs == 1)
    hipLaunchKernelGGL((k_leaf_down<R, 1>), dim3(nleaf, 1), dim3(256), 0, s, X, UL, mL, k, wt, r, q, b, kappa2,
                       leaf_origin, leaf_pts, n, nleaf, nrhs);
  else
    hipLaunchKernelGGL((k_leaf_down<R, LEAF_NV>), dim3(nleaf, ng), dim3(256), 0, s, X, UL, mL, k, wt, r, q, b,
                       kappa2, leaf_origin, leaf_pts, n, nleaf, nrhs);
  LSH_LAUNCH_CHECK();
}

// Transpose pass, leaves: q_tau = X_tau^T (g_tau + U_L rb_tau) (X given transposed)
template <typename R, int NV>
__global__ __launch_bounds__(256) void k_leaf_tdown(const cplx<R>* __restrict__ XT, const cplx<R>* __restrict__ UL,
                                                    int mL, int k, const cplx<R>* __restrict__ w,
                                                    const z64* __restrict__ g, z64* q, const I2* __restrict__ org,
                                                    const I2* __restrict__ pts, int n, int nleaf, int nrhs) {
  __shared__ cplx<R> us[NV][LEAF_MAX];
  __shared__ cplx<R> ws[NV][LEAF_MAX];
  const long t = blockIdx.x, r0 = (long)blockIdx.y * NV;
  const int nv = nrhs - r0 < NV ? (int)(nrhs - r0) : NV;
  const I2 o = org[t];
  for (int a = threadIdx.x; a < k; a += blockDim.x)
#pragma unroll
    for (int v = 0; v < NV; ++v) ws[v][a] = v < nv ? w[((r0 + v) * nleaf + t) * (long)k + a] : mk<R>(0, 0);
  __syncthreads();
  leaf_rows<R, NV>(UL, mL, k, ws, nv, [&](int i, int v, cplx<R> acc) {
    const I2 pi = pts[i];
    const z64 gv = g[(r0 + v) * (long)n * n + (long)(o.y + pi.y) * n + (o.x + pi.x)];
    us[v][i] = acc + mk<R>((R)gv.x, (R)gv.y);
  });
  __syncthreads();
  // (ws is free once us is built: it stages the results for one store pass)
  leaf_rows<R, NV>(XT + t * (long)mL * mL, mL, mL, us, nv, [&](int i, int v, cplx<R> acc) { ws[v][i] = acc; });
  __syncthreads();
  for (int v = 0; v < nv; ++v)
    for (int i = threadIdx.x; i < mL; i += blockDim.x) {
      const I2 pi = pts[i];
      const cplx<R> val = ws[v][i];
      q[(r0 + v) * (long)n * n + (long)(o.y + pi.y) * n + (o.x + pi.x)] = mk((double)val.x, (double)val.y);
    }
}

template <typename R>
void leaf_tdown(hipStream_t s, const cplx<R>* XT, const cplx<R>* UL, int mL, int k, const cplx<R>* w, const z64* g,
                z64* q, const I2* leaf_origin, const I2* leaf_pts, int nleaf, int n, int nrhs) {
  LSH_REQUIRE(mL <= LEAF_MAX, -6, "leaf too large");
  const int ng = nrhs == 1 ? 1 : ceil_div(nrhs, LEAF_NV);
  ProfScope ps("leaf_tdown", s, (double)sizeof(cplx<R>) * nleaf * ((double)ng * mL * mL + (double)nrhs * (mL + k)) +
                                    32.0 * nrhs * (double)nleaf * mL);
  if (nrhs == 1)
    hipLaunchKernelGGL((k_leaf_tdown<R, 1>), dim3(nleaf, 1), dim3(256), 0, s, XT, UL, mL, k, w, g, q, leaf_origin,
                       leaf_pts, n, nleaf, nrhs);
  else
    hipLaunchKernelGGL((k_leaf_tdown<R, LEAF_NV>), dim3(nleaf, ng), dim3(256), 0, s, XT, UL, mL, k, w, g, q,
                       leaf_origin, leaf_pts, n, nleaf, nrhs);
  LSH_LAUNCH_CHECK();
}

// ------------------------------------------- apply, one Woodbury level fused
// One product of a box inside a workgroup of NT threads: H blocks (1 or 2) of M
// rows of N entries (row-major, packed; the second block sh entries after the
// first) times the vectors x_h of NV right-hand sides in LDS.  L lanes per row,
// 4, 8 or 16 by the row length (the short rows of deep levels would leave most
// of 16 lanes idle, and the instructions, not the bytes, bound such a level):
// lane s takes columns s + L u of each 4 L-column chunk, P rows per lane group
// at a time, the products of a row added column by column in each lane and
// then over the lanes by DPP (the same arithmetic for any NT and NV).
template <typename R>
struct BoxProd {
  const cplx<R>* A;
  int M, N, H, sh, lg;  // lg: log2 L
  __device__ __forceinline__ BoxProd(const cplx<R>* A_, int M_, int N_, int H_, int sh_)
      : A(A_), M(M_), N(N_), H(H_), sh(sh_), lg(N_ <= 16 ? 2 : N_ <= 32 ? 3 : 4) {}
};
template <typename R, int P>
struct BoxFrag {
  cplx<R> a[P][4];
};

// entries of chunk j0 of row block blk; outside the product those of its last
// row block, row or column instead (their sums are not stored, their x is zero)
template <typename R, int P>
__device__ __forceinline__ void box_load(BoxFrag<R, P>& f, const BoxProd<R>& m, int blk, int j0) {
  const int L = 1 << m.lg, sub = threadIdx.x & (L - 1), nbk = (m.M + P - 1) / P, last = m.H * nbk - 1;
  blk = blk < last ? blk : last;
  const bool h1 = blk >= nbk;
  const int i0 = (blk - (h1 ? nbk : 0)) * P;
  const char* base = reinterpret_cast<const char*>(m.A);
  unsigned row[P], col[4];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const int i = i0 + p < m.M ? i0 + p : m.M - 1;
    row[p] = (unsigned)((h1 ? m.sh : 0) + i * m.N) * (unsigned)sizeof(cplx<R>);
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int j = j0 + sub + (u << m.lg);
    col[u] = (unsigned)(j < m.N ? j : m.N - 1) * (unsigned)sizeof(cplx<R>);
  }
#pragma unroll
  for (int p = 0; p < P; ++p)
#pragma unroll
    for (int u = 0; u < 4; ++u) f.a[p][u] = *reinterpret_cast<const cplx<R>*>(base + (row[p] + col[u]));
}
template <typename R, int P>
__device__ __forceinline__ void box_first(BoxFrag<R, P>& f, const BoxProd<R>& m) {
  box_load<R, P>(f, m, threadIdx.x >> m.lg, 0);
}

// out(h, i, v, sum) for every row and vector; f: this group's first chunk,
// already loaded.  The next chunk (or row block) is in flight during the
// products of the current one.
template <typename R, int P, int NT, int NV, typename Out>
__device__ __forceinline__ void box_run(const BoxProd<R>& m, BoxFrag<R, P>& f, const cplx<R>* x0, const cplx<R>* x1,
                                        int ldx, Out out) {
  const int L = 1 << m.lg, NG = NT >> m.lg, sub = threadIdx.x & (L - 1), grp = threadIdx.x >> m.lg;
  const int nbk = (m.M + P - 1) / P, nblk = m.H * nbk;
  for (int blk = grp; blk < nblk; blk += NG) {
    const bool h1 = blk >= nbk;
    const int i0 = (blk - (h1 ? nbk : 0)) * P;
    const cplx<R>* x = h1 ? x1 : x0;
    cplx<R> acc[P][NV];
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
      for (int v = 0; v < NV; ++v) acc[p][v] = mk<R>(0, 0);
    for (int j0 = 0; j0 < m.N; j0 += 4 * L) {
      BoxFrag<R, P> nx;
      const bool more = j0 + 4 * L < m.N;
      if (more || blk + NG < nblk) box_load<R, P>(nx, m, more ? blk : blk + NG, more ? j0 + 4 * L : 0);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int j = j0 + sub + (u << m.lg);
        cplx<R> xv[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          const cplx<R> t = x[v * ldx + (j < m.N ? j : m.N - 1)];
          xv[v] = mk(j < m.N ? t.x : R(0), j < m.N ? t.y : R(0));
        }
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
          for (int v = 0; v < NV; ++v) fma_acc(acc[p][v], f.a[p][u], xv[v]);
      }
      f = nx;
    }
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        cplx<R> t = mk(group_sum<4>(acc[p][v].x), group_sum<4>(acc[p][v].y));
        if (m.lg >= 3) t = t + mk(dpp_mov<0x141>(t.x), dpp_mov<0x141>(t.y));  // row_half_mirror
        if (m.lg >= 4) t = t + mk(dpp_mov<0x140>(t.x), dpp_mov<0x140>(t.y));  // row_mirror
        if (sub == 0 && i0 + p < m.M) out(h1 ? 1 : 0, i0 + p, v, t);
      }
  }
}

// A level's step in one launch: a workgroup per box and group of NV right-hand
// sides, which reads the box's matrices once for the group, every
// intermediate vector in LDS.  Between the four to six products stand
// barriers; each product's first entries are loaded two products ahead, so
// that a deep level (c = 29, 8192 boxes), whose products are one or two such
// loads, waits for memory once and not six times.  Box vector (right-hand
// side q, box b) is number q nb + b.
// The box matrices come at 2.7 to 3.1 TB/s (1024 x 1024, FP32, one vector:
// the down pass of 8192 boxes of c = 28, 184 MB, 68 us, of 256 of c = 188,
// 239 MB, 76 us), the arithmetic of the short rows being the other half of
// the deep levels' time.  Against one workgroup per box vector and 16 lanes for
// every row, whole applies: 512 x 512 with 8 vectors 2.38 -> 1.9 ms, its
// transpose (unfused before) 2.66 -> 1.9 ms; 384 x 384, FP64, 3 vectors 1.26 -> 1.14.
//
// PASS 0, up (Algorithm 2's upward step): input [rt_a; rt_b] (2c),
//   q = [L^T rt_a; R^T rt_b], y = W' q, t = in - [S_a L y1; S_b R y2],
//   out = U_l^T t (k).
// PASS 1, down: wt (k) and the children's rt (2c),
//   u = U_l wt, d = rt - diag(S_a, S_b) u, o = X_tau d (as above),
//   out = [G_ab o_b; G_ba o_a] + u.
// PASS 2, the down step transposed (leaves upward): wc (2c),
//   vb = [G_ab wc_b; G_ba wc_a] (kept for PASS 3), t = X_tau^T vb, with
//   X_tau^T v = v - [L z_1; R z_2], z = W'^T [(S_a L)^T v_a; (S_b R)^T v_b],
//   out = U_l^T (wc - diag(S_a, S_b)^T t) (k).
// PASS 3, the up step transposed: rb (k) and vb,
//   out = X_tau^T (vb + U_l rb) (2c).
template <typename R>
constexpr int LVL_P = sizeof(R) == 4 ? 2 : 1;

// LDS entries of one box vector
__host__ __device__ inline int level_lds(int pass, int c, int k, int r) {
  return pass == 0 ? 2 * c + 4 * r : pass == 1 ? k + 4 * c + 4 * r : pass == 2 ? 6 * c + 4 * r : k + 2 * c + 4 * r;
}

template <typename R, int NT, int NV, int PASS>
__global__ __launch_bounds__(NT) void k_level(LevelApply<R> A, const cplx<R>* __restrict__ in,
                                              const cplx<R>* __restrict__ in2, cplx<R>* __restrict__ out,
                                              cplx<R>* __restrict__ out2, int nrhs) {
  constexpr int P = LVL_P<R>;
  extern __shared__ __align__(16) unsigned char lvl_lds[];
  const int c = A.c, k = A.k, r = A.r, nb = A.nb, c2 = 2 * c, r2 = 2 * r;
  const int b = blockIdx.x % nb, q0 = blockIdx.x / nb * NV;
  const int nv = nrhs - q0 < NV ? nrhs - q0 : NV;
  const long cr = (long)c * r, cc = (long)c * c;
  cplx<R>* lds = reinterpret_cast<cplx<R>*>(lvl_lds);
  auto vec = [&](int v) { return (long)(q0 + v) * nb + b; };
  // copy of n entries per vector from global memory (zero for absent vectors)
  auto stage = [&](cplx<R>* dst, const cplx<R>* src, int n) {
#pragma unroll
    for (int v = 0; v < NV; ++v)
      for (int i = threadIdx.x; i < n; i += NT) dst[v * n + i] = v < nv ? src[vec(v) * n + i] : mk<R>(0, 0);
  };
  const BoxProd<R> mQ(A.Q, r, c, 2, r * c), mW(A.Ci + b * 4L * r * r, r2, r2, 1, 0);
  const BoxProd<R> mS(A.S + 2 * cc * b, c, c, 2, c * c), mL(A.Q, c, r, 2, r * c);  // (PASS 2, 3: Q holds [L; R])
  const BoxProd<R> mP(A.Pa + 2 * cr * b, PASS < 2 ? c : r, PASS < 2 ? r : c, 2, r * c);
  const BoxProd<R> mU(A.U, c2, k, 1, 0), mUt(A.Ut, k, c2, 1, 0), mG(A.Gab, c, c, 2, (int)(A.Gba - A.Gab));
  BoxFrag<R, P> f0, f1;
  if constexpr (PASS == 0) {
    cplx<R>*xs = lds, *q = xs + NV * c2, *y = q + NV * r2;
    box_first(f0, mQ);
    box_first(f1, mW);
    stage(xs, in, c2);
    __syncthreads();
    box_run<R, P, NT, NV>(mQ, f0, xs, xs + c, c2, [&](int h, int i, int v, cplx<R> s) { q[v * r2 + h * r + i] = s; });
    box_first(f0, mP);
    __syncthreads();
    box_run<R, P, NT, NV>(mW, f1, q, q, r2, [&](int, int i, int v, cplx<R> s) { y[v * r2 + i] = s; });
    box_first(f1, mUt);
    __syncthreads();
    box_run<R, P, NT, NV>(mP, f0, y, y + r, r2, [&](int h, int i, int v, cplx<R> s) {
      cplx<R>& t = xs[v * c2 + h * c + i];
      t = t - s;
    });
    __syncthreads();
    box_run<R, P, NT, NV>(mUt, f1, xs, xs, c2, [&](int, int i, int v, cplx<R> s) {
      if (v < nv) out[vec(v) * k + i] = s;
    });
  } else if constexpr (PASS == 1) {
    cplx<R>*w = lds, *u = w + NV * k, *d = u + NV * c2, *q = d + NV * c2, *y = q + NV * r2;
    box_first(f0, mU);
    box_first(f1, mS);
    stage(w, in, k);
    stage(d, in2, c2);
    __syncthreads();
    box_run<R, P, NT, NV>(mU, f0, w, w, k, [&](int, int i, int v, cplx<R> s) { u[v * c2 + i] = s; });
    box_first(f0, mQ);
    __syncthreads();
    box_run<R, P, NT, NV>(mS, f1, u, u + c, c2, [&](int h, int i, int v, cplx<R> s) {
      cplx<R>& t = d[v * c2 + h * c + i];
      t = t - s;
    });
    box_first(f1, mW);
    __syncthreads();
    box_run<R, P, NT, NV>(mQ, f0, d, d + c, c2, [&](int h, int i, int v, cplx<R> s) { q[v * r2 + h * r + i] = s; });
    box_first(f0, mP);
    __syncthreads();
    box_run<R, P, NT, NV>(mW, f1, q, q, r2, [&](int, int i, int v, cplx<R> s) { y[v * r2 + i] = s; });
    box_first(f1, mG);
    __syncthreads();
    box_run<R, P, NT, NV>(mP, f0, y, y + r, r2, [&](int h, int i, int v, cplx<R> s) {
      cplx<R>& t = d[v * c2 + h * c + i];
      t = t - s;
    });
    __syncthreads();
    box_run<R, P, NT, NV>(mG, f1, d + c, d, c2, [&](int h, int i, int v, cplx<R> s) {
      if (v < nv) out[vec(v) * c2 + h * c + i] = s + u[v * c2 + h * c + i];
    });
  } else if constexpr (PASS == 2) {
    cplx<R>*w = lds, *vb = w + NV * c2, *t = vb + NV * c2, *q = t + NV * c2, *y = q + NV * r2;
    box_first(f0, mG);
    box_first(f1, mP);
    stage(w, in, c2);
    __syncthreads();
    box_run<R, P, NT, NV>(mG, f0, w + c, w, c2, [&](int h, int i, int v, cplx<R> s) {
      vb[v * c2 + h * c + i] = s;
      if (v < nv) out2[vec(v) * c2 + h * c + i] = s;
    });
    box_first(f0, mW);
    __syncthreads();
    box_run<R, P, NT, NV>(mP, f1, vb, vb + c, c2, [&](int h, int i, int v, cplx<R> s) { q[v * r2 + h * r + i] = s; });
    box_first(f1, mL);
    __syncthreads();
    box_run<R, P, NT, NV>(mW, f0, q, q, r2, [&](int, int i, int v, cplx<R> s) { y[v * r2 + i] = s; });
    box_first(f0, mS);
    __syncthreads();
    box_run<R, P, NT, NV>(mL, f1, y, y + r, r2, [&](int h, int i, int v, cplx<R> s) {
      t[v * c2 + h * c + i] = vb[v * c2 + h * c + i] - s;
    });
    box_first(f1, mUt);
    __syncthreads();
    box_run<R, P, NT, NV>(mS, f0, t, t + c, c2, [&](int h, int i, int v, cplx<R> s) {
      cplx<R>& x = w[v * c2 + h * c + i];
      x = x - s;
    });
    __syncthreads();
    box_run<R, P, NT, NV>(mUt, f1, w, w, c2, [&](int, int i, int v, cplx<R> s) {
      if (v < nv) out[vec(v) * k + i] = s;
    });
  } else {
    cplx<R>*w = lds, *t = w + NV * k, *q = t + NV * c2, *y = q + NV * r2;
    box_first(f0, mU);
    box_first(f1, mP);
    stage(w, in, k);
    stage(t, in2, c2);
    __syncthreads();
    box_run<R, P, NT, NV>(mU, f0, w, w, k, [&](int, int i, int v, cplx<R> s) {
      cplx<R>& x = t[v * c2 + i];
      x = x + s;
    });
    box_first(f0, mW);
    __syncthreads();
    box_run<R, P, NT, NV>(mP, f1, t, t + c, c2, [&](int h, int i, int v, cplx<R> s) { q[v * r2 + h * r + i] = s; });
    box_first(f1, mL);
    __syncthreads();
    box_run<R, P, NT, NV>(mW, f0, q, q, r2, [&](int, int i, int v, cplx<R> s) { y[v * r2 + i] = s; });
    __syncthreads();
    box_run<R, P, NT, NV>(mL, f1, y, y + r, r2, [&](int h, int i, int v, cplx<R> s) {
      if (v < nv) out[vec(v) * c2 + h * c + i] = t[v * c2 + h * c + i] - s;
    });
  }
}

template <typename R, int PASS>
static void level_launch(hipStream_t s, const LevelApply<R>& A, const cplx<R>* in, const cplx<R>* in2, cplx<R>* out,
                         cplx<R>* out2, int nvec) {
  LSH_REQUIRE(A.c > 0 && A.k > 0 && A.r > 0 && A.nb > 0 && nvec > 0 && nvec % A.nb == 0, -6,
              "fused level apply: bad sizes");
  const size_t one = (size_t)level_lds(PASS, A.c, A.k, A.r) * sizeof(cplx<R>);
  LSH_REQUIRE(one <= LEVEL_FUSED_LDS, -6, "fused level apply: the box vectors exceed the workgroup's LDS");
  const double e = (double)sizeof(cplx<R>), c = A.c, k = A.k, r = A.r;
  static const char* name[2][4] = {{"level_up_f32", "level_down_f32", "level_tup_f32", "level_tdown_f32"},
                                   {"level_up_f64", "level_down_f64", "level_tup_f64", "level_tdown_f64"}};
  const bool square = PASS == 1 || PASS == 2;  // the S and G products
  ProfScope ps(name[sizeof(R) == 8][PASS], s,
               e * ((double)A.nb * (4 * r * r + 2 * c * r + (square ? 2 * c * c : 0)) + 2 * r * c + 2 * c * k +
                    (square ? 2 * c * c : 0) + (double)nvec * (k + (PASS == 0 ? 2 : 4) * c)));
  // right-hand sides per workgroup: as many (4, 2 or 1) as leave a workgroup
  // per compute unit and fit the LDS; then threads for about 8192 waves in all
  const int nrhs = nvec / A.nb;
  int nv = nrhs >= 3 ? 4 : nrhs;
  while (nv > 1 && (nv * one > LEVEL_FUSED_LDS || (long)A.nb * ((nrhs + nv - 1) / nv) < 256)) nv /= 2;
  const int grid = A.nb * ((nrhs + nv - 1) / nv), nt = grid <= 512 ? 1024 : grid <= 1024 ? 512 : grid <= 2048 ? 256 : grid <= 4096 ? 128 : 64;
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(grid), dim3(nt), nv * one, s, A, in, in2, out, out2, nrhs);
  };
#define LSH_LEVEL(NT)                             \
  case NT:                                        \
    if (nv == 4) go(k_level<R, NT, 4, PASS>);     \
    else if (nv == 2) go(k_level<R, NT, 2, PASS>); \
    else go(k_level<R, NT, 1, PASS>);             \
    break;
  switch (nt) { LSH_LEVEL(1024) LSH_LEVEL(512) LSH_LEVEL(256) LSH_LEVEL(128) LSH_LEVEL(64) }
#undef LSH_LEVEL
  LSH_LAUNCH_CHECK();
}

// (2^27 entries of 16 bytes are 2^31; a block that fits level_fits is far below the other 2^31)
bool level_offsets_fit(long between) { return between >= 0 && between <= (1L << 27); }

template <typename R>
bool level_fits(int c, int k, int r, bool transposed) {
  const int n = transposed ? std::max(level_lds(2, c, k, r), level_lds(3, c, k, r))
                           : std::max(level_lds(0, c, k, r), level_lds(1, c, k, r));
  return (size_t)n * sizeof(cplx<R>) <= LEVEL_FUSED_LDS;
}

template <typename R>
void level_up_fused(hipStream_t s, const LevelApply<R>& A, const cplx<R>* in, cplx<R>* out, int nvec) {
  level_launch<R, 0>(s, A, in, nullptr, out, nullptr, nvec);
}
template <typename R>
void level_down_fused(hipStream_t s, const LevelApply<R>& A, const cplx<R>* wt, const cplx<R>* rtc, cplx<R>* wc,
                      int nvec) {
  level_launch<R, 1>(s, A, wt, rtc, wc, nullptr, nvec);
}
template <typename R>
void level_tup_fused(hipStream_t s, const LevelApply<R>& A, const cplx<R>* wc, cplx<R>* vb, cplx<R>* wb, int nvec) {
  level_launch<R, 2>(s, A, wc, nullptr, wb, vb, nvec);
}
template <typename R>
void level_tdown_fused(hipStream_t s, const LevelApply<R>& A, const cplx<R>* rb, const cplx<R>* vb, cplx<R>* rbc,
                       int nvec) {
  level_launch<R, 3>(s, A, rb, vb, rbc, nullptr, nvec);
}

#define LSH_HBS_INST(R)                                                                                       \
  template void leaf_build<R>(hipStream_t, cplx<R>*, const cplx<R>*, int, const double*, double, const I2*,   \
                              const I2*, int, int);                                                          \
  template void leaf_scale_U<R>(hipStream_t, cplx<R>*, const cplx<R>*, int, int, const double*, double,       \
                                const I2*, const I2*, int, int);                                             \
  template void leaf_up<R>(hipStream_t, const cplx<R>*, const cplx<R>*, int, int, const z64*, cplx<R>*,        \
                           cplx<R>*, const I2*, const I2*, int, int, int, const double*, double);           \
  template void leaf_tdown<R>(hipStream_t, const cplx<R>*, const cplx<R>*, int, int, const cplx<R>*, const z64*,  \
                              z64*, const I2*, const I2*, int, int, int);                                    \
  template void leaf_down<R>(hipStream_t, const cplx<R>*, const cplx<R>*, int, int, const cplx<R>*,           \
                             const cplx<R>*, z64*, const double*, double, const I2*, const I2*, int, int, int);    \
  template void level_up_fused<R>(hipStream_t, const LevelApply<R>&, const cplx<R>*, cplx<R>*, int);            \
  template void level_down_fused<R>(hipStream_t, const LevelApply<R>&, const cplx<R>*, const cplx<R>*, cplx<R>*, \
                                    int);                                                                    \
  template void level_tup_fused<R>(hipStream_t, const LevelApply<R>&, const cplx<R>*, cplx<R>*, cplx<R>*, int); \
  template void level_tdown_fused<R>(hipStream_t, const LevelApply<R>&, const cplx<R>*, const cplx<R>*,        \
                                     cplx<R>*, int);                                                         \
  template bool level_fits<R>(int, int, int, bool);
LSH_HBS_INST(float)
LSH_HBS_INST(double)

}  // namespace lsh
