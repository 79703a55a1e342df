// Kernel-entry generator and FGMRES vector kernels.  All FP64.
#include <algorithm>
#include <cmath>

#include "../../include/lsh.h"
#include "ops.hpp"
#include "prof.hpp"
#include "wave.hpp"

namespace lsh {

// ------------------------------------------------------------ offset table
__global__ void k_offset_table(z64* T, int D, double h, double kappa, double t0r, double t0i) {
  const long e = blockIdx.x * (long)blockDim.x + threadIdx.x;
  const long W = D + 1;
  if (e >= W * W) return;
  const int dy = (int)(e / W), dx = (int)(e % W);
  z64 v;
  if (dx == 0 && dy == 0) {
    v = mk(t0r, t0i);
  } else {
    const double r = kappa * h * sqrt((double)dx * dx + (double)dy * dy);
    // (i/4) H0(r) = (i/4)(J0 + i Y0) = -Y0/4 + i J0/4
    v = mk(-0.25 * y0(r), 0.25 * j0(r));
  }
  T[e] = (h * h) * v;
}

void build_offset_table(hipStream_t s, z64* T, int D, double h, double kappa, double tau0_re, double tau0_im) {
  const long W = D + 1;
  hipLaunchKernelGGL(k_offset_table, dim3(ceil_div(W * W, 256)), dim3(256), 0, s, T, D, h, kappa, tau0_re,
                     tau0_im);
  LSH_LAUNCH_CHECK();
}

__global__ void k_table_add(z64* T, int D, const int* dxy, const z64* w, int cnt) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= cnt) return;
  const int dx = dxy[2 * k], dy = dxy[2 * k + 1];
  T[(long)dy * (D + 1) + dx] = T[(long)dy * (D + 1) + dx] + w[k];
}

void add_table_stencil(hipStream_t s, z64* T, int D, double h, const std::vector<StencilEntry>& stencil,
                       mem::Arena& scr) {
  std::vector<int> dxy;
  std::vector<z64> wv;
  for (auto& e : stencil) {  // one representative per offset (|dx|, |dy|): the stencil is symmetric
    if (e.dx < 0 || e.dy < 0 || (e.dx == 0 && e.dy == 0) || e.dx > D || e.dy > D) continue;
    dxy.push_back(e.dx);
    dxy.push_back(e.dy);
    wv.push_back(mk(h * h * e.re, h * h * e.im));
  }
  if (wv.empty()) return;
  int* ddxy = static_cast<int*>(scr.take(sizeof(int) * dxy.size()));
  z64* dw = static_cast<z64*>(scr.take(sizeof(z64) * wv.size()));
  LSH_HIP(hipMemcpyAsync(ddxy, dxy.data(), sizeof(int) * dxy.size(), hipMemcpyHostToDevice, s));
  LSH_HIP(hipMemcpyAsync(dw, wv.data(), sizeof(z64) * wv.size(), hipMemcpyHostToDevice, s));
  hipLaunchKernelGGL(k_table_add, dim3(ceil_div((int)wv.size(), 64)), dim3(64), 0, s, T, D, ddxy, dw,
                     (int)wv.size());
  LSH_LAUNCH_CHECK();
  LSH_HIP(hipStreamSynchronize(s));  // the host staging vectors die here
}

// --------------------------------------------------------- vector kernels
constexpr int MD_BLOCKS = 1024, MD_NT = 256, MD_MAXV = 128;

__global__ __launch_bounds__(MD_NT) void k_multidot(const z64* __restrict__ V, long ldv, int nv,
                                                    const z64* __restrict__ w, long N, z64* partial) {
  __shared__ z64 red[MD_MAXV][MD_NT / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int v = 0; v < nv; ++v) {
    const z64* Vv = V + v * ldv;
    z64 acc = mk(0.0, 0.0);
    for (long i = blockIdx.x * (long)MD_NT + threadIdx.x; i < N; i += (long)MD_BLOCKS * MD_NT)
      fma_acc(acc, conjg(Vv[i]), w[i]);
    for (int off = 32; off > 0; off >>= 1) {
      acc.x += __shfl_xor(acc.x, off);
      acc.y += __shfl_xor(acc.y, off);
    }
    if (lane == 0) red[v][wave] = acc;
  }
  __syncthreads();
  for (int v = threadIdx.x; v < nv; v += MD_NT) {
    z64 a = red[v][0];
    for (int k = 1; k < MD_NT / 64; ++k) a = a + red[v][k];
    partial[(long)v * MD_BLOCKS + blockIdx.x] = a;
  }
}

__global__ __launch_bounds__(256) void k_reduce_partials(const z64* partial, int nparts, z64* out) {
  __shared__ z64 red[256];
  const int v = blockIdx.x;
  z64 a = mk(0.0, 0.0);
  for (int k = threadIdx.x; k < nparts; k += 256) a = a + partial[(long)v * nparts + k];
  red[threadIdx.x] = a;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st) red[threadIdx.x] = red[threadIdx.x] + red[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[v] = red[0];
}

size_t multidot_partial_bytes(int nv) { return sizeof(z64) * (size_t)nv * MD_BLOCKS; }

void multidot(hipStream_t s, const z64* V, long ldv, int nv, const z64* w, long N, z64* out, z64* partial) {
  ProfScope ps("op_multidot", s, 16.0 * (double)N * (nv + 1));
  LSH_REQUIRE(nv <= MD_MAXV, -6, "multidot: too many vectors");
  hipLaunchKernelGGL(k_multidot, dim3(MD_BLOCKS), dim3(MD_NT), 0, s, V, ldv, nv, w, N, partial);
  LSH_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_reduce_partials, dim3(nv), dim3(256), 0, s, partial, MD_BLOCKS, out);
  LSH_LAUNCH_CHECK();
}

// One FGMRES step's classical Gram-Schmidt, twice, and the scaling of the new
// basis vector, for the group's vectors together (blockIdx.y), in four launches:
//   0  p0 = V^H w, one partial sum per workgroup
//   1  h1 = sum p0;  w -= V h1;  p1 = V^H w
//   2  h2 = sum p1;  w -= V h2;  p2 = |w|^2
//   3  |w|^2 = sum p2;  w /= |w| (left alone where that is not positive)
// Every workgroup adds up the partial sums it needs by itself, which costs
// less than a launch for them, and step 1's second look at its part of V finds
// it in L2.  About 256 workgroups in all share the vectors still running (bits
// of active), one per compute unit, so there are few partial sums.  Bound by
// the three passes over V (8 vectors of 512 x 512 against 6 each: 22 + 36 + 22
// + 8 us, V from the memory side's cache at up to 10 TB/s) and on small grids
// by the launches.  With nine launches for each vector by itself this took some
// 320 us, and the solve of 8 fields on 512 x 512 14.8 ms against 13.9.  (The
// workgroups go to running vectors only: 30 unpreconditioned iterations for
// one of eight on 1024 x 1024 take 26.4 ms, 46.7 with an eighth for each.)
constexpr int CGS_NT = 1024, CGS_E = 4, CGS_WG = 256, CGS_MAXV = LSH_MAX_ITERS;

template <int STEP>
__global__ __launch_bounds__(CGS_NT) void k_cgs(const z64* __restrict__ V, long ldv, int nv, z64* w, long N,
                                                unsigned active, const z64* __restrict__ pin, z64* __restrict__ pout,
                                                z64* h, int hs) {
  __shared__ z64 red[STEP <= 1 ? CGS_MAXV : 1][CGS_NT / 64];
  __shared__ z64 hv[STEP == 0 ? 1 : CGS_MAXV];
  const int q = blockIdx.y, nb = gridDim.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int k = 0; k < q; ++k) active &= active - 1;
  const int r = __builtin_ctz(active);  // the q-th running vector
  V += r * N;
  w += r * N;
  if (STEP > 0) {
    const int ns = STEP == 3 ? 1 : nv;
    for (int v = wave; v < ns; v += CGS_NT / 64) {
      const z64* p = pin + ((long)q * ns + v) * nb;
      z64 a = mk(0.0, 0.0);
      for (int k = lane; k < nb; k += 64) a = a + p[k];
      a = mk(group_sum<64>(a.x), group_sum<64>(a.y));
      if (lane == 0) {
        hv[v] = a;
        if (blockIdx.x == 0) h[(long)r * hs + (STEP == 3 ? nv : v)] = a;
      }
    }
    __syncthreads();
  }
  if (STEP == 3) {
    const double s = hv[0].x > 0 ? 1.0 / sqrt(hv[0].x) : 1.0;
    for (long i = blockIdx.x * (long)CGS_NT + tid; i < N; i += (long)nb * CGS_NT) w[i] = s * w[i];
    return;
  }
  z64 nrm = mk(0.0, 0.0);
  bool first = true;
  for (long i0 = blockIdx.x * (long)(CGS_NT * CGS_E) + tid; i0 - tid < N; i0 += (long)nb * CGS_NT * CGS_E) {
    // (what lies past the end is read as the last element and counted as zero:
    // no branch stands between the loads)
    z64 x[CGS_E];
    long ix[CGS_E];
#pragma unroll
    for (int e = 0; e < CGS_E; ++e) {
      const long i = i0 + e * CGS_NT;
      ix[e] = i < N ? i : N - 1;
      x[e] = w[ix[e]];
    }
    if (STEP > 0) {
#pragma unroll 4
      for (int v = 0; v < nv; ++v) {
        const z64* Vv = V + v * ldv;
        const z64 c = hv[v];
#pragma unroll
        for (int e = 0; e < CGS_E; ++e) x[e] = x[e] - Vv[ix[e]] * c;
      }
#pragma unroll
      for (int e = 0; e < CGS_E; ++e)
        if (i0 + e * CGS_NT < N) w[ix[e]] = x[e];
    }
#pragma unroll
    for (int e = 0; e < CGS_E; ++e)
      if (i0 + e * CGS_NT >= N) x[e] = mk(0.0, 0.0);
    if (STEP <= 1) {
#pragma unroll 4
      for (int v = 0; v < nv; ++v) {
        const z64* Vv = V + v * ldv;
        z64 acc = mk(0.0, 0.0);
#pragma unroll
        for (int e = 0; e < CGS_E; ++e) fma_acc(acc, conjg(Vv[ix[e]]), x[e]);
        acc = mk(group_sum<64>(acc.x), group_sum<64>(acc.y));
        if (lane == 0) red[v][wave] = first ? acc : red[v][wave] + acc;
      }
    } else {
#pragma unroll
      for (int e = 0; e < CGS_E; ++e) fma_acc(nrm, conjg(x[e]), x[e]);
    }
    first = false;
  }
  if (STEP == 2) {
    nrm = mk(group_sum<64>(nrm.x), group_sum<64>(nrm.y));
    if (lane == 0) red[0][wave] = nrm;
  }
  __syncthreads();
  const int ns = STEP == 2 ? 1 : nv;
  for (int v = tid; v < ns; v += CGS_NT) {
    z64 a = red[v][0];
    for (int k = 1; k < CGS_NT / 64; ++k) a = a + red[v][k];
    pout[((long)q * ns + v) * nb + blockIdx.x] = a;
  }
}

void cgs2(hipStream_t s, const z64* V, long ldv, int nv, z64* w, long N, int nr, unsigned active, z64* h1, z64* h2,
          int hs, z64* partial) {
  ProfScope ps("gram_schmidt", s, 16.0 * (double)N * (3 * nv + 7) * __builtin_popcount(active));
  LSH_REQUIRE(nv <= CGS_MAXV && nr >= 1 && nr <= 32, -6, "gram-schmidt: too many vectors");
  const int na = __builtin_popcount(active);
  if (na == 0) return;
  // the running vectors share the workgroups; every workgroup has a piece of
  // its vector: none writes an unset partial sum
  const int nb = (int)std::max(1L, std::min((long)(CGS_WG / na), (long)ceil_div(N, (long)(CGS_NT * CGS_E))));
  z64 *p0 = partial, *p1 = p0 + (size_t)na * nv * nb, *p2 = p1 + (size_t)na * nv * nb;  // (at most (2 nv + 1) CGS_WG)
  const dim3 grid(nb, na);
  hipLaunchKernelGGL(k_cgs<0>, grid, dim3(CGS_NT), 0, s, V, ldv, nv, w, N, active, p2, p0, h1, hs);
  LSH_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_cgs<1>, grid, dim3(CGS_NT), 0, s, V, ldv, nv, w, N, active, p0, p1, h1, hs);
  LSH_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_cgs<2>, grid, dim3(CGS_NT), 0, s, V, ldv, nv, w, N, active, p1, p2, h2, hs);
  LSH_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_cgs<3>, grid, dim3(CGS_NT), 0, s, V, ldv, nv, w, N, active, p2, p0, h2, hs);
  LSH_LAUNCH_CHECK();
}

__global__ void k_scale_invnorm(z64* y, const z64* x, const z64* nrm2, long N) {
  const double s = 1.0 / sqrt(nrm2[0].x);
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < N; i += (long)gridDim.x * blockDim.x)
    y[i] = s * x[i];
}

void scale_by_invnorm(hipStream_t s, z64* y, const z64* x, const z64* nrm2, long N) {
  hipLaunchKernelGGL(k_scale_invnorm, dim3(2048), dim3(256), 0, s, y, x, nrm2, N);
  LSH_LAUNCH_CHECK();
}

__global__ void k_lincomb(z64* y, const z64* __restrict__ V, long ldv, int nv, const z64* __restrict__ c, long N) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < N; i += (long)gridDim.x * blockDim.x) {
    z64 a = mk(0.0, 0.0);
    for (int v = 0; v < nv; ++v) fma_acc(a, V[v * ldv + i], c[v]);
    y[i] = a;
  }
}

void lincomb(hipStream_t s, z64* y, const z64* V, long ldv, int nv, const z64* c, long N) {
  hipLaunchKernelGGL(k_lincomb, dim3(2048), dim3(256), 0, s, y, V, ldv, nv, c, N);
  LSH_LAUNCH_CHECK();
}

__global__ void k_scale_real(z64* y, const z64* x, const double* b, double a, long N, long nb) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < N; i += (long)gridDim.x * blockDim.x)
    y[i] = (a * b[i % nb]) * x[i];
}

void scale_real(hipStream_t s, z64* y, const z64* x, const double* b, double a, long N) {
  hipLaunchKernelGGL(k_scale_real, dim3(2048), dim3(256), 0, s, y, x, b, a, N, N);
  LSH_LAUNCH_CHECK();
}

__global__ void k_sub_from(z64* y, const z64* x, long N) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < N; i += (long)gridDim.x * blockDim.x)
    y[i] = x[i] - y[i];
}

void sub_from(hipStream_t s, z64* y, const z64* x, long N) {
  hipLaunchKernelGGL(k_sub_from, dim3(2048), dim3(256), 0, s, y, x, N);
  LSH_LAUNCH_CHECK();
}

__global__ void k_conj(z64* y, const z64* x, long N) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < N; i += (long)gridDim.x * blockDim.x)
    y[i] = conjg(x[i]);
}

void conj_copy(hipStream_t s, z64* y, const z64* x, long N) {
  hipLaunchKernelGGL(k_conj, dim3(2048), dim3(256), 0, s, y, x, N);
  LSH_LAUNCH_CHECK();
}

__global__ void k_fill_zero(uint32_t* p, long n) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) p[i] = 0;
}

void fill_zero(hipStream_t s, void* p, size_t bytes) {
  if (!bytes) return;
  LSH_REQUIRE(bytes % 4 == 0, -1, "fill_zero: size must be a multiple of 4");
  long n = (long)(bytes / 4);
  int blocks = (int)((n + 255) / 256);
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_fill_zero, dim3(blocks), dim3(256), 0, s, static_cast<uint32_t*>(p), n);
  LSH_LAUNCH_CHECK();
}

}  // namespace lsh
