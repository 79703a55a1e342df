// FFT convolution operator (paper Sec. 2.2 end and Sec. 5: G + T is a
// convolution on the regular grid, applied by FFT).  All FP64.
//
// Three launches apply the operator to a group of vectors: rows of the data
// forward, columns forward times the spectrum and back, rows back.  The first
// two write their results transposed, so that every launch reads rows: a
// workgroup transforms ROWS neighbouring rows with the row index fastest over
// the lanes, and a transposed store is runs of ROWS entries.  Lengths are
// M = r 2^k >= 2n with r = 1, 3 or 5 (the grids are leaf 2^m a side), the
// whole batch of vectors is in each launch (grid y), and neighbouring row
// groups go to one XCD, whose L2 joins their parts of a line.
// The passes move 64 n M + 56 n^2 + 4 (M + 2)^2 bytes a vector; they are bound by
// those bytes on large grids and by the three launches on small ones.
// Against five launches a vector (transposes on their own) at powers of two:
// n = 64, 22.9 -> 14.4 us; n = 640 and four vectors, 318 -> 115-125 us (3.4 -> 2.3
// TB/s, 0.27 instead of 1.1 GB); n = 1024, 105 -> 68 us.
#include <cmath>

#include "ops.hpp"
#include "prof.hpp"

namespace lsh {
namespace {

constexpr double kC[8] = {1.0,
                          0.92387953251128675613,
                          0.70710678118654752440,
                          0.38268343236508977173,
                          0.0,
                          -0.38268343236508977173,
                          -0.70710678118654752440,
                          -0.92387953251128675613};  // cos(2 pi p / 16)
constexpr double kS[8] = {0.0,
                          0.38268343236508977173,
                          0.70710678118654752440,
                          0.92387953251128675613,
                          1.0,
                          0.92387953251128675613,
                          0.70710678118654752440,
                          0.38268343236508977173};  // sin(2 pi p / 16)

constexpr int brev(int i, int bits) {
  int r = 0;
  for (int b = 0; b < bits; ++b) r |= ((i >> b) & 1) << (bits - 1 - b);
  return r;
}
constexpr int lg(int R) { return R == 2 ? 1 : R == 4 ? 2 : R == 8 ? 3 : 4; }

// a * w_16^p (forward: w = exp(-2 pi i / 16); inverse: its conjugate)
template <int P, bool INV>
__device__ __forceinline__ z64 rot16(z64 a) {
  if (P == 0) return a;
  if (P == 4) return INV ? mk(-a.y, a.x) : mk(a.y, -a.x);
  const double c = kC[P], sn = INV ? kS[P] : -kS[P];
  return mk(a.x * c - a.y * sn, a.x * sn + a.y * c);
}

// In-register DFT of v[0 .. R): out[k] = sum_r v[r] w_R^(r k).  R = 2, 4, 8,
// 16 by radix-2 decimation in time (bit-reversed loads, natural-order
// result); R = 3, 5 by the sums and differences of v[p] and v[R - p].
template <int R, bool INV>
__device__ __forceinline__ void dft(z64* v) {
  z64 a[R];
  if constexpr (R == 3 || R == 5) {
    constexpr int H = R / 2;
    // cos and sin of 2 pi q / R, q = 1 .. H
    constexpr double c[2] = {R == 3 ? -0.5 : 0.30901699437494742410, -0.80901699437494742410};
    constexpr double s[2] = {R == 3 ? 0.86602540378443864676 : 0.95105651629515357212, 0.58778525229247312917};
    z64 sp[H], dp[H];
    a[0] = v[0];
#pragma unroll
    for (int p = 0; p < H; ++p) {
      sp[p] = v[p + 1] + v[R - 1 - p];
      dp[p] = v[p + 1] - v[R - 1 - p];
      a[0] = a[0] + sp[p];
    }
#pragma unroll
    for (int k = 1; k <= H; ++k) {
      z64 x = v[0], y = mk(0.0, 0.0);
#pragma unroll
      for (int p = 1; p <= H; ++p) {
        const int q = (p * k) % R, f = q <= H ? q : R - q;  // the angle 2 pi p k / R folded into (0, pi)
        x = x + c[f - 1] * sp[p - 1];
        y = q <= H ? y + s[f - 1] * dp[p - 1] : y - s[f - 1] * dp[p - 1];
      }
      const z64 iy = INV ? mk(-y.y, y.x) : mk(y.y, -y.x);  // -i y forward, i y inverse
      a[k] = x + iy;
      a[R - k] = x - iy;
    }
  } else {
    constexpr int B = lg(R);
#pragma unroll
    for (int i = 0; i < R; ++i) a[i] = v[brev(i, B)];
#pragma unroll
    for (int half = 1; half < R; half <<= 1)
#pragma unroll
      for (int i = 0; i < R; i += 2 * half)
#pragma unroll
        for (int p = 0; p < half; ++p) {
          z64 t;
          switch (p * (16 / (2 * half))) {  // compile-time after unrolling
            case 0: t = rot16<0, INV>(a[i + p + half]); break;
            case 1: t = rot16<1, INV>(a[i + p + half]); break;
            case 2: t = rot16<2, INV>(a[i + p + half]); break;
            case 3: t = rot16<3, INV>(a[i + p + half]); break;
            case 4: t = rot16<4, INV>(a[i + p + half]); break;
            case 5: t = rot16<5, INV>(a[i + p + half]); break;
            case 6: t = rot16<6, INV>(a[i + p + half]); break;
            default: t = rot16<7, INV>(a[i + p + half]); break;
          }
          const z64 u = a[i + p];
          a[i + p] = u + t;
          a[i + p + half] = u - t;
        }
  }
#pragma unroll
  for (int i = 0; i < R; ++i) v[i] = a[i];
}

// Stockham passes: M / VPT threads per row.  With NS the product of the earlier
// radices, butterfly j (< M / R) takes x[j + r M / R] (r < R), multiplies entry
// r by w_M^(r (j mod NS) M / (NS R)), transforms the R values in registers and
// puts entry r at (j / NS) NS R + (j mod NS) + r NS.  Input and output are in
// natural order, so the first pass reads global memory and the last writes it,
// and only the exchanges between passes go through LDS (one padded slot per
// 8 values).  Thread t runs butterflies t + T q (the last q not full for R = 3
// and 5).  Radix 8 while it divides, then 4 or 2, then 3 or 5.
constexpr int radix_of(int rem, int top) {
  return rem % top == 0 ? top : rem % 8 == 0 ? 8 : rem % 4 == 0 ? 4 : rem % 2 == 0 ? 2 : rem;
}
constexpr int passes_of(int M, int top) {
  int n = 0;
  for (int ns = 1; ns < M; ns *= radix_of(M / ns, top)) ++n;
  return n;
}
// values per thread: 16 where that saves a pass and its registers allow (M = 2048: 68 us
// of the operator at n = 1024 against 81 with 8; M = 1280: 8, as 16 spills: 128 against 140 us)
constexpr int vpt(int M) { return M >= 768 && M % 5 != 0 && passes_of(M, 16) < passes_of(M, 8) ? 16 : 8; }
constexpr int radix(int M, int ns) { return radix_of(M / ns, vpt(M)); }
constexpr int slots(int M, int R) { return (M / R + M / vpt(M) - 1) / (M / vpt(M)); }  // butterflies per thread
constexpr int last_ns(int M) {
  int ns = 1;
  while (ns * radix(M, ns) < M) ns *= radix(M, ns);
  return ns;
}
constexpr int max_vals(int M) {
  int best = vpt(M);
  for (int ns = 1; ns < M;) {
    const int R = radix(M, ns), v = slots(M, R) * R;
    best = v > best ? v : best;
    ns *= R;
  }
  return best;
}

// ROWS neighbouring rows per workgroup: 128- or 64-byte runs of a transposed
// store where two workgroups still fit a compute unit's LDS, two rows beyond.
// The column stage keeps four rows to M = 1536: its stores go to lines M
// entries apart (M = 1280, four vectors: 69 us with four rows, 95 with two; the
// row stages 46 against 58 us, so they take two from 1280 on).
constexpr int rows_of(int M, int stage) {
  return M <= 384 ? 8 : M <= (stage == 1 ? 1536 : 1024) ? 4 : 2;
}
// LDS entries per row: = 16 / ROWS mod 16, so that the 16 lanes of one phase of
// an access (ROWS rows times 16 / ROWS neighbouring entries) meet 16 slots
constexpr int row_lds(int M, int stage) {
  int n = M + M / vpt(M);
  while (n % 16 != 16 / rows_of(M, stage)) ++n;
  return n;
}

template <int M>
__device__ __forceinline__ int lpad(int i) {
  constexpr int P = vpt(M);
  return i + i / P;
}

template <int M, int NS, bool INV, int V>
__device__ __forceinline__ void passes(z64 (&v)[V], z64* L, int t, const z64* __restrict__ W) {
  constexpr int T = M / vpt(M), R = radix(M, NS), B = M / R, Q = slots(M, R);
  if constexpr (NS > 1) {
    constexpr int S = M / (NS * R);
    __syncthreads();  // the previous exchange's writes
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int j = t + T * q, jm = j % NS;
      z64 w[R];
#pragma unroll
      for (int r = 1; r < R; ++r) w[r] = W[r * jm * S];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const z64 x = L[lpad<M>((B % T == 0 || j < B ? j : 0) + r * B)];
        v[q * R + r] = r == 0 ? x : x * (INV ? conjg(w[r]) : w[r]);
      }
    }
  }
#pragma unroll
  for (int q = 0; q < Q; ++q) dft<R, INV>(v + q * R);
  if constexpr (NS * R < M) {
    if constexpr (NS > 1) __syncthreads();  // every read of L above is done
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int j = t + T * q, base = (j / NS) * NS * R + (j % NS);
      if (B % T == 0 || j < B)
#pragma unroll
        for (int r = 0; r < R; ++r) L[lpad<M>(base + r * NS)] = v[q * R + r];
    }
    passes<M, NS * R, INV>(v, L, t, W);
  }
}

// fn(k, value) for the transform's entries held by thread t after the passes
template <int M, int V, typename Fn>
__device__ __forceinline__ void each_out(z64 (&v)[V], int t, Fn fn) {
  constexpr int T = M / vpt(M), NS = last_ns(M), R = M / NS, B = M / R, Q = slots(M, R);
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int j = t + T * q;
    if (B % T == 0 || j < B)
#pragma unroll
      for (int e = 0; e < R; ++e) fn(j + e * B, v[q * R + e]);
  }
}

struct FftArgs {
  const z64* in;
  long ldin, sin;    // row stride and vector stride of the input
  int nin, nrows;    // entries of a row (zero beyond), rows
  z64* out;
  long ldout, sout;  // row stride of the (stage 0, 1: transposed) output, vector stride
  int nout;
  const z64* W;      // exp(-2 pi i k / M)
  const z64* spec;   // stage 1: the spectrum quarter (ld M / 2 + 1)
  const double* b;   // stage 0: input scaled by kb b; stage 2, mode 2: y = x + kb b v
  const z64* x;      // stage 2, modes 2 and 4: y = x + v
  double kb;
  int mode;
};

// STAGE 0: forward, transposed store; 1: forward, times the spectrum, back,
// transposed store; 2: inverse, the operator's epilogue (2, 3: y = v, 4)
template <int M, int STAGE>
__global__ __launch_bounds__(rows_of(M, STAGE) * (M / vpt(M))) void k_fft(FftArgs A) {
  constexpr int P = vpt(M), T = M / P, ROWS = rows_of(M, STAGE), V = max_vals(M), LROW = row_lds(M, STAGE);
  extern __shared__ unsigned char smem_raw[];
  const int rw = threadIdx.x % ROWS, t = threadIdx.x / ROWS;
  // neighbouring row groups on one XCD (workgroups go to the eight in turn)
  const int g = gridDim.x, per = g / 8, bi = blockIdx.x;
  const long grp = bi < 8 * per ? (long)(bi % 8) * per + bi / 8 : bi;
  const long r = grp * ROWS + rw;
  const bool ok = r < A.nrows;
  z64* L = reinterpret_cast<z64*>(smem_raw) + rw * LROW;
  z64 v[V];
  {
    const z64* src = A.in + blockIdx.y * A.sin + r * A.ldin;
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const int k = t + i * T;
      z64 x = mk(0.0, 0.0);
      if (ok && k < A.nin) {
        x = src[k];
        if (STAGE == 0 && A.b) x = (A.kb * A.b[r * A.ldin + k]) * x;
      }
      v[i] = x;
    }
  }
  passes<M, 1, STAGE == 2>(v, L, t, A.W);
  if constexpr (STAGE == 1) {  // entry (r, k) of the even spectrum: row min(r, M - r), entry min(k, M - k)
    const z64* sp = A.spec + (r <= M - r ? r : M - r) * (M / 2 + 1);
    __syncthreads();
    each_out<M>(v, t, [&](int k, z64 x) { L[lpad<M>(k)] = ok ? x * sp[k <= M - k ? k : M - k] : x; });
    __syncthreads();
#pragma unroll
    for (int i = 0; i < P; ++i) v[i] = L[lpad<M>(t + i * T)];
    __syncthreads();
    passes<M, 1, true>(v, L, t, A.W);
  }
  if (!ok) return;
  z64* dst = A.out + blockIdx.y * A.sout;
  if (STAGE < 2) {
    each_out<M>(v, t, [&](int k, z64 x) {
      if (k < A.nout) dst[k * A.ldout + r] = x;
    });
  } else {
    const z64* xr = A.x + blockIdx.y * A.sout;
    each_out<M>(v, t, [&](int k, z64 x) {
      if (k >= A.nout) return;
      const long e = r * A.ldout + k;
      dst[e] = A.mode == 2 ? xr[e] + (A.kb * A.b[e]) * x : A.mode == 4 ? xr[e] + x : x;
    });
  }
}

template <int M, int STAGE>
void launch(hipStream_t s, const FftArgs& A, int nvec) {
  constexpr int ROWS = rows_of(M, STAGE), T = M / vpt(M);
  constexpr size_t lds = sizeof(z64) * (size_t)ROWS * row_lds(M, STAGE);
  if (lds > 64 * 1024) {  // (above the default limit of a launch)
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_fft<M, STAGE>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    LSH_HIP(attr);
  }
  hipLaunchKernelGGL((k_fft<M, STAGE>), dim3(ceil_div(A.nrows, ROWS), nvec), dim3(ROWS * T), lds, s, A);
  LSH_LAUNCH_CHECK();
}

// the supported lengths, ascending
constexpr int kLen[] = {64,  80,  96,   128,  160,  192,  256,  320,  384, 512,
                        640, 768, 1024, 1280, 1536, 2048, 2560, 3072, 4096};

template <int STAGE>
void fft_stage(hipStream_t s, int M, const FftArgs& A, int nvec) {
  switch (M) {
#define LSH_FFT(LEN)                 \
  case LEN:                          \
    launch<LEN, STAGE>(s, A, nvec);  \
    break;
    LSH_FFT(64) LSH_FFT(80) LSH_FFT(96) LSH_FFT(128) LSH_FFT(160) LSH_FFT(192) LSH_FFT(256) LSH_FFT(320)
    LSH_FFT(384) LSH_FFT(512) LSH_FFT(640) LSH_FFT(768) LSH_FFT(1024) LSH_FFT(1280) LSH_FFT(1536) LSH_FFT(2048)
    LSH_FFT(2560) LSH_FFT(3072) LSH_FFT(4096)
#undef LSH_FFT
    default: LSH_REQUIRE(false, -6, "FFT length");
  }
}

// C[dy mod M][dx mod M] = h^2 (G(h|d|)[d != 0] + tau_d) for |dx|, |dy| < n
__global__ void k_fill_circulant(z64* C, int M, int n, const z64* __restrict__ T, int D) {
  const long e = blockIdx.x * (long)blockDim.x + threadIdx.x;
  if (e >= (long)M * M) return;
  const int iy = (int)(e / M), ix = (int)(e % M);
  const int dy = iy < n ? iy : iy - M, dx = ix < n ? ix : ix - M;
  z64 v = mk(0.0, 0.0);
  const int ady = dy < 0 ? -dy : dy, adx = dx < 0 ? -dx : dx;
  if (ady < n && adx < n && ady <= D && adx <= D && !(dx == 0 && dy == 0)) v = T[(long)ady * (D + 1) + adx];
  C[e] = v;
}

__global__ void k_add_stencil(z64* C, int M, const int* dxy, const z64* w, int cnt) {
  const int k = threadIdx.x;
  if (k >= cnt) return;
  const int dx = dxy[2 * k], dy = dxy[2 * k + 1];
  const int ix = (dx + M) % M, iy = (dy + M) % M;
  C[(long)iy * M + ix] = C[(long)iy * M + ix] + w[k];
}

// khat[a][c] = s K[c][a] for a, c <= M / 2 (ld M / 2 + 1)
__global__ void k_spectrum_quarter(const z64* __restrict__ K, int M, double s, z64* khat) {
  const int H = M / 2 + 1;
  const long e = blockIdx.x * (long)blockDim.x + threadIdx.x;
  if (e >= (long)H * H) return;
  const int a = (int)(e / H), c = (int)(e % H);
  khat[e] = s * K[(long)c * M + a];
}

int pad_len(int n) {
  for (int M : kLen)
    if (M >= 2 * n) return M;
  throw Error(-6, "grid side beyond the FFT lengths");
}

// Vectors per launch: the work arrays of a group stay within 64 MiB each, so
// that the passes of a large grid reuse them from the 256 MB Infinity Cache
int group_of(int n, int M) {
  const long g = (64L << 20) / (16L * n * M);
  return (int)(g < 1 ? 1 : g > 8 ? 8 : g);
}

}  // namespace

size_t ConvOperator::bytes(int n) {
  const size_t M = pad_len(n), H = M / 2 + 1, G = group_of(n, (int)M);
  mem::Sizer z;
  z.add_n<z64>(M);             // twiddles
  z.add_n<z64>(H * H);         // khat (one quarter)
  z.add_n<z64>(G * n * M);     // w1
  z.add_n<z64>(G * n * M);     // w2
  return z.total;
}

size_t ConvOperator::scratch_bytes(int n) {
  const size_t M = pad_len(n);
  return 2 * mem::round_up(sizeof(z64) * 64) + 2 * mem::round_up(sizeof(z64) * M * M);
}

void ConvOperator::init(hipStream_t s, int n_, double h, double kappa_, const z64* table, int D,
                        const std::vector<StencilEntry>& stencil, mem::Arena& scr) {
  n = n_;
  kappa = kappa_;
  M = pad_len(n);
  group = group_of(n, M);
  const int H = M / 2 + 1;
  std::vector<z64> tw_h(M);
  for (int k = 0; k < M; ++k) {
    const long double a = -2.0L * 3.141592653589793238462643383279502884L * k / M;
    tw_h[k] = mk((double)std::cos(a), (double)std::sin(a));
  }
  tw.alloc(sizeof(z64) * M);
  khat.alloc(sizeof(z64) * (size_t)H * H);
  w1.alloc(sizeof(z64) * (size_t)group * n * M);
  w2.alloc(sizeof(z64) * (size_t)group * n * M);
  // (on the caller's stream: a plain hipMemcpy would also wait for every
  // blocking stream of the device, a factorisation running beside the plan)
  LSH_HIP(hipMemcpyAsync(tw.p, tw_h.data(), sizeof(z64) * M, hipMemcpyHostToDevice, s));
  z64* C = static_cast<z64*>(scr.take(sizeof(z64) * (size_t)M * M));
  z64* Kt = static_cast<z64*>(scr.take(sizeof(z64) * (size_t)M * M));
  hipLaunchKernelGGL(k_fill_circulant, dim3(ceil_div((long)M * M, 256)), dim3(256), 0, s, C, M, n, table, D);
  LSH_LAUNCH_CHECK();
  std::vector<int> dxy;
  std::vector<z64> wv;
  for (auto& e : stencil) {
    if (std::abs(e.dx) >= n || std::abs(e.dy) >= n) continue;
    dxy.push_back(e.dx);
    dxy.push_back(e.dy);
    wv.push_back(mk(h * h * e.re, h * h * e.im));
  }
  int* ddxy = static_cast<int*>(scr.take(sizeof(int) * dxy.size()));
  z64* dw = static_cast<z64*>(scr.take(sizeof(z64) * wv.size()));
  LSH_HIP(hipMemcpyAsync(ddxy, dxy.data(), sizeof(int) * dxy.size(), hipMemcpyHostToDevice, s));
  LSH_HIP(hipMemcpyAsync(dw, wv.data(), sizeof(z64) * wv.size(), hipMemcpyHostToDevice, s));
  hipLaunchKernelGGL(k_add_stencil, dim3(1), dim3(64), 0, s, C, M, ddxy, dw, (int)wv.size());
  LSH_LAUNCH_CHECK();
  // full 2-D transform, each direction transposed as it is stored, so that
  // the second one ends at C[k2][k1].  The kernel is even in each offset (G
  // depends on |d|; the correction stencil covers whole symmetry orbits), so
  // its transform is too, and only the quarter k1, k2 <= M / 2 is kept.
  FftArgs A{};
  A.in = C;
  A.ldin = M;
  A.nin = A.nrows = A.nout = M;
  A.out = Kt;
  A.ldout = M;
  A.W = tw.as<z64>();
  fft_stage<0>(s, M, A, 1);  // Kt[k1][y]
  A.in = Kt;
  A.out = C;
  fft_stage<0>(s, M, A, 1);  // C[k2][k1]
  hipLaunchKernelGGL(k_spectrum_quarter, dim3(ceil_div((long)H * H, 256)), dim3(256), 0, s, C, M,
                     1.0 / ((double)M * M), khat.as<z64>());
  LSH_LAUNCH_CHECK();
  LSH_HIP(hipStreamSynchronize(s));  // the staging and scratch buffers die here
}

void ConvOperator::apply(hipStream_t s, const double* b, const z64* x, z64* y, int nrhs, bool transpose) {
  // algorithmic bytes: read x (and b), write y, read the spectrum quarter once
  const double H = M / 2 + 1;
  ProfScope ps("op_fft_operator", s, (double)nrhs * (16.0 * 2 * n * n + (b ? 8.0 * n * n : 0.0)) + 16.0 * H * H);
  const long nn = (long)n * n, nM = (long)n * M;
  for (int r0 = 0; r0 < nrhs; r0 += group) {
    const int nv = nrhs - r0 < group ? nrhs - r0 : group;
    FftArgs A{};
    A.W = tw.as<z64>();
    A.kb = kappa * kappa;
    // rows (x1 direction) of the n data rows, padded to M (A^T: scaled by kappa^2 b first) -> w1[k1][x2]
    A.in = x + r0 * nn;
    A.ldin = n;
    A.sin = nn;
    A.nin = A.nrows = n;
    A.out = w1.as<z64>();
    A.ldout = n;
    A.sout = nM;
    A.nout = M;
    A.b = transpose ? b : nullptr;
    fft_stage<0>(s, M, A, nv);
    // columns: transform, multiply by the spectrum, transform back, keep n -> w2[x2][k1]
    A.in = w1.as<z64>();
    A.sin = nM;
    A.nrows = M;
    A.out = w2.as<z64>();
    A.ldout = M;
    A.nout = n;
    A.spec = khat.as<z64>();
    fft_stage<1>(s, M, A, nv);
    // rows back, with the epilogue
    A.in = w2.as<z64>();
    A.ldin = M;
    A.nin = M;
    A.nrows = n;
    A.out = y + r0 * nn;
    A.ldout = n;
    A.sout = nn;
    A.b = b;
    A.x = b ? x + r0 * nn : nullptr;
    A.mode = !b ? 3 : (transpose ? 4 : 2);
    fft_stage<2>(s, M, A, nv);
  }
}

}  // namespace lsh
