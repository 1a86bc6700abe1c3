// The velocity on the grid from its half spectrum, for grids of 2^6 .. 2^10
// points an axis: the inverse real transform in three passes over memory.
//
//   k_fft_cols along k3: reads the caller's spectrum [k2][k3][k1][a], applies
//     the Biot-Savart law to a vorticity spectrum on the way in, writes
//     [x3][k2][k1][a];
//   k_fft_cols along k2, in place: [x3][x2][k1][a];
//   k_fft_rows along k1: each row's three components to real values, written
//     as the stored field's padded, interleaved rows with their periodic
//     copies (FP64 and FP32 storage), or over the row's own amplitudes as grid
//     values (16-bit storage, whose scale needs the whole field first).
//
// The components stay interleaved throughout, as the caller and the stored
// field have them.  Bound by HBM: each pass reads and writes the amplitudes
// once.  A general transform library needs a pass to separate the components
// and apply Biot-Savart and one to pack its planes besides its own passes:
// FP64 vorticity into FP32 storage, 512^3 7.68 ms with rocFFT, 4.17 here (the
// passes 1.49, 1.42 and 1.49 ms under a profiler, at 4.5, 4.6 and 3.4 TB/s);
// 1024^3 81.5 and 33.9 ms (14.5, 10.8 and 9.2).
//
// A column transform of length N = r1 r2 r3 is a Stockham transform in
// registers: a thread holds E elements of one column, the first stage's inputs
// come straight from memory and the last stage's outputs go straight back, and
// between stages the elements change threads through LDS, real parts first and
// then imaginary ones (half the LDS, so twice the workgroups).
//
// Inverse transforms, unnormalised: x_n = sum_k X_k exp(+2 pi i k n / N).
#include <cmath>

#include "device_common.h"
#include "launch.h"

namespace ptk {

namespace {

template <typename R>
struct alignas(2 * sizeof(R)) Cx {
  R x, y;
};
// A number of a buffer that is aligned as its real and imaginary parts are, which
// is all the caller's spectrum has to be (one load either way).
template <typename R>
__device__ __forceinline__ Cx<R> load(const Cx<R>* p) {
  struct Parts {
    R x, y;
  };
  const Parts v = *(const Parts*)p;
  return {v.x, v.y};
}
template <typename R>
__device__ __forceinline__ Cx<R> operator+(Cx<R> a, Cx<R> b) {
  return {a.x + b.x, a.y + b.y};
}
template <typename R>
__device__ __forceinline__ Cx<R> operator-(Cx<R> a, Cx<R> b) {
  return {a.x - b.x, a.y - b.y};
}
template <typename R>
__device__ __forceinline__ Cx<R> cmul(Cx<R> a, Cx<R> b) {
  return {fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x)};
}
template <typename R>
__device__ __forceinline__ Cx<R> times_i(Cx<R> a) {
  return {-a.y, a.x};
}

// a[0..r) -> its inverse transform, in order
template <int r, typename R>
__device__ __forceinline__ void butterfly(Cx<R>* a) {
  static_assert(r == 4 || r == 8 || r == 16, "radix");
  if constexpr (r == 4) {
    const Cx<R> t0 = a[0] + a[2], t1 = a[0] - a[2], t2 = a[1] + a[3], t3 = times_i(a[1] - a[3]);
    a[0] = t0 + t2;
    a[1] = t1 + t3;
    a[2] = t0 - t2;
    a[3] = t1 - t3;
  } else if constexpr (r == 8) {
    const R h = (R)0.70710678118654752440;
    Cx<R> e[4] = {a[0], a[2], a[4], a[6]}, o[4] = {a[1], a[3], a[5], a[7]};
    butterfly<4>(e);
    butterfly<4>(o);
    o[1] = {(o[1].x - o[1].y) * h, (o[1].x + o[1].y) * h};
    o[2] = times_i(o[2]);
    o[3] = {-(o[3].x + o[3].y) * h, (o[3].x - o[3].y) * h};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      a[k] = e[k] + o[k];
      a[k + 4] = e[k] - o[k];
    }
  } else {
    const R c1 = (R)0.92387953251128675613, s1 = (R)0.38268343236508977173, h = (R)0.70710678118654752440;
    Cx<R> m[4][4];
#pragma unroll
    for (int n = 0; n < 4; ++n) {
#pragma unroll
      for (int q = 0; q < 4; ++q) m[n][q] = a[n + 4 * q];
      butterfly<4>(m[n]);
    }
    // times exp(2 pi i n k / 16)
    m[1][1] = cmul(m[1][1], Cx<R>{c1, s1});
    m[1][2] = {(m[1][2].x - m[1][2].y) * h, (m[1][2].x + m[1][2].y) * h};
    m[1][3] = cmul(m[1][3], Cx<R>{s1, c1});
    m[2][1] = {(m[2][1].x - m[2][1].y) * h, (m[2][1].x + m[2][1].y) * h};
    m[2][2] = times_i(m[2][2]);
    m[2][3] = {-(m[2][3].x + m[2][3].y) * h, (m[2][3].x - m[2][3].y) * h};
    m[3][1] = cmul(m[3][1], Cx<R>{s1, c1});
    m[3][2] = {-(m[3][2].x + m[3][2].y) * h, (m[3][2].x - m[3][2].y) * h};
    m[3][3] = cmul(m[3][3], Cx<R>{-c1, -s1});
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      Cx<R> v[4] = {m[0][k], m[1][k], m[2][k], m[3][k]};
      butterfly<4>(v);
#pragma unroll
      for (int q = 0; q < 4; ++q) a[k + 4 * q] = v[q];
    }
  }
}

// Radices of a length
template <int N>
struct Plan;
template <> struct Plan<32> { static constexpr int r1 = 8, r2 = 4, r3 = 1; };
template <> struct Plan<64> { static constexpr int r1 = 8, r2 = 8, r3 = 1; };
template <> struct Plan<128> { static constexpr int r1 = 8, r2 = 4, r3 = 4; };
template <> struct Plan<256> { static constexpr int r1 = 8, r2 = 8, r3 = 4; };
template <> struct Plan<512> { static constexpr int r1 = 8, r2 = 8, r3 = 8; };
template <> struct Plan<1024> { static constexpr int r1 = 16, r2 = 16, r3 = 4; };

// index of element i in a column's LDS copy: a gap after every r1 elements, so
// that the first exchange's writes (r1 apart from thread to thread) spread
// over the banks
template <int N>
__device__ __forceinline__ int lds_index(int i) {
  return i + i / Plan<N>::r1;
}
template <int N>
constexpr int kLdsRows = N + N / Plan<N>::r1;

// One stage of a column held as E elements per thread, T = N / E threads
// (thread t has butterflies t, t + T, ...; element e = u * r + q is input or
// output q of butterfly t + u T).  L: product of the radices before.
// tw: exp(2 pi i j / TN), TN a multiple of N.
template <int N, int E, int r, int L, int TN, typename R>
__device__ __forceinline__ void stage(Cx<R>* v, int t, const Cx<R>* tw) {
  static_assert(E % r == 0, "whole butterflies");
  constexpr int T = N / E;
#pragma unroll
  for (int u = 0; u < E / r; ++u) {
    Cx<R>* a = v + u * r;
    if constexpr (L > 1) {
      // input p is multiplied by w^p, w = exp(2 pi i k / (L r)): powers that
      // need more than one product are not used
      const int k = (t + u * T) % L, s = k * (TN / (L * r));
      if constexpr (r == 4) {
#pragma unroll
        for (int p = 1; p < 4; ++p) a[p] = cmul(a[p], tw[p * s]);
      } else {
        const Cx<R> w1 = tw[s], w2 = tw[2 * s], w3 = tw[3 * s];
        a[1] = cmul(a[1], w1);
        a[2] = cmul(a[2], w2);
        a[3] = cmul(a[3], w3);
#pragma unroll
        for (int p = 4; p < r; p += 4) {
          const Cx<R> w4 = tw[p * s];
          a[p] = cmul(a[p], w4);
          a[p + 1] = cmul(a[p + 1], cmul(w4, w1));
          a[p + 2] = cmul(a[p + 2], cmul(w4, w2));
          a[p + 3] = cmul(a[p + 3], cmul(w4, w3));
        }
      }
    }
    butterfly<r>(a);
  }
}

// index of input q of butterfly b of a stage, and of output q
template <int N, int r>
__device__ __forceinline__ int in_index(int b, int q) {
  return b + q * (N / r);
}
template <int N, int r, int L>
__device__ __forceinline__ int out_index(int b, int q) {
  return b / L * (L * r) + b % L + q * L;
}

// outputs of the stage (r, L) to the inputs of the next (rn), one part at a
// time; NC: columns side by side in LDS
template <int N, int E, int r, int L, int rn, int NC, typename R>
__device__ __forceinline__ void exchange(Cx<R>* v, R* lds, int t) {
  constexpr int T = N / E;
#pragma unroll
  for (int part = 0; part < 2; ++part) {
#pragma unroll
    for (int e = 0; e < E; ++e)
      lds[lds_index<N>(out_index<N, r, L>(t + e / r * T, e % r)) * NC] = part ? v[e].y : v[e].x;
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const R f = lds[lds_index<N>(in_index<N, rn>(t + e / rn * T, e % rn)) * NC];
      if (part)
        v[e].y = f;
      else
        v[e].x = f;
    }
    __syncthreads();
  }
}

// every stage; on return element e is output q = e % r of the last stage's
// butterfly t + (e / r) T, at index in_index<N, rlast>
template <int N, int E, int TN, int NC, typename R>
__device__ __forceinline__ void transform(Cx<R>* v, R* lds, int t, const Cx<R>* tw) {
  using P = Plan<N>;
  stage<N, E, P::r1, 1, TN>(v, t, tw);
  exchange<N, E, P::r1, 1, P::r2, NC>(v, lds, t);
  stage<N, E, P::r2, P::r1, TN>(v, t, tw);
  if constexpr (P::r3 > 1) {
    exchange<N, E, P::r2, P::r1, P::r3, NC>(v, lds, t);
    stage<N, E, P::r3, P::r1 * P::r2, TN>(v, t, tw);
  }
}
template <int N>
constexpr int kLast = Plan<N>::r3 > 1 ? Plan<N>::r3 : Plan<N>::r2;

// Columns per workgroup and elements per thread: whole k1 (3 columns each), 192
// bytes or more of every row where 1024 threads and the LDS allow it.  (Rows'
// pieces are not aligned to cache lines; with 96-byte pieces the passes at
// 512^3 FP64 took 1.84 and 1.60 ms, with 192 1.49 and 1.43: 4.5 TB/s, a large
// copy's rate.)
template <int N, typename R>
constexpr int kColE = N == 1024 ? 16 : 8;
template <int N, typename R>
constexpr int kCols = sizeof(R) == 8 ? (N <= 256 ? 24 : 12) : (N <= 128 ? 48 : N == 256 ? 24 : 12);
// elements per thread of the rows' transforms
constexpr int kRowE = 8;

// Transforms of length N along the rows of `in` (row stride in_row, columns
// contiguous): workgroup = (plane, tile of columns).  Planes are in_plane and
// out_plane apart.  VORT: in is a vorticity spectrum [k2 plane][k3 row]
// [k1][a]; the Biot-Savart law makes it a velocity's.  Consecutive workgroups
// go round-robin to the 8 XCDs, so each XCD is given a contiguous range of
// tiles: neighbouring tiles share cache lines at their edges.
template <typename R, int N, bool VORT>
__global__ __launch_bounds__((kCols<N, R> * (N / kColE<N, R>))) void k_fft_cols(
    const Cx<R>* in, int64_t in_plane, int64_t in_row, Cx<R>* out, int64_t out_plane, int64_t out_row,
    const Cx<R>* __restrict__ tw) {
  using P = Plan<N>;
  constexpr int NC = kCols<N, R>, E = kColE<N, R>, T = N / E, COLS = 3 * (N / 2 + 1);
  constexpr int tiles = (COLS + NC - 1) / NC, total = N * tiles, per = (total + 7) / 8;
  static_assert(NC * T <= 1024 && NC * T % 64 == 0, "workgroup size");
  __shared__ R lds[kLdsRows<N> * NC];
  const int wg = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  if (wg >= total) return;
  const int plane = wg / tiles, tile = wg % tiles;
  const int c = threadIdx.x % NC, t = threadIdx.x / NC, col = tile * NC + c;
  const bool active = col < COLS;
  const Cx<R>* src = in + plane * in_plane + (active ? col : COLS - 1);
  Cx<R> v[E];
  if constexpr (VORT) {
    // u_a = i (k_b w_c - k_c w_b) / |k|^2, (a, b, c) cyclic
    const int k1 = (active ? col : COLS - 1) / 3, a = (active ? col : COLS - 1) % 3;
    const int b = a == 2 ? 0 : a + 1, d = b == 2 ? 0 : b + 1;
    const int n2 = N / 2, k2 = plane;
    const R q1 = (R)k1, q2 = (R)(k2 <= n2 ? k2 : k2 - N);
    Cx<R> wb[E], wd[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const Cx<R>* s = src + in_index<N, P::r1>(t + e / P::r1 * T, e % P::r1) * in_row;
      wb[e] = load(s + (b - a));
      wd[e] = load(s + (d - a));
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int k3 = in_index<N, P::r1>(t + e / P::r1 * T, e % P::r1);
      const R q3 = (R)(k3 <= n2 ? k3 : k3 - N);
      const R kk = q1 * q1 + q2 * q2 + q3 * q3;
      const R qb = a == 0 ? q2 : a == 1 ? q3 : q1, qd = a == 0 ? q3 : a == 1 ? q1 : q2;
      const R cr = qb * wd[e].x - qd * wb[e].x, ci = qb * wd[e].y - qd * wb[e].y;
      const bool zero = k1 == n2 || k2 == n2 || k3 == n2 || kk == (R)0;
      // c / kk: one division, then a correction of each quotient
      const R inv = (R)1 / (zero ? (R)1 : kk);
      R re = ci * inv, im = cr * inv;
      re = fma(fma(-re, kk, ci), inv, re);
      im = fma(fma(-im, kk, cr), inv, im);
      v[e] = zero ? Cx<R>{(R)0, (R)0} : Cx<R>{-re, im};
    }
  } else {
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = load(src + in_index<N, P::r1>(t + e / P::r1 * T, e % P::r1) * in_row);
  }
  transform<N, E, N, NC>(v, lds + c, t, tw);
  if (!active) return;
  Cx<R>* dst = out + plane * out_plane + col;
  constexpr int rl = kLast<N>;
#pragma unroll
  for (int e = 0; e < E; ++e) dst[in_index<N, rl>(t + e / rl * T, e % rl) * out_row] = v[e];
}

// rows per workgroup
template <int N>
constexpr int kRows = N >= 1024 ? 1 : N == 512 ? 2 : N == 256 ? 4 : N == 128 ? 8 : 16;

// The stored rows the real rows go to: the padded field (F the storage type),
// row (x3, x2) at each of its periodic places; or the grid values in R, each row
// at the place of its amplitudes (halo 0, no copies).
struct RowsOut {
  void* field;
  int64_t row_pitch, plane_pitch;  // bytes
  int P, lo;                       // padded extent and nodes below the grid (N and 0: in place)
};

// Real rows of length N from their N/2 + 1 amplitudes [k1][a]: a complex
// transform of length M = N/2 of Z_k = (X_k + conj X_{M-k}) + i exp(2 pi i k/N)
// (X_k - conj X_{M-k}), whose real and imaginary parts are the even and odd
// values.  (The imaginary parts of X_0 and X_M, which a Hermitian spectrum does
// not have, are left out.)  A workgroup's rows are in LDS before it writes any.
template <typename R, int N, typename F>
__global__ __launch_bounds__((kRows<N> * 3 * (N / 2 / kRowE))) void k_fft_rows(
    const Cx<R>* in, int64_t in_row, RowsOut o, const Cx<R>* __restrict__ tw) {
  constexpr int M = N / 2;
  using P = Plan<M>;
  constexpr int E = kRowE, T = M / E, RW = kRows<N>, NT = RW * 3 * T, ROW = 6 * (M + 1);
  static_assert(3 * kLdsRows<M> <= ROW && 3 * N <= ROW, "a row's LDS holds each of its forms");
  __shared__ __attribute__((aligned(16))) R lds[RW * ROW];
  constexpr int64_t groups = (int64_t)N * N / RW, per = (groups + 7) / 8;
  const int64_t wg = (int64_t)(blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (wg >= groups) return;
  const int64_t row0 = wg * RW;  // rows row0 .. row0 + RW - 1 of one plane (RW divides N)
  const int tid = threadIdx.x;
  for (int e = tid; e < RW * 3 * (M + 1); e += NT) {
    const int rw = e / (3 * (M + 1)), x = e - rw * (3 * (M + 1));
    *(Cx<R>*)(lds + rw * ROW + 2 * x) = in[(row0 + rw) * in_row + x];
  }
  __syncthreads();
  const int a = tid % 3, t = tid / 3 % T, rw = tid / (3 * T);
  R* my = lds + rw * ROW;
  Cx<R> v[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int k = in_index<M, P::r1>(t + e / P::r1 * T, e % P::r1);
    Cx<R> x = *(const Cx<R>*)(my + 2 * (3 * k + a)), y = *(const Cx<R>*)(my + 2 * (3 * (M - k) + a));
    if (k == 0) x.y = y.y = (R)0;
    y.y = -y.y;
    v[e] = (x + y) + times_i(cmul(x - y, tw[k]));
  }
  __syncthreads();
  transform<M, E, N, 3>(v, my + a, t, tw);
  constexpr int rl = kLast<M>;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int n = in_index<M, rl>(t + e / rl * T, e % rl);
    my[6 * n + a] = v[e].x;
    my[6 * n + 3 + a] = v[e].y;
  }
  __syncthreads();
  const int x3 = (int)(row0 / N), x2 = (int)(row0 % N);
  for (int q = 0; q < RW; ++q) {
    const R* src = lds + q * ROW;
    // padded coordinates z = x3 + lo (mod N) within [0, P)
    for (int z = (x3 + o.lo) % N; z < o.P; z += N)
      for (int y = (x2 + q + o.lo) % N; y < o.P; y += N) {
        F* dst = (F*)((unsigned char*)o.field + z * o.plane_pitch + y * o.row_pitch);
        for (int e = tid; e < 3 * o.P; e += NT) {
          int i = e - 3 * o.lo;
          i = i < 0 ? i + 3 * N : i >= 3 * N ? i - 3 * N : i;
          dst[e] = (F)src[i];
        }
      }
  }
}

template <typename R, int N>
hipError_t run_fft(const SpecTransform& p, bool vort, hipStream_t s) {
  constexpr int COLS = 3 * (N / 2 + 1), NC = kCols<N, R>, tiles = (COLS + NC - 1) / NC;
  constexpr unsigned grid = (unsigned)((N * tiles + 7) / 8 * 8);
  constexpr int threads = NC * (N / kColE<N, R>);
  const Cx<R>* in = (const Cx<R>*)p.spec;
  Cx<R>* mid = (Cx<R>*)p.mid;
  const Cx<R>* tw = (const Cx<R>*)p.twiddles;
  const int64_t rp = p.mid_row;
  // along k3: [k2][k3][cols] -> [x3][k2][cols]
  if (vort)
    k_fft_cols<R, N, true><<<grid, threads, 0, s>>>(in, (int64_t)N * COLS, COLS, mid, rp, rp * N, tw);
  else
    k_fft_cols<R, N, false><<<grid, threads, 0, s>>>(in, (int64_t)N * COLS, COLS, mid, rp, rp * N, tw);
  // along k2, in place
  k_fft_cols<R, N, false><<<grid, threads, 0, s>>>(mid, rp * N, rp, mid, rp * N, rp, tw);
  const RowsOut o{p.out, p.row_pitch, p.plane_pitch, p.P, p.lo};
  constexpr int RW = kRows<N>, rt = RW * 3 * (N / 2 / kRowE);
  constexpr unsigned rgrid = (unsigned)(((int64_t)N * N / RW + 7) / 8 * 8);
  if (p.out_f64)
    k_fft_rows<R, N, double><<<rgrid, rt, 0, s>>>(mid, rp, o, tw);
  else
    k_fft_rows<R, N, float><<<rgrid, rt, 0, s>>>(mid, rp, o, tw);
  return hipGetLastError();
}

}  // namespace

bool spec_transform_built(int64_t N) { return N == 64 || N == 128 || N == 256 || N == 512 || N == 1024; }

constexpr int64_t kTwiddles = 64 + 128 + 256 + 512 + 1024;

// complex numbers per row of the intermediate: rows start on 128-byte lines
int64_t spec_transform_row(int64_t N, int f64) {
  const int64_t line = f64 ? 8 : 16;
  return (3 * (N / 2 + 1) + line - 1) / line * line;
}

// Tables of every length, FP64 then FP32 ones: length N's starts N - 64 numbers
// into its precision's (64 + 128 + .. + N/2 = N - 64).
size_t spec_twiddle_bytes() { return (size_t)kTwiddles * (16 + 8); }

size_t spec_twiddle_offset(int64_t N, int f64) {
  return f64 ? (size_t)(N - 64) * 16 : (size_t)kTwiddles * 16 + (size_t)(N - 64) * 8;
}

void spec_twiddles(void* host) {
  for (int64_t j = 0; j < 1024; ++j) {
    const long double w = 6.283185307179586476925286766559L * (long double)j / 1024.0L;
    const long double c = cosl(w), s = sinl(w);
    for (int64_t N = 64, step = 16; N <= 1024; N *= 2, step /= 2) {
      if (j % step) continue;
      double* d = (double*)((char*)host + spec_twiddle_offset(N, 1)) + 2 * (j / step);
      float* f = (float*)((char*)host + spec_twiddle_offset(N, 0)) + 2 * (j / step);
      d[0] = (double)c;
      d[1] = (double)s;
      f[0] = (float)c;
      f[1] = (float)s;
    }
  }
}

hipError_t launch_spec_transform(const SpecTransform& p, int64_t N, int f64, int vorticity, hipStream_t s) {
#define PTK_FFT(n) \
  case n: return f64 ? run_fft<double, n>(p, vorticity != 0, s) : run_fft<float, n>(p, vorticity != 0, s);
  switch (N) {
    PTK_FFT(64)
    PTK_FFT(128)
    PTK_FFT(256)
    PTK_FFT(512)
    PTK_FFT(1024)
    default: return hipErrorInvalidValue;
  }
#undef PTK_FFT
}

}  // namespace ptk
