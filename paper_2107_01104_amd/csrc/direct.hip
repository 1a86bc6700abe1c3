// Interpolation and time steps straight from the stored field, without bins:
// 16 lanes per particle read its I^3 stencil from global memory.
//
// For launches with few particles per field node the tile-column sweep
// (interp.hip) stages far more of the field than the particles' stencils
// touch, and for small launches its time is the sort's and the re-binning's
// chain of launches.  Here a particle costs only its own stencil rows, needs no
// order, and in a frozen field needs no other particle, so a whole advance
// call of tracers is one launch.
//
// The lanes, the order of every sum and the plane references of the FP32
// gradient are those of the sweep (interp_device.h), so both give the same
// bits and the choice between them is invisible in the results.
//
// Bound by the memory pipeline: a particle's 64 rows (I = 8) are 96-byte
// segments at arbitrary 4-byte offsets, about 1.6 cache lines each.  Measured
// against the sort and sweep before it: 2e5 particles on 512^3 (FP32, I = 8,
// value + gradient) 1332 us a call, now 460 (1.2 GB of stencil nodes: 2.6 TB/s);
// 1000 on 32^3 (FP64, I = 4) 71 us, 32 so and 20 since the status words left the
// device; a Heun step of 10^4 on 32^3 as one call 169, 34 and 21 us.
#include "interp_device.h"

namespace ptk {

// node at p (the storage type, 2-, 4- or 8-byte aligned), widened exactly
template <int ST, typename V>
__device__ __forceinline__ void node_load(const unsigned char* p, V* v) {
  if constexpr (ST == ST_F64 || ST == ST_F32) {
    struct N3 {
      V x, y, z;
    };
    const N3 n = *(const N3*)p;
    v[0] = n.x;
    v[1] = n.y;
    v[2] = n.z;
  } else {
    const uint16_t* s = (const uint16_t*)p;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      if constexpr (ST == ST_BF16)
        v[q] = bf16_to_f32(s[q]);
      else
        v[q] = __half2float(__ushort_as_half(s[q]));
    }
  }
}

// u (and the gradient) at x, summed as in the sweep; r as lane_sums leaves it.
// c receives the cell.
template <int ST, int I, bool GRAD, typename V>
__device__ __forceinline__ void direct_sums(const InterpArgs& a, const V* cv, const V* cd, int j, int jj, int h,
                                            const double* x, V* r, int* c) {
  constexpr int HALF = I / 2;
  V t[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    double td;
    locate(x[d], a.N, a.invd, &c[d], &td);
    t[d] = (V)(td - 0.5);
  }
  // padded node coordinates of the stencil are c .. c + I - 1 on every axis
  const unsigned char* base = (const unsigned char*)a.field + (int64_t)(c[2] + h) * a.plane_pitch +
                              (int64_t)c[1] * a.row_pitch + (int64_t)(c[0] + jj) * StoreT<ST>::GB;
  constexpr bool SHIFT = GRAD && ST == ST_F32;
  float4 uc = make_float4(0.f, 0.f, 0.f, 0.f);
  const unsigned char* ref = nullptr;  // reference node of the particle's tile column in plane 0
  if constexpr (SHIFT) {
    constexpr int T = StoreT<ST>::T, TX = T + I - 1;
    const int X = min(c[0] / T * T + TX / 2, (int)a.P - 1), Y = min(c[1] / T * T + TX / 2, (int)a.P - 1);
    ref = (const unsigned char*)a.field + (int64_t)Y * a.row_pitch + (int64_t)X * 12;
    float u[3];
    node_load<ST>(ref + (int64_t)(c[2] + HALF - 1) * a.plane_pitch, u);
    uc = make_float4(u[0], u[1], u[2], 0.f);
  }
  Weights<I, GRAD, V> wt;
  lane_weights(cv, [&](V* o) {
#pragma unroll
    for (int p = 0; p < I; ++p) o[p] = cd[p];
  }, j, h, t[0], t[1], t[2], wt);
  V acc[3] = {0, 0, 0}, ad2[3] = {0, 0, 0}, ad3[3] = {0, 0, 0};
#pragma unroll
  for (int m = 0; m < HALF; ++m) {
    const unsigned char* plane = base + (int64_t)(2 * m) * a.plane_pitch;
    V s[3] = {0, 0, 0}, sd[3] = {0, 0, 0};
    V um[3] = {0, 0, 0};
    if constexpr (SHIFT) {
      node_load<ST>(ref + (int64_t)(c[2] + h + 2 * m) * a.plane_pitch, um);
      s[0] = um[0] - uc.x;
      s[1] = um[1] - uc.y;
      s[2] = um[2] - uc.z;
    }
    V v[I][3];
#pragma unroll
    for (int k = 0; k < I; ++k) node_load<ST>(plane + (int64_t)k * a.row_pitch, v[k]);
#pragma unroll
    for (int k = 0; k < I; ++k) {
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const V f = SHIFT ? v[k][q] - um[q] : v[k][q];
        s[q] = fma(wt.w2[k], f, s[q]);
        if constexpr (GRAD) sd[q] = fma(wt.dw2[k], f, sd[q]);
      }
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      acc[q] = fma(wt.w3[m], s[q], acc[q]);
      if constexpr (GRAD) {
        ad3[q] = fma(wt.dw3[m], s[q], ad3[q]);
        ad2[q] = fma(wt.w3[m], sd[q], ad2[q]);
      }
    }
  }
  lane_sums<GRAD, SHIFT>(wt.w1, wt.d1, acc, ad2, ad3, uc, j, h, r);
}

// the three components of u on every lane, scaled
template <int ST, bool GRAD, typename V>
__device__ __forceinline__ void share_value(const InterpArgs& a, const V* r, V* u) {
  if constexpr (GRAD) {
    u[0] = bcast<0>(r[0]);
    u[1] = bcast<0>(r[1]);
    u[2] = bcast<0>(r[2]);
  } else {
    u[0] = bcast<0>(r[0]);
    u[1] = bcast<4>(r[0]);
    u[2] = bcast<8>(r[0]);
  }
  if constexpr (ST == ST_BF16 || ST == ST_F16) {
#pragma unroll
    for (int q = 0; q < 3; ++q) u[q] *= (V)a.scale[q];
  }
}

// gradient totals r of this lane to row q of a.grad
template <int ST, typename V>
__device__ __forceinline__ void write_grad(const InterpArgs& a, int l16, const V* r, int64_t q) {
  const int sub = l16 & 3, ev = 6 * (l16 >> 3) + 3 * ((l16 >> 2) & 1) + sub;
  if (sub == 3 || ev < 3) return;
  V val = r[0];
  val = sub == 1 ? r[1] : val;
  val = sub == 2 ? r[2] : val;
  val *= (V)a.invd;
  if constexpr (ST == ST_BF16 || ST == ST_F16) val *= (V)(ev < 6 ? a.scale[0] : ev < 9 ? a.scale[1] : a.scale[2]);
  if (a.out_f64)
    ((double*)a.grad)[9 * q + (ev - 3)] = (double)val;
  else
    ((float*)a.grad)[9 * q + (ev - 3)] = (float)val;
}

template <int I, typename V>
__device__ __forceinline__ void table_row(const void* coef, int d, int jj, V* c) {
  const KernelTables* tab = (const KernelTables*)coef;
#pragma unroll
  for (int p = 0; p < I; ++p) {
    if constexpr (sizeof(V) == 8)
      c[p] = d ? tab->cder64[jj][p] : tab->cval64[jj][p];
    else
      c[p] = d ? tab->cder32[jj][p] : tab->cval32[jj][p];
  }
}

constexpr int kDirThreads = 256;
constexpr int kDirGroups = kDirThreads / 16;  // particles per block

// A launch may not reach 2^32 work-items, and a particle takes 16: calls of 2^28
// particles and more (small grids, or I = 4 on the largest) go in slices of
// half that, this launch's from particle a.first on.
constexpr int64_t kDirSlice = (int64_t)1 << 27;
static_assert(kDirSlice % kDirGroups == 0 && kDirSlice * 16 < (int64_t)1 << 32, "whole blocks, below 2^32 work-items");

int64_t direct_slice(int64_t np, int64_t first, unsigned* blocks, int* threads) {
  const int64_t n = np - first < kDirSlice ? np - first : kDirSlice;
  *blocks = (unsigned)((n + kDirGroups - 1) / kDirGroups);
  *threads = kDirThreads;
  return n;
}

template <int ST, int I, bool GRAD>
__global__ __launch_bounds__(kDirThreads) void k_direct(InterpArgs a, BinGeom g, uint32_t* keys) {
  using V = typename StoreT<ST>::acc;
  const int l16 = threadIdx.x & 15, j = l16 & 7, h = l16 >> 3;
  const int jj = j < I ? j : I - 1;
  const int64_t p = a.first + (int64_t)blockIdx.x * kDirGroups + (threadIdx.x >> 4);
  if (p >= a.np) return;  // (whole DPP rows: a particle's 16 lanes stay or leave together)
  const int64_t row = a.xrow ? (int64_t)a.xrow[p] : p;
  double x[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) x[d] = a.X[3 * row + d];
  V cv[I], cd[GRAD ? I : 1];
  table_row<I>(a.coef, 0, jj, cv);
  if constexpr (GRAD) table_row<I>(a.coef, 1, jj, cd);
  const bool ok = in_domain3(x[0], x[1], x[2]);
  int c[3];
  V r[3], u[3];
  direct_sums<ST, I, GRAD>(a, cv, cd, j, jj, h, x, r, c);
  share_value<ST, GRAD>(a, r, u);
  if (l16 == 0) {
    if (!ok) raise_flag(a.flag, kFlagDomain);
    if (keys) keys[p] = ok ? bin_key(c[0], c[1], c[2], g) : 0u;
  }
  const int64_t q = a.orig ? (int64_t)a.orig[p] : p;
  if (a.out && l16 < 3) {
    const V val = l16 == 0 ? u[0] : l16 == 1 ? u[1] : u[2];
    if (a.out_f64)
      ((double*)a.out)[3 * q + l16] = (double)val;
    else
      ((float*)a.out)[3 * q + l16] = (float)val;
  }
  if constexpr (GRAD) write_grad<ST>(a, l16, r, a.grad_orig ? (int64_t)a.grad_orig[p] : q);
}

// nsteps steps of tracers in a frozen field (Heun: the second stage may see
// another field, s.field2), positions and Adams-Bashforth history in place.
// The updates are those of step.hip's k_update, every operation a separately
// rounded binary64 one.  GRAD: the last step evaluates the gradient at its
// start position.
template <int ST, int I, bool GRAD>
__global__ __launch_bounds__(kDirThreads) void k_direct_steps(InterpArgs a, DirectSteps s) {
  using V = typename StoreT<ST>::acc;
  const int l16 = threadIdx.x & 15, j = l16 & 7, h = l16 >> 3;
  const int jj = j < I ? j : I - 1;
  const int64_t p = a.first + (int64_t)blockIdx.x * kDirGroups + (threadIdx.x >> 4);
  // Lanes without a particle leave before any read: positions and history are
  // written in place, and another particle's may be at any moment.  (The empty
  // asm has the arguments that follow fetched together with those the branch
  // waits for; behind it they cost a call of 20 us another 0.3.)
  asm volatile("" ::"s"(a.xrow), "s"(a.coef), "s"(a.field), "s"(a.row_pitch), "s"(a.plane_pitch), "s"(a.invd), "s"(a.N),
               "s"(s.X), "s"(s.hl), "s"(s.nsteps), "s"(s.kind), "s"(s.dt));
  if (p >= a.np) return;
  const int64_t row = a.xrow ? (int64_t)a.xrow[p] : p;
  double x[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) x[d] = s.X[3 * row + d];
  V cv[I];
  table_row<I>(a.coef, 0, jj, cv);
  bool ok = in_domain3(x[0], x[1], x[2]);
  // history: hist[e] = u_{n-1-e}, kept in registers over the steps
  V hist[4][3];
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int d = 0; d < 3; ++d) hist[e][d] = e < s.hl ? ((const V*)s.hist[e])[3 * p + d] : (V)0;
  int hl = s.hl, c[3];
  V r[3], k1[3];
  InterpArgs a2 = a;
  a2.field = s.field2;
#pragma unroll
  for (int q = 0; q < 3; ++q) a2.scale[q] = s.scale2[q];
  auto domain = [&](double& xn) {
    if (!in_domain(xn)) {
      ok = false;
      xn = 0.0;
    }
  };
  for (int n = 0; n < s.nsteps; ++n) {
    bool done = false;
    if constexpr (GRAD) {
      if (n == s.nsteps - 1) {
        V cd[I];
        table_row<I>(a.coef, 1, jj, cd);
        direct_sums<ST, I, true>(a, cv, cd, j, jj, h, x, r, c);
        share_value<ST, true>(a, r, k1);
        write_grad<ST>(a, l16, r, a.grad_orig ? (int64_t)a.grad_orig[p] : p);
        done = true;
      }
    }
    if (!done) {
      direct_sums<ST, I, false>(a, cv, (const V*)nullptr, j, jj, h, x, r, c);
      share_value<ST, false>(a, r, k1);
    }
    if (s.kind == kHeunCorrect) {
      double xs[3];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        xs[d] = x[d] + s.dt * (double)k1[d];
        domain(xs[d]);
      }
      V k2[3];
      direct_sums<ST, I, false>(a2, cv, (const V*)nullptr, j, jj, h, xs, r, c);
      share_value<ST, false>(a2, r, k2);
      const double hdt = 0.5 * s.dt;
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        x[d] = x[d] + hdt * ((double)k1[d] + (double)k2[d]);
        domain(x[d]);
      }
    } else {
      // order q = min(depth, hl + 1); order 1 is Euler
      const int q = min(s.depth, hl + 1);
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        if (q <= 1) {
          x[d] = x[d] + s.dt * (double)k1[d];
        } else {
          double inc = s.b[q - 1][0] * (double)k1[d];
          inc = inc + s.b[q - 1][1] * (double)hist[0][d];
          if (q > 2) inc = inc + s.b[q - 1][2] * (double)hist[1][d];
          if (q > 3) inc = inc + s.b[q - 1][3] * (double)hist[2][d];
          x[d] = x[d] + s.dt * inc;
        }
        domain(x[d]);
#pragma unroll
        for (int e = 3; e > 0; --e) hist[e][d] = hist[e - 1][d];
        hist[0][d] = k1[d];
      }
      hl = min(hl + 1, s.depth);
    }
  }
  if (l16 == 0 && !ok) raise_flag(a.flag, kFlagDomain);
  if (l16 < 3) {
    s.X[3 * row + l16] = l16 == 0 ? x[0] : l16 == 1 ? x[1] : x[2];
    if (s.kind == kAB) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e < hl) ((V*)s.hist[e])[3 * p + l16] = l16 == 0 ? hist[e][0] : l16 == 1 ? hist[e][1] : hist[e][2];
    }
  }
}

template <int ST, int I>
static hipError_t direct_one(InterpArgs a, const BinGeom& g, uint32_t* keys, const DirectSteps* st,
                             hipStream_t s) {
  int64_t n;
  for (a.first = 0; a.first < a.np; a.first += n) {
    unsigned grid;
    int threads;
    n = direct_slice(a.np, a.first, &grid, &threads);
    if (st) {
      if (a.grad)
        k_direct_steps<ST, I, true><<<grid, threads, 0, s>>>(a, *st);
      else
        k_direct_steps<ST, I, false><<<grid, threads, 0, s>>>(a, *st);
    } else if (a.grad) {
      k_direct<ST, I, true><<<grid, threads, 0, s>>>(a, g, keys);
    } else {
      k_direct<ST, I, false><<<grid, threads, 0, s>>>(a, g, keys);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int ST>
static hipError_t direct_st(int I, const InterpArgs& a, const BinGeom& g, uint32_t* keys, const DirectSteps* st,
                            hipStream_t s) {
  switch (I) {
    case 4: return direct_one<ST, 4>(a, g, keys, st, s);
    case 6: return direct_one<ST, 6>(a, g, keys, st, s);
    case 8: return direct_one<ST, 8>(a, g, keys, st, s);
    default: return hipErrorInvalidValue;
  }
}

static hipError_t direct_any(int storage, int I, const InterpArgs& a, const BinGeom& g, uint32_t* keys,
                             const DirectSteps* st, hipStream_t s) {
  if (a.np == 0) return hipSuccess;
  switch (storage) {
    case ST_F64: return direct_st<ST_F64>(I, a, g, keys, st, s);
    case ST_F32: return direct_st<ST_F32>(I, a, g, keys, st, s);
    case ST_BF16: return direct_st<ST_BF16>(I, a, g, keys, st, s);
    case ST_F16: return direct_st<ST_F16>(I, a, g, keys, st, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_direct(int storage, int I, const InterpArgs& a, const BinGeom& g, uint32_t* keys, hipStream_t s) {
  return direct_any(storage, I, a, g, keys, nullptr, s);
}

hipError_t launch_direct_steps(int storage, int I, const InterpArgs& a, const DirectSteps& st, hipStream_t s) {
  return direct_any(storage, I, a, BinGeom{}, nullptr, &st, s);
}

}  // namespace ptk
