// Device helpers shared by the interpolation kernels (interp.hip, direct.hip):
// storage types, DPP moves within a particle's 16 lanes, the weights and the
// sums over the lanes.  Both kernels evaluate a particle through these in the
// same order, so their results agree bit for bit.
#pragma once

#include <type_traits>

#include "device_common.h"
#include "launch.h"
#include "ptk_internal.h"

namespace ptk {

enum { ST_F64 = 0, ST_F32 = 1, ST_BF16 = 2, ST_F16 = 3 };

// 16-bit storage: the nodes are widened to FP32 (exactly) when they are staged
// into the LDS ring, so the sums read the same 16-byte nodes as FP32 storage
// and spend no instruction on conversions; HBM moves the 6-byte nodes.
template <int ST>
struct StoreT {
  using acc = float;
  static constexpr int T = kTileF32;   // tile edge in cells
  static constexpr int NB = 16;        // LDS bytes per node
  static constexpr int GB = 6;         // global (stored) bytes per node
  static constexpr int THREADS = 512;
};
template <>
struct StoreT<ST_F32> {
  using acc = float;
  static constexpr int T = kTileF32;
  static constexpr int NB = 16;
  static constexpr int GB = 12;
  static constexpr int THREADS = 512;
};
template <>
struct StoreT<ST_F64> {
  using acc = double;
  static constexpr int T = kTileF64;
  static constexpr int NB = 32;
  static constexpr int GB = 24;
  static constexpr int THREADS = 512;
};

// ---- DPP helpers (rows of 16 lanes = one particle group).  Every control
// used here reads a lane of the same row, so no lane keeps an old value and
// the moves need no initialised destination.
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
// 64-bit moves: one v_mov_b64_dpp for row_newbcast (the only control DPP
// has for 64-bit operands; the compiler splits the others into two 32-bit
// moves).  A 64-bit broadcast issues as fast as a 32-bit one.
// (the builtin's result is given a 64-bit type explicitly: inside a
// template the front end types the generic builtin's call as int)
template <int CTRL>
__device__ __forceinline__ long dpp64(long v) {
  const long r = __builtin_amdgcn_update_dpp(0L, v, CTRL, 0xF, 0xF, true);
  return r;
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  return __builtin_bit_cast(double, dpp64<CTRL>(__builtin_bit_cast(long, v)));
}
// value of lane L of this row
template <int L, typename V>
__device__ __forceinline__ V bcast(V v) {
  return dpp<0x150 + L>(v);
}
// lanes 0-7 of the row get lane L0's value, lanes 8-15 lane L1's: the second
// move writes only DPP banks 2 and 3 (lanes 8-15) over the first
template <int L0, int L1>
__device__ __forceinline__ float bcast2(float v) {
  const int a = __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x150 + L0, 0xF, 0xF, true);
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(a, __builtin_bit_cast(int, v), 0x150 + L1, 0xF, 0xC, false));
}
template <int L0, int L1>
__device__ __forceinline__ long bcast2_64(long b) {
  const long a = __builtin_amdgcn_update_dpp(0L, b, 0x150 + L0, 0xF, 0xF, true);
  const long r = __builtin_amdgcn_update_dpp(a, b, 0x150 + L1, 0xF, 0xC, false);
  return r;
}
template <int L0, int L1>
__device__ __forceinline__ double bcast2(double v) {
  return __builtin_bit_cast(double, bcast2_64<L0, L1>(__builtin_bit_cast(long, v)));
}

// Reduce-scatter of a particle's three value partials over the 16 lanes of a
// row (lane l16 = j + 8h): after it, lane (h, j) holds the row's total of
// value 2h + (j >> 2) (value 3 is the zero padding), summed over all 16 lanes.
// Five DPP additions instead of three full row sums (twelve).
template <typename V>
__device__ __forceinline__ V rowsum_scatter3(const V* e, int j, int h) {
  const V z = (V)0;
  // lanes l and l^8 (row_ror:8): the h = 0 half keeps values 0, 1, the h = 1
  // half keeps 2 and the padding
  const V k0 = h ? e[2] : e[0], k1 = h ? z : e[1];
  const V s0 = h ? e[0] : e[2], s1 = h ? e[1] : z;
  const V f0 = k0 + dpp<0x128>(s0);
  const V f1 = k1 + dpp<0x128>(s1);
  // lanes j and 7 - j of a half (row_half_mirror): j < 4 keeps f0, j >= 4 f1
  const bool hi = (j & 4) != 0;
  V g = (hi ? f1 : f0) + dpp<0x141>(hi ? f0 : f1);
  g += dpp<0xB1>(g);  // quad_perm [1,0,3,2]
  g += dpp<0x4E>(g);  // quad_perm [2,3,0,1]
  return g;
}

// f(integral_constant<int, K>) for K = B .. E-1
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

template <int NC, typename V>
__device__ __forceinline__ V horner(const V* c, V t) {
  V acc = c[NC - 1];
#pragma unroll
  for (int p = NC - 2; p >= 0; --p) acc = fma(acc, t, c[p]);
  return acc;
}

// Weights of one particle, split over its 16 lanes (lane j + 8h owns the x1
// offset j and the planes k = 2m + h): lanes 0-7 evaluate beta_j(t2), lanes 8-15
// beta_j(t3), all lanes beta_j(t1), and the row shares them with DPP.  cv, cd:
// the lane's rows of the value and derivative tables (cd unused without GRAD).
template <int I, bool GRAD, typename V>
struct Weights {
  V w1, d1, w2[I], dw2[GRAD ? I : 1], w3[I / 2], dw3[GRAD ? I / 2 : 1];
};

template <int I, bool GRAD, typename V, typename CD>
__device__ __forceinline__ void lane_weights(const V* cv, CD&& load_cd, int j, int h, V t1, V t2, V t3,
                                             Weights<I, GRAD, V>& w) {
  constexpr int HALF = I / 2;
  const V tsel = h ? t3 : t2;
  const V wsel = horner<I>(cv, tsel);
  w.w1 = horner<I>(cv, t1);
  if (j >= I) w.w1 = (V)0;
  static_for<0, I>([&](auto K) { w.w2[decltype(K)::value] = bcast<decltype(K)::value>(wsel); });
  static_for<0, HALF>([&](auto M) {
    constexpr int m = decltype(M)::value;
    w.w3[m] = bcast2<8 + 2 * m, 9 + 2 * m>(wsel);
  });
  if constexpr (GRAD) {
    V cd[I];
    load_cd(cd);
    const V dsel = horner<I - 1>(cd, tsel);
    w.d1 = horner<I - 1>(cd, t1);
    if (j >= I) w.d1 = (V)0;
    static_for<0, I>([&](auto K) { w.dw2[decltype(K)::value] = bcast<decltype(K)::value>(dsel); });
    static_for<0, HALF>([&](auto M) {
      constexpr int m = decltype(M)::value;
      w.dw3[m] = bcast2<8 + 2 * m, 9 + 2 * m>(dsel);
    });
  }
}

// The x1 weight and the sum over the particle's 16 lanes.  Values: lane (h, j)
// gets the total of value 2h + (j >> 2) in r[0].  With the gradient: lane l16
// ends with the totals of values 6 (l16 / 8) + 3 ((l16 / 4) & 1) + k, k = 0..2,
// in r[k], where value q < 3 is u_q and 3 + 3q + b is d u_q / d x_b before the
// 1/delta factor.  SHIFT adds the reference value uc back to u.
template <bool GRAD, bool SHIFT, typename V>
__device__ __forceinline__ void lane_sums(V w1, V d1, const V* acc, const V* ad2, const V* ad3, float4 uc, int j, int h,
                                          V* r) {
  V e[GRAD ? 12 : 3];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    e[q] = w1 * acc[q];
    if constexpr (GRAD) {
      e[3 + 3 * q + 0] = d1 * acc[q];
      e[3 + 3 * q + 1] = w1 * ad2[q];
      e[3 + 3 * q + 2] = w1 * ad3[q];
    }
  }
  if constexpr (!GRAD) {
    // lane (h, j) gets the total of value 2h + (j >> 2)
    r[0] = rowsum_scatter3(e, j, h);
  } else {
    // reduce-scatter: lanes l and l^8 split the 12 values 6/6, then lanes j and
    // 7-j of each half split their 6 values 3/3, then each quad sums its 3.
    // Lane l16 ends with the totals of values 6*(l16/8) + 3*((l16/4)&1) + k,
    // k = 0..2, in r[k].
    const int b2 = (j >> 2) & 1;
    V f[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      const V keep = h ? e[6 + k] : e[k];
      const V send = h ? e[k] : e[6 + k];
      f[k] = keep + dpp<0x128>(send);  // row_ror:8, the lane 8 away
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const V keep = b2 ? f[3 + k] : f[k];
      const V send = b2 ? f[k] : f[3 + k];
      V g = keep + dpp<0x141>(send);   // row_half_mirror, lane 7-j
      g += dpp<0xB1>(g);
      g += dpp<0x4E>(g);
      r[k] = g;
    }
    // lanes 0-3 hold the values: add back the particle plane's reference
    if constexpr (SHIFT) {
      if (h == 0 && b2 == 0) {
        r[0] += uc.x;
        r[1] += uc.y;
        r[2] += uc.z;
      }
    }
  }
}

}  // namespace ptk
