// Learned correction form: stencil features and the I = 4 Lagrange sum at
// particles, and a 195-128-128-3 SiLU network whose two hidden-layer products
// run on the matrix cores (BF16 operands, FP32 sums) -- training (forward,
// backward, Adam) and inference on binned particles.
//
// Matrix-core tiles: v_mfma_f32_32x32x16_bf16.  Lane l holds, of a 32 x 16 A
// tile, row l%32 and the 8 consecutive k starting at 8*(l/32); of a 16 x 32 B
// tile, column l%32 and the same k; of the 32 x 32 FP32 result, column l%32
// and rows 8*(v/4) + 4*(l/32) + v%4 in register v.  In training a workgroup of
// 8 waves takes 64 pairs; in inference a wave takes 32 particles by itself.
#include "device_common.h"
#include "launch.h"
#include "ptk_internal.h"

namespace ptk {

namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

constexpr int NF = kLearnedNFeat;   // 195 features
constexpr int FP = kLearnedPitch;   // 200: global feature row pitch
constexpr int K1 = 208;             // layer-1 k extent, padded to 13 x 16
constexpr int NH = 128, NO = 3;
constexpr int oW1 = 0, oB1 = NH * NF, oW2 = oB1 + NH, oB2 = oW2 + NH * NH, oW3 = oB2 + NH, oB3 = oW3 + NO * NH;
static_assert(oB3 + NO == kLearnedNParams, "parameter layout");
constexpr int ROWS = 64, NT = 256;
// LDS pitches in BF16 elements: rows of 16 x odd bytes, so that 32 lanes
// reading 16 bytes each from 32 consecutive rows cover all banks
constexpr int PX = 216;   // features (K1 + 8)
constexpr int PH = 136;   // hidden activations
constexpr int PT = 72;    // transposed tiles: 64 rows + 8
constexpr int PH2 = 132;  // FP32 h2 rows

__device__ __forceinline__ bf16x8 frag(const uint16_t* base, int pitch, int row, int k) {
  return __builtin_bit_cast(bf16x8, *(const uint4*)(base + row * pitch + k));
}
__device__ __forceinline__ f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
// logistic function through the hardware exponential and reciprocal
__device__ __forceinline__ float sigm(float z) { return __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }
__device__ __forceinline__ float silu(float z) { return z * sigm(z); }
__device__ __forceinline__ float dsilu(float z) {
  const float s = sigm(z);
  return s * (1.0f + z * (1.0f - s));
}
// row of result register v of this lane within a 32-row tile
__device__ __forceinline__ int acc_row(int v, int hi) { return 8 * (v >> 2) + 4 * hi + (v & 3); }

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
// two FP32 values rounded to BF16 (nearest even, one conversion instruction)
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  const bf16x2 v = {(__bf16)lo, (__bf16)hi};
  return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ uint16_t to_bf16(float x) { return __builtin_bit_cast(uint16_t, (__bf16)x); }

// value of lane L of this lane's group of 4
template <int L>
__device__ __forceinline__ int quad_bcast(int v) {
  return __builtin_amdgcn_mov_dpp(v, L * 0x55, 0xF, 0xF, true);
}

__device__ __forceinline__ float quad_sum(float v) {
  v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, true));
  v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x4E, 0xF, 0xF, true));
  return v;
}

// sums over a lane's group of 8 (DPP, every lane gets them) and of 16; shuffles
// through LDS would put an LDS round trip in every step of a phase's tail
template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
  return v + __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float sum8(float v) { return dpp_add<0x141>(dpp_add<0x4E>(dpp_add<0xB1>(v))); }
__device__ __forceinline__ float sum16(float v) { return dpp_add<0x140>(sum8(v)); }

typedef float f32x4a __attribute__((ext_vector_type(4), aligned(4)));

// Steps 1-3 of Sec. 2.2 for the particle of this lane's group of 4: lane k
// (k < 3) locates coordinate k, and the group shares cells and offsets.
// Returns whether this lane's coordinate is inside the domain (lane 3: true).
__device__ __forceinline__ bool locate_quad_x(double x, int k3, int N, double invd, int* c, double* td) {
  const bool ok = k3 == 3 || in_domain(x);
  int cc;
  double tt;
  locate(ok ? x : 0.0, N, invd, &cc, &tt);
  const long long tb = __double_as_longlong(tt);
  int lo = (int)(tb & 0xFFFFFFFFll), hi = (int)(tb >> 32);
#define PTK_Q(d)                                                                                   \
  c[d] = quad_bcast<d>(cc);                                                                        \
  td[d] = __longlong_as_double(((long long)(unsigned)quad_bcast<d>(hi) << 32) | (unsigned)quad_bcast<d>(lo));
  PTK_Q(0) PTK_Q(1) PTK_Q(2)
#undef PTK_Q
  return ok;
}

// the same from the particle's row of X: thread k3 loads coordinate min(k3, 2)
__device__ __forceinline__ bool locate_quad(const double* Xp, int k3, int N, double invd, int* c, double* td) {
  return locate_quad_x(Xp[k3 < 3 ? k3 : 2], k3, N, invd, c, td);
}

// One quarter of a particle's 4 x 4 x 4 stencil (the x3 plane k3): the loads
// of its 4 rows (4 nodes each: 12 consecutive floats, 4-byte aligned), ...
__device__ __forceinline__ void stencil_issue(const LearnedField& f, const int* c, int k3, float4 (&q)[4][3]) {
  const int64_t z = c[2] - 1 + k3 + f.halo_lo;
  const unsigned char* plane = (const unsigned char*)f.field + z * f.plane_pitch;
#pragma unroll
  for (int k2 = 0; k2 < 4; ++k2) {
    const int64_t y = c[1] - 1 + k2 + f.halo_lo;
    const f32x4a* row = (const f32x4a*)((const float*)(plane + y * f.row_pitch) + 3 * (c[0] - 1 + f.halo_lo));
#pragma unroll
    for (int e = 0; e < 3; ++e) {
      const f32x4a r = row[e];
      q[k2][e] = make_float4(r.x, r.y, r.z, r.w);
    }
  }
}

// ... and from them its 48 BF16 features, packed in pairs into fe[24] in
// feature order, and its part of the Lagrange I = 4 sum
__device__ __forceinline__ void stencil_sums(const LearnedField& f, const double* td, int k3, const float4 (&q)[4][3],
                                             uint32_t* fe, float* u) {
  float w[3][4];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const float t = (float)td[d];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float acc = f.l4[j][3];
#pragma unroll
      for (int p = 2; p >= 0; --p) acc = fmaf(acc, t, f.l4[j][p]);
      w[d][j] = acc;
    }
  }
  u[0] = u[1] = u[2] = 0.f;
#pragma unroll
  for (int k2 = 0; k2 < 4; ++k2) {
    const float4 q0 = q[k2][0], q1 = q[k2][1], q2 = q[k2][2];
    const float v[12] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w, q2.x, q2.y, q2.z, q2.w};
    const float w23 = w[2][k3] * w[1][k2];
#pragma unroll
    for (int k1 = 0; k1 < 4; ++k1) {
      const float ww = w23 * w[0][k1];
#pragma unroll
      for (int a = 0; a < 3; ++a) u[a] = fmaf(ww, v[3 * k1 + a], u[a]);
    }
#pragma unroll
    for (int qq = 0; qq < 6; ++qq) fe[6 * k2 + qq] = pack_bf16(v[2 * qq], v[2 * qq + 1]);
  }
}

__device__ __forceinline__ void stencil_plane(const LearnedField& f, const int* c, const double* td, int k3,
                                              uint32_t* fe, float* u) {
  float4 q[4][3];
  stencil_issue(f, c, k3, q);
  stencil_sums(f, td, k3, q, fe, u);
}

// ---------------------------------------------------------------- pairs
// thread = (particle, x3 plane of its stencil); caller order
__global__ __launch_bounds__(NT) void k_pairs(LearnedField f, const double* X, int64_t n, const float* uwide,
                                              uint16_t* feat, float* target, int* flag) {
  const int64_t g = (int64_t)blockIdx.x * NT + threadIdx.x;
  const int64_t p = min(g >> 2, n - 1);
  const int k3 = (int)(g & 3);
  const bool active = (g >> 2) < n;
  int c[3];
  double td[3];
  const bool ok = locate_quad(X + 3 * p, k3, f.N, f.invd, c, td);
  if (active && !ok) raise_flag(flag, kFlagDomain);
  uint32_t fe[24];
  float u[3];
  stencil_plane(f, c, td, k3, fe, u);
#pragma unroll
  for (int a = 0; a < 3; ++a) u[a] = quad_sum(u[a]);
  if (!active) return;
  if (feat) {
    uint2* dst = (uint2*)(feat + p * FP + 48 * k3);
#pragma unroll
    for (int q = 0; q < 12; ++q) dst[q] = make_uint2(fe[2 * q], fe[2 * q + 1]);
    if (k3 == 0) {
      uint32_t* tail = (uint32_t*)(feat + p * FP + 192);
      tail[0] = pack_bf16((float)td[0], (float)td[1]);
      tail[1] = (uint32_t)to_bf16((float)td[2]);
      tail[2] = 0u;
      tail[3] = 0u;
    }
  }
  if (target && k3 == 0) {
#pragma unroll
    for (int a = 0; a < 3; ++a) target[3 * p + a] = uwide[3 * p + a] - u[a];
  }
}

// ---------------------------------------------------------------- forward
// Training's forward pass for the 64 rows whose features are in sX; wave w takes
// hidden units 32 (w % 4) .. and rows 32 (w / 4) ..: h1 (BF16) in sH1 and its
// transpose in sH1t, h2 (FP32) in sH2 (the backward pass reads it by rows), the
// pre-activations' derivatives in ds1 and ds2.  sX and sH2 may alias.
__device__ __forceinline__ void forward_hidden(const uint16_t* sX, uint16_t* sH1, uint16_t* sH1t, float* sH2,
                                               const bf16x8 (&bw1)[13], const bf16x8 (&bw2)[8], float bias1,
                                               float bias2, f32x16& ds1, f32x16& ds2) {
  const int lane = threadIdx.x & 63, ub = (threadIdx.x >> 6) & 3, rt = threadIdx.x >> 8;
  const int r32 = lane & 31, hi = lane >> 5;
  const int J = 32 * ub + r32;
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  // (the A fragment of step s + 1 is read while step s's product runs)
  bf16x8 an = frag(sX, PX, 32 * rt + r32, 8 * hi);
#pragma unroll
  for (int s = 0; s < 13; ++s) {
    const bf16x8 a = an;
    if (s + 1 < 13) an = frag(sX, PX, 32 * rt + r32, 16 * (s + 1) + 8 * hi);
    acc = mfma(a, bw1[s], acc);
  }
#pragma unroll
  for (int v0 = 0; v0 < 16; v0 += 4) {
    float h[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float z = acc[v0 + q] + bias1;
      h[q] = silu(z);
      ds1[v0 + q] = dsilu(z);
    }
    const uint32_t p01 = pack_bf16(h[0], h[1]), p23 = pack_bf16(h[2], h[3]);
    const int r0 = 32 * rt + acc_row(v0, hi);
    sH1[r0 * PH + J] = (uint16_t)p01;
    sH1[(r0 + 1) * PH + J] = (uint16_t)(p01 >> 16);
    sH1[(r0 + 2) * PH + J] = (uint16_t)p23;
    sH1[(r0 + 3) * PH + J] = (uint16_t)(p23 >> 16);
    *(uint2*)(sH1t + J * PT + r0) = make_uint2(p01, p23);
  }
  __syncthreads();  // h1 complete; sX is dead from here on
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  an = frag(sH1, PH, 32 * rt + r32, 8 * hi);
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const bf16x8 a = an;
    if (s + 1 < 8) an = frag(sH1, PH, 32 * rt + r32, 16 * (s + 1) + 8 * hi);
    acc = mfma(a, bw2[s], acc);
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const float z = acc[v] + bias2;
    sH2[(32 * rt + acc_row(v, hi)) * PH2 + J] = silu(z);
    ds2[v] = dsilu(z);
  }
  __syncthreads();  // h2 complete
}

// The BF16 weight copies are kept in the order the fragments are loaded: element
// (unit J, input k) of a layer with KS steps of 16 inputs.  A wave's fragment is
// then 1 KB of consecutive bytes; from row-major copies each of its 64 lanes
// read its own cache line, and the 29 fragments of a training workgroup took
// 14 000 of its 35 000 cycles.
template <int KS>
__device__ __forceinline__ int frag_index(int J, int k) {
  return (((J >> 5) * KS + (k >> 4)) * 64 + ((k >> 3) & 1) * 32 + (J & 31)) * 8 + (k & 7);
}
template <int KS>
__device__ __forceinline__ void load_frags(const uint16_t* w, bf16x8 (&b)[KS]) {
  const int lane = threadIdx.x & 63, ub = (threadIdx.x >> 6) & 3;
#pragma unroll
  for (int s = 0; s < KS; ++s) b[s] = __builtin_bit_cast(bf16x8, ((const uint4*)w)[(ub * KS + s) * 64 + lane]);
}

// ---------------------------------------------------------------- training
// One workgroup: 64 consecutive pairs starting at row0 = 64 * blockIdx.x, eight
// waves (wave w: hidden units 32 (w % 4) .., rows 32 (w / 4) ..).  A workgroup is
// a serial chain of short phases: one takes 11.7 us (24 000 cycles; 15.3 us,
// 35 000, before the fragment order of the weights, the loads ahead of their
// phases and the sums by DPP), 256 of them 21.5 us (24.9), of which the last
// phases' stores of 43 MB of partials are a third.  Four waves on both row tiles
// each take the same time: the phases wait, they do not compute.
// Writes its part of the gradient (parameter layout) to gpart[blockIdx.x] and
// its sum of squared errors to lpart[blockIdx.x].
constexpr int NTB = 512;
__global__ __launch_bounds__(NTB, 2) void k_forward_backward(const uint16_t* feat, const float* target, int64_t batch,
                                                            const float* params, const uint16_t* w1b,
                                                            const uint16_t* w2b, const uint16_t* w2bt, float* gpart,
                                                            float* lpart, const uint16_t* feat_next) {
  // LDS regions (bytes): R0 transposed features [224][PT]; R1 transposed h1
  // [128][PT]; R2 features [64][PX] -> h2 FP32 [64][PH2] -> dz2 [64][PH] +
  // transposed dz2 [128][PT]; R3 h1 [64][PH] -> transposed dz1 [128][PT]
  constexpr int R0 = 224 * PT * 2, R1 = NH * PT * 2;
  constexpr int R2 = ROWS * PH * 2 + NH * PT * 2;  // the largest of its three uses
  static_assert(R2 >= ROWS * PX * 2 && R2 >= ROWS * PH2 * 4, "R2 size");
  constexpr int R3 = NH * PT * 2;
  static_assert(R3 >= ROWS * PH * 2, "R3 size");
  __shared__ __attribute__((aligned(16))) unsigned char lds[R0 + R1 + R2 + R3];
  __shared__ __attribute__((aligned(16))) float sW3[NO * NH];
  __shared__ __attribute__((aligned(16))) float sdy[ROWS * 4];  // [row][a], a quad a row
  __shared__ float sdw3[4 * NO * NH];  // dW3 sums of the four quarters of the rows
  __shared__ float sdb[2 * 2 * NH];    // db2 and db1 sums of the two row tiles
  __shared__ __attribute__((aligned(16))) float sred[NTB / 16];
  uint16_t* sXt = (uint16_t*)lds;
  uint16_t* sH1t = (uint16_t*)(lds + R0);
  unsigned char* r2 = lds + R0 + R1;
  uint16_t* sX = (uint16_t*)r2;
  float* sH2 = (float*)r2;
  uint16_t* sdZ2 = (uint16_t*)r2;
  uint16_t* sdZ2t = (uint16_t*)(r2 + ROWS * PH * 2);
  uint16_t* sH1 = (uint16_t*)(lds + R0 + R1 + R2);
  uint16_t* sdZ1t = sH1;

  const int t = threadIdx.x;
  const int lane = t & 63, wave = t >> 6, ub = wave & 3, rt = wave >> 2, r32 = lane & 31, hi = lane >> 5;
  const int J = 32 * ub + r32;
  const int64_t row0 = (int64_t)blockIdx.x * ROWS;
  float* gp = gpart + (int64_t)blockIdx.x * kLearnedNParams;

  // features -> sX (row-major) and sXt (transposed); entries 195.. are zero.
  // This thread's 16-byte pieces are loaded together (unconditionally, from
  // a clamped address), then stored.
  constexpr int FE = ROWS * (K1 / 8), FI = (FE + NTB - 1) / NTB;
  uint4 fq[FI];
#pragma unroll
  for (int i = 0; i < FI; ++i) {
    const int e = min(t + i * NTB, FE - 1);
    const int r = e / (K1 / 8), k0 = (e % (K1 / 8)) * 8;
    fq[i] = *(const uint4*)(feat + (row0 + r) * FP + (k0 < FP ? k0 : 0));
  }
  // the phases' other global operands, loaded ahead of them: this thread's
  // target, W3 and layer 1's fragments behind the features, layer 2's behind
  // the first barrier
  bf16x8 bw1[13], bw2[8], bw2t[8];
  const int orow = t >> 3, oa = min(t & 7, NO - 1);
  const float bias1 = params[oB1 + J], bias2 = params[oB2 + J], bias3 = params[oB3 + oa];
  const float tgt = target[(row0 + orow) * NO + oa];
  static_assert(NO * NH <= NTB && ROWS * 8 == NTB, "an element of W3 and an eighth of a row per thread");
  const float w3e = params[oW3 + min(t, NO * NH - 1)];
  load_frags(w1b, bw1);
  // the same rows of the next step's batch, read now so that they are in
  // this XCD's L2 when that step's workgroup (same block index, same XCD)
  // starts; their registers are consumed only at the end of the kernel
  uint4 fnext[FI];
  if (feat_next) {
#pragma unroll
    for (int i = 0; i < FI; ++i) {
      const int e = min(t + i * NTB, FE - 1);
      const int r = e / (K1 / 8), k0 = (e % (K1 / 8)) * 8;
      fnext[i] = *(const uint4*)(feat_next + (row0 + r) * FP + (k0 < FP ? k0 : 0));
    }
  }
#pragma unroll
  for (int i = 0; i < FI; ++i) {
    const int e = t + i * NTB;
    if (e >= FE) break;
    const int r = e / (K1 / 8), k0 = (e % (K1 / 8)) * 8;
    uint16_t v[8];
    {
      const uint32_t w[4] = {fq[i].x, fq[i].y, fq[i].z, fq[i].w};
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = k0 < FP ? (uint16_t)(w[j >> 1] >> (16 * (j & 1))) : (uint16_t)0;
    }
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (k0 + j >= NF) v[j] = 0;
    *(uint4*)(sX + r * PX + k0) = make_uint4((uint32_t)v[0] | ((uint32_t)v[1] << 16), (uint32_t)v[2] | ((uint32_t)v[3] << 16),
                                             (uint32_t)v[4] | ((uint32_t)v[5] << 16), (uint32_t)v[6] | ((uint32_t)v[7] << 16));
  }
  if (t < NO * NH) sW3[t] = w3e;
  __syncthreads();  // sX complete
  load_frags(w2b, bw2);
  load_frags(w2bt, bw2t);
  // sXt from sX: item (k, 8 rows from r0) per thread, consecutive threads on
  // consecutive k, so the 2-byte reads of a row are contiguous and the
  // 16-byte writes (row pitch 144 bytes) fall on distinct banks within each
  // quarter-wave; rows k >= K1 are zero
  for (int i = t; i < 224 * (ROWS / 8); i += NTB) {
    const int k = i % 224, r0 = (i / 224) * 8;
    uint16_t v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = k < K1 ? sX[(r0 + j) * PX + k] : (uint16_t)0;
    *(uint4*)(sXt + k * PT + r0) = make_uint4((uint32_t)v[0] | ((uint32_t)v[1] << 16), (uint32_t)v[2] | ((uint32_t)v[3] << 16),
                                              (uint32_t)v[4] | ((uint32_t)v[5] << 16), (uint32_t)v[6] | ((uint32_t)v[7] << 16));
  }
  // (layer 1 reads only sX: its barrier completes sXt too)

  f32x16 ds1, ds2;
  forward_hidden(sX, sH1, sH1t, sH2, bw1, bw2, bias1, bias2, ds1, ds2);

  // output layer, loss and dy = 2 (y - target) / (3 batch): eight threads a row,
  // every eighth quad of hidden units each
  float se = 0.f;
  {
    const int seg = t & 7;
    const float4* h = (const float4*)(sH2 + orow * PH2);
    const float4* w = (const float4*)sW3;
    float y[NO] = {0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < NH / 4; c += 8) {
      const float4 hc = h[c + seg];
#pragma unroll
      for (int a = 0; a < NO; ++a) {
        const float4 wc = w[a * (NH / 4) + c + seg];
        y[a] = fmaf(hc.x, wc.x, y[a]);
        y[a] = fmaf(hc.y, wc.y, y[a]);
        y[a] = fmaf(hc.z, wc.z, y[a]);
        y[a] = fmaf(hc.w, wc.w, y[a]);
      }
    }
#pragma unroll
    for (int a = 0; a < NO; ++a) y[a] = sum8(y[a]);
    if (seg < NO) {
      const float d = bias3 + (seg == 0 ? y[0] : seg == 1 ? y[1] : y[2]) - tgt;
      se = d * d;
      sdy[orow * 4 + seg] = 2.0f * d / (float)(NO * batch);
    }
  }
  se = sum16(se);
  if ((lane & 15) == 0) sred[t >> 4] = se;
  __syncthreads();
  if (t == 0) {
    float l = 0.f;
#pragma unroll
    for (int w = 0; w < NTB / 16; ++w) l += sred[w];
    lpart[blockIdx.x] = l;
  }
  // dW3[a][c] = sum_r dy[r][a] h2[r][c]: thread (c, quarter) sums its quarter of
  // the rows for the three a (the quarters are added after the barrier);
  // db3[a] = sum_r dy[r][a], wave 7 a lane per row
  static_assert(NTB == 4 * NH, "dW3 split");
  {
    const int c = t & (NH - 1), r0 = (t / NH) * (ROWS / 4);
    float g[NO] = {0.f, 0.f, 0.f};
#pragma unroll 8
    for (int r = r0; r < r0 + ROWS / 4; ++r) {
      const float h = sH2[r * PH2 + c];
      const float4 dy = *(const float4*)(sdy + 4 * r);
      g[0] = fmaf(dy.x, h, g[0]);
      g[1] = fmaf(dy.y, h, g[1]);
      g[2] = fmaf(dy.z, h, g[2]);
    }
#pragma unroll
    for (int a = 0; a < NO; ++a) sdw3[(t / NH) * NO * NH + a * NH + c] = g[a];
  }
  if (wave == 7) {
    static_assert(ROWS == 64, "a lane per row");
#pragma unroll
    for (int a = 0; a < NO; ++a) {
      const int g = __builtin_bit_cast(int, sum16(sdy[lane * 4 + a]));
      const float q0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(g, 0)),
                  q1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(g, 16)),
                  q2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(g, 32)),
                  q3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(g, 48));
      if (lane == 0) gp[oB3 + a] = (q0 + q1) + (q2 + q3);
    }
  }
  __syncthreads();  // every read of h2 is done: R2 now takes dz2
  for (int o = t; o < NO * NH; o += NTB)
    gp[oW3 + o] = (sdw3[o] + sdw3[NO * NH + o]) + (sdw3[2 * NO * NH + o] + sdw3[3 * NO * NH + o]);

  // dz2 = (dy W3) * silu'(z2), stored as BF16 row-major and transposed
  {
    const float w30 = sW3[J], w31 = sW3[NH + J], w32 = sW3[2 * NH + J];
    float db = 0.f;
#pragma unroll
    for (int v0 = 0; v0 < 16; v0 += 4) {
      float dz[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int r = 32 * rt + acc_row(v0 + q, hi);
        const float4 dy = *(const float4*)(sdy + 4 * r);
        const float dh = dy.x * w30 + dy.y * w31 + dy.z * w32;
        dz[q] = dh * ds2[v0 + q];
        db += dz[q];
      }
      const uint32_t p01 = pack_bf16(dz[0], dz[1]), p23 = pack_bf16(dz[2], dz[3]);
      const int r0 = 32 * rt + acc_row(v0, hi);
      sdZ2[r0 * PH + J] = (uint16_t)p01;
      sdZ2[(r0 + 1) * PH + J] = (uint16_t)(p01 >> 16);
      sdZ2[(r0 + 2) * PH + J] = (uint16_t)p23;
      sdZ2[(r0 + 3) * PH + J] = (uint16_t)(p23 >> 16);
      *(uint2*)(sdZ2t + J * PT + r0) = make_uint2(p01, p23);
    }
    db += __shfl_xor(db, 32);
    if (hi == 0) sdb[rt * NH + J] = db;
  }
  __syncthreads();

  // dh1 = dz2 W2 (unit J of layer 1), dz1 = dh1 * silu'(z1) -> transposed BF16
  {
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
    for (int s = 0; s < 8; ++s)
      acc = mfma(frag(sdZ2, PH, 32 * rt + r32, 16 * s + 8 * hi), bw2t[s], acc);
    float db = 0.f;
#pragma unroll
    for (int v0 = 0; v0 < 16; v0 += 4) {
      float dz[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        dz[q] = acc[v0 + q] * ds1[v0 + q];
        db += dz[q];
      }
      *(uint2*)(sdZ1t + J * PT + 32 * rt + acc_row(v0, hi)) =
          make_uint2(pack_bf16(dz[0], dz[1]), pack_bf16(dz[2], dz[3]));
    }
    db += __shfl_xor(db, 32);
    if (hi == 0) sdb[(2 + rt) * NH + J] = db;
  }
  // dW2[i][j] = sum_r dz2[r][i] h1[r][j]: rows i of tile ub, column tiles 2 rt
  // and 2 rt + 1
  {
    f32x16 acc[2];
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[q][v] = 0.f;
#pragma unroll
    for (int s = 0; s < ROWS / 16; ++s) {
      const bf16x8 a = frag(sdZ2t, PT, 32 * ub + r32, 16 * s + 8 * hi);
#pragma unroll
      for (int q = 0; q < 2; ++q) acc[q] = mfma(a, frag(sH1t, PT, 32 * (2 * rt + q) + r32, 16 * s + 8 * hi), acc[q]);
    }
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int v = 0; v < 16; ++v)
        gp[oW2 + (32 * ub + acc_row(v, hi)) * NH + 32 * (2 * rt + q) + r32] = acc[q][v];
  }
  __syncthreads();  // dz1 and the bias sums complete
  if (t < NH)
    gp[oB2 + t] = sdb[t] + sdb[NH + t];
  else if (t < 2 * NH)
    gp[oB1 + t - NH] = sdb[NH + t] + sdb[2 * NH + t];
  // dW1[i][f] = sum_r dz1[r][i] x[r][f] for f < 195: of the 7 column tiles, the
  // first four (rt = 0) or the last three
  {
    constexpr int NTP = 4;
    f32x16 acc[NTP];
#pragma unroll
    for (int q = 0; q < NTP; ++q)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[q][v] = 0.f;
    const int nt0 = rt * NTP, ntn = rt == 0 ? NTP : 7 - NTP;
#pragma unroll
    for (int s = 0; s < ROWS / 16; ++s) {
      const bf16x8 a = frag(sdZ1t, PT, 32 * ub + r32, 16 * s + 8 * hi);
#pragma unroll
      for (int q = 0; q < NTP; ++q)
        if (q < ntn) acc[q] = mfma(a, frag(sXt, PT, 32 * (nt0 + q) + r32, 16 * s + 8 * hi), acc[q]);
    }
#pragma unroll
    for (int q = 0; q < NTP; ++q) {
      const int fcol = 32 * (nt0 + q) + r32;
      if (q < ntn && fcol < NF)
#pragma unroll
        for (int v = 0; v < 16; ++v) gp[oW1 + (32 * ub + acc_row(v, hi)) * NF + fcol] = acc[q][v];
    }
  }
  if (feat_next) {
#pragma unroll
    for (int i = 0; i < FI; ++i) asm volatile("" ::"v"(fnext[i].x));
  }
}

// Sum of the workgroups' gradients, then (mode 1) one Adam step with BF16
// copies of W1, W2 (and W2 transposed), (mode 0) the gradient and loss only,
// (mode 2) the BF16 copies only.  A workgroup takes 64 parameters: wave q
// sums the q-th quarter of the partials (consecutive, in order, their loads
// in flight together), and wave 0 adds the four sums in order, so the order
// of every addition is fixed.
constexpr int UPD_E = 64;  // parameters per workgroup of k_update
__global__ __launch_bounds__(NT) void k_update(float* params, float* m, float* v, const float* gpart,
                                               const float* lpart, LearnedUpdate u, uint16_t* w1b, uint16_t* w2b,
                                               uint16_t* w2bt) {
  __shared__ float sq[4][UPD_E];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int e = blockIdx.x * UPD_E + lane;
  if (blockIdx.x == 0 && threadIdx.x == 0 && u.loss_out && u.mode != 2) {
    float l = 0.f;
    for (int w = 0; w < u.nparts; ++w) l += lpart[w];
    u.loss_out[0] = l * u.loss_scale;
  }
  float g = 0.f;
  if (u.mode != 2) {
    const int per = (u.nparts + 3) / 4;
    const int w0 = wave * per, w1 = min(u.nparts, w0 + per);
    if (e < kLearnedNParams) {
      int w = w0;
      for (; w + 16 <= w1; w += 16) {
        float part[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) part[k] = gpart[(int64_t)(w + k) * kLearnedNParams + e];
#pragma unroll
        for (int k = 0; k < 16; ++k) g += part[k];
      }
      for (; w < w1; ++w) g += gpart[(int64_t)w * kLearnedNParams + e];
    }
    sq[wave][lane] = g;
    __syncthreads();
    g = ((sq[0][lane] + sq[1][lane]) + sq[2][lane]) + sq[3][lane];
  }
  if (wave != 0 || e >= kLearnedNParams) return;
  float p = params[e];
  if (u.mode != 2) {
    if (u.mode == 0) {
      u.grad_out[e] = g;
      return;
    }
    const float mm = u.beta1 * m[e] + (1.0f - u.beta1) * g;
    const float vv = u.beta2 * v[e] + (1.0f - u.beta2) * g * g;
    m[e] = mm;
    v[e] = vv;
    p -= u.lr * (mm * u.c1) / (sqrtf(vv * u.c2) + u.eps);
    params[e] = p;
  }
  const uint16_t b = to_bf16(p);
  if (e < oB1) {
    w1b[frag_index<K1 / 16>(e / NF, e % NF)] = b;
  } else if (e >= oW2 && e < oB2) {
    const int j = (e - oW2) / NH, k = (e - oW2) % NH;
    w2b[frag_index<NH / 16>(j, k)] = b;
    w2bt[frag_index<NH / 16>(k, j)] = b;
  }
}

// ---------------------------------------------------------------- inference
// Particles in bin order (the k-th is the caller's orig[k]; orig is required).
// A wave takes 32 particles through the whole network by itself: two lanes per
// particle, lane l = particle l % 32 with the rows 2 (l / 32) and 2 (l / 32) + 1
// of its stencil's planes.  With the weights as the matrix instructions' A
// tile and the particles as B, a lane's 96 stencil values are its B fragments
// of layer 1 as they come from memory, and the hidden units that the result
// leaves in a lane are its B fragments of layer 2: the inputs of both layers
// are summed in the order that this distribution gives (layer1_piece,
// layer2_piece), and no value of a particle leaves its two lanes but the final
// sums.  So the waves need no barriers and share only the weights, in LDS.
// The stencil rows come in coalesced 16-byte pieces and change lanes through the
// wave's own LDS.  12.5e6 particles on 512^3 in the caller's order: 2.79 ms with
// two lanes reading their own rows (a cache access per lane: the address units
// busy 66%), 2.48 so (2.21 with the order of the chunks below); four waves staging 64 particles through LDS, the weights
// in registers, 2.75.  Without its gather it took 1.7 ms; the SiLUs (two
// transcendentals each) and the matrix instructions are not what bounds it, and
// neither more waves (12: 2.60) nor the next chunk's stencil in flight (256
// registers, 2.61) help: the vector, address and LDS pipes are each about half
// busy.
constexpr int INF_WAVES = 8, INF_PART = 32;

// 16-byte piece (unit tile ub, step s, lane) of a layer's A fragments <- pieces
// of the fragment-order copies (frag_index).  Layer 1: input 16 s + 8 hi + e
// stands for feature 48 (s / 3) + 24 hi + 8 (s % 3) + e (s < 12), step 12 for
// features 192 + 8 hi + e.
__device__ __forceinline__ uint4 layer1_piece(const uint4* w1b, int ub, int s, int lane) {
  const int f = s < 12 ? 48 * (s / 3) + 24 * (lane >> 5) + 8 * (s % 3) : 192 + 8 * (lane >> 5);
  return w1b[(ub * (K1 / 16) + (f >> 4)) * 64 + ((f >> 3) & 1) * 32 + (lane & 31)];
}
// Layer 2: the step's inputs e of half hi are the units in registers
// 8 (s % 2) + e of layer 1's tile s / 2: 16 s + 8 (e / 4) + 4 hi + e % 4.
__device__ __forceinline__ uint4 layer2_piece(const uint2* w2b, int ub, int s, int lane) {
  const int hi = lane >> 5, r = lane & 31, base = (ub * (NH / 16) + s) * 64;
  const uint2 a = w2b[2 * (base + r) + hi], b = w2b[2 * (base + 32 + r) + hi];
  return make_uint4(a.x, a.y, b.x, b.y);
}

__global__ __launch_bounds__(64 * INF_WAVES, INF_WAVES / 4) void k_infer(LearnedField f, const double* X, int64_t n,
                                                                         const uint32_t* orig, const float* params,
                                                                         const uint16_t* w1b, const uint16_t* w2b,
                                                                         float* out, int* flag) {
  constexpr int S1 = K1 / 16, S2 = NH / 16;
  __shared__ uint4 sW1[4 * S1 * 64], sW2[4 * S2 * 64];
  __shared__ __attribute__((aligned(16))) float sB1[NH], sB2[NH], sW3[NO * NH];
  __shared__ float4 sQ[INF_WAVES][4 * 3 * INF_PART];  // a wave's stencil plane: [row][particle][16-byte piece]
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, hi = lane >> 5;
  for (int e = t; e < 4 * S1 * 64; e += 64 * INF_WAVES)
    sW1[e] = layer1_piece((const uint4*)w1b, e / (S1 * 64), e / 64 % S1, e & 63);
  for (int e = t; e < 4 * S2 * 64; e += 64 * INF_WAVES)
    sW2[e] = layer2_piece((const uint2*)w2b, e / (S2 * 64), e / 64 % S2, e & 63);
  if (t < NH) {
    sB1[t] = params[oB1 + t];
    sB2[t] = params[oB2 + t];
  }
  if (t < NO * NH) sW3[t] = params[oW3 + t];
  const float b3[NO] = {params[oB3], params[oB3 + 1], params[oB3 + 2]};
  __syncthreads();

  // consecutive workgroups go round-robin to the 8 XCDs: XCD x takes a contiguous
  // range of the chunks and its waves go through it side by side, so that the
  // chunks in flight are neighbouring bins, which share their stencils' lines in
  // the XCD's L2 (a range per workgroup: 512^3 with 1.25e7 particles 2.43 ms,
  // now 2.21; 1024^3 with 1e8 23.6, now 22.4).  The workgroup varies faster
  // than the wave: what is left for the last round is spread over the CUs.
  const int64_t nchunks = (n + INF_PART - 1) / INF_PART;
  const int64_t per_xcd = gridDim.x / 8;
  const int64_t per = (nchunks + 7) / 8, step = per_xcd * INF_WAVES;
  const int64_t ch_end = min(nchunks, ((int64_t)(blockIdx.x & 7) + 1) * per);
  // row indices two chunks ahead, coordinates one chunk ahead (clamped to the
  // last particle; unconditional, so no branch merge waits for them)
  auto row_of = [&](int64_t ch) -> uint32_t { return orig[min(ch * INF_PART + (lane & 31), n - 1)]; };
  int64_t ch = (int64_t)(blockIdx.x & 7) * per + wave * per_xcd + (int64_t)(blockIdx.x >> 3);
  if (ch >= ch_end) return;
  uint32_t row = row_of(ch), row_n = row_of(ch + step);
  double x[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) x[d] = X[3 * (int64_t)row + d];
  for (; ch < ch_end; ch += step) {
    const int64_t p = ch * INF_PART + (lane & 31);
    const uint32_t dst = row;
    int c[3];
    float td[3];
    const bool ok = in_domain3(x[0], x[1], x[2]);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      double tt;
      locate(x[d], f.N, f.invd, &c[d], &tt);
      td[d] = (float)tt;
    }
    if (!ok && p < n) raise_flag(flag, kFlagDomain);
    // the chunk's stencil rows, 48 bytes each, in 16-byte pieces: consecutive
    // lanes take consecutive pieces (row pair by row pair, particle by particle),
    // so a row is one or two cache lines to the memory pipeline and not three
    // lanes' accesses each on its own
    const int64_t own = (int64_t)(c[2] - 1 + f.halo_lo) * f.plane_pitch + (int64_t)(c[1] - 1 + f.halo_lo) * f.row_pitch +
                        12 * (c[0] - 1 + f.halo_lo);
    float4 q[4][2][3];
    {
      const unsigned char* at[3];
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const int j = 64 * i + lane, pj = j % 96 / 3;
        const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)own, pj), up = (uint32_t)__shfl((int)(own >> 32), pj);
        at[i] = (const unsigned char*)f.field + (((int64_t)up << 32) | lo) + j / 96 * f.row_pitch + 16 * (j % 3);
      }
#pragma unroll
      for (int k3 = 0; k3 < 4; ++k3)
#pragma unroll
        for (int pr = 0; pr < 2; ++pr)
#pragma unroll
          for (int i = 0; i < 3; ++i) {
            const f32x4a v = *(const f32x4a*)(at[i] + k3 * f.plane_pitch + 2 * pr * f.row_pitch);
            q[k3][pr][i] = make_float4(v.x, v.y, v.z, v.w);
          }
    }
    // the next chunk's coordinates and the rows after them
    row = row_n;
    row_n = row_of(ch + 2 * step);
#pragma unroll
    for (int d = 0; d < 3; ++d) x[d] = X[3 * (int64_t)row + d];
    // the I = 4 Lagrange sum over this lane's planes
    float w[3][4];
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float acc = f.l4[j][3];
#pragma unroll
        for (int e = 2; e >= 0; --e) acc = fmaf(acc, td[d], f.l4[j][e]);
        w[d][j] = acc;
      }
    float u[3] = {0.f, 0.f, 0.f};
    bf16x8 b[S1];
    {
      uint32_t fe[48];
#pragma unroll
      for (int k3 = 0; k3 < 4; ++k3) {
        // the plane through the wave's LDS (its own instructions are in order):
        // this lane's rows are 2 hi and 2 hi + 1 of its particle.  Rows are 48
        // bytes from particle to particle: 16 lanes read 16 different slots.
        float4* sq = sQ[wave];
#pragma unroll
        for (int pr = 0; pr < 2; ++pr)
#pragma unroll
          for (int i = 0; i < 3; ++i) sq[192 * pr + 64 * i + lane] = q[k3][pr][i];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        float4 g[2][3];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int e = 0; e < 3; ++e) g[i][e] = sq[96 * (2 * hi + i) + 3 * (lane & 31) + e];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const float4 q0 = g[i][0], q1 = g[i][1], q2 = g[i][2];
          const float v[12] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w, q2.x, q2.y, q2.z, q2.w};
          const float w23 = w[2][k3] * (hi ? w[1][2 + i] : w[1][i]);
#pragma unroll
          for (int k1 = 0; k1 < 4; ++k1) {
            const float ww = w23 * w[0][k1];
#pragma unroll
            for (int a = 0; a < 3; ++a) u[a] = fmaf(ww, v[3 * k1 + a], u[a]);
          }
#pragma unroll
          for (int e = 0; e < 6; ++e) fe[12 * k3 + 6 * i + e] = pack_bf16(v[2 * e], v[2 * e + 1]);
        }
      }
#pragma unroll
      for (int s = 0; s < 12; ++s)
        b[s] = __builtin_bit_cast(bf16x8, make_uint4(fe[4 * s], fe[4 * s + 1], fe[4 * s + 2], fe[4 * s + 3]));
      const uint32_t t01 = pack_bf16(td[0], td[1]), t2 = (uint32_t)to_bf16(td[2]);
      b[12] = __builtin_bit_cast(bf16x8, make_uint4(hi ? 0u : t01, hi ? 0u : t2, 0u, 0u));
    }
    // layer 1, two unit tiles at a time; registers v of the result are units
    // 8 (v / 4) + 4 hi + v % 4 of their tile
    bf16x8 h1[S2];
#pragma unroll
    for (int ub = 0; ub < 4; ub += 2) {
      f32x16 acc[2];
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[r][v] = 0.f;
#pragma unroll
      for (int s = 0; s < S1; ++s)
#pragma unroll
        for (int r = 0; r < 2; ++r)
          acc[r] = mfma(__builtin_bit_cast(bf16x8, sW1[((ub + r) * S1 + s) * 64 + lane]), b[s], acc[r]);
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        uint32_t h[8];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float4 bb = *(const float4*)(sB1 + 32 * (ub + r) + 8 * k + 4 * hi);
          h[2 * k] = pack_bf16(silu(acc[r][4 * k] + bb.x), silu(acc[r][4 * k + 1] + bb.y));
          h[2 * k + 1] = pack_bf16(silu(acc[r][4 * k + 2] + bb.z), silu(acc[r][4 * k + 3] + bb.w));
        }
        h1[2 * (ub + r)] = __builtin_bit_cast(bf16x8, make_uint4(h[0], h[1], h[2], h[3]));
        h1[2 * (ub + r) + 1] = __builtin_bit_cast(bf16x8, make_uint4(h[4], h[5], h[6], h[7]));
      }
    }
    // layer 2 and the output layer's sums over this lane's units
    float y[NO] = {0.f, 0.f, 0.f};
#pragma unroll
    for (int ub = 0; ub < 4; ub += 2) {
      f32x16 acc[2];
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[r][v] = 0.f;
#pragma unroll
      for (int s = 0; s < S2; ++s)
#pragma unroll
        for (int r = 0; r < 2; ++r)
          acc[r] = mfma(__builtin_bit_cast(bf16x8, sW2[((ub + r) * S2 + s) * 64 + lane]), h1[s], acc[r]);
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int u0 = 32 * (ub + r) + 8 * k + 4 * hi;
          const float4 bb = *(const float4*)(sB2 + u0);
          const float hh[4] = {silu(acc[r][4 * k] + bb.x), silu(acc[r][4 * k + 1] + bb.y),
                               silu(acc[r][4 * k + 2] + bb.z), silu(acc[r][4 * k + 3] + bb.w)};
#pragma unroll
          for (int a = 0; a < NO; ++a) {
            const float4 ww = *(const float4*)(sW3 + a * NH + u0);
            y[a] = fmaf(hh[0], ww.x, y[a]);
            y[a] = fmaf(hh[1], ww.y, y[a]);
            y[a] = fmaf(hh[2], ww.z, y[a]);
            y[a] = fmaf(hh[3], ww.w, y[a]);
          }
        }
    }
    float r[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const float uu = u[a] + __shfl_xor(u[a], 32), yy = y[a] + __shfl_xor(y[a], 32);
      r[a] = uu + (b3[a] + yy);
    }
    if (hi == 0 && p < n) {
      float* o = out + 3 * (int64_t)dst;
      o[0] = r[0];
      o[1] = r[1];
      o[2] = r[2];
    }
  }
}

// ---------------------------------------------------------------- audit
__global__ void k_stride_gather(const double* X, int64_t stride, int64_t na, double* Xa) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= na) return;
  const int64_t p = i * stride;
  Xa[3 * i] = X[3 * p];
  Xa[3 * i + 1] = X[3 * p + 1];
  Xa[3 * i + 2] = X[3 * p + 2];
}

// sums[0] = sum |out[k i] - uw[i]|^2, sums[1] = sum |uw[i]|^2 in FP64; one block
__global__ __launch_bounds__(1024) void k_audit(const float* out, int64_t stride, int64_t na, const float* uw,
                                                double* sums) {
  __shared__ double se[1024], sr[1024];
  double e = 0.0, r = 0.0;
  for (int64_t i = threadIdx.x; i < na; i += 1024)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const double w = uw[3 * i + a];
      const double d = (double)out[3 * (i * stride) + a] - w;
      e += d * d;
      r += w * w;
    }
  se[threadIdx.x] = e;
  sr[threadIdx.x] = r;
  __syncthreads();
  for (int h = 512; h >= 1; h >>= 1) {
    if ((int)threadIdx.x < h) {
      se[threadIdx.x] += se[threadIdx.x + h];
      sr[threadIdx.x] += sr[threadIdx.x + h];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    sums[0] = se[0];
    sums[1] = sr[0];
  }
}

}  // namespace

hipError_t launch_learned_pairs(const LearnedField& f, const double* X, int64_t n, const float* uwide,
                                uint16_t* feat, float* target, int* flag, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = (4 * n + NT - 1) / NT;
  k_pairs<<<(unsigned)blocks, NT, 0, s>>>(f, X, n, uwide, feat, target, flag);
  return hipGetLastError();
}

hipError_t launch_learned_forward_backward(const uint16_t* feat, const float* target, int64_t batch,
                                           const float* params, const uint16_t* w1b, const uint16_t* w2b,
                                           const uint16_t* w2bt, float* gpart, float* lpart, hipStream_t s,
                                           const uint16_t* feat_next) {
  if (batch <= 0 || batch % ROWS) return hipErrorInvalidValue;
  k_forward_backward<<<(unsigned)(batch / ROWS), NTB, 0, s>>>(feat, target, batch, params, w1b, w2b, w2bt, gpart,
                                                             lpart, feat_next);
  return hipGetLastError();
}

hipError_t launch_learned_update(float* params, float* m, float* v, const float* gpart, const float* lpart,
                                 const LearnedUpdate& u, uint16_t* w1b, uint16_t* w2b, uint16_t* w2bt,
                                 hipStream_t s) {
  const int blocks = (kLearnedNParams + UPD_E - 1) / UPD_E;
  k_update<<<blocks, NT, 0, s>>>(params, m, v, gpart, lpart, u, w1b, w2b, w2bt);
  return hipGetLastError();
}

hipError_t launch_learned_infer(const LearnedField& f, const double* X, int64_t n, const uint32_t* orig,
                                const float* params, const uint16_t* w1b, const uint16_t* w2b, float* out,
                                int* flag, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (!orig) return hipErrorInvalidValue;  // the kernel reads every particle's row through it
  const int64_t nchunks = (n + INF_PART - 1) / INF_PART;
  // one workgroup a CU (the weights fill more than half of its LDS), a multiple
  // of the 8 XCDs
  const int64_t grid = min((nchunks + 7) / 8 * 8, (int64_t)256);
  k_infer<<<(unsigned)grid, 64 * INF_WAVES, 0, s>>>(f, X, n, orig, params, w1b, w2b, out, flag);
  return hipGetLastError();
}

hipError_t launch_stride_gather(const double* X, int64_t stride, int64_t na, double* Xa, hipStream_t s) {
  if (na <= 0) return hipSuccess;
  k_stride_gather<<<(unsigned)((na + 255) / 256), 256, 0, s>>>(X, stride, na, Xa);
  return hipGetLastError();
}

hipError_t launch_audit(const float* out, int64_t stride, int64_t na, const float* uw, double* sums,
                        hipStream_t s) {
  k_audit<<<1, 1024, 0, s>>>(out, stride, na, uw, sums);
  return hipGetLastError();
}

}  // namespace ptk
