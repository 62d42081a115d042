// lbm_closure.hip -- the learned boundary closure (include/lbm_closure.h):
// training-sample gathering on lattices and ensembles, and the network
// trainer (fused forward + backward per 64-row tile on BF16 MFMA with FP32
// accumulation, deterministic gradient reduction, Adam on FP32 masters).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstring>
#include <vector>

#include "lbm.h"
#include "lbm_closure.h"
#include "lbm_device.h"
#include "lbm_host.h"
#include "lbm_launch.h"
#include "lbm_mlp.h"
#include "lbm_sweep.h"

namespace lbm {

using mlp::bf16;
using mlp::bf16x8;
using mlp::f32x4;

// ------------------------------------------------------------------ sampling
__device__ inline void edge_normal(int edge, int& nx_, int& ny_) {
  nx_ = edge == E_LEFT ? -1 : (edge == E_RIGHT ? 1 : 0);
  ny_ = edge == E_BOTTOM ? -1 : (edge == E_TOP ? 1 : 0);
}

template <int S>
__device__ inline void load_node(const LatDesc& L, int parity, int x, int y, typename Codec<S>::R g[9]) {
  using C = Codec<S>;
  const typename C::T* A = static_cast<const typename C::T*>(buf_of(L, parity));
  const int idx = y * L.pitch + x;
#pragma unroll
  for (int i = 0; i < 9; ++i) g[i] = C::dec(A[i * L.plane + idx], L.ds[i]);
}

template <int S>
__device__ void site_features_body(const LatDesc& L, int parity, int x, int y, int edge, float* feat, float* mc) {
  using R = typename Codec<S>::R;
  int enx, eny;
  edge_normal(edge, enx, eny);
  const R rho0 = R(L.rho0);
  const Base<R> base(L);
  const R ref[3] = {R(L.m0[0]), R(L.m0[1]), R(L.m0[2])};
  R mom[3][3];  // depth 0..2 at k = 0
#pragma unroll
  for (int d = 0; d < 3; ++d) {
#pragma unroll
    for (int k = -1; k <= 1; ++k) {
      const int sx = x - d * enx - k * eny, sy = y - d * eny + k * enx;
      R g[9];
      load_node<S>(L, parity, sx, sy, g);
      float f[NODE_FEAT];
      strip_node_features<R>(g, rho0, base, ref, enx, eny, f);
#pragma unroll
      for (int q = 0; q < NODE_FEAT; ++q) feat[(3 * d + k + 1) * NODE_FEAT + q] = f[q];
      if (k == 0) moments<R>(g, rho0, base, mom[d][0], mom[d][1], mom[d][2]);
    }
  }
  // NSBC's m_c with a single normal (eqs. nes_2, nes_3)
  R m[3];
  const R gam = R(L.gamma), beta = R(L.beta);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const R mp = mom[0][c] - gam * normal_diff(mom[0][c], mom[1][c], mom[2][c], L.grad_order);
    m[c] = (R(1) - beta) * mp + beta * ref[c];
  }
  float rn[3], dn[3];
  to_normal_frame<R>(ref, base, enx, eny, rn);
  normal_frame_diff<R>(m, ref, enx, eny, dn);
  const float A = finish_inputs(feat, float(L.rho0), float(L.omega), dn, rn);
  mc[0] = dn[0];
  mc[1] = dn[1];
  mc[2] = dn[2];
  mc[3] = A;
}

// Moments of a site in the (n, t) frame; with `sub` (m_c - m0 and A of the
// previous step) the training residual ((m - m0) - (m_c - m0)) / A, the first
// difference formed at the lattice's precision.
template <int S>
__device__ void site_moments_body(const LatDesc& L, int parity, int x, int y, int edge, const float* sub, float* out) {
  using R = typename Codec<S>::R;
  int enx, eny;
  edge_normal(edge, enx, eny);
  R g[9], m[3];
  load_node<S>(L, parity, x, y, g);
  const Base<R> base(L);
  moments<R>(g, R(L.rho0), base, m[0], m[1], m[2]);
  if (sub) {
    const R ref[3] = {R(L.m0[0]), R(L.m0[1]), R(L.m0[2])};
    float d[3];
    normal_frame_diff<R>(m, ref, enx, eny, d);
#pragma unroll
    for (int c = 0; c < 3; ++c) out[c] = (d[c] - sub[c]) / sub[3];
  } else {
    to_normal_frame<R>(m, base, enx, eny, out);
  }
}

// Decode a site row; false when the strip (depth 0..2, tangential +-1) leaves the lattice.
__device__ inline bool site_of(const int32_t* s, int ens, int count, const LatDesc& single, const LatDesc* descs,
                               const LatDesc*& D, int& x, int& y, int& edge) {
  if (ens) {
    if (s[0] < 0 || s[0] >= count) return false;
    D = descs + s[0];
    x = s[1];
    y = s[2];
    edge = s[3];
  } else {
    D = &single;
    x = s[0];
    y = s[1];
    edge = s[2];
  }
  if (edge < 0 || edge > 3) return false;
  int enx, eny;
  edge_normal(edge, enx, eny);
  for (int d = 0; d < 3; ++d)
    for (int k = -1; k <= 1; ++k) {
      const int sx = x - d * enx - k * eny, sy = y - d * eny + k * enx;
      if (sx < 0 || sx >= D->nx || sy < 0 || sy >= D->ny) return false;
    }
  return true;
}

__global__ void k_site_features(LatDesc single, const LatDesc* __restrict__ descs, int ens, int count, int parity,
                                const int32_t* __restrict__ sites, int n, float* __restrict__ feat,
                                float* __restrict__ mc) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const LatDesc* D;
  int x, y, edge;
  float* f = feat + (size_t)i * mlp::IN;
  float* m = mc + (size_t)i * 4;
  if (!site_of(sites + 4 * i, ens, count, single, descs, D, x, y, edge)) {
    for (int q = 0; q < mlp::IN; ++q) f[q] = NAN;
    m[0] = m[1] = m[2] = m[3] = NAN;
    return;
  }
  const LatDesc L = *D;
  switch (L.store) {
    case ST_F64: site_features_body<ST_F64>(L, parity, x, y, edge, f, m); break;
    case ST_F32: site_features_body<ST_F32>(L, parity, x, y, edge, f, m); break;
    case ST_F16: site_features_body<ST_F16>(L, parity, x, y, edge, f, m); break;
    default: site_features_body<ST_BF16>(L, parity, x, y, edge, f, m); break;
  }
}

__global__ void k_site_moments(LatDesc single, const LatDesc* __restrict__ descs, int ens, int count, int parity,
                               const int32_t* __restrict__ sites, int n, const float* __restrict__ sub,
                               float* __restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const LatDesc* D;
  int x, y, edge;
  float* o = out + (size_t)i * 3;
  if (!site_of(sites + 4 * i, ens, count, single, descs, D, x, y, edge)) {
    o[0] = o[1] = o[2] = NAN;
    return;
  }
  const LatDesc L = *D;
  const float* sb = sub ? sub + (size_t)i * 4 : nullptr;
  switch (L.store) {
    case ST_F64: site_moments_body<ST_F64>(L, parity, x, y, edge, sb, o); break;
    case ST_F32: site_moments_body<ST_F32>(L, parity, x, y, edge, sb, o); break;
    case ST_F16: site_moments_body<ST_F16>(L, parity, x, y, edge, sb, o); break;
    default: site_moments_body<ST_BF16>(L, parity, x, y, edge, sb, o); break;
  }
}

hipError_t launch_site_features(const LatDesc* single, const LatDesc* descs, int count, int parity,
                                const int32_t* sites, int n, float* feat, float* mc, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  LatDesc dummy;
  std::memset(&dummy, 0, sizeof(dummy));
  k_site_features<<<dim3((n + 127) / 128), dim3(128), 0, s>>>(single ? *single : dummy, descs, single ? 0 : 1,
                                                              count, parity, sites, n, feat, mc);
  return hipGetLastError();
}

hipError_t launch_site_moments(const LatDesc* single, const LatDesc* descs, int count, int parity,
                               const int32_t* sites, int n, const float* sub, float* out, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  LatDesc dummy;
  std::memset(&dummy, 0, sizeof(dummy));
  k_site_moments<<<dim3((n + 127) / 128), dim3(128), 0, s>>>(single ? *single : dummy, descs, single ? 0 : 1,
                                                             count, parity, sites, n, sub, out);
  return hipGetLastError();
}

// ------------------------------------------------------------------ trainer
constexpr int NP_PAD = 10624;  // per-block stride of the partial-gradient buffer
constexpr int TB = 64;         // rows of a training tile
constexpr int TTHREADS = 256;  // 4 wavefronts of 16 rows
constexpr int TRAIN_BLOCKS = 256;  // one per CU; each walks tiles b, b + 256, ...
constexpr int train_blocks(int batch) { return (batch + TB - 1) / TB < TRAIN_BLOCKS ? (batch + TB - 1) / TB : TRAIN_BLOCKS; }
constexpr int STAT_BLOCKS = 256;
constexpr int STAT_COLS = mlp::IN + mlp::OUT;

using mlp::bf16x4;
// (vectors in caller memory that is only element-aligned)
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef __bf16 bf16x4u __attribute__((ext_vector_type(4), aligned(2)));

__device__ inline bf16x8 cat(bf16x4 a, bf16x4 b) { return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7); }
__device__ inline bf16x4 to_bf16(f32x4 v) { return bf16x4{(bf16)v[0], (bf16)v[1], (bf16)v[2], (bf16)v[3]}; }

// The trainer's wavefront works on 16 samples in the transposed form: every
// layer is Z^T = W X^T with the weights as the MFMA's A operand, so a lane
// (c = lane mod 16, g = lane div 16) holds, of sample c, the outputs
// 16 n + 4 g + r in accumulator n, element r.  Two such accumulators become the
// B operand of the next layer's K = 32 step (outputs 32 k + 8 g + j) by two row
// swaps between lanes, so no activation crosses LDS on the way forward or
// backward, and every sum runs in the order of forward16.
__device__ inline bf16x8 next_k(bf16x4 lo, bf16x4 hi) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  const u32x2 a = __builtin_bit_cast(u32x2, lo), b = __builtin_bit_cast(u32x2, hi);
  u32x4 o;
#pragma unroll
  for (int d = 0; d < 2; ++d) {
    // rows of 16 lanes (a0 a1 a2 a3), (b0 b1 b2 b3) -> (a0 a2 b0 b2), (a1 a3 b1 b3)
    const auto h = __builtin_amdgcn_permlane32_swap(a[d], b[d], false, false);
    const auto q = __builtin_amdgcn_permlane16_swap(h[0], h[1], false, false);
    o[d] = q[0];
    o[2 + d] = q[1];
  }
  return __builtin_bit_cast(bf16x8, o);
}

// Weights and biases of the forward pass in registers.
struct FwdRegs {
  bf16x8 w1[4][3], w2[4][2], w3[2];
  f32x4 b1[4], b2[4], b3;
  __device__ inline void load(const mlp::Net* net, int g) {
    using namespace mlp;
#pragma unroll
    for (int n = 0; n < 4; ++n) {
#pragma unroll
      for (int k = 0; k < 3; ++k) w1[n][k] = frag_k1(net->W1, IN, 16 * n, 32 * k);
#pragma unroll
      for (int k = 0; k < 2; ++k) w2[n][k] = frag_k1(net->W2, HID, 16 * n, 32 * k);
      b1[n] = *reinterpret_cast<const f32x4*>(net->b1 + 16 * n + 4 * g);
      b2[n] = *reinterpret_cast<const f32x4*>(net->b2 + 16 * n + 4 * g);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) w3[k] = frag_k1(net->W3, HID, 0, 32 * k);
    b3 = *reinterpret_cast<const f32x4*>(net->b3 + 4 * g);
  }
  // x: the lane's 8 inputs 32 k + 8 g + j of sample c; h1, h2: the hidden
  // layers as the next K steps; y: output r of sample c (lanes with g = 0)
  __device__ inline void run(const bf16x8 x[3], bf16x4 h1[4], bf16x4 h2[4], bf16x8 k1[2], bf16x8 k2[2],
                             f32x4& y) const {
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < 3; ++k) z = mlp::mfma(w1[n][k], x[k], z);
      h1[n] = mlp::tanh_bf16(z + b1[n]);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) k1[k] = next_k(h1[2 * k], h1[2 * k + 1]);
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < 2; ++k) z = mlp::mfma(w2[n][k], k1[k], z);
      h2[n] = mlp::tanh_bf16(z + b2[n]);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) k2[k] = next_k(h2[2 * k], h2[2 * k + 1]);
    y = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < 2; ++k) y = mlp::mfma(w3[k], k2[k], y);
    y += b3;
  }
};

// 4 x 4 transpose over the lanes 4 q .. 4 q + 3: lane i = lane mod 4 holds four
// values v[r] of its own sample and leaves with value i of the four lanes'
// samples.  Moved as bits: a non-finite value stays in its column and sample.
// (As a product with a matrix that picks columns an infinite value became NaN in
// all sixteen; a step at a batch of 4096 took 19.6 us with the products, 19.1 so.)
__device__ inline bf16x4 quad_transpose(bf16x4 v) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 d = __builtin_bit_cast(u32x2, v);
  const int i = threadIdx.x & 3;
  const uint32_t in = __builtin_amdgcn_mov_dpp(i < 2 ? d[1] : d[0], 0x4e, 0xf, 0xf, true);  // from lane i ^ 2
  const uint32_t lo = i < 2 ? d[0] : in, hi = i < 2 ? in : d[1];
  const uint32_t lo1 = __builtin_amdgcn_mov_dpp(lo, 0xb1, 0xf, 0xf, true);  // from lane i ^ 1
  const uint32_t hi1 = __builtin_amdgcn_mov_dpp(hi, 0xb1, 0xf, 0xf, true);
  // even lanes: the low halves (own, other); odd lanes: the high halves (other, own)
  const uint32_t sel = i & 1 ? 0x03020706u : 0x05040100u;
  return __builtin_bit_cast(bf16x4, u32x2{__builtin_amdgcn_perm(lo1, lo, sel), __builtin_amdgcn_perm(hi1, hi, sel)});
}

// LDS of the training kernel: the tile's inputs, activations and gradients as
// [column][sample], so that the weight gradients' operands (contraction over
// the 64 samples) are 16-byte reads.
constexpr int TS = TB + 8;
struct TrainLds {
  bf16 x[mlp::IN * TS], h1[mlp::HID * TS], h2[mlp::HID * TS], d1[mlp::HID * TS], d2[mlp::HID * TS], dy[16 * TS];
  float db1[4][mlp::HID], db2[4][mlp::HID], db3[4][4], loss[4];
};

// Forward and backward over the tiles of 64 samples that this block walks;
// writes the block's gradient sums (partial[block][NPARAM]) and its summed
// squared error.  Weight gradients stay in MFMA accumulators over all its
// tiles (wavefront w owns output rows 16 w .. 16 w + 15 of W1 and W2 and columns
// 16 w .. 16 w + 15 of W3), bias gradients in registers.
//
// What bounds it is the length of one tile's serial chain (about 2 us) at small
// batches and tanh at large ones; the weights are fetched once per block, and
// a batch of 65536 writes 256 partials (10.8 MB) instead of 1024.
__global__ __launch_bounds__(TTHREADS) void k_mlp_train(const mlp::Net* __restrict__ net, const bf16* __restrict__ W2t,
                                                       const bf16* __restrict__ X, const float* __restrict__ T,
                                                       int64_t nsrc, const int32_t* __restrict__ rows, int batch,
                                                       int ntiles, float* __restrict__ partial,
                                                       float* __restrict__ ploss) {
  using namespace mlp;
  __shared__ __attribute__((aligned(16))) TrainLds S;
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63, c = l & 15, g = l >> 4;
  const float inv = 2.f / (3.f * (float)batch);

  // source row of this lane's sample (4 lanes share one) in tile t, -1 if none
  auto source = [&](int t) -> int64_t {
    const int r = t * TB + 16 * w + c;
    if (t >= ntiles || r >= batch) return -1;
    const int64_t src = rows ? (int64_t)rows[r] : (int64_t)r;
    return src >= 0 && src < nsrc ? src : -1;
  };
  auto fetch = [&](int64_t src, bf16x8 x[3], float t3[3]) {
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int j = 0; j < 8; ++j) x[k][j] = (bf16)0.f;
    t3[0] = t3[1] = t3[2] = 0.f;
    if (src < 0) return;
#pragma unroll
    for (int k = 0; k < 3; ++k) x[k] = *reinterpret_cast<const bf16x8*>(X + (size_t)src * IN + 32 * k + 8 * g);
    if (g == 0) {
#pragma unroll
      for (int o = 0; o < OUT; ++o) t3[o] = T[(size_t)src * OUT + o];
    }
  };

  int64_t src = source(blockIdx.x);
  FwdRegs F;
  F.load(net, g);
  bf16x8 x[3];
  float t3[3];
  fetch(src, x, t3);
  bf16x8 w2t[4][2], w3t[4];
#pragma unroll
  for (int n = 0; n < 4; ++n) {
#pragma unroll
    for (int k = 0; k < 2; ++k) w2t[n][k] = frag_k1(W2t, HID, 16 * n, 32 * k);
#pragma unroll
    for (int j = 0; j < 8; ++j) w3t[n][j] = g == 0 && j < OUT ? net->W3[(j < OUT ? j : 0) * HID + 16 * n + c] : (bf16)0.f;
  }
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 gw1[6], gw2[4], gw3 = zero, gb1[4], gb2[4], gb3 = zero;
#pragma unroll
  for (int n = 0; n < 6; ++n) gw1[n] = zero;
#pragma unroll
  for (int n = 0; n < 4; ++n) gw2[n] = gb1[n] = gb2[n] = zero;
  float lsum = 0.f;
  // this wavefront's samples 4 (c / 4) .. + 3 of column 16 n + 4 g + c mod 4
  auto put_t = [&](bf16* dst, int n, bf16x4 v) {
    *reinterpret_cast<bf16x4*>(dst + (16 * n + 4 * g + (c & 3)) * TS + 16 * w + (c & ~3)) = quad_transpose(v);
  };
  // [column][sample] operand: columns m0 .. m0 + 15, samples 32 k .. 32 k + 31
  auto col = [&](const bf16* a, int m0, int k) {
    return *reinterpret_cast<const bf16x8*>(a + (m0 + c) * TS + 32 * k + 8 * g);
  };

  for (int t = blockIdx.x; t < ntiles; t += gridDim.x) {
    bf16x4 h1[4], h2[4];
    bf16x8 k1[2], k2[2], kd2[2];
    f32x4 y;
    F.run(x, h1, h2, k1, k2, y);
    // loss and dY = 2 (y - t) / (3 batch); output o of sample c in element o of the lanes with g = 0
    f32x4 dy = zero;
    if (g == 0 && src >= 0) {
#pragma unroll
      for (int o = 0; o < OUT; ++o) {
        const float e = y[o] - t3[o];
        lsum += e * e;
        dy[o] = e * inv;
      }
    }
    gb3 += dy;
    const bf16x4 none = {(bf16)0.f, (bf16)0.f, (bf16)0.f, (bf16)0.f};
    const bf16x8 kdy = cat(to_bf16(dy), none);  // outputs 0..3 in the lanes with g = 0, zero elsewhere
    // the next tile's inputs, in flight over the rest of this one
    src = source(t + gridDim.x);
    bf16x8 xn[3];
    fetch(src, xn, t3);
    // dZ2^T = (W3^T dY^T) * (1 - H2^2), dZ1^T = (W2^T dZ2^T) * (1 - H1^2)
    bf16x4 d1[4], d2[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      f32x4 z = mfma(w3t[n], kdy, zero);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float h = (float)h2[n][r];
        z[r] *= 1.f - h * h;
      }
      gb2[n] += z;
      d2[n] = to_bf16(z);
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) kd2[k] = next_k(d2[2 * k], d2[2 * k + 1]);
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      f32x4 z = zero;
#pragma unroll
      for (int k = 0; k < 2; ++k) z = mfma(w2t[n][k], kd2[k], z);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float h = (float)h1[n][r];
        z[r] *= 1.f - h * h;
      }
      gb1[n] += z;
      d1[n] = to_bf16(z);
    }
    // transposed to [column][sample], as bits throughout
#pragma unroll
    for (int k = 0; k < 3; ++k) {
#pragma unroll
      for (int j = 0; j < 8; ++j) S.x[(32 * k + 8 * g + j) * TS + 16 * w + c] = x[k][j];
      x[k] = xn[k];
    }
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      put_t(S.h1, n, h1[n]);
      put_t(S.h2, n, h2[n]);
      put_t(S.d1, n, d1[n]);
      put_t(S.d2, n, d2[n]);
    }
    put_t(S.dy, 0, to_bf16(dy));
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const bf16x8 a1 = col(S.d1, 16 * w, k), a2 = col(S.d2, 16 * w, k);
#pragma unroll
      for (int n = 0; n < 6; ++n) gw1[n] = mfma(a1, col(S.x, 16 * n, k), gw1[n]);
#pragma unroll
      for (int n = 0; n < 4; ++n) gw2[n] = mfma(a2, col(S.h1, 16 * n, k), gw2[n]);
      gw3 = mfma(col(S.dy, 0, k), col(S.h2, 16 * w, k), gw3);
    }
    __syncthreads();
  }

  // weight gradients: element r of a lane is row 4 g + r, column c of its 16 x 16 tile
  float* P = partial + (size_t)blockIdx.x * NP_PAD;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int m = 16 * w + 4 * g + r;
#pragma unroll
    for (int n = 0; n < 6; ++n) P[OFF_W1 + m * IN + 16 * n + c] = gw1[n][r];
#pragma unroll
    for (int n = 0; n < 4; ++n) P[OFF_W2 + m * HID + 16 * n + c] = gw2[n][r];
    if (4 * g + r < OUT) P[OFF_W3 + (4 * g + r) * HID + 16 * w + c] = gw3[r];
  }
  // bias gradients and the loss: over the 16 lanes that hold a column's samples, then over the wavefronts
  auto over16 = [](float v) {
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) v += __shfl_xor(v, o);
    return v;
  };
#pragma unroll
  for (int n = 0; n < 4; ++n)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float v1 = over16(gb1[n][r]), v2 = over16(gb2[n][r]);
      if (c == 0) {
        S.db1[w][16 * n + 4 * g + r] = v1;
        S.db2[w][16 * n + 4 * g + r] = v2;
      }
    }
#pragma unroll
  for (int o = 0; o < OUT; ++o) {
    const float v = over16(gb3[o]);
    if (l == 0) S.db3[w][o] = v;
  }
  lsum = over16(lsum);
  if (l == 0) S.loss[w] = lsum;
  __syncthreads();
  auto over4 = [](float a, float b, float d, float e) { return (a + b) + (d + e); };
  if (tid < HID) {
    P[OFF_B1 + tid] = over4(S.db1[0][tid], S.db1[1][tid], S.db1[2][tid], S.db1[3][tid]);
    P[OFF_B2 + tid] = over4(S.db2[0][tid], S.db2[1][tid], S.db2[2][tid], S.db2[3][tid]);
  } else if (tid < HID + OUT) {
    const int o = tid - HID;
    P[OFF_B3 + o] = over4(S.db3[0][o], S.db3[1][o], S.db3[2][o], S.db3[3][o]);
  } else if (tid == HID + OUT) {
    ploss[blockIdx.x] = over4(S.loss[0], S.loss[1], S.loss[2], S.loss[3]);
  }
}

// Sum the blocks' gradients; optionally return them, and optionally take an
// Adam step; refresh the BF16 copies and biases of the net.  A block takes 64
// parameters, its 16 wavefronts every 16th partial each (so a partial is one
// coalesced read and at most 16 lie in a thread's chain: one thread per
// parameter walked all of them, 238 us at 1024), added in a fixed order.  The
// last block sums the loss.
constexpr int APPLY_P = 64, APPLY_S = 16;
__global__ __launch_bounds__(APPLY_P* APPLY_S) void k_mlp_apply(
    const float* __restrict__ partial, const float* __restrict__ ploss, int nblocks, int batch,
    float* __restrict__ master, float* __restrict__ am, float* __restrict__ av, int adam, float lr, float bc1,
    float bc2, float* __restrict__ grads_out, float* __restrict__ loss_out, mlp::Net* __restrict__ net,
    bf16* __restrict__ W2t) {
  using namespace mlp;
  __shared__ float sum[APPLY_S][APPLY_P];
  const int q = threadIdx.x % APPLY_P, s = threadIdx.x / APPLY_P;
  const bool loss = blockIdx.x == gridDim.x - 1;
  const int p = loss ? NPARAM : blockIdx.x * APPLY_P + q;
  float g = 0.f;
  if (loss) {
    for (int b = s * APPLY_P + q; b < nblocks; b += APPLY_S * APPLY_P) g += ploss[b];
  } else if (p < NPARAM) {
#pragma unroll 4
    for (int b = s; b < nblocks; b += APPLY_S) g += partial[(size_t)b * NP_PAD + p];
  }
  sum[s][q] = g;
  __syncthreads();
  if (s != 0) return;
  g = 0.f;
#pragma unroll
  for (int k = 0; k < APPLY_S; ++k) g += sum[k][q];
  if (loss) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) g += __shfl_xor(g, o);
    if (q == 0 && loss_out && nblocks > 0) *loss_out = g / (3.f * (float)batch);
    return;
  }
  if (p >= NPARAM) return;
  float w = master[p];
  if (nblocks > 0) {
    if (grads_out) grads_out[p] = g;
    if (adam) {
      const float m = 0.9f * am[p] + 0.1f * g;
      const float v = 0.999f * av[p] + 0.001f * g * g;
      am[p] = m;
      av[p] = v;
      w -= lr * (m / bc1) / (sqrtf(v / bc2) + 1e-8f);
      master[p] = w;
    }
  }
  if (p < OFF_B1) {
    net->W1[p - OFF_W1] = (bf16)w;
  } else if (p < OFF_W2) {
    net->b1[p - OFF_B1] = w;
  } else if (p < OFF_B2) {
    const int k = p - OFF_W2;
    net->W2[k] = (bf16)w;
    W2t[(k % HID) * HID + k / HID] = (bf16)w;
  } else if (p < OFF_W3) {
    net->b2[p - OFF_B2] = w;
  } else if (p < OFF_B3) {
    net->W3[p - OFF_W3] = (bf16)w;
  } else {
    net->b3[p - OFF_B3] = w;
  }
}

__global__ void k_copy_f32(const float* __restrict__ src, int n, float* __restrict__ dst) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src[i];
}

// Outputs of n samples, 16 at a time per wavefront, the weights held in
// registers; bound by tanh (128 per sample), then by reading X once.
constexpr int FWD_BLOCKS = 512;
__global__ __launch_bounds__(TTHREADS) void k_mlp_forward(const mlp::Net* __restrict__ net,
                                                         const bf16* __restrict__ X, int64_t n,
                                                         float* __restrict__ Y) {
  using namespace mlp;
  const int l = threadIdx.x & 63, c = l & 15, g = l >> 4;
  const int64_t stride = (int64_t)gridDim.x * (TTHREADS / 64) * 16;
  int64_t row = ((int64_t)blockIdx.x * (TTHREADS / 64) + (threadIdx.x >> 6)) * 16 + c;
  FwdRegs F;
  F.load(net, g);
  bf16x8 x[3];
  auto fetch = [&](int64_t r) {
    const bf16* p = X + (r < n ? r : n - 1) * IN + 8 * g;
#pragma unroll
    for (int k = 0; k < 3; ++k) x[k] = *reinterpret_cast<const bf16x8*>(p + 32 * k);
  };
  fetch(row);
  for (; row - c < n; row += stride) {
    const bf16x8 xc[3] = {x[0], x[1], x[2]};
    if (row - c + stride < n) fetch(row + stride);
    bf16x4 h1[4], h2[4];
    bf16x8 k1[2], k2[2];
    f32x4 y;
    F.run(xc, h1, h2, k1, k2, y);
    if (g == 0 && row < n) {
#pragma unroll
      for (int o = 0; o < OUT; ++o) Y[row * OUT + o] = y[o];
    }
  }
}

// Column sums and sums of squares (fp64) of the raw inputs and the residuals:
// block b takes the b-th stretch of rows, STAT_ROWS at a time, a thread four
// neighbouring columns of one of them (and STAT_RES threads the residuals),
// then adds its rows' sums in a fixed order.  Bound by reading the samples
// once (300007 rows: 115 MB); with a thread per column it took 331 us.
constexpr int STAT_ROWS = 32, STAT_RES = 63, STAT_Q = mlp::IN / 4;
constexpr int STAT_THREADS = STAT_ROWS * STAT_Q + 64;
__global__ __launch_bounds__(STAT_THREADS) void k_stats_partial(const float* __restrict__ feat,
                                                                const float* __restrict__ resid, int64_t n,
                                                                double* __restrict__ part) {
  using namespace mlp;
  __shared__ double red[STAT_ROWS][IN + 1];
  __shared__ double res[2][64];
  const int tid = threadIdx.x;
  const int64_t per = (n + gridDim.x - 1) / gridDim.x;
  const int64_t r0 = (int64_t)blockIdx.x * per, r1 = r0 + per < n ? r0 + per : n;
  const int rr = tid / STAT_Q, c4 = 4 * (tid - rr * STAT_Q), k = tid - STAT_ROWS * STAT_Q;
  double s[4] = {0.0, 0.0, 0.0, 0.0}, q[4] = {0.0, 0.0, 0.0, 0.0};
  if (k < 0) {
#pragma unroll 4
    for (int64_t r = r0 + rr; r < r1; r += STAT_ROWS) {
      const f32x4u v = *reinterpret_cast<const f32x4u*>(feat + r * IN + c4);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const double d = (double)v[j];
        s[j] += d;
        q[j] += d * d;
      }
    }
  } else {
    if (k < STAT_RES) {
#pragma unroll 4
      for (int64_t i = r0 * OUT + k; i < r1 * OUT; i += STAT_RES) {
        const double d = (double)resid[i];
        s[0] += d;
        q[0] += d * d;
      }
    }
    res[0][k] = s[0];
    res[1][k] = q[0];
  }
  double* P = part + (size_t)blockIdx.x * STAT_COLS * 2;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    __syncthreads();
    if (k < 0) {
#pragma unroll
      for (int j = 0; j < 4; ++j) red[rr][c4 + j] = h ? q[j] : s[j];
    }
    __syncthreads();
    if (tid < IN) {
      double a = 0.0;
#pragma unroll
      for (int r = 0; r < STAT_ROWS; ++r) a += red[r][tid];
      P[2 * tid + h] = a;
    } else if (tid < STAT_COLS) {
      double a = 0.0;
#pragma unroll
      for (int r = 0; r < STAT_RES / OUT; ++r) a += res[h][OUT * r + tid - IN];
      P[2 * tid + h] = a;
    }
  }
}

// Mean, 1/std and output scales from the partial sums.  A strip-node input
// whose spread is below kNoiseFloor of the largest spread of the same moment
// over the nine strip nodes is dropped (weight 0): moments that vanish in
// exact arithmetic at the boundary row (e.g. the odd ones NSBC's
// non-equilibrium bounce-back cancels) hold only rounding noise there, and
// normalising that noise to unit spread would feed the network a
// precision-dependent random input.
constexpr double kNoiseFloor = 1e-3;

constexpr int FINAL_COLS = 128, FINAL_S = 8;
__global__ __launch_bounds__(FINAL_COLS* FINAL_S) void k_stats_final(const double* __restrict__ part, int nblocks,
                                                                    int64_t n, mlp::Net* __restrict__ net) {
  __shared__ double sd_s[mlp::IN];
  __shared__ double sum[FINAL_S][2][FINAL_COLS];
  const int c = threadIdx.x % FINAL_COLS, sl = threadIdx.x / FINAL_COLS;
  double s = 0.0, q = 0.0;
  if (c < STAT_COLS) {
#pragma unroll 8
    for (int b = sl; b < nblocks; b += FINAL_S) {
      s += part[((size_t)b * STAT_COLS + c) * 2];
      q += part[((size_t)b * STAT_COLS + c) * 2 + 1];
    }
  }
  sum[sl][0][c] = s;
  sum[sl][1][c] = q;
  __syncthreads();
  double mean = 0.0, sd = 0.0;
  s = q = 0.0;
  if (sl == 0 && c < STAT_COLS) {
#pragma unroll
    for (int k = 0; k < FINAL_S; ++k) {
      s += sum[k][0][c];
      q += sum[k][1][c];
    }
    mean = s / (double)n;
    const double var = q / (double)n - mean * mean;
    sd = var > 0.0 ? sqrt(var) : 0.0;
    if (c < mlp::IN) sd_s[c] = sd;
  }
  __syncthreads();
  if (sl != 0 || c >= STAT_COLS) return;
  if (c < mlp::IN) {
    // constant inputs (a spread at the fp64 rounding level of the mean) carry nothing
    bool used = c < mlp::NFEAT && sd > 1e-30 && sd > 1e-7 * fabs(mean);
    if (used && c < 9 * NODE_FEAT) {
      const int kind = c % NODE_FEAT;
      double top = 0.0;
      for (int j = 0; j < 9; ++j) top = fmax(top, sd_s[NODE_FEAT * j + kind]);
      used = sd > kNoiseFloor * top;
    }
    net->feat_mean[c] = used ? (float)mean : 0.f;
    net->feat_inv_std[c] = used ? (float)(1.0 / sd) : 0.f;
  } else {
    const double rms = sqrt(q / (double)n);
    net->out_scale[c - mlp::IN] = (float)(rms > 1e-30 ? rms : 1e-30);
  }
}

// Four neighbouring inputs of a row per thread, PACK_ROWS rows at a time (a
// thread keeps its columns' normalisation); bound by reading the samples and
// writing the packed ones (300007 rows: 180 MB, 62 us with a value per thread).
constexpr int PACK_ROWS = 8, PACK_THREADS = PACK_ROWS * mlp::IN / 4;
__global__ __launch_bounds__(PACK_THREADS) void k_pack(const mlp::Net* __restrict__ net,
                                                       const float* __restrict__ feat,
                                                       const float* __restrict__ resid, int64_t n,
                                                       bf16* __restrict__ x, float* __restrict__ t) {
  const int rr = threadIdx.x / (mlp::IN / 4), c = 4 * (threadIdx.x - rr * (mlp::IN / 4));
  float mean[4], inv[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    mean[j] = net->feat_mean[c + j];
    inv[j] = net->feat_inv_std[c + j];
  }
  const int64_t step = (int64_t)gridDim.x * PACK_ROWS;
#pragma unroll 4
  for (int64_t r = (int64_t)blockIdx.x * PACK_ROWS + rr; r < n; r += step) {
    const f32x4u v = *reinterpret_cast<const f32x4u*>(feat + r * mlp::IN + c);
    bf16x4u o;
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j] = (bf16)((v[j] - mean[j]) * inv[j]);
    *reinterpret_cast<bf16x4u*>(x + r * mlp::IN + c) = o;
  }
  if (!resid || !t) return;
  const int64_t all = n * mlp::OUT, ts = (int64_t)gridDim.x * PACK_THREADS;
  for (int64_t i = (int64_t)blockIdx.x * PACK_THREADS + threadIdx.x; i < all; i += ts)
    t[i] = resid[i] / net->out_scale[i % mlp::OUT];
}

__global__ void k_init_net(mlp::Net* __restrict__ net) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < mlp::OUT_PAD * mlp::HID) net->W3[i] = (bf16)0.f;
  if (i < mlp::OUT_PAD) net->b3[i] = 0.f;
  if (i < mlp::IN) {
    net->feat_mean[i] = 0.f;
    net->feat_inv_std[i] = i < mlp::NFEAT ? 1.f : 0.f;
  }
  if (i < 4) net->out_scale[i] = 1.f;
  if (i == 0) {
    net->trust = 0.f;
    net->kmin = 0.f;
  }
}

// Trust bound and gain of an exported blob: the gain scales the output scales
// (an under-relaxed correction for gain < 1).
__global__ void k_export_finish(mlp::Net* __restrict__ net, float trust, float gain, float kmin) {
  const int i = threadIdx.x;
  if (i < mlp::OUT) net->out_scale[i] *= gain;
  if (i == 0) {
    net->trust = trust;
    net->kmin = kmin;
  }
}

}  // namespace lbm

// ---------------------------------------------------------------------- C ABI
namespace {

using lbm::host::fail;

#define HIPCHK(expr)                                                                        \
  do {                                                                                      \
    hipError_t e_ = (expr);                                                                 \
    if (e_ != hipSuccess) return fail(LBM_ERR_HIP, "%s: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

struct MlpLayout {
  size_t off_master, off_m, off_v, off_net, off_w2t, off_partial, off_ploss, off_stats, off_grads, total;
};

MlpLayout mlp_layout(int32_t max_batch) {
  using lbm::host::round_up;
  MlpLayout L;
  size_t o = 0;
  const size_t np = sizeof(float) * lbm::NP_PAD;
  L.off_master = o;
  o = round_up(o + np, 256);
  L.off_m = o;
  o = round_up(o + np, 256);
  L.off_v = o;
  o = round_up(o + np, 256);
  L.off_net = o;
  o = round_up(o + sizeof(lbm::mlp::Net), 256);
  L.off_w2t = o;
  o = round_up(o + sizeof(lbm::mlp::bf16) * lbm::mlp::HID * lbm::mlp::HID, 256);
  const size_t blocks = (size_t)lbm::train_blocks(max_batch);
  L.off_partial = o;
  o = round_up(o + np * blocks, 256);
  L.off_ploss = o;
  o = round_up(o + sizeof(float) * blocks, 256);
  L.off_stats = o;
  o = round_up(o + sizeof(double) * 2 * lbm::STAT_COLS * lbm::STAT_BLOCKS, 256);
  L.off_grads = o;
  o = round_up(o + np, 256);
  L.total = o;
  return L;
}

}  // namespace

struct lbm_mlp {
  int32_t max_batch = 0;
  hipStream_t stream = nullptr;
  char* ws = nullptr;
  MlpLayout lay;
  int64_t step = 0;
  float* master() { return reinterpret_cast<float*>(ws + lay.off_master); }
  float* am() { return reinterpret_cast<float*>(ws + lay.off_m); }
  float* av() { return reinterpret_cast<float*>(ws + lay.off_v); }
  lbm::mlp::Net* net() { return reinterpret_cast<lbm::mlp::Net*>(ws + lay.off_net); }
  lbm::mlp::bf16* w2t() { return reinterpret_cast<lbm::mlp::bf16*>(ws + lay.off_w2t); }
  float* partial() { return reinterpret_cast<float*>(ws + lay.off_partial); }
  float* ploss() { return reinterpret_cast<float*>(ws + lay.off_ploss); }
  double* stats() { return reinterpret_cast<double*>(ws + lay.off_stats); }
  float* grads() { return reinterpret_cast<float*>(ws + lay.off_grads); }
};

namespace {

int check_batch(const lbm_mlp* m, int32_t batch) {
  if (!m) return fail(LBM_ERR_ARG, "trainer is NULL");
  if (batch < 1 || batch > m->max_batch) return fail(LBM_ERR_ARG, "batch %d outside [1, %d]", batch, m->max_batch);
  return LBM_OK;
}

hipError_t launch_apply(lbm_mlp* m, int nblocks, int batch, int adam, float lr, float bc1, float bc2, float* grads_out,
                        float* loss_out) {
  lbm::k_mlp_apply<<<dim3((lbm::mlp::NPARAM + lbm::APPLY_P - 1) / lbm::APPLY_P + 1), dim3(lbm::APPLY_P * lbm::APPLY_S),
                     0, m->stream>>>(m->partial(), m->ploss(), nblocks, batch, m->master(), m->am(), m->av(), adam, lr,
                                     bc1, bc2, grads_out, loss_out, m->net(), m->w2t());
  return hipGetLastError();
}

int run_train(lbm_mlp* m, const uint16_t* x, const float* t, int64_t nsamples, const int32_t* rows, int32_t batch,
              int adam, float lr, float* grads_out, float* loss_out) {
  int rc = check_batch(m, batch);
  if (rc) return rc;
  if (!x || !t) return fail(LBM_ERR_ARG, "x and t must not be NULL");
  if (nsamples < 1) return fail(LBM_ERR_ARG, "nsamples %lld < 1", (long long)nsamples);
  if (!rows && nsamples < batch) return fail(LBM_ERR_ARG, "batch %d > nsamples %lld", batch, (long long)nsamples);
  if (adam && !(lr > 0.f && std::isfinite(lr))) return fail(LBM_ERR_ARG, "learning rate %g", (double)lr);
  const int tiles = (batch + lbm::TB - 1) / lbm::TB, nb = lbm::train_blocks(batch);
  lbm::k_mlp_train<<<dim3(nb), dim3(lbm::TTHREADS), 0, m->stream>>>(
      m->net(), m->w2t(), reinterpret_cast<const lbm::mlp::bf16*>(x), t, nsamples, rows, batch, tiles, m->partial(),
      m->ploss());
  HIPCHK(hipGetLastError());
  float bc1 = 1.f, bc2 = 1.f;
  if (adam) {
    m->step += 1;
    bc1 = (float)(1.0 - std::pow(0.9, (double)m->step));
    bc2 = (float)(1.0 - std::pow(0.999, (double)m->step));
  }
  HIPCHK(launch_apply(m, nb, batch, adam, lr, bc1, bc2, grads_out, loss_out));
  return LBM_OK;
}

}  // namespace

namespace lbm {
namespace host {
// used by lbm_api.hip / lbm_ensemble.hip
hipError_t closure_features(const LatDesc* single, const LatDesc* descs, int count, int parity, const int32_t* sites,
                            int n, float* feat, float* mc, hipStream_t s) {
  return launch_site_features(single, descs, count, parity, sites, n, feat, mc, s);
}
hipError_t closure_moments(const LatDesc* single, const LatDesc* descs, int count, int parity, const int32_t* sites,
                           int n, const float* sub, float* out, hipStream_t s) {
  return launch_site_moments(single, descs, count, parity, sites, n, sub, out, s);
}
}  // namespace host
}  // namespace lbm

extern "C" {

int lbm_closure_net_bytes(size_t* bytes) {
  if (!bytes) return fail(LBM_ERR_ARG, "bytes is NULL");
  *bytes = sizeof(lbm::mlp::Net);
  return LBM_OK;
}

int lbm_mlp_workspace_bytes(int32_t max_batch, size_t* bytes) {
  if (!bytes) return fail(LBM_ERR_ARG, "bytes is NULL");
  if (max_batch < lbm::TB || max_batch > 65536 || max_batch % lbm::TB)
    return fail(LBM_ERR_ARG, "max_batch %d must be a multiple of %d in [%d, 65536]", max_batch, lbm::TB, lbm::TB);
  *bytes = mlp_layout(max_batch).total;
  return LBM_OK;
}

void lbm_mlp_destroy(lbm_mlp* m) {
  if (!m) return;
  (void)hipStreamSynchronize(m->stream);
  delete m;
}

int lbm_mlp_init(lbm_mlp** out, int32_t max_batch, void* workspace, size_t bytes, const float* params,
                 void* hip_stream) {
  if (!out) return fail(LBM_ERR_ARG, "out is NULL");
  *out = nullptr;
  size_t need = 0;
  int rc = lbm_mlp_workspace_bytes(max_batch, &need);
  if (rc) return rc;
  if (!workspace || ((uintptr_t)workspace & 255)) return fail(LBM_ERR_ARG, "workspace NULL or not 256-byte aligned");
  if (bytes < need) return fail(LBM_ERR_ARG, "workspace of %zu bytes < %zu required", bytes, need);
  if (!params) return fail(LBM_ERR_ARG, "params is NULL");
  lbm_mlp* m = new lbm_mlp();
  m->max_batch = max_batch;
  m->stream = static_cast<hipStream_t>(hip_stream);
  m->ws = static_cast<char*>(workspace);
  m->lay = mlp_layout(max_batch);
  hipError_t e = hipMemcpyAsync(m->master(), params, sizeof(float) * lbm::mlp::NPARAM, hipMemcpyDeviceToDevice,
                                m->stream);
  if (e == hipSuccess) e = hipMemsetAsync(m->am(), 0, sizeof(float) * lbm::NP_PAD, m->stream);
  if (e == hipSuccess) e = hipMemsetAsync(m->av(), 0, sizeof(float) * lbm::NP_PAD, m->stream);
  if (e == hipSuccess) {
    lbm::k_init_net<<<dim3(8), dim3(256), 0, m->stream>>>(m->net());
    e = hipGetLastError();
  }
  if (e == hipSuccess) {
    e = launch_apply(m, 0, 0, 0, 0.f, 1.f, 1.f, nullptr, nullptr);
  }
  if (e == hipSuccess) e = hipStreamSynchronize(m->stream);
  if (e != hipSuccess) {
    delete m;
    return fail(LBM_ERR_HIP, "trainer init: %s", hipGetErrorString(e));
  }
  *out = m;
  return LBM_OK;
}

int lbm_mlp_fit_normalization(lbm_mlp* m, const float* feat, const float* resid, int64_t n) {
  if (!m || !feat || !resid) return fail(LBM_ERR_ARG, "NULL argument");
  if (n < 2) return fail(LBM_ERR_ARG, "need at least 2 samples");
  lbm::k_stats_partial<<<dim3(lbm::STAT_BLOCKS), dim3(lbm::STAT_THREADS), 0, m->stream>>>(feat, resid, n, m->stats());
  HIPCHK(hipGetLastError());
  lbm::k_stats_final<<<dim3(1), dim3(lbm::FINAL_COLS * lbm::FINAL_S), 0, m->stream>>>(m->stats(), lbm::STAT_BLOCKS, n, m->net());
  HIPCHK(hipGetLastError());
  return LBM_OK;
}

int lbm_mlp_pack(lbm_mlp* m, const float* feat, const float* resid, int64_t n, uint16_t* x_out, float* t_out) {
  if (!m || !feat || !x_out) return fail(LBM_ERR_ARG, "NULL argument");
  if (n < 0) return fail(LBM_ERR_ARG, "n < 0");
  if (n == 0) return LBM_OK;
  const int64_t blocks = (n + lbm::PACK_ROWS - 1) / lbm::PACK_ROWS;
  lbm::k_pack<<<dim3((unsigned)std::min<int64_t>(blocks, 4096)), dim3(lbm::PACK_THREADS), 0, m->stream>>>(
      m->net(), feat, resid, n, reinterpret_cast<lbm::mlp::bf16*>(x_out), t_out);
  HIPCHK(hipGetLastError());
  return LBM_OK;
}

int lbm_mlp_train_step(lbm_mlp* m, const uint16_t* x, const float* t, int64_t nsamples, const int32_t* rows,
                       int32_t batch, float lr, float* loss_out) {
  return run_train(m, x, t, nsamples, rows, batch, 1, lr, nullptr, loss_out);
}

int lbm_mlp_grads(lbm_mlp* m, const uint16_t* x, const float* t, int64_t nsamples, const int32_t* rows,
                  int32_t batch, float* grads_out, float* loss_out) {
  if (!grads_out) return fail(LBM_ERR_ARG, "grads_out is NULL");
  return run_train(m, x, t, nsamples, rows, batch, 0, 0.f, grads_out, loss_out);
}

int lbm_mlp_forward(lbm_mlp* m, const uint16_t* x, int64_t n, float* y_out) {
  if (!m || !x || !y_out) return fail(LBM_ERR_ARG, "NULL argument");
  if (n <= 0) return n == 0 ? LBM_OK : fail(LBM_ERR_ARG, "n < 0");
  const int64_t tiles = (n + lbm::TB - 1) / lbm::TB;
  lbm::k_mlp_forward<<<dim3((unsigned)std::min<int64_t>(tiles, lbm::FWD_BLOCKS)), dim3(lbm::TTHREADS), 0, m->stream>>>(
      m->net(), reinterpret_cast<const lbm::mlp::bf16*>(x), n, y_out);
  HIPCHK(hipGetLastError());
  return LBM_OK;
}

int lbm_mlp_params(lbm_mlp* m, float* params_out) {
  if (!m || !params_out) return fail(LBM_ERR_ARG, "NULL argument");
  lbm::k_copy_f32<<<dim3((lbm::mlp::NPARAM + 255) / 256), dim3(256), 0, m->stream>>>(m->master(), lbm::mlp::NPARAM,
                                                                                    params_out);
  HIPCHK(hipGetLastError());
  return LBM_OK;
}

int lbm_mlp_normalization(lbm_mlp* m, float* mean_out, float* inv_std_out, float* scale_out) {
  if (!m) return fail(LBM_ERR_ARG, "trainer is NULL");
  lbm::mlp::Net* net = m->net();
  if (mean_out) HIPCHK(hipMemcpyAsync(mean_out, net->feat_mean, sizeof(float) * 96, hipMemcpyDeviceToDevice, m->stream));
  if (inv_std_out)
    HIPCHK(hipMemcpyAsync(inv_std_out, net->feat_inv_std, sizeof(float) * 96, hipMemcpyDeviceToDevice, m->stream));
  if (scale_out) HIPCHK(hipMemcpyAsync(scale_out, net->out_scale, sizeof(float) * 3, hipMemcpyDeviceToDevice, m->stream));
  return LBM_OK;
}

int lbm_mlp_set_normalization(lbm_mlp* m, const float* mean, const float* inv_std, const float* scale) {
  if (!m || !mean || !inv_std || !scale) return fail(LBM_ERR_ARG, "NULL argument");
  lbm::mlp::Net* net = m->net();
  HIPCHK(hipMemcpyAsync(net->feat_mean, mean, sizeof(float) * 96, hipMemcpyDeviceToDevice, m->stream));
  HIPCHK(hipMemcpyAsync(net->feat_inv_std, inv_std, sizeof(float) * 96, hipMemcpyDeviceToDevice, m->stream));
  HIPCHK(hipMemcpyAsync(net->out_scale, scale, sizeof(float) * 3, hipMemcpyDeviceToDevice, m->stream));
  return LBM_OK;
}

int lbm_mlp_export(lbm_mlp* m, float trust, float gain, float kmin, void* net_out) {
  if (!m || !net_out) return fail(LBM_ERR_ARG, "NULL argument");
  if (!(trust > 0.f)) return fail(LBM_ERR_ARG, "trust bound %g must be > 0", (double)trust);
  if (!(gain > 0.f) || !std::isfinite(gain)) return fail(LBM_ERR_ARG, "gain %g must be finite and > 0", (double)gain);
  if (!(kmin >= 0.f) || !std::isfinite(kmin)) return fail(LBM_ERR_ARG, "kmin %g must be finite and >= 0", (double)kmin);
  HIPCHK(hipMemcpyAsync(net_out, m->net(), sizeof(lbm::mlp::Net), hipMemcpyDeviceToDevice, m->stream));
  lbm::k_export_finish<<<dim3(1), dim3(32), 0, m->stream>>>(static_cast<lbm::mlp::Net*>(net_out), trust, gain,
                                                             kmin);
  HIPCHK(hipGetLastError());
  HIPCHK(hipStreamSynchronize(m->stream));
  return LBM_OK;
}

}  // extern "C"
