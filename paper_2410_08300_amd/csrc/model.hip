// Model executor (declared in include/convsel_model.h): a network of
// convolutions, linear layers, ReLU, pooling, residual adds and flattens run
// from one caller-provided device arena.  Planning is host-only: value shapes,
// resolved algorithms, filter packages, the largest convolution workspace,
// and an arena offset for every intermediate value, shared between values
// whose lifetimes do not overlap (greedy by size: each value goes to the
// lowest offset that no already-placed, simultaneously live value covers).
// The forward pass launches the library's convolution entry points and the
// small elementwise / pooling kernels below, and allocates nothing.
#include <algorithm>
#include <stdio.h>
#include <string>
#include <vector>

#include "../../include/convsel_model.h"
#include "common.hpp"
#include "kernels.hpp"

using convsel::bf16_t;
using convsel::elem;
using convsel::vec16;

namespace convsel {
conv_status_t conv2d_prepacked_residual(const void* x, const void* packed, const void* b, const void* res, void* y,
                                        const conv2d_desc_t* desc, conv_algo_t algo, void* workspace,
                                        size_t workspace_bytes, void* stream);
}

namespace {

// ---- kernels -------------------------------------------------------------

template <typename T>
__global__ __launch_bounds__(256) void relu_kernel(const T* __restrict__ x, T* __restrict__ y, int64_t n) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i < n) elem<T>::store(y + i, fmaxf(elem<T>::load(x + i), 0.f));
}

template <typename T>
__global__ __launch_bounds__(256) void add_kernel(const T* __restrict__ a, const T* __restrict__ b, T* __restrict__ y,
                                                  int64_t n, int relu) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i >= n) return;
  float v = elem<T>::load(a + i) + elem<T>::load(b + i);
  if (relu) v = fmaxf(v, 0.f);
  elem<T>::store(y + i, v);
}

// One output element per thread; consecutive threads take consecutive q.
// A workgroup covers 256 outputs of one plane (`tiles` workgroups per
// plane), so the plane is a per-workgroup quantity and the per-thread index
// arithmetic stays in 32 bits.  Max: padding never contributes.  Average:
// the window sum over the padded input divided by kh*kw.
template <typename T, bool MAX>
__global__ __launch_bounds__(256) void pool_kernel(const T* __restrict__ x, T* __restrict__ y, int tiles, int H,
                                                   int W, int P, int Q, int kh, int kw, int sh, int sw, int ph,
                                                   int pw) {
  const int plane = blockIdx.x / tiles;
  const int j = (blockIdx.x - plane * tiles) * 256 + threadIdx.x;
  if (j >= P * Q) return;
  const int p = j / Q, q = j - p * Q;
  const T* xp = x + static_cast<int64_t>(plane) * H * W;
  float acc = MAX ? -INFINITY : 0.f;
  const int ih0 = p * sh - ph, iw0 = q * sw - pw;
  if (kh <= 3 && kw <= 3) {  // uniform: all taps' loads issued together, then one wait
    float v[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      const int ih = ih0 + t / 3, iw = iw0 + t % 3;
      const bool ok = t / 3 < kh && t % 3 < kw && ih >= 0 && ih < H && iw >= 0 && iw < W;
      v[t] = elem<T>::load(xp + (ok ? ih * W + iw : 0));
      v[t] = ok ? v[t] : (MAX ? -INFINITY : 0.f);
    }
#pragma unroll
    for (int t = 0; t < 9; ++t) acc = MAX ? fmaxf(acc, v[t]) : acc + v[t];
    if (!MAX) acc /= static_cast<float>(kh * kw);
    elem<T>::store(y + static_cast<int64_t>(plane) * P * Q + j, acc);
    return;
  }
  for (int r = 0; r < kh; ++r) {
    const int ih = ih0 + r;
    if (ih < 0 || ih >= H) continue;
    const T* row = xp + ih * W;
    for (int s = 0; s < kw; ++s) {
      const int iw = iw0 + s;
      if (iw < 0 || iw >= W) continue;
      const float v = elem<T>::load(row + iw);
      acc = MAX ? fmaxf(acc, v) : acc + v;
    }
  }
  if (!MAX) acc /= static_cast<float>(kh * kw);
  elem<T>::store(y + static_cast<int64_t>(plane) * P * Q + j, acc);
}

// Global average: one wave per plane, lanes stride the plane, then a fixed
// butterfly over the 64 lanes (deterministic order).
template <typename T>
__global__ __launch_bounds__(256) void global_avgpool_kernel(const T* __restrict__ x, T* __restrict__ y, int64_t planes,
                                                             int HW) {
  const int64_t plane = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (plane >= planes) return;
  const T* xp = x + plane * HW;
  float acc = 0.f;
  for (int i = lane; i < HW; i += 64) acc += elem<T>::load(xp + i);
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) acc += __shfl_xor(acc, m, 64);
  if (lane == 0) elem<T>::store(y + plane, acc / static_cast<float>(HW));
}

// ---- the same on channels-last values (channels whole 16-byte units) ------

template <typename T>
__device__ __forceinline__ float unit_at(const vec16& v, int i) {
  return elem<T>::to_f32(convsel::vec16_get<T>(v, i));
}

// One 16-byte unit (8 bf16 or 4 fp32 channels of one output pixel) per thread.
template <typename T, bool MAX>
__global__ __launch_bounds__(256) void pool_nhwc_kernel(const T* __restrict__ x, T* __restrict__ y, int H,
                                                        int W, int P, int Q, int CU, int kh, int kw, int sh, int sw,
                                                        int ph, int pw, int64_t units) {
  constexpr int UE = elem<T>::per16;
  const int64_t u = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (u >= units) return;
  const int cu = static_cast<int>(u % CU);
  const int64_t j = u / CU;
  const int pq = static_cast<int>(j % (static_cast<int64_t>(P) * Q));
  const int64_t n = j / (static_cast<int64_t>(P) * Q);
  const int p = pq / Q, q = pq - p * Q;
  const int ih0 = p * sh - ph, iw0 = q * sw - pw;
  const T* xn = x + (n * H * W * CU + cu) * UE;
  float acc[UE];
#pragma unroll
  for (int i = 0; i < UE; ++i) acc[i] = MAX ? -INFINITY : 0.f;
  for (int r = 0; r < kh; ++r) {
    const int ih = ih0 + r;
    if (ih < 0 || ih >= H) continue;
    for (int s = 0; s < kw; ++s) {
      const int iw = iw0 + s;
      if (iw < 0 || iw >= W) continue;
      const vec16 v = convsel::load16(xn + (static_cast<int64_t>(ih) * W + iw) * CU * UE);
#pragma unroll
      for (int i = 0; i < UE; ++i) acc[i] = MAX ? fmaxf(acc[i], unit_at<T>(v, i)) : acc[i] + unit_at<T>(v, i);
    }
  }
  vec16 o = convsel::vec16_zero();
  const float k = static_cast<float>(kh * kw);
#pragma unroll
  for (int i = 0; i < UE; ++i) convsel::vec16_set<T>(o, i, elem<T>::from_f32(MAX ? acc[i] : acc[i] / k));
  __builtin_memcpy(y + u * UE, &o, 16);  // (the caller's tensor: element alignment)
}

// 3 x 3 pooling with stride 2 and padding 1 from N x C x H x W (W a multiple
// of 8, x 16-byte aligned) into channels-last: the step after a stem.  A
// workgroup takes 64 channels x 32 columns of one output row; a thread reads
// the 17 input columns of 8 outputs with two 16-byte loads and one element per
// row, and the tile is transposed in LDS.
//
// What bounds it: its bytes.  64 channels of 112 x 112, 32 images (51 MB read,
// 13 MB written): 26 us; one output per thread with nine 2-byte loads each took
// 32 us, and its result needed a transposition besides.
template <bool MAX>
__global__ __launch_bounds__(256) void pool3s2_to_nhwc_kernel(const bf16_t* __restrict__ x, bf16_t* __restrict__ y,
                                                              int C, int H, int W, int P, int Q, int qtiles,
                                                              int ctiles) {
  __shared__ __align__(16) uint16_t tile[32 * 72];  // [column][channel], rows of 72 values (nine 16-byte units)
  int b = blockIdx.x;
  const int qt = b % qtiles;
  b /= qtiles;
  const int p = b % P;
  b /= P;
  const int ct = b % ctiles;
  const int64_t n = b / ctiles;
  const int c = threadIdx.x >> 2, g = threadIdx.x & 3;
  const int q0 = qt * 32 + g * 8, iw = 2 * q0;
  float acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i] = MAX ? -INFINITY : 0.f;
  const bool on = ct * 64 + c < C && iw < W;
  const bf16_t* xp = x + (n * C + (on ? ct * 64 + c : 0)) * static_cast<int64_t>(H) * W;
  vec16 lo[3], hi[3];
  float left[3];
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    const int ih = 2 * p - 1 + r;
    const bool in = on && ih >= 0 && ih < H;
    const bf16_t* row = xp + (in ? static_cast<int64_t>(ih) * W : 0);
    const bool in_hi = in && iw + 8 < W, in_left = in && iw > 0;
    lo[r] = convsel::load16(row + (in ? iw : 0));
    hi[r] = convsel::load16(row + (in_hi ? iw + 8 : 0));
    left[r] = elem<bf16_t>::load(row + (in_left ? iw - 1 : 0));
    const uint32_t pad = MAX ? 0xff80ff80u : 0u;  // -infinity, or 0
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      lo[r].d[d] = in ? lo[r].d[d] : pad;
      hi[r].d[d] = in_hi ? hi[r].d[d] : pad;
    }
    if (!in_left) left[r] = MAX ? -INFINITY : 0.f;
  }
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    auto at = [&](int i) { return i < 0 ? left[r] : i < 8 ? unit_at<bf16_t>(lo[r], i) : unit_at<bf16_t>(hi[r], i - 8); };
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int s = 0; s < 3; ++s) acc[i] = MAX ? fmaxf(acc[i], at(2 * i - 1 + s)) : acc[i] + at(2 * i - 1 + s);
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) tile[(g * 8 + i) * 72 + c] = convsel::f32_to_bf16(MAX ? acc[i] : acc[i] / 9.f);
  __syncthreads();
  const int q = threadIdx.x >> 3, cu = threadIdx.x & 7;
  const int qo = qt * 32 + q;
  if (qo >= Q || ct * 64 + cu * 8 >= C) return;
  const vec16 v = convsel::load16(tile + q * 72 + cu * 8);
  convsel::store16(y + ((n * P + p) * Q + qo) * C + ct * 64 + cu * 8, v);
}

// Global average of N x HW x C: a workgroup takes 8 units of channels of one
// image, 32 threads per unit with two sums each, added up as a tree through LDS:
// the order of global_avgpool_kernel, bit for bit.
template <typename T>
__global__ __launch_bounds__(256) void global_avgpool_nhwc_kernel(const T* __restrict__ x, T* __restrict__ y, int HW,
                                                                  int CU, int ctiles) {
  constexpr int UE = elem<T>::per16;
  __shared__ float part[32][8 * UE + 1];
  const int ct = blockIdx.x % ctiles;
  const int64_t n = blockIdx.x / ctiles;
  const int cl = threadIdx.x & 7, pl = threadIdx.x >> 3, cu = ct * 8 + cl;
  float acc[2][UE];
#pragma unroll
  for (int k = 0; k < UE; ++k) acc[0][k] = acc[1][k] = 0.f;
  if (cu < CU)
    for (int i = pl; i < HW; i += 64) {
      const vec16 lo = convsel::load16(x + ((n * HW + i) * CU + cu) * UE);
      const bool both = i + 32 < HW;
      const vec16 hi = convsel::load16(x + ((n * HW + (both ? i + 32 : i)) * CU + cu) * UE);
#pragma unroll
      for (int k = 0; k < UE; ++k) {
        acc[0][k] += unit_at<T>(lo, k);
        acc[1][k] += both ? unit_at<T>(hi, k) : 0.f;
      }
    }
#pragma unroll
  for (int k = 0; k < UE; ++k) part[pl][cl * UE + k] = acc[0][k] + acc[1][k];
  __syncthreads();
  const int c = threadIdx.x;
  if (c >= 8 * UE || ct * 8 * UE + c >= CU * UE) return;
  float s[32];
#pragma unroll
  for (int i = 0; i < 32; ++i) s[i] = part[i][c];
#pragma unroll
  for (int m = 16; m >= 1; m >>= 1)
#pragma unroll
    for (int i = 0; i < m; ++i) s[i] += s[i + m];
  elem<T>::store(y + n * CU * UE + ct * 8 * UE + c, s[0] / static_cast<float>(HW));
}

unsigned blocks_for(int64_t n, int per = 256) { return static_cast<unsigned>((n + per - 1) / per); }

// ---- model ----------------------------------------------------------------

enum OpKind { OP_CONV, OP_RELU, OP_POOL, OP_GAP, OP_ADD, OP_FLATTEN };

struct Value {
  int ndim = 0;
  int64_t d[4] = {0, 0, 0, 0};
  int producer = -1;  // op index; -1 for the input
  int alias = -1;     // flatten: the value whose storage this one shares
  int falias = -1;    // planned: a fused add's output shares its convolution's storage
  int64_t offset = -1;
  int64_t bytes = 0;
  // planned: held channels-last (images between the convolutions of the
  // channels-last path), and the place of a channels-last copy of a value that
  // is not (-1: none), written just before its first reader cl_first
  bool cl = false;
  int64_t cl_offset = -1;
  int cl_first = -1, cl_last = -1;
  int64_t elems() const {
    int64_t e = 1;
    for (int i = 0; i < ndim; ++i) e *= d[i];
    return e;
  }
};

struct Op {
  OpKind kind;
  int in = -1, in2 = -1, out = -1;
  // convolution / linear
  bool linear = false;
  int64_t c = 0, k = 0, r = 1, s = 1;
  int32_t sh = 1, sw = 1, ph = 0, pw = 0, dh = 1, dw = 1, groups = 1;
  conv_algo_t algo = CONV_ALGO_DEFAULT, algo_run = CONV_ALGO_DEFAULT;
  const void* w = nullptr;
  const void* b = nullptr;
  int relu = 0;
  // planned: residual value added in this convolution's epilogue (an add
  // fused into it; -1: none), the ReLU that then follows it, and whether this
  // op (a fused add) is skipped
  int res = -1;
  int relu_eff = 0;
  bool skip = false;
  bool cl = false;    // planned: a convolution that runs the channels-last kernel
  bool copy = false;  // planned: and reads its input's channels-last copy
  convsel::Shape shape{};
  conv2d_desc_t desc{};
  int64_t pk_off = -1, pk_bytes = 0, bias_off = -1, ws_bytes = 0;
  // pooling
  int pool_kind = 0, kh = 1, kw = 1;
};

constexpr int64_t kAlign = 256;
int64_t align_up(int64_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

}  // namespace

struct convsel_model {
  int32_t dtype = CONV_F32;
  std::vector<Op> ops;
  std::vector<Value> vals;  // vals[0] is the input
  int output = -1;
  bool planned = false, bound = false;
  char* arena = nullptr;
  int64_t arena_bytes = 0, ws_off = 0, ws_bytes = 0;
  int64_t esize() const { return dtype == CONV_F32 ? 4 : 2; }
  int root(int v) const {
    for (;;) {
      if (vals[v].alias >= 0) v = vals[v].alias;
      else if (vals[v].falias >= 0) v = vals[v].falias;
      else return v;
    }
  }
};

namespace {

conv_status_t add_op(convsel_model_t* m, Op op, int32_t* out) {
  if (!m || !out) return CONV_ERR_INVALID_ARG;
  const int nv = (int)m->vals.size();
  if (op.in < 0 || op.in >= nv || (op.kind == OP_ADD && (op.in2 < 0 || op.in2 >= nv))) return CONV_ERR_INVALID_ARG;
  Value v;
  v.producer = (int)m->ops.size();
  op.out = nv;
  m->vals.push_back(v);
  m->ops.push_back(op);
  m->planned = m->bound = false;
  *out = op.out;
  return CONV_OK;
}

conv_status_t from_hip(hipError_t e) {
  if (e == hipSuccess) return CONV_OK;
  (void)hipGetLastError();
  return CONV_ERR_DEVICE;
}

template <typename T>
hipError_t launch_elementwise(const Op& op, const void* a, const void* b, void* y, const Value& vin, const Value& vout,
                              hipStream_t st) {
  switch (op.kind) {
    case OP_RELU:
      hipLaunchKernelGGL(relu_kernel<T>, dim3(blocks_for(vout.elems())), dim3(256), 0, st,
                         reinterpret_cast<const T*>(a), reinterpret_cast<T*>(y), vout.elems());
      break;
    case OP_ADD:
      hipLaunchKernelGGL(add_kernel<T>, dim3(blocks_for(vout.elems())), dim3(256), 0, st,
                         reinterpret_cast<const T*>(a), reinterpret_cast<const T*>(b), reinterpret_cast<T*>(y),
                         vout.elems(), op.relu);
      break;
    case OP_POOL: {
      // Planning keeps planes * tiles and every plane's size below 2^31.
      const int tiles = (int)blocks_for(vout.d[2] * vout.d[3]);
      const dim3 grid((unsigned)(vout.d[0] * vout.d[1] * tiles));
      if (op.pool_kind == 0)
        hipLaunchKernelGGL((pool_kernel<T, true>), grid, dim3(256), 0, st, reinterpret_cast<const T*>(a),
                           reinterpret_cast<T*>(y), tiles, (int)vin.d[2], (int)vin.d[3], (int)vout.d[2],
                           (int)vout.d[3], op.kh, op.kw, op.sh, op.sw, op.ph, op.pw);
      else
        hipLaunchKernelGGL((pool_kernel<T, false>), grid, dim3(256), 0, st, reinterpret_cast<const T*>(a),
                           reinterpret_cast<T*>(y), tiles, (int)vin.d[2], (int)vin.d[3], (int)vout.d[2],
                           (int)vout.d[3], op.kh, op.kw, op.sh, op.sw, op.ph, op.pw);
      break;
    }
    case OP_GAP:
      hipLaunchKernelGGL(global_avgpool_kernel<T>, dim3(blocks_for(vin.d[0] * vin.d[1], 4)), dim3(256), 0, st,
                         reinterpret_cast<const T*>(a), reinterpret_cast<T*>(y), vin.d[0] * vin.d[1],
                         (int)(vin.d[2] * vin.d[3]));
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Pooling and global average pooling with a channels-last value on either side.
template <typename T>
hipError_t launch_channels_last(const Op& op, const void* a, void* y, const Value& vin, const Value& vout, bool in_cl,
                                hipStream_t st) {
  const T* x = reinterpret_cast<const T*>(a);
  T* o = reinterpret_cast<T*>(y);
  constexpr int UE = elem<T>::per16;
  const int C = (int)vin.d[1], H = (int)vin.d[2], W = (int)vin.d[3];
  if (op.kind == OP_GAP) {
    const int ctiles = (C / UE + 7) / 8;
    hipLaunchKernelGGL(global_avgpool_nhwc_kernel<T>, dim3((unsigned)(vin.d[0] * ctiles)), dim3(256), 0, st, x, o,
                       H * W, C / UE, ctiles);
    return hipGetLastError();
  }
  const int P = (int)vout.d[2], Q = (int)vout.d[3];
  if (in_cl) {
    const int64_t units = vout.elems() / UE;
    auto go = [&](auto kern) {
      hipLaunchKernelGGL(kern, dim3(blocks_for(units)), dim3(256), 0, st, x, o, H, W, P, Q, C / UE, op.kh, op.kw,
                         op.sh, op.sw, op.ph, op.pw, units);
    };
    if (op.pool_kind == 0) go(pool_nhwc_kernel<T, true>);
    else go(pool_nhwc_kernel<T, false>);
    return hipGetLastError();
  }
  if constexpr (sizeof(T) == 2) {
    const int qtiles = (Q + 31) / 32, ctiles = (C + 63) / 64;
    auto go = [&](auto kern) {
      hipLaunchKernelGGL(kern, dim3((unsigned)(vin.d[0] * ctiles * P * qtiles)), dim3(256), 0, st, x, o, C, H, W, P, Q,
                         qtiles, ctiles);
    };
    if (op.pool_kind == 0) go(pool3s2_to_nhwc_kernel<true>);
    else go(pool3s2_to_nhwc_kernel<false>);
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
}

// A convolution of the channels-last path (operation number `index`): its
// input's copy first, when this is the first operation that reads one.
conv_status_t run_channels_last(const convsel_model& m, const Op& op, const void* x, const void* res, void* y,
                                int index, hipStream_t st) {
  if (op.copy) {
    const Value& in = m.vals[m.root(op.in)];
    char* copy = m.arena + in.cl_offset;
    if (in.cl_first == index) {
      const conv_status_t s =
          from_hip(convsel::launch_to_nhwc(op.shape.dtype, x, copy, op.shape.N, op.shape.C, op.shape.H * op.shape.W, st));
      if (s != CONV_OK) return s;
    }
    x = copy;
  }
  convsel::Shape s = op.shape;
  s.relu = op.relu_eff != 0;
  const void* b = op.b ? m.arena + op.bias_off : nullptr;
  if (s.G > 1) return from_hip(convsel::dw_nhwc_main(s, x, m.arena + op.pk_off, b, y, st));
  return from_hip(convsel::nhwc_main(s, x, m.arena + op.pk_off, b, y, res, m.vals[m.root(op.out)].cl, st));
}

convsel::Shape shape_of(const conv2d_desc_t& d) {
  int64_t P = 0, Q = 0;
  conv2d_output_shape(&d, &P, &Q);
  convsel::Shape s{};
  s.N = d.n; s.C = d.c; s.H = d.h; s.W = d.w; s.K = d.k; s.R = d.r; s.S = d.s; s.P = P; s.Q = Q;
  s.G = d.groups; s.Cg = d.c / d.groups; s.Kg = d.k / d.groups;
  s.sh = d.stride_h; s.sw = d.stride_w; s.ph = d.pad_h; s.pw = d.pad_w; s.dh = d.dil_h; s.dw = d.dil_w;
  s.dtype = d.dtype == CONV_F32 ? convsel::DT_F32 : convsel::DT_BF16;
  s.bias = d.has_bias != 0;
  s.relu = d.fuse_relu != 0;
  return s;
}

// The default choice of a model's layer: the fitted tree's, but for stride 2
// filters that the filter-row kernel serves implicit GEMM where the tree says
// precomputed indices.  3 -> 64 channels of 224 x 224, 7 x 7 stride 2, bf16, 1 to
// 64 images: 7.0 to 56 us against 10.7 to 83; not stride 4, whose rows it mostly
// skips (3 -> 96 of 300 x 300, 16 images, 76 against 20).
conv_algo_t default_of(const conv2d_desc_t& d) {
  const conv_algo_t al = conv2d_default_algo(&d);
  if (al == CONV_ALGO_IMPLICIT_PRECOMP_GEMM && d.stride_h == 2 && d.stride_w == 2 &&
      conv2d_check(&d, CONV_ALGO_IMPLICIT_GEMM) == CONV_OK && convsel::rows_applies(shape_of(d)))
    return CONV_ALGO_IMPLICIT_GEMM;
  return al;
}

// Channels-last planning.  An implicit GEMM convolution (one group, C and K whole
// 16-byte units) can run the channels-last kernel, which needs no transposition
// of its input, and a direct depthwise 3 x 3 layer one of its own; a value
// between two such operations is then held as N x H x W x C.  A value qualifies
// when everything that writes or reads it can handle that: those convolutions,
// pooling, global average pooling, and adds and ReLUs whose values all qualify;
// flattens only of 1 x 1 planes, where the two layouts are the same.  The
// model's input and output stay N x C x H x W; a convolution on either end reads
// a channels-last copy of its input (one copy per value, made by a transposing
// pass) or writes N x K x P x Q itself.  A convolution with no such neighbour
// keeps the kernels of its own: the transposing pass alone would cost more than
// it gains.
void plan_layouts(convsel_model& m, int out_root) {
  const int nv = (int)m.vals.size();
  for (Value& v : m.vals) {
    v.cl = false;
    v.cl_offset = -1;
    v.cl_first = v.cl_last = -1;
  }
  for (Op& op : m.ops) op.cl = op.copy = false;
  const int ue = m.dtype == CONV_F32 ? 4 : 8;
  std::vector<char> can(m.ops.size(), 0);  // convolutions the kernel serves
  // The caller's tensors may have any element alignment: read through a copy,
  // and by no kernel that takes 16-byte units of a plane.
  auto callers = [&](int root) { return root == 0 || root == out_root; };
  auto plane1 = [&](int v) { return m.vals[v].ndim == 2 || m.vals[v].d[2] * m.vals[v].d[3] == 1; };
  // Operation i reads the channels-last copy of its input.  Never through a
  // flatten, whose value is its root's storage in N x C x H x W order.
  auto read_copy = [&](size_t i) {
    Op& op = m.ops[i];
    Value& v = m.vals[m.root(op.in)];
    op.copy = true;
    v.cl_first = v.cl_first < 0 ? (int)i : std::min(v.cl_first, (int)i);
    v.cl_last = std::max(v.cl_last, (int)i);
  };
  for (size_t i = 0; i < m.ops.size(); ++i) {
    Op& op = m.ops[i];
    if (op.kind != OP_CONV) continue;
    const conv2d_desc_t& d = op.desc;
    op.shape = shape_of(d);
    const convsel::Shape& s = op.shape;
    if (op.algo_run == CONV_ALGO_DIRECT)  // depthwise: both its values channels-last, or neither
      can[i] = op.res < 0 && convsel::dw_nhwc_applies(s);
    else
      can[i] = op.algo_run == CONV_ALGO_IMPLICIT_GEMM && s.C % ue == 0 && s.K % ue == 0 && convsel::nhwc_applies(s);
  }
  // Candidates: storage roots, then those with an operation that cannot are
  // struck out until nothing changes; then the chains that do not pay.
  std::vector<char> cl(nv, 0);
  for (int v = 1; v < nv; ++v)
    cl[v] = m.vals[v].alias < 0 && m.vals[v].falias < 0 && v != out_root && m.vals[v].ndim == 4 &&
            m.vals[v].d[1] % ue == 0 && !plane1(v);
  for (bool changed = true; changed;) {
    changed = false;
    auto strike = [&](int v) {
      if (cl[v]) {
        cl[v] = 0;
        changed = true;
      }
    };
    auto same = [&](int a, int b) {  // both channels-last or neither
      if (cl[a] != cl[b]) {
        strike(a);
        strike(b);
      }
    };
    for (size_t i = 0; i < m.ops.size(); ++i) {
      const Op& op = m.ops[i];
      const int in = m.root(op.in), out = m.root(op.out);
      switch (op.kind) {
        case OP_CONV:
          if (!can[i]) {
            strike(in);
            strike(out);
          } else if (op.shape.G > 1) {
            same(in, out);
          }
          if (op.res >= 0) same(m.root(op.res), out);
          break;
        case OP_POOL: {
          const bool from_nchw = m.dtype == CONV_BF16 && op.kh == 3 && op.kw == 3 && op.sh == 2 && op.sw == 2 && op.ph == 1 && op.pw == 1 &&
                                 m.vals[op.in].d[3] % 8 == 0 && !callers(in);  // (pool3s2_to_nhwc_kernel)
          if (cl[in] && !cl[out] && !plane1(op.out)) strike(in);
          if (cl[out] && !cl[in] && !from_nchw) strike(out);
          break;
        }
        case OP_GAP:
          break;
        case OP_ADD:
          if (op.skip) break;
          same(m.root(op.in2), out);
          same(in, out);
          break;
        case OP_RELU:
          same(in, out);
          break;
        case OP_FLATTEN:
          if (!plane1(op.in)) strike(in);
          break;
      }
    }
  }
  // Chains: values that operations of the path connect, decided on one by one.
  std::vector<int> chain(nv);
  for (int v = 0; v < nv; ++v) chain[v] = v;
  auto find = [&](int v) {
    while (chain[v] != v) v = chain[v] = chain[chain[v]];
    return v;
  };
  auto join = [&](int a, int b) {
    if (cl[a] && cl[b]) chain[find(a)] = find(b);
  };
  for (const Op& op : m.ops) {
    if (op.kind == OP_FLATTEN || op.skip) continue;
    const int out = m.root(op.out);
    join(m.root(op.in), out);
    if (op.kind == OP_ADD) join(m.root(op.in2), out);
    if (op.kind == OP_CONV && op.res >= 0) join(m.root(op.res), out);
  }
  struct Chain {
    int64_t copied = 0;
    bool odd = false, depthwise = false, whole_rows = false;
    std::vector<int> copies;
  };
  std::vector<Chain> chains(nv);
  for (size_t i = 0; i < m.ops.size(); ++i) {
    const Op& op = m.ops[i];
    if (op.kind != OP_CONV || !can[i]) continue;
    const int in = m.root(op.in), out = m.root(op.out);
    if (!cl[in] && !cl[out]) continue;
    Chain& ch = chains[find(cl[in] ? in : out)];
    ch.depthwise = ch.depthwise || (op.shape.G > 1 && (m.dtype == CONV_F32 || op.shape.W % 8 != 0));
    ch.whole_rows = ch.whole_rows || (op.shape.G > 1 && op.shape.W % 8 == 0);
    ch.odd = ch.odd || op.shape.P * op.shape.Q % 8 != 0 || (op.shape.H * op.shape.W % 8 != 0 && op.shape.R == 1);
    if (!cl[in] && (!plane1(op.in) || callers(in)) &&
        std::find(ch.copies.begin(), ch.copies.end(), in) == ch.copies.end()) {
      ch.copies.push_back(in);
      ch.copied += m.vals[in].elems() * m.esize();
    }
  }
  // Copies have to pay.  On planes of whole 16-byte rows the N x C x H x W
  // kernels are as fast (28 x 28 bottleneck, 32 images: 46 us, channels-last 62,
  // of which the copy of its input 12), on others they repack planes or read
  // pixel pairs and take up to twice the time.  So a chain whose input needs
  // a copy goes channels-last only with such planes in it, or when the copy is
  // small (2 MB: 3 us, where the many launches of a small batch matter more).
  // Depthwise layers gain by themselves, in bf16 where the rows they read are no
  // whole 16 bytes (inverted blocks: 48 of 60 x 60, 22 images, 80 us, channels-last
  // 78; 32 of 14 x 14, 11 images, 28 and 20; but 48 of 56 x 56, 19 images, 61 and 68, and
  // 24 of 40 x 40, 8 images, 20.5 and 21.9): a chain with whole rows only keeps its
  // planes however small its copy.
  // fp32 networks go channels-last, all their chains, where they have depthwise
  // layers (96 -> 576 -> 96 of 14 x 14, 64 images, 87 us, channels-last 64; MobileNetV2
  // at batch 1 591, with the chains around its depthwise layers alone 496, with all
  // of them 388; three 28 x 28 bottlenecks before a depthwise block, batch 1, 173, 133, 122).
  bool depthwise = false;
  for (int v = 0; v < nv; ++v) depthwise = depthwise || (cl[v] && chains[find(v)].depthwise);
  auto pays = [&](const Chain& ch) {
    if (m.dtype == CONV_F32) return depthwise;
    return ch.depthwise || ch.odd || (!ch.whole_rows && ch.copied <= (2 << 20));
  };
  bool any = false, none = true;
  std::vector<char> keep(nv, 0);
  for (int v = 0; v < nv; ++v) {
    if (!cl[v]) continue;
    none = false;
    keep[v] = pays(chains[find(v)]);
    any = any || keep[v];
  }
  cl = keep;
  if (!any && (m.dtype == CONV_F32 || !none)) return;  // (else layers of 1 x 1 planes alone go the path)
  for (int v = 0; v < nv; ++v) m.vals[v].cl = cl[v];
  for (size_t i = 0; i < m.ops.size(); ++i) {
    Op& op = m.ops[i];
    if (op.kind != OP_CONV || !can[i]) continue;
    const int in = m.root(op.in), out = m.root(op.out);
    if (op.shape.G > 1 ? !cl[in]
                       : !cl[in] && !cl[out] &&
                             !(plane1(op.in) && !callers(in) && op.shape.P * op.shape.Q == 1))
      continue;
    op.cl = true;
    if (!cl[in] && (!plane1(op.in) || callers(in))) read_copy(i);
  }
  // A convolution between values that both stay as they are uses a copy that
  // exists anyway (the projection of a residual block beside its first layer).
  for (size_t i = 0; i < m.ops.size(); ++i) {
    Op& op = m.ops[i];
    if (op.kind != OP_CONV || !can[i] || op.cl || op.shape.G > 1) continue;
    if (m.vals[op.in].ndim != 4 || m.vals[m.root(op.in)].cl_first < 0) continue;
    op.cl = true;
    read_copy(i);
  }
}

}  // namespace

extern "C" {

conv_status_t convsel_model_create(int32_t dtype, convsel_model_t** model) {
  if (!model || (dtype != CONV_F32 && dtype != CONV_BF16)) return CONV_ERR_INVALID_ARG;
  convsel_model_t* m = new convsel_model_t();
  m->dtype = dtype;
  m->vals.push_back(Value());  // the input
  *model = m;
  return CONV_OK;
}

void convsel_model_destroy(convsel_model_t* model) { delete model; }

conv_status_t convsel_model_conv(convsel_model_t* model, int32_t in, int64_t c, int64_t k, int64_t r, int64_t s,
                                 int32_t stride_h, int32_t stride_w, int32_t pad_h, int32_t pad_w, int32_t dil_h,
                                 int32_t dil_w, int32_t groups, conv_algo_t algo, const void* w, const void* b,
                                 int32_t fuse_relu, int32_t* out) {
  if (!w || c < 1 || k < 1 || r < 1 || s < 1 || groups < 1 || (fuse_relu != 0 && fuse_relu != 1))
    return CONV_ERR_INVALID_ARG;
  if (conv2d_algo_name(algo)[0] == 'u') return CONV_ERR_INVALID_ARG;  // "unknown"
  Op op;
  op.kind = OP_CONV;
  op.in = in;
  op.c = c; op.k = k; op.r = r; op.s = s;
  op.sh = stride_h; op.sw = stride_w; op.ph = pad_h; op.pw = pad_w; op.dh = dil_h; op.dw = dil_w;
  op.groups = groups;
  op.algo = algo;
  op.w = w;
  op.b = b;
  op.relu = fuse_relu;
  return add_op(model, op, out);
}

conv_status_t convsel_model_linear(convsel_model_t* model, int32_t in, int64_t in_features, int64_t out_features,
                                   conv_algo_t algo, const void* w, const void* b, int32_t fuse_relu, int32_t* out) {
  if (!w || in_features < 1 || out_features < 1 || (fuse_relu != 0 && fuse_relu != 1)) return CONV_ERR_INVALID_ARG;
  if (conv2d_algo_name(algo)[0] == 'u') return CONV_ERR_INVALID_ARG;
  Op op;
  op.kind = OP_CONV;
  op.linear = true;
  op.in = in;
  op.c = in_features;
  op.k = out_features;
  op.algo = algo;
  op.w = w;
  op.b = b;
  op.relu = fuse_relu;
  return add_op(model, op, out);
}

conv_status_t convsel_model_relu(convsel_model_t* model, int32_t in, int32_t* out) {
  Op op;
  op.kind = OP_RELU;
  op.in = in;
  return add_op(model, op, out);
}

conv_status_t convsel_model_pool(convsel_model_t* model, int32_t in, int32_t kind, int32_t kh, int32_t kw,
                                 int32_t stride_h, int32_t stride_w, int32_t pad_h, int32_t pad_w, int32_t* out) {
  if ((kind != 0 && kind != 1) || kh < 1 || kw < 1 || stride_h < 1 || stride_w < 1 || pad_h < 0 || pad_w < 0 ||
      2 * pad_h > kh || 2 * pad_w > kw)
    return CONV_ERR_INVALID_ARG;
  Op op;
  op.kind = OP_POOL;
  op.in = in;
  op.pool_kind = kind;
  op.kh = kh; op.kw = kw; op.sh = stride_h; op.sw = stride_w; op.ph = pad_h; op.pw = pad_w;
  return add_op(model, op, out);
}

conv_status_t convsel_model_global_avgpool(convsel_model_t* model, int32_t in, int32_t* out) {
  Op op;
  op.kind = OP_GAP;
  op.in = in;
  return add_op(model, op, out);
}

conv_status_t convsel_model_add(convsel_model_t* model, int32_t a, int32_t b, int32_t fuse_relu, int32_t* out) {
  if (fuse_relu != 0 && fuse_relu != 1) return CONV_ERR_INVALID_ARG;
  Op op;
  op.kind = OP_ADD;
  op.in = a;
  op.in2 = b;
  op.relu = fuse_relu;
  return add_op(model, op, out);
}

conv_status_t convsel_model_flatten(convsel_model_t* model, int32_t in, int32_t* out) {
  Op op;
  op.kind = OP_FLATTEN;
  op.in = in;
  const conv_status_t st = add_op(model, op, out);
  if (st == CONV_OK) model->vals[*out].alias = in;
  return st;
}

conv_status_t convsel_model_set_output(convsel_model_t* model, int32_t value) {
  if (!model || value <= 0 || value >= (int32_t)model->vals.size()) return CONV_ERR_INVALID_ARG;
  model->output = value;
  model->planned = model->bound = false;
  return CONV_OK;
}

conv_status_t convsel_model_plan(convsel_model_t* model, int64_t n, int64_t c, int64_t h, int64_t w,
                                 size_t* arena_bytes) {
  if (!model || !arena_bytes || n < 1 || c < 1 || h < 1 || w < 1 || model->output < 0) return CONV_ERR_INVALID_ARG;
  convsel_model_t& m = *model;
  m.planned = m.bound = false;
  const int64_t es = m.esize();
  for (Op& op : m.ops) {
    op.res = -1;
    op.relu_eff = op.relu;
    op.skip = false;
  }
  for (Value& v : m.vals) v.falias = -1;
  Value& in = m.vals[0];
  in.ndim = 4;
  in.d[0] = n; in.d[1] = c; in.d[2] = h; in.d[3] = w;
  // Shapes and algorithms, in operation order.
  for (Op& op : m.ops) {
    const Value& a = m.vals[op.in];
    Value& o = m.vals[op.out];
    o.offset = -1;
    switch (op.kind) {
      case OP_CONV: {
        conv2d_desc_t& d = op.desc;
        if (op.linear) {
          const int64_t feat = a.ndim == 2 ? a.d[1] : (a.ndim == 4 ? a.d[1] * a.d[2] * a.d[3] : -1);
          if (feat != op.c || (a.ndim == 4 && a.d[2] * a.d[3] != 1)) return CONV_ERR_INVALID_ARG;
          d = conv2d_desc_t{a.d[0], op.c, 1, 1, op.k, 1, 1, 1, 1, 0, 0, 1, 1, 1, m.dtype, op.b != nullptr, op.relu};
        } else {
          if (a.ndim != 4 || a.d[1] != op.c) return CONV_ERR_INVALID_ARG;
          d = conv2d_desc_t{a.d[0], a.d[1], a.d[2], a.d[3], op.k, op.r, op.s, op.sh, op.sw, op.ph, op.pw,
                            op.dh, op.dw, op.groups, m.dtype, op.b != nullptr, op.relu};
        }
        conv_algo_t al = op.algo == CONV_ALGO_DEFAULT ? default_of(d) : op.algo;
        const conv_status_t st = conv2d_check(&d, al);
        if (st != CONV_OK) return st;
        op.algo_run = al;
        if (op.linear) {
          o.ndim = 2;
          o.d[0] = a.d[0]; o.d[1] = op.k; o.d[2] = o.d[3] = 0;
        } else {
          int64_t P = 0, Q = 0;
          conv2d_output_shape(&d, &P, &Q);
          o.ndim = 4;
          o.d[0] = a.d[0]; o.d[1] = op.k; o.d[2] = P; o.d[3] = Q;
        }
        break;
      }
      case OP_RELU:
        o.ndim = a.ndim;
        for (int i = 0; i < 4; ++i) o.d[i] = a.d[i];
        break;
      case OP_ADD: {
        const Value& b = m.vals[op.in2];
        if (a.ndim != b.ndim) return CONV_ERR_INVALID_ARG;
        for (int i = 0; i < a.ndim; ++i)
          if (a.d[i] != b.d[i]) return CONV_ERR_INVALID_ARG;
        o.ndim = a.ndim;
        for (int i = 0; i < 4; ++i) o.d[i] = a.d[i];
        break;
      }
      case OP_POOL: {
        if (a.ndim != 4 || a.elems() >= ((int64_t)1 << 31)) return CONV_ERR_INVALID_ARG;  // 32-bit plane offsets
        const int64_t P = (a.d[2] + 2 * op.ph - op.kh) / op.sh + 1;
        const int64_t Q = (a.d[3] + 2 * op.pw - op.kw) / op.sw + 1;
        if (a.d[2] + 2 * op.ph < op.kh || a.d[3] + 2 * op.pw < op.kw || P < 1 || Q < 1) return CONV_ERR_INVALID_ARG;
        o.ndim = 4;
        o.d[0] = a.d[0]; o.d[1] = a.d[1]; o.d[2] = P; o.d[3] = Q;
        break;
      }
      case OP_GAP:
        if (a.ndim != 4) return CONV_ERR_INVALID_ARG;
        o.ndim = 4;
        o.d[0] = a.d[0]; o.d[1] = a.d[1]; o.d[2] = o.d[3] = 1;
        break;
      case OP_FLATTEN:
        if (a.ndim != 4) return CONV_ERR_INVALID_ARG;
        o.ndim = 2;
        o.d[0] = a.d[0]; o.d[1] = a.d[1] * a.d[2] * a.d[3]; o.d[2] = o.d[3] = 0;
        break;
    }
    if (o.elems() >= ((int64_t)1 << 31)) return CONV_ERR_INVALID_ARG;
    o.bytes = o.elems() * es;
  }
  // Residual adds into implicit GEMM convolutions: an add of a convolution's
  // output X (read by nothing else, no ReLU of its own) and a value Y that
  // exists before that convolution runs becomes that convolution's epilogue
  // residual, y = relu(conv + b + Y); the add's output then shares X's storage.
  {
    const int nv0 = (int)m.vals.size();
    std::vector<int> uses(nv0, 0);
    for (const Op& op : m.ops) {
      ++uses[op.in];
      if (op.kind == OP_ADD) ++uses[op.in2];
    }
    ++uses[m.output];
    for (int i = 0; i < (int)m.ops.size(); ++i) {
      Op& add = m.ops[i];
      if (add.kind != OP_ADD) continue;
      int best = -1, other = -1;
      for (int side = 0; side < 2; ++side) {
        const int X = side == 0 ? add.in : add.in2, Y = side == 0 ? add.in2 : add.in;
        const int p = m.vals[X].producer;
        if (p < 0 || m.vals[X].alias >= 0 || uses[X] != 1) continue;
        const Op& c = m.ops[p];
        if (c.kind != OP_CONV || c.algo_run != CONV_ALGO_IMPLICIT_GEMM || c.relu_eff || c.res >= 0) continue;
        if (m.vals[m.root(Y)].producer >= p) continue;  // Y must exist when the convolution runs
        if (best < 0 || p > m.vals[best].producer) {
          best = X;
          other = Y;
        }
      }
      if (best < 0) continue;
      Op& c = m.ops[m.vals[best].producer];
      c.res = other;
      c.relu_eff = add.relu;
      c.desc.fuse_relu = add.relu;
      add.skip = true;
      m.vals[add.out].falias = best;
    }
  }
  // The output must come out of an operation, not be the input itself.
  const int out_root = m.root(m.output);
  if (out_root == 0) return CONV_ERR_UNSUPPORTED;
  plan_layouts(m, out_root);
  // Filter packages, biases and the largest workspace.
  int64_t off = 0;
  m.ws_bytes = 0;
  for (Op& op : m.ops) {
    if (op.kind != OP_CONV) continue;
    size_t pk = 0, ws = 0;
    if (op.cl)
      pk = op.shape.G > 1 ? convsel::dw_nhwc_packed_bytes(op.shape) : convsel::nhwc_packed_bytes(op.shape);
    else if (conv2d_packed_filter_bytes(&op.desc, op.algo_run, &pk) != CONV_OK ||
             conv2d_prepacked_workspace_bytes(&op.desc, op.algo_run, &ws) != CONV_OK)
      return CONV_ERR_INVALID_ARG;
    op.pk_off = off;
    op.pk_bytes = (int64_t)pk;
    off = align_up(off + (int64_t)pk);
    op.bias_off = -1;
    if (op.b) {
      op.bias_off = off;
      off = align_up(off + op.k * es);
    }
    op.ws_bytes = (int64_t)ws;
    m.ws_bytes = std::max(m.ws_bytes, (int64_t)ws);
  }
  // Lifetimes of the storage roots: [producer, last reader].
  const int nv = (int)m.vals.size();
  std::vector<int> last(nv, -1), first(nv, -1);
  for (int i = 0; i < nv; ++i)
    if (m.vals[i].alias < 0 && m.vals[i].falias < 0) first[i] = last[i] = m.vals[i].producer;
  for (int i = 0; i < (int)m.ops.size(); ++i) {
    const Op& op = m.ops[i];
    if (op.skip) continue;
    last[m.root(op.in)] = std::max(last[m.root(op.in)], i);
    if (op.kind == OP_ADD) last[m.root(op.in2)] = std::max(last[m.root(op.in2)], i);
    if (op.res >= 0) last[m.root(op.res)] = std::max(last[m.root(op.res)], i);
  }
  // The workspace, then the activations.
  m.ws_off = off;
  off = align_up(off + m.ws_bytes);
  const int64_t act_base = off;
  // Blocks to place: the storage roots and the channels-last copies.
  struct Block {
    int64_t need, offset;
    int first, last, value;
    bool copy;
  };
  std::vector<Block> order;
  for (int i = 0; i < nv; ++i) {
    const Value& v = m.vals[i];
    if (i > 0 && v.alias < 0 && v.falias < 0 && i != out_root)
      order.push_back({align_up(v.bytes), 0, first[i], last[i], i, false});
    if (v.cl_first >= 0) order.push_back({align_up(v.elems() * es), 0, v.cl_first, v.cl_last, i, true});
  }
  std::stable_sort(order.begin(), order.end(), [&](const Block& x, const Block& y) { return x.need > y.need; });
  std::vector<int> placed;
  int64_t act_top = 0;
  for (int v = 0; v < (int)order.size(); ++v) {
    // Intervals [offset, offset + bytes) of placed blocks live at the same time, sorted by offset.
    std::vector<std::pair<int64_t, int64_t>> busy;
    for (int u : placed)
      if (order[u].first <= order[v].last && order[v].first <= order[u].last)
        busy.push_back({order[u].offset, order[u].offset + order[u].need});
    std::sort(busy.begin(), busy.end());
    int64_t cand = 0;
    for (const auto& iv : busy) {
      if (cand + order[v].need <= iv.first) break;
      cand = std::max(cand, iv.second);
    }
    order[v].offset = cand;
    act_top = std::max(act_top, cand + order[v].need);
    placed.push_back(v);
  }
  for (const Block& bl : order) (bl.copy ? m.vals[bl.value].cl_offset : m.vals[bl.value].offset) = bl.offset + act_base;
  m.arena_bytes = act_base + act_top;
  *arena_bytes = (size_t)m.arena_bytes;
  m.planned = true;
  return CONV_OK;
}

conv_status_t convsel_model_output_shape(const convsel_model_t* model, int64_t dims[4], int32_t* ndim) {
  if (!model || !dims || !ndim || !model->planned) return CONV_ERR_INVALID_ARG;
  const Value& v = model->vals[model->output];
  *ndim = v.ndim;
  for (int i = 0; i < 4; ++i) dims[i] = i < v.ndim ? v.d[i] : 0;
  return CONV_OK;
}

conv_status_t convsel_model_value_placement(const convsel_model_t* model, int32_t v, int64_t* offset,
                                            int64_t* bytes) {
  if (!model || !offset || !bytes || !model->planned || v < 0 || v >= (int32_t)model->vals.size())
    return CONV_ERR_INVALID_ARG;
  const int r = model->root(v);
  *offset = (r == 0 || r == model->root(model->output)) ? -1 : model->vals[r].offset;
  *bytes = model->vals[v].bytes;
  return CONV_OK;
}

conv_status_t convsel_model_bind(convsel_model_t* model, void* arena, size_t arena_bytes, void* stream) {
  if (!model || !model->planned) return CONV_ERR_INVALID_ARG;
  convsel_model_t& m = *model;
  if ((int64_t)arena_bytes < m.arena_bytes || (m.arena_bytes > 0 && !arena) ||
      reinterpret_cast<uintptr_t>(arena) % kAlign != 0)
    return CONV_ERR_INVALID_ARG;
  m.bound = false;
  char* base = reinterpret_cast<char*>(arena);
  const hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  for (Op& op : m.ops) {
    if (op.kind != OP_CONV) continue;
    conv_status_t s = op.cl ? from_hip(op.shape.G > 1 ? convsel::dw_nhwc_pack(op.shape, op.w, base + op.pk_off, st)
                                                      : convsel::nhwc_pack(op.shape, op.w, base + op.pk_off, st))
                            : conv2d_pack_filters(op.w, base + op.pk_off, &op.desc, op.algo_run, stream);
    if (s != CONV_OK) return s;
    if (op.b) {
      s = from_hip(hipMemcpyAsync(base + op.bias_off, op.b, (size_t)(op.k * m.esize()), hipMemcpyDeviceToDevice, st));
      if (s != CONV_OK) return s;
    }
  }
  m.arena = base;
  m.bound = true;
  return CONV_OK;
}

conv_status_t convsel_model_forward(convsel_model_t* model, const void* x, void* y, void* stream) {
  if (!model || !model->bound || !x || !y) return CONV_ERR_INVALID_ARG;
  convsel_model_t& m = *model;
  const int out_root = m.root(m.output);
  const hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  auto ptr = [&](int v) -> char* {
    const int r = m.root(v);
    if (r == 0) return const_cast<char*>(reinterpret_cast<const char*>(x));
    if (r == out_root) return reinterpret_cast<char*>(y);
    return m.arena + m.vals[r].offset;
  };
  for (int i = 0; i < (int)m.ops.size(); ++i) {
    const Op& op = m.ops[i];
    const Value& vin = m.vals[op.in];
    const Value& vout = m.vals[op.out];
    conv_status_t s = CONV_OK;
    if (op.skip) continue;  // an add fused into its convolution
    switch (op.kind) {
      case OP_CONV:
        if (op.cl) {
          s = run_channels_last(m, op, ptr(op.in), op.res >= 0 ? ptr(op.res) : nullptr, ptr(op.out), i, st);
          break;
        }
        if (op.res >= 0)
          s = convsel::conv2d_prepacked_residual(
              ptr(op.in), m.arena + op.pk_off, op.b ? m.arena + op.bias_off : nullptr, ptr(op.res), ptr(op.out),
              &op.desc, op.algo_run, op.ws_bytes ? m.arena + m.ws_off : nullptr, (size_t)op.ws_bytes, stream);
        else
          s = conv2d_prepacked(ptr(op.in), m.arena + op.pk_off, op.b ? m.arena + op.bias_off : nullptr, ptr(op.out),
                               &op.desc, op.algo_run, op.ws_bytes ? m.arena + m.ws_off : nullptr, (size_t)op.ws_bytes,
                               stream);
        break;
      case OP_FLATTEN:
        break;
      case OP_POOL:
      case OP_GAP:
        if (m.vals[m.root(op.in)].cl || m.vals[m.root(op.out)].cl) {
          const bool in_cl = m.vals[m.root(op.in)].cl;
          s = from_hip(m.dtype == CONV_F32 ? launch_channels_last<float>(op, ptr(op.in), ptr(op.out), vin, vout, in_cl, st)
                                           : launch_channels_last<bf16_t>(op, ptr(op.in), ptr(op.out), vin, vout, in_cl, st));
          break;
        }
        [[fallthrough]];
      default:
        s = from_hip(m.dtype == CONV_F32
                         ? launch_elementwise<float>(op, ptr(op.in), op.in2 >= 0 ? ptr(op.in2) : nullptr,
                                                     ptr(op.out), vin, vout, st)
                         : launch_elementwise<bf16_t>(op, ptr(op.in), op.in2 >= 0 ? ptr(op.in2) : nullptr,
                                                      ptr(op.out), vin, vout, st));
        break;
    }
    if (s != CONV_OK) return s;
  }
  return CONV_OK;
}

conv_status_t convsel_model_describe(const convsel_model_t* model, char* buf, size_t len) {
  if (!model || !buf || len == 0) return CONV_ERR_INVALID_ARG;
  static const char* names[] = {"conv", "relu", "pool", "global_avgpool", "add", "flatten"};
  std::string d;
  char line[256];
  for (size_t i = 0; i < model->ops.size(); ++i) {
    const Op& op = model->ops[i];
    const Value& o = model->vals[op.out];
    const char* nm = op.kind == OP_CONV && op.linear ? "linear" : names[op.kind];
    snprintf(line, sizeof(line), "%zu %s v%d%s -> v%d [%lld %lld %lld %lld]", i, nm, op.in,
             op.kind == OP_ADD ? (std::string(" + v") + std::to_string(op.in2)).c_str() : "", op.out,
             (long long)o.d[0], (long long)o.d[1], (long long)o.d[2], (long long)o.d[3]);
    d += line;
    if (op.kind == OP_CONV) d += std::string(" algo=") + conv2d_algo_name(model->planned ? op.algo_run : op.algo);
    if (model->planned && op.cl) {
      d += " channels_last";
      if (op.shape.G == 1) {
        d += " " + convsel::nhwc_describe(op.shape);
        d += model->vals[model->root(op.out)].cl ? " out=nhwc" : " out=planes";
      }
      if (op.copy) d += " copy@" + std::to_string(model->vals[model->root(op.in)].cl_offset);
    }
    if (model->planned && op.res >= 0) d += " + v" + std::to_string(op.res);
    if (model->planned ? (op.kind == OP_CONV ? op.relu_eff : op.relu) : op.relu) d += " relu";
    if (model->planned && op.skip) d += " fused";
    if (model->planned) {
      snprintf(line, sizeof(line), " offset=%lld", (long long)(model->root(op.out) == model->root(model->output)
                                                                     ? -1
                                                                     : model->vals[model->root(op.out)].offset));
      d += line;
    }
    d += "\n";
  }
  if (model->planned) {
    snprintf(line, sizeof(line), "arena=%lld workspace=%lld@%lld", (long long)model->arena_bytes,
             (long long)model->ws_bytes, (long long)model->ws_off);
    d += line;
  }
  snprintf(buf, len, "%s", d.c_str());
  return CONV_OK;
}

}  // extern "C"
