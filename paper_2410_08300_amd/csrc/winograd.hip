// Winograd minimal filtering F(2x2, 3x3) (paper, Sec. V-B item (d), after
// Lavin and Gray 2016).  For a 4x4 input tile d and a 3x3 filter g, the 2x2
// output tile of the correlation is
//     Y = A^T [ (G g G^T) (.) (B^T d B) ] A
// with (.) the elementwise product, summed over input channels, so the
// 16 elementwise positions become 16 independent GEMMs:
//     M[xi,nu] (K x T) = U[xi,nu] (K x C) * V[xi,nu]^T (C x T).
// Four kernels: filter transform (U), input transform (V), the batched MFMA
// GEMM (gemm.hip), output transform (y).  U and V are kept in the data type
// (bf16 data: rounded after the fp32 transform), M in fp32.
//   B^T = [1 0 -1 0; 0 1 1 0; 0 -1 1 0; 0 1 0 -1]
//   G   = [1 0 0; 1/2 1/2 1/2; 1/2 -1/2 1/2; 0 0 1]
//   A^T = [1 1 1 0; 0 1 -1 -1]
#include "common.hpp"
#include "kernels.hpp"

namespace convsel {

namespace {

// U[xi*4+nu][k][c]; one thread per (k, c), c fastest (coalesced stores).
template <typename T>
__global__ __launch_bounds__(256) void wino_filter_kernel(const T* __restrict__ w, T* __restrict__ U, int K, int C) {
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (idx >= static_cast<int64_t>(K) * C) return;
  const T* g = w + idx * 9;
  float f[3][3];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) f[i][j] = elem<T>::to_f32(g[i * 3 + j]);
  // t = G f (4 x 3)
  float t[4][3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    t[0][j] = f[0][j];
    t[1][j] = 0.5f * (f[0][j] + f[1][j] + f[2][j]);
    t[2][j] = 0.5f * (f[0][j] - f[1][j] + f[2][j]);
    t[3][j] = f[2][j];
  }
  const int64_t plane = static_cast<int64_t>(K) * C;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float u[4] = {t[i][0], 0.5f * (t[i][0] + t[i][1] + t[i][2]), 0.5f * (t[i][0] - t[i][1] + t[i][2]),
                        t[i][2]};
#pragma unroll
    for (int j = 0; j < 4; ++j) U[(i * 4 + j) * plane + idx] = elem<T>::from_f32(u[j]);
  }
}

constexpr int CB = 32;  // channels per workgroup

// V[xi*4+nu][t][c] for the tiles of images n0 .. n0+nb-1 (t counted from n0).
// A workgroup stages four input rows of LPR columns for CB channels in LDS
// (a group of LPR lanes reads one row; all of a thread's reads are in flight
// together), which is the window of LPR/2 - 1 tiles of one tile row.  Each
// thread then transforms one channel of every eighth tile; consecutive threads
// write consecutive channels, 128 bytes (fp32) of each of V's 16 planes.  An
// odd channel pitch in LDS keeps the lanes' reads on distinct banks.
//
// What bounds it: V, four times the input, written once.  256 channels of
// 56 x 56, 8 images, fp32 (25.7 MB read, 102.8 MB written): 26.8 us; with eight
// tiles per workgroup, each element's row and column found by divisions, it
// took 45.6.
template <typename T, int LPR>
__global__ __launch_bounds__(256) void wino_input_kernel(const T* __restrict__ x, T* __restrict__ V, int C, int H,
                                                         int W, int ph, int pw, int TP, int TQ, int64_t n0,
                                                         int64_t Tc) {
  constexpr int TB = LPR / 2 - 1;            // tiles per workgroup along a tile row
  constexpr int GROUPS = 256 / LPR;          // rows read at a time
  constexpr int LOADS = CB * 4 / GROUPS;     // rows per thread
  constexpr int PITCH = 4 * LPR + 1;
  __shared__ float tile[CB * PITCH];
  const int tqb = (TQ + TB - 1) / TB;
  const int tp = blockIdx.x / tqb, tq0 = (blockIdx.x - tp * tqb) * TB;
  const int c0 = blockIdx.y * CB;
  const int nl = blockIdx.z;
  const int64_t n = n0 + nl;
  const int col = threadIdx.x % LPR, grp = threadIdx.x / LPR;
  const int ih0 = 2 * tp - ph, iw = 2 * tq0 - pw + col;
  const bool col_in = iw >= 0 && iw < W;
  const T* xn = x + (n * C + c0) * static_cast<int64_t>(H) * W;
  constexpr int BATCH = LOADS < 16 ? LOADS : 16;
#pragma unroll
  for (int l0 = 0; l0 < LOADS; l0 += BATCH) {
    T v[BATCH];
#pragma unroll
    for (int l = 0; l < BATCH; ++l) {
      const int row = (l0 + l) * GROUPS + grp, c = row >> 2, ih = ih0 + (row & 3);
      const bool in = col_in && c0 + c < C && ih >= 0 && ih < H;
      v[l] = xn[in ? (static_cast<int64_t>(c) * H + ih) * W + iw : 0];
      if (!in) v[l] = elem<T>::from_f32(0.f);
    }
#pragma unroll
    for (int l = 0; l < BATCH; ++l) {
      const int row = (l0 + l) * GROUPS + grp;
      tile[(row >> 2) * PITCH + (row & 3) * LPR + col] = elem<T>::to_f32(v[l]);
    }
  }
  __syncthreads();
  const int c = threadIdx.x % CB;
  if (c0 + c >= C) return;
  const int64_t plane = Tc * C;
  for (int tb = threadIdx.x / CB; tb < TB && tq0 + tb < TQ; tb += 256 / CB) {
    float d[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) d[i][j] = tile[c * PITCH + i * LPR + 2 * tb + j];
    // s = B^T d
    float s[4][4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      s[0][j] = d[0][j] - d[2][j];
      s[1][j] = d[1][j] + d[2][j];
      s[2][j] = d[2][j] - d[1][j];
      s[3][j] = d[1][j] - d[3][j];
    }
    const int64_t t = (static_cast<int64_t>(nl) * TP + tp) * TQ + tq0 + tb;
    T* vp = V + t * C + c0 + c;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float v[4] = {s[i][0] - s[i][2], s[i][1] + s[i][2], s[i][2] - s[i][1], s[i][1] - s[i][3]};
#pragma unroll
      for (int j = 0; j < 4; ++j) vp[(i * 4 + j) * plane] = elem<T>::from_f32(v[j]);
    }
  }
}

// Workgroups along a row of TQ tiles, lpr lanes to an input row.
int wino_row_blocks(int TQ, int lpr) { return (TQ + lpr / 2 - 2) / (lpr / 2 - 1); }

// Lanes per input row.  16, seven tiles a workgroup: the most workgroups, and the
// least LDS each (240 random inputs: within 5 percent of the best width in bf16
// and for few channels or tiles, where 32 and 64 lanes take up to twice as
// long: 5 channels of 54 x 54, two images, 2.7, 3.8 and 5.3 us).  In fp32, with more
// than a block of channels, blocks that they mostly fill and 2400 workgroups at 16
// lanes, V's 128-byte rows are what bounds it, and longer runs of them help: 32
// lanes (219 channels of 18 x 19, 26 images, 15.0 -> 12.5 us), or 64 where these
// leave no more lanes without a tile and V (14 KB for seven tiles) stays below 430
// MB (297 of 46 x 47, 10 images: 58.7, 40.5 and 35.6; but 343 of 56 x 56, 36
// images: 279, 252 and 364).
int wino_input_lanes(const Shape& s, int64_t nb) {
  const int TP = (int)((s.P + 1) / 2), TQ = (int)((s.Q + 1) / 2);
  const int64_t blocks = nb * TP * wino_row_blocks(TQ, 16) * ((s.C + CB - 1) / CB);
  const int64_t channels = (s.C + CB - 1) / CB * CB;  // (with those past C)
  if (s.dtype != DT_F32 || s.C <= CB || 8 * s.C < 5 * channels || blocks < 2400) return 16;
  return 2 * wino_row_blocks(TQ, 64) <= wino_row_blocks(TQ, 32) && blocks < 30000 ? 64 : 32;
}

template <typename T>
void launch_wino_input_typed(const Shape& s, const void* x, void* V, int64_t n0, int64_t nb, hipStream_t stream) {
  const int TP = (int)((s.P + 1) / 2), TQ = (int)((s.Q + 1) / 2);
  const int64_t Tc = nb * TP * TQ;
  const int best = wino_input_lanes(s, nb);
  const dim3 grid((unsigned)(TP * wino_row_blocks(TQ, best)), (unsigned)((s.C + CB - 1) / CB), (unsigned)nb);
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, stream, (const T*)x, (T*)V, (int)s.C, (int)s.H, (int)s.W, s.ph, s.pw,
                       TP, TQ, n0, Tc);
  };
  if constexpr (sizeof(T) == 4) {
    if (best == 64) return go(wino_input_kernel<T, 64>);
    if (best == 32) return go(wino_input_kernel<T, 32>);
  }
  go(wino_input_kernel<T, 16>);
}

// y tiles from M[xi*4+nu][k][t] (fp32); one thread per (k, t), t fastest.
template <typename T>
__global__ __launch_bounds__(256) void wino_output_kernel(const float* __restrict__ M, const T* __restrict__ bias,
                                                          T* __restrict__ y, int K, int P, int Q, int TP, int TQ,
                                                          int64_t n0, int64_t Tc, int relu) {
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (idx >= static_cast<int64_t>(K) * Tc) return;
  const int k = static_cast<int>(idx / Tc);
  const int64_t t = idx - static_cast<int64_t>(k) * Tc;
  const int tq = static_cast<int>(t % TQ);
  const int tp = static_cast<int>((t / TQ) % TP);
  const int64_t nl = t / (static_cast<int64_t>(TQ) * TP);
  const int64_t plane = static_cast<int64_t>(K) * Tc;
  float m[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) m[i][j] = M[(i * 4 + j) * plane + idx];
  // a = A^T m (2 x 4), out = a A (2 x 2)
  float a[2][4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    a[0][j] = m[0][j] + m[1][j] + m[2][j];
    a[1][j] = m[1][j] - m[2][j] - m[3][j];
  }
  const float bv = bias ? elem<T>::to_f32(bias[k]) : 0.f;
  const int64_t n = n0 + nl;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int p = 2 * tp + i;
    if (p >= P) continue;
    const float o[2] = {a[i][0] + a[i][1] + a[i][2], a[i][1] - a[i][2] - a[i][3]};
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int q = 2 * tq + j;
      if (q >= Q) continue;
      float v = o[j] + bv;
      if (relu) v = fmaxf(v, 0.f);
      y[((n * K + k) * P + p) * Q + q] = elem<T>::from_f32(v);
    }
  }
}

}  // namespace

hipError_t launch_wino_filter(const Shape& s, const void* w, void* U, hipStream_t stream) {
  const int64_t total = s.K * s.C;
  const dim3 grid((unsigned)((total + 255) / 256));
  if (s.dtype == DT_F32)
    hipLaunchKernelGGL(wino_filter_kernel<float>, grid, dim3(256), 0, stream, (const float*)w, (float*)U,
                       (int)s.K, (int)s.C);
  else
    hipLaunchKernelGGL(wino_filter_kernel<bf16_t>, grid, dim3(256), 0, stream, (const bf16_t*)w, (bf16_t*)U,
                       (int)s.K, (int)s.C);
  return hipGetLastError();
}

hipError_t launch_wino_input(const Shape& s, const void* x, void* V, int64_t n0, int64_t nb,
                             hipStream_t stream) {
  if (s.dtype == DT_F32) launch_wino_input_typed<float>(s, x, V, n0, nb, stream);
  else launch_wino_input_typed<bf16_t>(s, x, V, n0, nb, stream);
  return hipGetLastError();
}

hipError_t launch_wino_output(const Shape& s, const float* M, const void* b, void* y, int64_t n0, int64_t nb,
                              hipStream_t stream) {
  const int TP = (int)((s.P + 1) / 2), TQ = (int)((s.Q + 1) / 2);
  const int64_t Tc = nb * TP * TQ;
  const int64_t total = s.K * Tc;
  const dim3 grid((unsigned)((total + 255) / 256));
  if (s.dtype == DT_F32)
    hipLaunchKernelGGL(wino_output_kernel<float>, grid, dim3(256), 0, stream, M, (const float*)b, (float*)y,
                       (int)s.K, (int)s.P, (int)s.Q, TP, TQ, n0, Tc, s.relu ? 1 : 0);
  else
    hipLaunchKernelGGL(wino_output_kernel<bf16_t>, grid, dim3(256), 0, stream, M, (const bf16_t*)b,
                       (bf16_t*)y, (int)s.K, (int)s.P, (int)s.Q, TP, TQ, n0, Tc, s.relu ? 1 : 0);
  return hipGetLastError();
}

}  // namespace convsel
