// IM2COL (paper, Sec. II-B item (a); the "GEMM" algorithm of Sec. V-B item
// (c)): the column matrix that turns the convolution into a matrix product.
// Layout [image][group][P*Q][Cg*R*S]: one row per output pixel holding its
// receptive field in (c, r, s) order, zero where it leaves the image, so both
// GEMM operands (filters K x Cg*R*S and this matrix) are contiguous along the
// reduction.  A pure gather: every element is a bit copy of an input element.
//
// A workgroup writes a run of whole rows; consecutive threads write
// consecutive elements (coalesced stores), and the reads of neighbouring taps
// of one row fall on neighbouring input columns.
#include <algorithm>

#include "common.hpp"
#include "kernels.hpp"

namespace convsel {

namespace {

struct Im2colArgs {
  const void* x;
  void* col;
  int C, H, W, R, S, P, Q;
  int sh, sw, ph, pw, dh, dw;
  int G, Cg;
  int64_t n0;
  int64_t rows;       // nb * G * P * Q
  int rows_per_block;
};

template <typename T>
__global__ __launch_bounds__(256) void im2col_kernel(Im2colArgs a) {
  const int RS = a.R * a.S;
  const int crs = a.Cg * RS;
  const int PQ = a.P * a.Q;
  const int64_t row0 = static_cast<int64_t>(blockIdx.x) * a.rows_per_block;
  const int64_t rows_here = min(static_cast<int64_t>(a.rows_per_block), a.rows - row0);
  const int count = static_cast<int>(rows_here) * crs;
  const T* x = reinterpret_cast<const T*>(a.x);
  T* col = reinterpret_cast<T*>(a.col) + row0 * crs;
  for (int e = threadIdx.x; e < count; e += 256) {
    const int rl = e / crs, ci = e - rl * crs;
    const int64_t row = row0 + rl;
    const int pq = static_cast<int>(row % PQ);
    const int64_t ng = row / PQ;
    const int g = static_cast<int>(ng % a.G);
    const int64_t n = a.n0 + ng / a.G;
    const int c = ci / RS, rs = ci - c * RS;
    const int r = rs / a.S, s = rs - r * a.S;
    const int p = pq / a.Q, q = pq - p * a.Q;
    const int ih = p * a.sh - a.ph + r * a.dh, iw = q * a.sw - a.pw + s * a.dw;
    T v = elem<T>::from_f32(0.f);
    if (ih >= 0 && ih < a.H && iw >= 0 && iw < a.W)
      v = x[((n * a.C + g * a.Cg + c) * a.H + ih) * a.W + iw];
    col[e] = v;
  }
}

// The same matrix when a row's length Cg*R*S is a multiple of the 16-byte
// unit.  A workgroup owns PR x QT output pixels of one (image, group) and CC
// of its channels.  It stages the input rows those pixels read once in LDS,
// zero padding included, and then writes 16-byte units (UE consecutive
// (c, r, s) elements of one pixel) straight from there.  A thread keeps one
// unit position within the row for all its pixels, so the UE LDS offsets of
// its elements are worked out once and a unit costs UE LDS reads at
// constant offsets from its pixel's, the packing and one store.
//
// What bounds it: the column matrix's own bytes, R*S times the input, written
// once.  128 channels of 28 x 28, 3 x 3, 32 images, bf16 (57.8 MB written):
// 20.8 us, 2.8 TB/s, where a fill of that size takes 10; the rest is the
// staging round trips before the first store.  (Gathering each element from
// global memory with its own bounds check and tap step, as the kernel below
// does, took 57.8 us.)
struct Im2colTile {
  int CC, chunks;            // channels per workgroup, channel chunks per group
  int PR, QT, ptiles, qtiles;
  int IR, IC;                // staged input rows and columns per channel
  int plane;                 // LDS elements per channel: IR * IC rounded up to an odd number of banks
  int CU;                    // 16-byte units per pixel and full chunk
  uint32_t ir_magic, ic_magic;  // ceil(2^32 / d), 0 for d = 1: e / d for e < 2^16 as a high multiply
};

__device__ __forceinline__ int div_magic(int e, uint32_t m) {
  return m ? static_cast<int>(__umulhi(static_cast<uint32_t>(e), m)) : e;
}

template <typename T>
__global__ __launch_bounds__(256) void im2col_lds_kernel(Im2colArgs a, Im2colTile t) {
  constexpr int UE = elem<T>::per16;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ uint2 table[64];
  T* tile = reinterpret_cast<T*>(smem_raw);
  const int tid = threadIdx.x;
  // Pixel tiles fastest, then channel chunks, then (image, group).
  int b = blockIdx.x;
  const int qt = b % t.qtiles;
  b /= t.qtiles;
  const int pt = b % t.ptiles;
  b /= t.ptiles;
  const int chunk = b % t.chunks;
  const int ng = b / t.chunks;
  const int g = ng % a.G;
  const int64_t n = a.n0 + ng / a.G;
  const int p0 = pt * t.PR, q0 = qt * t.QT, c0 = chunk * t.CC;
  const int cc = min(t.CC, a.Cg - c0);
  const int pr = min(t.PR, a.P - p0), qn = min(t.QT, a.Q - q0);
  const T* x = reinterpret_cast<const T*>(a.x) + (n * a.C + g * a.Cg + c0) * static_cast<int64_t>(a.H) * a.W;
  const int h0 = p0 * a.sh - a.ph, w0 = q0 * a.sw - a.pw;
  const int count = cc * t.IR * t.IC;
  // Sixteen elements per thread in flight at a time.
  for (int e0 = tid; e0 < count; e0 += 16 * 256) {
    T v[16];
    int lo[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int e = e0 + i * 256;
      const int row = div_magic(e, t.ic_magic);
      const int col = e - row * t.IC;
      const int c = div_magic(row, t.ir_magic);
      const int ih = h0 + row - c * t.IR, iw = w0 + col;
      const bool in = e < count && ih >= 0 && ih < a.H && iw >= 0 && iw < a.W;
      v[i] = x[in ? (static_cast<int64_t>(c) * a.H + ih) * a.W + iw : 0];
      if (!in) v[i] = elem<T>::from_f32(0.f);
      lo[i] = e + c * (t.plane - t.IR * t.IC);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (e0 + i * 256 < count) tile[lo[i]] = v[i];
  }
  // Per pixel of the tile: LDS byte offset of its first tap, row of the image's column matrix.
  const int pixels = pr * qn;
  if (tid < pixels) {
    const int pl = tid / qn, ql = tid - pl * qn;
    table[tid] = make_uint2(static_cast<uint32_t>(pl * a.sh * t.IC + ql * a.sw) * sizeof(T),
                            static_cast<uint32_t>((p0 + pl) * a.Q + q0 + ql));
  }
  __syncthreads();

  const int RS = a.R * a.S;
  const int cu_here = cc * RS / UE;
  const int slots = 256 / t.CU;  // pixels written per pass
  const int cu = tid % t.CU, slot = tid / t.CU;
  if (slot >= slots || cu >= cu_here) return;
  uint32_t off[UE];  // byte offsets of this thread's elements from a pixel's first tap
#pragma unroll
  for (int i = 0; i < UE; ++i) {
    const int ci = cu * UE + i;
    const int c = ci / RS, rs = ci - c * RS;
    const int r = rs / a.S, s = rs - r * a.S;
    off[i] = static_cast<uint32_t>(c * t.plane + r * a.dh * t.IC + s * a.dw) * sizeof(T);
    asm volatile("" : "+v"(off[i]));  // one register each: the loop below only adds the pixel's offset
  }
  const uint32_t crs = static_cast<uint32_t>(a.Cg * RS);
  T* col = reinterpret_cast<T*>(a.col) + static_cast<int64_t>(ng) * a.P * a.Q * crs + c0 * RS + cu * UE;
  auto unit = [&](const uint2 px) {
    uint32_t e[UE];
#pragma unroll
    for (int i = 0; i < UE; ++i) e[i] = load_bits(reinterpret_cast<const T*>(smem_raw + (px.x + off[i])));
    vec16 v;
    pack16<T>(v, e);
    return v;
  };
  int px = slot;
  for (; px + slots < pixels; px += 2 * slots) {  // two units in flight
    const uint2 t0 = table[px], t1 = table[px + slots];
    const vec16 v0 = unit(t0), v1 = unit(t1);
    store16(col + static_cast<uint64_t>(t0.y) * crs, v0);
    store16(col + static_cast<uint64_t>(t1.y) * crs, v1);
  }
  if (px < pixels) {
    const uint2 t0 = table[px];
    store16(col + static_cast<uint64_t>(t0.y) * crs, unit(t0));
  }
}

// Tile of the LDS gather, or false where it does not serve the layer: rows
// that are no whole units, or filters so large that eight channels' units
// exceed a workgroup or their input rows 64 KiB of LDS.
bool im2col_tile(const Shape& s, Im2colTile& t) {
  const int ue = s.dtype == DT_F32 ? 4 : 8;
  const int64_t RS = s.R * s.S;
  if (s.Cg * RS % ue != 0) return false;
  // Channels: 128-byte multiples of the row (whole cache lines), at most a
  // workgroup's 256 units per pixel; all of them where there are fewer.
  int64_t cc = 512 / s.esize() / 4;  // 64 bf16, 32 fp32
  while (cc > ue && cc * RS / ue > 256) cc /= 2;
  if (cc >= s.Cg) cc = s.Cg;
  if (cc * RS / ue > 256) return false;
  // Pixels: rows of at most 64 columns, about 64 pixels (enough workgroups
  // for the CUs at the usual batches, and 16 to 64 units per thread).
  int64_t qt = s.Q < 64 ? s.Q : 64;
  int64_t pr = 64 / qt;
  if (pr < 1) pr = 1;
  if (pr > s.P) pr = s.P;
  const size_t limit = 60 * 1024;  // (the padding below adds at most three elements a channel)
  for (;;) {
    t.IR = (int)((pr - 1) * s.sh + (s.R - 1) * s.dh + 1);
    t.IC = (int)((qt - 1) * s.sw + (s.S - 1) * s.dw + 1);
    if ((size_t)cc * t.IR * t.IC * s.esize() <= limit && cc * t.IR * t.IC < 65536) break;
    if (pr > 1) pr = (pr + 1) / 2;
    else if (qt > 8) qt = (qt + 1) / 2;
    else if (cc > ue && cc % (2 * ue) == 0) cc /= 2;
    else return false;
  }
  // The lanes of a wave read one tap position of up to 64 consecutive
  // channels: an odd channel pitch in 4-byte banks keeps them apart.
  t.plane = s.dtype == DT_F32 ? (t.IR * t.IC) | 1 : (t.IR * t.IC + 1) / 2 * 2;
  if (s.dtype != DT_F32 && t.plane % 4 == 0) t.plane += 2;
  t.CC = (int)cc;
  t.chunks = (int)((s.Cg + cc - 1) / cc);
  t.PR = (int)pr;
  t.QT = (int)qt;
  t.ptiles = (int)((s.P + pr - 1) / pr);
  t.qtiles = (int)((s.Q + qt - 1) / qt);
  t.CU = (int)(cc * RS / ue);
  auto magic = [](int d) { return d == 1 ? 0u : (uint32_t)((((uint64_t)1 << 32) + d - 1) / d); };
  t.ir_magic = magic(t.IR);
  t.ic_magic = magic(t.IC);
  return true;
}

// The same matrix for the remaining layers whose rows are whole units
// (im2col_route): one thread per 16-byte unit of a row, consecutive threads along
// the row; the UE input elements are gathered with the tap indices stepped
// incrementally.
template <typename T>
__global__ __launch_bounds__(256) void im2col_vec_kernel(Im2colArgs a, int64_t units) {
  constexpr int UE = elem<T>::per16;
  const int RS = a.R * a.S;
  const int CU = a.Cg * RS / UE;  // units per row
  const int PQ = a.P * a.Q;
  const T* x = reinterpret_cast<const T*>(a.x);
  for (int64_t u = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; u < units;
       u += static_cast<int64_t>(gridDim.x) * 256) {
    const int64_t row = u / CU;
    const int cu = static_cast<int>(u - row * CU);
    const int pq = static_cast<int>(row % PQ);
    const int64_t ng = row / PQ;
    const int g = static_cast<int>(ng % a.G);
    const int64_t n = a.n0 + ng / a.G;
    const int p = pq / a.Q, q = pq - p * a.Q;
    const int ci0 = cu * UE;
    int c = ci0 / RS, rs = ci0 - c * RS;
    int r = rs / a.S, s = rs - r * a.S;
    const T* xn = x + (n * a.C + g * a.Cg) * static_cast<int64_t>(a.H) * a.W;
    const int h0 = p * a.sh - a.ph, w0 = q * a.sw - a.pw;
    uint32_t e[UE];
#pragma unroll
    for (int t = 0; t < UE; ++t) {
      const int ih = h0 + r * a.dh, iw = w0 + s * a.dw;
      const bool in = ih >= 0 && ih < a.H && iw >= 0 && iw < a.W;
      const uint32_t bits = load_bits(xn + (in ? (static_cast<int64_t>(c) * a.H + ih) * a.W + iw : 0));
      e[t] = in ? bits : 0u;
      if (++s == a.S) {
        s = 0;
        if (++r == a.R) {
          r = 0;
          ++c;
        }
      }
    }
    vec16 v;
    pack16<T>(v, e);
    store16(reinterpret_cast<T*>(a.col) + u * UE, v);
  }
}

}  // namespace

namespace {

enum Im2colKernel { IM2COL_LDS, IM2COL_VEC, IM2COL_ELEM };

// The kernel for the column matrix of nb images (`aligned`: col is 16-byte
// aligned), and its tile.
Im2colKernel im2col_route(const Shape& s, int64_t nb, bool aligned, Im2colTile& t) {
  const int64_t crs = s.Cg * s.R * s.S, ue = s.dtype == DT_F32 ? 4 : 8;
  if (!aligned || crs % ue != 0) return IM2COL_ELEM;
  const int64_t units = nb * s.G * s.P * s.Q * crs / ue;
  if (s.R * s.S == 1 || !im2col_tile(s, t)) return IM2COL_VEC;
  // Where the LDS tiles pay (the gather alone, 400 random layers, both ways):
  //  * not for single taps, which read every element once: 0.5 times as fast at
  //    best, and a hundredth on 1 x 1 planes;
  //  * with 750 units for a workgroup to write on average, which its setup and
  //    its staging round trip are spread over (fewer on small planes or with few
  //    channels: 92 channels a group of 2 x 2, 3 x 3 taps, 24.5 us by units,
  //    52.0 by tiles; 4 a group of 3 x 3, 17.9 and 121);
  //  * not for filters one column wide over single output rows, whose tiles
  //    hold no pixel twice (7 x 1, 320 channels of 71 x 71, 25 and 40 us);
  //  * with enough units in all (13 MB in bf16, 19 MB in fp32, whose units cost
  //    the other kernel half as many loads): below, a unit per thread fills
  //    the chip at once (one 64-channel 56 x 56 image, bf16, 3 x 3, with its product
  //    12.0 us by units, 17.9 by tiles; 12 channels of 78 x 78, fp32, 9.2 and 10.2).
  // Above these lines the tiles took 0.26 to 1.1 times as long, median 0.6.
  const int64_t blocks = nb * s.G * t.chunks * t.ptiles * t.qtiles;
  const bool once = s.S == 1 && t.IR * t.IC * 20 > t.PR * t.QT * s.R * 17;
  if (units < (s.dtype == DT_F32 ? 1200000 : 800000) || units < 750 * blocks || once) return IM2COL_VEC;
  return blocks < ((int64_t)1 << 31) ? IM2COL_LDS : IM2COL_VEC;
}

}  // namespace

hipError_t launch_im2col(const Shape& s, const void* x, void* col, int64_t n0, int64_t nb,
                         hipStream_t stream) {
  Im2colArgs a;
  a.x = x; a.col = col;
  a.C = (int)s.C; a.H = (int)s.H; a.W = (int)s.W; a.R = (int)s.R; a.S = (int)s.S;
  a.P = (int)s.P; a.Q = (int)s.Q;
  a.sh = s.sh; a.sw = s.sw; a.ph = s.ph; a.pw = s.pw; a.dh = s.dh; a.dw = s.dw;
  a.G = s.G; a.Cg = (int)s.Cg;
  a.n0 = n0;
  a.rows = nb * s.G * s.P * s.Q;
  const int64_t crs = s.Cg * s.R * s.S;
  Im2colTile t;
  const Im2colKernel kernel = im2col_route(s, nb, reinterpret_cast<uintptr_t>(col) % 16 == 0, t);
  if (kernel == IM2COL_LDS) {
    const int64_t blocks = nb * s.G * t.chunks * t.ptiles * t.qtiles;
    const size_t lds = (size_t)t.CC * t.plane * s.esize();
    if (s.dtype == DT_F32)
      hipLaunchKernelGGL(im2col_lds_kernel<float>, dim3((unsigned)blocks), dim3(256), lds, stream, a, t);
    else
      hipLaunchKernelGGL(im2col_lds_kernel<bf16_t>, dim3((unsigned)blocks), dim3(256), lds, stream, a, t);
    return hipGetLastError();
  }
  if (kernel == IM2COL_VEC) {
    const int64_t units = a.rows * (crs * s.esize() / 16);
    const int64_t blocks = std::min<int64_t>((units + 255) / 256, 65536);
    if (s.dtype == DT_F32)
      hipLaunchKernelGGL(im2col_vec_kernel<float>, dim3((unsigned)blocks), dim3(256), 0, stream, a, units);
    else
      hipLaunchKernelGGL(im2col_vec_kernel<bf16_t>, dim3((unsigned)blocks), dim3(256), 0, stream, a, units);
    return hipGetLastError();
  }
  a.rows_per_block = (int)(4096 / crs > 0 ? 4096 / crs : 1);
  const int64_t blocks = (a.rows + a.rows_per_block - 1) / a.rows_per_block;
  if (s.dtype == DT_F32)
    hipLaunchKernelGGL(im2col_kernel<float>, dim3((unsigned)blocks), dim3(256), 0, stream, a);
  else
    hipLaunchKernelGGL(im2col_kernel<bf16_t>, dim3((unsigned)blocks), dim3(256), 0, stream, a);
  return hipGetLastError();
}

const char* im2col_describe(const Shape& s, int64_t nb) {
  Im2colTile t;
  static const char* const names[] = {"im2col_lds_kernel", "im2col_vec_kernel", "im2col_kernel"};
  return names[im2col_route(s, nb, true, t)];
}

}  // namespace convsel
