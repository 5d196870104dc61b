// Batched MFMA GEMM with both operands reduction-contiguous ("NT"):
//   C[b][i][j] = sum_k A[b][i][k] * B[b][j][k]  (+ bias[i], ReLU)
// It is the multiply step of IM2COL + GEMM (A = filters, B = the column
// matrix, C = one image's output planes) and the 16 elementwise-product
// GEMMs of Winograd (A = U, B = V, C = M).  With `b_kmajor` set, B is read
// as B[b][k][j] instead (column-contiguous: an NCHW image as channels x
// pixels), which is the multiply step of KN2ROW; its tile is transposed on
// the way into LDS.
//
// Tiling: 256 threads = 4 waves in a 2 x 2 grid; a BM x BN tile per
// workgroup, (BM/2) x (BN/2) per wave as 32 x 32 MFMA blocks.  Each k-tile of
// BK reduction elements is staged in LDS as rows of BK (+ 16 bytes padding:
// an 80-byte row stride, an odd multiple of 16 bytes, so the per-lane 16-byte
// fragment reads of 32 consecutive rows hit distinct bank groups).  The next
// k-tile is fetched into registers while the MFMAs run on the current one.
#include <stdio.h>

#include <string>

#include "common.hpp"
#include "igemm_common.hpp"
#include "kernels.hpp"

namespace convsel {

namespace {

using namespace igemm;

constexpr int kThreads = 256;

template <typename T, int BM, int BN, bool VEC, bool OUT_F32, bool BKM>
__global__ __launch_bounds__(kThreads) void gemm_nt_kernel(GemmArgs g, int batch_base) {
  constexpr int UE = elem<T>::per16;  // elements per 16-byte unit
  constexpr int BK = 4 * UE;          // 32 bf16 or 16 fp32: two MFMA steps
  constexpr int KP = BK + UE;         // padded LDS row (elements)
  constexpr int UPR = BK / UE;        // 16-byte units per row = 4
  constexpr int UA = BM * UPR / kThreads;
  constexpr int UB = BN * UPR / kThreads;
  constexpr int MI = BM / 64, NJ = BN / 64;
  static_assert(UA >= 1 && UB >= 1, "tile too small");

  __shared__ __align__(16) T As[BM * KP];
  __shared__ __align__(16) T Bs[BN * KP];

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int i0 = blockIdx.y * BM, j0 = blockIdx.x * BN;
  const int b = batch_base + blockIdx.z;
  const int b0 = b / g.bdiv, b1 = b - b0 * g.bdiv;
  const T* A = reinterpret_cast<const T*>(g.A) + b0 * g.sA0 + b1 * g.sA1;
  const T* B = reinterpret_cast<const T*>(g.B) + b0 * g.sB0 + b1 * g.sB1;

  vec16 ra[UA], rb[UB];

  // One 16-byte unit (UE consecutive reduction elements) of row `row` of a
  // row-major operand, zero outside rows < nrows and k < Kred.  Loads are
  // unconditional from a valid address and masked afterwards, so a thread's
  // loads are all in flight together.
  auto load_unit = [&](const T* base, int row, int k, int nrows, int64_t ld) -> vec16 {
    if (VEC) {
      const bool ok = row < nrows && k < g.Kred;
      const vec16 v = load16(base + (ok ? row * ld + k : 0));
      vec16 r;
#pragma unroll
      for (int i = 0; i < 4; ++i) r.d[i] = ok ? v.d[i] : 0u;
      return r;
    } else {
      uint32_t e[UE];
#pragma unroll
      for (int i = 0; i < UE; ++i) {
        const bool ok = row < nrows && k + i < g.Kred;
        const uint32_t bits = load_bits(base + (ok ? row * ld + k + i : 0));
        e[i] = ok ? bits : 0u;
      }
      vec16 r;
      pack16<T>(r, e);
      return r;
    }
  };

  auto fetch = [&](int kt) {
    const int k0 = kt * BK;
#pragma unroll
    for (int u = 0; u < UA; ++u) {
      const int id = tid + u * kThreads;
      const int row = id / UPR, kc = (id % UPR) * UE;
      const int gi = i0 + row, gk = k0 + kc;
      ra[u] = load_unit(A, gi, gk, g.M, g.lda);
    }
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      const int id = tid + u * kThreads;
      if constexpr (BKM) {
        // UE consecutive columns of reduction row kr.
        const int kr = id / (BN / UE), jc = id % (BN / UE);
        const int gk = k0 + kr, gj = j0 + jc * UE;
        if (VEC && gk < g.Kred && gj + UE <= g.N) {
          rb[u] = load16(B + gk * g.ldb + gj);
        } else {
          uint32_t e[UE];
#pragma unroll
          for (int i = 0; i < UE; ++i) {
            const bool ok = gk < g.Kred && gj + i < g.N;
            const uint32_t bits = load_bits(B + (ok ? gk * g.ldb + gj + i : 0));
            e[i] = ok ? bits : 0u;
          }
          pack16<T>(rb[u], e);
        }
      } else {
        const int row = id / UPR, kc = (id % UPR) * UE;
        const int gj = j0 + row, gk = k0 + kc;
        rb[u] = load_unit(B, gj, gk, g.N, g.ldb);
      }
    }
  };
  auto stash = [&]() {
#pragma unroll
    for (int u = 0; u < UA; ++u) {
      const int id = tid + u * kThreads;
      store16(&As[(id / UPR) * KP + (id % UPR) * UE], ra[u]);
    }
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      const int id = tid + u * kThreads;
      if constexpr (BKM) {
        const int kr = id / (BN / UE), jc = id % (BN / UE);
#pragma unroll
        for (int i = 0; i < UE; ++i) Bs[(jc * UE + i) * KP + kr] = vec16_get<T>(rb[u], i);
      } else {
        store16(&Bs[(id / UPR) * KP + (id % UPR) * UE], rb[u]);
      }
    }
  };

  f32x16_t acc[MI][NJ];
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int nj = 0; nj < NJ; ++nj) acc[mi][nj] = zero16();

  const int nk = (g.Kred + BK - 1) / BK;
  fetch(0);
  stash();
  lds_sync();
  const int half = lane >> 5, l32 = lane & 31;
  for (int kt = 0; kt < nk; ++kt) {
    if (kt + 1 < nk) fetch(kt + 1);
#pragma unroll
    for (int st = 0; st < 2; ++st) {
      const int kofs = st * 2 * UE + half * UE;
      vec16 af[MI], bfr[NJ];
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) af[mi] = load16(&As[(wm * (BM / 2) + mi * 32 + l32) * KP + kofs]);
#pragma unroll
      for (int nj = 0; nj < NJ; ++nj) bfr[nj] = load16(&Bs[(wn * (BN / 2) + nj * 32 + l32) * KP + kofs]);
#pragma unroll
      for (int mi = 0; mi < MI; ++mi)
#pragma unroll
        for (int nj = 0; nj < NJ; ++nj) mfma_32x32<T>(acc[mi][nj], af[mi], bfr[nj]);
    }
    lds_sync();
    if (kt + 1 < nk) {
      stash();
      lds_sync();
    }
  }

  // Epilogue: bias, ReLU, store.  Lanes 0-31 write 32 consecutive j of one
  // row i, lanes 32-63 the same columns of row i+4.
  const int64_t cofs = b0 * g.sC0 + b1 * g.sC1;
  const T* bias = g.bias ? reinterpret_cast<const T*>(g.bias) + b1 * g.sBias1 : nullptr;
#pragma unroll
  for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
    for (int nj = 0; nj < NJ; ++nj) {
      const int j = j0 + wn * (BN / 2) + nj * 32 + l32;
      if (j >= g.N) continue;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int i = i0 + wm * (BM / 2) + mi * 32 + mfma_row(v, lane);
        if (i >= g.M) continue;
        float val = acc[mi][nj][v];
        if (bias) val += elem<T>::load(bias + i);
        if (g.relu) val = fmaxf(val, 0.f);
        const int64_t o = cofs + static_cast<int64_t>(i) * g.ldc + j;
        if (OUT_F32)
          reinterpret_cast<float*>(g.C)[o] = val;
        else
          elem<T>::store(reinterpret_cast<T*>(g.C) + o, val);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// "NT" GEMM through LDS DMA (both operands reduction-contiguous, 16-byte
// aligned rows, Kred whole 16-byte units).  The MFMA's A operand is a row of B
// (a pixel of IM2COL's column matrix, a Winograd tile) and its B operand a
// row of A (a filter), so each lane ends with four consecutive j of one i:
// the output row's order.
//
// A workgroup (4 waves, WJ x WI) owns TJ rows of B x TI rows of A and walks
// the reduction in k-tiles of 128 bytes (64 bf16, 32 fp32).  A k-tile stage
// is the TJ + TI rows of 128 bytes, two rows per 256-byte line with the
// 16-byte unit u of row r at position 8 (r & 1) + (u ^ ((r >> 1) & 7)) of line
// r >> 1, so 16 lanes reading one unit of 16 consecutive rows hit 16 distinct
// bank groups.  The stage is filled by `buffer_load ... lds` (no register
// round trip): DMA instruction J writes the stage's 16-byte units J*64 ..
// J*64+63, and each lane fetches the unit that the layout puts at its place
// (rows past the operand and reduction elements past Kred read zeros through
// the buffer range).  NST stages form a ring with NST - 1 k-tiles in flight
// and one barrier per k-tile.
//
// What bounds it: short reductions (4 to 18 k-tiles) make the first tile's
// latency and the epilogue half of a workgroup's time, so what counts is how
// many workgroups share a CU: two stages, 32 or 48 KiB of LDS, 5 or 3
// workgroups per CU for the 64 x 64 and 128 x 64 tiles.  VGG's 256 -> 256
// 56 x 56 fp32 layer (Winograd, 16 products of 256 x 6272 x 256): 160 us with
// the register-staged kernel above, 195 (four stages, 64 x 64), 130 (two
// stages); the fp32 matrix units' own time is 86 us.
template <int TJ, int TI, int WJ_, int NST_>
struct GemmDmaShape {
  static constexpr int WJ = WJ_;
  static constexpr int WI = 4 / WJ;
  static constexpr int MJ = TJ / WJ / 32, NI = TI / WI / 32;  // 32 x 32 blocks per wave
  static constexpr int ROWS = TJ + TI;
  static constexpr int STAGE = ROWS * 128;
  static constexpr int NST = NST_;
  static constexpr int NDMA = ROWS / 8 / 4;  // DMA instructions per wave and stage
  static_assert(WJ * WI == 4 && MJ >= 1 && NI >= 1 && TJ % 32 == 0 && TI % 32 == 0 && ROWS % 32 == 0, "tile");
  static_assert(NST * STAGE <= 160 * 1024 && NDMA * (NST - 1) <= 63, "stages");
};

template <typename T, int TJ, int TI, int WJ, int NST_, bool OUT_F32>
__global__ __launch_bounds__(256) void gemm_dma_kernel(GemmArgs g, int njt, int nit, uint32_t a_bytes,
                                                       uint32_t b_bytes) {
  using Sh = GemmDmaShape<TJ, TI, WJ, NST_>;
  constexpr int MJ = Sh::MJ, NI = Sh::NI, NST = Sh::NST, NDMA = Sh::NDMA, STAGE = Sh::STAGE;
  constexpr int ES = elem<T>::bytes, UE = elem<T>::per16, BK = 128 / ES;  // a k-tile is 128 bytes of a row
  extern __shared__ __align__(16) vec16 smem[];
  char* lds = reinterpret_cast<char*>(smem);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wj = wave % Sh::WJ, wi = wave / Sh::WJ;
  // Work units (batch item, j tile, i tile; i fastest) are dealt to the eight
  // XCDs in contiguous ranges (workgroup w runs on XCD w % 8): the i tiles
  // that read one j tile's rows of B follow each other on one L2.
  const int units = njt * nit * g.batch;
  const int per_xcd = (units + 7) >> 3;
  const int unit = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (unit >= units) return;  // uniform
  const int jt = unit / nit;
  const int b = jt / njt;
  const int j0 = (jt - b * njt) * TJ, i0 = (unit - jt * nit) * TI;
  const int b0 = b / g.bdiv, b1 = b - b0 * g.bdiv;
  const T* A = reinterpret_cast<const T*>(g.A) + b0 * g.sA0 + b1 * g.sA1;
  const T* B = reinterpret_cast<const T*>(g.B) + b0 * g.sB0 + b1 * g.sB1;
  const u32x4_t ar = dma_rsrc(A, a_bytes), br = dma_rsrc(B, b_bytes);
  const uint32_t lds0 = lds_address(lds);

  // This wave's DMA instructions: J = wave * NDMA + d.  Instructions below
  // TJ / 8 fill rows of B, the rest rows of A (a row boundary never falls
  // inside one: 64 units are 8 whole rows).
  uint32_t dvo[NDMA];
  int dku[NDMA];
#pragma unroll
  for (int d = 0; d < NDMA; ++d) {
    const int U = (wave * NDMA + d) * 64 + lane;
    const int line = U >> 4, pos = U & 15;
    const int row = 2 * line + (pos >> 3), u = (pos & 7) ^ (line & 7);
    const bool isb = row < TJ;
    const int grow = isb ? j0 + row : i0 + row - TJ;
    const bool ok = grow < (isb ? g.N : g.M);
    const int64_t ld = isb ? g.ldb : g.lda;
    dvo[d] = ok ? static_cast<uint32_t>((grow * ld + u * UE) * ES) : (isb ? b_bytes : a_bytes);
    dku[d] = u * UE;
  }
  const int nk = (g.Kred + BK - 1) / BK;
  auto issue = [&](int kt) {
    const uint32_t st = lds0 + (kt % NST) * STAGE;
    const uint32_t so = static_cast<uint32_t>(kt) * 128;
    const bool tail = (kt + 1) * BK > g.Kred;
#pragma unroll
    for (int d = 0; d < NDMA; ++d) {
      const int J = wave * NDMA + d;
      const bool isb = J < TJ / 8;
      const uint32_t vo = (!tail || kt * BK + dku[d] < g.Kred) ? dvo[d] : (isb ? b_bytes : a_bytes);
      dma16(isb ? br : ar, st + J * 1024, vo, so);
    }
  };

  // Fragment offsets within a stage: unit 2 t + half of row r.
  const int half = lane >> 5, l32 = lane & 31;
  auto frag = [&](int r, int u) { return (r >> 1) * 256 + ((8 * (r & 1) + (u ^ ((r >> 1) & 7))) << 4); };
  int aoff[MJ][4], boff[NI][4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
#pragma unroll
    for (int mj = 0; mj < MJ; ++mj) aoff[mj][t] = frag((wj * MJ + mj) * 32 + l32, 2 * t + half);
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) boff[ni][t] = frag(TJ + (wi * NI + ni) * 32 + l32, 2 * t + half);
  }

  f32x16_t acc[MJ][NI];
#pragma unroll
  for (int mj = 0; mj < MJ; ++mj)
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) acc[mj][ni] = zero16();

#pragma unroll
  for (int p = 0; p < NST - 1; ++p)
    if (p < nk) issue(p);
  for (int kt = 0; kt < nk; ++kt) {
    // k-tile kt has landed once at most the later tiles' DMAs are pending.
    const int later = min(nk - 1, kt + NST - 2) - kt;
    if (later >= 2 && NST == 4) CONVSEL_WAIT_VMCNT(2 * NDMA);
    else if (later >= 1) CONVSEL_WAIT_VMCNT(NDMA);
    else CONVSEL_WAIT_VMCNT(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();  // every wave's part of tile kt is in; every wave is done with tile kt - 1
    asm volatile("" ::: "memory");
    if (kt + NST - 1 < nk) issue(kt + NST - 1);  // into the stage of tile kt - 1
    const char* st = lds + (kt % NST) * STAGE;
    vec16 fa[2][MJ], fb[2][NI];
    auto read = [&](auto t_c) {
      constexpr int t = decltype(t_c)::value;
#pragma unroll
      for (int mj = 0; mj < MJ; ++mj) fa[t & 1][mj] = *reinterpret_cast<const vec16*>(st + aoff[mj][t]);
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) fb[t & 1][ni] = *reinterpret_cast<const vec16*>(st + boff[ni][t]);
    };
    read(std::integral_constant<int, 0>{});
    static_for<4>([&](auto t_c) {
      constexpr int t = decltype(t_c)::value;
      if constexpr (t + 1 < 4) read(std::integral_constant<int, t + 1>{});
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int d = 0; d < 4; ++d)
#pragma unroll
          for (int mj = 0; mj < MJ; ++mj)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
              acc[mj][ni] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(fa[t & 1][mj].d[d]),
                                                                 __uint_as_float(fb[t & 1][ni].d[d]), acc[mj][ni], 0, 0, 0);
      } else {
#pragma unroll
        for (int mj = 0; mj < MJ; ++mj)
#pragma unroll
          for (int ni = 0; ni < NI; ++ni) mfma_32x32<T>(acc[mj][ni], fa[t & 1][mj], fb[t & 1][ni]);
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  }

  // Epilogue: bias (per i), ReLU, four consecutive j per store.
  const int64_t cofs = b0 * g.sC0 + b1 * g.sC1;
  const T* bias = g.bias ? reinterpret_cast<const T*>(g.bias) + b1 * g.sBias1 : nullptr;
  const bool vst = ((cofs | g.ldc | g.sCj) & 3) == 0 && (g.jspan == 0 || g.jspan % 4 == 0) &&
                   reinterpret_cast<uintptr_t>(g.C) % 16 == 0;
  // Offset of column j in C (a folded batch maps j to its item's columns).
  auto col = [&](int j) -> int64_t {
    if (g.jspan == 0) return j;
    const int n = j / g.jspan;
    return n * g.sCj + (j - n * g.jspan);
  };
#pragma unroll
  for (int ni = 0; ni < NI; ++ni) {
    const int i = i0 + (wi * NI + ni) * 32 + l32;
    if (i >= g.M) continue;
    const float bv = bias ? elem<T>::load(bias + i) : 0.f;
    const int64_t row = cofs + static_cast<int64_t>(i) * g.ldc;
#pragma unroll
    for (int mj = 0; mj < MJ; ++mj) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int j = j0 + (wj * MJ + mj) * 32 + 8 * q + 4 * half;
        float v[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          v[t] = acc[mj][ni][4 * q + t] + bv;
          if (g.relu) v[t] = fmaxf(v[t], 0.f);
        }
        if constexpr (OUT_F32 || sizeof(T) == 4) {
          float* c = reinterpret_cast<float*>(g.C) + row;
          if (vst && j + 4 <= g.N) {
            *reinterpret_cast<float4*>(c + col(j)) = make_float4(v[0], v[1], v[2], v[3]);
          } else {
#pragma unroll
            for (int t = 0; t < 4; ++t)
              if (j + t < g.N) c[col(j + t)] = v[t];
          }
        } else {
          uint16_t* c = reinterpret_cast<uint16_t*>(g.C) + row;
          if (vst && j + 4 <= g.N) {
            *reinterpret_cast<uint2*>(c + col(j)) =
                make_uint2(f32x2_to_bf16x2(v[0], v[1]), f32x2_to_bf16x2(v[2], v[3]));
          } else {
#pragma unroll
            for (int t = 0; t < 4; ++t)
              if (j + t < g.N) c[col(j + t)] = f32_to_bf16(v[t]);
          }
        }
      }
    }
  }
}

template <typename T, int TJ, int TI, int WJ, int NST_, bool OUT_F32>
hipError_t launch_dma_tile(const GemmArgs& g, uint32_t a_bytes, uint32_t b_bytes, hipStream_t stream) {
  using Sh = GemmDmaShape<TJ, TI, WJ, NST_>;
  const auto kern = gemm_dma_kernel<T, TJ, TI, WJ, NST_, OUT_F32>;
  const size_t lds = (size_t)Sh::NST * Sh::STAGE;
  static bool attr = false;
  if (!attr) {
    const hipError_t e =
        hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    attr = true;
  }
  const int njt = (g.N + TJ - 1) / TJ, nit = (g.M + TI - 1) / TI;
  const int64_t units = (int64_t)njt * nit * g.batch;
  if (units >= ((int64_t)1 << 30)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(kern, dim3((unsigned)((units + 7) / 8 * 8)), dim3(256), lds, stream, g, njt, nit, a_bytes, b_bytes);
  return hipGetLastError();
}

// The DMA kernel serves operands whose rows are 16-byte aligned and whose
// per-batch extents fit a buffer range.
bool gemm_dma_ok(int dtype, const GemmArgs& g, uint32_t& a_bytes, uint32_t& b_bytes) {
  const int es = dtype == DT_F32 ? 4 : 2, ue = 16 / es;
  if (g.b_kmajor || g.Kred % ue != 0 || g.lda % ue != 0 || g.ldb % ue != 0) return false;
  if (g.sA0 % ue != 0 || g.sA1 % ue != 0 || g.sB0 % ue != 0 || g.sB1 % ue != 0) return false;
  if (reinterpret_cast<uintptr_t>(g.A) % 16 != 0 || reinterpret_cast<uintptr_t>(g.B) % 16 != 0) return false;
  if (g.M <= 0 || g.N <= 0 || g.Kred <= 0) return false;
  const int64_t ab = ((int64_t)(g.M - 1) * g.lda + g.Kred) * es, bb = ((int64_t)(g.N - 1) * g.ldb + g.Kred) * es;
  if (ab >= ((int64_t)1 << 31) || bb >= ((int64_t)1 << 31)) return false;
  a_bytes = (uint32_t)ab;
  b_bytes = (uint32_t)bb;
  return true;
}

// Tiles of the DMA kernel (GemmDmaShape).
struct DmaTile {
  int TJ, TI, WJ, NST;
};
constexpr DmaTile kDmaTiles[] = {{128, 256, 1, 3}, {128, 128, 2, 3}, {256, 64, 4, 3},
                                 {128, 64, 2, 2},  {64, 64, 2, 2},   {64, 64, 2, 4}};

int64_t tiles_of(const GemmArgs& g, int tj, int ti) {
  return (int64_t)((g.N + tj - 1) / tj) * ((g.M + ti - 1) / ti) * g.batch;
}

// Tile (TJ x TI) choice.  fp32: 64 x 64, whose five workgroups per CU keep the
// matrix units (a sixteenth of the bf16 rate) fed at any size (VGG block, two
// layers: 313 us against 322 to 383 with the larger tiles; whole calls of 142
// random fp32 IM2COL layers and 84 Winograd ones, against the register-staged
// kernel and the former gather and transform: 0.62 and 0.82 of the time in the
// geometric mean, at worst 1.16 and 1.10).  bf16 with at most
// 512 terms and more than two 64 x 64 tiles per CU takes those as well, several
// workgroups per CU hiding each other's start and end (504 random products: 0.81
// to 0.98 of the time with the larger tiles, at worst 1.06); longer reductions
// the largest tile whose grid fills the CUs, with TI no wider than M needs.
// Small problems take the 64 x 64 tile, and up to two workgroups per CU four
// stages (no more would share a CU at two either, and the k-tiles in flight are
// what hides their latency: 23 filters, 2350 pixels, 2160 terms, whole call 29 us
// with four stages, 35 with two; 48 filters, 20000 pixels, 288 terms 19 and 21).
int dma_tile(int dtype, const GemmArgs& g) {
  const int mr = (g.M + 63) / 64 * 64;
  if (dtype == DT_BF16 && (g.Kred > 512 || tiles_of(g, 64, 64) <= 512)) {
    if (mr >= 256 && tiles_of(g, 128, 256) >= 240) return 0;
    if (mr >= 128 && tiles_of(g, 128, 128) >= 240) return 1;
    if (tiles_of(g, 256, 64) >= 240) return 2;
    if (tiles_of(g, 128, 64) >= 240) return 3;
  }
  return tiles_of(g, 64, 64) > 512 ? 4 : 5;
}

// Products that the register-staged kernel runs faster than the DMA kernel:
// those bound by their stores.  A lane of the DMA kernel ends with four
// consecutive columns of a row, 32 rows a wave, which is four scattered stores
// instead of one where rows of C are no whole 16-byte units; its own lanes run
// along the rows.  Where its grid (128 columns, 64 or 128 rows) fills the chip
// (1176 random products, both ways, fp32 and bf16): such rows up to 256 terms 0.5
// to 1.05 of the DMA kernel's time (16 -> 106 channels of 62 x 62, Winograd, 17 images,
// fp32: 60 us against 113), up to 64 terms from 256 workgroups on, and up to 16
// terms on any large grid; rows of whole units up to 32 terms 0.7 to 1.05.  Not
// folded batches, whose items it would take one by one.
bool stores_bound(const GemmArgs& f) {
  if (f.jspan > 0) return false;
  const bool whole = f.ldc % 4 == 0 && f.sC0 % 4 == 0 && f.sC1 % 4 == 0 &&
                     reinterpret_cast<uintptr_t>(f.C) % 16 == 0;
  const int64_t grid = tiles_of(f, 128, f.M <= 64 ? 64 : 128);
  if (whole) return f.N > 1500 && grid > 512 && f.Kred <= 32;
  if (f.N > 1200 && ((grid > 340 && f.Kred <= 256) || (grid > 256 && f.Kred <= 64))) return true;
  return tiles_of(f, 64, 64) > 512 && f.Kred <= 16;
}

template <typename T, bool OUT_F32, int I>
hipError_t launch_dma_config(const GemmArgs& g, uint32_t a_bytes, uint32_t b_bytes, hipStream_t stream) {
  constexpr DmaTile t = kDmaTiles[I];
  return launch_dma_tile<T, t.TJ, t.TI, t.WJ, t.NST, OUT_F32>(g, a_bytes, b_bytes, stream);
}

template <typename T, bool OUT_F32>
hipError_t launch_dma(int tile, const GemmArgs& g, uint32_t a_bytes, uint32_t b_bytes, hipStream_t stream) {
  if (tile == 4) return launch_dma_config<T, OUT_F32, 4>(g, a_bytes, b_bytes, stream);
  if (tile == 5) return launch_dma_config<T, OUT_F32, 5>(g, a_bytes, b_bytes, stream);
  if constexpr (sizeof(T) == 2) {
    if (tile == 0) return launch_dma_config<T, OUT_F32, 0>(g, a_bytes, b_bytes, stream);
    if (tile == 1) return launch_dma_config<T, OUT_F32, 1>(g, a_bytes, b_bytes, stream);
    if (tile == 2) return launch_dma_config<T, OUT_F32, 2>(g, a_bytes, b_bytes, stream);
    if (tile == 3) return launch_dma_config<T, OUT_F32, 3>(g, a_bytes, b_bytes, stream);
  }
  return hipErrorInvalidValue;
}

template <typename T, int BM, int BN, bool OUT_F32, bool BKM>
hipError_t launch_tile(const GemmArgs& g, bool vec, hipStream_t stream) {
  const dim3 block(kThreads);
  for (int base = 0; base < g.batch; base += 65535) {
    const int nb = g.batch - base < 65535 ? g.batch - base : 65535;
    const dim3 grid((g.N + BN - 1) / BN, (g.M + BM - 1) / BM, nb);
    if (vec)
      hipLaunchKernelGGL((gemm_nt_kernel<T, BM, BN, true, OUT_F32, BKM>), grid, block, 0, stream, g, base);
    else
      hipLaunchKernelGGL((gemm_nt_kernel<T, BM, BN, false, OUT_F32, BKM>), grid, block, 0, stream, g, base);
  }
  return hipGetLastError();
}

template <typename T, bool OUT_F32>
hipError_t launch_typed(const GemmArgs& g, hipStream_t stream) {
  constexpr int UE = elem<T>::per16;
  const bool aligned = (reinterpret_cast<uintptr_t>(g.A) % 16 == 0) &&
                       (reinterpret_cast<uintptr_t>(g.B) % 16 == 0);
  const bool vec = aligned && g.lda % UE == 0 && g.ldb % UE == 0 && g.Kred % UE == 0 &&
                   g.sA0 % UE == 0 && g.sA1 % UE == 0 && g.sB0 % UE == 0 && g.sB1 % UE == 0;
  // Small M (filters per group) gets the 64-row tile so fewer MFMA rows idle.
  if (g.b_kmajor) {
    if (g.M <= 64) return launch_tile<T, 64, 128, OUT_F32, true>(g, vec, stream);
    return launch_tile<T, 128, 128, OUT_F32, true>(g, vec, stream);
  }
  if (g.M <= 64) return launch_tile<T, 64, 128, OUT_F32, false>(g, vec, stream);
  return launch_tile<T, 128, 128, OUT_F32, false>(g, vec, stream);
}

// How a product runs: the tile of the DMA kernel, or -1 for the register-staged
// one; `f` receives the arguments for the former.
int gemm_route(int dtype, const GemmArgs& g, GemmArgs& f, uint32_t& a_bytes, uint32_t& b_bytes) {
  // A batch that shares A and whose B items are consecutive rows is folded
  // into N when the items are narrow (IM2COL's small planes), so that the
  // tiles are full and the grid holds enough workgroups.
  f = g;
  if (g.batch > 1 && g.bdiv == 1 && g.sA0 == 0 && g.sB0 == (int64_t)g.N * g.ldb && g.N < 1024 &&
      (int64_t)g.N * g.batch < ((int64_t)1 << 31)) {
    f.jspan = g.N;
    f.sCj = g.sC0;
    f.N = g.N * g.batch;
    f.batch = 1;
    f.sB0 = f.sC0 = 0;
  }
  return gemm_dma_ok(dtype, f, a_bytes, b_bytes) && !stores_bound(f) ? dma_tile(dtype, f) : -1;
}

}  // namespace

hipError_t launch_gemm_nt(int dtype, const GemmArgs& g, hipStream_t stream) {
  uint32_t ab = 0, bb = 0;
  GemmArgs f;
  const int tile = gemm_route(dtype, g, f, ab, bb);
  if (tile >= 0) {
    if (dtype == DT_F32) return launch_dma<float, true>(tile, f, ab, bb, stream);
    return f.out_f32 ? launch_dma<bf16_t, true>(tile, f, ab, bb, stream)
                     : launch_dma<bf16_t, false>(tile, f, ab, bb, stream);
  }
  if (dtype == DT_F32) return launch_typed<float, true>(g, stream);
  return g.out_f32 ? launch_typed<bf16_t, true>(g, stream) : launch_typed<bf16_t, false>(g, stream);
}

std::string gemm_describe(int dtype, const GemmArgs& g) {
  uint32_t ab = 0, bb = 0;
  GemmArgs f;
  const int tile = gemm_route(dtype, g, f, ab, bb);
  const char* t = dtype == DT_F32 ? "f32" : "bf16";
  char buf[64];
  if (tile >= 0)
    snprintf(buf, sizeof(buf), "gemm_dma_kernel<%s,%d,%d,%d>", t, kDmaTiles[tile].TJ, kDmaTiles[tile].TI,
             kDmaTiles[tile].NST);
  else
    snprintf(buf, sizeof(buf), "gemm_nt_kernel<%s,%d,128>", t, g.M <= 64 ? 64 : 128);
  return buf;
}

}  // namespace convsel
