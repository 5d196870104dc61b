// Implicit GEMM on channels-last tensors (paper, Sec. V-B item (b)).
//
// With the channels of a pixel contiguous (N x H x W x Cp, Cp the channels
// rounded up to 16 bytes), the implicit column matrix needs no transposition
// at all: row `pixel` of it, for one filter tap, is a contiguous run of an
// input pixel's channels.  So both GEMM operands -- rows of filters, packed
// [K][tap][Cp], and rows of input pixels -- are copied to LDS by the
// buffer-to-LDS DMA in 128-byte pieces (a k-tile: 64 bf16 or 32 fp32 reduction
// terms), and a lane's address is its pixel's plus the tap's.  Pixels outside
// the image and rows past the tensors take an offset past the buffer, which
// copies zeros.  Strides, padding, dilation and filter sizes only change the
// addresses.
//
// A workgroup (4 waves, WJ x WI x WS) owns TJ pixels x TI filters.  The k-tile
// stage is the layout of the NT GEMM: TJ + TI rows of 128 bytes, two rows per
// 256-byte line, 16-byte unit u of row r at position 8 (r & 1) + (u ^
// ((r >> 1) & 7)) of line r >> 1, free of bank conflicts for the fragment
// reads.  NST stages form a ring, one barrier per k-tile.  WS = 4 splits the
// steps of a k-tile over the waves (small tiles, for grids that would leave
// CUs idle) and adds the four partial sums in LDS.
//
// What bounds it: the path from L2 to LDS, for every k-tile brings its TJ + TI
// rows (ResNet-50 at batch 32, 28 x 28, 128 -> 128 channels, 3 x 3: 15.3 us, of
// which the DMA alone takes 11.7, 21 TB/s over the chip, and the matrix
// instructions with their LDS reads alone 8.9), and around it a workgroup's
// start and end; so the tiles differ in how many workgroups share a CU and in
// how many k-tiles they have in flight.  The N x C x H x W kernels take, on
// 14 x 14 planes (32 images, per layer): 1024 -> 256 1 x 1 22.1 us, this one
// 11.0; 256 -> 1024 with the residual 19.9 and 12.4; 256 -> 256 3 x 3 15.7 and
// 17.3.  On 28 x 28 and 56 x 56 planes the two are within 10 percent.
// At batch 1 (7 x 7, 512 -> 512, 3 x 3) 11 us against 13 with their reduction.
//
// Output is channels-last (OUTC: filters are the MFMA's rows, so a lane holds
// four consecutive channels of one pixel) or N x K x P x Q (pixels are its
// rows).  Either way the tile is rounded, staged in LDS as output rows and
// stored, after the optional residual add, in 16-byte units along them (pixel
// by pixel along planes that are no whole units).
#include <stdio.h>

#include <algorithm>
#include <atomic>
#include <string>
#include <type_traits>

#include "common.hpp"
#include "igemm_common.hpp"
#include "kernels.hpp"

namespace convsel {

namespace {

using namespace igemm;

struct NhArgs {
  const void* x;       // input, moved back by the padding's bytes (never read there)
  const void* w;       // package [K][R*S][Cp]
  const void* b;
  const void* res;
  void* y;
  uint32_t x_bytes, w_bytes;
  int H, W, K, S, P, Q, PQ, NPQ;
  int sh, sw, ph, pw, dh, dw, R;
  int CU;              // 16-byte units per pixel
  uint32_t cu_magic, s_magic;  // ceil(2^32 / d), 0 for d = 1
  int ntap_units;      // R * S * CU: units of a filter row
  int nk;              // k-tiles: ceil(ntap_units / 8)
  int njt, nit, units;
  int relu;
};

__device__ __forceinline__ uint32_t magic_div(uint32_t e, uint32_t m) { return m ? __umulhi(e, m) : e; }

// Residual add and ReLU on one 16-byte unit of output values already rounded to T.
template <typename T>
__device__ __forceinline__ void nh_finish(vec16& v, const vec16& r, int relu) {
  if constexpr (sizeof(T) == 2) {
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      float lo = __uint_as_float(v.d[d] << 16) + __uint_as_float(r.d[d] << 16);
      float hi = __uint_as_float(v.d[d] & 0xffff0000u) + __uint_as_float(r.d[d] & 0xffff0000u);
      if (relu) {
        lo = fmaxf(lo, 0.f);
        hi = fmaxf(hi, 0.f);
      }
      v.d[d] = f32x2_to_bf16x2(lo, hi);
    }
  } else {
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      float f = __uint_as_float(v.d[d]) + __uint_as_float(r.d[d]);
      if (relu) f = fmaxf(f, 0.f);
      v.d[d] = __float_as_uint(f);
    }
  }
}

// G groups of four waves share a tile, group g taking k-tiles g, g + G, ... in
// a ring of its own.
template <typename T, int TJ_, int TI_, int WJ_, int WI_, int NST_, int G_ = 1>
struct NhTile {
  static constexpr int TJ = TJ_, TI = TI_, WJ = WJ_, WI = WI_, WS = 4 / (WJ_ * WI_), NST = NST_, G = G_;
  static constexpr int MJ = TJ / WJ / 32, NI = TI / WI / 32;
  static constexpr int NB = TJ / 32, NA = TI / 32;  // DMA instructions per wave and stage: pixels, filters
  static constexpr int STAGE = (TJ + TI) * 128;
  // One wave's output tile, and (WS = 4) the exchange of partial sums.
  static constexpr int STAGING = WS == 1 ? 4 * MJ * NI * 32 * 32 * elem<T>::bytes : G * 4 * 16 * 64 * 4;
  static constexpr int LDS = G * NST * STAGE > STAGING ? G * NST * STAGE : STAGING;
  static_assert(WJ * WI * WS == 4 && MJ >= 1 && NI >= 1 && (WS == 1 ? G == 1 : MJ * NI == 1), "waves");
  static_assert((NB + NA) * (NST - 1) <= 63 && LDS <= 160 * 1024, "stages");
};

// What the output is: channels-last, planes of whole 16-byte units (bf16: or half
// units), or planes of any size.  (A form each: with the last one in the same
// kernel the others ran 5 percent longer.)
enum { NH_OUT_PIXELS, NH_OUT_PLANES, NH_OUT_ODD_PLANES };

// GEN: the tap is a lane's own and part of its offset; otherwise all lanes are on
// one tap, whose offset is the DMA's scalar offset (nh_uniform_taps()).
template <typename T, typename Tl, bool GEN, int OUT>
__global__ __launch_bounds__(256 * Tl::G) void nhwc_conv_kernel(NhArgs a) {
  constexpr bool OUTC = OUT == NH_OUT_PIXELS;
  constexpr int TJ = Tl::TJ, TI = Tl::TI, MJ = Tl::MJ, NI = Tl::NI, NB = Tl::NB, NA = Tl::NA, NST = Tl::NST;
  constexpr int ES = elem<T>::bytes, UE = elem<T>::per16, WS = Tl::WS, G = Tl::G;
  extern __shared__ __align__(16) vec16 smem[];
  char* lds = reinterpret_cast<char*>(smem);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) & 3);
  const int grp = G == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
  char* ring = lds + grp * (NST * Tl::STAGE);
  const int wj = wave % Tl::WJ, wi = (wave / Tl::WJ) % Tl::WI, ws = wave / (Tl::WJ * Tl::WI);
  // Units (pixel tile, filter tile; filter tiles fastest) go to the XCDs in
  // contiguous ranges, so the tiles that read the same pixels share an L2.
  const int per_xcd = (a.units + 7) >> 3;
  const int unit = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (unit >= a.units) return;  // uniform
  const int jt = unit / a.nit;
  const int j0 = jt * TJ, i0 = (unit - jt * a.nit) * TI;
  const u32x4_t xr = dma_rsrc(a.x, a.x_bytes), wr = dma_rsrc(a.w, a.w_bytes);
  const uint32_t lds0 = lds_address(ring);

  // DMA lanes: instruction J of a stage fills its 16-byte units J*64 + lane,
  // that is unit u of row 2 line + ((lane >> 3) & 1), line = J*4 + lane/16.
  uint32_t bvo[NB], avo[NA], bu[NB], au[NA];
  uint32_t rmask[NB], cmask[NB];  // rows r and columns s of the filter that fall inside the image
  const int rows_taps = a.R, cols_taps = a.S;
#pragma unroll
  for (int d = 0; d < NB; ++d) {
    const int line = (wave * NB + d) * 4 + (lane >> 4);
    const int row = 2 * line + ((lane >> 3) & 1);
    bu[d] = (lane & 7) ^ (line & 7);
    const int j = j0 + row;
    const int jj = min(j, a.NPQ - 1);
    const int n = jj / a.PQ, pq = jj - n * a.PQ;
    const int p = pq / a.Q, q = pq - p * a.Q;
    const int ih = p * a.sh, iw = q * a.sw;  // in the padded image
    bvo[d] = static_cast<uint32_t>((n * a.H + ih) * a.W + iw) * (a.CU * 16) + (GEN ? 0 : bu[d] * 16);
    uint32_t rm = 0, cm = 0;
    if (j < a.NPQ) {
      for (int r = 0; r < rows_taps; ++r) {
        const int h = ih + r * a.dh - a.ph;
        rm |= (h >= 0 && h < a.H ? 1u : 0u) << r;
      }
      for (int s = 0; s < cols_taps; ++s) {
        const int v = iw + s * a.dw - a.pw;
        cm |= (v >= 0 && v < a.W ? 1u : 0u) << s;
      }
    }
    rmask[d] = rm;
    cmask[d] = cm;
  }
#pragma unroll
  for (int d = 0; d < NA; ++d) {
    const int line = TJ / 2 + (wave * NA + d) * 4 + (lane >> 4);
    const int row = 2 * line + ((lane >> 3) & 1) - TJ;
    au[d] = (lane & 7) ^ (line & 7);
    avo[d] = i0 + row < a.K ? static_cast<uint32_t>((i0 + row) * a.ntap_units + au[d]) * 16 : a.w_bytes;
  }

  // Issue cursor (uniform taps): tap (ir, is), 128-byte piece ic of the pixel.
  const int pieces = a.CU >> 3;
  int ir = 0, is = 0, ic = 0, ikt = grp, slot = 0;  // (slot: the ring stage of k-tile ikt)
  uint32_t vcur[NB];
  auto tap_lanes = [&]() {
#pragma unroll
    for (int d = 0; d < NB; ++d) vcur[d] = ((rmask[d] >> ir) & (cmask[d] >> is) & 1u) ? bvo[d] : a.x_bytes;
  };
  auto advance = [&](int by) {
    for (ic += by; ic >= pieces;) {
      ic -= pieces;
      if (++is == a.S) {
        is = 0;
        ++ir;
      }
    }
  };
  if constexpr (!GEN) {
    if constexpr (G > 1) advance(grp);
    tap_lanes();
  }
  auto issue = [&]() {  // k-tile ikt into its stage
    const uint32_t st = lds0 + slot * Tl::STAGE;
    slot = slot == NST - 1 ? 0 : slot + 1;
    if constexpr (!GEN) {
      const uint32_t so = static_cast<uint32_t>((ir * a.dh * a.W + is * a.dw) * a.CU + ic * 8) * 16;
#pragma unroll
      for (int d = 0; d < NB; ++d) dma16(xr, st + (wave * NB + d) * 1024, vcur[d], so);
      if (ic + G >= pieces) {
        advance(G);
        tap_lanes();
      } else {
        ic += G;
      }
    } else {
#pragma unroll
      for (int d = 0; d < NB; ++d) {
        const uint32_t e = static_cast<uint32_t>(ikt) * 8 + bu[d];
        const uint32_t tap = magic_div(e, a.cu_magic), cu = e - tap * a.CU;
        const uint32_t r = magic_div(tap, a.s_magic), s = tap - r * a.S;
        const bool ok = e < static_cast<uint32_t>(a.ntap_units) && ((rmask[d] >> r) & (cmask[d] >> s) & 1u);
        const uint32_t vo = bvo[d] + ((r * a.dh * a.W + s * a.dw) * a.CU + cu) * 16;
        dma16(xr, st + (wave * NB + d) * 1024, ok ? vo : a.x_bytes, 0u);
      }
    }
    const uint32_t wo = static_cast<uint32_t>(ikt) * 128;
    const bool tail = GEN && (ikt + 1) * 8 > a.ntap_units;
#pragma unroll
    for (int d = 0; d < NA; ++d) {
      const uint32_t vo = tail && ikt * 8 + static_cast<int>(au[d]) >= a.ntap_units ? a.w_bytes : avo[d];
      dma16(wr, st + TJ * 128 + (wave * NA + d) * 1024, vo, wo);
    }
    ikt += G;
  };

  // Fragment offsets within a stage: unit 2 t + half of row r.
  const int half = lane >> 5, l32 = lane & 31;
  auto frag = [&](int r, int u) { return (r >> 1) * 256 + ((8 * (r & 1) + (u ^ ((r >> 1) & 7))) << 4); };
  constexpr int TS = 4 / WS;  // steps of a k-tile per wave
  int poff[MJ][TS], foff[NI][TS];
#pragma unroll
  for (int t = 0; t < TS; ++t) {
#pragma unroll
    for (int mj = 0; mj < MJ; ++mj) poff[mj][t] = frag((wj * MJ + mj) * 32 + l32, 2 * (t * WS + ws) + half);
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) foff[ni][t] = frag(TJ + (wi * NI + ni) * 32 + l32, 2 * (t * WS + ws) + half);
  }

  f32x16_t acc[MJ][NI];
#pragma unroll
  for (int mj = 0; mj < MJ; ++mj)
#pragma unroll
    for (int ni = 0; ni < NI; ++ni) acc[mj][ni] = zero16();
  // fp32 sums go k-tile by k-tile (32 terms each, then added to the total): one
  // chain over the whole reduction rounds more than the split reductions of the
  // N x C x H x W kernels do (simulated, relative error: 240 terms 2.0e-7, in
  // k-tiles 1.0e-7; 576 terms 3.0e-7 and 1.0e-7).  With the steps split over the
  // waves the chains are short already.  Costs 5 percent (inverted block, 96-576-96,
  // 14 x 14, 64 images: 60.8 us as one chain, 64.0).
  constexpr bool BLOCKED = sizeof(T) == 4 && WS == 1;

  const int nk = G == 1 ? a.nk : (a.nk - grp + G - 1) / G;      // this group's k-tiles
  const int rounds = G == 1 ? nk : (a.nk + G - 1) / G;          // (the groups' barriers are common)
#pragma unroll
  for (int p = 0; p < NST - 1; ++p)
    if (p < nk) issue();

  // Bias of this lane's channels, requested now and used after the last k-tile:
  // OUTC, four consecutive channels per register group (group ws alone with WS
  // = 4); else one channel per block.  Channels past K read the last ones.
  constexpr int BG = OUTC ? (WS == 4 ? 1 : 4) : 1, BL = OUTC ? 4 : 1;
  typename elem<T>::storage bias[NI][BG][BL];
#pragma unroll
  for (int ni = 0; ni < NI; ++ni)
#pragma unroll
    for (int g = 0; g < BG; ++g) {
      const int ch = i0 + (wi * NI + ni) * 32 + (OUTC ? 8 * (WS == 4 ? ws : g) + 4 * half : l32);
#pragma unroll
      for (int t = 0; t < BL; ++t) bias[ni][g][t] = 0;
      if (a.b) __builtin_memcpy(&bias[ni][g][0], reinterpret_cast<const T*>(a.b) + min(ch, a.K - BL), BL * ES);
    }
  auto bias_of = [&](int ni, int g, int t) {
    T v;
    __builtin_memcpy(&v, &bias[ni][BG == 1 ? 0 : g][OUTC ? t : 0], ES);
    return elem<T>::to_f32(v);
  };
  int stage = 0;
  for (int kt = 0; kt < rounds; ++kt) {
    // k-tile kt has landed once at most the later tiles' DMAs are pending.
    const int later = min(nk - 1, kt + NST - 2) - kt;
    constexpr int PER = NB + NA;
    if constexpr (NST >= 3) {
      if (later == NST - 2) CONVSEL_WAIT_VMCNT((NST - 2) * PER);
      else if (NST >= 4 && later >= 1) CONVSEL_WAIT_VMCNT(PER);
      else CONVSEL_WAIT_VMCNT(0);
    } else {
      CONVSEL_WAIT_VMCNT(0);
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();  // every wave's part of k-tile kt is in, every wave is done with k-tile kt - 1
    asm volatile("" ::: "memory");
    if (kt + NST - 1 < nk) issue();  // into the stage of k-tile kt - 1
    if (G > 1 && kt >= nk) continue;  // a group with one k-tile less
    const char* st = ring + stage * Tl::STAGE;
    stage = stage == NST - 1 ? 0 : stage + 1;
    vec16 fp[2][MJ], ff[2][NI];
    auto read = [&](auto t_c) {
      constexpr int t = decltype(t_c)::value;
#pragma unroll
      for (int mj = 0; mj < MJ; ++mj) fp[t & 1][mj] = *reinterpret_cast<const vec16*>(st + poff[mj][t]);
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) ff[t & 1][ni] = *reinterpret_cast<const vec16*>(st + foff[ni][t]);
    };
    f32x16_t part[MJ][NI];
    if constexpr (BLOCKED) {
#pragma unroll
      for (int mj = 0; mj < MJ; ++mj)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) part[mj][ni] = zero16();
    }
    read(std::integral_constant<int, 0>{});
    static_for<TS>([&](auto t_c) {
      constexpr int t = decltype(t_c)::value;
      if constexpr (t + 1 < TS) read(std::integral_constant<int, t + 1>{});
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int mj = 0; mj < MJ; ++mj)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
          f32x16_t& sum = BLOCKED ? part[mj][ni] : acc[mj][ni];
          if constexpr (OUTC) mfma_32x32<T>(sum, ff[t & 1][ni], fp[t & 1][mj]);
          else mfma_32x32<T>(sum, fp[t & 1][mj], ff[t & 1][ni]);
        }
      __builtin_amdgcn_sched_barrier(0);
    });
    if constexpr (BLOCKED) {
#pragma unroll
      for (int mj = 0; mj < MJ; ++mj)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) acc[mj][ni] += part[mj][ni];
    }
  }
  lds_sync();  // no wave reads the stages any more: the output is staged in their place

  // Block (mj, ni) of the accumulators: lane column l32 is a pixel (OUTC) or a
  // channel, register 4 g + t row 8 g + 4 half + t of the other kind.
  const T* res = reinterpret_cast<const T*>(a.res);
  T* y = reinterpret_cast<T*>(a.y);
  const bool relu_now = a.relu && !res;
  if constexpr (WS == 4) {
    // Partial sums of the waves: wave w of the first group adds up and stores
    // row group w.
    float* part = reinterpret_cast<float*>(lds);
#pragma unroll
    for (int v = 0; v < 16; ++v) part[((grp * 4 + ws) * 16 + v) * 64 + lane] = acc[0][0][v];
    lds_sync();
    if (grp > 0) return;
    float v4[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      float s = 0.f;
#pragma unroll
      for (int w = 0; w < 4 * G; ++w) s += part[(w * 16 + 4 * ws + t) * 64 + lane];
      v4[t] = s + bias_of(0, 0, t);
      if (relu_now) v4[t] = fmaxf(v4[t], 0.f);
    }
    if constexpr (OUTC) {
      const int j = j0 + l32, ch = i0 + 8 * ws + 4 * half;
      if (j >= a.NPQ || ch >= a.K) return;  // (K is a multiple of 4)
      const int64_t o = static_cast<int64_t>(j) * a.K + ch;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        if (res) {
          v4[t] = elem<T>::to_f32(elem<T>::from_f32(v4[t])) + elem<T>::load(res + o + t);
          if (a.relu) v4[t] = fmaxf(v4[t], 0.f);
        }
      }
      if constexpr (sizeof(T) == 2)
        *reinterpret_cast<uint2*>(y + o) = make_uint2(f32x2_to_bf16x2(v4[0], v4[1]), f32x2_to_bf16x2(v4[2], v4[3]));
      else
        *reinterpret_cast<float4*>(y + o) = make_float4(v4[0], v4[1], v4[2], v4[3]);
    } else {
      const int k = i0 + l32;
      if (k >= a.K) return;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int j = j0 + 8 * ws + 4 * half + t;
        if (j >= a.NPQ) return;
        const int n = j / a.PQ;
        const int64_t o = (static_cast<int64_t>(n) * a.K + k) * a.PQ + (j - n * a.PQ);
        float f = v4[t];
        if (res) {
          f = elem<T>::to_f32(elem<T>::from_f32(f)) + elem<T>::load(res + o);
          if (a.relu) f = fmaxf(f, 0.f);
        }
        elem<T>::store(y + o, f);
      }
    }
    return;
  } else {
    // This wave's output rows: ROWS (pixels or channels) of COLS values.
    constexpr int ROWS = (OUTC ? MJ : NI) * 32, COLS = (OUTC ? NI : MJ) * 32;
    constexpr int U = COLS / UE;  // 16-byte units per row
    char* stg = lds + wave * (MJ * NI * 32 * 32 * ES);
#pragma unroll
    for (int mj = 0; mj < MJ; ++mj)
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) {
        const int rb = OUTC ? mj : ni, cb = OUTC ? ni : mj;
        const int row = rb * 32 + l32;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          float v[4];
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            v[t] = acc[mj][ni][4 * g + t] + bias_of(ni, g, t);
            if (relu_now) v[t] = fmaxf(v[t], 0.f);
          }
          const int col = cb * 32 + 8 * g + 4 * half;
          char* at = stg + row * (U * 16) + (((col / UE) ^ (row & (U - 1))) << 4) + (col % UE) * ES;
          if constexpr (sizeof(T) == 2)
            *reinterpret_cast<uint2*>(at) = make_uint2(f32x2_to_bf16x2(v[0], v[1]), f32x2_to_bf16x2(v[2], v[3]));
          else
            *reinterpret_cast<float4*>(at) = make_float4(v[0], v[1], v[2], v[3]);
        }
      }
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): this wave's staging writes are done
    __builtin_amdgcn_wave_barrier();
    constexpr int RPI = 64 / U, PASSES = ROWS / RPI;
    const int rrow = lane / U, u = lane % U;
    const int rbase = OUTC ? j0 + wj * MJ * 32 : i0 + wi * NI * 32;
    const int cbase = (OUTC ? i0 + wi * NI * 32 : j0 + wj * MJ * 32) + u * UE;
    vec16 d[PASSES];
#pragma unroll
    for (int it = 0; it < PASSES; ++it) {
      const int row = rrow + RPI * it;
      d[it] = *reinterpret_cast<const vec16*>(stg + row * (U * 16) + ((u ^ (row & (U - 1))) << 4));
    }
    if constexpr (OUTC) {
      if (cbase >= a.K) return;  // (K is a multiple of UE)
      const int64_t o0 = static_cast<int64_t>(rbase + rrow) * a.K + cbase;
      const int64_t step = static_cast<int64_t>(RPI) * a.K;
      const int left = a.NPQ - rbase - rrow;
      if (res) {
        vec16 r[PASSES];
#pragma unroll
        for (int it = 0; it < PASSES; ++it) r[it] = RPI * it < left ? load16(res + o0 + it * step) : vec16_zero();
#pragma unroll
        for (int it = 0; it < PASSES; ++it) nh_finish<T>(d[it], r[it], a.relu);
      }
#pragma unroll
      for (int it = 0; it < PASSES; ++it)
        if (RPI * it < left) store16(y + o0 + it * step, d[it]);
    } else if constexpr (OUT == NH_OUT_PLANES) {
      // UE consecutive pixels of a channel: a whole unit of one image, or (bf16,
      // planes of whole half units) two halves.
      if (cbase >= a.NPQ) return;
      const int n = cbase / a.PQ, pq = cbase - n * a.PQ;
      const int64_t o0 = (static_cast<int64_t>(n) * a.K + rbase + rrow) * a.PQ + pq;
      const int64_t step = static_cast<int64_t>(RPI) * a.PQ;
      const int left = a.K - rbase - rrow;
      if (a.PQ % UE == 0) {
        if (res) {
          vec16 r[PASSES];
#pragma unroll
          for (int it = 0; it < PASSES; ++it) {
            r[it] = vec16_zero();
            if (RPI * it < left) __builtin_memcpy(&r[it], res + o0 + it * step, 16);
          }
#pragma unroll
          for (int it = 0; it < PASSES; ++it) nh_finish<T>(d[it], r[it], a.relu);
        }
#pragma unroll
        for (int it = 0; it < PASSES; ++it)  // (the caller's tensor: element alignment)
          if (RPI * it < left) __builtin_memcpy(y + o0 + it * step, &d[it], 16);
      } else if constexpr (sizeof(T) == 2) {
        // Two half units of four pixels, each in one image.
        int64_t o[2];
        bool in[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int j = cbase + 4 * h, n2 = j / a.PQ;
          in[h] = j < a.NPQ;
          o[h] = (static_cast<int64_t>(n2) * a.K + rbase + rrow) * a.PQ + (j - n2 * a.PQ);
        }
        if (res) {
          vec16 r[PASSES];
#pragma unroll
          for (int it = 0; it < PASSES; ++it) {
            r[it] = vec16_zero();
#pragma unroll
            for (int h = 0; h < 2; ++h)
              if (RPI * it < left && in[h]) __builtin_memcpy(&r[it].d[2 * h], res + o[h] + it * step, 8);
          }
#pragma unroll
          for (int it = 0; it < PASSES; ++it) nh_finish<T>(d[it], r[it], a.relu);
        }
#pragma unroll
        for (int it = 0; it < PASSES; ++it)
#pragma unroll
          for (int h = 0; h < 2; ++h)
            if (RPI * it < left && in[h]) __builtin_memcpy(y + o[h] + it * step, &d[it].d[2 * h], 8);
      }
    } else {
      // Planes of no whole units: one pixel per lane, so that a wave's stores run
      // along a channel's pixels.  (Eight pixels of a lane one after the other
      // instead, a store's lanes 16 bytes apart: 4 -> 126 channels, 2 x 2, 55
      // images of 47 x 47 outputs, whole layer 47.7 us, this way 24.1.)
      constexpr int LPX = COLS < 64 ? COLS : 64, RL = 64 / LPX;  // lanes along a row, rows per pass
      const int left = a.K - rbase - lane / LPX;
#pragma unroll
      for (int cb = 0; cb < COLS; cb += LPX) {
        const int col = cb + lane % LPX, j = j0 + wj * MJ * 32 + col;
        if (j >= a.NPQ || left <= 0) continue;
        const int n = j / a.PQ;
        const int64_t o0 = (static_cast<int64_t>(n) * a.K + rbase + lane / LPX) * a.PQ + (j - n * a.PQ);
        constexpr int BATCH = ROWS / RL < 16 ? ROWS / RL : 16;  // residuals requested together
#pragma unroll
        for (int it0 = 0; it0 < ROWS / RL; it0 += BATCH) {
          T r[BATCH];
          if (res) {
#pragma unroll
            for (int t = 0; t < BATCH; ++t)  // (rows past K read the first one)
              r[t] = res[RL * (it0 + t) < left ? o0 + static_cast<int64_t>(RL * (it0 + t)) * a.PQ : o0];
          }
#pragma unroll
          for (int t = 0; t < BATCH; ++t) {
            const int row = lane / LPX + RL * (it0 + t);
            if (RL * (it0 + t) >= left) continue;
            float f = elem<T>::load(reinterpret_cast<const T*>(
                stg + row * (U * 16) + (((col / UE) ^ (row & (U - 1))) << 4) + (col % UE) * ES));
            if (res) {
              f += elem<T>::to_f32(r[t]);
              if (a.relu) f = fmaxf(f, 0.f);
            }
            elem<T>::store(y + o0 + static_cast<int64_t>(RL * (it0 + t)) * a.PQ, f);
          }
        }
      }
    }
  }
}

// Filter package: [K][R*S][Cp] from K x C x R x S, zero channels past C.  One
// thread per 16-byte unit.
template <typename T>
__global__ __launch_bounds__(256) void nhwc_pack_kernel(const T* __restrict__ w, T* __restrict__ pk, int C, int RS,
                                                        int CU, int64_t units) {
  constexpr int UE = elem<T>::per16;
  const int64_t u = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (u >= units) return;
  const int cu = static_cast<int>(u % CU);
  const int64_t kt = u / CU;
  const int tap = static_cast<int>(kt % RS);
  const T* src = w + (kt / RS) * C * RS + tap;
  uint32_t e[UE];
#pragma unroll
  for (int i = 0; i < UE; ++i) {
    const int c = cu * UE + i;
    const uint32_t bits = load_bits(src + static_cast<int64_t>(c < C ? c : 0) * RS);
    e[i] = c < C ? bits : 0u;
  }
  vec16 v;
  pack16<T>(v, e);
  store16(pk + u * UE, v);
}

// ---- depthwise 3 x 3 ------------------------------------------------------------
// A thread owns one 16-byte unit of channels and PR x QN output pixels (two rows
// at stride 1, one at stride 2; 7 or 4 columns): its input units are requested
// together (pixels outside the image read zeros past the buffer) and each feeds
// up to nine taps from registers.  Consecutive lanes take consecutive channel
// units, so every access is whole lines.
//
// What bounds it: its bytes, and the one round trip of a thread's reads (576
// channels of 14 x 14, 64 images, fp32, 58 MB: 15.9 us with 2 x 7 pixels a
// thread, 19.0 with 2 x 4, 20.6 with 1 x 4; the N x C x H x W kernel takes 21.5).
// Seven columns where they pad a row no more than four do.
struct DwArgs {
  const void* x;
  const void* w;  // [9][C]
  const void* b;
  void* y;
  uint32_t x_bytes;
  int H, W, P, Q, CU, ph, pw, pstrips, qstrips, relu;
  int64_t threads;
};

template <typename T, int ST, int QN>
__global__ __launch_bounds__(256) void dw3_nhwc_kernel(DwArgs a) {
  constexpr int UE = elem<T>::per16, PR = ST == 1 ? 2 : 1;
  constexpr int IR = (PR - 1) * ST + 3, IC = (QN - 1) * ST + 3;
  const int64_t id = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (id >= a.threads) return;
  const int cu = static_cast<int>(id % a.CU);
  int64_t rest = id / a.CU;
  const int q0 = static_cast<int>(rest % a.qstrips) * QN;
  rest /= a.qstrips;
  const int p0 = static_cast<int>(rest % a.pstrips) * PR;
  const int n = static_cast<int>(rest / a.pstrips);
  const __amdgpu_buffer_rsrc_t xr = make_rsrc(a.x, a.x_bytes);
  vec16 in[IR][IC];
#pragma unroll
  for (int i = 0; i < IR; ++i) {
    const int h = p0 * ST - a.ph + i;
    const bool hin = h >= 0 && h < a.H;
#pragma unroll
    for (int j = 0; j < IC; ++j) {
      const int w = q0 * ST - a.pw + j;
      const uint32_t off = static_cast<uint32_t>(((n * a.H + h) * a.W + w) * a.CU + cu) * 16;
      in[i][j] = buf_load16(xr, hin && w >= 0 && w < a.W ? off : a.x_bytes, 0);
    }
  }
  const T* wp = reinterpret_cast<const T*>(a.w) + cu * UE;
  vec16 wt[9];
#pragma unroll
  for (int t = 0; t < 9; ++t) wt[t] = load16(wp + static_cast<int64_t>(t) * a.CU * UE);
  float bias[UE];
#pragma unroll
  for (int e = 0; e < UE; ++e) bias[e] = a.b ? elem<T>::load(reinterpret_cast<const T*>(a.b) + cu * UE + e) : 0.f;
  T* y = reinterpret_cast<T*>(a.y);
#pragma unroll
  for (int i = 0; i < PR; ++i)
#pragma unroll
    for (int j = 0; j < QN; ++j) {
      float acc[UE];
#pragma unroll
      for (int e = 0; e < UE; ++e) acc[e] = 0.f;
#pragma unroll
      for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int s = 0; s < 3; ++s)
#pragma unroll
          for (int e = 0; e < UE; ++e)
            acc[e] = fmaf(elem<T>::to_f32(vec16_get<T>(in[i * ST + r][j * ST + s], e)),
                          elem<T>::to_f32(vec16_get<T>(wt[r * 3 + s], e)), acc[e]);
      vec16 v = vec16_zero();
#pragma unroll
      for (int e = 0; e < UE; ++e) {
        float f = acc[e] + bias[e];
        if (a.relu) f = fmaxf(f, 0.f);
        vec16_set<T>(v, e, elem<T>::from_f32(f));
      }
      const int p = p0 + i, q = q0 + j;
      if (p < a.P && q < a.Q) store16(y + (((static_cast<int64_t>(n) * a.P + p) * a.Q + q) * a.CU + cu) * UE, v);
    }
}

// Depthwise filters C x 1 x 3 x 3 as [9][C].
template <typename T>
__global__ __launch_bounds__(256) void dw3_pack_kernel(const T* __restrict__ w, T* __restrict__ pk, int C) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < 9 * C) pk[i] = w[(i % C) * 9 + i / C];
}

// N x C x HW to N x HW x Cp (zeros in the channels past C).  A workgroup
// transposes 64 pixels x 64 (bf16) or 32 (fp32) channels through LDS: reads
// run along the pixels, writes along the channels in 16-byte units.
template <typename T>
__global__ __launch_bounds__(256) void to_nhwc_kernel(const T* __restrict__ x, T* __restrict__ y, int C, int HW,
                                                      int CU, int ptiles, int ctiles, int vec) {
  constexpr int UE = elem<T>::per16, TC = 128 / elem<T>::bytes;
  constexpr int PITCH = 64 + (sizeof(T) == 2 ? 2 : 1);
  __shared__ T tile[TC * PITCH];
  int b = blockIdx.x;
  const int ct = b % ctiles;
  b /= ctiles;
  const int pt = b % ptiles;
  const int64_t n = b / ptiles;
  const int c0 = ct * TC, p0 = pt * 64;
  const T* xn = x + (n * C + c0) * static_cast<int64_t>(HW) + p0;
  if (vec) {  // whole 16-byte units of pixels
    constexpr int PU = 64 / UE, IT = TC * PU / 256;
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const int e = threadIdx.x + i * 256, c = e / PU, pu = e % PU;
      const bool in = c0 + c < C && p0 + pu * UE < HW;
      vec16 v = load16(in ? xn + static_cast<int64_t>(c) * HW + pu * UE : x);
#pragma unroll
      for (int k = 0; k < UE; ++k)
        tile[c * PITCH + pu * UE + k] = in ? vec16_get<T>(v, k) : elem<T>::from_f32(0.f);
    }
  } else {
    const int px = threadIdx.x & 63;
    constexpr int IT = TC / 4;
    T v[IT];
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const int c = (threadIdx.x >> 6) + 4 * i;
      const bool in = c0 + c < C && p0 + px < HW;
      v[i] = in ? xn[static_cast<int64_t>(c) * HW + px] : elem<T>::from_f32(0.f);
    }
#pragma unroll
    for (int i = 0; i < IT; ++i) tile[((threadIdx.x >> 6) + 4 * i) * PITCH + px] = v[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int e = threadIdx.x + i * 256, px = e >> 3, cu = e & 7;
    if (p0 + px >= HW || c0 / UE + cu >= CU) continue;
    uint32_t bits[UE];
#pragma unroll
    for (int k = 0; k < UE; ++k) bits[k] = load_bits(tile + (cu * UE + k) * PITCH + px);
    vec16 v;
    pack16<T>(v, bits);
    store16(y + ((n * HW + p0 + px) * CU + c0 / UE + cu) * UE, v);
  }
}

// ---- host side ------------------------------------------------------------

uint32_t magic_of(int d) { return d == 1 ? 0u : (uint32_t)((((uint64_t)1 << 32) + d - 1) / d); }

// Tiles and their measured costs, microseconds: a launch of nk k-tiles, w
// workgroups per CU of which `occ` run together, takes about
//   base + max(w * nk * through, ceil(w / occ) * nk * latency) + w * tile
// (fitted, relative error, to the 52 channels-last convolutions of ResNet-50
// at batch 32, each run with every tile; median error 3 to 5 percent).  The
// sum over those layers with the tile this picks is 812 us; 811 with the best
// measured one for each, 870 with the best single tile.
// On layers it was not fitted to (220 random ones, bf16, 3 x 3 to 7 x 7, 9 to 512
// channels, copy included): 1.04 times the best tile's time in the geometric mean,
// 1.65 at worst; in sum 5.24 ms, with the best tile of each 4.88, with the best
// single tile 7.17.
// In fp32 the matrix instructions bound a k-tile (a sixteenth of the bf16 rate):
// mfma32 is what one takes on a CU to itself.
struct NhConfig {
  int TJ, TI, WJ, WI, NST, G;  // NhTile
  int occ;
  double base, through, latency, tile, mfma32;
};
constexpr NhConfig kNhConfigs[] = {
    {128, 128, 2, 2, 2, 1, 2, 5.33, 0.05, 0.755, 2.08, 1.9},
    {64, 128, 2, 2, 3, 1, 2, 4.62, 0.230, 0.369, 1.38, 0.95},
    {64, 128, 2, 2, 2, 1, 3, 4.96, 0.293, 0.683, 0.91, 0.95},
    {64, 64, 2, 2, 4, 1, 2, 3.26, 0.174, 0.243, 1.11, 0.48},
    {64, 64, 2, 2, 2, 1, 5, 3.88, 0.174, 0.632, 0.64, 0.48},
    {32, 32, 1, 1, 8, 1, 2, 3.3, 0.10, 0.18, 0.9, 0.21},   // steps split over the waves
    {32, 32, 1, 1, 4, 4, 1, 3.8, 0.05, 0.06, 1.2, 0.21},   // and k-tiles over four groups of waves
};
constexpr int kNumNh = sizeof(kNhConfigs) / sizeof(kNhConfigs[0]);

int nh_units_per_pixel(const Shape& s) {
  const int ue = s.dtype == DT_F32 ? 4 : 8;
  return (int)((s.C + ue - 1) / ue);
}

// One tap for all lanes of a k-tile: where the tiles do not span taps (Cp whole
// 128-byte pieces), and every tap's offset stays within the buffer.  The range
// check that zeroes lanes outside the image may be made against the buffer's size
// less the scalar offset, which must not go below zero.  Larger offsets belong to
// taps outside the image for every pixel (padding of at least N * H rows).
bool nh_uniform_taps(const Shape& s) {
  const int64_t cu = nh_units_per_pixel(s);
  const int64_t last = ((s.R - 1) * s.dh * s.W + (s.S - 1) * s.dw + 1) * cu - 8;
  return cu % 8 == 0 && last <= (s.N * s.H * s.W + s.ph * s.W + s.pw) * cu;
}

int nh_config(const Shape& s) {
  const int64_t npq = s.N * s.P * s.Q;
  const double nk = (double)((s.R * s.S * nh_units_per_pixel(s) + 7) / 8);
  int best = 0;
  double bt = 0;
  for (int c = 0; c < kNumNh; ++c) {
    const NhConfig& t = kNhConfigs[c];
    const int64_t units = ((npq + t.TJ - 1) / t.TJ) * ((s.K + t.TI - 1) / t.TI);
    const int64_t w = (units + 255) / 256;
    const double through = s.dtype == DT_F32 ? std::max(t.through, t.mfma32) : t.through;
    const double us = t.base + std::max((double)w * nk * through, (double)((w + t.occ - 1) / t.occ) * nk * t.latency) +
                      (double)w * t.tile;
    if (c == 0 || us < bt) {
      best = c;
      bt = us;
    }
  }
  return best;
}

template <typename T, typename Tl, bool GEN, int OUT>
hipError_t nh_launch(const NhArgs& a, hipStream_t stream) {
  const auto kern = nhwc_conv_kernel<T, Tl, GEN, OUT>;
  if (Tl::LDS > 64 * 1024) {
    static std::atomic<bool> set{false};
    if (!set.load()) {
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, Tl::LDS);
      if (e != hipSuccess) return e;
      set.store(true);
    }
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)((a.units + 7) / 8 * 8)), dim3(256 * Tl::G), Tl::LDS, stream, a);
  return hipGetLastError();
}

template <typename T, typename Tl>
hipError_t nh_dispatch_tile(NhArgs& a, bool gen, bool outc, hipStream_t st) {
  a.njt = (a.NPQ + Tl::TJ - 1) / Tl::TJ;
  a.nit = (a.K + Tl::TI - 1) / Tl::TI;
  a.units = a.njt * a.nit;
  if (outc) return gen ? nh_launch<T, Tl, true, NH_OUT_PIXELS>(a, st) : nh_launch<T, Tl, false, NH_OUT_PIXELS>(a, st);
  // (The tile whose waves split the steps stores pixel by pixel anyway.)
  constexpr int ODD = Tl::WS == 1 ? NH_OUT_ODD_PLANES : NH_OUT_PLANES;
  if (a.PQ % 4 != 0) return gen ? nh_launch<T, Tl, true, ODD>(a, st) : nh_launch<T, Tl, false, ODD>(a, st);
  return gen ? nh_launch<T, Tl, true, NH_OUT_PLANES>(a, st) : nh_launch<T, Tl, false, NH_OUT_PLANES>(a, st);
}

template <typename T, int I>
hipError_t nh_dispatch_config(NhArgs& a, bool gen, bool outc, hipStream_t st) {
  constexpr NhConfig c = kNhConfigs[I];
  return nh_dispatch_tile<T, NhTile<T, c.TJ, c.TI, c.WJ, c.WI, c.NST, c.G>>(a, gen, outc, st);
}

template <typename T>
hipError_t nh_dispatch(NhArgs& a, int cfg, bool gen, bool outc, hipStream_t st) {
  static_assert(kNumNh == 7, "one line each");
  switch (cfg) {
    case 0: return nh_dispatch_config<T, 0>(a, gen, outc, st);
    case 1: return nh_dispatch_config<T, 1>(a, gen, outc, st);
    case 2: return nh_dispatch_config<T, 2>(a, gen, outc, st);
    case 3: return nh_dispatch_config<T, 3>(a, gen, outc, st);
    case 4: return nh_dispatch_config<T, 4>(a, gen, outc, st);
    case 5: return nh_dispatch_config<T, 5>(a, gen, outc, st);
    case 6: return nh_dispatch_config<T, 6>(a, gen, outc, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

bool nhwc_applies(const Shape& s) {
  const int ue = s.dtype == DT_F32 ? 4 : 8;
  const int64_t cu = (s.C + ue - 1) / ue, lim = (int64_t)1 << 31;
  if (s.G != 1 || s.N < 1 || s.R > 31 || s.S > 31) return false;
  // Offsets are 32-bit byte offsets below 2^31 from the (padding-shifted) base.
  if ((s.N * s.H * s.W + s.ph * s.W + s.pw + (s.R * s.dh + 1) * s.W + s.S * s.dw) * cu * 16 >= lim) return false;
  if (s.K * s.R * s.S * cu * 16 >= lim) return false;
  // The copy's workgroups (64 pixels of one image, 8 units) of 256 threads: a grid holds fewer than 2^32 threads.
  if (s.N * ((s.H * s.W + 63) / 64) * ((cu + 7) / 8) >= (int64_t)1 << 24) return false;
  return s.R * s.S * cu < 65536 && s.N * s.P * s.Q + 128 < lim;
}

size_t nhwc_packed_bytes(const Shape& s) { return (size_t)s.K * s.R * s.S * nh_units_per_pixel(s) * 16; }
size_t nhwc_input_bytes(const Shape& s) { return (size_t)s.N * s.H * s.W * nh_units_per_pixel(s) * 16; }

namespace {
hipError_t nh_pack(const Shape& s, const void* w, void* pk, int CU, hipStream_t stream) {
  const int64_t units = s.K * s.R * s.S * CU;
  const dim3 grid((unsigned)((units + 255) / 256));
  if (s.dtype == DT_F32)
    hipLaunchKernelGGL(nhwc_pack_kernel<float>, grid, dim3(256), 0, stream, (const float*)w, (float*)pk, (int)s.C,
                       (int)(s.R * s.S), CU, units);
  else
    hipLaunchKernelGGL(nhwc_pack_kernel<bf16_t>, grid, dim3(256), 0, stream, (const bf16_t*)w, (bf16_t*)pk, (int)s.C,
                       (int)(s.R * s.S), CU, units);
  return hipGetLastError();
}

hipError_t nh_copy(int dtype, const void* x, void* y, int64_t N, int64_t C, int64_t HW, int CU, hipStream_t stream) {
  const int ue = dtype == DT_F32 ? 4 : 8;
  const int ptiles = (int)((HW + 63) / 64), ctiles = (CU + 7) / 8;
  const int vec = HW % ue == 0 && reinterpret_cast<uintptr_t>(x) % 16 == 0;
  const dim3 grid((unsigned)(N * ptiles * ctiles));
  if (dtype == DT_F32)
    hipLaunchKernelGGL(to_nhwc_kernel<float>, grid, dim3(256), 0, stream, (const float*)x, (float*)y, (int)C, (int)HW,
                       CU, ptiles, ctiles, vec);
  else
    hipLaunchKernelGGL(to_nhwc_kernel<bf16_t>, grid, dim3(256), 0, stream, (const bf16_t*)x, (bf16_t*)y, (int)C,
                       (int)HW, CU, ptiles, ctiles, vec);
  return hipGetLastError();
}
}  // namespace

hipError_t nhwc_pack(const Shape& s, const void* w, void* pk, hipStream_t stream) {
  return nh_pack(s, w, pk, nh_units_per_pixel(s), stream);
}

hipError_t launch_to_nhwc(int dtype, const void* x, void* y, int64_t N, int64_t C, int64_t HW, hipStream_t stream) {
  const int ue = dtype == DT_F32 ? 4 : 8;
  return nh_copy(dtype, x, y, N, C, HW, (int)((C + ue - 1) / ue), stream);
}

// ---- depthwise 3 x 3 layers: x, y channels-last with C whole 16-byte units ----

bool dw_nhwc_applies(const Shape& s) {
  const int64_t ue = 16 / s.esize();
  return s.G == s.C && s.K == s.C && s.R == 3 && s.S == 3 && s.dh == 1 && s.dw == 1 && s.sh == s.sw && s.sh <= 2 &&
         s.C % ue == 0 && s.N >= 1 && s.N * s.H * s.W * s.C * s.esize() < ((int64_t)1 << 31) - 64 && s.C < (1 << 24);
}

size_t dw_nhwc_packed_bytes(const Shape& s) { return (size_t)9 * s.C * s.esize(); }

hipError_t dw_nhwc_pack(const Shape& s, const void* w, void* pk, hipStream_t stream) {
  const dim3 grid((unsigned)((9 * s.C + 255) / 256));
  if (s.dtype == DT_F32)
    hipLaunchKernelGGL(dw3_pack_kernel<float>, grid, dim3(256), 0, stream, (const float*)w, (float*)pk, (int)s.C);
  else
    hipLaunchKernelGGL(dw3_pack_kernel<bf16_t>, grid, dim3(256), 0, stream, (const bf16_t*)w, (bf16_t*)pk, (int)s.C);
  return hipGetLastError();
}

hipError_t dw_nhwc_main(const Shape& s, const void* x, const void* pk, const void* b, void* y, hipStream_t stream) {
  DwArgs a;
  a.x = x; a.w = pk; a.b = b; a.y = y;
  a.x_bytes = (uint32_t)(s.N * s.H * s.W * s.C * s.esize());
  a.H = (int)s.H; a.W = (int)s.W; a.P = (int)s.P; a.Q = (int)s.Q;
  a.CU = (int)(s.C * s.esize() / 16);
  a.ph = s.ph; a.pw = s.pw;
  a.pstrips = (int)(s.sh == 1 ? (s.P + 1) / 2 : s.P);
  const bool wide = (s.Q + 6) / 7 * 7 <= (s.Q + 3) / 4 * 4;
  a.qstrips = (int)(wide ? (s.Q + 6) / 7 : (s.Q + 3) / 4);
  a.relu = s.relu ? 1 : 0;
  a.threads = s.N * a.pstrips * a.qstrips * a.CU;
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3((unsigned)((a.threads + 255) / 256)), dim3(256), 0, stream, a);
  };
  auto typed = [&](auto t) {
    using T = decltype(t);
    if (s.sh == 1) wide ? go(dw3_nhwc_kernel<T, 1, 7>) : go(dw3_nhwc_kernel<T, 1, 4>);
    else wide ? go(dw3_nhwc_kernel<T, 2, 7>) : go(dw3_nhwc_kernel<T, 2, 4>);
  };
  if (s.dtype == DT_F32) typed(0.f);
  else typed(bf16_t{});
  return hipGetLastError();
}

// ---- single layers -----------------------------------------------------------
// A layer called by itself takes N x C x H x W: a batch of its images is copied
// to channels-last in the workspace, then convolved.  The copy and the filter
// package together stay within 32 MiB (the static scratch, so no layer that ran
// there is refused), in batches of equal size.
namespace {
constexpr size_t kLayerBytes = (size_t)32 << 20;
}  // namespace

// The layer with the channels its copy holds: C, or C rounded up to whole
// 128-byte pieces where that adds at most a seventh (all lanes of a k-tile are
// then on one tap, which saves each its own tap arithmetic).
namespace {
Shape nh_layer_shape(const Shape& s) {
  const int64_t step = 128 / s.esize(), up = (s.C + step - 1) / step * step;
  Shape b = s;
  if ((up - s.C) * 7 <= s.C) b.C = b.Cg = up;
  return b;
}

// Images per batch, 0 where one image does not fit.
int64_t nh_layer_batch(const Shape& l) {
  const size_t pk = align256(nhwc_packed_bytes(l));
  const size_t img = (size_t)l.H * l.W * nh_units_per_pixel(l) * 16;
  if (pk + img > kLayerBytes) return 0;
  const int64_t nb = std::min<int64_t>(l.N, (int64_t)((kLayerBytes - pk) / img));
  const int64_t batches = (l.N + nb - 1) / nb;
  return (l.N + batches - 1) / batches;
}
}  // namespace

bool nhwc_layer_applies(const Shape& s) {
  if (s.dtype != DT_BF16 || s.N < 1 || s.G != 1) return false;
  Shape l = nh_layer_shape(s);
  l.N = nh_layer_batch(l);
  return l.N >= 1 && nhwc_applies(l);
}

size_t nhwc_layer_packed_bytes(const Shape& s) { return nhwc_packed_bytes(nh_layer_shape(s)); }

size_t nhwc_layer_bytes(const Shape& s) {
  const Shape l = nh_layer_shape(s);
  return align256((size_t)nh_layer_batch(l) * l.H * l.W * nh_units_per_pixel(l) * 16);
}

hipError_t nhwc_layer_pack(const Shape& s, const void* w, void* pk, hipStream_t stream) {
  return nh_pack(s, w, pk, nh_units_per_pixel(nh_layer_shape(s)), stream);
}

hipError_t nhwc_layer_main(const Shape& s, const void* x, const void* pk, const void* b, void* y, void* copy,
                           hipStream_t stream, const void* res) {
  Shape l = nh_layer_shape(s);
  const int64_t nb = nh_layer_batch(l);
  if (nb < 1 || !copy) return hipErrorInvalidValue;
  const int64_t in = s.C * s.H * s.W * s.esize(), out = s.K * s.P * s.Q * s.esize();
  for (int64_t n0 = 0; n0 < s.N; n0 += nb) {
    l.N = std::min(nb, s.N - n0);
    hipError_t e = nh_copy(s.dtype, reinterpret_cast<const char*>(x) + n0 * in, copy, l.N, s.C, s.H * s.W,
                           nh_units_per_pixel(l), stream);
    if (e != hipSuccess) return e;
    e = nhwc_main(l, copy, pk, b, reinterpret_cast<char*>(y) + n0 * out,
                  res ? reinterpret_cast<const char*>(res) + n0 * out : nullptr, false, stream);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t nhwc_main(const Shape& s, const void* x, const void* pk, const void* b, void* y, const void* res,
                     bool out_nhwc, hipStream_t stream) {
  NhArgs a;
  const int CU = nh_units_per_pixel(s);
  const int64_t shift = (s.ph * s.W + s.pw) * (int64_t)CU * 16;
  a.x = reinterpret_cast<const char*>(x) - shift;
  a.x_bytes = (uint32_t)(nhwc_input_bytes(s) + shift);
  a.w = pk;
  a.w_bytes = (uint32_t)nhwc_packed_bytes(s);
  a.b = b; a.res = res; a.y = y;
  a.H = (int)s.H; a.W = (int)s.W; a.K = (int)s.K; a.S = (int)s.S; a.R = (int)s.R;
  a.P = (int)s.P; a.Q = (int)s.Q; a.PQ = (int)(s.P * s.Q); a.NPQ = (int)(s.N * s.P * s.Q);
  a.sh = s.sh; a.sw = s.sw; a.ph = s.ph; a.pw = s.pw; a.dh = s.dh; a.dw = s.dw;
  a.CU = CU;
  a.cu_magic = magic_of(CU);
  a.s_magic = magic_of((int)s.S);
  a.ntap_units = (int)(s.R * s.S) * CU;
  a.nk = (a.ntap_units + 7) / 8;
  a.relu = s.relu ? 1 : 0;
  const int cfg = nh_config(s);
  const bool gen = !nh_uniform_taps(s);
  return s.dtype == DT_F32 ? nh_dispatch<float>(a, cfg, gen, out_nhwc, stream)
                           : nh_dispatch<bf16_t>(a, cfg, gen, out_nhwc, stream);
}

std::string nhwc_describe(const Shape& s) {
  const NhConfig& c = kNhConfigs[nh_config(s)];
  char buf[96];
  snprintf(buf, sizeof(buf), "tile=%dx%d stages=%d groups=%d taps=%s", c.TJ, c.TI, c.NST, c.G,
           nh_uniform_taps(s) ? "uniform" : "per_lane");
  return buf;
}

std::string nhwc_layer_describe(const Shape& s) {
  Shape l = nh_layer_shape(s);
  l.N = nh_layer_batch(l);
  char buf[384];
  snprintf(buf, sizeof(buf),
           "implicit_gemm kernels=nhwc_pack_kernel;to_nhwc_kernel;nhwc_conv_kernel<bf16> %s k_tiles=%d "
           "images_per_launch=%lld (channels-last copy of the input, rows of pixels and filters copied to LDS by DMA)",
           nhwc_describe(l).c_str(), (int)((s.R * s.S * nh_units_per_pixel(l) + 7) / 8), (long long)l.N);
  return buf;
}

}  // namespace convsel
