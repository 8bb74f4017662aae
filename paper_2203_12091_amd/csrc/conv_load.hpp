// Operand loading of the int8 contraction kernels (k_conv.hip, k_pred.hip):
// LDS slab layout, the LDS-DMA ring's primitives, the walks over a tile's
// slabs, and the launch arguments.
#pragma once

#include <limits.h>
#include <math.h>

#include <type_traits>

#include "fls.hpp"

namespace fxpq {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v4i_a4 __attribute__((ext_vector_type(4), aligned(4)));  // dword-aligned 16 bytes
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int BK = 64;
// Cache policy of the int32 accumulator stores: non-temporal (the tensor is
// read once, by the FL search that follows, not by this kernel).
constexpr int kAccPolicy = 2;

// LDS slab layout: rows of 64 bytes (four 16-byte chunks), no padding; chunk
// c of row r sits at chunk position c ^ f(r) with f(r) = (r >> 2) & 3.  The
// MFMA operand reads (lane l: row l % 32, one chunk) then run at the full
// ds_read_b128 rate on gfx950 (measured: 1.5x slower with f = (r >> 1) ^
// (r >> 3), 3x without a swizzle); the 16-byte stores of whole rows are
// insensitive to it.
__device__ inline int lds_swz(int row) { return (row >> 2) & 3; }
__device__ inline int lds_off(int row, int chunk) {
  return row * 64 + ((chunk ^ lds_swz(row)) & 3) * 16;
}

// FAST64: C % 64 == 0, register-staged slabs; GEN16: C % 16 == 0; RGB4: the
// 4-channel padded input; DMA64: C % 64 == 0, slabs loaded straight into a
// three-stage LDS ring (global_load_lds), two slabs in flight.  HALO4 /
// HALO8: C % 64 == 0, tiles of whole output-image rows whose input patch
// (up to 256 / 512 pixels per channel chunk) is loaded into LDS once and read
// by every filter tap, weights through the DMA ring.  SPLIT64, SPLIT32:
// C % 64 == 0, 64 x 64 / 32 x 32 tiles whose depth the four waves split
// (SplitTile).  DMA16, SPLIT64G, SPLIT32G: the same for C % 16 == 0.
enum Loader { LD_FAST64 = 0, LD_GEN16 = 1, LD_RGB4 = 2, LD_DMA64 = 3, LD_HALO4 = 4, LD_HALO8 = 5,
              LD_RGB8 = 6, LD_SPLIT64 = 7, LD_SPLIT32 = 8, LD_DMA16 = 9, LD_SPLIT64G = 10,
              LD_SPLIT32G = 11 };
constexpr int split_t(int loader) {
  return loader == LD_SPLIT64 || loader == LD_SPLIT64G ? 2
         : (loader == LD_SPLIT32 || loader == LD_SPLIT32G ? 1 : 0);
}
// Loaders through the LDS ring of whole blocks; any C % 16 == 0 (not only 64).
constexpr bool is_ring(int loader) { return loader == LD_DMA64 || loader == LD_DMA16; }
constexpr bool is_gen(int loader) {
  return loader == LD_DMA16 || loader == LD_SPLIT64G || loader == LD_SPLIT32G;
}

constexpr bool is_halo(int loader) { return loader == LD_HALO4 || loader == LD_HALO8; }

// Weight stages of the halo tiles' LDS ring (HD - 1 slabs in flight).
constexpr int kHaloStages = 3;

// 16-byte padding sources of the LDS-ring loader: code 0, and code -128 for
// inputs stored as u - 128 (both the value 0).
__device__ int4 kPadVec[2] = {{0, 0, 0, 0},
                              {(int)0x80808080, (int)0x80808080, (int)0x80808080, (int)0x80808080}};

// s_waitcnt immediate that waits until at most n vector memory operations are
// outstanding (gfx9 encoding: vmcnt split over bits 3:0 and 15:14; expcnt and
// lgkmcnt left at their maxima, i.e. not waited for).
template <int N>
__device__ inline void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

// One 16-byte global -> LDS load per lane (global_load_lds_dwordx4): lane l's
// bytes land at lds + 16 l.  Issued as inline asm so that the compiler does
// not add its own conservative wait for these LDS writes before later LDS
// reads (it cannot tell the ring stages apart); the ring waits explicitly
// (wait_vmcnt) and orders with ring_barrier().  M0 holds the wave-uniform LDS
// address; the s_nop separates its write from the load.
__device__ inline void dma16(const int8_t* g, int8_t* lds) {
  const uint32_t l = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)lds);
  asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(g), "{m0}"(l) : "memory");
}

// Workgroup barrier without the memory fence __syncthreads() adds: that fence
// would wait for every outstanding LDS-ring load.  The empty asm statements
// keep the compiler from moving memory accesses across it.
__device__ inline void ring_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
enum Epi { EPI_ACC = 0, EPI_MM = 1, EPI_WIN = 2, EPI_REQ = 3 };

struct ConvArgs {
  const int8_t* x;
  const int8_t* w;
  const int32_t* colsum;
  int32_t* acc;
  int N, H, W, C, K, R, S, stride, pad, Ho, Wo;
  int M;        // rows
  int kdepth;   // R * S * C
  int wrow;     // bytes per weight row (kdepth, or padded to 64 for RGB4)
  int x_type;
  int want_mm;  // reduce min / max of the epilogue values
  SrcDev ep;    // kind == FXPQ_SRC_ACC when an epilogue is given
  int has_ep;
  double* mm_part;
  unsigned* mm_ticket;  // small grids: the last block writes the total to mm_out
  double* mm_out;
  // EPI_ACC: store only when the FL-search plan asks for the general pass
  int only_if_general;
  const FlsPlan* plan_in;
  // EPI_WIN
  int wl, sign_req, fl_lo, fl_hi;
  const double* mm;      // min / max of the C-Block values
  long long* part_i;
  double* part_f;
  FlsPlan* plan;
  fxpq_fmt* fmt_win;
  unsigned* flags;
  // EPI_REQ
  const fxpq_fmt* fmt_req;
  int8_t* y;
  int y_type;
  // predicted C-Block: row-tile workers and column tiles; in deferred mode
  // block 0 records the decision's inputs
  int workers, ntm, ntn;
  PredJob* job;
  unsigned* job_miss;
  int64_t job_per_thread;
  // halo tiles: hG images of hTH output rows each (hG > 1 only with hTH ==
  // Ho), hTPI tiles per image (hG == 1), input patch hPH x hPW per image;
  // stores of rows that do not exist go to `sink` (32 int32)
  int hG, hTH, hTPI, hPH, hPW;
  // C % 16 walks: 64 channels as filter rows, taps and channels, and in the input
  int gen_r, gen_s, gen_c;
  int64_t gen_step;
  // RGB8: 16-byte chunks (four taps) per filter row; four chunks as rows and chunks
  int rgb_chunks, rgb_step_r, rgb_step_c;
  int32_t* sink;
};

// Tile configurations: block BM x BN, four waves of (32 TM) x (32 TN) (32 x 64 in
// 128 x 64 tiles), MINW
// waves per SIMD requested from the register allocator.
enum TileCfg { TC_256x64 = 0, TC_128x128 = 1, TC_256x128 = 2, TC_H224x256 = 3, TC_H128x256 = 4,
               TC_64x64 = 5, TC_32x32 = 6, TC_128x64 = 7 };

// Accumulators per thread of a configuration (the per-thread bound of the
// fused window epilogue).
constexpr int conv_per_thread(int cfg) { return cfg == TC_256x128 ? 128 : 64; }

// Slabs of a BM x BN tile, 64 bytes of depth each, loaded straight into an LDS
// stage (C % 64 == 0): each of WAVES waves fills 1 KB pieces (16 rows of 64
// bytes), piece q = WAVES j + wave, lane l -> row 16 q + l / 4, physical chunk l % 4, which holds
// logical chunk (l % 4) ^ f(row) of the swizzled layout.  The channel chunks
// are walked outermost and the filter taps innermost.  The walk is incremental:
// a scalar tap (ir, is) with its offsets, each row's address of tap (0, 0)
// fixed, so that a slab costs a few vector instructions per load (the divisions
// and 64-bit products of addressing every slab from its number took longer than
// its MFMAs: 14x14x256 3x3 at batch 256 ran 56 -> 48 us plain, 74 -> 66 us
// predicted).
//
// GEN: any C % 16 == 0.  The depth is walked in order, and a slab's four chunks
// may belong to different taps: each lane walks the taps of its own chunk (the
// same in all its pieces), 64 channels on per slab, and chunks past the depth
// take zero weights.  Against slabs staged through registers, plain / predicted:
// 760 x 32 x 2000 in split tiles 31.9 / 38.7 -> 10.3 / 12.2 us, 50176 x 256 x 1296
// in 128 x 128 tiles 49.5 / 53.7 -> 42.1 / 47.6.
template <int BM, int BN, int WAVES = 4, bool GEN = false>
struct RingLoad {
  static constexpr int AJ = BM / (16 * WAVES), BJ = BN / (16 * WAVES);
  static constexpr int kOps = AJ + BJ;  // loads per wave and slab
  int64_t arow[AJ];                     // address of (ih0, iw0, chunk), used where it is valid
  int aih[AJ], aiw[AJ];
  const int8_t* bsrc[BJ];
  int64_t padp, rowskip;
  int ir, is, ic;  // next slab: filter tap, first channel (GEN: of the lane's chunk)
  int64_t atap;    // (ir * W + is) * C + ic
  int btap;        // (ir * S + is) * C + ic
  int kt, kc;      // GEN: next slab of the tile, the lane's chunk

  __device__ inline void cols(const ConvArgs& a, int a_off, int n0, int wave, int lane) {
    kc = ((lane & 3) ^ lds_swz(lane >> 2)) & 3;
#pragma unroll
    for (int j = 0; j < BJ; ++j) {
      const int row = 16 * (WAVES * j + wave) + (lane >> 2);
      const int col = n0 + row;
      const int cc = col < a.K ? col : a.K - 1;
      bsrc[j] = a.w + (int64_t)cc * a.wrow + (GEN ? 0 : kc * 16);
    }
    padp = (int64_t)(uintptr_t)&kPadVec[a_off];
    rowskip = (int64_t)(a.W - a.S) * a.C;
    seek(a, 0);
  }
  // Rows m0 .. m0 + BM - 1, from their first slab.
  __device__ inline void rows(const ConvArgs& a, int m0, int wave, int lane) {
    const int hw_out = a.Ho * a.Wo;
#pragma unroll
    for (int j = 0; j < AJ; ++j) {
      const int row = 16 * (WAVES * j + wave) + (lane >> 2);
      const int grow = m0 + row;
      const bool ok = grow < a.M;
      const int rr = ok ? grow : a.M - 1;
      const int n = rr / hw_out, rem = rr - n * hw_out;
      const int oh = rem / a.Wo, ow = rem - oh * a.Wo;
      aih[j] = ok ? oh * a.stride - a.pad : INT_MIN / 2;  // no row: never inside
      aiw[j] = ow * a.stride - a.pad;
      arow[j] = (int64_t)(uintptr_t)a.x +
                (((int64_t)n * a.H + (oh * a.stride - a.pad)) * a.W + aiw[j]) * a.C +
                (GEN ? 0 : kc * 16);
    }
  }
  // The walk at slab q of a tile.
  __device__ inline void seek(const ConvArgs& a, int q) {
    if constexpr (GEN) {
      btap = q * BK + kc * 16;
      const int tap = btap / a.C;
      ic = btap - tap * a.C;
      ir = tap / a.S;
      is = tap - ir * a.S;
      kt = q;
    } else {
      const int taps = a.R * a.S, chunk = q / taps, tap = q - chunk * taps;
      ir = tap / a.S;
      is = tap - ir * a.S;
      ic = chunk * BK;
      btap = tap * a.C + ic;
    }
    atap = ((int64_t)ir * a.W + is) * a.C + ic;
  }
  // Issues load i (of kOps) of the next slab into stage (sa, sb).
  __device__ inline void load(const ConvArgs& a, int i, int8_t* sa, int8_t* sb, int wave) {
    if (i < AJ) {
      const bool ok = (unsigned)(aih[i] + ir) < (unsigned)a.H && (unsigned)(aiw[i] + is) < (unsigned)a.W;
      const int64_t p = ok ? arow[i] + atap : padp;
      dma16(reinterpret_cast<const int8_t*>(p), &sa[(WAVES * i + wave) * 1024]);
    } else if constexpr (GEN) {
      const int8_t* p = bsrc[i - AJ] + btap;
      dma16(ir < a.R ? p : reinterpret_cast<const int8_t*>(&kPadVec[0]), &sb[(WAVES * (i - AJ) + wave) * 1024]);
    } else {
      dma16(bsrc[i - AJ] + btap, &sb[(WAVES * (i - AJ) + wave) * 1024]);
    }
  }
  // Steps to the slab after; true when that was the tile's last slab (the walk
  // is back at the first one).
  __device__ inline bool advance(const ConvArgs& a) {
    if constexpr (GEN) {
      if (++kt == (a.kdepth + BK - 1) / BK) {
        seek(a, 0);
        return true;
      }
      // 64 channels on: gen_r filter rows, gen_s taps, gen_c channels; a wrap of
      // the channels moves one tap on, one of the taps a row
      ic += a.gen_c;
      const bool cw = ic >= a.C;
      ic -= cw ? a.C : 0;
      is += a.gen_s + (cw ? 1 : 0);
      const bool sw = is >= a.S;
      is -= sw ? a.S : 0;
      ir += a.gen_r + (sw ? 1 : 0);
      atap += a.gen_step + (sw ? rowskip : 0);
      btap += BK;
      return false;
    }
    // next tap; after the last, the next channel chunk
    atap += a.C;
    btap += a.C;
    if (++is == a.S) {
      is = 0;
      atap += rowskip;
      if (++ir == a.R) {
        ir = 0;
        ic += BK;
        if (ic >= a.C) ic = 0;
        atap = ic;
        btap = ic;
        return ic == 0;
      }
    }
    return false;
  }
  // All of the next slab's loads.
  __device__ inline bool issue(const ConvArgs& a, int8_t* sa, int8_t* sb, int wave) {
#pragma unroll
    for (int i = 0; i < kOps; ++i) load(a, i, sa, sb, wave);
    return advance(a);
  }
};

// Slabs staged through registers (C % 64, C % 16 or padded RGB): thread t loads
// chunk t % 4 of rows t / 4 + 64 i.  Loads are unconditional (from a valid
// address when the element does not exist); the pad / zero value replaces them
// at the LDS store.  A select right after the load would let the compiler branch
// around the load and then wait at the join for the loads just issued, i.e. for
// the next slab before this slab's MFMAs.
template <int BM, int BN, int LOADER>
struct StagedLoad {
  static constexpr int ACH = BM / 64, BCH = BN / 64;
  const int8_t* abase[ACH];
  int ih0[ACH], iw0[ACH];
  bool aval[ACH];
  const int8_t* bptr[BCH];
  v4i regA[ACH], regB[BCH];
  bool aok[ACH], bok[BCH];
  // LD_RGB8: pixel index of the row at (ih0, 0) within its image, dword shift of
  // the loaded pixels (0 inside the image), the next chunk's filter row and its
  // chunk within the row
  int rgb_p[ACH], rgb_d[ACH];
  int rgb_r, rgb_c;
  int kt;          // next slab of the tile
  // LD_FAST64, LD_GEN16: filter tap and channel of the next chunk (uniform /
  // per thread), advanced slab by slab
  int ir, is, ic;

  __device__ inline void cols(const ConvArgs& a, int n0, int tid) {
#pragma unroll
    for (int i = 0; i < BCH; ++i) {
      int col = n0 + (tid >> 2) + 64 * i;
      int cc = col < a.K ? col : a.K - 1;
      bptr[i] = a.w + (int64_t)cc * a.wrow;
    }
  }
  __device__ inline void rows(const ConvArgs& a, int m0, int tid) {
    const int hw_out = a.Ho * a.Wo;
#pragma unroll
    for (int i = 0; i < ACH; ++i) {
      int row = m0 + (tid >> 2) + 64 * i;
      aval[i] = row < a.M;
      int rr = aval[i] ? row : a.M - 1;
      int n = rr / hw_out, rem = rr - n * hw_out;
      int oh = rem / a.Wo, ow = rem - oh * a.Wo;
      ih0[i] = oh * a.stride - a.pad;
      iw0[i] = ow * a.stride - a.pad;
      abase[i] = a.x + (int64_t)n * a.H * a.W * a.C;
    }
    restart(a, tid);
    if constexpr (LOADER == LD_RGB8) {
#pragma unroll
      for (int i = 0; i < ACH; ++i) {
        rgb_p[i] = ih0[i] * a.W;
        if (!aval[i]) ih0[i] = INT_MIN / 2;  // no row: never inside
      }
    }
  }
  // The walk at the first slab of the same rows.
  __device__ inline void restart(const ConvArgs& a, int tid) {
    kt = 0;
    ir = is = ic = 0;
    if constexpr (LOADER == LD_RGB8) {
      rgb_r = (tid & 3) / a.rgb_chunks;
      rgb_c = (tid & 3) - rgb_r * a.rgb_chunks;
    } else if constexpr (LOADER == LD_GEN16) {
      ic = (tid & 3) * 16;
      wrap(a);
    }
  }
  __device__ inline void wrap(const ConvArgs& a) {
    while (ic >= a.C) {
      ic -= a.C;
      if (++is == a.S) is = 0, ++ir;
    }
  }
  // Loads the next slab into registers; true after the tile's last one (rows()
  // starts the next tile).
  __device__ inline bool gload(const ConvArgs& a, int ktiles, int tid, int padw, const int* rs_tab) {
    const int kc = tid & 3;
    // FAST64 walks the depth channel chunk by channel chunk with the filter
    // taps innermost, so that consecutive slabs read neighbouring pixels of
    // the same channels (cache reuse); the integer sums do not depend on the
    // order.
    const int k0 = (LOADER == LD_FAST64) ? (ir * a.S + is) * a.C + ic : kt * BK;
    if constexpr (LOADER == LD_FAST64) {
#pragma unroll
      for (int i = 0; i < ACH; ++i) {
        int ih = ih0[i] + ir, iw = iw0[i] + is;
        bool ok = aval[i] && ih >= 0 && ih < a.H && iw >= 0 && iw < a.W;
        const int8_t* p = abase[i] + (ok ? ((int64_t)ih * a.W + iw) * a.C + ic + kc * 16 : 0);
        regA[i] = *reinterpret_cast<const v4i*>(p);
        aok[i] = ok;
      }
      if (++is == a.S) {
        is = 0;
        if (++ir == a.R) {
          ir = 0;
          ic += BK;
        }
      }
    } else if constexpr (LOADER == LD_GEN16) {
      bool kin = k0 + kc * 16 < a.kdepth;
#pragma unroll
      for (int i = 0; i < ACH; ++i) {
        int ih = ih0[i] + ir, iw = iw0[i] + is;
        bool ok = kin && aval[i] && ih >= 0 && ih < a.H && iw >= 0 && iw < a.W;
        const int8_t* p = abase[i] + (ok ? ((int64_t)ih * a.W + iw) * a.C + ic : 0);
        regA[i] = *reinterpret_cast<const v4i*>(p);
        aok[i] = ok;
      }
      ic += BK;
      wrap(a);
    } else if constexpr (LOADER == LD_RGB8) {
      // filters re-laid as [r][chunk][4 taps][c] (rgb8_setup): a chunk is four
      // neighbouring pixels of one input row, one 16-byte load from column iw
      // clamped to [0, W - 4] (W >= 4); at the image borders the LDS store
      // shifts them and pads the pixels outside the row (the taps past S have
      // zero weights: their pixels only need to be readable).  Rows past R are
      // zero filter rows; a row outside the image is all padding (shift 8).
      const int r = rgb_r < a.R ? rgb_r : INT_MIN / 2, rw = rgb_r * a.W;
#pragma unroll
      for (int i = 0; i < ACH; ++i) {
        const int iw = iw0[i] + 4 * rgb_c, iwc = min(max(iw, 0), a.W - 4);
        const bool ok = (unsigned)(ih0[i] + r) < (unsigned)a.H;
        const unsigned px = ok ? (unsigned)(rgb_p[i] + rw + iwc) : 0u;
        regA[i] = *reinterpret_cast<const v4i_a4*>(abase[i] + (uint64_t)px * 4);
        rgb_d[i] = ok ? iw - iwc : 8;
        aok[i] = true;
      }
      // four chunks on
      rgb_r += a.rgb_step_r;
      rgb_c += a.rgb_step_c;
      const bool wrap_c = rgb_c >= a.rgb_chunks;
      rgb_c -= wrap_c ? a.rgb_chunks : 0;
      rgb_r += wrap_c;
    } else {  // LD_RGB4: four 4-byte pixels per 16-byte chunk
#pragma unroll
      for (int i = 0; i < ACH; ++i) {
        v4i v;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          int rs = (k0 + kc * 16 + 4 * j) >> 2;
          int t = (rs < 128) ? rs_tab[rs] : -1;
          int word = padw;
          if (t >= 0 && aval[i]) {
            int ih = ih0[i] + (t >> 16), iw = iw0[i] + (t & 0xFFFF);
            if (ih >= 0 && ih < a.H && iw >= 0 && iw < a.W)
              word = *reinterpret_cast<const int*>(abase[i] + ((int64_t)ih * a.W + iw) * 4);
          }
          v[j] = word;
        }
        regA[i] = v;
        aok[i] = true;
      }
    }
#pragma unroll
    for (int i = 0; i < BCH; ++i) {
      const int k = k0 + kc * 16;
      const bool kin = LOADER != LD_GEN16 || k < a.kdepth;
      regB[i] = *reinterpret_cast<const v4i*>(bptr[i] + (kin ? k : 0));
      bok[i] = kin;
    }
    return ++kt == ktiles;
  }
  __device__ inline void lstore(int8_t* sa, int8_t* sb, int tid, int padw) const {
    const int kc = tid & 3;
    const v4i padv = {padw, padw, padw, padw};
#pragma unroll
    for (int i = 0; i < ACH; ++i) {
      v4i v = aok[i] ? regA[i] : padv;
      if constexpr (LOADER == LD_RGB8) {
        const int d = rgb_d[i];
        if (d != 0) {  // image border or missing row (no loads in here)
          v4i o;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int m = j + d;
            const int pk = m <= 0 ? v[0] : (m == 1 ? v[1] : (m == 2 ? v[2] : v[3]));
            o[j] = (m >= 0 && m < 4) ? pk : padw;
          }
          v = o;
        }
      }
      *reinterpret_cast<v4i*>(&sa[lds_off((tid >> 2) + 64 * i, kc)]) = v;
    }
#pragma unroll
    for (int i = 0; i < BCH; ++i)
      *reinterpret_cast<v4i*>(&sb[lds_off((tid >> 2) + 64 * i, kc)]) = bok[i] ? regB[i] : v4i{0, 0, 0, 0};
  }
};

// The (row, filter column) of each tap of the padded RGB layout's packed filters.
__device__ inline void rgb4_table(const ConvArgs& a, int* rs_tab) {
  for (int i = threadIdx.x; i < 128; i += 256) rs_tab[i] = (i < a.R * a.S) ? ((i / a.S) << 16) | (i % a.S) : -1;
  __syncthreads();
}

// MFMAs of one staged slab: two 32-deep steps over a wave's TM x TN tile.  All
// fragments of the slab are read first, then the MFMAs run: the LDS latency is
// paid once per slab (interleaving reads and MFMAs on a few reused registers
// paid it before every pair of MFMAs).  between(i) comes before MFMA i: vector
// instructions there run while the reads (i = 0) or the MFMA before are under
// way (the ring's loads, 40 instructions a slab, moved there from before the
// reads: 14x14x256 3x3 at batch 256 47.3 -> 43.2 us plain, a chain of 72 slabs
// in four blocks 32.6 -> 27.1).
template <int TM, int TN, typename F>
__device__ __attribute__((always_inline)) inline void slab_mfma(const int8_t* sa, const int8_t* sb,
                                                                int row0, int col0, int lane,
                                                                v16i (&acc)[TM][TN], F between) {
  v4i af[2][TM], bf[2][TN];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
    for (int mi = 0; mi < TM; ++mi)
      af[kk][mi] = *reinterpret_cast<const v4i*>(
          &sa[lds_off(row0 + mi * 32 + (lane & 31), kk * 2 + (lane >> 5))]);
#pragma unroll
    for (int ni = 0; ni < TN; ++ni)
      bf[kk][ni] = *reinterpret_cast<const v4i*>(
          &sb[lds_off(col0 + ni * 32 + (lane & 31), kk * 2 + (lane >> 5))]);
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int kk = 0; kk < 2; ++kk)
#pragma unroll
    for (int mi = 0; mi < TM; ++mi)
#pragma unroll
      for (int ni = 0; ni < TN; ++ni) {
        between((kk * TM + mi) * TN + ni);
        acc[mi][ni] =
            __builtin_amdgcn_mfma_i32_32x32x32_i8(af[kk][mi], bf[kk][ni], acc[mi][ni], 0, 0, 0);
      }
}
template <int TM, int TN>
__device__ inline void slab_mfma(const int8_t* sa, const int8_t* sb, int row0, int col0, int lane,
                                 v16i (&acc)[TM][TN]) {
  slab_mfma<TM, TN>(sa, sb, row0, col0, lane, acc, [](int) {});
}

// A 32 T x 32 T tile (T = 1, 2) whose depth the block's four waves split: each
// wave walks its quarter of the slabs through a ring of its own (three stages,
// two slabs in flight; no barriers, a wave waits for its own loads only), then
// the partial accumulators are added through LDS.  T = 2 leaves wave w with the
// 32 x 32 subtile (w / 2, w % 2), T = 1 with its four accumulators per thread
// 4 w .. 4 w + 3, in out[0 .. 3].
constexpr int kSplitD = 2;  // slabs in flight
template <int T>
constexpr int kSplitStage = T * 64 * 64;  // bytes of a stage: 32 T rows, 32 T columns
template <int T>
constexpr int kSplitLds = 4 * (kSplitD + 1) * kSplitStage<T>;
template <int T, bool GEN>
struct SplitTile {
  static constexpr int D = kSplitD, ST = kSplitStage<T>, SA = 32 * T * 64;
  using Ring = RingLoad<32 * T, 32 * T, 1, GEN>;
  static constexpr int OPS = Ring::kOps, MFMAS = 2 * T * T, PER = (OPS + MFMAS - 1) / MFMAS;
  Ring ld;
  int n;         // this wave's slabs
  int8_t* ring;  // its stages

  // Sends the first slabs' loads.
  __device__ __attribute__((always_inline)) inline void start(const ConvArgs& a, int a_off, int m0,
                                                              int n0, int ktiles, int wave,
                                                              int lane, int8_t* lds) {
    const int q0 = (int)((int64_t)ktiles * wave / 4);
    n = (int)((int64_t)ktiles * (wave + 1) / 4) - q0;
    ring = lds + wave * (D + 1) * ST;
    ld.cols(a, a_off, n0, 0, lane);
    ld.rows(a, m0, 0, lane);
    ld.seek(a, q0);
    for (int i = 0; i < D && i < n; ++i) (void)ld.issue(a, ring + i * ST, ring + i * ST + SA, 0);
  }
  __device__ __attribute__((always_inline)) inline void finish(const ConvArgs& a, int wave, int lane,
                                                               int8_t* lds, v16i& out) {
    v16i acc[T][T];
#pragma unroll
    for (int t = 0; t < T * T; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[t / T][t % T][e] = 0;
    int8_t* cur = ring;
    for (int s = 0; s < n - D; ++s) {
      wait_vmcnt<OPS*(D - 1)>();
      asm volatile("" ::: "memory");
      int8_t* st = cur == ring ? ring + D * ST : cur - ST;
      slab_mfma<T, T>(cur, cur + SA, 0, 0, lane, acc, [&](int i) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < PER; ++j)
          if (i * PER + j < OPS) ld.load(a, i * PER + j, st, st + SA, 0);
        __builtin_amdgcn_sched_barrier(0);
      });
      (void)ld.advance(a);
      cur = cur == ring + D * ST ? ring : cur + ST;
    }
    for (int left = min(D, n); left > 0; --left) {
      if (left > 1) wait_vmcnt<OPS>();
      else wait_vmcnt<0>();
      asm volatile("" ::: "memory");
      slab_mfma<T, T>(cur, cur + SA, 0, 0, lane, acc);
      cur = cur == ring + D * ST ? ring : cur + ST;
    }
    add_waves(acc, wave, lane, lds, out);
  }
  __device__ __attribute__((always_inline)) static inline void add_waves(const v16i (&acc)[T][T],
                                                                         int wave, int lane,
                                                                         int8_t* lds, v16i& out) {
    // 16-byte pieces (wave, subtile t, group g of four accumulators, lane); the
    // rings have been read
    static_assert(4 * T * T * 4 * 64 * 16 <= kSplitLds<T>, "partial sums fit the rings");
    __syncthreads();
    v4i* red = reinterpret_cast<v4i*>(lds);
#pragma unroll
    for (int t = 0; t < T * T; ++t) {
      const v16i& v = acc[t / T][t % T];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const v4i p = {v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
        if ((T == 2 ? t : g) != wave) red[((wave * T * T + t) * 4 + g) * 64 + lane] = p;
        else
#pragma unroll
          for (int j = 0; j < 4; ++j) out[(T == 2 ? 4 * g : 0) + j] = p[j];
      }
    }
    __syncthreads();
#pragma unroll
    for (int o = 1; o < 4; ++o) {
      const int from = (wave + o) & 3;
#pragma unroll
      for (int g = 0; g < (T == 2 ? 4 : 1); ++g) {
        const v4i v = red[((from * T * T + (T == 2 ? wave : 0)) * 4 + (T == 2 ? g : wave)) * 64 + lane];
#pragma unroll
        for (int j = 0; j < 4; ++j) out[4 * g + j] += v[j];
      }
    }
  }
};

// Tile shape and grid of a conv; loader choice and the geometry in `a`.
dim3 conv_setup(const fxpq_conv_desc& d, const void* x, int x_type, const int8_t* w,
                const int32_t* colsum, const SrcDev* ep, ConvArgs& a, int& loader, int& cfg, int cus,
                int halo = FXPQ_TILING_GEMM, bool wide_ok = true);
// Grids that leave CUs idle: 64 x 64 or 32 x 32 tiles with split depth instead.
void split_setup(ConvArgs& a, int& loader, int& cfg, dim3& grid, int cus);
// The padded RGB layout: re-lays the filters into the handle's buffer, filter
// rows padded to whole 16-byte chunks of four taps, and switches to the loader
// that reads four pixels at a time.  plain: the contraction alone.
void rgb8_setup(const Ctx& c, const fxpq_conv_desc& d, ConvArgs& a, int& loader, bool plain);

}  // namespace fxpq
