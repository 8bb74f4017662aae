// C-Blocks over codes wider than 8 bits (Sec. "Integer-Only Inference": the
// first and last layers start at 32-bit activations and weights, Sec.
// "Initial Design Generation"), on the int8 matrix cores.
//
// A code of up to 32 bits is written in base 256.  Input codes x split into
// np_x byte planes: planes below the top hold the unsigned bytes (stored as
// byte - 128, the U8OFF storage the int8 contraction already corrects with the
// weight column sums), the top plane holds the rest (signed storage for
// signed formats).  Weight codes split into balanced digits in [-128, 127]
// (int8 as they are).  Then
//     sum_k x_k w_k = sum_{p,q} 256^(p+q) sum_k xp_k wq_k,
// each inner sum an ordinary int8 contraction with exact int32 accumulation;
// the combine kernel adds them with exact shifts in 128-bit integers and
// applies the C-Block epilogue in integers, writing int64 values at the
// epilogue's scale (an FXPQ_SRC_INT source for the FxP-QLayer that follows).
#include <type_traits>

#include "conv_load.hpp"

namespace fxpq {

namespace {

constexpr int kMaxPlanes = 5;  // balanced base-256 digits of a 32-bit code

__device__ inline void flag(unsigned* flags, unsigned bit) { atomicOr(flags, bit); }

// Byte planes of the inputs and digit planes of the weights with their column
// sums, in one launch: block b < K takes weight row b, the others the inputs,
// four values per thread and step (16-byte loads, one dword per plane and
// store; value by value with byte stores the 3.2 M inputs of a 16 x 224 x 224
// image batch took 28 us).
__global__ __launch_bounds__(kThreads) void k_split(const int32_t* __restrict__ x, int64_t nx,
                                                    int np_x, int sign_x, int64_t xs,
                                                    int8_t* __restrict__ px,
                                                    const int32_t* __restrict__ w, int64_t wrow,
                                                    int K, int np_w, int sign_w, int64_t ws,
                                                    int8_t* __restrict__ pw, int R, int S, int chunks,
                                                    int32_t* __restrict__ cs, unsigned* flags) {
  __shared__ long long sh[8];
  bool bad = false;
  if ((int)blockIdx.x < K) {
    long long sum[kMaxPlanes];
#pragma unroll
    for (int p = 0; p < kMaxPlanes; ++p) sum[p] = 0;
    const int64_t row = (int64_t)blockIdx.x * wrow;
    for (int64_t i = 4 * threadIdx.x; i < wrow; i += 4 * kThreads) {
      v4i v = {0, 0, 0, 0};
      if (chunks) {  // padded RGB, filter rows of whole chunks of four taps
        const int r = (int)i / (16 * chunks), t = ((int)i - r * 16 * chunks) >> 2;
        if (r < R && t < S) v = *reinterpret_cast<const v4i_a4*>(w + row + (r * S + t) * 4);
      } else {
        v = *reinterpret_cast<const v4i_a4*>(w + row + i);
      }
      // unsigned codes are read as uint32 (the storage of 32-bit ones)
      int64_t r[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) r[e] = sign_w ? (int64_t)v[e] : (int64_t)(uint32_t)v[e];
#pragma unroll
      for (int p = 0; p < kMaxPlanes; ++p) {
        if (p >= np_w) break;
        unsigned pack = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int d = (int)((r[e] + 128) & 255) - 128;
          pack |= (unsigned)(d & 255) << (8 * e);
          sum[p] += d;
          r[e] = (r[e] - d) >> 8;
        }
        *reinterpret_cast<unsigned*>(pw + p * ws + row + i) = pack;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) bad |= r[e] != 0;
    }
#pragma unroll
    for (int p = 0; p < kMaxPlanes; ++p) {
      if (p >= np_w) break;
      const long long t = block_reduce(sum[p], OpAddL(), sh);
      if (threadIdx.x == 0) cs[(int64_t)p * K + blockIdx.x] = (int32_t)t;
    }
  } else {
    for (int64_t i = 4 * ((blockIdx.x - K) * (int64_t)kThreads + threadIdx.x); i < nx;
         i += 4 * (int64_t)(gridDim.x - K) * kThreads) {
      const v4i v = *reinterpret_cast<const v4i_a4*>(x + i);
      for (int p = 0; p < np_x; ++p) {
        const bool top = p == np_x - 1;
        unsigned pack = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          // the top plane holds the rest: signed, or (unsigned codes are read
          // as uint32, the storage of 32-bit ones) a byte - 128 like the others
          const int t = sign_x || !top ? v[e] >> (8 * p) : (int)((uint32_t)v[e] >> (8 * p));
          if (top) bad |= sign_x ? (t < -128 || t > 127) : (uint32_t)t > 255u;
          pack |= (unsigned)((top && sign_x ? t : t - 128) & 255) << (8 * e);
        }
        *reinterpret_cast<unsigned*>(px + p * xs + i) = pack;
      }
    }
  }
  if (bad) flag(flags, FXPQ_FLAG_CODE);
}

// Bits of |v| (0 for v == 0).
__device__ inline int bits128(__int128 v) {
  unsigned __int128 m = v < 0 ? (unsigned __int128)(-v) : (unsigned __int128)v;
  unsigned long long hi = (unsigned long long)(m >> 64), lo = (unsigned long long)m;
  return hi ? 128 - __builtin_clzll(hi) : (lo ? 64 - __builtin_clzll(lo) : 0);
}

// v * 2^sh, with `bad` set where the result would not stay below 2^120.
__device__ inline __int128 shl_checked(__int128 v, int sh, bool& bad) {
  if (v == 0) return 0;
  if (sh > 119 || bits128(v) + sh > 120) {
    bad = true;
    return 0;
  }
  return v * ((__int128)1 << sh);
}

// Bits of |v| (0 for v == 0).
__device__ inline int bits64(int64_t v) {
  const unsigned long long m = v < 0 ? 0ull - (unsigned long long)v : (unsigned long long)v;
  return m ? 64 - __builtin_clzll(m) : 0;
}

// v * 2^sh, with `bad` set where the result would not stay below 2^62.
__device__ inline int64_t shl62(int64_t v, int sh, bool& bad) {
  if (v == 0) return 0;
  if (sh > 61 || bits64(v) + sh > 62) {
    bad = true;
    return 0;
  }
  return v * ((int64_t)1 << sh);
}

// The C-Block epilogue on an exact contraction value a (bias, Scale
// multiply and offset, ReLU; every step exact): 128-bit arithmetic, or int64
// where the host has shown the contraction stays below 2^62 (every step then
// checked against 2^62).  bad: the value leaves [-2^62, 2^62] (written as 0).
__device__ inline int64_t wide_epi(__int128 a, const EpiRaw& r, const EpiU& u, const SrcDev& ep,
                                   bool& bad) {
  bool b = false;
  __int128 t = shl_checked(a, u.sh_acc, b);
  if (ep.bias) t += shl_checked((__int128)r.b, u.sh_bias, b);
  if (ep.scale) {
    if (bits128(t) > 90) b = true;
    else t *= (__int128)r.sc;
  }
  t = shl_checked(t, u.sh_mid, b);
  if (ep.shift) t += shl_checked((__int128)r.sh, u.sh_shift, b);
  if (ep.ep_relu && t < 0) t = 0;
  b |= bits128(t) > 62;
  bad |= b;
  return b ? 0 : (int64_t)t;
}

__device__ inline int64_t wide_epi(int64_t a, const EpiRaw& r, const EpiU& u, const SrcDev& ep,
                                   bool& bad) {
  bool b = false;
  int64_t t = shl62(a, u.sh_acc, b);
  if (ep.bias) t += shl62((int64_t)r.b, u.sh_bias, b);
  if (ep.scale) {
    if (bits64(t) + 32 > 62) {
      int64_t m;
      b |= __builtin_mul_overflow(t, (int64_t)r.sc, &m);
      t = m;
    } else {
      t *= (int64_t)r.sc;
    }
  }
  t = shl62(t, u.sh_mid, b);
  if (ep.shift) t += shl62((int64_t)r.sh, u.sh_shift, b);
  if (ep.ep_relu && t < 0) t = 0;
  b |= bits64(t) > 62;
  bad |= b;
  return b ? 0 : t;
}

// The epilogue of N contraction values of one channel: store(e, value) for
// each, true where the value exists.  int64: one bound per value, in fp64,
// shows for the whole wave that no step leaves 2^62 (the steps' own checks are
// three quarters of their instructions: 64 x 224 x 224 padded RGB 7x7 at 16 bits,
// the whole C-Block, 737 -> 626 us); else, and in 128 bits, checked step by step.
template <int N, typename F>
__device__ __forceinline__ void wide_store(int64_t (&t)[N], const EpiRaw& r, const EpiU& u,
                                           const SrcDev& ep, bool& bad, F store) {
  constexpr double kRoom = 0x1p61;
  const double pa = ldexp(1.0, u.sh_acc), mid = ldexp(1.0, u.sh_mid);
  const double B = ep.bias ? ldexp(fabs((double)r.b), u.sh_bias) : 0.0;
  const double S = ep.shift ? ldexp(fabs((double)r.sh), u.sh_shift) : 0.0;
  const double sc = ep.scale ? fabs((double)r.sc) * mid : mid;
  bool ok = B < kRoom && S < kRoom && imax(imax(u.sh_acc, u.sh_bias), imax(u.sh_mid, u.sh_shift)) < 62;
#pragma unroll
  for (int e = 0; e < N; ++e) {
    const double A = fabs((double)t[e]) * pa;
    ok = ok && A < kRoom && (A + B) * sc < kRoom;
  }
  if (__all(ok)) {
    const int64_t b = ep.bias ? (int64_t)r.b * ((int64_t)1 << u.sh_bias) : 0;
    const int64_t sh = ep.shift ? (int64_t)r.sh * ((int64_t)1 << u.sh_shift) : 0;
#pragma unroll
    for (int e = 0; e < N; ++e) {
      int64_t x = t[e] * ((int64_t)1 << u.sh_acc) + b;
      if (ep.scale) x *= (int64_t)r.sc;
      x = x * ((int64_t)1 << u.sh_mid) + sh;
      if (ep.ep_relu) x = x > 0 ? x : 0;
      store(e, x);
    }
    return;
  }
  // rolled: the values move down by one each time
#pragma nounroll
  for (int e = 0; e < N; ++e) {
    bool b = false;
    const int64_t x = wide_epi(t[0], r, u, ep, b);
    if (store(e, x)) bad |= b;
#pragma unroll
    for (int i = 0; i + 1 < N; ++i) t[i] = t[i + 1];
  }
}
template <int N, typename F>
__device__ __forceinline__ void wide_store(__int128 (&t)[N], const EpiRaw& r, const EpiU& u,
                                           const SrcDev& ep, bool& bad, F store) {
#pragma unroll
  for (int e = 0; e < N; ++e) {
    bool b = false;
    const int64_t x = wide_epi(t[e], r, u, ep, b);
    if (store(e, x)) bad |= b;
  }
}

// WIDE: the plane sums may exceed 2^62 (combined in 128 bits); otherwise the
// host has shown |sum| < 2^62 and the whole value stays in int64.
template <bool WIDE>
__global__ __launch_bounds__(kThreads) void k_wide_combine(const int32_t* __restrict__ acc,
                                                           int64_t mk, int np_x, int np_w,
                                                           SrcDev ep, int64_t* __restrict__ v,
                                                           int32_t* d_scale, unsigned* flags) {
  const EpiU u = epi_uniform(ep);
  if (blockIdx.x == 0 && threadIdx.x == 0) *d_scale = u.s_out;
  const int K = ep.channels;
  const int64_t step = (int64_t)gridDim.x * kThreads;
  const int cstep = (int)(step % K);
  int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x;
  int c = (int)(i % K);
  bool bad = false;
  for (; i < mk; i += step) {
    const EpiRaw r = epi_channel_load(ep, c);
    using Acc = typename std::conditional<WIDE, __int128, int64_t>::type;
    Acc a = 0;
    for (int p = 0; p < np_x; ++p)
      for (int q = 0; q < np_w; ++q)
        a += (Acc)acc[(int64_t)(p * np_w + q) * mk + i] * ((Acc)1 << (8 * (p + q)));
    v[i] = wide_epi(a, r, u, ep, bad);
    c += cstep;
    if (c >= K) c -= K;
  }
  if (bad) flag(flags, FXPQ_FLAG_RANGE);
}

// ---------------------------------------------------------------------------
// One contraction for the whole wide C-Block.  The plane pairs (p, q) are
// walked by shift g = p + q; the pairs of one shift accumulate in the same
// int32 matrix-core accumulators (a pair's sum is at most depth * 2^14 in
// magnitude, the host bounds the group), which then fold into an exact wide
// register accumulator W += (acc + corr_g) * 256^g, corr_g adding back
// 128 * (the weight plane's column sum) for every input plane stored as
// byte - 128.  The epilogue runs on W in the same kernel: no per-pair
// tensors and no combine pass.
//
// Tiles of 32 x 32 where 128 x 64 ones leave CUs idle: the sequence of slabs (64 bytes of depth of one pair)
// is split over the block's four waves, each with its own LDS stages and no
// barriers, and the waves' W are added through LDS at the end.  The walk over
// a pair's depth is incremental.  (128 x 64 tiles with barriers and the
// addresses of every slab from its number spent their time there: the whole
// C-Block 30 x 20 x 3168 at 16 bits 326 -> 51 us, 4536 x 128 x 144 77 -> 42, 4 x 46
// x 46 padded RGB 7x7 76 -> 34.)
// ---------------------------------------------------------------------------

// Walk over the plane pairs in shift order.
struct PairWalk {
  int g, p;
  __device__ inline void start() { g = p = 0; }
  __device__ inline void next(const WideFusedArgs& a) {
    if (p < min(g, a.np_x - 1)) {
      ++p;
    } else {
      ++g;
      p = max(g - a.np_w + 1, 0);
    }
  }
  __device__ inline int q() const { return g - p; }
  // input planes stored as byte - 128
  __device__ inline bool off(const WideFusedArgs& a) const { return p < a.np_x - 1 || !a.sign_x; }
};

// The geometry and walk of the first plane pair for the 8-bit loaders.
__device__ inline ConvArgs conv_args(const WideFusedArgs& a) {
  ConvArgs c{};
  c.x = a.px; c.w = a.pw;
  c.H = a.H; c.W = a.W; c.C = a.C; c.K = a.K; c.R = a.R; c.S = a.S;
  c.stride = a.stride; c.pad = a.pad; c.Ho = a.Ho; c.Wo = a.Wo; c.M = a.M;
  c.kdepth = a.kdepth; c.wrow = a.wrow;
  c.gen_r = a.gen_r; c.gen_s = a.gen_s; c.gen_c = a.gen_c; c.gen_step = a.gen_step;
  c.rgb_chunks = a.chunks;
  c.rgb_step_r = a.chunks ? 4 / a.chunks : 0;
  c.rgb_step_c = a.chunks ? 4 % a.chunks : 0;
  return c;
}

// A tap of the packed padded RGB filters: its filter row and column, and its
// byte offset from tap (0, 0)'s pixel.  Past the last tap: never inside an image
// (no row or column index, INT_MIN / 2 for a missing row among them, plus
// INT_MIN / 2 is one of an image that has as many rows and columns).
struct alignas(16) RgbTap {
  int r, s;
  int64_t off;
};

// Slabs of C % 16 == 0 inputs: the ring of the 8-bit contraction, moved from
// plane pair to plane pair.
struct WideRing {
  static constexpr int D = kSplitD, ST = kSplitStage<1>, SA = 32 * 64;
  using Ring = RingLoad<32, 32, 1, true>;
  static constexpr int OPS = Ring::kOps, MFMAS = 2, PER = (OPS + MFMAS - 1) / MFMAS;
  Ring ld;
  ConvArgs ca;
  PairWalk at;
  int left;  // slabs not yet sent
  int8_t *ring, *cur;

  __device__ inline void pair(const WideFusedArgs& a, int p0, int q0) {
#pragma unroll
    for (int j = 0; j < Ring::AJ; ++j) ld.arow[j] += (at.p - p0) * a.xs;
#pragma unroll
    for (int j = 0; j < Ring::BJ; ++j) ld.bsrc[j] += (at.q() - q0) * a.ws;
    ld.padp = (int64_t)(uintptr_t)&kPadVec[at.off(a) ? 1 : 0];
  }
  __device__ inline void advance(const WideFusedArgs& a) {
    --left;
    if (ld.advance(ca) && left > 0) {
      const int p0 = at.p, q0 = at.q();
      at.next(a);
      pair(a, p0, q0);
    }
  }
  __device__ inline void start(const WideFusedArgs& a, const PairWalk& first, int kt, int n, int m0,
                               int n0, int lane, int8_t* lds, const RgbTap*) {
    ca = conv_args(a);
    at = first;
    left = n;
    ring = cur = lds;
    ld.cols(ca, 0, n0, 0, lane);
    ld.rows(ca, m0, 0, lane);
    pair(a, 0, 0);
    ld.seek(ca, kt);
    for (int i = 0; i < D && i < n; ++i) {
#pragma unroll
      for (int k = 0; k < OPS; ++k) ld.load(ca, k, ring + i * ST, ring + i * ST + SA, 0);
      advance(a);
    }
  }
  // The next slab's MFMAs; `follow` slabs come after it.
  __device__ inline void slab(const WideFusedArgs& a, int lane, int follow, v16i (&acc)[1][1]) {
    if (follow >= D) {
      wait_vmcnt<OPS*(D - 1)>();
      asm volatile("" ::: "memory");
      int8_t* st = cur == ring ? ring + D * ST : cur - ST;
      slab_mfma<1, 1>(cur, cur + SA, 0, 0, lane, acc, [&](int i) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < PER; ++k)
          if (i * PER + k < OPS) ld.load(ca, i * PER + k, st, st + SA, 0);
        __builtin_amdgcn_sched_barrier(0);
      });
      advance(a);
    } else {
      if (follow > 0) wait_vmcnt<OPS>();
      else wait_vmcnt<0>();
      asm volatile("" ::: "memory");
      slab_mfma<1, 1>(cur, cur + SA, 0, 0, lane, acc);
    }
    cur = cur == ring + D * ST ? ring : cur + ST;
  }
};

// Slabs of padded RGB inputs (C == 4): a 16-byte chunk is four taps, gathered
// as dwords through a table of the taps' rows, columns and offsets, staged
// through registers one slab ahead.
struct WideRgb {
  static constexpr int ST = kSplitStage<1>, SA = 32 * 64, PC = 2;  // 16-row pieces
  PairWalk at;
  int kt, ktiles, left, taps;
  const int8_t *xb[PC], *wb[PC];
  int ih0[PC], iw0[PC];
  v4i ra[PC], rb[PC];
  int8_t* ring;
  const RgbTap* tab;
  int st;

  __device__ inline void gload(const WideFusedArgs& a, int lane) {
    const int kc = lane & 3, padw = at.off(a) ? (int)0x80808080 : 0;
    const int64_t px = at.p * a.xs;
    RgbTap tp[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) tp[e] = tab[kt * 16 + kc * 4 + e];
#pragma unroll
    for (int i = 0; i < PC; ++i) {
      bool ok[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        ok[e] = (unsigned)(ih0[i] + tp[e].r) < (unsigned)a.H &&
                (unsigned)(iw0[i] + tp[e].s) < (unsigned)a.W;
        // (a readable address where the tap is outside: loads without branches)
        const int8_t* ad = xb[i] + px + tp[e].off;
        ra[i][e] = *reinterpret_cast<const int*>(ok[e] ? ad : a.px);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) ra[i][e] = ok[e] ? ra[i][e] : padw;
      rb[i] = *reinterpret_cast<const v4i*>(wb[i] + at.q() * a.ws + kt * 64);
    }
    if (++kt == ktiles) {
      kt = 0;
      if (--left > 0) at.next(a);
    } else {
      --left;
    }
  }
  __device__ inline void lstore(int lane) {
    int8_t* sa = ring + st * ST;
#pragma unroll
    for (int i = 0; i < PC; ++i) {
      *reinterpret_cast<v4i*>(&sa[lds_off(16 * i + (lane >> 2), lane & 3)]) = ra[i];
      *reinterpret_cast<v4i*>(&sa[SA + lds_off(16 * i + (lane >> 2), lane & 3)]) = rb[i];
    }
  }
  __device__ inline void start(const WideFusedArgs& a, const PairWalk& first, int kt0, int n, int m0,
                               int n0, int lane, int8_t* lds, const RgbTap* table) {
    at = first;
    kt = kt0;
    ktiles = a.wrow / 64;
    left = n;
    ring = lds;
    tab = table;
    st = 0;
    const int hw_out = a.Ho * a.Wo;
#pragma unroll
    for (int i = 0; i < PC; ++i) {
      const int row = m0 + 16 * i + (lane >> 2);
      const int rr = row < a.M ? row : a.M - 1;
      const int im = rr / hw_out, rem = rr - im * hw_out;
      const int oh = rem / a.Wo, ow = rem - oh * a.Wo;
      ih0[i] = row < a.M ? oh * a.stride - a.pad : INT_MIN / 2;
      iw0[i] = ow * a.stride - a.pad;
      xb[i] = a.px + (((int64_t)im * a.H + (oh * a.stride - a.pad)) * a.W + iw0[i]) * 4;
      const int col = n0 + 16 * i + (lane >> 2);
      wb[i] = a.pw + (int64_t)(col < a.K ? col : a.K - 1) * a.wrow + (lane & 3) * 16;
    }
    if (n > 0) {
      gload(a, lane);
      lstore(lane);
    }
  }
  __device__ inline void slab(const WideFusedArgs& a, int lane, int follow, v16i (&acc)[1][1]) {
    if (follow > 0) gload(a, lane);
    slab_mfma<1, 1>(ring + st * ST, ring + st * ST + SA, 0, 0, lane, acc);
    st ^= 1;
    if (follow > 0) lstore(lane);
  }
};

template <bool WIDE, bool RGB>
__global__ __launch_bounds__(kThreads) void k_wide_split(WideFusedArgs a) {
  using Acc = typename std::conditional<WIDE, __int128, int64_t>::type;
  using Load = typename std::conditional<RGB, WideRgb, WideRing>::type;
  constexpr int STAGES = RGB ? 2 : kSplitD + 1;
  __shared__ __attribute__((aligned(16))) int8_t lds[4 * STAGES * kSplitStage<1>];
  __shared__ RgbTap tab[RGB ? 128 : 1];  // at most 128 taps
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m0 = blockIdx.x * 32, n0 = blockIdx.y * 32;
  const int ktiles = (a.wrow + 63) / 64;
  if constexpr (RGB) {
    for (int i = tid; i < ktiles * 16; i += kThreads) {
      const int r = i / a.S, s = i - r * a.S;
      tab[i] = i < a.R * a.S ? RgbTap{r, s, ((int64_t)r * a.W + s) * 4} : RgbTap{INT_MIN / 2, INT_MIN / 2, 0};
    }
    __syncthreads();
  }
  const int total = a.np_x * a.np_w * ktiles;
  const int s0 = (int)((int64_t)total * wave / 4), n = (int)((int64_t)total * (wave + 1) / 4) - s0;
  PairWalk at;
  at.start();
  for (int j = s0 / ktiles; j > 0; --j) at.next(a);
  int kt = s0 % ktiles;
  Load ld;
  ld.start(a, at, kt, n, m0, n0, lane, lds + wave * STAGES * kSplitStage<1>, tab);
  const EpiU u = epi_uniform(a.ep);
  if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) *a.d_scale = u.s_out;

  v16i acc[1][1];
  Acc W[16];
  int corr = 0;
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    acc[0][0][e] = 0;
    W[e] = 0;
  }
  const int col = n0 + (lane & 31), cc = col < a.K ? col : a.K - 1;
  // the accumulators of shift g into W
  auto fold = [&](int g) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      W[e] += ((Acc)acc[0][0][e] + (Acc)corr) * ((Acc)1 << (8 * g));
      acc[0][0][e] = 0;
    }
    corr = 0;
  };
  for (int s = 0; s < n; ++s) {
    if (kt == 0 && at.off(a)) {
      // byte - 128 storage: 128 * colsum of this weight plane per column, by
      // the wave that has the pair's first slab
      corr += 128 * a.cs[(int64_t)at.q() * a.K + cc];
    }
    ld.slab(a, lane, n - 1 - s, acc);
    if (++kt == ktiles) {
      kt = 0;
      const int g = at.g;
      at.next(a);
      if (at.g != g) fold(g);
    }
  }
  fold(at.g);  // (nothing left when the last slab ended its shift)

  // the waves' sums, accumulators 4 w .. 4 w + 3 to wave w, two at a time
  constexpr int MINE = 4, RED = 2;
  static_assert(4 * 4 * RED * 64 * 8 <= sizeof(lds), "exchange fits the stages");
  unsigned long long* red = reinterpret_cast<unsigned long long*>(lds);
  Acc mine[MINE];
#pragma unroll
  for (int part = 0; part < MINE / RED; ++part) {
#pragma unroll
    for (int half = 0; half < (WIDE ? 2 : 1); ++half) {
      __syncthreads();
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int e = 0; e < RED; ++e) {
          const Acc v = W[4 * t + part * RED + e];
          red[((wave * 4 + t) * RED + e) * 64 + lane] = (unsigned long long)(half ? v >> (WIDE ? 64 : 0) : v);
        }
      __syncthreads();
#pragma unroll
      for (int e = 0; e < RED; ++e) {
        Acc sum = half ? mine[part * RED + e] : (Acc)0;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const unsigned long long v = red[((w * 4 + wave) * RED + e) * 64 + lane];
          if constexpr (WIDE) sum += half ? (Acc)v << 64 : (Acc)(unsigned __int128)v;
          else sum += (Acc)v;
        }
        mine[part * RED + e] = sum;
      }
    }
  }
  // epilogue
  bool bad = false;
  const EpiRaw r = epi_channel_load(a.ep, cc);
  wide_store(mine, r, u, a.ep, bad, [&](int e, int64_t x) __attribute__((always_inline)) -> bool {
    const int row = m0 + 8 * wave + 4 * (lane >> 5) + e;
    const bool in = row < a.M && col < a.K;
    if (in) a.v[(int64_t)row * a.K + col] = x;
    return in;
  });
  if (bad) flag(a.flags, FXPQ_FLAG_RANGE);
}

// Grids that fill the chip: tiles of 128 x 64 shared by the block's waves (32
// rows each; 64 x 64, 32 x 32 each, for 128-bit sums: twice the columns held 128
// registers of sums and spilled as many), slabs through the LDS ring or, padded RGB with filter rows of
// whole 16-byte chunks, staged through registers four pixels at a time.  Two
// blocks per CU hide each other's waits (64 x 64 split tiles hold 128 registers
// of int64 sums per thread, one block: 64 x 224 x 224 padded RGB, the whole
// C-Block, 1398 us; pixel by pixel with the addresses from the slab's number
// 976; this 737).
template <bool WIDE, bool RGB>
__global__ __launch_bounds__(kThreads, 2) void k_wide_tile(WideFusedArgs a) {
  using Acc = typename std::conditional<WIDE, __int128, int64_t>::type;
  constexpr int BM = WIDE ? 64 : 128, BN = 64, TN = WIDE ? 1 : 2;
  constexpr int SA = BM * 64, ST = (BM + BN) * 64;
  using Load = typename std::conditional<RGB, StagedLoad<BM, BN, LD_RGB8>, RingLoad<BM, BN, 4, true>>::type;
  constexpr int D = kSplitD, STAGES = RGB ? 2 : D + 1;
  __shared__ __attribute__((aligned(16))) int8_t stage[STAGES * ST];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m0 = blockIdx.x * BM, n0 = blockIdx.y * BN;
  const int row0 = (WIDE ? wave >> 1 : wave) * 32, col0 = WIDE ? (wave & 1) * 32 : 0;  // of the wave
  const int ktiles = (a.wrow + 63) / 64;
  const int total = a.np_x * a.np_w * ktiles;
  const ConvArgs ca = conv_args(a);
  PairWalk at, in;  // pair of the slab computed, of the slab loaded
  at.start();
  in.start();
  Load ld;
  int sent = 0;  // slabs loaded
  auto next_pair = [&]() __attribute__((always_inline)) {
    const int p0 = in.p, q0 = in.q();
    in.next(a);
    const int64_t dx = (in.p - p0) * a.xs, dw = (in.q() - q0) * a.ws;
    if constexpr (RGB) {
#pragma unroll
      for (int i = 0; i < Load::ACH; ++i) ld.abase[i] += dx;
#pragma unroll
      for (int i = 0; i < Load::BCH; ++i) ld.bptr[i] += dw;
      ld.restart(ca, tid);
    } else {
#pragma unroll
      for (int j = 0; j < Load::AJ; ++j) ld.arow[j] += dx;
#pragma unroll
      for (int j = 0; j < Load::BJ; ++j) ld.bsrc[j] += dw;
      ld.padp = (int64_t)(uintptr_t)&kPadVec[in.off(a) ? 1 : 0];
    }
  };
  v16i acc[1][TN];
  Acc W[TN][16];
  int corr[TN];
#pragma unroll
  for (int ni = 0; ni < TN; ++ni) {
    corr[ni] = 0;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      acc[0][ni][e] = 0;
      W[ni][e] = 0;
    }
  }
  int kt = 0;
  // before and after a slab's MFMAs
  auto begin_slab = [&]() __attribute__((always_inline)) {
    if (kt == 0 && at.off(a)) {
#pragma unroll
      for (int ni = 0; ni < TN; ++ni) {
        const int col = n0 + col0 + ni * 32 + (lane & 31);
        corr[ni] += 128 * a.cs[(int64_t)at.q() * a.K + (col < a.K ? col : a.K - 1)];
      }
    }
  };
  auto end_slab = [&]() __attribute__((always_inline)) {
    if (++kt < ktiles) return;
    kt = 0;
    const int g = at.g;
    at.next(a);
    if (at.g == g) return;
#pragma unroll
    for (int ni = 0; ni < TN; ++ni) {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        W[ni][e] += ((Acc)acc[0][ni][e] + corr[ni]) * ((Acc)1 << (8 * g));
        acc[0][ni][e] = 0;
      }
      corr[ni] = 0;
    }
  };
  if constexpr (RGB) {
    ld.cols(ca, n0, tid);
    ld.rows(ca, m0, tid);
    int padw = 0;  // of the slab in the registers
    auto load = [&]() __attribute__((always_inline)) {
      padw = in.off(a) ? (int)0x80808080 : 0;
      if (ld.gload(ca, ktiles, tid, 0, nullptr) && ++sent < a.np_x * a.np_w) next_pair();
    };
    load();
    ld.lstore(stage, stage + SA, tid, padw);
    __syncthreads();
    for (int s = 0; s < total; ++s) {
      int8_t *cur = stage + (s & 1) * ST, *next = stage + ((s & 1) ^ 1) * ST;
      begin_slab();
      if (s + 1 < total) load();
      slab_mfma<1, TN>(cur, cur + SA, row0, col0, lane, acc);
      if (s + 1 < total) ld.lstore(next, next + SA, tid, padw);
      __syncthreads();
      end_slab();
    }
  } else {
    constexpr int OPS = Load::kOps;
    static_assert(OPS <= 2 * TN, "every load comes before an MFMA of the slab");
    ld.cols(ca, 0, n0, wave, lane);
    ld.rows(ca, m0, wave, lane);
    ld.padp = (int64_t)(uintptr_t)&kPadVec[in.off(a) ? 1 : 0];
    auto advance = [&]() __attribute__((always_inline)) {
      ++sent;
      if (ld.advance(ca) && sent < total) next_pair();
    };
    for (int i = 0; i < D && i < total; ++i) {
#pragma unroll
      for (int k = 0; k < OPS; ++k) ld.load(ca, k, stage + i * ST, stage + i * ST + SA, wave);
      advance();
    }
    int8_t* cur = stage;
    for (int s = 0; s < total; ++s) {
      begin_slab();
      // (loads of the column sums only make the waits longer)
      if (s + D - 1 < total) wait_vmcnt<OPS*(D - 1)>();
      else wait_vmcnt<0>();
      ring_barrier();
      int8_t* st = cur == stage ? stage + D * ST : cur - ST;
      const bool more = s + D < total;
      slab_mfma<1, TN>(cur, cur + SA, row0, col0, lane, acc, [&](int i) __attribute__((always_inline)) {
        if (more && i < OPS) ld.load(ca, i, st, st + SA, wave);
        __builtin_amdgcn_sched_barrier(0);
      });
      if (more) advance();
      cur = cur == stage + D * ST ? stage : cur + ST;
      end_slab();
    }
  }
  const EpiU u = epi_uniform(a.ep);
  if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) *a.d_scale = u.s_out;
  bool bad = false;
#pragma unroll
  for (int ni = 0; ni < TN; ++ni) {
    const int col = n0 + col0 + ni * 32 + (lane & 31);
    const EpiRaw r = epi_channel_load(a.ep, col < a.K ? col : a.K - 1);
    wide_store(W[ni], r, u, a.ep, bad, [&](int e, int64_t x) __attribute__((always_inline)) -> bool {
      const int row = m0 + row0 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
      const bool in = row < a.M && col < a.K;
      if (in) a.v[(int64_t)row * a.K + col] = x;
      return in;
    });
  }
  if (bad) flag(a.flags, FXPQ_FLAG_RANGE);
}

// Accumulators outside [-2^(bits-1), 2^(bits-1) - 1]: one atomic add per block.
__global__ __launch_bounds__(kThreads) void k_acc_overflow(const int32_t* __restrict__ acc,
                                                           int64_t n, int bits,
                                                           unsigned long long* count) {
  __shared__ unsigned long long part[kThreads / 64];
  const int64_t lo = -((int64_t)1 << (bits - 1)), hi = ((int64_t)1 << (bits - 1)) - 1;
  unsigned long long c = 0;
  for (int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kThreads) {
    const int64_t a = acc[i];
    c += (a < lo || a > hi) ? 1 : 0;
  }
  for (int off = 32; off > 0; off >>= 1) c += __shfl_down(c, off, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long t = 0;
    for (int w = 0; w < kThreads / 64; ++w) t += part[w];
    if (t) atomicAdd(count, t);
  }
}

int stream_blocks(int64_t n) {
  int64_t b = (n + kThreads - 1) / kThreads;
  return (int)(b < 4096 ? (b < 1 ? 1 : b) : 4096);
}

}  // namespace

hipError_t launch_wide_split(const Ctx& c, const int32_t* x, int64_t nx, int np_x, int sign_x,
                             int64_t xs, int8_t* px, const int32_t* w, int64_t wrow, int K,
                             int np_w, int sign_w, int64_t ws, int8_t* pw, int R, int S,
                             int chunks, int32_t* cs) {
  k_split<<<K + stream_blocks((nx + 3) / 4), kThreads, 0, c.stream>>>(
      x, nx, np_x, sign_x, xs, px, w, wrow, K, np_w, sign_w, ws, pw, R, S, chunks, cs, c.sc.flags);
  return hipGetLastError();
}

hipError_t launch_acc_overflow(const Ctx& c, const int32_t* acc, int64_t n, int bits,
                               int64_t* count) {
  k_acc_overflow<<<stream_blocks(n), kThreads, 0, c.stream>>>(
      acc, n, bits, reinterpret_cast<unsigned long long*>(count));
  return hipGetLastError();
}

// Fused contraction's variant: 32 x 32 split tiles up to eight per CU (fewer
// 128 x 64 tiles than CUs: 4536 x 128 x 144, 568 split tiles, 44 us against 57 in
// 72 tiles; 10 x 207 x 207 padded RGB, 6500 split tiles, 182 against 115 in 813),
// and for padded RGB whose filter rows do not fit the packed rows as whole
// chunks; else 128 x 64 tiles.  128-bit sums: split tiles, but 64 x 64 ones for
// grids above 24 split tiles per CU with at most 16 slabs (the split tiles'
// exchange of sums, 16 barriers, outweighs the contraction) and full column
// tiles.  24 / 32 by 16 / 24 bits (9 / 16 slabs), us, split -> 64 x 64: 802816 x 64
// x 16 711 -> 555, 837 -> 734; 200704 x 128 x 48 360 -> 289, 428 -> 384; but 50176
// x 64 x 16 (3136 split tiles) 57 -> 54, 67 -> 71, 802816 x 16 x 64 408 -> 589, and
// 12544 x 512 x 256 (36 slabs) 126 -> 132.
static bool wide_split_tiles(const Ctx& c, const WideFusedArgs& a, bool wide) {
  const int64_t ct = (a.K + 31) / 32, tiles = (int64_t)((a.M + 31) / 32) * ct;
  if (!wide) return tiles <= 8 * c.cus;
  return tiles <= 24 * c.cus || a.np_x * a.np_w * ((a.wrow + 63) / 64) > 16 || ct % 2 != 0;
}

int wide_chunks(const Ctx& c, const WideFusedArgs& a, bool wide) {
  const int chunks = (a.S + 3) / 4;
  // (LD_RGB8's pixel indices within an image are 32-bit)
  if (a.C != 4 || a.W < 4 || (int64_t)a.H * a.W > INT_MAX || wide_split_tiles(c, a, wide) ||
      a.R * chunks * 16 > a.wrow)
    return 0;
  return chunks;
}

hipError_t launch_wide_fused(const Ctx& c, const WideFusedArgs& args, bool wide) {
  WideFusedArgs a = args;
  const bool rgb = a.C == 4;
  if (!rgb) {  // 64 channels as filter rows, taps and channels
    a.gen_r = BK / a.C / a.S;
    a.gen_s = BK / a.C % a.S;
    a.gen_c = BK % a.C;
    a.gen_step = ((int64_t)a.gen_r * a.W + a.gen_s) * a.C + a.gen_c;
  }
  if (wide_split_tiles(c, a, wide) || (rgb && !a.chunks)) {
    const dim3 grid((unsigned)((a.M + 31) / 32), (unsigned)((a.K + 31) / 32));
    if (wide && rgb) k_wide_split<true, true><<<grid, kThreads, 0, c.stream>>>(a);
    else if (wide) k_wide_split<true, false><<<grid, kThreads, 0, c.stream>>>(a);
    else if (rgb) k_wide_split<false, true><<<grid, kThreads, 0, c.stream>>>(a);
    else k_wide_split<false, false><<<grid, kThreads, 0, c.stream>>>(a);
  } else {
    const int bm = wide ? 64 : 128;
    const dim3 grid((unsigned)((a.M + bm - 1) / bm), (unsigned)((a.K + 63) / 64));
    if (wide && rgb) k_wide_tile<true, true><<<grid, kThreads, 0, c.stream>>>(a);
    else if (wide) k_wide_tile<true, false><<<grid, kThreads, 0, c.stream>>>(a);
    else if (rgb) k_wide_tile<false, true><<<grid, kThreads, 0, c.stream>>>(a);
    else k_wide_tile<false, false><<<grid, kThreads, 0, c.stream>>>(a);
  }
  return hipGetLastError();
}

hipError_t launch_wide_combine(const Ctx& c, const int32_t* acc, int64_t mk, int np_x, int np_w,
                               const SrcDev& ep, int64_t* v, int32_t* d_scale) {
  // |sum_{p,q} acc_pq 256^(p+q)| < pairs * 2^31 * 256^(np_x + np_w - 2): int64 when below 2^62
  const int pairs = np_x * np_w;
  const int lg = pairs <= 1 ? 0 : 32 - __builtin_clz((unsigned)(pairs - 1));  // ceil(log2 pairs)
  const bool wide = 31 + 8 * (np_x + np_w - 2) + lg >= 62;
  if (wide)
    k_wide_combine<true><<<stream_blocks(mk), kThreads, 0, c.stream>>>(acc, mk, np_x, np_w, ep, v,
                                                                       d_scale, c.sc.flags);
  else
    k_wide_combine<false><<<stream_blocks(mk), kThreads, 0, c.stream>>>(acc, mk, np_x, np_w, ep,
                                                                        v, d_scale, c.sc.flags);
  return hipGetLastError();
}

}  // namespace fxpq
