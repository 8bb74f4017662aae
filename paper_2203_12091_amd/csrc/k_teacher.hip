// FP32 teacher: the full-precision network whose activations are the
// reference of the layer error in the per-layer sensitivity sweep (Sec.
// "Data-Structures Sensitivity to Quantization"; the full-precision model as
// teacher, Sec. "Quantization Parameters Optimization").  Its arithmetic is
// fixed so that any implementation gets the same bits:
//   conv / FC   fp64 sum of the fp32 x fp32 products (exact in fp64) in the
//               order r, s, c with padded taps skipped, rounded once to fp32;
//   BN-as-Scale one fp32 fma per value; bias one fp32 add;
//   ReLU        every value <= 0 becomes +0;
//   residual    one fp32 add, then ReLU;
//   max-pool    the largest in-range tap;
//   avg-pool    (float)(fp64 sum in pixel order / pixels).
// Reference data only: computed once per sweep, outside its timing.
#include <limits.h>
#include <math.h>

#include "common.hpp"

namespace fxpq {

// x NHWC fp32, w RSCK fp32 (output channels contiguous), y NHWK fp32.  Every
// output is one fp64 fma chain over k = (r, s, c) in the defined order, so the
// work splits over outputs only.  v_mfma_f64_16x16x4 adds its four products
// one after the other, in ascending k, each with its own rounding (compared
// with the fma chain over 3 M random outputs of wide exponent range: the same
// bits), so the chain runs on the matrix cores: a wave computes (16 T)^2
// outputs, a block 2 x 2 waves, slabs of KT consecutive k staged in LDS (the
// next slab's loads in flight meanwhile).  A padded tap (and k past the end) is
// staged as the pixel value 0: 0 * w leaves the chain as it is for finite w
// (it starts at +0 and never becomes -0).  Once a slab holds an infinite or NaN
// weight, the tile goes on with scalar fmas that skip padded taps.
// Bound by the fp64 matrix cores: 149 clocks per instruction and wave measured
// in a bare loop, 33 TFLOP/s with one wave per SIMD and 37 to 47 with four;
// vector fmas reach 62 bare, but 8 x 4 outputs per thread, whose operands the
// LDS has to feed, ran at 20.  Measured at 32 images (one output per thread ->
// now): 3x3 128 -> 128 at 28x28 1122 -> 216 us, 3x3 64 -> 64 at 56x56 1189 ->
// 205 us, 3x3 512 -> 512 at 7x7 1502 -> 260 us, 7x7 RGB 1854 -> 275 us.
typedef double v4d __attribute__((ext_vector_type(4)));

template <int T, int KT, bool VEC>
__global__ __launch_bounds__(256, 4) void k_teacher_conv(const float* __restrict__ x,
                                                         const float* __restrict__ w,
                                                         float* __restrict__ y, int N, int H,
                                                         int W, int C, int K, int R, int S,
                                                         int stride, int pad, int Ho, int Wo) {
  constexpr int BM = 32 * T, BN = 32 * T;
  // Slabs are staged as doubles, four values per thread and operand.  A row
  // holds, per 8 k, the operands of two steps side by side: k at 8 (k / 8) +
  // 2 (k % 4) + (k % 8) / 4, and is padded by two doubles: sixteen rows' 16
  // bytes on distinct banks.
  constexpr int RS = KT + 2;
  auto pos = [](int k) { return (k & ~7) + 2 * (k & 3) + ((k & 7) >> 2); };
  static_assert(BM * KT == 1024, "four values per thread and slab");
  __shared__ __attribute__((aligned(16))) double As[2][BM * RS];
  __shared__ __attribute__((aligned(16))) double Bs[2][BN * RS];
  // per pixel of the tile: (row, column) of tap (0, 0) and its element offset
  __shared__ __attribute__((aligned(16))) int4 geo[BM];
  __shared__ int nonfinite;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wrow = (wave >> 1) * 16 * T, wcol = (wave & 1) * 16 * T;
  const int64_t M = (int64_t)N * Ho * Wo;
  const int64_t depth = (int64_t)R * S * C;
  const int64_t ntn = (K + BN - 1) / BN, tiles = ((M + BM - 1) / BM) * ntn;
  // this thread stages k = ak .. ak + 3 of pixel ap, channels bn .. bn + 3 of k = bk
  const int ak = tid % (KT / 4) * 4, ap = tid / (KT / 4);
  const int bk = tid / (BN / 4), bn = tid % (BN / 4) * 4;
  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int64_t m0 = tile / ntn * BM;
    const int n0 = (int)(tile % ntn) * BN;
    __syncthreads();  // the previous tile's last slab is read
    if (tid == 0) nonfinite = 0;
    if (tid < BM) {
      const int64_t m = m0 + tid < M ? m0 + tid : M - 1;
      const int64_t n = m / ((int64_t)Ho * Wo);
      const int rem = (int)(m - n * Ho * Wo);
      const int ih = rem / Wo * stride - pad, iw = rem % Wo * stride - pad;
      const int64_t at = ((n * H + ih) * W + iw) * C;
      // no pixel: outside for every tap
      geo[tid] = make_int4(m0 + tid < M ? ih : INT_MIN / 2, iw, (int)(unsigned)at, (int)(at >> 32));
    }
    const float* pw = w + (int64_t)bk * K + n0 + bn;
    __syncthreads();  // geo is written, nonfinite cleared
    const int4 gp = geo[ap];
    const float* px = x + (int64_t)((uint64_t)(unsigned)gp.w << 32 | (unsigned)gp.z);
    v4d acc[T][T];
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
      for (int j = 0; j < T; ++j) acc[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
    float ra[4], rb[4];
    bool aok[4], bok[4];
    int lr = 0, ls = 0, lc = ak;  // tap and channel of the staged k
    int64_t lk = 0;               // first k of the slab
    auto wrap = [&](int& r, int& s, int& c) {
      while (c >= C) {
        c -= C;
        if (++s == S) s = 0, ++r;
      }
    };
    wrap(lr, ls, lc);
    // Loads are unconditional (from a valid address where there is no value);
    // the zeros go in at the LDS store.  VEC: C and K are multiples of 4 and x
    // and w are 16-byte aligned, so four values share their tap and bounds.
    auto gload = [&]() {
      if constexpr (VEC) {
        const bool a1 = (lk + ak < depth) & ((unsigned)(gp.x + lr) < (unsigned)H) &
                        ((unsigned)(gp.y + ls) < (unsigned)W);
        const bool b1 = (lk + bk < depth) & (n0 + bn < K);
        const float4 av = *reinterpret_cast<const float4*>(a1 ? px + ((int64_t)lr * W + ls) * C + lc : x);
        const float4 bv = *reinterpret_cast<const float4*>(b1 ? pw : w);
        ra[0] = av.x, ra[1] = av.y, ra[2] = av.z, ra[3] = av.w;
        rb[0] = bv.x, rb[1] = bv.y, rb[2] = bv.z, rb[3] = bv.w;
        aok[0] = aok[1] = aok[2] = aok[3] = a1;
        bok[0] = bok[1] = bok[2] = bok[3] = b1;
      } else {
        int r = lr, s = ls, c = lc;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          aok[e] = (lk + ak + e < depth) & ((unsigned)(gp.x + r) < (unsigned)H) &
                   ((unsigned)(gp.y + s) < (unsigned)W);
          ra[e] = *(aok[e] ? px + ((int64_t)r * W + s) * C + c : x);
          bok[e] = (lk + bk < depth) & (n0 + bn + e < K);
          rb[e] = *(bok[e] ? pw + e : w);
          ++c;
          wrap(r, s, c);
        }
      }
      pw += (int64_t)KT * K;
    };
    auto lstore = [&](int st) {
      unsigned big = 0u;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        As[st][ap * RS + pos(ak + e)] = (double)(aok[e] ? ra[e] : 0.0f);
        const float v = bok[e] ? rb[e] : 0.0f;
        const unsigned mag = __float_as_uint(v) & 0x7FFFFFFFu;
        big = big > mag ? big : mag;
        Bs[st][(bn + e) * RS + pos(bk)] = (double)v;
      }
      if (big >= 0x7F800000u) nonfinite = 1;
      // on to the next slab
      lk += KT;
      lc += KT;
      wrap(lr, ls, lc);
    };
    gload();
    lstore(0);
    __syncthreads();
    int st = 0;
    int64_t k0 = 0;
    for (; k0 < depth && !nonfinite; k0 += KT) {
      const bool more = k0 + KT < depth;
      if (more) gload();
      const double* sa = &As[st][(wrow + (lane & 15)) * RS + 2 * (lane >> 4)];
      const double* sb = &Bs[st][(wcol + (lane & 15)) * RS + 2 * (lane >> 4)];
#pragma unroll
      for (int g = 0; g < KT; g += 8) {
        double2 av[T], bv[T];
#pragma unroll
        for (int i = 0; i < T; ++i) {
          av[i] = *reinterpret_cast<const double2*>(sa + i * 16 * RS + g);
          bv[i] = *reinterpret_cast<const double2*>(sb + i * 16 * RS + g);
        }
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int i = 0; i < T; ++i)
#pragma unroll
            for (int j = 0; j < T; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(q ? av[i].y : av[i].x, q ? bv[j].y : bv[j].x,
                                                               acc[i][j], 0, 0, 0);
      }
      st ^= 1;
      if (more) lstore(st);
      __syncthreads();
    }
    for (; k0 < depth; k0 += KT) {  // an infinite or NaN weight was seen
      if (k0 + KT < depth) gload();
#pragma unroll
      for (int i = 0; i < T; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int p = wrow + 16 * i + (lane >> 4) + 4 * v;
          const int ph = geo[p].x, pwc = geo[p].y;
#pragma nounroll
          for (int k = 0; k < KT && k0 + k < depth; ++k) {
            const int tap = (int)((k0 + k) / C), r = tap / S, s = tap - r * S;
            if ((unsigned)(ph + r) >= (unsigned)H || (unsigned)(pwc + s) >= (unsigned)W) continue;
            const double a = As[st][p * RS + pos(k)];
#pragma unroll
            for (int j = 0; j < T; ++j)
              acc[i][j][v] = fma(a, Bs[st][(wcol + 16 * j + (lane & 15)) * RS + pos(k)], acc[i][j][v]);
          }
        }
      st ^= 1;
      if (k0 + KT < depth) lstore(st);
      __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t m = m0 + wrow + 16 * i + (lane >> 4) + 4 * v;
#pragma unroll
        for (int j = 0; j < T; ++j) {
          const int n = n0 + wcol + 16 * j + (lane & 15);
          if (m < M && n < K) y[m * K + n] = (float)acc[i][j][v];
        }
      }
  }
}

// The same chains one output per thread, output channels fastest so a wave reads
// few input pixels and consecutive filters: for outputs whose 32 x 32 tiles would be
// mostly padding (narrow_teacher).  Bound by the loads of the pixels, which
// neighbouring threads share.
__global__ __launch_bounds__(256) void k_teacher_narrow(const float* x, const float* w, float* y,
                                                        int N, int H, int W, int C, int K, int R,
                                                        int S, int stride, int pad, int Ho, int Wo) {
  const int64_t total = (int64_t)N * Ho * Wo * K;
  for (int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; o < total;
       o += (int64_t)gridDim.x * blockDim.x) {
    const int k = (int)(o % K);
    int64_t pix = o / K;
    const int ow = (int)(pix % Wo);
    pix /= Wo;
    const int oh = (int)(pix % Ho);
    const int n = (int)(pix / Ho);
    double acc = 0.0;
    for (int r = 0; r < R; ++r) {
      const int ih = oh * stride - pad + r;
      if (ih < 0 || ih >= H) continue;
      for (int s = 0; s < S; ++s) {
        const int iw = ow * stride - pad + s;
        if (iw < 0 || iw >= W) continue;
        const float* xp = x + (((int64_t)n * H + ih) * W + iw) * C;
        const float* wp = w + ((int64_t)(r * S + s) * C) * K + k;
        for (int c = 0; c < C; ++c) acc = fma((double)xp[c], (double)wp[(int64_t)c * K], acc);
      }
    }
    y[o] = (float)acc;
  }
}

// Per channel (innermost, `channels` of them): fmaf(t, a1, a2) or t + bias,
// then ReLU.  In place allowed.
__global__ __launch_bounds__(256) void k_teacher_affine(const float* t, int64_t n, int channels,
                                                        const float* a1, const float* a2,
                                                        const float* bias, int relu, float* y) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int c = (int)(i % channels);
    float v = t[i];
    if (a1) v = fmaf(v, a1[c], a2[c]);
    else if (bias) v = v + bias[c];
    if (relu) v = v > 0.0f ? v : 0.0f;
    y[i] = v;
  }
}

__global__ __launch_bounds__(256) void k_teacher_add(const float* a, const float* b, int64_t n,
                                                     int relu, float* y) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    float v = a[i] + b[i];
    if (relu) v = v > 0.0f ? v : 0.0f;
    y[i] = v;
  }
}

// NHWC max-pool; out-of-range taps are skipped.
__global__ __launch_bounds__(256) void k_teacher_maxpool(const float* x, float* y, int N, int H,
                                                         int W, int C, int ks, int stride, int pad,
                                                         int Ho, int Wo) {
  const int64_t total = (int64_t)N * Ho * Wo * C;
  for (int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; o < total;
       o += (int64_t)gridDim.x * blockDim.x) {
    const int c = (int)(o % C);
    int64_t pix = o / C;
    const int ow = (int)(pix % Wo);
    pix /= Wo;
    const int oh = (int)(pix % Ho);
    const int n = (int)(pix / Ho);
    float m = -INFINITY;
    for (int r = 0; r < ks; ++r) {
      const int ih = oh * stride - pad + r;
      if (ih < 0 || ih >= H) continue;
      for (int s = 0; s < ks; ++s) {
        const int iw = ow * stride - pad + s;
        if (iw < 0 || iw >= W) continue;
        m = fmaxf(m, x[(((int64_t)n * H + ih) * W + iw) * C + c]);
      }
    }
    y[o] = m;
  }
}

// x [n][hw][c] -> y [n][c].
__global__ __launch_bounds__(256) void k_teacher_avgpool(const float* x, float* y, int N, int hw,
                                                         int C) {
  const int64_t total = (int64_t)N * C;
  for (int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; o < total;
       o += (int64_t)gridDim.x * blockDim.x) {
    const int c = (int)(o % C);
    const int n = (int)(o / C);
    double acc = 0.0;
    for (int p = 0; p < hw; ++p) acc = acc + (double)x[((int64_t)n * hw + p) * C + c];
    y[o] = (float)(acc / (double)hw);
  }
}

static int elem_grid(int64_t n) {
  int64_t b = (n + 255) / 256;
  return (int)(b < 65536 ? (b < 1 ? 1 : b) : 65536);
}

// Outputs that one thread each computes faster than 32 x 32 tiles: few and
// shallow ones (a tile takes its 32 channels and 32 of depth whatever exists of
// them), and up to eight channels of a few input channels.  us, per output / in
// tiles, pixels x channels, depth: 784 x 64, 1 5.1 / 6.4; 12544 x 16, 9 5.2 / 7.2, x 64
// 10 / 10; 6240 x 269, 4 9.0 / 10.9; 100352 x 16, 4 9.1 / 11.8, x 24 12 / 12;
// 802816 x 4, 4 15 / 61, x 16 52 / 63, x 24 75 / 64; 802816 x 1, 9 10 / 77, x 8 57 /
// 79, x 12 84 / 80; 802816 x 8, 147 (3 input channels) 374 / 439, 100352 x 4 31 / 69,
// x 12 67 / 69, but 784 x 4 17 / 11; 16 input channels, 100352 x 4, 144 25 / 50, x 8
// 37 / 51, x 2 66 / 56, x 6 144 / 57; 64, x 4, 576 218 / 185.
static bool narrow_teacher(int64_t M, int K, int C, int64_t depth) {
  const int64_t one = K * (depth + 3);  // about a pixel's work
  if (one <= (C <= 4 ? 128 : 64) || (depth <= 16 && M * one <= (depth <= 9 ? 12000000 : 2500000))) return true;
  if (K > 8) return false;
  if (C <= 4) return depth <= 32 || M >= 65536;
  return C <= 16 && M >= 65536 && (K == 1 || K % 4 == 0);
}

hipError_t launch_teacher_conv(const Ctx& c, const fxpq_conv_desc& d, const float* x,
                               const float* w, float* y) {
  const int Ho = (d.h + 2 * d.pad - d.r) / d.stride + 1;
  const int Wo = (d.w + 2 * d.pad - d.s) / d.stride + 1;
  const int64_t M = (int64_t)d.n * Ho * Wo;
  if (narrow_teacher(M, d.k, d.c, (int64_t)d.r * d.s * d.c)) {
    k_teacher_narrow<<<elem_grid(M * d.k), 256, 0, c.stream>>>(x, w, y, d.n, d.h, d.w, d.c, d.k, d.r, d.s,
                                                               d.stride, d.pad, Ho, Wo);
    return hipGetLastError();
  }
  auto blocks = [&](int b) { return ((M + b - 1) / b) * ((d.k + b - 1) / b); };
  auto run = [&](auto kernel, int b) {
    const int64_t tiles = blocks(b);
    kernel<<<(int)(tiles < (1 << 20) ? tiles : (1 << 20)), 256, 0, c.stream>>>(
        x, w, y, d.n, d.h, d.w, d.c, d.k, d.r, d.s, d.stride, d.pad, Ho, Wo);
  };
  const bool vec = d.c % 4 == 0 && d.k % 4 == 0 && ((uintptr_t)x | (uintptr_t)w) % 16 == 0;
  // 64 x 64 blocks with at least four per CU, else 32 x 32 with slabs twice as
  // deep (3x3 64 -> 64 at 56x56, 6.1 large blocks per CU: 205 against 216 us;
  // 3x3 256 -> 256 at 14x14, 1.5: 248 against 227 us; 2 images of 512 -> 512
  // at 7x7: 295 against 106 us)
  if (blocks(64) >= 4 * (int64_t)c.cus) vec ? run(k_teacher_conv<2, 16, true>, 64) : run(k_teacher_conv<2, 16, false>, 64);
  else vec ? run(k_teacher_conv<1, 32, true>, 32) : run(k_teacher_conv<1, 32, false>, 32);
  return hipGetLastError();
}

hipError_t launch_teacher_affine(const Ctx& c, const float* t, int64_t n, int channels,
                                 const float* a1, const float* a2, const float* bias, int relu,
                                 float* y) {
  k_teacher_affine<<<elem_grid(n), 256, 0, c.stream>>>(t, n, channels, a1, a2, bias, relu, y);
  return hipGetLastError();
}

hipError_t launch_teacher_add(const Ctx& c, const float* a, const float* b, int64_t n, int relu,
                              float* y) {
  k_teacher_add<<<elem_grid(n), 256, 0, c.stream>>>(a, b, n, relu, y);
  return hipGetLastError();
}

hipError_t launch_teacher_maxpool(const Ctx& c, const float* x, int n, int h, int w, int ch,
                                  int ks, int stride, int pad, float* y) {
  const int Ho = (h + 2 * pad - ks) / stride + 1, Wo = (w + 2 * pad - ks) / stride + 1;
  k_teacher_maxpool<<<elem_grid((int64_t)n * Ho * Wo * ch), 256, 0, c.stream>>>(
      x, y, n, h, w, ch, ks, stride, pad, Ho, Wo);
  return hipGetLastError();
}

hipError_t launch_teacher_avgpool(const Ctx& c, const float* x, int n, int hw, int ch, float* y) {
  k_teacher_avgpool<<<elem_grid((int64_t)n * ch), 256, 0, c.stream>>>(x, y, n, hw, ch);
  return hipGetLastError();
}

}  // namespace fxpq
