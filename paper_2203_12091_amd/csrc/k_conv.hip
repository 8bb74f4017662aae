// Quantized convolution / FC (the C-Block contraction, Sec. "Integer-Only
// Inference"): implicit GEMM over NHWC int8 codes and KRSC int8 weights with
// int32 accumulation on the gfx950 int8 matrix cores (v_mfma_i32_32x32x32_i8).
//
//   rows    m = (n, oh, ow)          M = N * Ho * Wo
//   columns j = output channel       N = K
//   depth   k = (r, s, c), c fastest K = R * S * C
//
// A block computes a BM x BN tile with 4 waves (64 x 64 each, 2 x 2 MFMA tiles,
// at 128 x 128), stepping through depth in 64-byte slabs staged in LDS (a ring
// of three filled by LDS-DMA, or two stages through registers, the next slabs'
// loads in flight during the current slab's MFMAs); for grids that leave CUs
// idle the four waves share one small tile and split its depth (split_setup).
// No im2col buffer: each thread gathers its rows' 16-byte chunks straight from
// the NHWC tensor, with zero padding (code 0, or -128 for codes stored as
// u - 128, both meaning the value 0).
//
// Epilogue: for inputs stored as u - 128 the exact accumulator is restored by
// adding 128 * (sum of the filter's codes).  Then, by mode:
//   EPI_ACC  store the int32 accumulators; optionally reduce the exact min /
//            max of the C-Block values (bias, Scale, ReLU applied in fp64,
//            exact below 2^53) for the FxP-QLayer;
//   EPI_MM   only the min / max;
//   EPI_WIN  the window partial sums of the exact FL search over the C-Block
//            values (the same sums the streaming window pass forms);
//   EPI_REQ  the C-Block values requantized to the searched format (Eq. 1-2).
// (The predicted FxP-QLayer has its own kernel, k_pred.hip.)
// A C-Block whose contraction is shallow (R * S * C small next to the output)
// is cheaper to recompute three times than to write, and read twice, as
// int32: the fused launcher runs EPI_MM, EPI_WIN and EPI_REQ over the same
// operands, and stores int32 accumulators only when the window pass cannot
// decide and the exact general pass needs them.
#include "conv_load.hpp"

namespace fxpq {

template <int BM, int BN, int TM, int TN, int MINW, int LOADER, int EPI>
__global__ __launch_bounds__(256, MINW) void k_qconv(ConvArgs a) {
  constexpr int SPLIT = split_t(LOADER);
  constexpr int E = SPLIT == 1 ? 4 : 16;  // accumulators per thread and MFMA tile
  constexpr int WROWS = 2 * E * TM, WCOLS = 32 * TN;
  constexpr int WGN = BN / WCOLS;  // waves along N
  static_assert((BM / WROWS) * WGN == 4, "four waves per block");
  constexpr int PER_THREAD = TM * TN * 16;
  // LDS slabs: two stages for the register-staged loaders; the ring of the
  // DMA loader is declared with it.
  constexpr int NST = (is_ring(LOADER) || SPLIT) ? 1 : 2;
  __shared__ __attribute__((aligned(16))) int8_t As[NST][SPLIT ? 16 : BM * 64];
  __shared__ __attribute__((aligned(16))) int8_t Bs[NST][SPLIT ? 16 : BN * 64];
  __shared__ int rs_tab[128];
  __shared__ double shd[8];
  __shared__ WinShared wsh;

  // Decisions every block takes identically before any load.
  WinSetup ws;
  QFmt qf;
  if constexpr (EPI == EPI_ACC) {
    if (a.only_if_general && (!a.plan_in->need_general || a.plan_in->status)) return;
  } else if constexpr (EPI == EPI_WIN) {
    ws = win_setup<FXPQ_SRC_ACC>(a.ep, a.mm, a.wl, a.sign_req, a.fl_lo, a.fl_hi, MODE_SEARCH,
                                 PER_THREAD);
    if (ws.verdict != 0) {
      if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0)
        win_verdict_write(ws, a.wl, a.fl_lo, a.fl_hi, a.plan, a.fmt_win, a.flags);
      return;
    }
  } else if constexpr (EPI == EPI_REQ) {
    const int sv = src_scale(a.ep);
    if (a.y_type == FXPQ_I8) qf = qfmt_setup<FXPQ_I8>(a.fmt_req, sv, a.flags);
    else if (a.y_type == FXPQ_U8OFF) qf = qfmt_setup<FXPQ_U8OFF>(a.fmt_req, sv, a.flags);
    else qf = qfmt_setup<FXPQ_C8>(a.fmt_req, sv, a.flags);
    if (!qf.ok) return;
  }

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform per wave
  const int wm = wave / WGN, wn = wave % WGN;
  // Tile of this block.  Blocks are dealt to the 8 XCDs round-robin by linear
  // id; remapped so that each XCD takes a contiguous run of tiles in
  // row-block-major order, i.e. the column tiles of one row block run on the
  // same XCD and share its L2 copy of the input rows.
  int tm = blockIdx.x, tn = blockIdx.y;
  {
    const int T = gridDim.x * gridDim.y;
    if (T % 8 == 0) {
      const int L = blockIdx.y * gridDim.x + blockIdx.x;
      const int t = (L % 8) * (T / 8) + L / 8;
      tm = t / gridDim.y;
      tn = t - tm * gridDim.y;
    }
  }
  int m0 = tm * BM;
  const int n0 = tn * BN;
  // Halo tiles: output rows oh0 .. oh0 + hTH - 1 (all columns) of images
  // img0 .. img0 + hG - 1; vrows of the BM rows exist.
  int img0 = 0, oh0 = 0, vrows = BM;
  if constexpr (is_halo(LOADER)) {
    if (a.hG > 1) {
      img0 = tm * a.hG;
      vrows = min(a.hG, a.N - img0) * a.Ho * a.Wo;
    } else {
      img0 = tm / a.hTPI;
      oh0 = (tm - img0 * a.hTPI) * a.hTH;
      vrows = min(a.hTH, a.Ho - oh0) * a.Wo;
    }
    m0 = (img0 * a.Ho + oh0) * a.Wo;
  }

  // Inputs stored as u - 128 (branch-free, so the operand loads need not wait
  // for the format).
  const int fin_sign = *(a.has_ep ? &a.ep.fin->sign : &kEpiOne);
  const int a_off = (a.x_type == FXPQ_U8OFF) || (a.x_type == FXPQ_C8 && fin_sign == 0);
  const int padw = a_off ? (int)0x80808080 : 0;

  if (LOADER == LD_RGB4) rgb4_table(a, rs_tab);

  v16i acc[TM][TN];
#pragma unroll
  for (int mi = 0; mi < TM; ++mi)
#pragma unroll
    for (int ni = 0; ni < TN; ++ni)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[mi][ni][e] = 0;

  auto compute = [&](const int8_t* sa, const int8_t* sb) {
    slab_mfma<TM, TN>(sa, sb, wm * WROWS, wn * WCOLS, lane, acc);
  };

  // Per-channel epilogue operands of this thread's output columns, loaded
  // before the main loop so that their latency overlaps it.
  const bool want_vals = (EPI != EPI_ACC) || a.want_mm;
  int csum[TN];
  EpiRaw eraw[TN];
  auto epi_loads = [&]() {
#pragma unroll
    for (int ni = 0; ni < TN; ++ni) {
      const int col = n0 + wn * WCOLS + ni * 32 + (lane & 31);
      const int cc = col < a.K ? col : a.K - 1;
      csum[ni] = *(a_off ? a.colsum + cc : &kEpiZero);
      if (want_vals) eraw[ni] = epi_channel_load(a.ep, cc);
    }
  };
  const int ktiles = (a.kdepth + BK - 1) / BK;
  const int hw_out = a.Ho * a.Wo;
  const int taps = a.R * a.S;

  if constexpr (SPLIT != 0) {
    __shared__ __attribute__((aligned(16))) int8_t ring[kSplitLds<SPLIT>];
    SplitTile<SPLIT, is_gen(LOADER)> st;
    epi_loads();
    st.start(a, a_off, m0, n0, ktiles, wave, lane, ring);
    st.finish(a, wave, lane, ring, acc[0][0]);
  } else if constexpr (is_ring(LOADER)) {
    RingLoad<BM, BN, 4, is_gen(LOADER)> ld;
    ld.cols(a, a_off, n0, wave, lane);
    ld.rows(a, m0, wave, lane);
    constexpr int OPS = decltype(ld)::kOps;
    static_assert(OPS < 2 * TM * TN, "every load and the walk's step come before an MFMA of the slab");
    constexpr int D = 2;                // slabs in flight (3: two blocks per CU instead of three, 30% slower)
    constexpr int ST = (BM + BN) * 64;  // bytes of a stage: rows, then columns
    __shared__ __attribute__((aligned(16))) int8_t stage[(D + 1) * ST];
    // Slab kt sits in stage kt % (D + 1).  Waiting: this wave's pieces of slab
    // kt have landed (the next D - 1 slabs' may still be in flight); after the
    // barrier every wave's have, and every wave has finished reading the stage
    // of slab kt - 1, which slab kt + D takes.  Its loads go out between the
    // MFMAs.
    epi_loads();
    for (int i = 0; i < D && i < ktiles; ++i) ld.issue(a, stage + i * ST, stage + i * ST + BM * 64, wave);
    int8_t* cur = stage;
    for (int kt = 0; kt < ktiles - D; ++kt) {
      wait_vmcnt<OPS * (D - 1)>();
      ring_barrier();
      int8_t* st = cur == stage ? stage + D * ST : cur - ST;
      slab_mfma<TM, TN>(cur, cur + BM * 64, wm * WROWS, wn * WCOLS, lane, acc,
                        [&](int i) __attribute__((always_inline)) {
        if (i < OPS) ld.load(a, i, st, st + BM * 64, wave);
        else if (i == OPS) ld.advance(a);
        __builtin_amdgcn_sched_barrier(0);
      });
      cur = cur == stage + D * ST ? stage : cur + ST;
    }
    for (int left = min(D, ktiles); left > 0; --left) {
      if (left > 1) wait_vmcnt<OPS>();
      else wait_vmcnt<0>();
      ring_barrier();
      compute(cur, cur + BM * 64);
      cur = cur == stage + D * ST ? stage : cur + ST;
    }
  } else if constexpr (is_halo(LOADER)) {
    // Patch row R (pixel of the padded input patch) of a chunk sits at LDS row
    // R of a patch buffer; the DMA pieces of 16 rows are dealt to the waves as
    // in LD_DMA64.  Filter tap (r, s) of output row p reads patch row
    // pbase(p) + r * hPW + s.  Weights: one 64-byte slab per (chunk, tap).
    static_assert(WGN == 4, "halo tiles split the block's columns over the four waves");
    constexpr int AJ = (LOADER == LD_HALO8) ? 8 : 4, BJ = BN / 64;
    constexpr int NPR = 64 * AJ;  // patch rows per buffer
    constexpr int HD = kHaloStages;
    __shared__ __attribute__((aligned(16))) int8_t P0[NPR * 64], P1[NPR * 64];
    __shared__ __attribute__((aligned(16))) int8_t Bst[HD][BN * 64];
    const int ppx = a.hPH * a.hPW;
    const int npx = a.hG * ppx;
    const int8_t* psrc[AJ];
    bool pok[AJ];
#pragma unroll
    for (int j = 0; j < AJ; ++j) {
      const int R = 16 * (4 * j + wave) + (lane >> 2);
      const int g = R / ppx, rem = R - g * ppx;
      const int py = rem / a.hPW, px = rem - py * a.hPW;
      const int ih = oh0 * a.stride - a.pad + py, iw = px - a.pad, img = img0 + g;
      pok[j] = R < npx && img < a.N && ih >= 0 && ih < a.H && iw >= 0 && iw < a.W;
      const int lch = ((lane & 3) ^ lds_swz(R)) & 3;
      psrc[j] = a.x + (pok[j] ? (((int64_t)img * a.H + ih) * a.W + iw) * a.C + lch * 16 : 0);
    }
    const int8_t* bsrc[BJ];
#pragma unroll
    for (int j = 0; j < BJ; ++j) {
      const int row = 16 * (4 * j + wave) + (lane >> 2);
      const int col = n0 + row;
      const int cc = col < a.K ? col : a.K - 1;
      bsrc[j] = a.w + (int64_t)cc * a.wrow + (((lane & 3) ^ lds_swz(row)) & 3) * 16;
    }
    // patch row of tap (0, 0) for each of this lane's output rows
    int pbase[TM];
    const int rows_img = a.hTH * a.Wo;
#pragma unroll
    for (int mi = 0; mi < TM; ++mi) {
      const int p = mi * 32 + (lane & 31);
      const int g = p / rows_img, q = p - g * rows_img;
      const int ohl = q / a.Wo, ow = q - ohl * a.Wo;
      pbase[mi] = (p < vrows) ? g * ppx + ohl * a.stride * a.hPW + ow * a.stride : 0;
    }
    const int8_t* padp = reinterpret_cast<const int8_t*>(&kPadVec[a_off]);
    auto issue = [&](int kt, int8_t* sb) {
      const int cchunk = kt / taps;
      const int rs = kt - cchunk * taps;
      const int c0 = cchunk * BK;
      if (rs == 0) {
        int8_t* pb = (cchunk & 1) ? P1 : P0;
#pragma unroll
        for (int j = 0; j < AJ; ++j) dma16(pok[j] ? psrc[j] + c0 : padp, &pb[(4 * j + wave) * 1024]);
      }
      const int k0 = rs * a.C + c0;
#pragma unroll
      for (int j = 0; j < BJ; ++j) dma16(bsrc[j] + k0, &sb[(4 * j + wave) * 1024]);
    };
    auto compute_tap = [&](int kt, const int8_t* sb) {
      const int cchunk = kt / taps;
      const int rs = kt - cchunk * taps;
      const int r = rs / a.S, sx = rs - r * a.S;
      const int toff = r * a.hPW + sx;
      const int8_t* pb = (cchunk & 1) ? P1 : P0;
      v4i af[2][TM], bf[2][TN];
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
          af[kk][mi] = *reinterpret_cast<const v4i*>(&pb[lds_off(pbase[mi] + toff, kk * 2 + (lane >> 5))]);
#pragma unroll
        for (int ni = 0; ni < TN; ++ni)
          bf[kk][ni] = *reinterpret_cast<const v4i*>(
              &sb[lds_off(wn * WCOLS + ni * 32 + (lane & 31), kk * 2 + (lane >> 5))]);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
#pragma unroll
          for (int ni = 0; ni < TN; ++ni)
            acc[mi][ni] =
                __builtin_amdgcn_mfma_i32_32x32x32_i8(af[kk][mi], bf[kk][ni], acc[mi][ni], 0, 0, 0);
    };
    // Ring of HD weight stages: slab kt + HD - 1 is issued at step kt into
    // the stage slab kt - 1 used.  Waiting at step kt: slab kt's loads have
    // landed while the (up to HD - 2) later slabs' may be in flight; at most
    // one of those carries a chunk's patch (a chunk has taps >= HD - 1 slabs).
    auto wait_slab = [&](int kt) {
      const int later = min(HD - 2, ktiles - 1 - kt);
      bool patch = false;
      for (int j = 1; j <= later; ++j) patch = patch || (kt + j) % taps == 0;
      switch (later * 2 + (patch ? 1 : 0)) {
        case 0: wait_vmcnt<0>(); break;
        case 2: wait_vmcnt<BJ>(); break;
        case 3: wait_vmcnt<BJ + AJ>(); break;
        case 4: wait_vmcnt<2 * BJ>(); break;
        case 5: wait_vmcnt<2 * BJ + AJ>(); break;
        case 6: wait_vmcnt<3 * BJ>(); break;
        default: wait_vmcnt<3 * BJ + AJ>(); break;
      }
    };
    static_assert(HD >= 3 && HD <= 5, "ring depth");
    epi_loads();
#pragma unroll
    for (int j = 0; j < HD - 1; ++j)
      if (j < ktiles) issue(j, Bst[j]);
    for (int kt0 = 0; kt0 < ktiles; kt0 += HD) {
#pragma unroll
      for (int j = 0; j < HD; ++j) {
        const int kt = kt0 + j;
        if (kt < ktiles) {
          wait_slab(kt);
          ring_barrier();
          if (kt + HD - 1 < ktiles) issue(kt + HD - 1, Bst[(j + HD - 1) % HD]);
          compute_tap(kt, Bst[j]);
        }
      }
    }
  } else {
    StagedLoad<BM, BN, LOADER> ld;
    ld.cols(a, n0, tid);
    ld.rows(a, m0, tid);
    ld.gload(a, ktiles, tid, padw, rs_tab);
    epi_loads();
    ld.lstore(As[0], Bs[0], tid, padw);
    __syncthreads();
    for (int kt = 0; kt < ktiles; ++kt) {
      const int buf = kt & 1;
      if (kt + 1 < ktiles) ld.gload(a, ktiles, tid, padw, rs_tab);
      compute(As[buf], Bs[buf]);
      if (kt + 1 < ktiles) ld.lstore(As[buf ^ 1], Bs[buf ^ 1], tid, padw);
      __syncthreads();
    }
  }

  // ---- epilogue ----
  // Visits this thread's in-range accumulators (restored for u - 128 inputs)
  // with the channel's epilogue constants.
  EpiU eu;
  if (want_vals) eu = epi_uniform(a.ep);
  const bool full = m0 + BM <= a.M && n0 + BN <= a.K;
  auto visit = [&](auto&& f) {
#pragma unroll
    for (int ni = 0; ni < TN; ++ni) {
      const int col = n0 + wn * WCOLS + ni * 32 + (lane & 31);
      const int corr = 128 * csum[ni];
      double Mc = 1.0, Ac = 0.0;
      if (want_vals) epi_channel_raw(a.ep, eu, eraw[ni], Mc, Ac);
#pragma unroll
      for (int mi = 0; mi < TM; ++mi) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const int row = m0 + wm * WROWS + mi * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
          if (full || (row < a.M && col < a.K)) f(acc[mi][ni][e] + corr, Mc, Ac, row, col);
        }
      }
    }
  };
  const double relo = a.ep.ep_relu ? 0.0 : -INFINITY;  // ReLU as max(v, relo)
  const int bid = blockIdx.y * gridDim.x + blockIdx.x;

  if constexpr (EPI == EPI_ACC || EPI == EPI_MM) {
    // The epilogue value is a monotonic function of the accumulator within a
    // channel (v = relu(acc * M + A), rounding included), so the min / max of
    // the values are those of the channel's extreme accumulators: track the
    // integer extremes per column, evaluate the epilogue on them only.
    int lo[TN], hi[TN];
#pragma unroll
    for (int ni = 0; ni < TN; ++ni) {
      lo[ni] = INT_MAX;
      hi[ni] = INT_MIN;
    }
    if constexpr (is_halo(LOADER)) {
      // Rows past vrows do not exist (padding of the last MFMA row tile, or a
      // partial tile): their stores go to a scratch sink, their values are not
      // counted (branch-free selects).
#pragma unroll
      for (int ni = 0; ni < TN; ++ni) {
        const int col = n0 + wn * WCOLS + ni * 32 + (lane & 31);
        const int corr = 128 * csum[ni];
        int32_t* dst = a.acc + (int64_t)m0 * a.K + col;
        int32_t* sink = a.sink + (lane & 31);
#pragma unroll
        for (int mi = 0; mi < TM; ++mi) {
#pragma unroll
          for (int e = 0; e < E; ++e) {
            const int lr = mi * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
            const bool ok = lr < vrows;
            const int v = acc[mi][ni][e];
            if constexpr (EPI == EPI_ACC)
              __builtin_nontemporal_store(v + corr, ok ? dst + (int64_t)lr * a.K : sink);
            lo[ni] = min(lo[ni], ok ? v : INT_MAX);
            hi[ni] = max(hi[ni], ok ? v : INT_MIN);
          }
        }
      }
    } else if (full && a.K < (1 << 21)) {
      // Full tile: buffer stores with the row offset in a scalar register (at
      // most 132 rows of 4-byte values below the descriptor's 2 GiB).
      __amdgpu_buffer_rsrc_t rs;
      int vo[TN];
      if constexpr (EPI == EPI_ACC) {
        rs = __builtin_amdgcn_make_buffer_rsrc(a.acc + (int64_t)(m0 + wm * WROWS) * a.K, (short)0,
                                               0x7fffffff, 0x00020000);
#pragma unroll
        for (int ni = 0; ni < TN; ++ni)
          vo[ni] = (4 * (lane >> 5) * a.K + n0 + wn * WCOLS + ni * 32 + (lane & 31)) * 4;
      }
#pragma unroll
      for (int ni = 0; ni < TN; ++ni) {
        const int corr = 128 * csum[ni];
#pragma unroll
        for (int mi = 0; mi < TM; ++mi) {
#pragma unroll
          for (int e = 0; e < E; ++e) {
            const int v = acc[mi][ni][e];
            if constexpr (EPI == EPI_ACC)
              __builtin_amdgcn_raw_buffer_store_b32(
                  v + corr, rs, vo[ni], (mi * 32 + 8 * (e >> 2) + (e & 3)) * a.K * 4, kAccPolicy);
            lo[ni] = min(lo[ni], v);
            hi[ni] = max(hi[ni], v);
          }
        }
      }
    } else {
#pragma unroll
      for (int ni = 0; ni < TN; ++ni) {
        const int col = n0 + wn * WCOLS + ni * 32 + (lane & 31);
        const int corr = 128 * csum[ni];
#pragma unroll
        for (int mi = 0; mi < TM; ++mi) {
#pragma unroll
          for (int e = 0; e < E; ++e) {
            const int row = m0 + wm * WROWS + mi * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
            if (row < a.M && col < a.K) {
              const int v = acc[mi][ni][e];
              if constexpr (EPI == EPI_ACC)
                __builtin_nontemporal_store(v + corr, a.acc + (int64_t)row * a.K + col);
              lo[ni] = min(lo[ni], v);
              hi[ni] = max(hi[ni], v);
            }
          }
        }
      }
    }
    if (!want_vals) return;
    double mn = INFINITY, mx = -INFINITY;
#pragma unroll
    for (int ni = 0; ni < TN; ++ni) {
      if (lo[ni] > hi[ni]) continue;  // no in-range value in this column
      double Mc, Ac;
      epi_channel_raw(a.ep, eu, eraw[ni], Mc, Ac);
      const int corr = 128 * csum[ni];
      const double f0 = fmax(fma((double)(lo[ni] + corr), Mc, Ac), relo);
      const double f1 = fmax(fma((double)(hi[ni] + corr), Mc, Ac), relo);
      mn = fmin(mn, fmin(f0, f1));
      mx = fmax(mx, fmax(f0, f1));
    }
    mn = block_reduce(mn, OpMin(), shd);
    mx = block_reduce(mx, OpMax(), shd);
    if (a.mm_ticket) {
      ticket_minmax(mn, mx, bid, gridDim.x * gridDim.y, a.mm_part, a.mm_ticket, a.mm_out);
    } else if (tid == 0) {
      a.mm_part[2 * bid] = mn;
      a.mm_part[2 * bid + 1] = mx;
    }
  } else if constexpr (EPI == EPI_WIN) {
    const FlsU& u = ws.u;
    const WinCtx wc = win_ctx(u, ws);
    WinAcc wa;
    win_acc_zero(wa);
    // W = v * 2^(sigma - sv): fold the integer scaling into the constants.
    const double wsc = u.wscale;
#define FXPQ_WIN_VISIT(NN, C0)                                              \
  visit([&](int v, double Mc, double Ac, int, int) {                        \
    const double W = fmax(fma((double)v, Mc * wsc, Ac * wsc), relo);       \
    win_consume<false, NN, C0>(wc, wa, W);                                  \
  })
    switch (win_variant(u, ws, a.mm)) {
      case 0: FXPQ_WIN_VISIT(false, false); break;
      case 1: FXPQ_WIN_VISIT(false, true); break;
      case 2: FXPQ_WIN_VISIT(true, false); break;
      default: FXPQ_WIN_VISIT(true, true); break;
    }
#undef FXPQ_WIN_VISIT
    win_write_partials_int(wa, 1, bid, a.part_i, a.part_f, wsh);
  } else {  // EPI_REQ
    visit([&](int v, double Mc, double Ac, int row, int col) {
      const double val = fmax(fma((double)v, Mc, Ac), relo);
      a.y[(int64_t)row * a.K + col] = (int8_t)quant_one(val, qf);
    });
  }
}

template <int BM, int BN, int TM, int TN, int MINW, int EPI>
static void conv_dispatch_loader(int loader, dim3 grid, hipStream_t st, const ConvArgs& a) {
  // (256 x 64 tiles take the staged loaders, the others the ring; 256 x 128 ones
  // only C % 64 == 0)
  if constexpr (BN == 64) {
    if (loader == LD_FAST64) k_qconv<BM, BN, TM, TN, MINW, LD_FAST64, EPI><<<grid, 256, 0, st>>>(a);
    else if (loader == LD_GEN16) k_qconv<BM, BN, TM, TN, MINW, LD_GEN16, EPI><<<grid, 256, 0, st>>>(a);
    else if constexpr (EPI == EPI_ACC) {
      if (loader == LD_RGB8) k_qconv<BM, BN, TM, TN, MINW, LD_RGB8, EPI><<<grid, 256, 0, st>>>(a);
      else k_qconv<BM, BN, TM, TN, MINW, LD_RGB4, EPI><<<grid, 256, 0, st>>>(a);
    }
  } else if constexpr (BM == 256) {
    k_qconv<BM, BN, TM, TN, MINW, LD_DMA64, EPI><<<grid, 256, 0, st>>>(a);
  } else {
    if (loader == LD_DMA64) k_qconv<BM, BN, TM, TN, MINW, LD_DMA64, EPI><<<grid, 256, 0, st>>>(a);
    else k_qconv<BM, BN, TM, TN, MINW, LD_DMA16, EPI><<<grid, 256, 0, st>>>(a);
  }
}

// First-layer filters [k][(r S + s) 4 + c] (rows of wrow bytes) re-laid as
// [k][r][s < 4 chunks][c] (rows of wrow8 bytes, zeros past R, S).
__global__ void k_rgb8_weights(const int8_t* w, int K, int R, int S, int wrow, int8_t* out,
                               int wrow8, int chunks) {
  const int64_t n = (int64_t)K * wrow8;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int k = (int)(i / wrow8), b = (int)(i - (int64_t)k * wrow8);
    const int r = b / (16 * chunks), t = b - r * 16 * chunks, s = t >> 2, c = t & 3;
    out[i] = (r < R && s < S) ? w[(int64_t)k * wrow + (r * S + s) * 4 + c] : (int8_t)0;
  }
}

// Plain / predicted call, us, pixel by pixel -> by chunks: 64 x 224 x 224, 11x11
// stride 4 35.6 / 71.0 -> 29.9 / 43.6; 32 x 224 x 224, 3x3 84.9 / 112.5 -> 83.4 /
// 96.8 (two chunks per filter row -> one); 256 x 224 x 224, 7x7 stride 2 204.5 /
// 274.8 -> 194.2 / 263.9 (addresses from the image row instead of 64-bit products).
// A plain call of less than four slabs (up to 5x5) stays pixel by pixel: the re-lay's
// launch takes 2 us and its loads no less (by chunks -> pixel by pixel, 1600 x 688,
// 3x3 13.9 -> 11.9; 401408 x 64, 3x3 29.8 -> 27.2, 5x5 33.3 -> 33.7, 7x7 35.6 -> 44.0;
// but predicted 40.8 -> 54.5, 47.2 -> 62.7, 51.0 -> 79.5).
void rgb8_setup(const Ctx& c, const fxpq_conv_desc& d, ConvArgs& a, int& loader, bool plain) {
  // (the loader's pixel indices within an image are 32-bit)
  if (loader != LD_RGB4 || d.w < 4 || (int64_t)d.h * d.w > INT_MAX || !c.sc.rgb_w) return;
  const int chunks = (d.s + 3) / 4;
  const int64_t wrow8 = ((int64_t)d.r * chunks * 16 + 63) / 64 * 64;
  if (d.k * wrow8 > (int64_t)kRgbWBytes || (plain && wrow8 < 4 * BK)) return;
  const int64_t n = d.k * wrow8;
  k_rgb8_weights<<<(int)((n + 255) / 256), 256, 0, c.stream>>>(a.w, d.k, d.r, d.s, a.wrow, c.sc.rgb_w,
                                                               (int)wrow8, chunks);
  a.w = c.sc.rgb_w;
  a.wrow = (int)wrow8;
  a.kdepth = (int)wrow8;
  a.rgb_chunks = chunks;
  a.rgb_step_r = 4 / chunks;
  a.rgb_step_c = 4 % chunks;
  loader = LD_RGB8;
}

// Convolutions the halo tiles take: 3x3 filters (stride 1 or 2), 64-channel
// multiples in, 256-channel multiples out, contraction deep enough to be
// bound by the matrix cores.
static bool ep_halo_ok(const fxpq_conv_desc& d) {
  return d.r == 3 && d.s == 3 && (d.stride == 1 || d.stride == 2) && d.pad <= 2 && d.c % 64 == 0 &&
         d.k % 256 == 0 && d.r * d.s * d.c >= 1024;
}

dim3 conv_setup(const fxpq_conv_desc& d, const void* x, int x_type, const int8_t* w,
                       const int32_t* colsum, const SrcDev* ep, ConvArgs& a, int& loader,
                       int& cfg, int cus, int halo, bool wide_ok) {
  a.x = static_cast<const int8_t*>(x);
  a.w = w;
  a.colsum = colsum;
  a.N = d.n; a.H = d.h; a.W = d.w; a.C = d.c; a.K = d.k; a.R = d.r; a.S = d.s;
  a.stride = d.stride; a.pad = d.pad;
  a.Ho = (d.h + 2 * d.pad - d.r) / d.stride + 1;
  a.Wo = (d.w + 2 * d.pad - d.s) / d.stride + 1;
  a.M = d.n * a.Ho * a.Wo;
  a.kdepth = d.r * d.s * d.c;
  loader = (d.c % 64 == 0) ? LD_FAST64 : (d.c == 4 ? LD_RGB4 : LD_GEN16);
  a.wrow = (loader == LD_RGB4) ? (a.kdepth + 63) / 64 * 64 : a.kdepth;
  if (loader == LD_RGB4) a.kdepth = a.wrow;
  a.x_type = x_type;
  a.has_ep = ep != nullptr;
  if (ep) a.ep = *ep;
  // 256 x 64 tiles for narrow outputs; 256 x 128 (128 x 64 per wave: fewer LDS
  // bytes per MFMA, two blocks per CU) for deep contractions with enough tiles
  // to fill the chip; else 128 x 128 (three blocks per CU).
  const int64_t tiles_256x128 = (int64_t)((a.M + 255) / 256) * ((d.k + 127) / 128);
  if (d.k <= 64 || loader == LD_RGB4) cfg = TC_256x64;
  else if (wide_ok && loader == LD_FAST64 && a.kdepth >= 512 && 2 * tiles_256x128 >= 3 * (int64_t)cus)
    cfg = TC_256x128;
  else cfg = TC_128x128;
  // outside the narrow tiles: slabs through the LDS ring
  if (cfg != TC_256x64) loader = loader == LD_FAST64 ? LD_DMA64 : LD_DMA16;
  // (64 channels = gen_r S + gen_s taps and gen_c channels)
  a.gen_r = BK / d.c / d.s;
  a.gen_s = BK / d.c % d.s;
  a.gen_c = BK % d.c;
  a.gen_step = ((int64_t)a.gen_r * d.w + a.gen_s) * d.c + a.gen_c;
  // 3x3 filters over small images with 256-channel multiples, on request:
  // halo tiles of whole output rows (224 rows in 7 MFMA row tiles, else 128
  // in 4) when the patch fits 512 LDS rows and, first choice, the tiles fill
  // the chip.  (Measured slower than the implicit-GEMM tiles on ResNet-50's
  // 14x14 and 7x7 layers: one block per CU cannot hide the LDS and barrier
  // latency of each slab.)
  if (halo == FXPQ_TILING_HALO && loader == LD_DMA64 && ep_halo_ok(d)) {
    for (int opt = 0; opt < 2; ++opt) {
      const int bm = opt == 0 ? 224 : 128;
      const int howo = a.Ho * a.Wo;
      int G, TH;
      if (howo <= bm) {
        G = bm / howo;
        TH = a.Ho;
      } else {
        G = 1;
        TH = bm / a.Wo;
        if (TH < 1) continue;
      }
      const int PH = (TH - 1) * d.stride + d.r, PW = (a.Wo - 1) * d.stride + d.s;
      const int npx = G * PH * PW;
      if (npx > 512) continue;
      const int tpi = (a.Ho + TH - 1) / TH;
      const int64_t tm = (G > 1) ? (d.n + G - 1) / G : (int64_t)d.n * tpi;
      const int64_t tiles = tm * (d.k / 256);
      if (opt == 0 && tiles < cus) continue;
      a.hG = G;
      a.hTH = TH;
      a.hTPI = tpi;
      a.hPH = PH;
      a.hPW = PW;
      loader = npx <= 256 ? LD_HALO4 : LD_HALO8;
      cfg = opt == 0 ? TC_H224x256 : TC_H128x256;
      return dim3((unsigned)tm, d.k / 256);
    }
  }
  switch (cfg) {
    case TC_256x64: return dim3((a.M + 255) / 256, (d.k + 63) / 64);
    case TC_256x128: return dim3((a.M + 255) / 256, (d.k + 127) / 128);
    default: return dim3((a.M + 127) / 128, (d.k + 127) / 128);
  }
}

// Split tiles where they all fit the chip at once: 32 x 32 tiles up to two per
// CU (their LDS allows three), else 64 x 64 tiles up to one per CU (one fits).
// Plain contraction with its min / max and predicted call, us, 128 x 128 or
// 256 x 64 tiles / 64 x 64 / 32 x 32:
//   64 x 4096 x 9216   51.7 60.5 / 28.7 33.2 / 20.5 24.4  (256 tiles of 32)
//   8 x 512 x 4608     27.2 35.7 / 13.9 18.9 / 10.6 14.5  (16)
//   392 x 512 x 4608   27.3 35.7 / 14.1 19.1 / 11.1 15.1  (208)
//   1568 x 256 x 2304  18.3 26.0 / 11.6 16.4 / 11.3 15.7  (392)
//   6272 x 128 x 1152  13.2 20.1 / 10.7 15.3 / 14.0 19.2  (784)
//   25088 x 64 x 256   11.5 17.2 / 13.8 16.2 / --         (392 of 64)
//   10816 x 384 x 1728 18.7 26.4 / 32.3 36.6 / --         (1014 of 64)
// Between the two, 128 x 64 tiles where 128 x 128 ones take at most two thirds of
// the CUs: 6272 x 256 x 2304 (98 tiles of 128 x 128) 19.0 22.9 -> 15.7 20.3, 3136 x
// 512 x 4608 (100) 28.7 34.6 -> 23.6 28.5, 10816 x 256 x 2304 (170) 21.3 25.6 ->
// 19.5 24.0, 12544 x 256 x 2304 (196) 19.7 24.1 -> 20.6 24.6.  (Two groups of four
// waves on half the depth each in one 128 x 128 tile gave nothing: a slab's LDS
// traffic is what a CU waits for.)
void split_setup(ConvArgs& a, int& loader, int& cfg, dim3& grid, int cus) {
  if (loader != LD_FAST64 && loader != LD_DMA64 && loader != LD_GEN16 && loader != LD_DMA16) return;
  auto tiles = [&](int t) { return (int64_t)((a.M + t - 1) / t) * ((a.K + t - 1) / t); };
  int t;
  if (tiles(32) <= 2 * cus) t = 32;
  else if (tiles(64) <= cus) t = 64;
  else {
    if (cfg == TC_128x128 && 3 * tiles(128) <= 2 * cus) {
      cfg = TC_128x64;
      grid = dim3((a.M + 127) / 128, (a.K + 63) / 64);
    }
    return;
  }
  if (loader == LD_GEN16 || loader == LD_DMA16) loader = t == 32 ? LD_SPLIT32G : LD_SPLIT64G;
  else loader = t == 32 ? LD_SPLIT32 : LD_SPLIT64;
  cfg = t == 32 ? TC_32x32 : TC_64x64;
  grid = dim3((a.M + t - 1) / t, (a.K + t - 1) / t);
}

template <int EPI>
static void conv_run(const ConvArgs& a, int loader, int cfg, dim3 grid, hipStream_t st) {
  if constexpr (EPI == EPI_ACC) {
    if (cfg == TC_128x64) {
      if (loader == LD_DMA64) k_qconv<128, 64, 1, 2, 3, LD_DMA64, EPI><<<grid, 256, 0, st>>>(a);
      else k_qconv<128, 64, 1, 2, 3, LD_DMA16, EPI><<<grid, 256, 0, st>>>(a);
      return;
    }
    if (cfg == TC_64x64) {
      if (loader == LD_SPLIT64) k_qconv<64, 64, 1, 1, 1, LD_SPLIT64, EPI><<<grid, 256, 0, st>>>(a);
      else k_qconv<64, 64, 1, 1, 1, LD_SPLIT64G, EPI><<<grid, 256, 0, st>>>(a);
      return;
    }
    if (cfg == TC_32x32) {
      if (loader == LD_SPLIT32) k_qconv<32, 32, 1, 1, 1, LD_SPLIT32, EPI><<<grid, 256, 0, st>>>(a);
      else k_qconv<32, 32, 1, 1, 1, LD_SPLIT32G, EPI><<<grid, 256, 0, st>>>(a);
      return;
    }
    if (cfg == TC_H224x256) {
      if (loader == LD_HALO4) k_qconv<224, 256, 7, 2, 1, LD_HALO4, EPI><<<grid, 256, 0, st>>>(a);
      else k_qconv<224, 256, 7, 2, 1, LD_HALO8, EPI><<<grid, 256, 0, st>>>(a);
      return;
    }
    if (cfg == TC_H128x256) {
      if (loader == LD_HALO4) k_qconv<128, 256, 4, 2, 1, LD_HALO4, EPI><<<grid, 256, 0, st>>>(a);
      else k_qconv<128, 256, 4, 2, 1, LD_HALO8, EPI><<<grid, 256, 0, st>>>(a);
      return;
    }
  }
  constexpr int W3 = 3;
  if (cfg == TC_256x64)
    conv_dispatch_loader<256, 64, 2, 2, W3, EPI>(loader, grid, st, a);
  else if (cfg == TC_256x128) {
    conv_dispatch_loader<256, 128, 4, 2, 2, EPI>(loader, grid, st, a);
  } else
    conv_dispatch_loader<128, 128, 2, 2, W3, EPI>(loader, grid, st, a);
}

hipError_t launch_conv(const Ctx& c, const fxpq_conv_desc& d, const void* x, int x_type,
                       const int8_t* w, const int32_t* colsum, const SrcDev* ep, int32_t* acc,
                       double* d_minmax) {
  ConvArgs a{};
  int loader;
  int cfg;
  dim3 grid = conv_setup(d, x, x_type, w, colsum, ep, a, loader, cfg, c.cus, c.conv_tiling);
  split_setup(a, loader, cfg, grid, c.cus);
  a.acc = acc;
  a.sink = c.sc.sink;
  a.want_mm = (ep != nullptr && d_minmax != nullptr);
  a.mm_part = c.sc.minmax_part;
  const int nb = (int)(grid.x * grid.y);
  a.mm_ticket = ticket_for(c, nb);
  a.mm_out = d_minmax;
  bool timed = timer_begin(c, FXPQ_TIMER_QCONV);
  rgb8_setup(c, d, a, loader, true);
  conv_run<EPI_ACC>(a, loader, cfg, grid, c.stream);
  timer_end(c, timed, 2.0 * (double)a.M * (double)d.k * (double)(d.r * d.s * d.c));
  if (a.want_mm && !a.mm_ticket) return launch_minmax_fin(c, a.mm_part, nb, d_minmax);
  return hipGetLastError();
}

int conv_fused_blocks(const fxpq_conv_desc& d, int cus, bool rgb_ok) {
  ConvArgs a{};
  int loader;
  int cfg;
  const dim3 grid = conv_setup(d, nullptr, 0, nullptr, nullptr, nullptr, a, loader, cfg, cus);
  if (loader == LD_RGB4 && !rgb_ok) return -1;
  return (int)(grid.x * grid.y);
}

// Conv + epilogue + FxP-QLayer (FL search, requantization) with the int32
// accumulators recomputed instead of stored.  `ep` is the ACC source of the
// C-Block values, its x pointing at the fallback int32 buffer.
hipError_t launch_conv_fused(const Ctx& c, const fxpq_conv_desc& d, const void* x, int x_type,
                             const int8_t* w, const int32_t* colsum, const SrcDev& ep, int wl,
                             int sign, int fl_lo, int fl_hi, fxpq_fmt* out, int8_t* y, int y_type,
                             double* d_minmax) {
  ConvArgs a{};
  int loader;
  int cfg;
  const dim3 grid = conv_setup(d, x, x_type, w, colsum, &ep, a, loader, cfg, c.cus);
  const int nb = (int)(grid.x * grid.y);
  const double ops = 2.0 * (double)a.M * (double)d.k * (double)(d.r * d.s * d.c);
  const int64_t n = (int64_t)a.M * d.k;
  // 1. min / max of the C-Block values
  a.want_mm = 1;
  a.mm_part = c.sc.minmax_part;
  bool timed = timer_begin(c, FXPQ_TIMER_CBLOCK_PASS);
  conv_run<EPI_MM>(a, loader, cfg, grid, c.stream);
  timer_end(c, timed, ops);
  hipError_t e = launch_minmax_fin(c, a.mm_part, nb, d_minmax);
  if (e != hipSuccess) return e;
  // 2. window partial sums, then the exact decision
  a.wl = wl;
  a.sign_req = sign;
  a.fl_lo = fl_lo;
  a.fl_hi = fl_hi;
  a.mm = d_minmax;
  const int set = fls_begin(c);
  a.part_i = c.sc.win_part + (size_t)set * kWinSlots * kWinPart;
  a.part_f = c.sc.win_part_f + (size_t)set * kWinSlots * kWinPartF;
  a.plan = static_cast<FlsPlan*>(c.sc.plan);
  a.fmt_win = out;
  a.flags = c.sc.flags;
  timed = timer_begin(c, FXPQ_TIMER_CBLOCK_PASS);
  conv_run<EPI_WIN>(a, loader, cfg, grid, c.stream);
  timer_end(c, timed, ops);
  e = launch_fls_window_fin(c, ep, set, wl, sign, fl_lo, 1, fl_hi, MODE_SEARCH, conv_per_thread(cfg),
                            d_minmax, out);
  if (e != hipSuccess) return e;
  // 3. only when the plan asks for the general pass: int32 accumulators, then
  //    the exact search over every remaining candidate
  ConvArgs g = a;
  g.acc = static_cast<int32_t*>(const_cast<void*>(ep.x));
  g.want_mm = 0;
  g.only_if_general = 1;
  g.plan_in = static_cast<const FlsPlan*>(c.sc.plan);
  conv_run<EPI_ACC>(g, loader, cfg, grid, c.stream);
  e = launch_fls_general(c, ep, n, wl, fl_lo, fl_hi, d_minmax, out, nullptr);
  if (e != hipSuccess) return e;
  // 4. codes in the searched format
  a.fmt_req = out;
  a.y = y;
  a.y_type = y_type;
  timed = timer_begin(c, FXPQ_TIMER_CBLOCK_PASS);
  conv_run<EPI_REQ>(a, loader, cfg, grid, c.stream);
  timer_end(c, timed, ops);
  return hipGetLastError();
}

}  // namespace fxpq
