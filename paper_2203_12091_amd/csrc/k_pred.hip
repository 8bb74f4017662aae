// Predicted C-Block (fxpq_cblock_predicted): the int8 contraction of k_conv.hip
// followed by the predicted FxP-QLayer in one pass.  The epilogue forms the
// window partial sums of the exact FL search at the window the previous call's
// min / max give, writes the codes of the candidate the previous call chose
// and reduces this call's min / max; no int32 accumulators.  The decision
// (k_pred_fin / k_pred_decide) checks the prediction.
//
// A block keeps its column tile and walks several row tiles: the window's
// set-up, the channels' constants, the weights' addresses and the block
// reduction are paid once per block instead of once per tile (they took about
// as many instructions as the 64 values per thread of a tile), and the next
// tile's first slabs load during the epilogue.  Bound by vector arithmetic
// where the contraction is shallow (about 18 instructions per value), by the
// contraction's operand delivery where it is deep.  Two blocks per CU: the
// state between the tiles takes 209-248 registers, and at three blocks (168)
// it spilled about a hundred of them.  One block per tile against this, batch
// 256, predicted call: 56x56 64 -> 256 1x1 228 -> 166 us, 28x28 128 -> 512 1x1
// 128 -> 101, 14x14 256 -> 1024 1x1 80 -> 65, 14x14 256 3x3 66 -> 58 (with the
// loads between the MFMAs, see slab_mfma), 7x7 512 3x3 66 -> 53.
#include "conv_load.hpp"

namespace fxpq {

// Values that all lanes hold, moved to scalar registers (results of vector
// arithmetic stay in vector registers otherwise).
__device__ inline int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ inline double uniform(double v) {
  return __hiloint2double(uniform(__double2hiint(v)), uniform(__double2loint(v)));
}

template <int BM, int BN, int LOADER>
__global__ __launch_bounds__(256, 2) void k_cblock_pred(ConvArgs a) {
  constexpr int SPLIT = split_t(LOADER);
  constexpr int TM = SPLIT ? 1 : BM * BN / 8192, TN = SPLIT ? 1 : 2;  // MFMA tiles per wave
  constexpr int NG = SPLIT == 1 ? 1 : 4;      // groups of four accumulators per thread and tile
  constexpr int WROWS = 8 * NG * TM, WCOLS = 32 * TN;
  constexpr int WGN = BN / WCOLS;  // waves along N
  static_assert((BM / WROWS) * WGN == 4, "four waves per block");
  // bound on the values per thread and tile (one for all tile shapes, so that
  // the decision does not depend on the shape)
  constexpr int PER_THREAD = 64;
  constexpr int NST = is_ring(LOADER) ? 3 : 2;  // LDS stages
  constexpr int SA = BM * 64, SB = BN * 64;
  __shared__ __attribute__((aligned(16))) int8_t stage[SPLIT ? kSplitLds<SPLIT> : NST * (SA + SB)];
  __shared__ int rs_tab[128];
  __shared__ WinShared wsh;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform per wave
  const int wm = wave / WGN, wn = wave % WGN;
  // Blocks are dealt to the 8 XCDs round-robin by id; remapped so that each XCD
  // takes a contiguous run of row-block-major tiles, i.e. the column tiles of a
  // run of rows share its L2 copy of the input.
  int t = blockIdx.x;
  if (gridDim.x % 8 == 0) t = (blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
  const int worker = t / a.ntn, n0 = (t - worker * a.ntn) * BN;
  const int tm0 = (int)((int64_t)a.ntm * worker / a.workers);
  const int tm1 = (int)((int64_t)a.ntm * (worker + 1) / a.workers);

  // The uniform inputs of the set-up, by scalar loads before anything else.
  const double pmm[2] = {a.mm[0], a.mm[1]};
  const fxpq_fmt prev = *a.fmt_win, fin = *a.ep.fin;
  SrcDev ep = a.ep;
  ep.fin = &fin;
  // Inputs stored as u - 128.
  const int a_off = (a.x_type == FXPQ_U8OFF) || (a.x_type == FXPQ_C8 && fin.sign == 0);
  const int padw = a_off ? (int)0x80808080 : 0;
  if (LOADER == LD_RGB4) rgb4_table(a, rs_tab);
  const int ktiles = (a.kdepth + BK - 1) / BK;
  const int total = (tm1 - tm0) * ktiles;

  // Per-channel operands of this thread's output columns.
  int csum[TN];
  EpiRaw eraw[TN];
#pragma unroll
  for (int ni = 0; ni < TN; ++ni) {
    const int col = n0 + wn * WCOLS + ni * 32 + (lane & 31);
    const int cc = col < a.K ? col : a.K - 1;
    csum[ni] = *(a_off ? a.colsum + cc : &kEpiZero);
    eraw[ni] = epi_channel_load(ep, cc);
  }

  // The first slabs' loads go out before the set-up, which runs meanwhile (in
  // small grids the set-up and the waits for the channel constants and the
  // first slabs, one after the other, took 3.5 of a call's 9 us).
  using Load = std::conditional_t<
      SPLIT != 0, SplitTile<SPLIT == 0 ? 1 : SPLIT, is_gen(LOADER)>,
      std::conditional_t<is_ring(LOADER), RingLoad<BM, BN, 4, is_gen(LOADER)>, StagedLoad<BM, BN, LOADER>>>;
  Load ld;
  int ti = tm0;  // tile being loaded
  bool ended = false;
  constexpr int D = NST - 1, ST = SA + SB;  // LDS ring: slabs in flight, bytes of a stage
  auto advance = [&](auto& l) __attribute__((always_inline)) {
    if (l.advance(a) && ++ti < tm1) l.rows(a, ti * BM, wave, lane);
  };
  auto issue = [&](auto& l, int8_t* st) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < l.kOps; ++i) l.load(a, i, st, st + SA, wave);
    advance(l);
  };
  if constexpr (SPLIT != 0) {
    ld.start(a, a_off, tm0 * BM, n0, ktiles, wave, lane, stage);
  } else if constexpr (is_ring(LOADER)) {
    ld.cols(a, a_off, n0, wave, lane);
    ld.rows(a, tm0 * BM, wave, lane);
    for (int i = 0; i < D && i < total; ++i) issue(ld, stage + i * ST);
  } else {
    ld.cols(a, n0, tid);
    ld.rows(a, tm0 * BM, tid);
    ended = ld.gload(a, ktiles, tid, padw, rs_tab);
  }

  if (a.job && blockIdx.x == 0 && tid == 0)
    *a.job = PredJob{a.ep, a.wl, a.sign_req, a.fl_lo, a.fl_hi, 1, a.job_per_thread,
                     const_cast<double*>(a.mm), a.fmt_win, a.job_miss, a.part_i, a.part_f};
  // the window of the predicted min / max (verdict != 0: none to evaluate,
  // the decision counts the call a miss; the min / max still go out)
  const WinSetup ws = win_setup<FXPQ_SRC_ACC>(ep, pmm, a.wl, a.sign_req, a.fl_lo, a.fl_hi,
                                              MODE_SEARCH, PER_THREAD);
  v16i acc[TM][TN];
  // The accumulators start at the restoring term 128 * (sum of the filter's
  // codes) of inputs stored as u - 128 (zero otherwise), so the matrix cores
  // return the restored accumulator (exact in int32 like it).
  auto acc_start = [&]() {
#pragma unroll
    for (int ni = 0; ni < TN; ++ni)
#pragma unroll
      for (int mi = 0; mi < TM; ++mi)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[mi][ni][e] = 128 * csum[ni];
  };

  const FlsU& u = ws.u;
  const bool win = uniform(ws.verdict) == 0;
  const int pj = uniform(pred_pick(ws, prev));
  const int qmax = uniform((int)u.qmax), qmin = uniform((int)u.qmin);
  const unsigned xorw = u.sign ? 0u : 0x80808080u;
  const double relo = uniform(a.ep.ep_relu ? 0.0 : -INFINITY);  // ReLU as max(v, relo)
  WinCtx wc{};
  if (win) wc = win_ctx(u, ws);
  wc.qmin = uniform(wc.qmin);
  wc.qmax = uniform(wc.qmax);
  // The window sums are formed from x = W 2^(b0 - sigma), the value in units of
  // the first candidate's step, straight from the accumulator (multiplier and
  // addend scaled by that power of two): its code is rne(x), the second
  // candidate's rne(2 x), the clipping bound's argument x 2^(bce - b0).  Sums
  // of x q and x^2 are those of W q and W^2 scaled by 2^(b0 - sigma) and its
  // square, exactly (every term keeps its bits); they are scaled back before
  // the block reduction.  Where the first candidate cannot saturate, the second
  // candidate's code comes from the low bits of x plus a rounding constant,
  // clamped as an integer, then converted back, and the written candidate's
  // sum q^2 from dot products of its packed codes (exact integers).
  const int ex = win ? uniform(ws.b0 - u.sigma) : 0, ece = win ? uniform(ws.bce - ws.b0) : 0;
  const double xce_hi = uniform(ldexp(wc.qmax, -ece)), xce_lo = uniform(ldexp(wc.qmin, -ece));
  const double up = uniform(ldexp(1.0, -ex));
  const EpiU eu = epi_uniform(ep);
  double Mx[TN], Ax[TN];
#pragma unroll
  for (int ni = 0; ni < TN; ++ni) {
    epi_channel_raw(ep, eu, eraw[ni], Mx[ni], Ax[ni]);
    // columns past the tensor's hold zeros, which add nothing to any sum
    const bool in = n0 + wn * WCOLS + ni * 32 + (lane & 31) < a.K;
    Mx[ni] = in ? ldexp(Mx[ni], ex) : 0.0;
    Ax[ni] = in ? ldexp(Ax[ni], ex) : 0.0;
  }
  // Sums over the block's tiles.  One tile's sums of x q are exact in fp64 (the
  // bound of the window's set-up) and then added as integers.
  WinAcc wa;
  win_acc_zero(wa);
  long long wq[kWindow] = {0, 0};
  // min / max from the integer extremes of each column (the epilogue is
  // monotonic in the accumulator within a channel)
  int lo[TN], hi[TN];
#pragma unroll
  for (int ni = 0; ni < TN; ++ni) {
    lo[ni] = INT_MAX;
    hi[ni] = INT_MIN;
  }
  // byte selectors of the code transpose (v_perm: bytes 0-3 this lane's dword,
  // 4-7 the partner's): step 1 pairs lanes j, j ^ 1 (even lanes keep bytes 0
  // and 2 of both, odd lanes bytes 1 and 3), step 2 lanes j, j ^ 2 (the low or
  // high halves of both)
  const int qj = lane & 3;
  const unsigned s1 = (qj & 1) ? 0x03070105u : 0x06020400u;
  const unsigned s2 = (qj & 2) ? 0x03020706u : 0x05040100u;
  // tiles of BM rows store through a buffer descriptor: row offsets in scalars,
  // columns past the tensor's dropped by its range (their tiles took the general
  // form before: 401408 x 96 x 16 83 -> 52 us)
  int vo[TN];
#pragma unroll
  for (int ni = 0; ni < TN; ++ni)
    vo[ni] = n0 + wn * WCOLS + ni * 32 + ((lane & 31) & ~3) < a.K
                 ? (4 * (lane >> 5) + qj) * a.K + n0 + wn * WCOLS + ni * 32 + ((lane & 31) & ~3)
                 : INT_MIN;  // past the descriptor's range: dropped

  // The codes leave as dwords: a lane holds one column at 4 consecutive rows
  // (e = 4g .. 4g + 3), and a 4 x 4 byte transpose inside each lane quad (one
  // partner exchange and one per-lane byte permute per step) gives lane 4k + j
  // row j at 4 consecutive columns.
  auto pack4 = [&](const int (&c)[4]) __attribute__((always_inline)) -> unsigned {
    const unsigned p01 = __builtin_amdgcn_perm((unsigned)c[1], (unsigned)c[0], 0x0C0C0400u);
    const unsigned p23 = __builtin_amdgcn_perm((unsigned)c[3], (unsigned)c[2], 0x0C0C0400u);
    return __builtin_amdgcn_perm(p23, p01, 0x05040100u);
  };
  auto transpose4 = [&](unsigned w4) __attribute__((always_inline)) -> unsigned {
    w4 = __builtin_amdgcn_perm((unsigned)__builtin_amdgcn_mov_dpp((int)w4, 0xB1, 0xF, 0xF, false), w4, s1);
    w4 = __builtin_amdgcn_perm((unsigned)__builtin_amdgcn_mov_dpp((int)w4, 0x4E, 0xF, 0xF, false), w4, s2);
    return w4 ^ xorw;
  };
  // The tile's sums of W q = 2^(sigma - b0) x q, as integers.
  auto add_tile = [&]() __attribute__((always_inline)) {
    wq[0] += exact_i64(wa.PL[0] * up);
    wq[1] += exact_i64(wa.PL[1] * up);
  };

  // A tile of BM rows of a window whose first candidate does not saturate: its
  // values' min / max, its window sums and the codes of candidate PJ as bytes
  // (q - 128 when unsigned).  NN: no negative values.  Straight-line code.
  auto tile_full = [&](int m0, auto nn, auto pj_) __attribute__((always_inline)) {
    constexpr bool NN = decltype(nn)::value;
    constexpr int PJ = decltype(pj_)::value ? 1 : 0;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        a.y + (int64_t)(m0 + wm * WROWS) * a.K, (short)0, 0x7fffffff, 0x00020000);
    wa.PL[0] = wa.PL[1] = 0.0;
    int dq = 0;  // sum q^2 of the written candidate
#pragma unroll
    for (int ni = 0; ni < TN; ++ni) {
#pragma unroll
      for (int mi = 0; mi < TM; ++mi) {
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          int c[4];
#pragma unroll
          for (int jj = 0; jj < 4; ++jj) {
            static_assert(kWindow == 2, "two window candidates");
            const int v = acc[mi][ni][4 * g + jj];
            lo[ni] = min(lo[ni], v);
            hi[ni] = max(hi[ni], v);
            // a window with negative values is never a ReLU layer's (its
            // values are >= 0, so is the previous call's minimum): no max with
            // the ReLU bound there; a prediction that says otherwise is a miss
            // anyway (its window's variant differs from the actual one)
            double x = fma((double)v, Mx[ni], Ax[ni]);
            if (NN) x = max64s(x, relo);
            wa.V2 = fma(x, x, wa.V2);
            // every value of a hit lies within [qmin - 1/2, qmax + 1/2] at the
            // first candidate's step (one at qmax + 1/2 has the same error
            // term with the code qmax)
            double q0 = rint(x);
            int c0 = 0;
            if (PJ == 0) {
              q0 = min64(q0, wc.qmax);
              c0 = (int)q0;
            } else {
              wa.A[0] = fma(q0, q0, wa.A[0]);
            }
            wa.PL[0] = fma(x, q0, wa.PL[0]);
            const int c1 = NN ? min(rne_lo(x + kRne1), qmax) : med3i(rne_lo(x + kRne1), qmin, qmax);
            const double q1 = (double)c1;
            if (PJ == 0) wa.A[1] = fma(q1, q1, wa.A[1]);
            wa.PL[1] = fma(x, q1, wa.PL[1]);
            // clipping error at bce: (x - x clamped to its range [qmin, qmax]
            // 2^(b0 - bce))^2, in units scaled by 2^(2 (b0 - bce)) (exactly
            // those of (t - qmax)^+ and (t - qmin)^- with t = x 2^(bce - b0),
            // scaled back below); one-sided without negative values
            double xcl = min64(x, xce_hi);
            if (!NN) xcl = max64(xcl, xce_lo);
            const double e = x - xcl;
            wa.CE[0] = fma(e, e, wa.CE[0]);
            c[jj] = PJ ? c1 : c0;
          }
          const unsigned w4 = pack4(c);
          if (NN) dq = (int)__builtin_amdgcn_udot4(w4, w4, (unsigned)dq, false);
          else dq = __builtin_amdgcn_sdot4((int)w4, (int)w4, dq, false);
          __builtin_amdgcn_raw_buffer_store_b32(transpose4(w4), rs, vo[ni], (mi * 32 + 8 * g) * a.K, 0);
        }
      }
    }
    wa.A[PJ] += (double)dq;
    add_tile();
  };
  // Any other tile: values past the tensor's rows add nothing, both
  // candidates' codes are clamped in fp64 (a first candidate that saturates: x
  // is not bounded by the codes' range; or an unsigned format forced on
  // negative values), or only the min / max (no window).  A rolled loop over
  // eight accumulators a time, which move down by as many registers: unrolled,
  // its checks took more registers than the block has.
  auto tile_any = [&](int m0, auto wn_) __attribute__((always_inline)) {
    constexpr bool WIN = decltype(wn_)::value;
    wa.PL[0] = wa.PL[1] = 0.0;
#pragma unroll
    for (int ni = 0; ni < TN; ++ni) {
      const int col = n0 + wn * WCOLS + ni * 32 + (lane & 31);
      const int scol = n0 + wn * WCOLS + ni * 32 + ((lane & 31) & ~3);
      int rbase = m0 + wm * WROWS + 4 * (lane >> 5);
#pragma nounroll
      for (int it = 0; it < (TM * NG + 1) / 2; ++it, rbase += 16) {
#pragma unroll
        for (int g = 0; g < (NG < 2 ? NG : 2); ++g) {
          int c[4];
#pragma unroll
          for (int jj = 0; jj < 4; ++jj) {
            const int v = acc[0][ni][4 * g + jj];
            const bool ok = rbase + 8 * g + jj < a.M && col < a.K;
            lo[ni] = min(lo[ni], ok ? v : INT_MAX);
            hi[ni] = max(hi[ni], ok ? v : INT_MIN);
            if constexpr (WIN) {
              double x = max64s(fma((double)v, Mx[ni], Ax[ni]), relo);
              x = ok ? x : 0.0;
              wa.V2 = fma(x, x, wa.V2);
              const double q0 = max64(min64(rint(x), wc.qmax), wc.qmin);
              const double q1 = max64(min64(rint(x + x), wc.qmax), wc.qmin);
              wa.A[0] = fma(q0, q0, wa.A[0]);
              wa.PL[0] = fma(x, q0, wa.PL[0]);
              wa.A[1] = fma(q1, q1, wa.A[1]);
              wa.PL[1] = fma(x, q1, wa.PL[1]);
              const double e = x - max64(min64(x, xce_hi), xce_lo);
              wa.CE[0] = fma(e, e, wa.CE[0]);
              c[jj] = (int)(pj ? q1 : q0);
            }
          }
          if constexpr (WIN) {
            const unsigned w4 = transpose4(pack4(c));
            const int srow = rbase + 8 * g + qj;
            if (srow < a.M && scol < a.K)
              *reinterpret_cast<unsigned*>(a.y + (int64_t)srow * a.K + scol) = w4;
          }
        }
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            if (NG == 1) break;
            if (e < 8) acc[mi][ni][e] = acc[mi][ni][e + 8];
            else if (mi + 1 < TM) acc[mi][ni][e] = acc[mi + 1][ni][e - 8];
          }
      }
    }
    if (WIN) add_tile();
  };
  // The straight-line form: the first candidate does not saturate, and the
  // codes fit the dot product (signed, or no negative values).
  const int var = win ? win_variant(u, ws, a.mm) : 0;  // 2 NN + C0
  // (its stores' offsets within 64 rows of output stay below the descriptor's range)
  const bool fast = win && (var == 2 || (var == 0 && u.sign)) && a.K < (1 << 25);
  // Wave priorities: the two blocks of a CU run the same phases, and where both
  // wait for one unit at once the other idles.  With the contraction ahead
  // (deep: the matrix cores are what a tile waits for) or the epilogue ahead
  // (shallow: vector arithmetic is) the blocks shift against each other.
  // Batch 256, no priorities / contraction ahead / epilogue ahead: 28x28 128
  // 3x3 67.8 / 62.5 / 65.2 us, 14x14 256 3x3 56.7 / 54.3 / 56.1, 28x28 512 -> 128
  // 1x1 (8 slabs) 49.6 / 48.3 / 48.2, 14x14 256 -> 1024 1x1 (4 slabs) 62.9 / 63.1
  // / 60.4, 28x28 128 -> 512 1x1 (2) 100.1 / 97.3 / 92.7, 56x56 64 -> 256 1x1
  // (1) 170 / 169 / 162.
  const bool deep = ktiles >= 8;
  auto contraction_prio = [&]() __attribute__((always_inline)) {
    if (deep) __builtin_amdgcn_s_setprio(2);
    else __builtin_amdgcn_s_setprio(0);
  };
  auto epilogue_prio = [&]() __attribute__((always_inline)) {
    if (deep) __builtin_amdgcn_s_setprio(0);
    else __builtin_amdgcn_s_setprio(2);
  };
  // Epilogue of row tile tm; true when it issued exactly TM * TN * 4 stores.
  // All of it is inlined: as a function of its own (the compiler's choice for
  // code of this size) it keeps this kernel's state in memory, and its
  // branches span more than a branch instruction reaches: their long form
  // takes the registers of the return address.
  auto finish_tile = [&](int tm) __attribute__((always_inline)) -> bool {
    epilogue_prio();
    const int m0 = tm * BM;
    using F = std::false_type;
    using T = std::true_type;
    if (fast && m0 + BM <= a.M) {
      if (var) {
        if (pj) tile_full(m0, T(), T());
        else tile_full(m0, T(), F());
      } else {
        if (pj) tile_full(m0, F(), T());
        else tile_full(m0, F(), F());
      }
      return true;
    }
    if (win) tile_any(m0, T());
    else tile_any(m0, F());
    return false;
  };

  if constexpr (SPLIT != 0) {
    for (int tm = tm0; tm < tm1; ++tm) {
      if (tm > tm0) {
        __syncthreads();  // the sums have been read: the tile's slabs may land
        ld.start(a, a_off, tm * BM, n0, ktiles, wave, lane, stage);
      }
      ld.finish(a, wave, lane, stage, acc[0][0]);
#pragma unroll
      for (int e = 0; e < 4 * NG; ++e) acc[0][0][e] += 128 * csum[0];
      (void)finish_tile(tm);
    }
  } else if constexpr (is_ring(LOADER)) {
    // Slab s of the block's sequence sits in stage s % NST; at step s the loads
    // of slab s have landed, those of s + 1 .. s + D - 1 and, issued at the
    // step, s + D are in flight, across tile ends too.  vmcnt counts in order
    // and includes the epilogues' stores: after the loads of slab s come those
    // of the next slabs and the stores of the tiles that ended within the last
    // D steps (`ends`, bit i: a full tile ended at step s - 1 - i; a partial
    // tile's stores are not counted, which only waits longer).
    constexpr int OPS = Load::kOps, STORES = TM * TN * 4;
    static_assert(D <= 3 && OPS * (D - 1) + D * STORES < 64, "vmcnt range");
    static_assert(OPS < 2 * TM * TN, "every load and the walk's step come before an MFMA of the slab");
    int8_t* cur = stage;
    int s = 0;
    unsigned ends = 0;
    // one slab; STEADY: no tile ended within the last D steps, D more to come
    auto step = [&](auto steady) __attribute__((always_inline)) {
      constexpr bool STEADY = decltype(steady)::value;
      asm volatile("" ::: "memory");  // the stores counted below stay above
      if (STEADY) {
        wait_vmcnt<OPS * (D - 1)>();
      } else if (s + D - 1 < total) {
        const int n = __builtin_popcount(ends & ((1u << D) - 1));
        if (n == 0) wait_vmcnt<OPS * (D - 1)>();
        else if (n == 1) wait_vmcnt<OPS * (D - 1) + STORES>();
        else if (n == 2) wait_vmcnt<OPS * (D - 1) + 2 * STORES>();
        else wait_vmcnt<OPS * (D - 1) + D * STORES>();
      } else {
        wait_vmcnt<0>();
      }
      ring_barrier();
      int8_t* st = cur == stage ? stage + D * ST : cur - ST;
      if (STEADY) {
        slab_mfma<TM, TN>(cur, cur + SA, wm * WROWS, wn * WCOLS, lane, acc,
                          [&](int i) __attribute__((always_inline)) {
          if (i < OPS) ld.load(a, i, st, st + SA, wave);
          else if (i == OPS) advance(ld);
          __builtin_amdgcn_sched_barrier(0);
        });
      } else {
        slab_mfma<TM, TN>(cur, cur + SA, wm * WROWS, wn * WCOLS, lane, acc,
                          [&](int i) __attribute__((always_inline)) {
          if (i == 0 && s + D < total) issue(ld, st);
        });
      }
      cur = cur == stage + D * ST ? stage : cur + ST;
      ++s;
    };
    for (int tm = tm0; tm < tm1; ++tm) {
      contraction_prio();
      acc_start();
      int kt = 0;
      while (kt < ktiles) {
        if (kt >= D) {
          // (a loop of its own: the conditions of the other steps, a dozen
          // taken branches, cost a block that waits for memory 0.14 us a slab)
          const int e = min(ktiles, kt + total - D - s);
          for (; kt < e; ++kt) step(std::true_type());
          if (kt >= ktiles) break;
        }
        step(std::false_type());
        ++kt;
        ends <<= 1;
      }
      const bool counted = finish_tile(tm);
      ends = (ktiles >= D ? 0u : ends) | (counted ? 1u : 0u);
    }
  } else {
    ld.lstore(stage, stage + SA, tid, padw);
    contraction_prio();
    acc_start();
    __syncthreads();
    int tm = tm0, kt = 0;  // tile and slab being computed
    for (int s = 0; s < total; ++s) {
      int8_t* cur = stage + (s & 1) * (SA + SB);
      int8_t* next = stage + ((s & 1) ^ 1) * (SA + SB);
      if (s + 1 < total) {
        if (ended) ld.rows(a, ++ti * BM, tid);
        ended = ld.gload(a, ktiles, tid, padw, rs_tab);
      }
      slab_mfma<TM, TN>(cur, cur + SA, wm * WROWS, wn * WCOLS, lane, acc);
      if (s + 1 < total) ld.lstore(next, next + SA, tid, padw);
      __syncthreads();
      if (++kt == ktiles) {
        kt = 0;
        (void)finish_tile(tm++);
        contraction_prio();
        if (tm < tm1) acc_start();
      }
    }
  }

  if (win) {
    // sum W^2 = 2^(2 (sigma - b0)) sum x^2, exact powers of two
    wa.V2 *= up * up;
    wa.CE[0] = ldexp(wa.CE[0], 2 * ece);
    win_write_partials_wq(wa, wq, 1, blockIdx.x, a.part_i, a.part_f, wsh);
  }
  double mn = INFINITY, mx = -INFINITY;
#pragma unroll
  for (int ni = 0; ni < TN; ++ni) {
    if (lo[ni] > hi[ni] || n0 + wn * WCOLS + ni * 32 + (lane & 31) >= a.K) continue;  // no value
    double Mc, Ac;
    epi_channel(ep, eu, n0 + wn * WCOLS + ni * 32 + (lane & 31), Mc, Ac);
    const double f0 = fmax(fma((double)lo[ni], Mc, Ac), relo);
    const double f1 = fmax(fma((double)hi[ni], Mc, Ac), relo);
    mn = fmin(mn, fmin(f0, f1));
    mx = fmax(mx, fmax(f0, f1));
  }
  // into the slots, beside the window sums (no per-block partials to finish)
  mm_slot_add(mn, mx, blockIdx.x, a.part_i);
}

// Launches one tile shape: row-tile workers times column tiles, as many blocks
// as the chip holds at once where the rows suffice (split evenly; a multiple of
// the XCDs where there are enough).
template <int BM, int BN, int LOADER>
static void pred_run(const Ctx& c, ConvArgs a) {
  auto kernel = k_cblock_pred<BM, BN, LOADER>;
  const int resident = resident_blocks(c, (const void*)kernel);
  a.ntm = (a.M + BM - 1) / BM;
  a.ntn = (a.K + BN - 1) / BN;
  int workers = imax(1, (resident > 0 ? resident : 2 * c.cus) / a.ntn);
  if (workers >= a.ntm) workers = a.ntm;
  else if (workers >= 64) workers &= ~7;
  // a thread's sums of W q, below 2^53 per tile, stay within 63 bits
  workers = imax(workers, (a.ntm + 1023) / 1024);
  a.workers = workers;
  kernel<<<workers * a.ntn, 256, 0, c.stream>>>(a);
}

// Predicted C-Block (conv + epilogue + FxP-QLayer in one contraction): the
// epilogue evaluates the window of the min / max in d_minmax (the previous
// call's) and writes the codes of the candidate the format in `out` picks;
// the decision checks the prediction and sets *miss when it fails.
hipError_t launch_conv_pred(const Ctx& c, const fxpq_conv_desc& d, const void* x, int x_type,
                            const int8_t* w, const int32_t* colsum, const SrcDev& ep, int wl,
                            int sign, int fl_lo, int fl_hi, fxpq_fmt* out, int8_t* y,
                            double* d_minmax, unsigned* miss) {
  ConvArgs a{};
  int loader;
  int cfg;
  // no 256 x 128 tiles: their 128 accumulators per thread and the window
  // state of this epilogue do not fit the registers of two blocks per CU
  dim3 grid = conv_setup(d, x, x_type, w, colsum, &ep, a, loader, cfg, c.cus, FXPQ_TILING_GEMM, false);
  split_setup(a, loader, cfg, grid, c.cus);
  a.want_mm = 1;
  a.wl = wl;
  a.sign_req = sign;
  a.fl_lo = fl_lo;
  a.fl_hi = fl_hi;
  a.mm = d_minmax;
  // deferred mode: the call's own slot set and record, no decision launch
  const int job = c.pred_jobs_n ? (*c.pred_jobs_n)++ : -1;
  const int set = job < 0 ? fls_begin(c) : 0;
  if (job < 0) {
    a.part_i = c.sc.win_part + (size_t)set * kWinSlots * kWinPart;
    a.part_f = c.sc.win_part_f + (size_t)set * kWinSlots * kWinPartF;
  } else {
    a.part_i = c.sc.pred_slots_i + (size_t)job * kWinSlots * kWinPart;
    a.part_f = c.sc.pred_slots_f + (size_t)job * kWinSlots * kWinPartF;
    a.job = c.sc.pred_jobs + job;
    a.job_miss = miss;
    a.job_per_thread = conv_per_thread(cfg);
  }
  a.fmt_win = out;
  a.y = y;
  a.y_type = FXPQ_C8;
  a.flags = c.sc.flags;
  bool timed = timer_begin(c, FXPQ_TIMER_CBLOCK_PRED);
  rgb8_setup(c, d, a, loader, false);
  switch (loader) {
    case LD_SPLIT64: pred_run<64, 64, LD_SPLIT64>(c, a); break;
    case LD_SPLIT64G: pred_run<64, 64, LD_SPLIT64G>(c, a); break;
    case LD_SPLIT32: pred_run<32, 32, LD_SPLIT32>(c, a); break;
    case LD_SPLIT32G: pred_run<32, 32, LD_SPLIT32G>(c, a); break;
    case LD_FAST64: pred_run<256, 64, LD_FAST64>(c, a); break;
    case LD_GEN16: pred_run<256, 64, LD_GEN16>(c, a); break;
    case LD_RGB8: pred_run<256, 64, LD_RGB8>(c, a); break;
    case LD_RGB4: pred_run<256, 64, LD_RGB4>(c, a); break;
    case LD_DMA64:
      if (cfg == TC_128x64) pred_run<128, 64, LD_DMA64>(c, a);
      else pred_run<128, 128, LD_DMA64>(c, a);
      break;
    default:
      if (cfg == TC_128x64) pred_run<128, 64, LD_DMA16>(c, a);
      else pred_run<128, 128, LD_DMA16>(c, a);
      break;
  }
  timer_end(c, timed, 2.0 * (double)a.M * (double)d.k * (double)(d.r * d.s * d.c));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || job >= 0) return e;
  return launch_pred_fin(c, ep, set, wl, sign, fl_lo, fl_hi, conv_per_thread(cfg), d_minmax, out,
                         miss);
}

}  // namespace fxpq
