// Kernel 2 for lattices of up to 64 * kLinearWaves units: forward / backward scores as
// scaled probabilities.
//
// The recursion of rnnt_k2_lattice.h with the scores as probabilities, not logarithms:
//   alpha(t,u) = alpha(t-1,u) p_blank(t-1,u) + alpha(t,u-1) p_label(t,u-1)
// so a step of a diagonal is two products, a lane shift and a fused multiply-add in
// float64, where the log-add costs a conversion, an exponential, a logarithm and a
// conversion back on the same dependent chain.  Every lane (one unit each) holds its score
// as m * 2^E, with E an integer that stays fixed for a chunk of 8 diagonals and is set
// anew, from m's exponent, between chunks; a neighbour's value enters times 2^(E' - E).
//
// What bounds a sweep is one wave's instruction issue (about 5 cycles an instruction) and that
// chain, so the sweeping waves do little else: each has a loader wave, which reads the cells
// of 8 frames x 8 units as whole 128-byte lines into registers, several chunks ahead, and
// writes them to LDS by diagonal; a step then reads one 16-byte row slot at a constant
// offset, with no address arithmetic and no clamping (cells outside the utterance come back
// as 0 from the bounded buffer, and 0 is the absent arc).  Kernel 2, this sweep against the
// log2 one (event-timed): losses only, B=32 T=300 U=60, 25.2 -> 19.9 us; with scores, B=16
// T=150 U=40 19.0 -> 15.4, B=32 T=250 U=80 36.5 -> 34.2 (W-Transducer 45.9 -> 36), B=64 T=500
// U=150 86.7 -> 73, B=16 T=400 U=300 182 -> 115, B=8 T=400 U=383 223 -> 132 us.  A chunk is
// ~640 cycles without scores to store, ~810 with, ~1400 with a neighbouring wave to exchange
// with.  A wave touching the weights' lines ahead of the loaders changed nothing: not memory.
//
// A chunk's scales are set from the scores four diagonals before it starts, in the shadow of
// the steps in between, so that its start costs the chain one scaling.  A wave takes its
// neighbour's values two chunks late, so that they too are in registers before their use.
//
// Exactness.  A probability below 2^-kLinearMinLog2 is stored by kernel 1 as its (negative)
// log2 instead.  When a sweep met such a weight or a NaN, when a valid score at a chunk's end
// lay outside [2^-kMinExp, 2^kMaxExp] of its lane's scale, or when some score up to 7 lanes
// upstream lay more than kMaxRise binary orders above a lane, the block sweeps again with an
// exponent of its own for every value (SLOW: no range limit, about ten times slower a step).
// What a kept sweep loses to underflow in a chunk is below 2^-1022 in some lane's scale,
// reaches another lane's scale multiplied by at most 2^kMaxRise, and valid scores there are
// at least 2^-kMinExp: 2^-40 of any of them.  A score's fall (from the middle of a chunk to the end
// of the next) is largest where the first chunks climb the labels of frame 0: under 170 on N(0, 3^2)
// logits, 240 with an alignment's symbols raised by 8 nats, 250 by 12, 320 by 16 and 390 by 20 (N(0,
// 2^2)); the rise over 7 lanes stays under 360 in all of them.  So one column has its limits at 410
// and 572 (at 320 and 662, B=4 T=500 U=20 V=64 raised by 20 nats took 200 us a call, not 50).  Across
// columns the rise is taken over up to 14 lanes, and the limits lie at 320 and 662 (at 410 and 572,
// B=8 T=300 U=200 V=64 raised by 12 nats took 296 us, not 105).
//
// Scores are stored by diagonal as before, 8 bytes a node: m with its low 24 mantissa bits
// replaced by E (28 bits of m stay: 4e-9 relative, against the ~1e-7 of the float32
// posteriors formed from them).  A sweep whose E would not fit (a path below 2^-8300000) is
// run in log2 units by one wave (lattice_sweep); the two flags of an utterance tell
// kernel 2b which of its arrays hold log2 scores.
#pragma once

#include <type_traits>

#include "rnnt_device.h"
#include "rnnt_k2_lattice.h"

namespace rnnt {

constexpr int kChunk = 8;          // diagonals per chunk; also frames and units of a loaded tile
constexpr int kTileRing = 24;      // LDS rows (diagonals) per column of 64 units
constexpr int kTilesAhead = 4;     // chunks of weights in flight in a loader's registers
constexpr int kScaleStep = 4;      // the next chunk's scales are set after this many steps
constexpr int kWaveLag = 2;        // chunks between a wave and the neighbour it takes values from
template <int NW>
constexpr int kMinExp = NW == 1 ? 410 : 320;
constexpr int kMaxExp = 450;  // with kMinExp and the weights' 2^-200: products of two scores and a weight are normal
template <int NW>
constexpr int kMaxRise = 1022 - 40 - kMinExp<NW>;  // lost terms stay below the kept ones
constexpr int kMaxScale = (1 << 23) - 4096;  // |E| of a stored score
constexpr int kNoScale = -(1 << 30);
constexpr int kLowest = static_cast<int>(0x80000000u);
static_assert(kTileRing >= 3 * kChunk - 1, "the next chunk being read and a tile being written");

// LDS barrier: this wave's global loads and stores stay in flight.
__device__ __forceinline__ void k2_lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The whole-wave shifts by one lane (0x138 up, 0x130 down); the end lane keeps `fill`, or 0.
template <int CTRL, bool ZERO = false>
__device__ __forceinline__ int wave_move(int x, int fill) {
  return __builtin_amdgcn_update_dpp(ZERO ? 0 : fill, x, CTRL, 0xf, 0xf, ZERO);
}
template <int CTRL, bool ZERO = false>
__device__ __forceinline__ double wave_move(double x, double fill) {
  const int lo = wave_move<CTRL, ZERO>(static_cast<int>(__double2loint(x)), static_cast<int>(__double2loint(fill)));
  const int hi = wave_move<CTRL, ZERO>(static_cast<int>(__double2hiint(x)), static_cast<int>(__double2hiint(fill)));
  return __hiloint2double(hi, lo);
}

// m * 2^e in a float64 and a separate integer exponent, summed without overflow.
struct Scaled {
  double m;
  int e;
};
__device__ __forceinline__ Scaled scaled_add(Scaled a, Scaled b) {
  constexpr int kNone = -(1 << 30);
  const int ea = a.m == 0.0 ? kNone : a.e + __builtin_amdgcn_frexp_exp(a.m);
  const int eb = b.m == 0.0 ? kNone : b.e + __builtin_amdgcn_frexp_exp(b.m);
  const int e = max(ea, eb);
  const int da = min(max(a.e - e, -2100), 2100), db = min(max(b.e - e, -2100), 2100);
  return Scaled{ldexp(a.m, da) + ldexp(b.m, db), e};
}

// m scaled to [0.5, 1), its exponent moved into e.
__device__ __forceinline__ Scaled scaled_norm(Scaled a) {
  const int ex = __builtin_amdgcn_frexp_exp(a.m);
  return Scaled{ldexp(a.m, -ex), a.e + ex};
}
// A weight of kernel 1's coded form (rnnt_device.h).
__device__ __forceinline__ Scaled scaled_weight(double w) {
  const double f = floor(w);
  if (w < 0.0) return Scaled{w <= 0.5 * kNoArc ? 0.0 : exp2(w - f), static_cast<int>(max(f, -1e9))};
  return Scaled{w < 0x1p-1000 ? 0.0 : w, 0};
}
__device__ __forceinline__ Scaled scaled_mul(Scaled a, Scaled b) { return Scaled{a.m * b.m, a.e + b.e}; }

typedef const volatile __attribute__((address_space(3))) u32x4* lds_volatile_u32x4;

constexpr int kTileRow = kWave * 16;  // bytes of an LDS row: one column's cells of a diagonal
template <int NW>
struct LinearShared {
  alignas(16) unsigned char tile[NW][kTileRing * kTileRow];
  // what a wave passes to its neighbour for chunk g, in slot g & 3 (slot w of the first index:
  // between waves w and w + 1; the last one is of zeros, for the wave without a neighbour): the
  // value of each step, the chunk's scale and the largest scale of the last 8 lanes; SLOW: a
  // scale per step
  alignas(16) double xch[NW][4][kChunk];
  alignas(16) int xexp[NW][4][kChunk];
  alignas(8) int xhead[NW][4][2];
  double sink[NW > 1 ? kWave + kChunk : 1];  // takes the steps' writes of the other lanes
};

// One sweep by a block of NW sweeping waves of 64 units and NW loader waves behind them;
// every thread returns whether its part has to be done in the next slower form.
template <int NW, int VAR, int MODE, bool FWD, bool SLOW>
__device__ __forceinline__ int linear_sweep(const LatticeParams& p, LinearShared<NW>& sh, int b, int T, int U) {
  constexpr int kRow = kTileRow;
  constexpr bool fwd = FWD;
  const int tid = threadIdx.x;
  const int lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const bool loader = wave >= NW;
  const int wv = loader ? wave - NW : wave;  // the column of 64 units this wave serves
  const int ub = wv * kWave;
  const int u = ub + lane;
  const int U1 = p.U_max + 1;
  const int D = T - 1 + U;
  const int n_chunk = (D + kChunk - 1) / kChunk;
  const int lag = kWaveLag * (fwd ? wv : NW - 1 - wv);  // chunks behind the first column
  const int n_round = n_chunk + kWaveLag * (NW - 1);
  const double2* __restrict__ w_utt = p.lp2 + static_cast<int64_t>(b) * p.T_max * U1;
  int bad = 0;

  if (loader) {
    // tile g: frames t0 .. t0+7 of every 8 units of the column, t0 = 8 g - 8 (u / 8) forward,
    // D - 15 - 8 g - 8 (u / 8) backward.  Lane (i, k) holds frame t0 + i, unit 8 j + k: step
    // 8 g + i + k forward, 8 g + 14 - i - k backward, so tile g and the one before hold every
    // cell of chunk g.  Frames outside [0, T) are past the buffer (a negative offset is above
    // 2^31), units past U are sent past it: they read 0.
    const __amdgpu_buffer_rsrc_t rsrc = make_buffer(w_utt, static_cast<int64_t>(T) * U1 * 16);
    const int i = lane >> 3, k = lane & 7;
    const int row_b = U1 * 16;
    const int step_g = (fwd ? kChunk : -kChunk) * row_b;
    const int step_j = 128 - kChunk * row_b;  // 8 units on, 8 frames back
    // byte offset of tile -1's cell for j = 0
    int off = ((fwd ? -kChunk : D - 15 + kChunk) - ub + i) * row_b + (ub + k) * 16;
    const int k_max = U - ub - k;  // unit 8 j + k of the column exists while 8 j <= k_max
    const int slot = fwd ? i + k : 14 - i - k;  // row of the cell after the tile's first row
    u32x4 buf[kTilesAhead][8];
    auto issue = [&](u32x4 (&x)[8]) {
#pragma unroll
      for (int j = 0; j < 8; ++j)
        x[j] = buffer_load16<false>(rsrc, 8 * j <= k_max ? off + j * step_j : kOutOfRange);
      off += step_g;
      __builtin_amdgcn_sched_barrier(0);
    };
    int ring = kTileRing - kChunk;  // first LDS row of the tile to write: tile -1 ends where chunk 0 starts
    uint32_t sign = 0;  // sign bit: some weight is in log2 form
    auto put = [&](const u32x4 (&x)[8]) {
#pragma unroll
      for (int j = 0; j < 8; ++j) sign |= x[j].y | x[j].w;
      int row = ring + slot;
      row -= row >= kTileRing ? kTileRing : 0;
      unsigned char* dst = &sh.tile[wv][row * kRow + k * 16];
#pragma unroll
      for (int j = 0; j < 8; ++j) *reinterpret_cast<u32x4*>(dst + j * 128) = x[j];
      ring += kChunk;
      ring -= ring >= kTileRing ? kTileRing : 0;
    };
    // tiles -1, 0 and 1 before the first round, then one tile a round, kTilesAhead in flight
#pragma unroll
    for (int q = 0; q < kTilesAhead; ++q) issue(buf[q]);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      put(buf[q]);
      issue(buf[q]);
    }
    k2_lds_barrier();
    k2_lds_barrier();  // chunk 0 has been read
    for (int r = 0; r < lag; ++r) k2_lds_barrier();  // the rounds before this column's first chunk
    // the sweeping wave reads chunk g + 1 ahead of its use, tile g + 2 is written; the way out leaves the loop, so
    // that the waits of the next turn count only loads that were issued on every path to it
    const int n_left = n_round - lag;
    for (int g0 = 0;; g0 += kTilesAhead) {
      bool out = false;
#pragma unroll
      for (int q = 0; q < kTilesAhead; ++q) {
        if (g0 + q >= n_left) {
          out = true;
          break;
        }
        put(buf[(q + 3) % kTilesAhead]);
        issue(buf[(q + 3) % kTilesAhead]);
        k2_lds_barrier();
      }
      if (out) break;
    }
    if (!SLOW && static_cast<int>(sign) < 0) bad = 1;
  } else {
    __builtin_amdgcn_s_setprio(3);
    const int ND = p.T_max + p.U_max;
    double* __restrict__ scores = (fwd ? p.alpha : p.beta) + static_cast<int64_t>(b) * (ND + 1) * p.u_pad;
    const __amdgpu_buffer_rsrc_t s_rsrc = make_buffer(scores, static_cast<int64_t>(ND + 1) * p.u_pad * 8);
    const int row_bytes = p.u_pad * 8;
    const Scaled w_close = scaled_weight(w_utt[static_cast<int64_t>(T - 1) * U1 + U].x);
    // a closing blank below the scales' range (its logit masked with a finite number, -1e30): the clamp of
    // scaled_weight would be the loss, and the first score has no exponent to be stored with
    if (w_close.m != 0.0 && w_close.e < -kMaxScale) bad = 1;
    const bool first_lane = fwd ? u == 0 : u == U;  // the node the sweep starts from
    const Scaled start = fwd ? Scaled{1.0, 0} : scaled_norm(w_close);
    double m = first_lane ? start.m : 0.0;
    int E = first_lane ? start.e : 0;
    Scaled acc{0.0, 0};  // W-Transducer: the sum of this lane's scores up to the chunk
    auto store_score = [&](int d, double x, int ex) {
      const int lo = (__double2loint(x) & static_cast<int>(0xff000000)) | (ex & 0xffffff);
      const u32x2 v = {static_cast<uint32_t>(lo), static_cast<uint32_t>(__double2hiint(x))};
      __builtin_amdgcn_raw_buffer_store_b64(v, s_rsrc, u * 8, __builtin_amdgcn_readfirstlane(d * row_bytes), 0);
    };
    // whether unit uu's node of diagonal d lies in the utterance
    auto valid_at = [&](int d, int uu) { return uu >= d - (T - 1) && uu <= min(d, U) && uu >= 0; };
    if (MODE != kLossOnly && first_lane) store_score(fwd ? 0 : D, m, m == 0.0 ? kZeroScore : E);
    const bool has_in = NW > 1 && (fwd ? wv > 0 : wv < NW - 1);    // a neighbour to take values from
    const bool has_out = NW > 1 && (fwd ? wv < NW - 1 : wv > 0);   // ... to pass them to
    const int in_slot = !has_in ? NW - 1 : fwd ? wv - 1 : wv;
    const int out_slot = fwd ? min(wv, NW > 1 ? NW - 2 : 0) : max(wv - 1, 0);
    const bool out_lane = has_out && lane == (fwd ? kWave - 1 : 0);
    constexpr int kToNext = fwd ? 0x138 : 0x130;  // the lane shift that brings the neighbour's value
    if (NW > 1 && wv == 0 && lane < 4 * kChunk) {
      sh.xch[NW - 1][lane / kChunk][lane % kChunk] = 0.0;
      sh.xexp[NW - 1][lane / kChunk][lane % kChunk] = 0;
      sh.xhead[NW - 1][lane / kChunk][lane & 1] = (lane & 1) ? kNoScale : 0;
    }
    int ring = 0;
    auto read_chunk = [&](double2 (&w)[kChunk]) {  // the weights of the next chunk
      const unsigned char* src = &sh.tile[wv][ring * kRow + lane * 16];
#pragma unroll
      for (int s = 0; s < kChunk; ++s) {
        // volatile: one 16-byte read, into registers of its own.  Split in two by the compiler, the
        // halves left dead registers that it gave to the steps, which then waited for the reads
        const u32x4 x = *(lds_volatile_u32x4)(src + s * kRow);
        w[s].x = __hiloint2double(static_cast<int>(x.y), static_cast<int>(x.x));
        w[s].y = __hiloint2double(static_cast<int>(x.w), static_cast<int>(x.z));
      }
      ring += kChunk;
      ring -= ring >= kTileRing ? kTileRing : 0;
    };

    const Scaled wild = VAR == 0 ? Scaled{0.0, 0}
                        : fwd    ? Scaled{u == 0 ? 1.0 : 0.0, 0}
                                 : Scaled{u != U ? 0.0 : VAR == 1 ? w_close.m : 1.0, VAR == 1 ? w_close.e : 0};
    // ^ the wild-card arcs that end where a lane has no neighbour: weight 1 from alpha(0,0) = 1 into
    // (t, 0); from (t, U) to (T-1, U) (beta = w_close) or to the final state
    int worst = 0;  // sign bit: a score or a scale out of range

    // ---- SLOW: chunk g step by step, a = (m, E) an exponent to every value
    auto slow_chunk = [&](int g, const double2 (&w)[kChunk]) {
      const int d_cur = fwd ? g * kChunk : D - g * kChunk;  // the diagonal m is of
      const int n_step = min(kChunk, D - g * kChunk);
      Scaled a{m, E};
#pragma unroll 1
      for (int s = 0; s < n_step; ++s) {
        double2 ws = w[0];
#pragma unroll
        for (int k = 1; k < kChunk; ++k) {
          ws.x = s == k ? w[k].x : ws.x;
          ws.y = s == k ? w[k].y : ws.y;
        }
        if (VAR != 0) acc = scaled_add(acc, a);
        const Scaled wl = scaled_weight(ws.y);
        const Scaled out = fwd ? scaled_mul(a, wl) : a;
        Scaled in{0.0, 0};
        if (NW > 1) {
          in.m = sh.xch[in_slot][g & 3][s];
          in.e = sh.xexp[in_slot][g & 3][s];
          if (out_lane) {
            sh.xch[out_slot][g & 3][s] = out.m;
            sh.xexp[out_slot][g & 3][s] = out.e;
          }
        }
        in = Scaled{wave_move<kToNext>(out.m, in.m), wave_move<kToNext>(out.e, in.e)};
        if (!fwd) in = scaled_mul(in, wl);
        a = scaled_norm(scaled_add(scaled_mul(a, scaled_weight(ws.x)), in));
        if (VAR != 0) a = scaled_norm(scaled_add(a, wild));
        const int d = fwd ? d_cur + 1 + s : d_cur - 1 - s;
        if (!valid_at(d, u)) a.m = 0.0;
        if (a.m != 0.0 && (a.e > kMaxScale || a.e < -kMaxScale)) bad = 1;
        if (MODE != kLossOnly) store_score(d, a.m, a.m == 0.0 ? kZeroScore : a.e);
      }
      m = a.m;
      E = a.e;
    };

    // ---- the scaled form
    // the rows of a whole chunk's steps as constant scalar offsets
    int row_off[kChunk];
#pragma unroll
    for (int q = 0; q < kChunk; ++q) row_off[q] = __builtin_amdgcn_readfirstlane(q * row_bytes);
    if (!SLOW) E = start.e;  // every lane: none but the first is reached
    double ratio = 1.0;      // 2^(the neighbour's scale - this lane's), of the chunk
    double x_in[kChunk];     // the neighbour's values for the chunk (NW > 1)
    int rise_in = kNoScale;  // its largest scale near the edge
    // a lane above U holds no node and its scale no meaning; less kNoScale the limit stays below 2^31
    // (at 2^30 - 1 a scale above 1, as W-Transducer scores reach, wrapped and sent the sweep to SLOW)
    const int rise_limit = u <= U ? kMaxRise<NW> : 1 << 29;
    auto read_in = [&](int g, double (&x)[kChunk], int& e, int& rise) {
#pragma unroll
      for (int s = 0; s < kChunk; ++s) x[s] = sh.xch[in_slot][g & 3][s];
      e = sh.xhead[in_slot][g & 3][0];
      rise = sh.xhead[in_slot][g & 3][1];
    };
    // the scores of diagonal d: valid ones must be positive, normal (class 0x100) and in range.
    // Sign bits: set in `out` where the lane has no node there, in `low` and `high` out of range
    auto check_scores = [&](int d, double x) {
      const int out = (u - (d - (T - 1))) | (min(d, U) - u);
      int ex = __builtin_amdgcn_frexp_exp(x);
      ex = __builtin_amdgcn_class(x, 0x100) ? ex : -100000;
      worst |= ((ex + kMinExp<NW>) | (kMaxExp - ex)) & ~out;
    };
    auto fast_chunk = [&](int g, const double2 (&w)[kChunk], double2 (&w_next)[kChunk], auto whole_tag) {
      constexpr bool whole = decltype(whole_tag)::value;
      const int d_cur = fwd ? g * kChunk : D - g * kChunk;  // the diagonal m is of
      const int n_step = whole ? kChunk : D - g * kChunk;
      double x_next[kChunk];
      int e_in = 0, rise_next = kNoScale;
      if (NW > 1 && whole) read_in(g + 1, x_next, e_in, rise_next);
      if (whole) read_chunk(w_next);
      const int e_bits = E & 0xffffff;
      const int chunk_off = u * 8 + (fwd ? d_cur + 1 : d_cur - kChunk) * row_bytes;
      // no node of that lane is left (its arc would keep a lane alive that no other score follows)
      const bool wild_over = fwd ? d_cur >= T - 1 : d_cur <= U;
      const double c = VAR == 0 || wild_over ? 0.0 : ldexp(wild.m, min(max(wild.e - E, -2000), 1000));
      double sum = 0.0;
      double* const x_out = out_lane ? &sh.xch[out_slot][g & 3][0] : &sh.sink[NW > 1 ? lane : 0];
      int E_next = E;
      double ratio_next = 1.0;
#pragma unroll
      for (int s = 0; s < (whole ? kChunk : kChunk - 1); ++s) {
        if (!whole && s >= n_step) break;
        const double wb = w[s].x, wl = w[s].y;
        if (VAR != 0) sum += m;
        const double t = VAR != 0 ? fma(m, wb, c) : m * wb;
        const double out = fwd ? m * wl : m;
        if (NW > 1) x_out[s] = out;
        const double k = fwd ? ratio : wl * ratio;
        if (NW > 1) x_in[s] = wave_move<kToNext>(out, x_in[s]);
        m = fma(NW > 1 ? x_in[s] : wave_move<kToNext, true>(out, 0.0), k, t);
        if (MODE != kLossOnly) {
          if (whole) {
            const int lo = (__double2loint(m) & static_cast<int>(0xff000000)) | e_bits;
            const u32x2 x = {static_cast<uint32_t>(lo), static_cast<uint32_t>(__double2hiint(m))};
            __builtin_amdgcn_raw_buffer_store_b64(x, s_rsrc, chunk_off, row_off[fwd ? s : kChunk - 1 - s], 0);
          } else {
            store_score(fwd ? d_cur + 1 + s : d_cur - 1 - s, m, E);
          }
        }
        if (whole && s == kScaleStep - 1) {
          // the next chunk's scales; lanes the sweep has not reached take the last reached one's
          const int d = fwd ? d_cur + kScaleStep : d_cur - kScaleStep;
          const int front = (fwd ? min(d, U) : max(d - (T - 1), 0)) - ub;
          E_next = E + __builtin_amdgcn_frexp_exp(m);
          int e_front = __builtin_amdgcn_readlane(E_next, min(max(front, 0), kWave - 1));
          if (NW > 1 && (fwd ? front < 0 : front >= kWave)) e_front = e_in;
          E_next = (fwd ? lane > front : lane < front) ? e_front : E_next;
          const int diff = wave_move<kToNext>(E_next, e_in) - E_next;
          ratio_next = ldexp(1.0, min(max(diff, -1100), 1000));
        }
        if (s == 0) {
          // this chunk's scales: the largest of a node up to 7 lanes upstream (across the wave's
          // edge: of the neighbour's last 8 lanes, for all of them) against each lane's
          int rise = m != 0.0 ? E : kNoScale;
#pragma unroll
          for (int q = 0; q < kChunk - 1; ++q) rise = max(rise, wave_move<kToNext>(rise, kLowest));  // one v_max with the shift in it
          if (out_lane) {
            sh.xhead[out_slot][g & 3][0] = E;
            sh.xhead[out_slot][g & 3][1] = rise;
          }
          if (NW > 1) rise = (fwd ? lane < kChunk - 1 : lane > kWave - kChunk) ? max(rise, rise_in) : rise;
          worst |= rise_limit - (rise - E);
          worst |= (kMaxScale - E) | (E + kMaxScale);
        }
      }
      check_scores(fwd ? d_cur + n_step : d_cur - n_step, m);
      if (VAR != 0) acc = scaled_add(acc, Scaled{sum, E});
      if (whole) {
        m = ldexp(m, E - E_next);
        E = E_next;
        ratio = ratio_next;
        rise_in = rise_next;
        if (NW > 1) {
#pragma unroll
          for (int s = 0; s < kChunk; ++s) x_in[s] = x_next[s];
        }
      }
    };
    double2 wa[kChunk], wb[kChunk];
    auto chunk = [&](int g, const double2 (&w)[kChunk], double2 (&w_next)[kChunk]) {
      if (SLOW) {
        read_chunk(w_next);
        slow_chunk(g, w);
      } else if (D - g * kChunk >= kChunk) {
        fast_chunk(g, w, w_next, std::true_type{});
      } else {
        fast_chunk(g, w, w_next, std::false_type{});
      }
    };
    k2_lds_barrier();  // tiles -1, 0 and 1 are in LDS
    read_chunk(wa);
    k2_lds_barrier();
    for (int r = 0; r < lag; ++r) k2_lds_barrier();  // every wave passes one a round
    if (!SLOW && NW > 1) {
      int e0;
      read_in(0, x_in, e0, rise_in);
    }
    for (int g = 0; g < n_round - lag; g += 2) {
      if (g < n_chunk) chunk(g, wa, wb);
      k2_lds_barrier();
      if (g + 1 >= n_round - lag) break;
      if (g + 1 < n_chunk) chunk(g + 1, wb, wa);
      k2_lds_barrier();
    }
    if (!SLOW && worst < 0) bad = 1;
    Scaled total{m, E};
    if (VAR != 0 && (fwd ? VAR == 1 && u == U : u == 0)) {
      // (t,U) -> (T-1,U), t <= T-2, resp. (0,0) -> (t,0), t >= 1: no later node reads the sum
      total = scaled_norm(scaled_add(total, acc));
      if (MODE != kLossOnly) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");  // after the step's store of the node
        store_score(fwd ? D : 0, total.m, total.m == 0.0 ? kZeroScore : total.e);
      }
    }
    if (fwd && u == U) {
      Scaled P = scaled_mul(total, w_close);
      if (VAR == 2) P = scaled_add(P, acc);  // (t,U) -> final
      const double lnP2 = P.m == 0.0 ? kNoArc : log2(P.m) + static_cast<double>(P.e);
      p.lnp2_fwd[b] = lnP2;
      if (p.loss_f32) p.loss_f32[b] = static_cast<float>(-lnP2 / kLog2eD);
    }
    __builtin_amdgcn_s_setprio(0);
  }
  return bad;
}

template <int NW, int VAR, int MODE>
__global__ __launch_bounds__(128 * NW) void k2_linear(LatticeParams p) {
  __shared__ LinearShared<NW> sh;
  const int b = blockIdx.x;
  const bool fwd = blockIdx.y == 0;
  const int tid = threadIdx.x;
  const int T = p.logit_lens[b];
  const int U = p.label_lens[b];
  const bool ok = T >= 1 && T <= p.T_max && U >= 0 && U <= p.U_max;
  int bad_label = 0;
  if (ok) {
    for (int u = tid; u < U; u += blockDim.x) {
      const int y = p.labels[static_cast<int64_t>(b) * p.U_max + u];
      if (y < 0 || y >= p.V || y == p.blank) bad_label = 1;
    }
  }
  bad_label = __syncthreads_or(bad_label);
  if (tid == 0) p.status[b] = (ok && !bad_label) ? 0 : 1;  // both sweeps store the same
  if (!ok || bad_label) {
    if (tid == 0 && fwd) {
      p.lnp2_fwd[b] = __builtin_nan("");
      if (p.loss_f32) p.loss_f32[b] = __builtin_nanf("");
    }
    return;  // the whole block
  }

  int bad = fwd ? linear_sweep<NW, VAR, MODE, true, false>(p, sh, b, T, U)
                : linear_sweep<NW, VAR, MODE, false, false>(p, sh, b, T, U);
  bad = __syncthreads_or(bad);
  if (bad) {
    bad = fwd ? linear_sweep<NW, VAR, MODE, true, true>(p, sh, b, T, U)
              : linear_sweep<NW, VAR, MODE, false, true>(p, sh, b, T, U);
    bad = __syncthreads_or(bad);
  }
  // the utterance's flags: in place of its backward ln P, which only the dense form reports
  if (tid == 0) reinterpret_cast<int32_t*>(p.lnp2_bwd + b)[fwd ? 0 : 1] = bad;
  if (bad && tid < kWave) {
    constexpr int K = units_per_lane(kWave * NW);
    constexpr int PF = K >= 3 ? 2 : 4;
    lattice_sweep<K, PF, VAR, MODE, kWeightsCoded, 1>(p, b, fwd ? 0 : 1, tid, T, U);
  }
}

}  // namespace rnnt
