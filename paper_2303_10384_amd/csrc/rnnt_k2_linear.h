// Kernel 2 for lattices of up to six columns of 64 units (scaled_sweep_columns): forward / backward
// scores as scaled probabilities.
//
// The recursion of rnnt_k2_lattice.h with the scores as probabilities, not logarithms:
//   alpha(t,u) = alpha(t-1,u) p_blank(t-1,u) + alpha(t,u-1) p_label(t,u-1)
// where the log-add has a conversion, an exponential, a logarithm and a conversion back on its
// dependent chain.  Every lane (one unit each) holds its score as m * 2^e, e an integer of its own.
// A step takes the larger of its two sources' exponents and scales the two weights by what the others
// lie below it (off the chain of the scores): two products, a lane shift and a fused multiply-add, and
// an exponent's shift and maximum beside them.  Every kNormEvery steps m goes back to [0.5, 1), its
// exponent into e.
//
// Range.  There is none to be checked.  A lane whose exponent came from upstream along k <= kNormEvery arcs
// since the last normalisation also holds that path's value, so its m is at least 2^-(200 k + 1), weights being
// no less than 2^-kLinearMinLog2: a normal number, beside which what a term loses to underflow (2^-1074) is
// below 2^-270.  Smaller weights are marked (rnnt_device.h).  Chunks that meet one decode their
// weights, with exponents of their own where they are below 2^-1000, and normalise every step.
// (An exponent fixed for a chunk of eight diagonals, as this kernel had first, makes a step two instructions
// shorter, but each of its limits was met: by steep climbs on plain N(0, 3^2) logits, by alignments raised by
// 20 to 40 nats, by any marked weight; the sweep was then done again, in all 3.5 times the time.
// Checked and redone chunk by chunk, the decision at each chunk's end cost the chain 550 cycles.)
//
// What bounds a sweep is one wave's instruction issue (about 5 cycles an instruction, 14 to a step) and
// its chains, so the sweeping waves do little else: each has a loader wave, which reads the cells
// of 8 frames x 8 units as whole 128-byte lines into registers, several chunks ahead, and
// writes them to LDS by diagonal; a step then reads one 16-byte row slot at a constant
// offset, with no address arithmetic and no clamping (cells outside the utterance come back
// as 0 from the bounded buffer, and 0 is the absent arc).  A wave takes its neighbour's values two
// chunks late, so that they too are in registers before their use.
//
// Kernel 2, the log2 sweep / this one with an exponent a chunk / this one (event-timed, us): losses only, B=16
// T=400 U=60 31 / 23.5 / 26.6, U=150 47 / 45 / 48, U=300 151 / 93 / 79; with scores, B=16 T=400 U=60 38 / 28 / 30
// (W-Transducer 50 / 31 / 37), B=32 T=250 U=80 36.5 / 34.1 / 34.6 (46 / 37 / 40), B=64 T=500 U=150 73 / 82 / 81,
// B=8 T=300 U=200 60 / 56 / 59, B=16 T=400 U=300 182 / 115 / 93, B=8 T=400 U=383 223 / 223 / 106.  The same with
// symbols raised by 40 nats: 38 / 161 / 30 (U=60), 60 / 243 / 59 (U=200); T=400 U=300 on N(0, 3^2) 182 / 398 / 93.
// Blanks masked in every frame, B=8 T=600 U=120: by -inf 67 / 331 / 85, by -1e4 67 / 387 / 98.
//
// Scores are stored by diagonal as before, 8 bytes a node: m with its low 24 mantissa bits
// replaced by e (28 bits of m stay: 4e-9 relative, against the ~1e-7 of the float32
// posteriors formed from them).  An e below kLowestExp stays there, nothing beside a path probability
// above 2^kLogScoresBelow; below that the sweep is run in log2 units by one wave (lattice_sweep).  The two
// flags of an utterance tell kernel 2b which of its arrays hold log2 scores.
#pragma once

#include <type_traits>

#include "rnnt_device.h"
#include "rnnt_k2_lattice.h"

namespace rnnt {

constexpr int kChunk = 8;          // diagonals per chunk; also frames and units of a loaded tile
constexpr int kTileRing = 24;      // LDS rows (diagonals) per column of 64 units
constexpr int kTilesAhead = 4;     // chunks of weights in flight in a loader's registers
constexpr int kNormEvery = 4;      // steps between two normalisations of a score
constexpr int kWaveLag = 2;        // chunks between a wave and the neighbour it takes values from
constexpr int kLogScoresBelow = -(1 << 22);  // a path probability under 2^this has its scores in log2 units
static_assert(kChunk % kNormEvery == 0 && kNormEvery * static_cast<int>(kLinearMinLog2) < 850,
              "every wave normalises in the same steps, and m stays a normal number between two");
static_assert(kTileRing >= 3 * kChunk - 1, "the next chunk being read and a tile being written");

// LDS barrier: this wave's global loads and stores stay in flight.
__device__ __forceinline__ void k2_lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The whole-wave shifts by one lane (0x138 up, 0x130 down); the end lane keeps `fill`.
template <int CTRL>
__device__ __forceinline__ int wave_move(int x, int fill) {
  return __builtin_amdgcn_update_dpp(fill, x, CTRL, 0xf, 0xf, false);
}
template <int CTRL>
__device__ __forceinline__ double wave_move(double x, double fill) {
  const int lo = wave_move<CTRL>(static_cast<int>(__double2loint(x)), static_cast<int>(__double2loint(fill)));
  const int hi = wave_move<CTRL>(static_cast<int>(__double2hiint(x)), static_cast<int>(__double2hiint(fill)));
  return __hiloint2double(hi, lo);
}

// Sum without overflow; a zero's exponent does not count.
__device__ __forceinline__ Scaled scaled_add(Scaled a, Scaled b) {
  const int ea = a.m == 0.0 ? kNoScale : a.e + __builtin_amdgcn_frexp_exp(a.m);
  const int eb = b.m == 0.0 ? kNoScale : b.e + __builtin_amdgcn_frexp_exp(b.m);
  const int e = max(ea, eb);
  const int da = min(max(a.e - e, -2100), 2100), db = min(max(b.e - e, -2100), 2100);
  return Scaled{ldexp(a.m, da) + ldexp(b.m, db), e};
}

// m scaled to [0.5, 1), its exponent moved into e.
__device__ __forceinline__ Scaled scaled_norm(Scaled a) {
  const int ex = __builtin_amdgcn_frexp_exp(a.m);
  return Scaled{ldexp(a.m, -ex), a.e + ex};
}
__device__ __forceinline__ Scaled scaled_mul(Scaled a, Scaled b) { return Scaled{a.m * b.m, a.e + b.e}; }

typedef const volatile __attribute__((address_space(3))) u32x4* lds_volatile_u32x4;

// A tile's weight as the loader leaves it: a log2 (-1 and below) as -m 2^0 with m = 2^fraction in [1, 2],
// whose float32 leaves the low 29 bits free, and minus its exponent in them; any other as it is.
__device__ __forceinline__ void split_log2(uint32_t& lo, uint32_t& hi) {
  const double w = __hiloint2double(static_cast<int>(hi), static_cast<int>(lo));
  const double f = floor(w);
  const double m = max(static_cast<double>(fast_exp2(static_cast<float>(w - f))), 1.0);
  const int e = static_cast<int>(max(f, static_cast<double>(kLowestWeight)));
  const bool is_log2 = w <= -1.0;
  lo = is_log2 ? static_cast<uint32_t>(-e) : lo;
  hi = is_log2 ? static_cast<uint32_t>(__double2hiint(m)) | 0x80000000u : hi;
}
// ... as mantissa and exponent.  LOG2S: some weight of the tile is a log2.
template <bool LOG2S>
__device__ __forceinline__ Scaled tile_weight(double w) {
  const bool is_log2 = LOG2S && w <= -1.0;
  const int lo = __double2loint(w);
  Scaled o{__hiloint2double(__double2hiint(w) & 0x7fffffff, is_log2 ? 0 : lo), is_log2 ? -lo : 0};
  const bool none = o.m < 0x1p-1010;
  o.m = none ? 0.0 : o.m;
  o.e = none ? kNoWeight : o.e;
  return o;
}

constexpr int kTileRow = kWave * 16;  // bytes of an LDS row: one column's cells of a diagonal
template <int NW>
struct LinearShared {
  alignas(16) unsigned char tile[NW][kTileRing * kTileRow];
  alignas(8) int marked[NW][4][2];  // of chunk g's tiles, in slot g & 3: some weight is marked, some is a log2
  // what a wave passes to its neighbour in the steps of chunk g, in slot g & 3 (slot w of the first
  // index: between waves w and w + 1; the last one for the wave without a neighbour)
  alignas(16) double xch[NW][4][kChunk];
  alignas(16) int xexp[NW][4][kChunk];
  // takes the steps' writes of the other lanes
  double sink[NW > 1 ? kWave + kChunk : 1];
  int sink_exp[NW > 1 ? kWave + kChunk : 1];
};

// One sweep by a block of NW sweeping waves of 64 units and NW loader waves behind them;
// every thread returns whether the sweep has to be done in log2 units.
template <int NW, int VAR, int MODE, bool FWD>
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
    // byte offset of tile -1's cell for j = 0; unsigned, the longest utterances' frames past T lie above 2^31 too
    uint32_t off = static_cast<uint32_t>(((fwd ? -kChunk : D - 15 + kChunk) - ub + i)) * static_cast<uint32_t>(row_b) +
                   static_cast<uint32_t>((ub + k) * 16);
    const int k_max = U - ub - k;  // unit 8 j + k of the column exists while 8 j <= k_max
    const int slot = fwd ? i + k : 14 - i - k;  // row of the cell after the tile's first row
    u32x4 buf[kTilesAhead][8];
    auto issue = [&](u32x4 (&x)[8]) {
#pragma unroll
      for (int j = 0; j < 8; ++j)
        x[j] = buffer_load16<false>(
            rsrc, 8 * j <= k_max ? static_cast<int>(off + static_cast<uint32_t>(j * step_j)) : kOutOfRange);
      off += static_cast<uint32_t>(step_g);
      __builtin_amdgcn_sched_barrier(0);
    };
    int ring = kTileRing - kChunk;  // first LDS row of the tile to write: tile -1 ends where chunk 0 starts
    int n_put = 0;
    uint32_t top_before = 0;
    auto put = [&](const u32x4 (&x)[8]) {
      uint32_t top = 0;  // the largest upper word: marked weights have the sign bit, log2 ones are -1 and below
#pragma unroll
      for (int j = 0; j < 8; ++j) top = max(top, max(x[j].y, x[j].w));
      const uint32_t both = max(top, top_before);  // tile g completes chunk g
      const bool any_marked = __builtin_amdgcn_ballot_w64(both >= 0x80000000u) != 0;
      const bool any_log2 = __builtin_amdgcn_ballot_w64(both >= 0xbff00000u) != 0;
      if (lane == 0) {
        sh.marked[wv][(n_put + 3) & 3][0] = any_marked;
        sh.marked[wv][(n_put + 3) & 3][1] = any_log2;
      }
      top_before = top;
      ++n_put;
      int row = ring + slot;
      row -= row >= kTileRing ? kTileRing : 0;
      unsigned char* dst = &sh.tile[wv][row * kRow + k * 16];
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(top >= 0xbff00000u) != 0, 0)) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          uint32_t y[4] = {x[j].x, x[j].y, x[j].z, x[j].w};
          split_log2(y[0], y[1]);
          split_log2(y[2], y[3]);
          *reinterpret_cast<u32x4*>(dst + j * 128) = u32x4{y[0], y[1], y[2], y[3]};
        }
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j) *reinterpret_cast<u32x4*>(dst + j * 128) = x[j];
      }
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
  } else {
    __builtin_amdgcn_s_setprio(3);
    const int ND = p.T_max + p.U_max;
    double* __restrict__ scores = (fwd ? p.alpha : p.beta) + static_cast<int64_t>(b) * (ND + 1) * p.u_pad;
    const __amdgpu_buffer_rsrc_t s_rsrc = make_buffer(scores, static_cast<int64_t>(ND + 1) * p.u_pad * 8);
    const int row_bytes = p.u_pad * 8;
    const Scaled w_close = scaled_weight(w_utt[static_cast<int64_t>(T - 1) * U1 + U].x);
    const bool first_lane = fwd ? u == 0 : u == U;  // the node the sweep starts from
    const Scaled start = fwd ? Scaled{1.0, 0} : scaled_norm(w_close);
    // the score of the diagonal reached, m * 2^e; a lane the sweep has not reached holds 0
    double m = first_lane ? start.m : 0.0;
    int e = first_lane && m != 0.0 ? max(start.e, kLowestExp) : kNoScale;
    Scaled acc{0.0, 0};  // W-Transducer: the sum of this lane's scores up to the chunk
    auto score_words = [&](double x, int ex) {  // the stored form
      const int lo = (__double2loint(x) & static_cast<int>(0xff000000)) | (ex & 0xffffff);
      return u32x2{static_cast<uint32_t>(lo), static_cast<uint32_t>(__double2hiint(x))};
    };
    auto store_score = [&](int d, double x, int ex) {
      __builtin_amdgcn_raw_buffer_store_b64(score_words(x, ex), s_rsrc, u * 8,
                                            __builtin_amdgcn_readfirstlane(d * row_bytes), 0);
    };
    if (MODE != kLossOnly && first_lane) store_score(fwd ? 0 : D, m, e);
    const bool has_in = NW > 1 && (fwd ? wv > 0 : wv < NW - 1);    // a neighbour to take values from
    const bool has_out = NW > 1 && (fwd ? wv < NW - 1 : wv > 0);   // ... to pass them to
    const int in_slot = !has_in ? NW - 1 : fwd ? wv - 1 : wv;
    const int out_slot = fwd ? min(wv, NW > 1 ? NW - 2 : 0) : max(wv - 1, 0);
    const bool out_lane = has_out && lane == (fwd ? kWave - 1 : 0);
    constexpr int kToNext = fwd ? 0x138 : 0x130;  // the lane shift that brings the neighbour's value
    // what enters where there is no neighbour: nothing, or a wild-card arc: of weight 1 from
    // alpha(0,0) = 1 into (t, 0); from (t, U) to (T-1, U) (beta = w_close) or to the final state
    const Scaled edge = fwd && VAR != 0 ? Scaled{1.0, 0} : Scaled{0.0, kNoScale};
    const Scaled final_arc = VAR == 1 ? w_close : Scaled{1.0, 0};
    if (NW > 1 && wv == 0 && lane < 4 * kChunk) {
      sh.xch[NW - 1][lane / kChunk][lane % kChunk] = edge.m;
      sh.xexp[NW - 1][lane / kChunk][lane % kChunk] = edge.e;
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

    double x_in[kChunk];  // the neighbour's values for the chunk (NW > 1)
    int e_in[kChunk];
    auto read_in = [&](int g, double (&x)[kChunk], int (&ex)[kChunk]) {
#pragma unroll
      for (int s = 0; s < kChunk; ++s) {
        x[s] = sh.xch[in_slot][g & 3][s];
        ex[s] = sh.xexp[in_slot][g & 3][s];
      }
    };
    // the rows of a whole chunk's steps as constant scalar offsets
    int row_off[kChunk];
#pragma unroll
    for (int q = 0; q < kChunk; ++q) row_off[q] = __builtin_amdgcn_readfirstlane(q * row_bytes);

    double in = edge.m;  // lane 0 resp. 63 keep theirs: the shifts write over it
    int ei = edge.e;

    // Chunk g, n_step diagonals of it.  WHOLE: all kChunk.  MARKED: some weights are (1) marked, (2) log2s; then
    // all are decoded in the steps, with exponents of their own, and every step normalises its score.
    auto steps = [&](int g, const double2 (&w)[kChunk], int n_step, auto whole_tag, auto marked_tag) {
      constexpr bool WHOLE = decltype(whole_tag)::value;
      constexpr int MARKED = decltype(marked_tag)::value;
      const int d_cur = fwd ? g * kChunk : D - g * kChunk;  // the diagonal m is of
      const int store_off = u * 8 + (fwd ? d_cur + 1 : d_cur - kChunk) * row_bytes;
      double* const x_out = out_lane ? &sh.xch[out_slot][g & 3][0] : &sh.sink[NW > 1 ? lane : 0];
      int* const e_out = out_lane ? &sh.xexp[out_slot][g & 3][0] : &sh.sink_exp[NW > 1 ? lane : 0];
      double sum = 0.0;  // of m, in e's scale
#pragma unroll
      for (int s = 0; s < kChunk; ++s) {
        if (!WHOLE && s >= n_step) break;
        Scaled wb{w[s].x, 0}, wl{w[s].y, 0};
        int n;
        if (MARKED != 0) {
          wb = tile_weight<MARKED == 2>(w[s].x);
          wl = tile_weight<MARKED == 2>(w[s].y);
        }
        if (VAR != 0) {
          if (MARKED != 0) acc = scaled_add(acc, Scaled{m, e});
          else sum += m;
        }
        const double out = fwd ? m * wl.m : m;
        const int et = e + wb.e, eo = fwd ? e + wl.e : e;
        if (NW > 1) {
          x_out[s] = out;
          e_out[s] = eo;
          in = x_in[s];
          ei = e_in[s];
        }
        in = wave_move<kToNext>(out, in);
        ei = wave_move<kToNext>(eo, ei);
        // the scaling goes into the weights, off the chain of the scores (the exponents' own chain does not wait
        // for them between normalisations)
        if (fwd || VAR != 0) {
          double r = fwd ? in : in * wl.m;
          int er = fwd ? ei : ei + wl.e;
          if (!fwd) {  // the label arc that unit U lacks
            r = u == U ? final_arc.m : r;
            er = u == U ? final_arc.e : er;
          }
          n = max(et, er);
          m = fma(r, ldexp(1.0, er - n), m * ldexp(wb.m, et - n));
        } else {
          const int er = ei + wl.e;
          n = max(et, er);
          m = fma(in, ldexp(wl.m, er - n), m * ldexp(wb.m, et - n));
        }
        if (VAR != 0 && MARKED == 0) sum = ldexp(sum, et - n);
        e = n;
        if (MARKED != 0 || s % kNormEvery == kNormEvery - 1) {
          const int ex = __builtin_amdgcn_frexp_exp(m);
          const bool none = m == 0.0;
          if (VAR != 0 && MARKED == 0) {
            if (s == kChunk - 1) acc = scaled_add(acc, Scaled{sum, e});
            else sum = ldexp(sum, -ex);  // of up to four scores, m above 2^-802: no overflow
          }
          m = __builtin_amdgcn_frexp_mant(m);
          e = none ? kNoScale : max(e + ex, kLowestExp);
        }
        if (MODE != kLossOnly) {
          if (WHOLE)
            __builtin_amdgcn_raw_buffer_store_b64(score_words(m, e), s_rsrc, store_off, row_off[fwd ? s : kChunk - 1 - s],
                                                  0);
          else
            store_score(fwd ? d_cur + 1 + s : d_cur - 1 - s, m, e);
        }
      }
    };
    double2 wa[kChunk], wb[kChunk];
    int marked = 0, log2s = 0;  // of the chunk ahead's weights
    using std::integral_constant;
    auto chunk = [&](int g, const double2 (&w)[kChunk], double2 (&w_next)[kChunk]) {
      if (D - g * kChunk >= kChunk) {
        double x_next[kChunk];
        int e_next[kChunk];
        if (NW > 1) read_in(g + 1, x_next, e_next);
        read_chunk(w_next);
        const int marked_next = sh.marked[wv][(g + 1) & 3][0], log2s_next = sh.marked[wv][(g + 1) & 3][1];
        if (__builtin_expect(marked == 0, 1)) {
          steps(g, w, kChunk, std::true_type{}, integral_constant<int, 0>{});
        } else {
          if (log2s == 0) steps(g, w, kChunk, std::true_type{}, integral_constant<int, 1>{});
          else steps(g, w, kChunk, std::true_type{}, integral_constant<int, 2>{});
        }
        marked = __builtin_amdgcn_readfirstlane(marked_next);
        log2s = __builtin_amdgcn_readfirstlane(log2s_next);
        if (NW > 1) {
#pragma unroll
          for (int s = 0; s < kChunk; ++s) {
            x_in[s] = x_next[s];
            e_in[s] = e_next[s];
          }
        }
      } else {
        steps(g, w, D - g * kChunk, std::false_type{}, integral_constant<int, 2>{});  // the last one, whatever its weights
      }
    };
    k2_lds_barrier();  // tiles -1, 0 and 1 are in LDS
    read_chunk(wa);
    marked = __builtin_amdgcn_readfirstlane(sh.marked[wv][0][0]);
    log2s = __builtin_amdgcn_readfirstlane(sh.marked[wv][0][1]);
    k2_lds_barrier();
    for (int r = 0; r < lag; ++r) k2_lds_barrier();  // every wave passes one a round
    if (NW > 1) read_in(0, x_in, e_in);
    for (int g = 0; g < n_round - lag; g += 2) {
      if (g < n_chunk) chunk(g, wa, wb);
      k2_lds_barrier();
      if (g + 1 >= n_round - lag) break;
      if (g + 1 < n_chunk) chunk(g + 1, wb, wa);
      k2_lds_barrier();
    }
    Scaled total{m, e};
    if (VAR != 0 && (fwd ? VAR == 1 && u == U : u == 0)) {
      // (t,U) -> (T-1,U), t <= T-2, resp. (0,0) -> (t,0), t >= 1: no later node reads the sum
      total = scaled_norm(scaled_add(total, acc));
      if (MODE != kLossOnly) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");  // after the step's store of the node
        store_score(fwd ? D : 0, total.m, total.m == 0.0 ? kNoScale : total.e);
      }
    }
    // below 2^kLogScoresBelow the scores' stored exponents would not do (nor the clamps of the weights'
    // and scores' exponents far below that)
    if (fwd && u == U) {
      Scaled P = scaled_mul(total, w_close);
      if (VAR == 2) P = scaled_add(P, acc);  // (t,U) -> final
      const double lnP2 = P.m == 0.0 ? kNoArc : log2(P.m) + static_cast<double>(P.e);
      p.lnp2_fwd[b] = lnP2;
      if (p.loss_f32) p.loss_f32[b] = static_cast<float>(-lnP2 / kLog2eD);
      bad = P.m != 0.0 && lnP2 < kLogScoresBelow;
    }
    if (!fwd && u == 0) bad = total.m != 0.0 && total.e + __builtin_amdgcn_frexp_exp(total.m) < kLogScoresBelow;
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

  int bad = fwd ? linear_sweep<NW, VAR, MODE, true>(p, sh, b, T, U) : linear_sweep<NW, VAR, MODE, false>(p, sh, b, T, U);
  bad = __syncthreads_or(bad);
  // the utterance's flags: in place of its backward ln P, which only the dense form reports
  if (tid == 0) reinterpret_cast<int32_t*>(p.lnp2_bwd + b)[fwd ? 0 : 1] = bad;
  if (bad && tid < kWave) {
    constexpr int K = units_per_lane(kWave * NW);
    constexpr int PF = K >= 3 ? 2 : 4;
    lattice_sweep<K, PF, VAR, MODE, kWeightsCoded, 1>(p, b, fwd ? 0 : 1, tid, T, U);
  }
}

}  // namespace rnnt
