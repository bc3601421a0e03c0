// Launch templates of kernel 1 (row log-normaliser and gather): row-group shape
// from V, blocking of the diagonals, and the template instance for the dtype.
// Included by the three units that instantiate one output form each
// (rnnt_launch_k1_lattice.hip, rnnt_launch_k1_rows.hip, rnnt_launch_k1_dense.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "rnnt_launch.h"

namespace rnnt {
namespace k1 {
namespace {  // each including unit keeps its own copy

// ---- kernel 1 ---------------------------------------------------------------

// Lanes per row G and interior chunks per lane NB: the smallest G*NB that
// covers a row's interior chunks (at most V / EPC of them) with NB <= 5; rows
// with more go in pieces of 64 * kPieceChunks (2, 3 and 8 chunks a lane were slower).
struct K1Shape {
  int G, NB;
  bool fast;
};

template <typename T>
K1Shape k1_shape(int V) {
  constexpr int EPC = ElemTraits<T>::kPerChunk;
  const int interior = V / EPC;
  K1Shape best{64, 5, false};
  int best_slots = 1 << 30;
  // ties go to the larger G (fewer chunks per lane; measured faster on 16-bit rows of
  // 1025, where G = 32 x NB = 4 and G = 64 x NB = 2 tie), down to two chunks per lane: at
  // one chunk a row's fixed work (geometry, boundary elements, reduction) outweighs its
  // loads, and half the lanes take it for half the cost (16-bit rows of 513, 32 x 2 against
  // 64 x 1: 59.8 against 64.6 us; float32 rows of 128, 16 x 2 against 32 x 1: 57 against 61 us)
  for (int g : {8, 16, 32, 64}) {
    for (int nb = 1; nb <= 5; ++nb) {
      const int slots = g * nb;
      if (slots >= interior && (slots < best_slots || (slots == best_slots && nb > 1))) {
        best = K1Shape{g, nb, true};
        best_slots = slots;
      }
    }
  }
  return best;
}

// one block per frame of an utterance, split into the fewest blocks of at most `cap`
// units, of equal size up to one unit (81 units: 27 + 27 + 27, not 32 + 32 + 17).  16-bit
// rows: cap = kMaxRowsPerBlock.  float32 rows: 128 KB of logits, between 32 rows (rows of
// 1025: 48 and 64 rows were slower) and kMaxRowsPerBlock: a block of 32 short rows is one
// round of its row groups, all start-up and no rows in flight (rows of 32, 301 units: K1
// 99 us in blocks of 31 rows, 51 us in blocks of 151; rows of 257, 61 units: 82 and 60 us)
// Where that leaves fewer blocks than the chip holds at once (256 CUs of eight blocks),
// blocks of more than kBlockRounds rounds of their G-lane row groups are cut further (one
// utterance, T = 200, 61 units, bf16 rows of 1025: 15.6 -> 11.7 us; two, rows of 5003:
// 64 -> 35 us; with 4096 blocks in place of 2048, 800 frames of 101 bf16 rows of 1025
// went from 24 to 28 us).
constexpr int kBlockBytes = 128 << 10;
constexpr int kFillBlocks = 2048;
constexpr int kBlockRounds = 4;
void k1_blocking(PopulateParams& p, int elem_bytes, int G) {
  int cap = kMaxRowsPerBlock;
  if (elem_bytes == 4) {
    const int64_t rows = kBlockBytes / (static_cast<int64_t>(p.V) * elem_bytes);
    cap = rows < 32 ? 32 : rows < kMaxRowsPerBlock ? static_cast<int>(rows) : kMaxRowsPerBlock;
  }
  const int U1 = p.U_max + 1;
  const int64_t frames = static_cast<int64_t>(p.B) * p.T_max;
  p.n_ublk = (U1 + cap - 1) / cap;
  const int least = kBlockRounds * (256 / G);  // rows of kBlockRounds rounds
  while (frames * p.n_ublk < kFillBlocks && (U1 + p.n_ublk - 1) / p.n_ublk > least) ++p.n_ublk;
  p.rows_per_block = (U1 + p.n_ublk - 1) / p.n_ublk;
}

constexpr int kPieceChunks = 4;

template <typename T, int G, int NB, int OUT, bool FAST, bool NT = true, bool LONG = false>
hipError_t launch_k1_g(PopulateParams p, hipStream_t stream) {
  k1_blocking(p, static_cast<int>(sizeof(T)), G);
  const int64_t blocks = static_cast<int64_t>(p.B) * p.T_max * p.n_ublk;
  const int64_t runs = (blocks + kXcdRun - 1) / kXcdRun;  // whole rounds of the XCD-major numbering
  const int64_t grid = (runs + kXcds - 1) / kXcds * kXcds * kXcdRun;
  if (grid > 0x7fffffffLL) return hipErrorInvalidConfiguration;
  hipLaunchKernelGGL((k1_populate<T, G, NB, OUT, FAST, NT, LONG>), dim3(static_cast<uint32_t>(grid)), dim3(256), 0,
                     stream, p);
  return hipGetLastError();
}

// the two load forms; the populate step on its own has no gradient after it
template <typename T, int G, int NB, int OUT, bool LONG>
hipError_t launch_k1_nt(const PopulateParams& p, hipStream_t stream) {
  if constexpr (OUT != kK1Dense) {
    if (p.keep_logits) return launch_k1_g<T, G, NB, OUT, true, false, LONG>(p, stream);
  }
  return launch_k1_g<T, G, NB, OUT, true, true, LONG>(p, stream);
}

template <typename T, int G, int OUT>
hipError_t launch_k1_nb(int nb, const PopulateParams& p, hipStream_t stream) {
  switch (nb) {
    case 1: return launch_k1_nt<T, G, 1, OUT, false>(p, stream);
    case 2: return launch_k1_nt<T, G, 2, OUT, false>(p, stream);
    case 3: return launch_k1_nt<T, G, 3, OUT, false>(p, stream);
    case 4: return launch_k1_nt<T, G, 4, OUT, false>(p, stream);
    default: return launch_k1_nt<T, G, 5, OUT, false>(p, stream);
  }
}

// A block's rows are consecutive; the fast path addresses them through one
// buffer resource with 32-bit offsets.
bool k1_span_fits(PopulateParams p, int elem_bytes) {
  k1_blocking(p, elem_bytes, 64);
  return static_cast<int64_t>(p.rows_per_block) * p.V * elem_bytes + 64 < 0x7fffffffLL;
}

template <typename T, int OUT>
hipError_t launch_k1(const PopulateParams& p, hipStream_t stream) {
  const K1Shape ks = k1_shape<T>(p.V);
  if (!k1_span_fits(p, static_cast<int>(sizeof(T)))) return launch_k1_g<T, 64, 5, OUT, false>(p, stream);
  if (!ks.fast) return launch_k1_nt<T, 64, kPieceChunks, OUT, true>(p, stream);
  switch (ks.G) {
    case 8: return launch_k1_nb<T, 8, OUT>(ks.NB, p, stream);
    case 16: return launch_k1_nb<T, 16, OUT>(ks.NB, p, stream);
    case 32: return launch_k1_nb<T, 32, OUT>(ks.NB, p, stream);
    default: return launch_k1_nb<T, 64, OUT>(ks.NB, p, stream);
  }
}

template <int OUT>
hipError_t launch_k1_dtype(rnnt_dtype_t dt, const PopulateParams& p, hipStream_t stream) {
  switch (dt) {
    case RNNT_DTYPE_F32: return launch_k1<float, OUT>(p, stream);
    case RNNT_DTYPE_BF16: return launch_k1<bf16_t, OUT>(p, stream);
    default: return launch_k1<f16_t, OUT>(p, stream);
  }
}

}  // namespace
}  // namespace k1
}  // namespace rnnt
