"""Host-side model of the kernels' grids and index arithmetic (no GPU).

Before any launch, this checks for every workload shape that each block of
each kernel only addresses memory inside the buffers it is given, that the
gradient kernel's chunk -> (row, column) mapping reproduces the flat index
exactly, and that 32-bit intermediates cannot overflow.  The formulas mirror
the launch code in csrc/rnnt_api.hip and the kernels' index expressions.
"""
import os
import re

import numpy as np
import pytest

from paper_2303_10384_amd.workloads import WORKLOADS

_CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2303_10384_amd", "csrc")
_K1_SRC = os.path.join(_CSRC, "rnnt_k1_populate.h")
# consecutive populate blocks per XCD turn, as the kernel source defines it
K1_XCD_RUN = int(re.search(r"#define RNNT_K1_XCD_RUN (\d+)", open(_K1_SRC).read()).group(1))
# whether sweeps of 65..256 units run one unit per lane over several wavefronts
K2_MULTI_WAVE = int(re.search(r"#define RNNT_K2_MULTI_WAVE (\d+)",
                              open(os.path.join(_CSRC, "rnnt_launch_k2.h")).read()).group(1))


def units_per_lane(U1):
    return next(k for k in (1, 2, 3, 4, 6, 8, 12, 16, 24, 32) if U1 <= 64 * k)


def sweep_shape(U1):
    """(wavefronts per sweep, units per lane) of the lattice sweeps."""
    K = units_per_lane(U1)
    return (K, 1) if K2_MULTI_WAVE and K in (2, 3, 4) else (1, K)

EPC = {"f32": 4, "bf16": 8, "f16": 8}
SHAPES = [(w.B, w.T_max, w.U_max, w.V, w.dtype) for w in WORKLOADS.values()] + [
    (3, 7, 0, 2, "f32"), (2, 5, 4, 3, "bf16"), (1, 1, 1023, 5, "f32"), (4, 9, 63, 4097, "f16"),
    (5, 3, 64, 7, "bf16"), (2, 2, 127, 8, "f32"), (2, 4, 300, 6, "f32"), (1, 3, 700, 5, "bf16"),
    (1, 2, 1023, 3, "bf16"), (1, 3, 1535, 4, "f32"), (1, 2, 2047, 3, "bf16"), (3, 7, 5, 4100, "f32"), (3, 7, 5, 8200, "bf16"), (3, 7, 5, 2600, "f16")]


def _constant(path, name):
    """The value of `constexpr int name = ...;` (whole numbers, shifts and products of them)."""
    expr = re.search(r"constexpr int %s = ([0-9 <*]+);" % name, open(os.path.join(_CSRC, path)).read()).group(1)
    return int(eval(expr, {"__builtins__": {}}))


K1_BLOCK_BYTES = _constant("rnnt_launch_k1.h", "kBlockBytes")
K1_FILL_BLOCKS = _constant("rnnt_launch_k1.h", "kFillBlocks")
K1_BLOCK_ROUNDS = _constant("rnnt_launch_k1.h", "kBlockRounds")
K1_PIECE_CHUNKS = _constant("rnnt_launch_k1.h", "kPieceChunks")
K1_MAX_ROWS = _constant("rnnt_k1_populate.h", "kMaxRowsPerBlock")


def k1_shape(V, epc):
    """(lanes per row, interior chunks per lane, whether a row fits the registers of one)."""
    interior = V // epc
    best, best_slots = (64, 5, False), 1 << 30
    for g in (8, 16, 32, 64):
        for nb in range(1, 6):
            if g * nb >= interior and (g * nb < best_slots or (g * nb == best_slots and nb > 1)):
                best, best_slots = (g, nb, True), g * nb
    return best


def k1_blocking(B, T, U, V, esz, G):
    """(blocks a frame, rows a block at most)."""
    cap = K1_MAX_ROWS if esz != 4 else min(max(K1_BLOCK_BYTES // (V * esz), 32), K1_MAX_ROWS)
    U1 = U + 1
    n_ublk = -(-U1 // cap)
    while B * T * n_ublk < K1_FILL_BLOCKS and -(-U1 // n_ublk) > K1_BLOCK_ROUNDS * (256 // G):
        n_ublk += 1
    return n_ublk, -(-U1 // n_ublk)


@pytest.mark.parametrize("run", sorted({1, K1_XCD_RUN, 16}))
@pytest.mark.parametrize("B,T,U,V,dt", SHAPES)
def test_populate_kernel_addresses(B, T, U, V, dt, run):
    epc = EPC[dt]
    esz = {"f32": 4, "bf16": 2, "f16": 2}[dt]
    n_elem = B * T * (U + 1) * V
    G, NB, fast = k1_shape(V, epc)
    pieces = not fast  # rows past the registers go in pieces of 64 * K1_PIECE_CHUNKS interior chunks
    if pieces:
        G, NB = 64, K1_PIECE_CHUNKS
    n_ublk, rows_per_block = k1_blocking(B, T, U, V, esz, G)  # equal blocks up to one unit
    assert 1 <= rows_per_block <= K1_MAX_ROWS and n_ublk * rows_per_block >= U + 1
    # (a frame cut to few rounds may end in blocks past its units: they return at once)
    blocks = B * T * n_ublk
    grid = -(-(-(-blocks // run)) // 8) * 8 * run
    assert grid < 2**31
    # XCD-major numbering: physical block i (XCD i % 8, its k-th block, k = i // 8) ->
    # logical ((k // run) * 8 + i % 8) * run + k % run, a bijection onto [0, blocks) once
    # the logical numbers >= blocks (the grid's round-up) are dropped
    i = np.arange(grid, dtype=np.int64)
    k = i // 8
    lb = ((k // run) * 8 + i % 8) * run + k % run
    kept = np.sort(lb[lb < blocks])
    assert np.array_equal(kept, np.arange(blocks))
    # the launcher checks the span with blocks of 64-lane groups, the largest that long rows have
    fast = k1_blocking(B, T, U, V, esz, 64)[1] * V * esz + 64 < 0x7fffffff
    # every row a block can reach with full lengths (t < T, u <= U)
    b, t, u = np.meshgrid(np.arange(B), np.arange(T), np.arange(U + 1), indexing="ij")
    b, t, u = b.ravel(), t.ravel(), u.ravel()
    row = (b.astype(np.int64) * T + t) * (U + 1) + u
    e0 = row * V
    c0 = e0 // epc
    mis = e0 - c0 * epc
    nch = (mis + V + epc - 1) // epc
    assert np.all((c0 + nch - 1) * epc < n_elem)
    assert np.all(e0 + V <= n_elem)
    whole = c0 + nch <= n_elem // epc
    assert np.all(((c0 + nch) * epc <= n_elem)[whole])
    if fast:
        # interior chunks [kf, kl] fit G*NB lanes-chunks; every clamped index stays in [0, nch)
        first_partial = mis != 0
        last_partial = (mis + V) % epc != 0
        kf = first_partial.astype(np.int64)
        kl = nch - 1 - last_partial.astype(np.int64)
        if pieces:  # lane k0 + 64 q of piece pc: every interior chunk once, the others past the buffer
            n_pc = -(-(V // epc) // (64 * NB))
            assert np.all(kl - kf + 1 <= n_pc * 64 * NB) and np.all(kl - kf + 1 > (n_pc - 1) * 64 * NB - epc)
            assert int(nch.max() + n_pc * 64 * NB) * 16 < 2**31  # k * 16 in 32 bits, from an offset past the buffer too
        else:
            assert np.all(kl - kf + 1 <= G * NB)
        assert np.all(np.maximum(kl, 0) < nch) and np.all(kf <= nch)
    # only rows reaching into the tensor's final partial chunk read element-wise
    assert np.all((e0 + V > (n_elem // epc) * epc)[~whole])
    if fast:
        # per-block buffer: from the first chunk of the block's first row (unit u_lo) to
        # the end of its last row; row j of the block at element e_rel0 + j * V
        ublk = u // rows_per_block
        u_lo = ublk * rows_per_block
        n_rows = np.minimum(rows_per_block, U + 1 - u_lo)
        j = u - u_lo
        row_lo = (b.astype(np.int64) * T + t) * (U + 1) + u_lo
        e_first = row_lo * V
        c_base = e_first // epc
        c_end = (e_first + n_rows * V + epc - 1) // epc
        assert np.all((c_end - c_base) * 16 < 2**31)
        e_rel = (e_first - c_base * epc) + j * V
        assert np.array_equal(e_rel, e0 - c_base * epc)
        off0 = (e_rel - mis) * esz
        assert np.all(off0 >= 0) and np.all(off0 + nch * 16 <= (c_end - c_base) * 16)
        assert np.all(e_rel * esz < 2**31)
        # rows per block fit the LDS arrays
        assert n_rows.max() <= 256
    # lattice-form writes at the row index, inside the B * T * (U+1) cell arrays
    assert row.max() < B * T * (U + 1) and row.min() >= 0


# (logits, gradient): a chunk is 16 bytes of the gradient, 128 threads a block where that is float32
GRADS = [(*s, s[4]) for s in SHAPES] + [(*s, "f32") for s in SHAPES if s[4] != "f32"]


@pytest.mark.parametrize("B,T,U,V,dt,gdt", GRADS)
def test_gradient_kernel_chunk_mapping(B, T, U, V, dt, gdt):
    epc = EPC[gdt]
    n_elem = B * T * (U + 1) * V
    n_rows = B * T * (U + 1)
    tile = (128 if gdt == "f32" else 256) * 2  # threads x chunks per thread
    chunks = -(-n_elem // epc)
    blocks = -(-chunks // tile)
    assert blocks < 2**31
    rng = np.random.default_rng(0)
    blk = np.unique(np.concatenate([np.arange(min(blocks, 64)), np.arange(max(0, blocks - 64), blocks),
                                    rng.integers(0, blocks, size=256)])).astype(np.int64)
    tile0 = blk * tile
    e_tile = tile0 * epc
    r_tile = e_tile // V
    v_tile = e_tile - r_tile * V
    assert np.all(v_tile < V)
    for cl in (0, 1, tile // 2 - 1, tile // 2, tile - 1):
        c = tile0 + cl
        e0 = c * epc
        live = e0 < n_elem
        off = v_tile + cl * epc
        assert np.all(off < 2**32)
        # split_row: e / V as a product with the rounded 1 / V, at most one off
        q = (e_tile.astype(np.float64) * (1.0 / V)).astype(np.int64)
        assert np.all(np.abs(q - r_tile) <= 1)
        dr = off // V
        r = r_tile + dr
        v = off - dr * V
        assert np.all((r * V + v)[live] == e0[live])
        assert np.all(r[live] < n_rows)
        if V >= epc:
            split = v + epc > V
            # the second row of a split chunk exists unless the chunk runs past the end
            assert np.all(((r + 1 < n_rows) | (e0 + epc > n_elem))[live & split])


@pytest.mark.parametrize("B,T,U,V,dt", SHAPES)
def test_lattice_kernel_addresses(B, T, U, V, dt):
    """Log2 sweep (the loss past six columns of units, rnnt_lattice_scores, and a scaled sweep's fallback): weights of any step e read at the cell clamped into the utterance,
    diagonal ec = clamp(e, 0, D), unit clamp(u, ec - (T_b-1), min(ec, U_b)), a valid cell,
    stored at its row (b, ec - u, u);
    alpha stored in row min(d, D+1), beta in row d (or the spare row ND when d < 0), each row
    u_pad = 64*K wide; the posterior kernel reads alpha, beta only at diagonals <= D."""
    U1 = U + 1
    ND = T + U
    NW, K = sweep_shape(U1)
    u_pad = 64 * units_per_lane(U1)
    assert NW * 64 * K == u_pad  # unit u in column u whatever the waves
    n_cells = B * T * U1  # kernel 1's lattice form: one cell per logits row
    n_scores = B * (ND + 1) * u_pad
    lanes = np.concatenate([w * 64 * K + np.arange(64) * K for w in range(NW)])  # each lane's first unit
    for Tb, Ub in [(T, U), (1, 0), (max(1, T // 2), U // 2), (1, U), (T, 0)]:
        D = Tb - 1 + Ub
        PF = 1 if K >= 24 else 2 if K >= 16 else min(24, 48 // K)
        for bb in {0, B - 1}:
            for e in range(-PF - 2, D + PF + 2):  # every diagonal a load or store step can name
                ec = min(max(e, 0), D)
                for k in range(K):
                    uc = np.minimum(np.maximum(lanes + k, ec - (Tb - 1)), min(ec, Ub))
                    tc = ec - uc
                    assert np.all((tc >= 0) & (tc < Tb) & (uc >= 0) & (uc <= Ub))  # a cell kernel 1 wrote
                    w = (bb * T + tc) * U1 + uc  # row (t, u) of utterance bb
                    assert np.all(w >= 0) and np.all(w < n_cells)
                    rows = []
                    if 1 <= e <= D + PF - 1:  # forward steps d = 1 .. (last block's end)
                        rows.append(min(e, D + 1))
                    if -PF + 1 <= e <= D - 1:  # backward steps d = D-1 .. (last block's end)
                        rows.append(e if e >= 0 else ND)
                    for row in rows:
                        a = (bb * (ND + 1) + row) * u_pad + lanes + k
                        assert np.all(a >= 0) and np.all(a < n_scores)
        # spare rows never overlap the rows the posterior kernel reads (d <= D)
        assert D + 1 <= ND


@pytest.mark.parametrize("NW", [2, 3, 4])
@pytest.mark.parametrize("D", [0, 1, 23, 24, 25, 47, 48, 330, 649])
def test_lattice_multi_wave_schedule(NW, D):
    """Several wavefronts per sweep: wave w runs segment g = r - lag(w) of PF steps in round r
    (lag w forward, NW-1-w backward) and every wave passes one barrier per round.  Each value a
    wave takes from its neighbour (slot [pair][r-1 & 1][s] in round r) was written by that
    neighbour in round r-1 for the same diagonal, and is not overwritten before it is read; the
    LDS slots stay inside [NW-1][2][PF]."""
    PF = 24  # one unit per lane
    n_seg = (D + PF - 1) // PF
    n_rounds = n_seg + NW - 1
    for sweep in ("forward", "backward"):
        writes = {}  # (pair, half, s) -> list of (round, diagonal)
        reads = []   # (round, pair, half, s, diagonal)
        active = {w: 0 for w in range(NW)}
        for r in range(n_rounds):  # the same trip count for every wave: equal barrier counts
            for w in range(NW):
                lag = w if sweep == "forward" else NW - 1 - w
                g = r - lag
                if not (0 <= g < n_seg):
                    continue
                active[w] += 1
                for s in range(PF):
                    d = 1 + g * PF + s if sweep == "forward" else D - 1 - g * PF - s
                    producer = w < NW - 1 if sweep == "forward" else w > 0
                    consumer = w > 0 if sweep == "forward" else w < NW - 1
                    if producer:
                        pair = w if sweep == "forward" else w - 1
                        assert 0 <= pair < NW - 1
                        writes.setdefault((pair, r & 1, s), []).append((r, d))
                    if consumer:
                        pair = w - 1 if sweep == "forward" else w
                        assert 0 <= pair < NW - 1
                        reads.append((r, pair, (r - 1) & 1, s, d))
        assert all(n == n_seg for n in active.values())  # every wave runs every segment once
        for r, pair, half, s, d in reads:
            # the latest write to the slot before round r: made in round r-1, for diagonal d
            before = [(rw, dw) for rw, dw in writes.get((pair, half, s), []) if rw < r]
            assert before and before[-1] == (r - 1, d)
            # and the next write to that slot comes after round r's barrier
            assert all(rw > r for rw, _ in writes[(pair, half, s)] if rw >= r)


@pytest.mark.parametrize("T,U", [(1, 0), (2, 0), (5, 0), (1, 7), (2, 1), (30, 17), (250, 80), (24, 0), (25, 23),
                                 (500, 150), (3, 255), (40, 300), (7, 700), (3, 1000), (2, 1535), (9, 2047)])
def test_wildcard_sums_take_each_frame_once(T, U):
    """W-Transducer sweeps: the owning lane stores the value of step s of a segment in LDS
    slot s, and after the segment lane s adds it to its own sum when the step's diagonal is
    in range.  Every frame's term enters exactly once: alpha(t, U) for t <= T-2 (forward;
    t = 0 from the start when U = 0) and beta(t, 0) for 1 <= t <= T-1 (backward; t = T-1
    from the start when U = 0), and the stash and sink indices stay inside their arrays."""
    nw, K = sweep_shape(U + 1)
    PF = 1 if K >= 24 else 2 if K >= 16 else min(24, 48 // K)
    D = T - 1 + U
    n_seg = (D + PF - 1) // PF
    fwd, bwd = [], []
    if U == 0 and T >= 2:
        fwd.append(0)
        bwd.append(T - 1)
    for g in range(n_seg):
        d0f, d0b = 1 + g * PF, D - 1 - g * PF
        for lane in range(64):
            for s_ in range(PF):
                assert 0 <= lane + s_ < 64 + PF  # the sink of the lanes without a value
            if lane < PF:  # min(lane, PF - 1) is the slot read; lanes >= PF add nothing
                d = d0f + lane
                if U <= d <= U + T - 2:
                    fwd.append(d - U)
                d = d0b - lane
                if 1 <= d <= T - 1:
                    bwd.append(d)
    assert sorted(fwd) == list(range(0, T - 1))
    assert sorted(bwd) == list(range(1, T))


@pytest.mark.parametrize("B,T,U,V,dt,gdt", GRADS)
def test_gradient_kernel_fast_path_buffer(B, T, U, V, dt, gdt):
    """Blocks on the buffer-load path: no partial chunk inside, a per-block buffer of at
    most one tile (offsets fit 32 bits), every live chunk's offset inside it, dead chunks
    past its end; the row-record indices of dead chunks are clamped into the records."""
    epc = EPC[gdt]
    chunk_bytes = epc * {"f32": 4, "bf16": 2, "f16": 2}[dt]  # of logits: 16, or 8 under a float32 gradient
    assert chunk_bytes in (8, 16)
    n_elem = B * T * (U + 1) * V
    n_rows = B * T * (U + 1)
    tile = (128 if gdt == "f32" else 256) * 2  # threads x chunks per thread
    n_chunks = -(-n_elem // epc)
    n_full = n_elem // epc
    blocks = -(-n_chunks // tile)
    for blk in sorted(b for b in {0, 1, blocks // 2, blocks - 2, blocks - 1} if 0 <= b < blocks):
        tile0 = blk * tile
        general = V < epc or (n_elem % epc != 0 and tile0 + tile > n_full)
        if general:
            # at most the last block holds the partial chunk
            assert V < epc or blk == blocks - 1
            continue
        tile_bytes = min(tile, n_full - tile0) * chunk_bytes
        assert 0 < tile_bytes <= tile * chunk_bytes < 2**31
        cl = np.arange(tile)
        live = tile0 + cl < n_full
        assert np.all((cl * chunk_bytes < tile_bytes) == live)
        e_tile = tile0 * epc
        r_tile, v_tile = e_tile // V, e_tile % V
        r = np.minimum(r_tile + (v_tile + cl * epc) // V, n_rows - 1)
        assert np.all(r >= 0) and np.all(np.minimum(r + 1, n_rows - 1) < n_rows)
    assert 0x80000000 > tile * 16  # the out-of-range offset lies past every block's buffer


@pytest.mark.parametrize("B,T,U,V,dt", SHAPES)
def test_posterior_kernel_tiles_cover_every_row_once(B, T, U, V, dt):
    """Posterior kernel: block (b, tile) walks item i -> t = t0 + i % 8, d = t0 + i // 8, u = d - t
    over 8 * (7 + U + 1) items; kept items (t < min(t0+8, T), 0 <= u <= U) are every row once."""
    TT = 8
    U1 = U + 1
    n_tiles = -(-T // TT)
    assert B * n_tiles < 2**31
    seen = np.zeros((T, U1), np.int64)
    for tile in range(n_tiles):
        t0 = tile * TT
        i = np.arange(TT * (TT - 1 + U1))
        t = t0 + i % TT
        d = t0 + i // TT
        u = d - t
        keep = (t < min(t0 + TT, T)) & (u >= 0) & (u <= U)
        np.add.at(seen, (t[keep], u[keep]), 1)
        # consecutive items of one diagonal are consecutive cells (coalesced loads)
        assert np.all(np.diff(u[:TT]) == -1)
    assert np.all(seen == 1)


@pytest.mark.parametrize("B,T,U,V,dt", SHAPES)
def test_viterbi_kernel_addresses(B, T, U, V, dt):
    """Forced-alignment kernel: decision words stored at row min(d, D+1), one per lane slot (K a
    row) or one per wave (NW a row); the backtrace stages blocks of 64 diagonals, lane l loading
    the words of diagonal 64 w + l at byte offset ((64 w + l) cols + c) * 8: never negative, and past
    the utterance's (T_max+U_max+1)*cols words only beyond the last row (a buffer load there reads
    0), under 2^31 bytes."""
    U1 = U + 1
    ND = T + U
    NW, K = sweep_shape(U1)
    cols = units_per_lane(U1)  # decision words per diagonal: one per lane slot, or one per wave
    assert cols == (NW if NW > 1 else K)
    words = (ND + 1) * cols
    lanes = np.arange(64)
    for Tb, Ub in [(T, U), (1, 0), (max(1, T // 2), U // 2), (1, U), (T, 0)]:
        D = Tb - 1 + Ub
        PF = 1 if K >= 24 else 2 if K >= 16 else min(24, 48 // K)
        for d in range(1, D + PF):
            row = min(d, D + 1)
            for wv in range(NW):
                for lane in range(64):
                    assert 0 <= row * cols + (wv if NW > 1 else min(lane, K - 1)) < words
        # unit u's word column and bit: (u % K, u // K) in one wave, (u // 64, u % 64) over several
        for u in range(Ub + 1):
            c, bit = (u // 64, u % 64) if NW > 1 else (u % K, u // K)
            assert 0 <= c < cols and 0 <= bit < 64
        for w in range(D // 64 + 1):
            for k in range(cols):
                idx = (64 * w + lanes) * cols + k
                assert np.all(idx >= 0) and np.all(idx * 8 < 2 ** 31)
                # a word past the stored rows is a diagonal past ND: masked off by the walk (d <= D)
                assert np.all((idx < words) | (64 * w + lanes > ND))


def _walk_by_diagonal(dec, t, U, var):
    """The backtrace one diagonal per step (the plain definition): at node (t, u) a set bit
    means entered by the label arc (or, at u = 0, by the initial wild-card arc)."""
    u, start, frames = U, 0, {}
    while t + u > 0:
        bit = dec[t + u][u]
        label = u > 0 and (bit or t == 0)
        jumped = var != 0 and bit and u == 0
        if label:
            frames[u - 1] = t
            u -= 1
        elif jumped:
            start = t
            break
        else:
            t -= 1
    return frames, start


def _walk_by_label_moves(dec, t, U, var, ND):
    """The kernel's backtrace: one step per label move, unit u's bits over a block of 64
    diagonals taken as one 64-bit mask (the ballot), the highest set bit in [max(u, 1), d]."""
    u, start, frames = U, 0, {}
    d = t + u
    w = d // 64
    steps = 0
    while d > 0 and (var != 0 or u > 0):
        steps += 1
        if d < 64 * w:
            w -= 1
            assert d >= 64 * w  # at most one block down per step
        base = 64 * w
        bits = 0
        for lane in range(64):
            if base + lane <= ND and dec[base + lane][u]:
                bits |= 1 << lane
        lo, hi = max(u, 1) - base, d - base
        assert lo <= hi <= 63
        m = bits & ((1 << (hi + 1)) - 1) & ~((1 << max(lo, 0)) - 1)
        if u > 0:
            if m:
                dl = base + m.bit_length() - 1
            elif u >= base:
                dl = u
            else:
                d = base - 1
                continue
            frames[u - 1] = dl - u
            u -= 1
            d = dl - 1
        else:
            if m:
                start = base + m.bit_length() - 1
                break
            d = base - 1
    assert steps <= U + (t + U) // 64 + 1
    return frames, start


@pytest.mark.parametrize("var", [0, 1, 2])
@pytest.mark.parametrize("T,U,density", [(1, 0, 0.5), (3, 1, 0.5), (7, 5, 0.2), (70, 3, 0.05), (5, 130, 0.9),
                                         (200, 80, 0.3), (150, 150, 0.5), (64, 64, 0.0), (65, 63, 1.0)])
def test_viterbi_walk_by_label_moves(var, T, U, density):
    """The block-ballot backtrace reaches the same frames and start frame as the walk one
    diagonal at a time, on random decision bits (any bits define a valid walk)."""
    rng = np.random.default_rng(T * 1000 + U + var)
    ND = T - 1 + U
    for _ in range(5):
        dec = rng.random((ND + 65, U + 1)) < density
        for t_end in {T - 1, max(0, T // 2)}:
            assert _walk_by_label_moves(dec, t_end, U, var, ND) == _walk_by_diagonal(dec, t_end, U, var)


@pytest.mark.parametrize("U_max,columns", [(0, 1), (63, 1), (64, 2), (127, 2), (128, 3), (192, 4), (255, 4), (256, 5),
                                           (319, 5), (320, 6), (383, 6), (384, 0), (2047, 0)])
def test_columns_of_the_scaled_sweep(U_max, columns):
    """Which sweep a lattice takes depends on its padded units alone: the GPU tests' shapes of up to 383 units
    reach one to six columns of the scaled sweep whatever their frames."""
    import paper_2303_10384_amd as P
    assert P.load_library().rnnt_scaled_sweep_columns(U_max) == columns


CHUNK = _constant("rnnt_k2_linear.h", "kChunk")
RING = _constant("rnnt_k2_linear.h", "kTileRing")
WAVE_LAG = _constant("rnnt_k2_linear.h", "kWaveLag")
NOTHING = (-1, -1)  # a cell that was never written, or holds the 0 of an offset past the buffer


class ScaledSweep:
    """One sweep of the scaled form: which cells its loaders put where in LDS between which barriers, and
    what its sweeping waves read.  A phase is the work between two barriers."""

    def __init__(self, T_max, U_max, T, U, fwd):
        self.NW = (U_max + 64) // 64
        self.T, self.U, self.U1, self.D, self.fwd = T, U, U_max + 1, T - 1 + U, fwd
        self.size = T * self.U1 * 16
        self.n_chunk = -(-self.D // CHUNK)
        self.n_round = self.n_chunk + WAVE_LAG * (self.NW - 1)

    def lag(self, wv):
        return WAVE_LAG * (wv if self.fwd else self.NW - 1 - wv)

    def tile(self, wv, g):
        """Cells of tile g: [(LDS row after the tile's first, unit in the column, (frame, unit) or NOTHING)]."""
        lane = np.arange(64)
        i, k = lane >> 3, lane & 7
        ub, row_b = wv * 64, self.U1 * 16
        off = ((-CHUNK if self.fwd else self.D - 15 + CHUNK) - ub + i) * row_b + (ub + k) * 16
        off = off + (g + 1) * (CHUNK if self.fwd else -CHUNK) * row_b
        slot = i + k if self.fwd else 14 - i - k
        cells = []
        for j in range(8):
            o = off + j * (128 - CHUNK * row_b)
            assert np.all((o > -2**31) & (o < 2**32))  # unsigned 32 bits: below 0 is at or above 2^31
            exists = 8 * j <= self.U - ub - k
            unsigned = np.where(exists, o, 0x80000000) & 0xffffffff  # as the buffer's bounds check sees it
            inside = unsigned < self.size
            frame = (self.D - 15 - CHUNK * g if not self.fwd else CHUNK * g) - ub - 8 * j + i
            unit = ub + 8 * j + k
            assert np.array_equal(inside, exists & (frame >= 0) & (frame < self.T))
            assert np.all(unit[inside] <= self.U) and np.array_equal((o // row_b)[inside], frame[inside])
            assert np.array_equal((o % row_b // 16)[inside], unit[inside])
            for n in range(64):
                cells.append((int(slot[n]), int(8 * j + k[n]), (int(frame[n]), int(unit[n])) if inside[n] else NOTHING))
        return cells

    def check_column(self, wv):
        lag, ring = self.lag(wv), {}
        marks = {}
        n_left = self.n_round - lag
        # loader: tiles -1, 0, 1 in phase 0, tile g + 2 in the round of chunk g
        puts = [(0, -1), (0, 0), (0, 1)] + [(2 + lag + g, g + 2) for g in range(n_left)]
        # sweeping wave: chunk 0 in phase 1, chunk g + 1 in the round of chunk g where that is whole
        reads = [(1, 0)] + [(2 + lag + g, g + 1) for g in range(min(n_left, self.n_chunk)) if self.D - CHUNK * g >= CHUNK]
        phases = {}
        for ph, g in puts:
            phases.setdefault(ph, ([], []))[0].append(g)
        for ph, g in reads:
            phases.setdefault(ph, ([], []))[1].append(g)
        for ph in sorted(phases):
            written = set()
            new = {}
            for g in phases[ph][0]:
                first = RING - CHUNK + (g + 1) * CHUNK
                for slot, col, cell in self.tile(wv, g):
                    assert 0 <= slot <= 14 and 0 <= col < 64
                    key = ((first + slot) % RING, col)
                    assert key not in written or ph == 0
                    written.add(key)
                    new[key] = cell
                marks[g & 3] = (ph, g)
            for g in phases[ph][1]:
                for s in range(CHUNK):
                    row = (g * CHUNK + s) % RING
                    d = g * CHUNK + s if self.fwd else self.D - 1 - g * CHUNK - s
                    for col in range(64):
                        u = wv * 64 + col
                        t = d - u
                        want = (t, u) if 0 <= t < self.T and u <= self.U else NOTHING
                        assert (row, col) not in written, "a row is written while it is read"
                        got = ring.get((row, col), NOTHING)
                        if g * CHUNK + s < self.D or want == NOTHING:  # a step of the sweep, or nothing there
                            assert got == want, (wv, g, s, u, got, want)
                # its marks were left by tile g, in an earlier phase
                assert marks[g & 3][1] == g and marks[g & 3][0] < ph
            ring.update(new)
        # barriers: two before the rounds, the rounds before the first chunk, one a round
        assert 2 + lag + n_left == 2 + self.n_round

    def check_exchange(self):
        """A wave reads the slot of chunk g + 1 in the round of chunk g (and slot 0 before its first round): written by
        its neighbour for that chunk, in an earlier phase, and not written again meanwhile."""
        for wv in range(self.NW):
            src = wv - 1 if self.fwd else wv + 1
            if not 0 <= src < self.NW:
                continue
            lag, lag_src = self.lag(wv), self.lag(src)
            writes = {2 + lag_src + g: g for g in range(min(self.n_round - lag_src, self.n_chunk))}
            wanted = [(2 + lag, 0)] if self.n_chunk else []
            wanted += [(2 + lag + g, g + 1) for g in range(min(self.n_round - lag, self.n_chunk))
                       if self.D - CHUNK * g >= CHUNK and g + 1 < self.n_chunk]
            for ph, g in wanted:
                before = [(p, c) for p, c in writes.items() if c % 4 == g % 4 and p < ph]
                assert before and max(before)[1] == g
                assert writes.get(ph, g + 1) % 4 != g % 4

    def check_stores(self, T_max, U_max):
        """Every step stores a row of its utterance's scores, in the columns the waves own."""
        u_pad = 64 * units_per_lane(U_max + 1)
        assert 64 * self.NW <= u_pad and (T_max + U_max + 1) * u_pad * 8 < 2**31
        for g in range(self.n_chunk):
            d_cur = CHUNK * g if self.fwd else self.D - CHUNK * g
            n = min(CHUNK, self.D - CHUNK * g)
            for s in range(n):
                d = d_cur + 1 + s if self.fwd else d_cur - 1 - s
                assert 0 <= d <= self.D <= T_max + U_max
                if n == CHUNK:  # a constant row offset from the chunk's first row
                    assert d == (d_cur + 1 if self.fwd else d_cur - CHUNK) + (s if self.fwd else CHUNK - 1 - s)


@pytest.mark.parametrize("T,U", [(1, 0), (1, 7), (2, 1), (9, 0), (8, 1), (17, 63), (16, 64), (30, 65), (25, 127), (40, 192),
                                 (3, 256), (33, 320), (11, 383), (90, 9), (57, 70)])
def test_scaled_sweep_tiles_and_exchange(T, U):
    """Every step reads the weights of its own cell, 0 where it has none; no LDS row is overwritten before it is
    read or while it is; the exchange and the marks likewise; all waves pass the same barriers; utterances of the
    padded shape, of one frame, without units and ending inside an earlier column."""
    for T_b, U_b in {(T, U), (1, U), (T, 0), (max(1, T // 2), U // 2), (max(1, T - 3), max(0, U - 1))}:
        for fwd in (True, False):
            m = ScaledSweep(T, U, T_b, U_b, fwd)
            for wv in range(m.NW):
                m.check_column(wv)
            m.check_exchange()
            m.check_stores(T, U)


def test_scaled_sweep_of_the_longest_utterances():
    """Byte offsets of the loaders stay in 32 bits, past the buffer where they should be, at the largest
    shapes the library takes (T_max * (U_max + 1) * 16 and the scores' rows under 2^31 bytes)."""
    for U_max in (0, 63, 64, 383):
        u_pad = 64 * units_per_lane(U_max + 1)
        T = min((2**31 - 1) // (16 * (U_max + 1)), (2**31 - 1) // (u_pad * 8) - U_max - 1)
        for fwd in (True, False):
            m = ScaledSweep(T, U_max, T, U_max, fwd)
            for wv in {0, m.NW - 1}:
                for g in (-1, 0, 1, m.n_chunk // 2, m.n_chunk - 1, m.n_round + 1, m.n_round + 3):
                    m.tile(wv, g)
