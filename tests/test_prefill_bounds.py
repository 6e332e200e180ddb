"""CPU replay of the prefill GEMM's address arithmetic (no GPU).

For every work item of a launch and every one of its 512 threads, the index
arithmetic of ffn_prefill_kernel (work-item mapping, tile descriptor, the
one unconditional 4-byte load per thread, the packed weight loads of every K
block, the row-scale and expert-row loads with their stand-in rows, and the
output stores) is recomputed here, and each address is checked against the
size of the buffer it points into.  The same for ffn_prefill_wide_kernel (256-row
tiles, both operands asynchronously into LDS), with a simulation of the work
queues that hand out its items.  Shapes: the tiny layer, ragged tail
tiles with skewed routing, the DeepSeek-V3 prefill chunk (8192 tokens,
uniform) and the streamed path's launch over one group of G experts in
every chunk (an expert's rows of all chunks numbered as one run of launch
rows mapped to sorted positions and tokens by row tables, scales of a ring
whose end is the group's last slot).
"""
import numpy as np
import pytest

BM, BN, THREADS, XCD, TILE_BYTES, BAND_ROWS = 128, 256, 512, 8, 2048, 1024
WIDE, QUEUE_DESCS, WORKGROUPS = 256, 4, 256  # the wide kernel's rows per tile; its counters in the last entries


def _max_mtiles(R, E):
    return (R + BM - 1) // BM + min(R, E)


def _describe(chunk_offsets, n_units, max_mtiles, rows=BM):
    """prefill_tiles_kernel: per expert u its rows (one chunk: sorted positions
    [off[u], off[u+1]); several chunks: launch rows [vstart[u], vstart[u] +
    M_u), M_u summed over the chunks), the m-tile scan and the descriptors."""
    one = len(chunk_offsets) == 1
    m = [sum(int(oc[u + 1] - oc[u]) for oc in chunk_offsets) for u in range(n_units)]
    vstart = np.concatenate([[0], np.cumsum(m)]).astype(np.int64)
    cnt = [(x + rows - 1) // rows if x > 0 else 0 for x in m]
    start = np.concatenate([[0], np.cumsum(cnt)]).astype(np.int64)
    desc = {}
    for u in range(n_units):
        o0 = int(chunk_offsets[0][u]) if one else int(vstart[u])
        for b in range(start[u], start[u] + cnt[u]):
            if b < max_mtiles:
                desc[b] = (u, int(start[u]), o0, o0 + m[u])
    return start, vstart, desc


def _row_tables(chunk_offsets, n_units, chunk_rows, chunk_tokens, sorted_src, topk, vstart):
    """prefill_rows_kernel: launch row -> (sorted position, token)."""
    n = int(vstart[-1])
    pos = np.full(n, -1, np.int64)
    tok = np.full(n, -1, np.int64)
    for u in range(n_units):
        v = int(vstart[u])
        for c, oc in enumerate(chunk_offsets):
            p0, cnt = int(oc[u]), int(oc[u + 1] - oc[u])
            pp = c * chunk_rows + p0 + np.arange(cnt)
            pos[v:v + cnt] = pp
            tok[v:v + cnt] = np.asarray(sorted_src)[pp] // topk + c * chunk_tokens
            v += cnt
    assert np.all(pos >= 0)
    return pos, tok


def _tile_of(desc, n_tiles, item, rows=BM):
    e, s0, o0, o1 = desc[item // n_tiles]
    mcount = (o1 - o0 + rows - 1) // rows
    local = item - s0 * n_tiles
    kband = BAND_ROWS // rows
    band = local // (kband * n_tiles)
    width = min(kband, mcount - band * kband)
    ntx, mt = divmod(local - band * kband * n_tiles, width)
    mt += band * kband
    q = (o1 - o0 + 31) >> 5
    base, extra = divmod(q, mcount)
    first = o0 + 32 * (mt * base + min(mt, extra))
    groups = base + (1 if mt < extra else 0)
    return e, first, min(32 * groups, o1 - first), ntx


def _packed_lane_offset(h, kq, r):
    return 1024 * h + 512 * (kq & 1) + 256 * (kq >> 1) + 16 * r


def replay(gateup, E, N, K, topk, a_rows, offsets, sorted_src, R, n_chunks=1, chunk_rows=0, chunk_tokens=0,
           max_mtiles=None):
    """Checks every address one launch computes; returns the number of items run.

    E: experts of the launch (its weight stacks); offsets: [E+1] for one
    chunk, or a list of n_chunks such windows (chunk c's rows start at c *
    chunk_rows, its sorted_src entries are chunk-relative slots); a_rows:
    rows of the activation operand (tokens for gate/up, routed rows for
    down); R: rows of the sorted order (sorted_src, the row tables and the
    outputs).
    """
    nb = K // 128
    n_tiles = N // 128 if gateup else N // BN
    chunk_offsets = offsets if n_chunks > 1 else [offsets]
    if max_mtiles is None:
        max_mtiles = _max_mtiles(R, E)
    start, vstart, desc = _describe(chunk_offsets, E, max_mtiles)
    tables = n_chunks > 1
    if tables:
        row_pos, row_tok = _row_tables(chunk_offsets, E, chunk_rows, chunk_tokens, sorted_src, topk, vstart)
        assert row_pos.size <= R
    total = min(int(start[E]), max_mtiles)
    real = total * n_tiles
    grid = (max_mtiles * n_tiles + XCD - 1) // XCD * XCD
    per = (real + XCD - 1) // XCD
    tid = np.arange(THREADS)
    lane, wave = tid & 63, tid >> 6
    r32, g2 = lane & 31, lane >> 5
    scale_entries = E * (N // 128) * nb
    ran = 0
    for block in range(grid):
        slot = block // XCD
        if slot >= per:
            continue
        item = (block % XCD) * per + slot
        if item >= real:
            continue
        ran += 1
        e, m0, mc, nt = _tile_of(desc, n_tiles, item)
        assert 0 <= e < E
        assert 0 < mc <= BM and m0 >= 0 and m0 + mc <= R
        # (1) one 4-byte load per thread: a row index (sorted_src, or a row
        # table) or a weight scale; GATEUP with tables also the row's position.
        ti = np.minimum(tid, mc - 1)
        tw = np.where(tid < BM, 0, np.minimum(tid - BM, 2 * nb - 1))
        h, b = tw // nb, tw % nb
        wrow = e * (N // 128) + (nt if gateup else 2 * nt + h)
        sidx = wrow * nb + b
        has_index = gateup or tables
        uses_src = (tid < BM) & has_index
        table_len = row_pos.size if tables else R
        assert np.all(np.where(uses_src, m0 + ti < table_len, (sidx >= 0) & (sidx < scale_entries)))
        # (2) packed weights: every K block (the ring loads clamp to nb - 1).
        grp = nt * (128 // 16) + wave if gateup else nt * (BN // 16) + 2 * wave + (r32 >> 4)
        w0 = e * N * K + grp * nb * TILE_BYTES + _packed_lane_offset(0, 2 * g2, r32 & 15)
        assert np.all(w0 >= 0)
        assert np.all(w0 + (nb - 1) * TILE_BYTES + 1536 + 16 <= E * N * K)
        # (3) activation rows and their scales (stand-in rows for invalid or
        # missing ones: the tile's last row, row 0 if that one is invalid),
        # and the output rows.
        rows = np.arange(BM)
        vrow = m0 + np.minimum(rows, mc - 1)
        if tables:
            pos = row_pos[vrow]
            srow = row_tok[vrow] if gateup else pos
        else:
            pos = m0 + rows
            srow = np.asarray(sorted_src)[vrow] // topk if gateup else pos
        arow = np.where((rows < mc) & (srow >= 0) & (srow < a_rows), srow, -1)
        a_last = arow[mc - 1] if arow[mc - 1] >= 0 else 0
        ar = np.where(arow >= 0, arow, a_last)
        assert np.all((ar >= 0) & (ar < a_rows))
        assert np.all(ar * nb + (nb - 1) < a_rows * nb)                    # row-scale loads
        c = np.concatenate([tid, tid + THREADS])
        a_off = ar[c >> 3] * K + (c & 7) * 16
        assert np.all(a_off + (nb - 1) * 128 + 16 <= a_rows * K)           # expert-row loads
        orow = pos[:mc]
        assert np.all((orow >= 0) & (orow < R))
        # (4) stores of the rows below mc, at their output rows.
        if gateup:
            row = c >> 3
            live = row < mc
            q_off = orow[np.minimum(row, mc - 1)] * N + nt * 128 + (c & 7) * 16
            assert np.all(q_off[live] + 16 <= R * N)
            assert np.all(orow * (N // 128) + nt < R * (N // 128))
        else:
            for j in range(4):
                t = j * 32 + r32
                live = t < mc
                dst = orow[np.minimum(t, mc - 1)] * N + nt * BN + wave * 32 + g2 * 4
                assert np.all(dst[live] + 3 * 8 + 4 <= R * N)
    return ran


def _swz(row, c):
    return row * 128 + ((c ^ ((row >> 1) & 7)) << 4)


def drain(real, grid, rng):
    """The wide kernel's work queues: workgroups in a random order of events, each taking its place in its own
    XCD's range first, then the next of that range, then of the others.  Returns the items in the order taken."""
    assert grid % XCD == 0
    per, team = -(-real // XCD), grid // XCD
    counters, taken = [0] * XCD, []

    def at(x, i):
        return x * per + i if i < per and x * per + i < real else -1

    def take(wg):
        home = wg % XCD
        for x in [home] + [(home + d) % XCD for d in range(1, XCD)]:
            if x != home and at(x, team + counters[x]) < 0:
                continue
            i = team + counters[x]
            counters[x] += 1
            if at(x, i) >= 0:
                return at(x, i)
        return -1

    running = [(wg, at(wg % XCD, wg // XCD)) for wg in range(grid)]
    while running:
        rng.shuffle(running)
        again = []
        for wg, item in running:
            if item >= 0:
                taken.append(item)
                again.append((wg, take(wg)))  # asked for before the tile, used after it
        running = again
    return taken


def replay_wide(gateup, E, N, K, topk, a_rows, offsets, sorted_src, R, n_chunks=1, chunk_rows=0, chunk_tokens=0,
                max_mtiles=None):
    """Checks every address of a launch of wide tiles (arguments as replay); returns the number of items run."""
    nb = K // 128
    assert nb % 4 == 0 and 4 <= nb <= 64
    assert a_rows * K <= 1 << 32
    n_tiles = N // 128 if gateup else N // BN
    chunk_offsets = offsets if n_chunks > 1 else [offsets]
    table = _max_mtiles(R, E) if max_mtiles is None else max_mtiles  # entries of the workspace
    limit = table - QUEUE_DESCS                                      # the counters take the last ones
    assert QUEUE_DESCS * 16 == 2 * XCD * 4
    assert -(-R // WIDE) + min(R, E) <= limit                        # else the library takes narrow tiles
    start, vstart, desc = _describe(chunk_offsets, E, limit, WIDE)
    assert int(start[E]) <= limit
    tables = n_chunks > 1
    if tables:
        row_pos, row_tok = _row_tables(chunk_offsets, E, chunk_rows, chunk_tokens, sorted_src, topk, vstart)
    real = int(start[E]) * n_tiles
    grid = min(-(-limit * n_tiles // XCD) * XCD, WORKGROUPS)
    items = drain(real, grid, np.random.default_rng(real))
    assert sorted(items) == list(range(real))
    tid = np.arange(THREADS)
    lane, wave = tid & 63, tid >> 6
    r32, g2 = lane & 31, lane >> 5
    wr, wc = wave & 3, wave >> 2
    for item in items:
        e, m0, mc, nt = _tile_of(desc, n_tiles, item, WIDE)
        assert 0 <= e < E and 0 < mc <= WIDE and m0 >= 0 and m0 + mc <= R
        groups = (mc + 31) >> 5
        grp0 = np.where(wc == 1, (groups + 1) >> 1, 0)
        nq = np.where(wc == 1, groups >> 1, (groups + 1) >> 1)
        assert np.all(grp0 + nq <= 8) and np.all(nq <= 4)
        # (1) row indices (a sorted position's slot, or row tables), weight scales: dwords.
        ti = np.minimum((wave & 3) * 64 + lane, mc - 1)
        if gateup or tables:
            assert np.all(m0 + ti < (row_pos.size if tables else R))
        h = np.minimum(wave - 4, 1)[(wave == 4) | (wave == 5)]
        wrow = e * (N // 128) + (nt if gateup else 2 * nt + h)
        assert np.all(wrow * nb + nb - 1 < E * (N // 128) * nb)  # min(lane, nb - 1)
        # (2) weights: two 16-row groups per wave, 2 KB per K block.
        grp = nt * (128 // 16) + wave if gateup else nt * (BN // 16) + 2 * wave + 1
        w0 = (e * (N // 16) + grp) * nb * TILE_BYTES + lane * 16
        assert np.all(w0 + (nb - 1) * TILE_BYTES + 1024 + 16 <= E * N * K)
        # (3) expert rows and their scales, with stand-in rows; 32-bit offsets.
        rows = np.arange(WIDE)
        vrow = m0 + np.minimum(rows, mc - 1)
        if tables:
            pos = row_pos[vrow]
            srow = row_tok[vrow] if gateup else pos
        else:
            pos = m0 + rows
            srow = np.asarray(sorted_src)[vrow] // topk if gateup else pos
        arow = np.where((rows < mc) & (srow >= 0) & (srow < a_rows), srow, -1)
        safe = np.where(arow >= 0, arow, max(int(arow[mc - 1]), 0))
        assert np.all((safe >= 0) & (safe < a_rows))
        for i in range(4):  # waves below `groups`: 8 rows of 128 bytes per load, swizzled into LDS
            t = 32 * wave + 8 * i + (lane >> 3)
            a_off = safe[t] * K + (((lane & 7) ^ ((t >> 1) & 7)) << 4)
            live = wave < groups
            assert np.all(a_off[live] < 1 << 32)
            assert np.all(a_off[live] + (nb - 1) * 128 + 16 <= a_rows * K)
            assert np.all((wave * 4096 + i * 1024 + lane * 16 + 16)[live] <= WIDE * 128)
        s_off = safe[(wave & 3) * 64 + lane] * (nb * 4)
        live = (wave < 4) & (wave * 64 < mc)
        assert np.all(s_off[live] < 1 << 32) and np.all(s_off[live] % 16 == 0)
        assert np.all(s_off[live] + 16 * (nb // 4 - 1) + 16 <= a_rows * nb * 4)
        # (4) LDS reads of the K loop: groups grp0 .. grp0 + nq - 1 (a wave without groups reads none).
        for q in range(4):
            off = grp0 * 4096 + _swz(r32, 4 * (q >> 1) + 2 * g2 + (q & 1)) + np.maximum(nq - 1, 0) * 4096
            assert np.all(off[nq > 0] + 16 <= WIDE * 128)
        assert np.all(((grp0 + nq - 1) * 32 + r32)[nq > 0] < WIDE)
        # (5) stores of the rows below mc, at their output rows.
        orow = pos[:mc]
        assert np.all((orow >= 0) & (orow < R))
        if gateup:
            for i in range(4):
                c = tid + i * THREADS
                row = c >> 3
                live = row < mc
                assert np.all(row < WIDE)
                q_off = orow[np.minimum(row, mc - 1)] * N + nt * 128 + (c & 7) * 16
                assert np.all(q_off[live] + 16 <= R * N)
            assert np.all(orow * (N // 128) + nt < R * (N // 128))
        else:
            for b in range(4):
                t = (grp0 + b) * 32 + r32
                live = (b < nq) & (t < mc)
                dst = orow[np.minimum(t, mc - 1)] * N + nt * BN + wr * 64 + g2 * 4
                assert np.all(dst[live] + 32 + 3 * 8 + 4 <= R * N)
    return len(items)


def _routing(T, E, k, zipf_s, seed):
    rng = np.random.default_rng(seed)
    logp = np.zeros(E) if zipf_s == 0 else -zipf_s * np.log(np.arange(1, E + 1))
    g = rng.gumbel(size=(T, E))
    return np.argsort(-(logp[None, :] + g), axis=1, kind="stable")[:, :k].astype(np.int32)


def _sorted(ids, E):
    flat = ids.reshape(-1)
    order = np.argsort(flat, kind="stable").astype(np.int64)
    offsets = np.concatenate([[0], np.cumsum(np.bincount(flat, minlength=E))]).astype(np.int64)
    return offsets, order


def _run_layer(H, I, E, k, T, zipf_s, seed, replay=replay):
    ids = _routing(T, E, k, zipf_s, seed)
    offsets, src = _sorted(ids, E)
    R = T * k
    n_gu = replay(True, E, I, H, k, T, offsets, src, R)
    n_dn = replay(False, E, H, I, k, R, offsets, None, R)
    return n_gu, n_dn, offsets


@pytest.mark.parametrize("rows", [BM, WIDE])
def test_work_items_cover_every_tile_once(rows):
    """The work-item order (an expert's m-tiles in bands of 1024 rows, each band
    n-tile major) is a bijection onto (m-tile, n-tile) pairs, and an expert's
    m-tiles partition its rows, for experts of 0 to 21 m-tiles (one band, two
    and a partial third) and ragged tails."""
    rng = np.random.default_rng(3)
    m = [0, 1, 31, 128, 129, 1000, 1024, 1025, 2047, 2560] + list(rng.integers(0, 2700, 20))
    offsets = np.concatenate([[0], np.cumsum(m)]).astype(np.int64)
    for n_tiles in (1, 3, 16, 28):
        start, _, desc = _describe([offsets], len(m), 10**9, rows)
        seen = {}
        for item in range(int(start[-1]) * n_tiles):
            e, first, mc, nt = _tile_of(desc, n_tiles, item, rows)
            assert 0 <= nt < n_tiles and 0 < mc <= rows
            assert (e, first, nt) not in seen
            seen[(e, first, nt)] = mc
        for u in range(len(m)):
            for nt in range(n_tiles):
                pos = int(offsets[u])
                for f, c in sorted((f, c) for (e, f, t), c in seen.items() if e == u and t == nt):
                    assert f == pos
                    pos += c
                assert pos == int(offsets[u + 1])


@pytest.mark.parametrize("H,I,E,k,T,zipf_s", [
    (256, 128, 8, 2, 16, 0.0),        # the tiny layer
    (512, 256, 16, 4, 300, 1.2),      # ragged tails, skewed routing
    (1024, 384, 4, 4, 700, 0.0),      # k = E, several m-tiles per expert
])
def test_prefill_addresses_small_shapes(H, I, E, k, T, zipf_s):
    n_gu, n_dn, _ = _run_layer(H, I, E, k, T, zipf_s, 0)
    assert n_gu > 0 and n_dn > 0


@pytest.mark.parametrize("rows,T", [(BM, 8192), (WIDE, 8192)])
def test_prefill_addresses_deepseek_prefill_chunk(rows, T):
    """8192 tokens, uniform top-8 of 256 experts, narrow tiles (unaligned row scales) and wide ones: the last
    expert has far more than 32 rows, so its down tiles on the last n-tile reach
    the end of the scale table."""
    n_gu, n_dn, offsets = _run_layer(7168, 2048, 256, 8, T, 0.0, 0, replay if rows == BM else replay_wide)
    assert offsets[256] - offsets[255] > 32
    assert n_gu == 16 * sum(-(-int(m) // rows) for m in np.diff(offsets) if m > 0)
    assert n_dn == 28 * (n_gu // 16)


@pytest.mark.parametrize("H,I,E,k,T,zipf_s", [
    (512, 512, 16, 4, 700, 1.2),      # fewer items than workgroups, ragged tails
    (1024, 512, 5, 3, 1501, 0.0),     # a few hundred items
    (8192, 512, 4, 4, 900, 0.5),      # 64 K blocks, k = E
])
def test_wide_tile_addresses_small_shapes(H, I, E, k, T, zipf_s):
    n_gu, n_dn, _ = _run_layer(H, I, E, k, T, zipf_s, 0, replay_wide)
    assert n_gu > 0 and n_dn > 0


def test_queues_hand_out_every_item_once():
    """Ranges shorter than their workgroups, item counts that 8 does not divide, one range only, many rounds."""
    rng = np.random.default_rng(1)
    for grid in (8, 64, 256):
        for real in (0, 1, 7, 8, 9, 63, 65, 255, 256, 257, 300, 1000, 4097):
            assert sorted(drain(real, grid, rng)) == list(range(real))


@pytest.mark.parametrize("rows,T", [(BM, 1500), (WIDE, 6000)])
def test_prefill_addresses_streamed_group_over_chunks(rows, T):
    """The streamed path's launch pair of one group of G experts over all
    chunks: each chunk sorted on its own (offsets and chunk-relative slots),
    an expert's tiles spanning chunks through the row tables (the last chunk
    partial), the
    weight and scale stacks holding exactly the G experts (a group that ends
    at the ring's last slot)."""
    H, I, E, k, G, chunk = 7168, 2048, 256, 8, 16, T // 3 + 12
    ids = _routing(T, E, k, 0.8, 1)
    n_chunks = -(-T // chunk)
    offs, srcs = [], []
    for c in range(n_chunks):
        o, s = _sorted(ids[c * chunk:(c + 1) * chunk], E)
        offs.append(o)
        srcs.append(s)
    src_all = np.concatenate(srcs)       # chunk c's entries at c * chunk * k (the last chunk partial)
    R = T * k
    assert src_all.size == R
    for e0 in (0, 112, E - G):
        window = [o[e0:e0 + G + 1] for o in offs]
        mm = (R + 127) // 128 + G
        for gateup in (True, False):
            n = (replay if rows == BM else replay_wide)(
                gateup, G, I if gateup else H, H if gateup else I, k, T if gateup else R, window, src_all, R,
                n_chunks=n_chunks, chunk_rows=chunk * k, chunk_tokens=chunk, max_mtiles=mm)
            rows_u = [sum(int(o[e0 + u + 1] - o[e0 + u]) for o in offs) for u in range(G)]
            tiles = sum(-(-m // rows) for m in rows_u)
            assert n == tiles * (I // 128 if gateup else H // 256)
