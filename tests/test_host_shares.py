"""Invariants of the kernels' work-share arithmetic (which workgroup works on which tiles, which
workgroups share a block or a head), evaluated on the host through the library.

The kernels rely on: every tile is dealt out exactly once, in contiguous runs, those of an XCD's
workgroups balanced within one tile; a share has no more tiles than there are accumulators for; what
several workgroups finish together is shared inside one XCD."""
import ctypes as C

import pytest

from paper_2505_23219_amd import binding as B


@pytest.mark.parametrize("M", [1, 16, 64, 65, 128])
def test_which_linear_layers_are_taken(M):
    """Narrow matrices always (up to 639 tiles of 16 rows); wide ones up to what eight passes over 256
    compute units deal out in shares of 8 tiles, of 4 above 64 rows of x: 262144 and 131072 rows."""
    lib = B.lib()
    for N in (1, 16, 130, 4096, 10224, 10225, 12288, 22016, 32000, 131072, 131073, 152064, 262144, 262145, 400000):
        for K in (8, 4096, 13824):
            want = (N + 15) // 16 < 640 or N <= (262144 if M <= 64 else 131072)
            assert lib.ghd_debug_admitted(M, N, K, 256) == want, (N, K)


def test_cuts_of_known_shapes():
    """(whole tiles, tiles per share, parts, workgroups) of 7B- and 13B-shaped layers inside a step: wide
    matrices go whole-tile; output projections too up to some 30 rows of x, and in parts above; down
    projections, with their long k range, always in parts."""
    lib = B.lib()
    out = (C.c_int * 5)()
    for (M, N, K), want in [((1, 4096, 4096), [1, 1, 1, 256]), ((17, 4096, 4096), [1, 1, 1, 256]), ((64, 4096, 4096), [0, 4, 4, 256]),
                            ((1, 4096, 11008), [0, 4, 4, 256]), ((64, 4096, 11008), [0, 4, 4, 256]),
                            ((1, 5120, 5120), [1, 2, 1, 256]), ((64, 5120, 5120), [0, 5, 4, 256]), ((64, 5120, 13824), [0, 8, 6, 240]),
                            ((64, 12288, 4096), [1, 3, 1, 256]), ((64, 22016, 4096), [1, 6, 1, 256]),
                            ((128, 22016, 4096), [1, 6, 1, 256]), ((128, 32000, 4096), [1, 8, 1, 256]),
                            ((64, 40000, 4096), [1, 5, 1, 512])]:
        lib.ghd_debug_cut(M, N, K, 256, 0, out)
        assert list(out)[:4] == want, (M, N, K, list(out))


def attn_share(lib, nh, ntile, j, G, head):
    out = (C.c_int * 6)()
    lib.ghd_debug_attn_share(nh, ntile, j, G, head, out)
    return list(out)


@pytest.mark.parametrize("nh,ntile,G", [
    (32, 33, 256), (40, 129, 256), (32, 1, 256), (4, 3, 256), (2, 5, 256), (256, 2, 256), (100, 17, 256),
    (1, 40, 256), (7, 9, 256), (3, 2, 8), (5, 4, 16), (9, 3, 24), (4, 6, 7), (300, 2, 256),
])
def test_attention_share_invariants(nh, ntile, G):
    """Every (head, key tile) pair belongs to exactly one workgroup; the parts of a head are
    consecutive workgroups of one XCD, at most 64 of them (the merge keeps one part per
    lane), each with a contiguous, non-empty tile range, in order."""
    lib = B.lib()
    nx = 8 if G % 8 == 0 else 1
    Gx = G // nx
    for head in range(nh):
        parts = {}
        for j in range(G):
            first, np_, me, t0, t1, mine = attn_share(lib, nh, ntile, j, G, head)
            if not mine or me >= np_:
                continue
            parts[me] = (j, first, np_, t0, t1)
        assert parts, head
        np_ = next(iter(parts.values()))[2]
        first = next(iter(parts.values()))[1]
        assert sorted(parts) == list(range(np_)) and 1 <= np_ <= 64
        pos = 0
        for me in range(np_):
            j, f, n, t0, t1 = parts[me]
            assert (f, n) == (first, np_) and j == first + me
            assert j // Gx == first // Gx                 # one XCD
            assert t0 == pos and t1 > t0
            pos = t1
        assert pos == ntile
        sizes = [parts[me][4] - parts[me][3] for me in range(np_)]
        assert max(sizes) - min(sizes) <= 1 and sizes[-1] == min(sizes)   # the last part gets a short range


def tile_range(lib, ntiles, gx, i):
    out = (C.c_int * 2)()
    lib.ghd_debug_tile_range(ntiles, gx, i, out)
    return list(out)


@pytest.mark.parametrize("gx", [32, 2, 7, 64, 96, 256])
def test_tile_range_is_the_even_deal(gx):
    """The division-free form that the kernels evaluate, from one tile to the most that a launch has:
    XCD x has the tiles [x n / 8, (x + 1) n / 8), its workgroup w the w-th of gx equal runs of them."""
    lib = B.lib()
    for ntiles in list(range(1, 70)) + [255, 256, 257, 320, 1376, 2000, 8 * gx, 8 * gx + 1, 64 * gx, 64 * gx - 3, 16384]:
        for i in range(0, 8 * gx, 1 if gx <= 32 else 37):
            x, w = i % 8, i // 8
            i0, U = ntiles * x // 8, ntiles * (x + 1) // 8 - ntiles * x // 8
            ge = min(U, gx)                                            # workgroups that get a tile
            want = [i0 + U * w // ge, i0 + U * (w + 1) // ge] if w < ge else [0, 0]
            got = tile_range(lib, ntiles, gx, i)
            assert got == want or (got[0] == got[1] and want[0] == want[1]), (ntiles, gx, i)


@pytest.mark.parametrize("ntiles,gx", [(768, 32), (256, 32), (1376, 32), (2000, 64), (320, 32), (3, 32), (16384, 256), (41, 7)])
def test_tile_ranges_cover_every_tile_once(ntiles, gx):
    """Contiguous in workgroup order inside an XCD, balanced within one tile, nothing left out."""
    lib = B.lib()
    covered = 0
    for x in range(8):
        pos, sizes = ntiles * x // 8, []
        for w in range(gx):
            c0, c1 = tile_range(lib, ntiles, gx, w * 8 + x)
            if c0 == c1:
                continue
            assert c0 == pos and c1 > c0
            sizes.append(c1 - c0)
            pos = c1
        assert pos == ntiles * (x + 1) // 8
        covered += sum(sizes)
        if sizes:
            assert max(sizes) - min(sizes) <= 1 and len(sizes) == min(gx, sum(sizes))
    assert covered == ntiles


@pytest.mark.parametrize("M", [1, 16, 17, 33, 48, 64, 65, 96, 97, 128])
def test_linear_cut_covers_every_tile_and_fits(M):
    """How a launch is cut: whole tiles, or parts whose workgroups are all resident (at most 32
    on each XCD), with a k-step for each of eight wavefronts, of no more tiles than there are
    accumulators for."""
    lib = B.lib()
    out, grp = (C.c_int * 5)(), (C.c_int * 2)()
    for N in (1, 16, 64, 130, 1000, 1280, 4096, 5003, 5120, 10224, 10240, 22016, 32000, 262144):
        for K in (8, 40, 256, 688, 1280, 3416, 4096, 11008, 65536):
            for solo in (0, 1):
                lib.ghd_debug_cut(M, N, K, 256, solo, out)
                whole, tiles, parts, grid, rows = list(out)
                ntiles, nks = (N + 15) // 16, (K + 31) // 32
                mt = (M + 15) // 16 if M <= 64 else 6 if M <= 96 else 8
                assert 1 <= tiles <= 8 and grid % 8 == 0
                lib.ghd_debug_groups(M, N, K, 256, solo, grp)
                if whole:
                    # (groups of workgroups with different rows of x have the same tiles each)
                    gx = grid // 8 // grp[1]
                    assert parts == 1 and grid == 8 * gx * grp[1]
                    ranges = [tile_range(lib, ntiles, gx, i) for i in range(8 * gx)]
                    assert max(b - a for a, b in ranges) <= tiles
                    assert sorted(t for a, b in ranges for t in range(a, b)) == list(range(ntiles))
                    assert not rows or (solo and mt <= 4)
                else:
                    assert grp[1] == 1 and not rows and tiles * mt <= 32 and 2 <= parts <= nks // 8 and ntiles < 640
                    per_xcd = grid // 8 // parts
                    assert grid == per_xcd * parts * 8 <= 256 and per_xcd * 8 * tiles >= ntiles


@pytest.mark.parametrize("M", [1, 17, 32, 33, 37, 48, 64, 65, 80, 96, 97, 128])
def test_row_groups_cover_every_row_once(M):
    """Whole tiles dealt out to several groups of workgroups: every group has all the tiles, at most one a
    workgroup, and its own rows; together they have all rows, and none reads past the rows of
    the packed activation layout.  Narrow matrices of few tiles only, and nothing else is in groups."""
    lib = B.lib()
    cut, grp = (C.c_int * 5)(), (C.c_int * 2)()
    seen = 0
    for N in (1, 40, 300, 896, 1024, 1280, 2048, 2049, 4096, 9000, 10240):
        for K in (8, 688, 896, 3416, 11008):
            for solo in (0, 1):
                lib.ghd_debug_cut(M, N, K, 256, solo, cut)
                lib.ghd_debug_groups(M, N, K, 256, solo, grp)
                whole, tiles, parts, grid, rows = list(cut)
                mt, groups = list(grp)
                ntiles, need = (N + 15) // 16, (M + 15) // 16
                layout = 1 if need <= 1 else 2 if need <= 2 else 4 if need <= 4 else 8
                if groups == 1:
                    assert mt >= need
                    continue
                seen += 1
                assert whole and tiles == 1 and ntiles < 640 and mt in (1, 2, 4)
                assert mt * (groups - 1) < need <= mt * groups <= layout
                gx = grid // 8 // groups
                assert gx >= 2 and grid == 8 * gx * groups <= 256
                ranges = [tile_range(lib, ntiles, gx, i) for i in range(8 * gx)]
                assert sorted(t for a, b in ranges for t in range(a, b)) == list(range(ntiles))
                # (the kernel's way from a workgroup's number to its group: a multiplication)
                magic = (1 << 32) // gx + 1
                assert [(w * magic) >> 32 for w in range(gx * groups)] == [w // gx for w in range(gx * groups)]
    assert seen > 0 or M <= 16


def test_uneven_shares_of_calls_that_read_x_as_it_lies():
    """17 to 32 rows by narrow matrices of more tiles than workgroups, calls of their own: one launch in whole tiles that reads x as
    it lies while rows are few, packing and parts where that is less (or x would be packed anyway)."""
    lib, out = B.lib(), (C.c_int * 5)()
    for (M, N, K), whole in [((18, 4539, 2096), 1), ((17, 4142, 2344), 1), ((17, 5027, 2848), 1), ((18, 4503, 2712), 1), ((19, 4478, 2384), 1),
                             ((21, 4173, 2152), 1), ((17, 8748, 2848), 1), ((22, 8382, 2848), 1), ((28, 8626, 2848), 1),
                             ((28, 4966, 3080), 0), ((30, 5099, 3048), 0), ((32, 5027, 3080), 0), ((24, 5120, 5120), 0), ((26, 9375, 6256), 0)]:
        lib.ghd_debug_cut(M, N, K, 256, 1, out)
        assert out[0] == whole and out[4] == whole, (M, N, K, list(out))


def test_which_launches_take_four_k_steps_in_a_turn():
    """Workgroups of one whole tile with up to 64 rows of x, from 56 k-steps on: with single k-steps in turn calls of their own of
    5 to 16 rows were 2 to 12% slower than with a k range for each wavefront.  Nothing else."""
    lib = B.lib()
    for (M, N, K, solo), want in [((8, 4096, 11008, 1), 4), ((12, 1118, 3744, 1), 4), ((9, 3311, 4960, 1), 4), ((16, 4096, 4096, 1), 4),
                                  ((18, 1365, 2704, 1), 4), ((40, 79, 4816, 1), 4), ((35, 2882, 2872, 1), 4), ((1, 4096, 4096, 0), 4),
                                  ((8, 4096, 1792, 1), 4), ((8, 4096, 1760, 1), 1), ((8, 5000, 4096, 1), 1), ((80, 2000, 4096, 1), 1),
                                  ((64, 22016, 4096, 0), 1), ((1, 4096, 11008, 0), 1), ((3, 655, 9584, 1), 1)]:
        assert lib.ghd_debug_run(M, N, K, 256, solo) == want, (M, N, K, solo)


@pytest.mark.parametrize("tmin", [1, 2, 4])
@pytest.mark.parametrize("nh,ntile", [(32, 33), (40, 129), (32, 1), (4, 3), (256, 2), (7, 9), (1, 40), (100, 17)])
def test_attention_parts_are_not_made_too_small(nh, ntile, tmin):
    """With at least tmin tiles wanted per part: still every tile once, in order, no empty part,
    and no more parts than give each tmin tiles (the last may have fewer)."""
    lib = B.lib()
    out = (C.c_int * 6)()
    for head in range(nh):
        parts = {}
        for j in range(256):
            lib.ghd_debug_attn_share_min(nh, ntile, tmin, j, 256, head, out)
            first, np_, me, t0, t1, mine = list(out)
            if mine and me < np_:
                parts[me] = (j, first, np_, t0, t1)
        np_ = parts[0][2]
        assert sorted(parts) == list(range(np_)) and np_ <= -(-ntile // tmin)
        pos = 0
        for me in range(np_):
            j, first, n, t0, t1 = parts[me]
            assert (j, n, t0) == (first + me, np_, pos) and t1 > t0
            pos = t1
        assert pos == ntile


@pytest.mark.parametrize("n", [2, 7, 32])
def test_exchange_counts_each_launch_by_itself(n):
    """The workgroups that exchange partial results count themselves in with their XCD numbers, on a
    line that every layer of a call uses again.  Whichever XCD each launch begins with, workgroups that
    share one pass, over as many layers as a model may have; one workgroup elsewhere fails that
    launch for the others, and only that."""
    lib = B.lib()
    epochs = 48
    start = [(5 * e * e + 3 * e) % 8 for e in range(epochs)]          # another XCD from launch to launch
    xcd = [s for s in start for _ in range(n)]
    ok = (C.c_int * epochs)()
    lib.ghd_debug_exchange((C.c_int * len(xcd))(*xcd), epochs, n, ok)
    assert list(ok) == [n] * epochs
    stray = 20
    xcd[stray * n] = (xcd[stray * n] + 1) % 8
    lib.ghd_debug_exchange((C.c_int * len(xcd))(*xcd), epochs, n, ok)
    assert ok[stray] < n and [o for e, o in enumerate(ok) if e != stray] == [n] * (epochs - 1)


def test_attention_shares_are_those_of_integer_division():
    """The kernels divide by reciprocals in floats: the same heads and tile boundaries as whole-number division
    gives, over all head counts, grids and lengths that a call may have."""
    import random
    rng = random.Random(7)
    lib, out = B.lib(), (C.c_int * 6)()
    for _ in range(40000):
        nh, G, tmin = rng.randint(1, 256), 8 * rng.choice([32, rng.randint(2, 32)]), rng.choice([1, 4])
        most = (2 ** 31 - 1) // 64 // 64           # keys of 64 channels or more, offsets of 32 bits
        ntile = min(rng.choice([rng.randint(1, 70), rng.randint(1, 3000), rng.randint(1, most), most]), (2 ** 31 - 1) // nh)
        j = rng.randrange(G)
        Gx = G // 8
        x, w = j // Gx, j % Gx
        h0, h1 = nh * x // 8, nh * (x + 1) // 8
        if h0 == h1:
            continue
        head, Hx = rng.randrange(h0, h1), h1 - h0
        hl = head - h0
        lo, hi = (Hx * w // Gx, Hx * (w + 1) // Gx) if Hx >= Gx else (((w + 1) * Hx - 1) // Gx, ((w + 1) * Hx - 1) // Gx + 1)
        want = [-1] * 5 + [0]
        if lo <= hl < hi:
            first, n, me = j, 1, 0
            if Hx < Gx:
                a, b = Gx * hl // Hx, Gx * (hl + 1) // Hx
                first, n, me = x * Gx + a, min(b - a, -(-ntile // tmin)), w - a
            t = [-(-ntile * i // n) for i in (me, me + 1)] if me < n else [0, 0]
            want = [first, n, me] + t + [1]
        lib.ghd_debug_attn_share_min(nh, ntile, tmin, j, G, head, out)
        assert list(out) == want, (nh, ntile, tmin, G, j, head)


def test_rows_of_the_qkv_matrix_are_found_without_division():
    """Every row of QKV matrices of all head counts: the epilogue's arithmetic finds the part, head and position that the
    packing put there."""
    lib, out = B.lib(), (C.c_int * 6)()
    for nh in list(range(1, 42)) + [64, 100, 128, 256]:
        for d in (64, 128):
            n = 3 * nh * d
            for p in range(0, n, 4) if n < 20000 else sorted({*range(0, n, 244), *range(0, n, nh * d // 8), n - 4}):
                lib.ghd_debug_qkv_row(p, nh, d, out)
                assert list(out[:3]) == list(out[3:]), (p, nh, d, list(out))


def test_which_x_out_the_residual_stream_is_not_kept_in():
    """Copied at the end where a byte of x_out is one of x_in's, of parent[]'s or of the workspace buffer's; kept there beside them."""
    fn = B.lib().ghd_debug_x_out_copied
    fn.argtypes = [C.c_void_p, C.c_void_p, C.c_void_p, C.c_int, C.c_int, C.c_void_p, C.c_size_t]
    M, H, ws_bytes = 7, 64, 4096
    n = 4 * M * H
    far = 1 << 30
    for size, args in [(n // 2, lambda at: (at, far, far)), (4 * M, lambda at: (far, at, far)), (ws_bytes, lambda at: (far, far, at))]:
        for x in (1 << 20, 1 << 40):
            for at, meets in [(x - size, 0), (x - size + 1, 1), (x, 1), (x + n // 2, 1), (x + n - 1, 1), (x + n, 0)]:
                x_in, parent, ws = args(at)
                assert fn(x, x_in, parent, M, H, ws, ws_bytes) == meets, (size, x, at)


@pytest.fixture(params=[-1, 1])
def recip_ulps(request):
    """Reciprocals as far off as the hardware's may be."""
    B.lib().ghd_debug_recip_ulps(request.param)
    yield request.param
    B.lib().ghd_debug_recip_ulps(0)


def test_attention_shares_with_the_hardwares_reciprocals(recip_ulps):
    test_attention_shares_are_those_of_integer_division()


def test_rows_of_the_qkv_matrix_with_the_hardwares_reciprocals(recip_ulps):
    test_rows_of_the_qkv_matrix_are_found_without_division()


@pytest.mark.parametrize("ulps", [-1, 0, 1])
def test_heads_that_are_one_part(ulps):
    """Attention calls in one launch have the fewest tiles of a part at 0, a head a workgroup at most and as many workgroups as
    that takes: every head is one workgroup's, with all its tiles, whatever the head count and the length."""
    lib, out = B.lib(), (C.c_int * 6)()
    lib.ghd_debug_recip_ulps(ulps)
    try:
        for nh in range(1, 257):
            G = min(256, 8 * -(-nh // 8))
            for ntile in (1, 2, 3, 7, 12, 64, 1000, 2 ** 19 - 1):
                for head in {0, nh // 3, nh // 2, nh - 1}:
                    whole = []
                    for j in range(G):
                        lib.ghd_debug_attn_share_min(nh, ntile, 0, j, G, head, out)
                        first, n, me, t0, t1, mine = list(out)
                        if mine and me < n:
                            whole.append((first == j, n, me, t0, t1))
                        else:
                            assert t0 == t1 or not mine
                    assert whole == [(True, 1, 0, 0, ntile)], (nh, ntile, head, whole)
    finally:
        lib.ghd_debug_recip_ulps(0)
