"""The launches that calls become, on the CPU: the engine's host code against a stand-in for the
HIP runtime that notes every launch."""
import os

import pytest

from paper_2601_20309_amd import binding as B
from tests import launches as L

pytestmark = pytest.mark.skipif(not os.path.exists(L.HIPCC), reason="needs hipcc")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    return L.build(str(tmp_path_factory.mktemp("launches")))


def test_two_launches_at_once_both_take_shares_or_neither(exe):
    """Both directions by a kernel each: fixed shares on both sides up to 24 rounds of each
    side's waves, else drawn steps beyond 8 rounds; vectors of 8 bytes, configured launches and chunks
    of layers of 1 MiB and more always by 8; a launch that has the link to itself by 24, one that carries both ways by 8."""
    zero = B.KV_PATH_ZEROCOPY

    def drawn(out_kib, in_kib, dim, **kw):
        block = 4 * dim * kw.get("layers", 1)
        kw = {"path": zero, **kw}
        got = L.launches(exe, [L.move(out_kib * 1024 // block, in_kib * 1024 // block, dim, **kw)])[0]
        return [x["drawn"] for x in got]

    whole = 2048                                                               # segments of 4 KiB: rounds of 288 KiB each way
    assert drawn(3000, 3000, whole) == [0, 0]
    assert drawn(24 * 288, 24 * 288, whole) == [0, 0]
    assert drawn(24 * 288, 24 * 288 + 8, whole) == [1, 1]
    assert drawn(24 * 288 + 8, 24 * 288, whole) == [1, 1]
    assert drawn(7000, 5000, whole) == [1, 1]
    assert drawn(7000, 2304, whole) == [1, 0]                                  # 8 rounds in: over before it matters
    assert drawn(7000, 2312, whole) == [1, 1]
    assert drawn(24 * 192, 2 * 24 * 192, whole) == [1, 1]                      # in-heavy: rounds of 192 KiB out and of 288 in
    assert drawn(16 * 192, 24 * 288, whole) == [0, 0]
    assert drawn(6000, 6000, whole, layers=8, chunk_layers=4) == [1] * 4       # 3000 KiB a launch, layer by layer
    assert drawn(1800, 1800, whole, layers=8, chunk_layers=4) == [0] * 4       # under 1 MiB: rounds of 64 and 96 KiB
    assert drawn(2000, 2000, 420, host_layout=1) == [1, 1]                     # 840-byte segments: 8-byte vectors
    assert drawn(3000, 3000, whole, vecs_per_lane=2, wg_lanes=64) == [1, 1]
    assert drawn(1500, 0, whole) == [0] and drawn(0, 2200, whole) == [0]
    assert drawn(1700, 0, whole) == [1] and drawn(0, 2400, whole) == [1]
    assert drawn(1000, 1000, whole, path=B.KV_PATH_AUTO) == [0] and drawn(1200, 1200, whole, path=B.KV_PATH_AUTO) == [1]


def test_more_waves_for_tiles_of_512_bytes(exe):
    """8-byte vectors in tiles of 64: what comes in alone gets 1.5 times the waves, both ways only
    where groups are several tiles no more than a third empty (segments of a layer-first pool; blocks of a block-first one)."""
    def waves(seg, out_mib, in_mib, **kw):
        kw = {"host_layout": 1, "layers": 4, **kw}
        block = 2 * kw["layers"] * seg
        return L.launches(exe, [L.move((out_mib << 20) // block, (in_mib << 20) // block, seg // 2, **kw)])[0][0]["waves"]

    def base(table, vecs, tiles):
        return int(table * 1.4 / (vecs / (64 * tiles)))

    for seg, vecs, tiles, more in [(328, 41, 1, False), (360, 45, 1, False), (392, 49, 1, False), (1000, 125, 3, False),
                                   (1016, 127, 3, False), (1048, 131, 3, True), (1160, 145, 3, True), (1400, 175, 3, True)]:
        both, heavy, alone = base(120, vecs, tiles), base(112, vecs, tiles), base(80, vecs, tiles)
        assert waves(seg, 24, 24) == both + both // 2 * more, seg
        assert waves(seg, 12, 30) == heavy + heavy // 2 * more, seg
        assert waves(seg, 0, 30) == alone + alone // 2, seg
        assert waves(seg, 30, 0) == base(64, vecs, tiles), seg
    assert waves(200, 24, 24, host_layout=0, layers=8) == base(120, 400, 7) * 3 // 2


@pytest.mark.parametrize("layout", [B.KV_HOST_BLOCK_FIRST, B.KV_HOST_LAYER_FIRST])
def test_bench_names_the_kernels_that_run(exe, layout):
    """bench.py names the kernel of its step from the call's sizes: the engine launches that one,
    in either pool layout, with chunks of layers, under a workgroup cap, and with lists of different lengths."""
    import bench
    from paper_2601_20309_amd import workloads as W
    sh = W.KVShape(32, 8, 128, 16, n_hbm_blocks=9, n_host_slots=9)            # blocks of 2 MiB
    small = W.KVShape(2, 1, 128, 16, n_hbm_blocks=9, n_host_slots=9)          # of 16 KiB
    plans = [(s, path, n_out, n_in, kw) for s in (sh, small) for path in ("sdma_staged", "fused", "zerocopy")
             for n_out, n_in in ((128, 128), (224, 224), (224, 225), (900, 2000), (2000, 700), (896, 897))
             for kw in ({}, {"chunk_layers": 1}, {"max_copy_wgs": 8})]
    code = {name: n for n, name in B.PATH_NAMES.items()}
    got = L.launches(exe, [L.move(no, ni, s.head_dim, layers=s.n_layers, heads=s.n_kv_heads, tokens=s.block_size, path=code[path],
                                  host_layout=layout, **kw) for s, path, no, ni, kw in plans])
    for (s, path, no, ni, kw), launches in zip(plans, got):
        named = bench.step_kernels(path, s, layout, no, ni, **kw)
        assert set(named) == {x["kernel"] for x in launches}, (s.n_layers, path, no, ni, kw)


def kinds(n, dim, **kw):
    return [L.move(n, n, dim, **kw), L.move(n, 0, dim, **kw), L.move(0, n, dim, **kw)]


@pytest.mark.parametrize("layout", [B.KV_HOST_BLOCK_FIRST, B.KV_HOST_LAYER_FIRST])
@pytest.mark.parametrize("dim,tokens", list(L.SHARES))
def test_lengths_that_end_the_fixed_share(exe, dim, tokens, layout):
    """L.SHARES: by a block more the waves draw, both ways, out and in, at every vector width."""
    for kind, n in enumerate(L.SHARES[dim, tokens][layout]):
        kw = dict(dim=dim, tokens=tokens, layers=6, host_layout=layout)
        below, above = L.launches(exe, [kinds(n, **kw)[kind], kinds(n + 1, **kw)[kind]])
        assert [below[0]["drawn"], above[0]["drawn"]] == [0, 1], kind


@pytest.mark.parametrize("vecs", list(L.ROUNDS))
def test_rounds_of_the_default_shapes(exe, vecs):
    """L.ROUNDS: the waves and steps that the engine launches; full rounds and the end of the fixed share lie between two of
    the lengths."""
    lengths = L.round_lengths(vecs)
    for kind, (waves, steps) in enumerate(L.ROUNDS[vecs]):
        got = {n: L.launches(exe, [kinds(n, 8 * vecs)[kind]])[0][0] for n in lengths}
        assert got[max(lengths)]["waves"] == waves and all(x["steps"] == n * steps for n, x in got.items())
        limit = L.BOTH_WAYS if kind == 0 else L.ONE_WAY
        for r in (1, 2, 3, limit):
            n = r * waves // steps
            assert n in got and n + 1 in got and n * steps <= r * waves < (n + 1) * steps
        assert [got[n]["drawn"] for n in (limit * waves // steps, limit * waves // steps + 1)] == [0, 1]


@pytest.mark.parametrize("vecs", [64, 75])
@pytest.mark.parametrize("wgs,lanes", [(1, 64), (3, 64), (1, 256), (2, 320)])
def test_lengths_around_the_limits_of_configured_shapes(exe, wgs, lanes, vecs):
    """L.configured_lengths: of each kind some take fixed shares and some draw, the nearest two a block apart, and some
    draw four steps at a time."""
    lengths = L.configured_lengths(wgs, lanes, vecs)
    for kind in range(3):
        calls = [kinds(n, 8 * vecs, layers=2, max_copy_wgs=wgs, wg_lanes=lanes, vecs_per_lane=1)[kind] for n in lengths]
        got = [x[0] for x in L.launches(exe, calls)]
        drawn = [x["drawn"] for x in got]
        first = drawn.index(1)
        assert drawn == sorted(drawn) and first > 0 and lengths[first] == lengths[first - 1] + 1
        assert got[-1]["waves"] == wgs * lanes // 64 and got[-1]["steps"] > 9 * got[-1]["waves"]


def test_tiles_of_short_reader_passes(exe):
    """Rows of a tile: even and at most eight, with no more rows than a wave's share makes them in as
    many rounds; tiles cover the list; from 13 rows a wave on tiles of eight."""
    for wgs in (0, 1, 3, 300):
        waves = 4 * (wgs or 1408)
        ns = sorted({max(1, rows * waves // 2 + d) for rows in range(1, 14) for d in (-1, 0, 1)})  # blocks of two rows
        for n, got in zip(ns, L.launches(exe, [L.read(n, 512, max_wgs=wgs) for n in ns])):
            x = got[-1]
            each = -(-2 * n // waves)
            rounds = -(-each // 8)
            want = -(-each // rounds)
            assert x["rows"] == (want + want % 2 if each <= 12 else 8), (wgs, n)
            assert x["tiles"] * 4 * x["rows"] >= 2 * n > (x["tiles"] - 1) * 4 * x["rows"]
