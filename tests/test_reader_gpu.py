"""The synthetic decode reader against the oracle's checksum, alone and while a
rotation runs."""
import numpy as np
import pytest
import torch

from oracle import kv_oracle as O
from paper_2601_20309_amd import binding as B
from paper_2601_20309_amd import workloads as W
from tests.gpu_harness import GpuCase, make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["tiny", "ragged", "small8b"])
def test_reader_checksum_matches_oracle(name):
    case, rot = make_case(name, B.KV_HOST_BLOCK_FIRST, B.KV_PATH_AUTO)
    sh = case.shape
    rng = np.random.default_rng(1)
    for ids, passes, wgs in [(rng.permutation(sh.n_hbm_blocks)[: sh.n_hbm_blocks // 2], 1, 0),
                             (np.arange(sh.n_hbm_blocks), 3, 0),
                             (np.array([5, 5, 7]), 2, 3),
                             (np.array([], dtype=np.int32), 1, 0)]:
        rc, want = O.read_checksum(case.oshape, case.ref_cache.view(np.uint8), ids)
        assert rc == 0
        assert case.eng.kv_reader_start(ids, passes, wgs) == 0
        rc, got, ms = case.eng.kv_reader_wait()
        assert rc == 0 and len(ms) == passes
        assert got == (want * passes) % (1 << 64)
    assert case.eng.kv_reader_start([sh.n_hbm_blocks], 1) == B.KV_ERANGE
    assert case.eng.kv_reader_start([0], 0) == B.KV_EINVAL
    assert case.eng.kv_reader_wait()[0] == B.KV_EINVAL     # nothing started
    case.close()


@pytest.mark.parametrize("path", [B.KV_PATH_AUTO, B.KV_PATH_SDMA_STAGED])
def test_reader_runs_beside_a_rotation(path):
    """Reader over blocks the rotation does not name, started first, rotation on
    top of it: both results must be what each gives alone."""
    case, rot = make_case("small8b", B.KV_HOST_BLOCK_FIRST, path)
    named = set(rot.out_ids.tolist()) | set(rot.in_ids.tolist())
    others = np.array([b for b in range(case.shape.n_hbm_blocks) if b not in named], dtype=np.int32)
    rc, want = O.read_checksum(case.oshape, case.ref_cache.view(np.uint8), others)
    assert case.eng.kv_reader_start(others, 8) == 0
    case.rotate(rot)
    rc, got, ms = case.eng.kv_reader_wait()
    assert rc == 0 and got == (want * 8) % (1 << 64)
    case.check()
    # swapped-out blocks are only read by the rotation: a reader may share them
    assert case.eng.kv_reader_start(rot.out_ids, 2) == 0
    case.rotate(rot.inverse())
    rc, want2 = O.read_checksum(case.oshape, case.ref_cache.view(np.uint8), rot.out_ids)
    # (the inverse rotation rewrites out_ids with their own bytes, so the sum is stable)
    rc, got2, _ = case.eng.kv_reader_wait()
    assert got2 == (want2 * 2) % (1 << 64)
    case.check()
    case.close()


def test_reader_on_block_first_cache():
    case, rot = make_case("small8b", B.KV_HOST_BLOCK_FIRST, B.KV_PATH_AUTO, hbm_layout=B.KV_HBM_BLOCK_FIRST)
    ids = np.random.default_rng(4).permutation(case.shape.n_hbm_blocks)[:100]
    rc, want = O.read_checksum(case.oshape, case.ref_cache.view(np.uint8), ids)
    assert case.eng.kv_reader_start(ids, 2) == 0
    rc, got, _ = case.eng.kv_reader_wait()
    assert rc == 0 and got == (2 * want) % (1 << 64)
    case.close()


@pytest.mark.parametrize("vecs", [1, 3, 63, 64, 65, 192, 511, 512, 513, 2049])
def test_reader_tiles_that_span_segments(vecs):
    """Segments of `vecs` 16-byte vectors: a tile (2048 vectors, rows of 64) begins and
    ends inside segments, spans many, or is one of several in a segment; lists of
    one block, with repeats, and long enough that workgroups claim tiles beyond
    their fixed share (few workgroups).  A sum of whole numbers: equal or wrong."""
    sh = W.KVShape(2, 1, 8 * vecs, 1, n_hbm_blocks=max(24, 12288 // vecs), n_host_slots=4)
    rng = np.random.default_rng(vecs)
    cache = rng.integers(0, 65536, 4 * sh.n_hbm_blocks * 8 * vecs, dtype=np.uint16)
    for hbm_layout in (B.KV_HBM_LAYER_FIRST, B.KV_HBM_BLOCK_FIRST):
        case = GpuCase(sh, B.KV_HOST_BLOCK_FIRST, B.KV_PATH_AUTO, cache, cache[:4 * 4 * 8 * vecs], hbm_layout=hbm_layout)
        every = rng.permutation(sh.n_hbm_blocks)
        for ids, passes, wgs in [(every, 2, 0), (every, 3, 1), (every, 1, 3), (every[:1], 2, 0),
                                 (np.array([5, 5, 7, 5]), 1, 0), (every[:-3], 2, 2)]:
            rc, want = O.read_checksum(case.oshape, case.ref_cache.view(np.uint8), ids)
            assert rc == 0 and case.eng.kv_reader_start(ids, passes, wgs) == 0
            rc, got, _ = case.eng.kv_reader_wait()
            assert rc == 0 and got == (want * passes) % (1 << 64), (hbm_layout, len(ids), passes, wgs)
        case.close()


@pytest.mark.parametrize("vecs", [64, 75])
def test_reader_claims_every_tile_once(vecs):
    """Passes long enough that tiles are claimed: groups of several workgroups, grids
    that the 64 counters do not divide and smaller ones, claims of one, two and four
    tiles, tiles taken from other groups (64 rounds of the grid and more), and the
    default grid.  A tile left out or read twice changes the sum."""
    nb = (3 << 29) // (64 * vecs)                                        # 1.5 GiB of blocks of 4 segments
    sh = W.KVShape(2, 1, 8 * vecs, 1, n_hbm_blocks=nb, n_host_slots=4)
    cache = torch.randint(-2**62, 2**62, (4, nb, 2 * vecs), device="cuda")      # 64-bit words of the [plane][block] segments
    block = sum((w & 0xFFFFFFFF).sum(1) + ((w >> 32) & 0xFFFFFFFF).sum(1) for w in cache).cpu().numpy()
    torch.cuda.synchronize()
    eng = B.Engine(B.make_config(sh), cache.data_ptr())
    ids = np.random.default_rng(vecs).integers(0, nb, 2 * nb).astype(np.int32)
    for wgs, rounds, passes in [(0, 69, 2), (0, 30, 1), (1, 300, 2), (40, 5, 2), (63, 130, 1), (64, 66, 1), (65, 30, 2), (65, 200, 2),
                                (100, 100, 1), (127, 65, 1), (128, 4, 1), (129, 90, 2), (1000, 40, 1)]:
        n = min(2 * nb, (2 * rounds + 1) * (wgs or 1408) * 1024 // (4 * vecs) + 1)      # (rounds + 1/2) * workgroups tiles of 2048 vectors
        assert eng.kv_reader_start(ids[:n], passes, wgs) == 0
        rc, got, _ = eng.kv_reader_wait()
        assert rc == 0 and got == int(block[ids[:n]].sum()) * passes % (1 << 64), (wgs, rounds, passes)
    eng.kv_destroy()


@pytest.mark.parametrize("vecs", [64, 5])
@pytest.mark.parametrize("blocks", [65536, 65537])
def test_reader_lists_in_arguments(blocks, vecs):
    """Lists at and beyond what a launch's arguments hold, two ids to a word where the
    cache has at most 65536 blocks, with the highest ids among them, of odd and even
    lengths; fixed shares only and claimed tiles in turn, so that each pass finds the
    counters that another one drew from at zero."""
    sh = W.KVShape(1, 1, 8 * vecs, 1, n_hbm_blocks=blocks, n_host_slots=4)
    cache = torch.randint(-2**62, 2**62, (2, blocks, 2 * vecs), device="cuda")
    block = sum((w & 0xFFFFFFFF).sum(1) + ((w >> 32) & 0xFFFFFFFF).sum(1) for w in cache).cpu().numpy()
    torch.cuda.synchronize()
    eng = B.Engine(B.make_config(sh), cache.data_ptr())
    rng = np.random.default_rng(blocks)
    for n, passes, wgs in [(1, 1, 0), (2, 2, 0), (895, 1, 0), (896, 1, 1), (897, 2, 2), (1791, 3, 1), (1792, 1, 0), (1793, 2, 1), (5000, 1, 3),
                           (1792, 2, 1), (7, 1, 0)]:
        ids = rng.integers(0, blocks, n).astype(np.int32)
        ids[-1] = blocks - 1
        assert eng.kv_reader_start(ids, passes, wgs) == 0
        rc, got, _ = eng.kv_reader_wait()
        assert rc == 0 and got == int(block[ids].sum()) * passes % (1 << 64), (n, passes, wgs)
    eng.kv_destroy()


@pytest.mark.parametrize("vecs", [64, 192, 105, 2048])
def test_reader_short_passes(vecs):
    """Passes of every number of rows per wave up to the most that counts as short and one
    more, where tiles go back to eight rows: the last workgroup's tile full, of one row and
    of one vector, lists in the arguments, there in pairs and in memory, whole rows to a
    segment and rows that straddle them, the whole grid (there up to 75 MiB) and a few workgroups."""
    nb = 2100 if vecs == 2048 else 20000
    sh = W.KVShape(1, 1, 8 * vecs, 1, n_hbm_blocks=nb, n_host_slots=4)
    cache = torch.randint(-2**62, 2**62, (2, nb, 2 * vecs), device="cuda")
    block = sum((w & 0xFFFFFFFF).sum(1) + ((w >> 32) & 0xFFFFFFFF).sum(1) for w in cache).cpu().numpy()
    torch.cuda.synchronize()
    eng = B.Engine(B.make_config(sh), cache.data_ptr())
    rng = np.random.default_rng(vecs)
    for wgs in (1, 3, 40, 150, 300, 0):
        for rows in range(1, 14):
            most = rows * 4 * (wgs or 1408) * 64 // (2 * vecs)           # blocks that this many rows a wave hold
            for n in {most - 1, most, most + 1, most - 2 * (wgs or 1408)} & set(range(1, 2 * nb + 1)):
                ids = rng.integers(0, nb, n).astype(np.int32)
                passes = 1 + n % 2
                assert eng.kv_reader_start(ids, passes, wgs) == 0
                rc, got, _ = eng.kv_reader_wait()
                assert rc == 0 and got == int(block[ids].sum()) * passes % (1 << 64), (wgs, rows, n)
    eng.kv_destroy()
