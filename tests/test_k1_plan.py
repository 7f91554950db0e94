"""Host logic of the LM heads' launches. asv_k1_plan: which tile family covers which 256-id slabs,
and each launch's K loop, weight copy policy and tile order. asv_k1_cut and asv_draft_cut: the
slabs of other widths that take the plan's place, and the draft head's. asv_verify and
asv_draft_step launch from the same records. CPU only: no GPU call."""
import math

import numpy as np
import pytest

import paper_2609_02897_amd as asv
from paper_2609_02897_amd import _build

COST = {128: 62, 192: 80, 256: 98}      # per-round costs of the tile families (tile pick)


@pytest.fixture(scope="module", autouse=True)
def built():
    if not _build.is_built(_build.OUT):
        _build.build_library()


def _launch(tile_rows, slab0, n_slabs, row_tiles, k_loop, stream_w, blk_slabs=0, blk_rows=0):
    return dict(tile_rows=tile_rows, slab0=slab0, n_slabs=n_slabs, row_tiles=row_tiles,
                k_loop=k_loop, stream_w=stream_w, blk_slabs=blk_slabs, blk_rows=blk_rows)


@pytest.mark.parametrize("N,V,expected", [
    # up to 64 rows one 64-row tile a slab (cut anew: test_documented_cuts)
    (60, 128256, [_launch(64, 0, 501, 1, 0, 1)]),
    (60, 151936, [_launch(64, 0, 594, 1, 0, 1)]),
    # 378 rows: 128-row tiles fill one round on 85 slabs (three row tiles: default policy),
    # 192-row tiles take the other 509 (two row tiles: non-temporal W)
    (378, 151936, [_launch(128, 0, 85, 3, 3, 0), _launch(192, 85, 509, 2, 2, 1)]),
    # 2048 rows: 23 slabs of 192-row tiles (11 row tiles: blocked order), then 256-row tiles
    (2048, 128256, [_launch(192, 0, 23, 11, 2, 0, 8, 4), _launch(256, 23, 478, 8, 2, 0)]),
    # 3048 rows: 256-row tiles only, twelve row tiles, blocks of 8 slabs x 4 row tiles
    (3048, 151936, [_launch(256, 0, 594, 12, 2, 0, 8, 4)]),
])
def test_documented_plans(N, V, expected):
    assert asv.k1_plan(N, V, 256) == expected


def _rounds(tiles, cus):
    return (tiles + cus - 1) // cus


def _estimate(launches, cus):
    return sum(_rounds(k["n_slabs"] * k["row_tiles"], cus) * COST[k["tile_rows"]]
               for k in launches)


def test_plan_invariants():
    """Over random shapes: the launches cover the slabs once, in order; every launch follows
    the stated rules; above 64 rows the plan's estimate is no worse than any single family's."""
    rng = np.random.default_rng(2609)
    for _ in range(3000):
        N = int(rng.choice([rng.integers(1, 65), rng.integers(65, 600), rng.integers(600, 6000)]))
        V = int(rng.integers(1, 300000))
        cus = int(rng.choice([8, 32, 80, 104, 256, 304]))
        forced = int(rng.choice([0, 0, 0, 64, 128, 192, 256]))
        got = asv.k1_plan(N, V, cus, forced)
        S = (V + 255) // 256
        c = max(1, cus // 8)
        assert 1 <= len(got) <= 2
        assert got[0]["slab0"] == 0 and sum(k["n_slabs"] for k in got) == S
        if len(got) == 2:
            assert got[1]["slab0"] == got[0]["n_slabs"] and got[0]["tile_rows"] != got[1]["tile_rows"]
        if forced:
            assert len(got) == 1 and got[0]["tile_rows"] == forced
        elif N <= 64:
            assert len(got) == 1 and got[0]["tile_rows"] == 64
        else:
            assert all(k["tile_rows"] in (128, 192, 256) for k in got)
            single = min(_rounds(S * math.ceil(N / r), cus) * COST[r] for r in COST)
            assert _estimate(got, cus) <= single, (N, V, cus, got)
        for k in got:
            rt = math.ceil(N / k["tile_rows"])
            assert k["row_tiles"] == rt
            if k["tile_rows"] == 64:
                assert k["k_loop"] == 0
            else:
                assert k["k_loop"] == (3 if k["tile_rows"] == 128 else 2)
            assert k["stream_w"] == (1 if rt <= 2 else 0)
            blocked = rt > 4 and c / rt + rt > c / 4 + 4
            assert (k["blk_slabs"], k["blk_rows"]) == ((max(1, c // 4), 4) if blocked else (0, 0))


def _cut(main=(0, 0, 0, 0), tail=(0, 0, 0, 0)):
    return dict(zip(("main_slabs", "main_ids", "main_tile_ids", "main_tile_rows"), main),
                **dict(zip(("tail_slabs", "tail_ids", "tail_tile_ids", "tail_tile_rows"), tail)),
                records=main[0] + tail[0])


@pytest.mark.parametrize("N,V,expected", [
    # one workgroup per CU: an equal share of the ids on the 128- or the 256-id tile
    (60, 32000, _cut((250, 128, 128, 64))),
    (60, 50000, _cut((250, 200, 256, 64))),
    # two per CU
    (60, 60000, _cut((500, 120, 128, 64))),
    (60, 128256, _cut((501, 256, 256, 64))),
    # whole rounds of two per CU, the rest on 64-id tiles
    (60, 151936, _cut((1024, 128, 128, 64), (326, 64, 64, 64))),
    # past 2^18 ids the plan's widths
    (60, 300000, _cut((1172, 256, 256, 64))),
    # no whole round of 256-id slabs: one round of narrower ones alone
    (120, 32000, _cut(tail=(250, 128, 128, 128))),
    (190, 32000, _cut(tail=(250, 128, 128, 192))),
    # one round, then the rest on narrower slabs, one a CU
    (120, 73728, _cut((256, 256, 256, 128), (256, 32, 64, 128))),
    (230, 81920, _cut((256, 256, 256, 256), (256, 64, 64, 256))),
    # two rounds: the rest on 64-row tiles
    (190, 151936, _cut((512, 256, 256, 192), (82, 256, 256, 64))),
    # the plan's launches as they are
    (378, 151936, None), (250, 98304, None), (513, 34000, None), (2048, 128256, None),
])
def test_documented_cuts(N, V, expected):
    assert asv.k1_cut(N, V, 256) == expected


@pytest.mark.parametrize("B,V,expected", [
    # one 64-id slab a CU (and a few more at one or two requests): tiles that hold no more
    (1, 16000, _cut((250, 64, 64, 32))), (8, 5000, _cut((79, 64, 64, 32))),
    (9, 16384, _cut((256, 64, 64, 64))), (2, 20480, _cut((320, 64, 64, 32))),
    (3, 16385, _cut((228, 72, 128, 64))), (2, 20481, _cut((233, 88, 128, 64))),
    (1, 32000, _cut((250, 128, 128, 64))), (16, 48000, _cut((250, 192, 256, 64))),
    (17, 32000, _cut((250, 128, 128, 128))), (32, 48000, _cut((250, 192, 192, 128))),
    (32, 64000, _cut((250, 256, 256, 128))), (40, 32000, _cut((250, 128, 128, 256))),
])
def test_documented_draft_cuts(B, V, expected):
    assert asv.draft_cut(B, V, 256) == expected


def _check_cut(c, V):
    """The slabs cover ids 0 .. V - 1 once, none is empty and each fits its tile."""
    assert c["records"] == c["main_slabs"] + c["tail_slabs"] > 0
    at = 0
    for part in ("main", "tail"):
        n, ids = c[part + "_slabs"], c[part + "_ids"]
        if n == 0:
            assert [c[f"{part}_{f}"] for f in ("ids", "tile_ids", "tile_rows")] == [0, 0, 0]
            continue
        assert 0 < ids <= c[part + "_tile_ids"] and at + (n - 1) * ids < V
        at = at + n * ids
    assert at >= V


def test_cut_invariants():
    """Over random shapes and at the rules' own lines: every cut covers the vocabulary once, and the
    records it writes fit the workspace, whatever the CU count."""
    rng = np.random.default_rng(97)
    lines = [(N, V + d) for N in (1, 64, 65, 128, 192, 256, 257, 384, 385, 512)
             for V in (5, 8192, 16384, 32768, 57344, 65536, 98304, 131072, 196608, 1 << 18)
             for d in (-1, 0, 1)]
    drawn = [(int(rng.choice([rng.integers(1, 65), rng.integers(65, 513), rng.integers(513, 4000)])),
              int(np.exp(rng.uniform(np.log(4), np.log(400000))))) for _ in range(3000)]
    seen = set()
    for i, (N, V) in enumerate(lines + drawn):
        cus = 256 if i % 2 else int(rng.choice([8, 32, 80, 104, 304, 1000]))
        c = asv.k1_cut(N, V, cus)
        assert asv.k1_cut(N, V, cus, 128) is None and asv.k1_cut(N, V, cus, 256) is None
        assert (c is not None) if N <= 64 else (c is None or N <= 512)
        if c:
            _check_cut(c, V)
            assert 12 * N * c["records"] <= asv.workspace_bytes(1, N, 64, V), (N, V, cus, c)
            seen.add((c["main_tile_ids"], c["main_tile_rows"], c["tail_tile_ids"], c["tail_tile_rows"]))
        B = -(-N // 8)
        d = asv.draft_cut(B, V, cus)
        _check_cut(d, V)
        assert 36 * 4 * B * d["records"] <= asv.draft_workspace_bytes(B, 64, V), (B, V, cus, d)
    assert len(seen) > 15


def test_plan_of_the_largest_sizes_is_quick():
    """The two-family search is bounded: one CU and the largest accepted grid plan at once."""
    import time
    asv.k1_plan(100, 1000, 256)               # loads the library (runtime start-up) untimed
    t0 = time.perf_counter()
    got = asv.k1_plan((1 << 15) - 64, (1 << 30) - 1, 1)   # 2^22 slabs x 511 64-row tiles
    assert time.perf_counter() - t0 < 0.5
    assert sum(k["n_slabs"] for k in got) == ((1 << 30) - 1 + 255) // 256


@pytest.mark.parametrize("args", [(0, 1000, 256, 0), (10, 0, 256, 0), (10, 1000, 0, 0),
                                  (10, 1000, 256, 100)])
def test_plan_rejects(args):
    with pytest.raises(asv.AsvError):
        asv.k1_plan(*args)
    with pytest.raises(asv.AsvError):
        asv.k1_cut(*args)


@pytest.mark.parametrize("args", [(0, 1000, 256), (1, 3, 256), (1, 1000, 0), (1 << 22, 1000, 256)])
def test_draft_cut_rejects(args):
    with pytest.raises(asv.AsvError):
        asv.draft_cut(*args)
