"""The tile kernel (rows by tree groups), the block GEMM kernel and the
many-trees-per-lane kernel against the CPU oracle, at the sizes where their
branches meet: leaf ids identical, scores within 1e-5 (1 + |oracle|) (sums are
taken in double and rounded once, 6e-8)."""
import numpy as np
import pytest

import paper_2010_04804_amd as hb
from paper_2010_04804_amd import synth
from test_gpu_parity import check, need_gpu, run, say  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ROWS = 49_152  # 192 rows per CU: the smallest batch of the tile kernel


def _forest(kind, size, F, T, K=1, ld=1, seed=0, spread=1, base=False):
    rng = np.random.Generator(np.random.PCG64(seed))
    thr = lambda r, f: r.standard_normal(f.size)
    leaves = lambda r, n: r.normal(0.0, 0.05, (n, ld) if ld > 1 else n)
    if kind == "perfect":
        m = synth.perfect_forest(rng, T, size, F, thr, leaves, leaf_dim=ld)
    else:
        m = synth.leafwise_forest(rng, T, size, 12, 0.7, F, thr, lambda r, n: r.normal(0.0, 0.05, n))
        if ld > 1:
            m["leaf_value"] = rng.normal(0.0, 0.05, m["feature"].size * ld).astype(np.float32)
            m["leaf_dim"] = ld
    if spread > 1:
        m["feature"] = np.where(m["feature"] >= 0, m["feature"] * spread, -1).astype(np.int32)
        m["n_features"] = F * spread
    K = max(K, ld)
    m.update(n_outputs=K, tree_class=(np.arange(T) % K).astype(np.int32) if K > 1 and ld == 1 else None,
             aggregation="mean" if ld > 1 else "sum", transform="softmax" if K > 1 and ld == 1 else "none",
             base_score=np.linspace(-1, 1, K).astype(np.float32) if base else None)
    return m


def _both(m, X, strategy, expect, label, expect_ids=None):
    """Scores with leaf ids (and a workspace) and without either, each on the
    kernel its plan names."""
    h = hb.compile(m, strategy=strategy, device=0)
    n = X.shape[0]
    plan = [p["kernel"] for p in h.plan(n, strategy)]
    plan_ids = [p["kernel"] for p in h.plan(n, strategy, hb.workspace_bytes(h, n, strategy), leaves=True)]
    say(label, plan, plan_ids)
    assert plan[0].startswith(expect), plan
    assert plan_ids[0].startswith(expect_ids or expect), plan_ids
    s, ids = run(h, X, strategy)
    check(m, X, s, ids, label)
    s, none = run(h, X, strategy, leaves=False, workspace=False)
    assert none is None
    check(m, X, s, None, label + " scores only")
    return h


# kind, depth or leaves, columns, trees, classes, leaf values, rows past ROWS, column spread, strategy, kernel;
# with leaf ids the fast kernel takes the cases of few columns and perfect trees (FAST_IDS)
FAST_IDS = {(1, 300): "fast_kernel<3, 1, 2, 512", (5, 28): "fast_kernel<0, 5, 2, 512",
            (7, 40): "fast_kernel<3, 7, 16, 512", (8, 54): "fast_kernel<3, 8, 16, 512"}
CASES = [
    ("perfect", 8, 130, 33, 1, 1, 0, 1, "ptt", "tile_kernel<true, false, 1, false"),     # a chunk and a tree
    ("perfect", 7, 203, 5, 1, 1, 1, 1, "ptt", "tile_kernel<true, false, 1, false"),      # fewer trees than a chunk
    ("perfect", 1, 300, 70, 2, 1, 127, 1, "ptt", "tile_kernel<true, false, 2, false"),   # one level
    ("perfect", 6, 450, 40, 1, 1, 65, 1, "ptt", "tile_kernel<true, "),                   # about the widest tile
    ("perfect", 6, 64, 37, 5, 5, 3, 1, "ptt", "tile_kernel<true, false, 16, true"),      # 5-vector leaves
    ("perfect", 5, 28, 64, 2, 2, 77, 1, "ptt", "tile_kernel<true, false, 2, true"),      # 2-vectors, narrow rows
    ("perfect", 7, 40, 66, 3, 1, 20_001, 1, "ptt", "tile_kernel<true, false, 16, false"),
    ("perfect", 11, 28, 9, 1, 1, 1, 3, "ptt", "tile_kernel<true, "),                     # deep, through a column list
    ("perfect", 12, 20, 6, 16, 1, 0, 1, "ptt", "tile_kernel<true, true, 16, false"),     # ranks, 16 classes
    ("perfect", 8, 54, 700, 7, 1, 30_000, 1, "ptt", "tile_kernel<true, "),
    ("leafwise", 200, 150, 35, 1, 1, 5, 1, "tt", "tile_kernel<false, false, 1, false"),
    ("leafwise", 40, 260, 64, 2, 2, 64, 1, "tt", "tile_kernel<false, false, 2, true"),
    ("leafwise", 1500, 28, 4, 3, 1, 1, 1, "tt", "tile_kernel<false, false, 16, false"),  # trees past the fast tables
    ("leafwise", 31, 170, 21, 4, 4, 2, 2, "tt", "tile_kernel<false, false, 16, true"),
]


@pytest.mark.parametrize("kind,size,F,T,K,ld,extra,spread,strategy,expect", CASES)
def test_tile_kernel(kind, size, F, T, K, ld, extra, spread, strategy, expect):
    m = _forest(kind, size, F, T, K, ld, seed=size + F + T, spread=spread, base=K > 1)
    n = ROWS + extra
    X = np.random.Generator(np.random.PCG64(n + F)).standard_normal((n, F * spread)).astype(np.float32)
    _both(m, X, strategy, expect, f"tile {kind}{size} F{F}x{spread} T{T} K{K} ld{ld} n{n}",
          FAST_IDS.get((size, F))).close()


@pytest.mark.parametrize("kind,size,F,T,strategy", [
    ("perfect", 11, 24, 10, "ptt"), ("perfect", 6, 140, 36, "ptt"), ("leafwise", 60, 140, 30, "tt")])
def test_tile_missing_categories_and_infinities(kind, size, F, T, strategy):
    """NaN with both default directions, category sets, ties, and infinite
    thresholds and inputs, in fp32 and rank tiles; node ids permuted, so the
    leaf ids come from a table."""
    m = synth.permute_nodes(_forest(kind, size, F, T, seed=3 * F + T), seed=5)
    n = ROWS + 19
    rng = np.random.Generator(np.random.PCG64(F))
    X = rng.standard_normal((n, F)).astype(np.float32)
    inner = np.flatnonzero(m["feature"] >= 0)
    m["threshold"] = m["threshold"].copy()
    m["threshold"][rng.choice(inner, 40)] = np.inf
    m["threshold"][rng.choice(inner, 40)] = -np.inf
    m["threshold"][rng.choice(inner, 40)] = -0.0
    X[rng.random(X.shape) < 0.02] = np.inf
    X[rng.random(X.shape) < 0.02] = -np.inf
    X[rng.random(X.shape) < 0.02] = 0.0
    tie = rng.choice(inner, 200)
    X[rng.integers(0, n, 200), m["feature"][tie]] = m["threshold"][tie]
    m, X = synth.with_categories(m, X, seed=F, cat_cols=[1, 5], n_categories=3)
    m, X = synth.with_missing(m, X, seed=T, p_missing=0.05)
    _both(m, X, strategy, "tile_kernel<", f"tile special {kind}{size} F{F} {strategy}").close()


def test_tile_unaligned_leaf_ids():
    """Leaf ids one int past a 16-byte boundary, and input rows four bytes past
    one: the scalar paths write every id and nothing around them."""
    m = _forest("perfect", 6, 132, 36, seed=9)
    h = hb.compile(m, device=0)
    n, T, F = ROWS + 33, 36, 132
    X = np.random.Generator(np.random.PCG64(1)).standard_normal((n, F)).astype(np.float32)
    xbuf = torch.zeros(n * F + 1, dtype=torch.float32, device="cuda")
    xbuf[1:] = torch.from_numpy(X).cuda().reshape(-1)
    buf = torch.full((n * T + 8,), -7, dtype=torch.int32, device="cuda")
    sc = torch.empty((n, 1), dtype=torch.float32, device="cuda")
    hb.predict_ptr(h, xbuf.data_ptr() + 4, n, sc.data_ptr(), buf.data_ptr() + 4, "ptt",
                   torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    b = buf.cpu().numpy()
    assert b[0] == -7 and np.all(b[1 + n * T:] == -7)
    check(m, X, sc.cpu().numpy(), b[1:1 + n * T].reshape(n, T), "tile unaligned")
    h.close()


@pytest.mark.parametrize("kind,size,F,T,K,ld,n", [
    ("perfect", 7, 40, 300, 2, 2, 16_000), ("perfect", 7, 40, 300, 2, 2, 15_001), ("perfect", 7, 33, 300, 5, 5, 1025),
    ("perfect", 11, 20, 33, 1, 1, 4097), ("perfect", 12, 20, 64, 3, 1, 1100), ("leafwise", 31, 40, 101, 1, 1, 2000),
    ("leafwise", 200, 30, 130, 3, 1, 8192), ("leafwise", 60, 20, 300, 2, 2, 4_000)])
def test_tile_tree_split(kind, size, F, T, K, ld, n):
    """With a workspace, batches of 1,025 to 16,384 rows divide the trees of a
    row tile among workgroups, whose last leaf-id group may be short: ids and
    scores as without the split."""
    m = _forest(kind, size, F, T, K, ld, seed=size + n, base=True)
    strategy = "ptt" if kind == "perfect" else "tt"
    h = hb.compile(m, strategy=strategy, device=0)
    for leaves in (False, True):
        plan = [p["kernel"] for p in h.plan(n, strategy, hb.workspace_bytes(h, n, strategy), leaves)]
        say("tile split", kind, size, F, T, K, ld, n, leaves, plan)
        assert plan[0].startswith("tile_kernel<") and plan[1].startswith("split_finish"), plan
    X = np.random.Generator(np.random.PCG64(n)).standard_normal((n, F)).astype(np.float32)
    s, ids = run(h, X, strategy)
    check(m, X, s, ids, f"tile split {kind}{size} T{T} n{n}")
    s, _ = run(h, X, strategy, leaves=False)
    check(m, X, s, None, f"tile split {kind}{size} T{T} n{n} scores only")
    h.close()


@pytest.mark.parametrize("kind,size,F,T,ld,n,workspace", [
    ("perfect", 9, 60, 100, 2, 50_003, False),      # chunks of 6 trees, one per flush
    ("perfect", 8, 60, 400, 2, 8_000, True)])       # tree split in parts of 30 trees, chunks of 6
def test_tile_leaf_ids_start_at_any_tree(kind, size, F, T, ld, n, workspace):
    """Leaf-id rows 16-byte aligned (T a multiple of four) and flushes that
    start at no multiple of four trees and end on a lane's first or second
    one: every id is written, and nothing around the output."""
    m = _forest(kind, size, F, T, ld, ld, seed=size + T)
    strategy = "ptt" if kind == "perfect" else "tt"
    h = hb.compile(m, strategy=strategy, device=0)
    X = np.random.Generator(np.random.PCG64(n)).standard_normal((n, F)).astype(np.float32)
    Xd = torch.from_numpy(X).cuda()
    nws = hb.workspace_bytes(h, n, strategy) if workspace else 0
    plan = [p["kernel"] for p in h.plan(n, strategy, nws, leaves=True)]
    say("tile ids", kind, size, F, T, ld, n, nws, plan)
    assert plan[0].startswith("tile_kernel<") and (len(plan) == 2) == workspace, plan
    buf = torch.full((n * T + 8,), -7, dtype=torch.int32, device="cuda")
    sc = torch.empty((n, max(1, ld)), dtype=torch.float32, device="cuda")
    ws = torch.empty(max(nws, 8), dtype=torch.uint8, device="cuda")
    hb.predict_ptr(h, Xd.data_ptr(), n, sc.data_ptr(), buf.data_ptr() + 16, strategy,
                   torch.cuda.current_stream().cuda_stream, ws.data_ptr() if nws else None, nws)
    torch.cuda.synchronize()
    b = buf.cpu().numpy()
    assert np.all(b[:4] == -7) and np.all(b[4 + n * T:] == -7)
    check(m, X, sc.cpu().numpy(), b[4:4 + n * T].reshape(n, T), f"tile ids {kind}{size} T{T} n{n}")
    h.close()


@pytest.mark.parametrize("T,K,ld,n", [(1, 1, 1, 32_768), (3, 1, 1, 32_769), (5, 2, 1, 32_895), (9, 3, 3, 33_000),
                                      (4, 16, 1, 32_801)])
def test_gemm_block_kernel(T, K, ld, n):
    """Fewer trees than the four tree groups, ragged row tiles, class trees and
    vector leaves on the block GEMM kernel, with ties and NaN in the rows."""
    m = _forest("perfect", 8, 20, T, K, ld, seed=T + n, base=True)
    rng = np.random.Generator(np.random.PCG64(n))
    X = rng.standard_normal((n, 20)).astype(np.float32)
    X[rng.random(X.shape) < 0.02] = np.nan
    inner = rng.choice(np.flatnonzero(m["feature"] >= 0), 500)
    X[rng.integers(0, n, 500), m["feature"][inner]] = m["threshold"][inner]
    _both(m, X, "gemm", "gemm_block_kernel<", f"gemm block T{T} K{K} ld{ld} n{n}").close()


@pytest.mark.parametrize("kind,size", [("perfect", 5), ("leafwise", 30)])
@pytest.mark.parametrize("T,K,ld,n", [(513, 1, 1, 2), (1023, 1, 1, 65), (2049, 1, 1, 3), (2500, 7, 1, 5), (2100, 2, 2, 33),
                                      (2060, 5, 5, 9), (700, 12, 1, 7), (1100, 9, 9, 4), (600, 3, 1, 300)])
def test_lanes_many_trees(kind, size, T, K, ld, n):
    """Tree counts past the lanes of a workgroup: 256 to 1,024 lanes per row,
    one and four trees per lane, the halving sums of 1 to 16 outputs."""
    m = _forest(kind, size, 12, T, K, ld, seed=T + n)
    X = np.random.Generator(np.random.PCG64(n)).standard_normal((n, 12)).astype(np.float32)
    strategy = "ptt" if kind == "perfect" else "tt"
    _both(m, X, strategy, "lanes", f"lanes {kind} T{T} K{K} ld{ld} n{n}").close()


@pytest.mark.parametrize("F,K", [(40_952, 1), (40_832, 12)])
def test_lanes_widest_rows(F, K):
    """Rows that leave LDS for the four waves' sums and nothing more stay on
    the trees-across-lanes kernel."""
    m = _forest("perfect", 8, F, 162, K, seed=K)
    inner = np.flatnonzero(m["feature"] >= 0)
    m["feature"][inner] = np.arange(inner.size) % F  # every column is used
    X = np.random.Generator(np.random.PCG64(F)).standard_normal((9, F)).astype(np.float32)
    _both(m, X, "ptt", "lanes_kernel<", f"lanes F{F} K{K}").close()


def test_lanes_leafwise_four_trees():
    """Four leaf-wise trees per lane only where a row has more than 256 lanes."""
    m = _forest("leafwise", 30, 12, 1200, seed=4)
    h = hb.compile(m, strategy="tt", device=0)
    for n, kernel in [(200, "lanes4_kernel<false, 1, false>"), (257, "lanes_kernel<false, 1, false, 1>"),
                      (512, "lanes_kernel<false, 1, false, 1>")]:
        assert [p["kernel"] for p in h.plan(n, "tt")] == [kernel]
    h.close()


def test_tile_tree_split_of_narrow_rows():
    """The leaf-wise tree split goes to the tile kernel on rows wide enough
    to leave the fast kernel few waves on a CU, or for few walks; with leaf
    ids, beyond 3M walks, only in flushes of 16 trees."""
    tile, fast = "tile_kernel<", "fast_kernel<"
    for leaves_, F, T, n, kernel, kernel_ids in [
            (31, 12, 150, 4_500, tile, tile), (31, 12, 800, 4_500, fast, fast), (31, 28, 800, 16_000, fast, fast),
            (31, 60, 800, 4_500, tile, fast), (255, 50, 800, 3_000, tile, tile), (255, 50, 800, 6_500, tile, fast)]:
        h = hb.compile(_forest("leafwise", leaves_, F, T, seed=F + T), strategy="tt", device=0)
        for ids, expect in ((False, kernel), (True, kernel_ids)):
            plan = [p["kernel"] for p in h.plan(n, "tt", hb.workspace_bytes(h, n, "tt"), ids)]
            assert plan[0].startswith(expect), (leaves_, F, T, n, ids, plan)
        h.close()


@pytest.mark.parametrize("D,K", [(9, 1), (10, 1), (9, 3), (10, 12)])
def test_tile_tables_left_out(D, K):
    """Scalar leaves of depth 9 or 10 on at most 64 columns have no tile
    tables: the fast kernel holds every batch of them."""
    m = _forest("perfect", D, 64, 13, K, seed=D)
    h = hb.compile(m, strategy="ptt", device=0)
    for n in (2_000, 16_000, 50_000, 70_000, 300_000):
        for ws in (0, hb.workspace_bytes(h, n, "ptt")):
            plan = [p["kernel"] for p in h.plan(n, "ptt", ws)]
            assert plan[0].startswith(("fast_kernel<", "lanes_kernel<")), (D, K, n, ws, plan)
    h.close()


def _deep_columns(T, F, counts, draw):
    """Perfect trees of depth 12 whose decision nodes test column c counts[c]
    times (the columns of the rest drawn from those past counts), thresholds
    from draw(rng, column, number)."""
    rng = np.random.Generator(np.random.PCG64(T))
    m = _forest("perfect", 12, F, T, seed=T)
    inner = rng.permutation(np.flatnonzero(m["feature"] >= 0))
    f = rng.integers(len(counts), max(F - 3, len(counts) + 1), inner.size)  # (the last three columns: no node)
    f[:sum(counts)] = np.repeat(np.arange(len(counts)), counts)
    m["feature"][inner] = f
    m["threshold"] = m["threshold"].copy()
    for c in range(F):
        at = inner[f == c]
        m["threshold"][at] = draw(rng, c, at.size)
    return m


@pytest.mark.parametrize("F,n", [(16, ROWS + 37), (16, 3_001), (180, ROWS + 5)])
def test_tile_ranks_of_sampled_columns(F, n):
    """Columns with more distinct thresholds (58,001 and 36,003) than fit in
    LDS: every second (16 columns) or fourth (180) passes through it and the
    last steps of a search are taken in global memory. Short columns and columns that no node
    tests lie beside them; rows hold ties with any of the thresholds, their
    neighbours, infinities and NaN."""
    def draw(rng, c, k):
        t = rng.standard_normal(k).astype(np.float32)
        if k > 8:
            t[:4] = [np.inf, -np.inf, -0.0, 0.0]
        return t

    m = _deep_columns(40, F, (58_001, 36_003), draw)
    rng = np.random.Generator(np.random.PCG64(n))
    X = rng.standard_normal((n, F)).astype(np.float32)
    for c in range(F - 3):
        t = np.unique(m["threshold"][m["feature"] == c])
        assert c > 1 or t.size > 35_000
        pick = rng.choice(t, n)
        near = np.nextafter(pick, rng.choice(np.float32([np.inf, -np.inf]), n))
        X[:, c] = np.select([rng.random(n) < 0.3, rng.random(n) < 0.6], [pick, near], X[:, c])
        X[rng.random(n) < 0.02, c] = np.nan
        X[rng.random(n) < 0.02, c] = rng.choice([np.inf, -np.inf])
    _both(m, X, "ptt", "tile_kernel<true, true, 1, false" if n >= ROWS else "lanes", f"tile sampled ranks F{F} n{n}",
          "tile_kernel<true, true, 1, false").close()


@pytest.mark.parametrize("distinct,ranked", [(65_534, True), (65_535, False)])
def test_tile_rank_limit(distinct, ranked):
    """16-bit ranks hold a column of 65,534 distinct thresholds; one more and
    the model keeps the fp32 tile."""
    def draw(rng, c, k):
        return rng.permutation(np.arange(k)).astype(np.float32) if c == 0 else rng.standard_normal(k)

    m = _deep_columns(17, 5, (distinct,), draw)
    n = ROWS + 3
    rng = np.random.Generator(np.random.PCG64(distinct))
    X = rng.standard_normal((n, 5)).astype(np.float32)
    X[:, 0] = rng.integers(-2, distinct + 2, n) + rng.choice([0.0, 0.5], n)
    X[:8, 0] = [-1, 0, distinct - 1, distinct - 2, distinct, np.inf, -np.inf, np.nan]
    _both(m, X, "ptt", f"tile_kernel<true, {'true' if ranked else 'false'}, 1, false", f"tile rank limit {distinct}").close()
