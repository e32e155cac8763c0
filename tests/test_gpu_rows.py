"""Rows of chosen shapes through whole steps on the GPU, against the oracle,
bit for bit: the row kernels at the sizes where a batch, a block width or a
table begins or ends, and the value distributions that leave their common
paths (rows sorted by id, one cluster of large values, massive ties, constant
rows, few finite logits, signed zeros, values at the ends of the counted
range and beyond it).

Every draft row is given by its place in the frontier, so both sides see the
same row for the same node whatever the tree is.
"""

import os

import numpy as np
import pytest
import torch

from oracle import rheo
from oracle.drivers import run_philox
from oracle.harness import node_table

pytestmark = pytest.mark.gpu

KEY = 0x1F2E3D4C5B6A7988


@pytest.fixture(scope="module")
def dev():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2609_21827_amd import binding
    binding.load_library()
    return "cuda"


def _shape(kind, x, rng):
    """The rows x [n, V] (fp32) given the value distribution `kind`."""
    n, V = x.shape
    if kind == "sorted":
        x = -np.sort(-x, axis=1)
    elif kind == "sorted_up":
        x = np.sort(x, axis=1)
    elif kind == "cluster":                 # the largest values in one run of ids
        x[:, V // 3:V // 3 + min(V // 4, 700)] += 9
    elif kind == "ties":
        x = np.round(x)
    elif kind == "const":
        x[:] = -1.25
    elif kind == "few":                     # about 40 finite logits
        x[:, 40:][rng.random((n, V - 40)) < 0.9995] = -np.inf
    elif kind == "signed_zeros":            # the top of the row: zeros of both signs
        x = -np.abs(x)
        x[:, rng.integers(0, V, 60)] = 0.0
        x[:, rng.integers(0, V, 60)] = -0.0
    elif kind == "edges":                   # magnitudes around 2^-11 and 2^9
        e = np.array([2.0 ** -11, 2.0 ** -11 * (1 - 2 ** -8), 2.0 ** -12, 1e-30, 511.0,
                      -2.0 ** -11, -2.0 ** -10, -511.0, -512.0, -513.0, -1e30, 0.0, -0.0])
        x[:, :: max(1, V // 200)] = rng.choice(e, x[:, :: max(1, V // 200)].shape)
    elif kind == "small":                   # every value below 2^-11
        x *= 1e-5
    elif kind == "large":                   # the top of the row above 2^9
        x = x * 3 + 515
    elif kind == "zeros":                   # a padded vocabulary's columns, and scattered ones
        x[:, V - V // 16:] = 0.0
        x[rng.random((n, V)) < 0.05] = -0.0
    elif kind == "zeros_small":             # both, and values below 2^-11 that are listed
        x[rng.random((n, V)) < 0.05] = 0.0
        x[:, rng.integers(0, V, 60)] = 1e-4
        x[:, rng.integers(0, V, 60)] = -2e-5
    elif kind == "half_zeros":              # lanes that meet on a word
        x[rng.random((n, V)) < 0.5] = 0.0
    elif kind == "few_values":
        x = np.round(x / 3) * 3
    elif kind == "zero_cross":              # the support spans zero
        x = x * 0.01
    return x


def _rows(rng, n, V, dtype, kind, spread=2.0):
    x = (rng.standard_normal((n, V)) * spread).astype(np.float32)
    x = torch.from_numpy(np.ascontiguousarray(_shape(kind, x, rng), dtype=np.float32))
    return x.to(torch.bfloat16) if dtype == "bf16" else x


def _check(V, dtype, support, kind, seed, m=1, K=5, depth=3, T=1.0, full=False, method="rheo",
           env=None, same=False):
    from paper_2609_21827_amd.binding import Tree
    rng = np.random.default_rng(seed)
    unit = 8 if dtype == "bf16" else 4
    stride = (V + unit - 1) // unit * unit
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    base = _rows(rng, 1, V, dtype, kind)
    rows = []
    for n in [1] + [K] * (depth - 1) + [1 + K + (depth - 1) * K * K]:
        r = base.repeat(n, 1) if same else _rows(rng, n, V, dtype, kind)
        rows.append(r)
    R = min(20, K + (depth - 1) * K * K)
    rows[-1] = rows[-1][:R + 1]
    dev_rows = []
    for r in rows:
        p = torch.zeros((r.shape[0], stride), dtype=td)
        p[:, :V] = r
        dev_rows.append(p.to("cuda"))

    os.environ.update(env or {})
    try:
        tree = Tree(batch=1, vocab=V, pool=K, leads=m, depth=depth, support=support, dtype=td,
                    row_stride=stride, construct_full=full, method=method)
    finally:
        for k in env or {}:
            del os.environ[k]
    try:
        for _ in range(2):                  # a second step on the same handle
            tree.begin_step()
            for r in dev_rows[:-1]:
                tree.expand_level(r, T, KEY)
            nodes = {k: v.cpu().numpy()[0] for k, v in tree.read_nodes().items()}
            tree.prune(R)
            par, tok = (x.cpu().numpy()[0] for x in tree.pruned_view())
            mask, dep = (x.cpu().numpy()[0] for x in tree.tree_mask())
            acc, alen, fin = (x.cpu().numpy()[0] for x in tree.verify(dev_rows[-1], T, KEY))
        assert tree.device_error() == 0
    finally:
        tree.close()

    cfg = rheo.TreeConfig(K=K, m=m, depth=depth, n_expand=K, support=support, construct_full=full,
                          mode="topk" if method == "topk" else "rheo",
                          verifier="rrsw" if method == "rrsw" else "rheo")
    f32 = [r.float().numpy() for r in rows]
    out = {}

    def draft_dist(node, nodes_):
        j = 0
        if node.depth:
            level = rheo.frontier_of_level(nodes_[:1 + K + (node.depth - 1) * K * K], node.depth, K)
            j = [x.uid for x in level].index(node.uid)
        return rheo.node_dist_from_logits(f32[node.depth][j], m, T, support, False, "canonical", full)

    def process():
        onodes = yield from rheo.build_tree(cfg, T, draft_dist, 0)
        pt = rheo.prune(onodes, R)
        out["n"], out["pt"] = onodes, pt
        a, u = yield from rheo.verify(
            onodes, pt, lambda i: rheo.target_weights(f32[-1][i], T), cfg.verifier)
        return a, u

    oacc, ou = run_philox(process(), KEY, 0)
    tab = node_table(out["n"])
    for k in tab:
        assert np.array_equal(nodes[k], tab[k]), (k, np.nonzero(nodes[k] != tab[k])[0][:8])
    pt = out["pt"]
    assert list(par) == list(pt.parent)
    assert list(tok) == [-1] + [out["n"][u].token for u in pt.order[1:]]
    om, od = rheo.tree_mask(out["n"], pt)
    assert np.array_equal(mask, np.array(om, dtype=np.uint8)) and list(dep) == od
    assert list(acc[:int(alen)]) == list(oacc) and int(fin) == ou


KINDS = ["plain", "sorted", "sorted_up", "cluster", "ties", "const", "few", "signed_zeros",
         "zero_cross"]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("dtype,V,support", [("bf16", 9001, 128), ("f32", 5003, 100),
                                             ("bf16", 9001, 400)])
def test_row_distributions(dev, kind, dtype, V, support):
    _check(V, dtype, support, kind, 11)


@pytest.mark.parametrize("dtype,V,support,env", [
    # one and two batches of a 512-thread block, and one vector more or less
    ("bf16", 32768, 128, None), ("bf16", 32769, 128, None), ("bf16", 32760, 256, None),
    ("f32", 16384, 128, None), ("f32", 16387, 128, None),
    # the same for 256-thread blocks, up to their last vector
    ("bf16", 16384, 128, {"RHEO_ROW_NARROW": "1"}), ("bf16", 131072, 64, {"RHEO_ROW_NARROW": "1"}),
    ("f32", 65536, 256, {"RHEO_ROW_NARROW": "1"}),
    # supports around the classes of the row kernel
    ("bf16", 20011, 256, None), ("bf16", 20011, 257, None), ("bf16", 20011, 1024, None),
    # the longest rows, and fp32 rows of 1024-thread blocks
    ("bf16", 262143, 128, None), ("bf16", 262143, 512, None), ("f32", 131072, 128, None),
    ("f32", 131073, 128, None), ("f32", 262143, 256, None), ("f32", 196608, 300, None),
])
def test_row_sizes(dev, dtype, V, support, env):
    _check(V, dtype, support, "plain", 12, depth=2, env=env)


# whole-vocabulary construction totals: from counts of the values (bf16), with
# values listed apart, counts that overflow, values past the counted range
@pytest.mark.parametrize("kind", ["plain", "edges", "small", "large", "const", "few", "sorted_up",
                                  "signed_zeros"])
@pytest.mark.parametrize("dtype,V,support,T", [("bf16", 9001, 64, 1.0), ("f32", 5003, 64, 1.0),
                                               ("bf16", 140001, 300, 0.7)])
def test_construct_full_rows(dev, kind, dtype, V, support, T):
    _check(V, dtype, support, kind, 13, depth=2, T=T, full=True)


@pytest.mark.parametrize("R", [1, 7, 61, 200, 465])
@pytest.mark.parametrize("same", [False, True])
def test_prune_budgets(dev, R, same):
    """Budgets across the tree, distinct and massively tied scores (the same
    row at every node), against the node records of the same step."""
    from paper_2609_21827_amd.binding import Tree
    rng = np.random.default_rng(5)
    V, K, depth, B = 2048, 8, 8, 3
    tree = Tree(batch=B, vocab=V, pool=K, leads=1, depth=depth, support=64, dtype=torch.float32)
    try:
        tree.begin_step()
        for n in [1] + [K] * (depth - 1):
            r = torch.zeros((B * n, V)) if same else torch.from_numpy(
                rng.standard_normal((B * n, V)).astype(np.float32) * 3)
            tree.expand_level(r.to("cuda"), 1.0, KEY)
        nodes = {k: v.cpu().numpy() for k, v in tree.read_nodes().items()}
        R = min(R, nodes["token"].shape[1] - 1)
        tree.prune(R)
        par, tok = (x.cpu().numpy() for x in tree.pruned_view())
        mask, dep = (x.cpu().numpy() for x in tree.tree_mask())
        assert tree.device_error() == 0
    finally:
        tree.close()
    for b in range(B):
        n = {k: v[b] for k, v in nodes.items()}
        path = [()]
        for u in range(1, len(n["token"])):
            path.append(path[n["parent"][u]] + (int(n["slot"][u]),))
        order = sorted(range(1, len(path)), key=lambda u: (-n["score"][u], n["depth"][u], path[u]))
        kept = [0] + order[:R]
        place = {u: i for i, u in enumerate(kept)}
        assert list(par[b]) == [-1] + [place[n["parent"][u]] for u in kept[1:]]
        assert list(tok[b]) == [-1] + [n["token"][u] for u in kept[1:]]
        assert list(dep[b]) == [n["depth"][u] for u in kept]
        want = np.zeros((R + 1, R + 1), dtype=np.uint8)
        for i in range(R + 1):
            j = i
            while j >= 0:
                want[i, j] = 1
                j = par[b][j]
        assert np.array_equal(mask[b], want)


@pytest.mark.parametrize("kind", ["plain", "flat", "const", "onehot", "mixed"])
@pytest.mark.parametrize("K,depth", [(15, 15), (12, 8), (3, 3)])
def test_prune_piles(dev, kind, K, depth):
    """Scores that pile up: equal and nearly equal ones below 2^-63, scores of 0
    (one token a row has all the weight), both beside ordinary ones; trees of
    more nodes than a block has threads; budgets up to every node."""
    from paper_2609_21827_amd.binding import Tree
    rng = np.random.default_rng(9)
    V, B = 2048, 2
    tree = Tree(batch=B, vocab=V, pool=K, leads=1, depth=depth, support=64, dtype=torch.float32)
    rows = []
    for n in [1] + [K] * (depth - 1):
        x = rng.standard_normal((B, n, V)).astype(np.float32) * 3
        if kind == "flat":
            x *= 1e-3
        elif kind == "const":
            x[:] = 0.5
        elif kind != "plain":
            hot = np.ones((B, n), bool) if kind == "onehot" else rng.random((B, n)) < 0.5
            for b, j in zip(*np.nonzero(hot)):
                x[b, j, rng.integers(V)] += 60
        rows.append(torch.from_numpy(x).to("cuda"))
    N = 1 + K + (depth - 1) * K * K
    views = {}
    try:
        for R in sorted({1, min(60, N - 1), N // 2, N - 1}):
            tree.begin_step()
            for x in rows:
                tree.expand_level(x, 1.0, KEY)
            nodes = {k: v.cpu().numpy() for k, v in tree.read_nodes().items()}
            tree.prune(R)
            views[R] = [v.cpu().numpy() for v in tree.pruned_view()]
        assert tree.device_error() == 0
    finally:
        tree.close()
    for b in range(B):
        n = {k: v[b] for k, v in nodes.items()}
        path = [()]
        for u in range(1, N):
            path.append(path[n["parent"][u]] + (int(n["slot"][u]),))
        order = [0] + sorted(range(1, N), key=lambda u: (-n["score"][u], n["depth"][u], path[u]))
        place = {u: i for i, u in enumerate(order)}
        for R, (par, tok) in views.items():
            assert list(par[b]) == [-1] + [place[n["parent"][u]] for u in order[1:R + 1]], (b, R)
            assert list(tok[b]) == [-1] + [n["token"][u] for u in order[1:R + 1]], (b, R)


# dense mode on both of its routes, one block a row (bf16: on one, two and more
# batches of 32768, up to the longest row) and the chunked kernels: the counts'
# edges as above, ties of the last listed construction weight, the draw's batch
# and slot
@pytest.mark.parametrize("row", ["1", "0"])
@pytest.mark.parametrize("kind", ["plain", "edges", "small", "large", "const", "sorted", "sorted_up",
                                  "ties", "signed_zeros", "zero_cross"])
@pytest.mark.parametrize("V,m,K,T,method", [(9001, 1, 5, 1.0, "rheo"), (32769, 0, 12, 0.7, "rrsw"),
                                            (70000, 3, 4, 1.5, "topk"), (163841, 2, 4, 1.0, "rheo")])
def test_dense_rows(dev, kind, V, m, K, T, method, row):
    _check(V, "bf16", 0, kind, 14, m=m, K=K, depth=2, T=T, method=method,
           env={"RHEO_EXPAND_ROW": row})


@pytest.mark.parametrize("row", ["1", "0"])
@pytest.mark.parametrize("dtype,V", [("bf16", 32760), ("bf16", 32768), ("bf16", 131073),
                                     ("bf16", 262143), ("bf16", 300), ("f32", 5003)])
def test_dense_sizes(dev, dtype, V, row):
    _check(V, dtype, 0, "plain", 15, depth=2, env={"RHEO_EXPAND_ROW": row})


# the route that the sizes choose: few rows of one batch and a little more, by rows
# and chunked
@pytest.mark.parametrize("V", [32768, 32776])
def test_dense_route(dev, V):
    _check(V, "bf16", 0, "plain", 16, depth=3)


# rows of hardly more elements than the support, of more elements than a block
# holds candidates but of few vectors, and of few finite logits: the threshold
# bounds nothing and the selection is exact from the row, digit by digit
@pytest.mark.parametrize("kind", ["plain", "ties", "const", "few", "cluster", "signed_zeros",
                                  "zero_cross", "small", "large"])
@pytest.mark.parametrize("dtype,V,support,env", [
    ("bf16", 1000, 128, None), ("bf16", 2051, 1024, None), ("bf16", 8253, 1024, None),
    ("bf16", 1000, 128, {"RHEO_ROW_NARROW": "1"}), ("bf16", 3001, 700, {"RHEO_EXPAND_ROW": "0"}),
    ("f32", 2003, 512, None), ("f32", 2051, 1024, None), ("f32", 1003, 900, None),
    ("f32", 3001, 700, {"RHEO_EXPAND_ROW": "0"}), ("bf16", 700, 0, {"RHEO_EXPAND_ROW": "1"}),
])
def test_short_rows(dev, kind, dtype, V, support, env):
    _check(V, dtype, support, kind, 17, depth=2, env=env)


# rows that the counts of the dense and the whole-vocabulary kernels cover only
# in part or not at all, on one, five and eight batches of 32768
@pytest.mark.parametrize("kind", ["zeros", "zeros_small", "half_zeros", "few_values", "small", "large",
                                  "edges", "const"])
@pytest.mark.parametrize("V,support,full", [(9001, 0, False), (140001, 0, False), (262143, 0, False),
                                            (9001, 64, True), (140001, 300, True)])
def test_uncounted_rows(dev, kind, V, support, full):
    _check(V, "bf16", support, kind, 18, m=2, depth=2, T=0.9, full=full,
           env={"RHEO_EXPAND_ROW": "1"})
