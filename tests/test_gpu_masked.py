"""GPU parity on masked vocabularies: logits of -inf (the truncation of
Sec. 3.2; padded vocabularies; constrained decoding), in both dtypes, on
every expand path (chunked, one block per row, large supports, dense), with
masks shared by draft and target and masks of the target alone; rows with
fewer finite logits than the support (the support ends with masked tokens
in id order); and the undefined cases, which set device error bit 9 (512).
The bar is the one of the other parity tests: bit-exact.
"""

import numpy as np
import pytest
import torch

import synth
from test_gpu_configs import run_all
from test_gpu_parity import run_parity

pytestmark = pytest.mark.gpu

W = synth.WORKLOADS


@pytest.fixture(scope="module")
def dev():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2609_21827_amd import binding
    binding.load_library()
    return "cuda"


@pytest.mark.parametrize("over", [
    # fewer finite logits than the support (about 100 of 128, 50 of 128)
    dict(V=1003, dtype="bf16", support=128, mask=0.9),
    dict(V=1001, dtype="f32", support=128, mask=0.95),
    # a small support, target-only masks too, three sequences
    dict(V=1003, dtype="bf16", support=6, mask=0.5, mask_target=0.1, B=3),
    # a large support (sorted tail) with about 120 finite of 300
    dict(V=4099, dtype="bf16", support=300, mask=0.97),
    # a padded vocabulary: the last 500 ids masked in every row
    dict(V=1003, dtype="bf16", support=128, mask_tail=500),
    # the support is the whole row, half of it masked
    dict(V=300, dtype="bf16", support=1024, mask=0.5, K=6),
    # leads: none, two
    dict(V=1003, dtype="bf16", support=64, mask=0.8, m=0, mask_target=0.2),
    dict(V=1003, dtype="f32", support=64, mask=0.8, m=2, K=6),
    # dense distributions (support = V)
    dict(V=1003, dtype="bf16", support=0, mask=0.9),
    dict(V=1001, dtype="f32", support=0, mask=0.5, mask_target=0.2),
])
@pytest.mark.parametrize("row", ["auto", "0"])
def test_masked_edge_shapes(dev, over, row):
    kw = dict(recipe="zipf", K=5, depth=3, R=12, sigma=1.5, sigma_t=0.8)
    kw.update(over)
    w = W["tiny"].with_(name="masked_edge", **kw)
    tree_kw = {}
    if w.V % 8:
        tree_kw["row_stride"] = (w.V + 7) // 8 * 8
    env = {"RHEO_EXPAND_ROW": row} if row != "auto" else None
    run_parity(w, range(3), list(range(w.B)), dev=dev, tree_kw=tree_kw, env=env)


@pytest.mark.parametrize("base,over", [
    ("llama2", dict(mask=0.5, mask_target=0.05)),
    ("llama2", dict(mask=0.999)),                 # about 32 finite logits, S = 128
    ("llama3", dict(mask=0.5, mask_target=0.05)),
    ("llama3", dict(mask=0.999)),                 # about 128 finite, around S
    ("llama3", dict(mask_tail=256)),
    ("llama2", dict(mask=0.9, support=0)),
])
def test_masked_workloads(dev, base, over):
    w = W[base].with_(name=base + "_masked", **over)
    run_parity(w, range(2), [0], dev=dev)


@pytest.mark.parametrize("over", [
    dict(mask=0.9, mask_target=0.02),
    dict(mask=0.999),                             # rows below S finite: exact fallback
])
def test_masked_headline_all_sequences(dev, over):
    # the batched shape: one block per row on every level
    run_all(W["headline"].with_(name="headline_masked", **over), [0], dev)


def test_masked_headline_dense(dev):
    run_all(W["headline_dense"].with_(name="headline_dense_masked", mask=0.5, B=16), [0], dev)


def test_undefined_rows_set_error_bit(dev):
    """A draft row whose x_{m+1} is masked, and a target row without a finite
    logit, set device error bit 9; a walk that reaches such a target row
    ends with the failure result; the other sequences are unaffected."""
    from paper_2609_21827_amd.driver import make_tree, replay_step, run_step
    w = W["headline"].with_(name="undef", B=8, depth=3, R=20)
    tree = make_tree(w, device=dev)
    rec = {}
    ref = run_step(tree, w, 0, device=dev, record=rec)
    torch.cuda.synchronize()
    assert tree.device_error() == 0
    # the root target row of sequence 3: all -inf (every walk starts there)
    target = rec["target"].clone()
    target[3, 0, :] = float("-inf")
    out = [x.cpu() for x in replay_step(tree, dict(rec, target=target), w.R)]
    assert tree.device_error() == 512
    assert int(out[1][3]) == -1 and int(out[2][3]) == -1 and bool((out[0][3] == -1).all())
    for b in range(w.B):
        if b != 3:
            assert all(torch.equal(o[b], r[b]) for o, r in zip(out, ref)), b
    tree.close()
    # sequence 5's root draft row with m = 1 finite logit: x_2 is -inf
    tree = make_tree(w, device=dev)
    draft = [d.clone() for d in rec["draft"]]
    keep = int(torch.argmax(draft[0][5, 0, :w.V].float()))
    v = draft[0][5, 0, keep].clone()
    draft[0][5, 0, :] = float("-inf")
    draft[0][5, 0, keep] = v
    out = [x.cpu() for x in replay_step(tree, dict(rec, draft=draft), w.R)]
    assert tree.device_error() & 512
    for b in range(w.B):
        if b != 5:
            assert all(torch.equal(o[b], r[b]) for o, r in zip(out, ref)), b
    tree.close()


@pytest.mark.parametrize("over,env", [
    (dict(V=1003, dtype="bf16", support=128), None),
    (dict(V=1003, dtype="bf16", support=128), {"RHEO_EXPAND_ROW": "0"}),
    (dict(V=4099, dtype="f32", support=300, m=0), None),
    (dict(V=4099, dtype="bf16", support=64, construct_full=True), None),
    (dict(V=1003, dtype="bf16", support=0), {"RHEO_EXPAND_ROW": "1"}),
    (dict(V=1003, dtype="bf16", support=0, m=2), {"RHEO_EXPAND_ROW": "0"}),
    (dict(V=1001, dtype="f32", support=0), None),
])
def test_fully_masked_draft_rows(dev, over, env):
    """Draft rows without a finite logit, at the root, at one node of level 1
    and at every node of level 2: reported by error bit 9, the tree whole all
    the same (scores that are NaN rank above the others and tie: every
    frontier entry and pruned index is taken), the other sequences unaffected."""
    import os
    from paper_2609_21827_amd.driver import make_tree, run_step
    w = W["tiny"].with_(name="undef_rows", recipe="zipf", K=5, n_expand=5, depth=4, R=30, B=8,
                        sigma=1.5, sigma_t=0.8, **over)
    K, NE, B, D = w.K, w.n_expand, w.B, w.depth
    os.environ.update(env or {})
    try:
        tree = make_tree(w, device=dev, row_stride=(w.V + 7) // 8 * 8)
    finally:
        for k in env or {}:
            del os.environ[k]
    rec = {}

    def step(drafts):
        tree.begin_step()
        front = []
        for rows in drafts:
            tree.expand_level(rows, rec["T"], rec["rng_key"])
            front.append([x.cpu().numpy() for x in tree.frontier_view()])
        nodes = {k: v.cpu().numpy() for k, v in tree.read_nodes().items()}
        tree.prune(w.R)
        views = [x.cpu().numpy() for x in (*tree.pruned_view(), *tree.tree_mask())]
        out = [x.cpu().numpy() for x in tree.verify(rec["target"], rec["T"], rec["rng_key"])]
        return front, nodes, views, out

    run_step(tree, w, 0, device=dev, record=rec)
    ref = step(rec["draft"])
    assert tree.device_error() == 0
    drafts = [d.clone() for d in rec["draft"]]
    drafts[0][1] = float("-inf")
    drafts[1][4, 2] = float("-inf")
    drafts[2][6] = float("-inf")
    for _ in range(2):                  # both values of the children words' mark
        front, nodes, views, out = step(drafts)
    err = tree.device_error()
    tree.close()
    assert err & 512 and not err & (16 | 64 | 128 | 256), err
    for b in (0, 2, 3, 5, 7):
        for x, y in zip([*nodes.values(), *views, *out], [*ref[1].values(), *ref[2], *ref[3]]):
            assert np.array_equal(x[b], y[b]), b
    par, tok, mask, dep = views
    for b in range(B):
        n = {k: v[b] for k, v in nodes.items()}
        score = np.where(np.isnan(n["score"]), np.inf, n["score"])
        path = [()]
        for u in range(1, len(score)):
            path.append(path[n["parent"][u]] + (int(n["slot"][u]),))
        best = lambda uids: sorted(uids, key=lambda u: (-score[u], n["depth"][u], path[u]))
        for level in range(D - 1):
            first = 1 if level == 0 else 1 + K + (level - 1) * NE * K
            kept = best(range(first, first + (1 if level == 0 else NE) * K))[:NE]
            assert list(front[level][0][b]) == [(u - first) // K for u in kept], (b, level)
            assert list(front[level][1][b]) == [n["token"][u] for u in kept], (b, level)
        kept = [0] + best(range(1, len(score)))[:w.R]
        place = {u: i for i, u in enumerate(kept)}
        want = [-1] + [place.get(int(n["parent"][u]), -1) for u in kept[1:]]
        assert list(par[b]) == want, b
        assert list(tok[b]) == [-1] + [n["token"][u] for u in kept[1:]], b
        assert list(dep[b]) == [n["depth"][u] for u in kept], b
        for i in range(w.R + 1):
            for j in range(w.R + 1):
                p = i
                for _ in range(16):
                    p = want[p] if p > j else p
                assert mask[b][i][j] == (p == j), (b, i, j)
        assert np.all((out[2][b] >= -1) & (out[2][b] < w.V))
