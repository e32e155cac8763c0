"""rheo_create_static: a tree whose device state lives in the library's
static scratch array (no device allocation) gives the same results, bit
for bit, as a tree from rheo_create -- on two calls in a row on one device,
the second with a smaller input (a dense tree, in the region the first one
used), over two steps each."""

import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

W = synth.WORKLOADS


@pytest.fixture(scope="module")
def dev():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2609_21827_amd import binding
    binding.load_library()
    return "cuda"


def _steps(tree, w, steps, dev):
    from paper_2609_21827_amd.driver import run_step
    out = []
    for s in steps:
        acc, alen, fin = run_step(tree, w, s, device=dev)
        nodes = {k: v.cpu().numpy() for k, v in tree.read_nodes().items()}
        pv = [x.cpu().numpy() for x in tree.pruned_view()]
        out.append((acc.numpy(), alen.numpy(), fin.numpy(), nodes, pv))
    torch.cuda.synchronize()
    assert tree.device_error() == 0
    return out


def test_static_tree_matches_allocated_tree(dev):
    from paper_2609_21827_amd.driver import make_tree
    first = W["headline"].with_(name="static_a", B=16, depth=5, R=40)
    second = W["llama2"].with_(name="static_b", B=3, support=0, depth=4, R=20)
    assert second.B * second.V < first.B * first.V
    for w in (first, second):
        ref_tree = make_tree(w, device=dev)
        ref = _steps(ref_tree, w, [0, 1], dev)
        ref_tree.close()
        st = make_tree(w, device=dev, static=True)
        got = _steps(st, w, [0, 1], dev)
        st.close()
        for (a1, l1, f1, n1, p1), (a2, l2, f2, n2, p2) in zip(got, ref):
            assert np.array_equal(a1, a2) and np.array_equal(l1, l2) and np.array_equal(f1, f2)
            for k in n1:
                assert np.array_equal(n1[k], n2[k]), (w.name, k)
            for x, y in zip(p1, p2):
                assert np.array_equal(x, y), w.name


@pytest.mark.parametrize("static", [True, False])
def test_recreated_tree_starts_clean(dev, static):
    """The first step of a tree whose memory an earlier tree of the same shape
    used: every tree numbers its exchanges alike, so a word left there would
    pass for its own (a chunk total not yet overwritten gave the final sample
    of another target row)."""
    from paper_2609_21827_amd.driver import make_tree, replay_step, run_step
    w = W["headline"].with_(name="again", B=16, depth=2, R=12)
    rec, ref = [{}, {}], []
    tree = make_tree(w, device=dev)
    for s in (0, 1):
        ref.append(run_step(tree, w, s, device=dev, record=rec[s]))
    torch.cuda.synchronize()
    tree.close()
    for i in range(8):
        tree = make_tree(w, device=dev, static=static)
        out = [x.cpu() for x in replay_step(tree, rec[i % 2], w.R)]
        assert tree.device_error() == 0
        tree.close()
        assert all(torch.equal(o, r) for o, r in zip(out, ref[i % 2])), i


@pytest.mark.parametrize("dense", [False, True])
def test_smaller_tree_leaves_larger_one_its_lds(dev, dense):
    """A tree whose prune kernel, and in dense mode whose row kernel, takes most of
    a compute unit's LDS still runs after a smaller tree of the kind is created."""
    import os
    from paper_2609_21827_amd.binding import Tree
    V, K, depth, R = (262143, 4, 2, 12) if dense else (2048, 15, 13, 500)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)

    def make(V, depth):
        return Tree(batch=1, vocab=V, pool=K, leads=1, depth=depth, support=0 if dense else 64,
                    dtype=torch.bfloat16, row_stride=(V + 7) // 8 * 8)

    os.environ["RHEO_EXPAND_ROW"] = "1"
    try:
        large = make(V, depth)
        draft = [torch.randn((n, large.row_stride), generator=g, device="cuda").mul_(3).bfloat16()
                 for n in [1] + [K] * (depth - 1)]
        target = torch.randn((R + 1, large.row_stride), generator=g, device="cuda").mul_(3).bfloat16()

        def step():
            large.begin_step()
            for rows in draft:
                large.expand_level(rows, 1.0, 77)
            large.prune(R)
            return [x.cpu() for x in (*large.pruned_view(), *large.verify(target, 1.0, 77))]

        ref = step()
        small = make(1000, 2)
        out = step()
        assert large.device_error() == 0
        small.close()
        large.close()
    finally:
        del os.environ["RHEO_EXPAND_ROW"]
    assert all(torch.equal(o, r) for o, r in zip(out, ref))
