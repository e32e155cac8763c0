"""The decoding steps whose speed counts, and how each is set up and run.

One case is one whole step of the tree machinery for a batch of sequences, the
calls a serving loop makes between its draft and target forwards: begin_step,
expand_level at every depth, prune, pruned_view and tree_mask (what the target
forward needs) and verify.  The frontier of each level is read in place
(frontier_view).  Every output is a whole number that follows from exact
integer decisions, so two correct implementations agree on every one of them.

Logits are drawn on the GPU from the seed alone.  All rows of a sequence share
a base (a Zipf log-prior over a random token order plus noise); each draft row
and each target row adds noise of its own, so that target rows agree with draft
rows about as a draft model's do, whichever nodes the tree keeps.  ``peak`` is
the share of sequences whose rows are nearly one-hot (a confident model: long
accepted paths), ``mask`` the share of the vocabulary at -inf in a sequence's
draft and target rows (constrained decoding, a padded vocabulary).
"""

import math

import torch

from paper_2609_21827_amd.binding import Tree

_DEFAULTS = dict(B=1, V=128256, dtype="bf16", K=8, m=1, n_expand=0, depth=7, R=60, T=1.0,
                 support=128, full=False, tempered=False, method="rheo", mask=0.0, peak=0.0)


def _case(**kw):
    c = dict(_DEFAULTS)
    c.update(kw)
    return c


def listed():
    return [
        # one sequence at a time, a small vocabulary with fp32 logits: a local
        # assistant; launches and latency are all there is
        _case(name="b1_v32k_f32", V=32000, dtype="f32", depth=6),
        # one sequence, a large vocabulary, sampling below temperature 1
        _case(name="b1_v128k", T=0.6),
        # a handful of sequences and nothing round: odd vocabulary, padded
        # rows, fewer parents than slots, two leads, the leads-first verifier
        _case(name="b6_v50k_odd", B=6, V=50001, K=6, m=2, n_expand=4, depth=5, R=39, T=0.8,
              method="rrsw"),
        # the headline serving batch
        _case(name="b64_v128k", B=64),
        # the same batch with a wider, deeper tree
        _case(name="b64_k10", B=64, K=10, depth=8, R=64),
        # the largest batch: wide tree, larger vocabulary, a confident model in
        # a quarter of the sequences
        _case(name="b128_v152k", B=128, V=151936, K=10, depth=8, R=80, T=0.8, peak=0.25),
        # a wide support: little of the draft's mass truncated
        _case(name="b64_s1024", B=64, support=1024),
        # the tree built on the whole vocabulary's softmax, only the sampled
        # slot's tail truncated
        _case(name="b32_full", B=32, full=True),
        # no truncation at all: the whole vocabulary is the support
        _case(name="b64_dense", B=64, support=0),
        # the same for a few sequences with fp32 logits
        _case(name="b4_dense_f32", B=4, V=32000, dtype="f32", depth=6, support=0),
        # fp32 logits of a large vocabulary (an LM head in full precision)
        _case(name="b16_v128k_f32", B=16, dtype="f32", support=256),
        # the largest vocabulary the library takes, odd, half of it masked
        _case(name="b16_v262k_mask", B=16, V=262143, depth=6, mask=0.5),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: batches of 1 to 128, vocabularies of 8 thousand to
    262143, both types, every mode, the methods and options, sizes mostly odd."""
    c = _case()
    c["V"] = _log_int(rng, 8192, 262143)
    c["dtype"] = rng.choice(["bf16", "bf16", "f32"])
    c["K"] = rng.randint(4, 12)
    c["m"] = rng.choice([0, 1, 1, 1, 2, 3])
    c["n_expand"] = rng.choice([0, 0, rng.randint(2, c["K"])])
    c["depth"] = rng.randint(3, 8)
    c["T"] = rng.choice([0.2, 0.6, 0.8, 1.0, 1.0, 1.5])
    mode = rng.choice(["sparse", "sparse", "sparse", "full", "dense"])
    if mode == "dense":
        c["support"] = 0
    else:
        c["support"] = min(rng.choice([128, 128, 128, 256, 512, 1024, _log_int(rng, 64, 1024)]),
                           _max_support(c))
        c["full"] = mode == "full"
    c["tempered"] = rng.random() < 0.2
    c["method"] = rng.choice(["rheo", "rheo", "rheo", "rrsw", "topk"])
    c["mask"] = rng.choice([0.0, 0.0, 0.0, 0.3, 0.9])
    c["peak"] = rng.choice([0.0, 0.0, 0.25])
    nodes = c["K"] + (c["depth"] - 1) * _ne(c) * c["K"]
    c["R"] = min(nodes, rng.randint(20, 96))
    # as many sequences as cost no more than the largest listed case
    cost = _draft_bytes(c, 1) * (4 if mode != "sparse" else 2 if c["support"] > 256 else 1)
    c["B"] = min(_log_int(rng, 1, 128), max(1, int(1.2e9 / cost)))
    return c


def _ne(c):
    return c["n_expand"] or c["K"]


def _max_support(c):
    """The widest support rheo_create takes for this vocabulary."""
    chunk = 65536 if c["dtype"] == "bf16" else 32768
    return min(1024, 2048 // ((c["V"] + chunk - 1) // chunk))


def _esz(c):
    return 2 if c["dtype"] == "bf16" else 4


def _stride(c):
    """Elements between rows: V rounded up to whole 16-byte units."""
    unit = 16 // _esz(c)
    return (c["V"] + unit - 1) // unit * unit


def _draft_bytes(c, B):
    return B * (1 + (c["depth"] - 1) * _ne(c)) * c["V"] * _esz(c)


def _rows(c, g, base, n, sigma):
    """[B, n, stride] logit rows: the sequence's base plus noise per row."""
    B, V = c["B"], c["V"]
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    out = torch.zeros((B, n, _stride(c)), dtype=dt, device="cuda")
    step = max(1, (1 << 28) // (n * V))          # at most 1 GiB of fp32 at a time
    for b0 in range(0, B, step):
        b1 = min(B, b0 + step)
        x = torch.randn((b1 - b0, n, V), generator=g, device="cuda")
        out[b0:b1, :, :V] = x.mul_(sigma).add_(base[b0:b1, None, :])
    return out


def prepare(case, seed):
    c = case
    B, V = c["B"], c["V"]
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    log_rank = torch.log1p(torch.arange(V, dtype=torch.float32, device="cuda"))
    base = torch.empty((B, V), dtype=torch.float32, device="cuda")
    for b in range(B):
        base[b] = log_rank[torch.randperm(V, generator=g, device="cuda")]
    base.mul_(-1.1)
    base.add_(torch.randn((B, V), generator=g, device="cuda"), alpha=1.3)
    if c["peak"] > 0:
        hot = torch.rand(B, generator=g, device="cuda") < c["peak"]
        tok = torch.randint(0, V, (B,), generator=g, device="cuda")
        base[torch.arange(B, device="cuda"), tok] += 12.0 * hot
    if c["mask"] > 0:
        base[torch.rand((B, V), generator=g, device="cuda") < c["mask"]] = -math.inf
    P = [1] + [_ne(c)] * (c["depth"] - 1)
    drafts = [_rows(c, g, base, p, 0.5) for p in P]
    target = _rows(c, g, base, c["R"] + 1, 0.5)
    key = int(torch.randint(0, 2 ** 62, (1,), generator=g, device="cuda"))
    tree = Tree(batch=B, vocab=V, pool=c["K"], leads=c["m"], depth=c["depth"],
                support=c["support"], n_expand=c["n_expand"], construct_tempered=c["tempered"],
                row_stride=_stride(c), method=c["method"], construct_full=c["full"],
                dtype=torch.bfloat16 if c["dtype"] == "bf16" else torch.float32)
    n, i32 = c["R"] + 1, dict(dtype=torch.int32, device="cuda")
    return dict(case=c, tree=tree, drafts=drafts, target=target, key=key,
                frontier=tree.frontier_view(),
                view=(torch.empty((B, n), **i32), torch.empty((B, n), **i32)),
                mask=(torch.empty((B, n, n), dtype=torch.uint8, device="cuda"),
                      torch.empty((B, n), **i32)),
                out=(torch.empty((B, c["depth"]), **i32), torch.empty((B,), **i32),
                     torch.empty((B,), **i32)))


def run(state):
    c, tree = state["case"], state["tree"]
    T, key = c["T"], state["key"]
    tree.begin_step()
    for rows in state["drafts"]:
        tree.expand_level(rows, T, key)
    tree.prune(c["R"])
    parent, token = tree.pruned_view(out=state["view"])
    mask, depth = tree.tree_mask(out=state["mask"])
    accepted, length, final = tree.verify(state["target"], T, key, out=state["out"])
    return dict(frontier_parent=state["frontier"][0], frontier_token=state["frontier"][1],
                parent=parent, token=token, mask=mask, depth=depth,
                accepted=accepted, length=length, final=final)


def work(case):
    """Every draft row read once, the root's target row of every sequence (how many
    more a walk reads follows from the draws) and the outputs; one operation per logit."""
    c = case
    n = c["R"] + 1
    rows = c["B"] * (1 + (c["depth"] - 1) * _ne(c)) + c["B"]
    out = c["B"] * (n * 8 + n * n + n * 4 + c["depth"] * 4 + 8)
    return dict(bytes=rows * c["V"] * _esz(c) + out, flops=rows * c["V"])


def tolerance(case):
    """Whole numbers from exact integer decisions: the same for everybody."""
    return "exact"


def exact(case, seed):
    """No output is a rounded number: there is nothing to compare in 64 bits."""
    return None
