"""Captured prefill calls give every replay's own result.

The one-launch form hands its chunk terms over by flags that hold the call's tag, which a graph repeats; the packed
form chooses its row groups from the offsets, which a graph's caller may rewrite.  Each replay reads new inputs
(copied in place), with eager calls on the same workspace between, and has to equal the eager call on them bit by bit.
"""
import pytest
import torch

import paper_2607_14568_amd as gdn
from paper_2607_14568_amd import inputs

pytestmark = pytest.mark.gpu
NAMES = ("q", "k", "v", "g", "beta", "S0")
EVEN, LONG = [200, 150, 193, 256, 130, 180, 129, 190], [900, 64, 100, 100, 64, 100, 50, 50]


def _inputs(seed, lengths, io, H, d):
    x = inputs.make_prefill(B=1, T=700 if lengths is None else 0, H=H, dk=d, dv=d, io=io, seed=seed, s0_std=0.05, g_shift=-3.0,
                            lengths=lengths)
    return {n: x[n].cuda() for n in NAMES + (() if lengths is None else ("cu_seqlens",))}


@pytest.mark.parametrize("form,io,H,d", [("one launch", "bf16", 4, 128), ("no workspace", "bf16", 16, 64),
                                         ("packed", "bf16", 8, 128), ("packed", "bf16", 2, 128), ("one launch", "f32", 2, 64)])
def test_replays(form, io, H, d):
    print("case: graph", form, io, H, d, flush=True)
    cuts = [LONG, EVEN, LONG, EVEN] if form == "packed" else [None] * 4
    assert sum(LONG) == sum(EVEN)
    sets = [_inputs(30 + i, c, io, H, d) for i, c in enumerate(cuts)]
    x = {n: t.clone() for n, t in sets[0].items()}
    n_seqs = 0 if cuts[0] is None else len(cuts[0])
    ws = torch.empty(gdn.gdn_chunk_prefill_workspace_bytes(1, x["q"].shape[1], H, d, d, 64, n_seqs,
                                                           gdn.GDN_F32 if io == "f32" else gdn.GDN_BF16),
                     dtype=torch.uint8, device="cuda")

    def call(x, o, S_T):
        kw = dict(cu_seqlens=x.get("cu_seqlens"), o=o, S_T=S_T)
        args = [x[n] for n in NAMES]
        if form == "no workspace":
            return gdn.gdn_chunk_prefill_noalloc(*args, **kw)
        return gdn.gdn_chunk_prefill(*args, workspace=ws, **kw)

    def out():
        return torch.empty_like(x["v"]), torch.empty_like(x["S0"])

    want = []
    for s in sets:
        r = out()
        call(s, *r)
        want.append(r)
    got = out()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(x, *got)
    for i, s in enumerate(sets):
        for n, t in s.items():
            x[n].copy_(t)
        for t in got:
            t.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(got[0], want[i][0]) and torch.equal(got[1], want[i][1]), i
        if i == 1:   # an eager call with a tag of its own in between
            call(sets[0], *out())
