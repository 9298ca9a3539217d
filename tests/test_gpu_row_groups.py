"""GPU parity of the bf16 prefill where its launch rules switch, against the fp64 oracle.

More chain workgroups than compute units: a workgroup then takes two groups of 16 state rows, with a ring of
three chunks (dense input always, packed input of two workgroups per compute unit by the lengths of its prompts,
chosen on the device, of three and more always).  Chunk
counts around the ring and its unrolled loop, partial last chunks, an empty sequence, both value widths, the
input transforms and snapshots.  And the chunk terms, formed by one wave per chunk: chunk lengths around every
16-token block edge.  Bars as the other prefill tests (max|x - ref| / max|ref| <= 2e-2 for bf16 io).
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2607_14568_amd as gdn
import parity
from paper_2607_14568_amd import inputs

pytestmark = pytest.mark.gpu
TOL = 2e-2
f64 = inputs.as_f64
RAW = gdn.GDN_QK_L2NORM | gdn.GDN_GATE_LOGITS


def _run(recipe, snap=0, workspace=None):
    raw = recipe.get("raw", False)
    print("case:", recipe, "snap", snap, flush=True)
    x = inputs.make_prefill(io="bf16", s0_std=0.05, **recipe)
    d = {k: (v.cuda() if isinstance(v, torch.Tensor) else v) for k, v in x.items()}
    kw = dict(flags=RAW if raw else 0, cu_seqlens=d["cu_seqlens"], workspace=workspace)
    args = (d["q"], d["k"], d["v"], d["g"], d["beta"], d["S0"])
    if snap:
        o, S_T, snaps = gdn.gdn_chunk_prefill_snapshots_ex(*args, snap_every=snap, **kw)
    else:
        o, S_T = gdn.gdn_chunk_prefill_ex(*args, **kw)
    torch.cuda.synchronize()
    cu = None if x["cu_seqlens"] is None else x["cu_seqlens"].numpy()
    ref = oracle.recurrence_ex(*(f64(x[n]) for n in ("q", "k", "v", "g", "beta", "S0")), cu_seqlens=cu, qk_l2norm=raw,
                               gate_logits=raw)
    parity.check(f64(o), ref[0], f64(S_T), ref[1], TOL, str(recipe), cu_seqlens=cu)
    if snap:   # snapshot j is the state after j * snap * 64 tokens: the final state of a prompt cut there
        starts, S0 = ([0] if cu is None else cu[:-1]), f64(x["S0"])
        for s, j in [(s, j) for s in range(len(starts)) for j in range(snaps.shape[1])]:
            n = (j + 1) * snap * 64
            if cu is not None and n >= cu[s + 1] - cu[s]:
                continue   # no such cut inside this prompt
            rows, first = (slice(None), S0) if cu is None else (slice(0, 1), S0[s:s + 1])
            cut = oracle.recurrence_ex(*(f64(x[m])[rows, starts[s]:starts[s] + n] for m in ("q", "k", "v", "g", "beta")), first,
                                       qk_l2norm=raw, gate_logits=raw)
            assert oracle.max_rel_err(f64(snaps[:, j] if cu is None else snaps[s:s + 1, j]), cut[1]) < TOL


def _cus():
    return torch.cuda.get_device_properties(0).multi_processor_count


@pytest.mark.parametrize("T", [1, 64, 65, 129, 193, 256, 330, 385, 449])
def test_two_row_groups_dense(T):
    """384 chain workgroups of 16 rows (3 prompts, 16 heads): 192 of 32 rows; 1 to 8 chunks."""
    assert 3 * 16 * 128 // 16 > _cus()
    _run(dict(B=3, T=T, H=16, dk=128, dv=128, seed=500 + T))


@pytest.mark.parametrize("dk,dv,raw,snap", [(64, 128, False, 0), (128, 64, True, 0), (64, 64, True, 2), (128, 128, False, 3)])
def test_two_row_groups_forms(dk, dv, raw, snap):
    """Other widths, transforms and snapshots (B chosen so that 16-row workgroups need two rounds)."""
    assert (3 if dv == 128 else 5) * 16 * dv // 16 > _cus()
    _run(dict(B=3 if dv == 128 else 5, T=457, H=16, H_k=8, dk=dk, dv=dv, seed=600 + dk + dv, raw=raw), snap)


def test_two_row_groups_packed():
    """512 workgroups of 16 rows over packed prompts of 0 to 6 chunks."""
    _run(dict(B=1, T=0, H=8, dk=128, dv=128, seed=700, lengths=[1, 0, 63, 64, 65, 193, 384, 130]))


@pytest.mark.parametrize("lengths,groups", [([200, 150, 193, 256, 130, 180, 129, 190], 2), ([577, 64, 1, 0, 65, 64, 0, 30], 1)])
@pytest.mark.parametrize("dk,dv,raw,snap", [(128, 128, False, 0), (64, 64, True, 0), (128, 64, False, 2), (64, 128, True, 0),
                                            (128, 128, True, 1)])
def test_packed_row_groups(dk, dv, raw, snap, lengths, groups):
    """Two workgroups of 16 rows per compute unit: prompts of like length take two row groups, prompts with one long
    one among them one (its chain is the call).  The choice, kept in the workspace's header, and the results."""
    n, H = len(lengths), 1024 // dv
    assert 2 * _cus() <= n * H * dv // 16 < 3 * _cus()
    ws = torch.zeros(gdn.gdn_chunk_prefill_workspace_bytes(1, sum(lengths), H, dk, dv, 64, n, gdn.GDN_BF16), dtype=torch.uint8,
                     device="cuda")
    _run(dict(B=1, T=0, H=H, H_k=H // 2, dk=dk, dv=dv, seed=720 + dk + dv, lengths=lengths, raw=raw), snap, ws)
    assert ws[64:68].view(torch.int32).item() == groups


@pytest.mark.parametrize("dk,dv,raw,snap", [(128, 128, True, 0), (64, 64, False, 0), (128, 64, False, 2), (64, 128, True, 1)])
def test_packed_two_row_groups(dk, dv, raw, snap):
    """Three workgroups of 16 rows per compute unit and more: two row groups whatever the lengths."""
    H = 2048 // dv
    assert 7 * H * dv // 16 >= 3 * _cus()
    _run(dict(B=1, T=0, H=H, H_k=H // 2, dk=dk, dv=dv, seed=740 + dk + dv, lengths=[1, 0, 65, 193, 384, 130, 64], raw=raw), snap)


@pytest.mark.parametrize("d,raw", [(64, False), (128, False), (64, True), (128, True)])
def test_chunk_terms_block_edges(d, raw):
    """One sequence per chunk length around the 16-token blocks: the one-launch form."""
    _run(dict(B=1, T=0, H=2, dk=d, dv=d, seed=800 + d, raw=raw, lengths=[1, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64]))
