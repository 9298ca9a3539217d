"""GPU parity of the fp32 sequential prefill at the chunk counts where its chain can go wrong, against the fp64 oracle.

The chain keeps two chunks resident by parity and forms the outputs one chunk behind: one chunk and no chunk,
even and odd counts, partial last chunks, every pair of widths, packed prompts, the input transforms and
snapshots.  Bar as the other prefill tests (max|x - ref| / max|ref| <= 2e-4 for fp32 io).
"""
import pytest
import torch

import oracle
import paper_2607_14568_amd as gdn
import parity
from paper_2607_14568_amd import inputs

pytestmark = pytest.mark.gpu
f64 = inputs.as_f64


@pytest.mark.parametrize("dk,dv", [(64, 64), (128, 64), (64, 128), (128, 128)])
@pytest.mark.parametrize("lengths,raw,snap", [([1, 0, 64, 65], False, 0), ([128, 129, 17, 192], True, 0), ([200], False, 1),
                                              ([321], True, 2)])
def test_chain_chunk_counts(dk, dv, lengths, raw, snap):
    print("case:", dk, dv, lengths, raw, snap, flush=True)
    x = inputs.make_prefill(B=1, T=0, H=4, H_k=2, dk=dk, dv=dv, io="f32", seed=900 + dk + dv + len(lengths), s0_std=0.05,
                            lengths=lengths, raw=raw)
    d = {k: (v.cuda() if isinstance(v, torch.Tensor) else v) for k, v in x.items()}
    args = (d["q"], d["k"], d["v"], d["g"], d["beta"], d["S0"])
    kw = dict(flags=gdn.GDN_QK_L2NORM | gdn.GDN_GATE_LOGITS if raw else 0, cu_seqlens=d["cu_seqlens"])
    if snap:
        o, S_T, snaps = gdn.gdn_chunk_prefill_snapshots_ex(*args, snap_every=snap, **kw)
    else:
        o, S_T = gdn.gdn_chunk_prefill_ex(*args, **kw)
    torch.cuda.synchronize()
    tokens = [f64(x[n]) for n in ("q", "k", "v", "g", "beta")]
    tf = dict(qk_l2norm=raw, gate_logits=raw)
    cu = x["cu_seqlens"].numpy()
    ref = oracle.recurrence_ex(*tokens, f64(x["S0"]), cu_seqlens=cu, **tf)
    parity.check(f64(o), ref[0], f64(S_T), ref[1], 2e-4, "%d %d %s" % (dk, dv, lengths), cu_seqlens=cu)
    for j in range(snaps.shape[1] if snap else 0):   # the state after (j + 1) * snap chunks of the only sequence
        n = (j + 1) * snap * 64
        cut = oracle.recurrence_ex(*(t[:, :n] for t in tokens), f64(x["S0"]), **tf)
        assert oracle.max_rel_err(f64(snaps[:, j]), cut[1]) < 2e-4
