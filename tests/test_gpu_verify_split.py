"""Launches whose draft rows are selected by a kernel of their own (more rows
than the two-row workgroups take, or more than 32768 logits): against the
oracle, and against the whole-row selection, at the edges of the launch shapes
(one chunk past a power of two, a row that ends inside a register slot), with
rows that the draft kernel must leave to the row kernel (-inf entries, values on
a coarse grid whose ties straddle the threshold, one value only), trees,
placeholders, a temperature and vanilla SJD. Decisions are compared as
everywhere: bit-exact but for near-ties within 1e-6."""
import numpy as np
import pytest
import torch

from oracle.parity import compare_verify
from synth_inputs import verify_inputs
from test_gpu_verify import run_both

pytestmark = pytest.mark.gpu

CASES = [
    # V, B, L, top_k, T, flags (1: adaptive continuation, 2: drafting)
    (256, 20, 32, 37, 1.0, 3),
    (4096, 40, 16, 700, 0.8, 3),
    (4100, 45, 30, 300, 1.0, 3),
    (8620, 41, 32, 2000, 1.0, 0),
    (16384, 41, 32, 2000, 1.0, 1),
    (16388, 18, 32, 2048, 1.3, 2),
    (32768, 9, 64, 1, 1.0, 3),
    (32772, 1, 20, 500, 1.0, 3),
    (65536, 2, 33, 2000, 1.0, 3),
]


@pytest.mark.parametrize("V,B,L,top_k,T,flags", CASES, ids=[f"V{c[0]}-rows{c[1] * c[2]}" for c in CASES])
def test_split_launches_match_oracle(orc, V, B, L, top_k, T, flags):
    K, D, D_in = 3, 2, 2
    inp = verify_inputs(B, L, V, top_k=top_k, seed=V + L, K=K, D=D, D_in=D_in, temperature=T)
    g = torch.Generator().manual_seed(V)
    n_s = L - (K - 1) * D_in
    inp["meta"][:, 1] = torch.randint(0, n_s + 1, (B,), generator=g)
    # draft rows that the candidates cannot decide, at windows' first rows
    inp["draft"][0, 0, 5::7] = -float("inf")
    if L > 3:
        inp["draft"][0, 2] = torch.round(inp["draft"][0, 2] * 2) / 2
        inp["draft"][B - 1, 3] = 1.25
        inp["cur"][B - 1, 1, 3::5] = -float("inf")
    inp["meta"][0, 1] = inp["meta"][B - 1, 1] = n_s
    trials = sorted({0, B // 2, B - 1})
    got, ref = run_both(orc, inp, K=K, D=D, top_k=top_k, T=T, flags=flags, want_p=False, oracle_trials=trials)
    compare_verify(got, ref, K=K, D=D, label=f"split V={V}")
    # every trial against the whole-row selection (its normalisers add in
    # another order: the same decisions but for fp64 near-ties)
    import paper_2603_18599_amd as sjd
    from paper_2603_18599_amd.sjd import SJD_FULL_SELECT, verify_outputs
    dev = {k: v.cuda() for k, v in inp.items()}
    res = []
    for extra in (0, SJD_FULL_SELECT):
        out = verify_outputs(B, L, K, D)
        rows = torch.zeros(B, L, 2, dtype=torch.int32, device="cuda")
        sjd.sjd_verify(dev["cur"], dev["draft"], dev["draft_tok"], dev["meta"], out, K=K, D=D, top_k=top_k,
                       temperature=T, flags=flags | extra, seed=1, step=0, sib=dev["sib"], out_rows=rows)
        torch.cuda.synchronize()
        res.append(dict({k: v.cpu() for k, v in out.items()}, rows=rows.cpu()))
    differ = {k: int((res[0][k] != res[1][k]).sum()) for k in res[0]}
    assert not any(differ.values()), differ
