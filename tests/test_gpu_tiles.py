"""Window forward at the edges of the activation tiles (32 rows x 64 columns)
and of the kernels that write them: widths that end inside a 256-column norm
chunk, one column tile, windows whose rows end inside an 8-row group or a 32-row
tile, narrow and wide row groups, against the oracle's forward.

Tolerance: activations carry 16 significant bits (relative rounding 2^-17) at
about eight points per layer, and the logits are sums of such values; 2^-11 of
the largest logit is 64 times one rounding, while a misplaced or missing tile
entry moves logits by their own size."""
import numpy as np
import pytest
import torch

from model_util import make_engine, oracle_first_window, setup, weights_device, weights_numpy
from synth_inputs import model_config

pytestmark = pytest.mark.gpu

SHAPES = [
    dict(d_model=64, n_heads=1, n_kv_heads=1, ffn_dim=64, L=1, K=1, D=0, n_prompt=2),
    dict(d_model=320, n_heads=5, n_kv_heads=1, ffn_dim=192, L=9, K=2, D=2, n_prompt=50),
    dict(d_model=576, n_heads=9, n_kv_heads=3, ffn_dim=1088, L=33, K=4, D=3, n_prompt=97),
    dict(d_model=1088, n_heads=4, n_kv_heads=2, head_dim=128, ffn_dim=2816, L=31, K=4, D=3, n_prompt=130),
    dict(d_model=2112, n_heads=16, n_kv_heads=4, head_dim=128, ffn_dim=4160, L=64, K=4, D=3, n_prompt=75),
]


@pytest.mark.parametrize("over", SHAPES, ids=[f"d{s['d_model']}-L{s['L']}" for s in SHAPES])
def test_window_forward_at_tile_edges(orc, over):
    cfg = model_config("tiny", weights_f32=False, **over)
    w, prompt = setup(cfg, wseed=21, pseed=22, device="cuda")
    print(f"case {over}", flush=True)
    eng = make_engine(cfg, weights_device(w))
    eng.prefill(prompt.cuda(), 7)
    logits = torch.empty(cfg["L"], cfg["V"], dtype=torch.float32, device="cuda")
    eng.forward_window(logits)
    torch.cuda.synchronize()
    got = logits.cpu().numpy()
    eng.close()
    ref = oracle_first_window(orc, cfg, weights_numpy(w), prompt.numpy().astype(np.int32), 7)
    err = np.abs(got - ref).max()
    print(f"max |logit error| = {err:.3e}, max |logit| = {np.abs(ref).max():.3f}", flush=True)
    assert np.isfinite(got).all()
    assert err <= np.abs(ref).max() * 2.0 ** -11, err
