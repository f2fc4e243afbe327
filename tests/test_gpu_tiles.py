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


# Narrow models run each projection with its consumer as one kernel, wider ones
# (and SJD_TUNE contexts, whose timed candidates are the split kernels) as two;
# short caches of 64-dim heads take the one-kernel attention. Under one plan the
# results have the same bits. Shapes: more splits than k-steps, uneven splits, a
# projection too long for one kernel, 128-dim heads, grouped heads, one to four
# streams, prompts of one and of several prefill windows, window rows past a
# 32-row tile, caches of more chunks than the one-kernel attention takes.
NARROW = [
    (dict(d_model=64, n_heads=1, n_kv_heads=1, ffn_dim=64, L=1, K=1, D=0, n_prompt=3), "2,5,3,1"),
    (dict(d_model=320, n_heads=5, n_kv_heads=1, ffn_dim=1600, L=9, K=2, D=2, n_prompt=33), "4,1,5,22"),
    (dict(d_model=576, n_heads=6, n_kv_heads=2, head_dim=128, ffn_dim=1536, L=33, K=4, D=3, n_prompt=97), "8,7,3,9"),
    (dict(d_model=960, n_heads=15, n_kv_heads=15, ffn_dim=2816, L=32, K=4, D=3, n_prompt=64, batch=4), "8,8,5,22"),
    (dict(d_model=512, n_heads=8, n_kv_heads=4, ffn_dim=1024, L=20, K=4, D=3, n_prompt=200, cfg_w=3.0), "3,32,17,31"),
    (dict(d_model=256, n_heads=4, n_kv_heads=4, ffn_dim=1024, L=64, K=4, D=3, n_prompt=470, max_seq=1000), "2,2,2,4"),
    (dict(d_model=448, n_heads=7, n_kv_heads=7, ffn_dim=2560, L=25, K=4, D=3, n_prompt=135), "3,5,2,31"),
    (dict(d_model=384, n_heads=41, n_kv_heads=1, ffn_dim=2624, L=26, K=4, D=3, n_prompt=135), "3,9,2,13"),
]


@pytest.mark.parametrize("over,plan", NARROW, ids=[f"d{o['d_model']}-L{o['L']}" for o, _ in NARROW])
def test_narrow_models_match_the_split_kernels_bitwise(monkeypatch, over, plan):
    from paper_2603_18599_amd.sjd import SJD_AC, SJD_PD, SJD_TUNE
    monkeypatch.setenv("SJD_SPLITS", plan)
    # (shapes without a recorded plan: windows of more than 32 rows take the closed
    # form on both sides)
    base = model_config("tiny", weights_f32=False, vocab_size=1056, V=1056, **over)
    w, prompt = setup(base, wseed=31, pseed=32, device="cuda")
    dev = weights_device(w)
    B, L = base.get("batch", 1), base["L"]
    got = []
    for flags in (SJD_AC | SJD_PD, SJD_AC | SJD_PD | SJD_TUNE):
        print(f"case {over} flags {flags}", flush=True)
        eng = make_engine(dict(base, flags=flags), dev)
        for b in range(B):
            p = prompt[:len(prompt) - b].cuda()
            if base.get("cfg_w"):
                eng.prefill_cfg(p, p[7:].contiguous(), 5, image=b)
            else:
                eng.prefill_image(b, p, 5 + b)
        logits = torch.zeros(32 * (B - 1) + L, base["V"], device="cuda")
        metas = torch.zeros(2, B, 8, dtype=torch.int32, device="cuda")
        for t in range(2):
            eng.step(1.0, 200, 5, t, out_meta=metas[t])
        eng.forward_window(logits)
        torch.cuda.synchronize()
        got.append((logits.cpu(), metas.cpu()))
        eng.close()
    assert torch.equal(got[0][1], got[1][1])
    for b in range(B):
        assert torch.equal(got[0][0][32 * b:32 * b + L], got[1][0][32 * b:32 * b + L])


@pytest.mark.parametrize("n_prompt,batch", [(215, 1), (215, 2), (250, 1)])
def test_attention_launch_shape_follows_the_fill_bitwise(monkeypatch, n_prompt, batch):
    """Narrow contexts of at most 512 positions attend in one kernel while the
    fill is short and in two beyond: a generation that crosses the line, in
    prefill or between steps (each step synchronised, so that the host knows the
    fill; a second image far behind the first), against the split kernels."""
    from paper_2603_18599_amd.sjd import SJD_AC, SJD_PD, SJD_TUNE
    monkeypatch.setenv("SJD_SPLITS", "4,4,4,4")
    base = model_config("tiny", weights_f32=False, d_model=512, n_heads=8, n_kv_heads=4, ffn_dim=1024, vocab_size=1056,
                        V=1056, L=32, K=4, D=3, n_prompt=n_prompt, batch=batch, max_seq=512)
    w, prompt = setup(base, wseed=61, pseed=62, device="cuda")
    dev = weights_device(w)
    got = []
    for flags in (SJD_AC | SJD_PD, SJD_AC | SJD_PD | SJD_TUNE):
        print(f"prompt {n_prompt} batch {batch} flags {flags}", flush=True)
        eng = make_engine(dict(base, flags=flags), dev)
        for again in range(2):  # the second generation starts below the line again
            for b in range(batch):
                eng.prefill_image(b, prompt[:n_prompt - 100 * b].cuda(), 5 + b)
            logits = torch.zeros(32 * batch, base["V"], device="cuda")
            meta = torch.zeros(batch, 8, dtype=torch.int32, device="cuda")
            for t in range(24):
                eng.step(1.0, 8, 5, t, out_meta=meta)
                torch.cuda.synchronize()
                got.append(meta.cpu())
            eng.forward_window(logits)
            got.append(logits.cpu())
            assert int(meta[0, 7]) + 32 > 256  # (cached rows plus the window)
        eng.close()
    half = len(got) // 2
    assert all(torch.equal(a, b) for a, b in zip(got[:half], got[half:]))


def test_gemm_widths_agree_bitwise(monkeypatch):
    """The column blocks a GEMM workgroup takes do not change a result: a plan
    that runs six wide (8 blocks at 16 splits of 96 blocks: 192 workgroups eight
    wide, 256 six wide) against four
    wide."""
    cfg = model_config("tiny", weights_f32=False, d_model=1088, n_heads=4, n_kv_heads=2, head_dim=128, ffn_dim=1536,
                       L=23, K=4, D=3, n_prompt=20)
    w, prompt = setup(cfg, wseed=41, pseed=42, device="cuda")
    dev = weights_device(w)
    got = []
    for plan in ("4,4,16:8,4", "4,4,16,4"):
        print(f"case {plan}", flush=True)
        monkeypatch.setenv("SJD_SPLITS", plan)
        eng = make_engine(cfg, dev)
        eng.prefill(prompt.cuda(), 3)
        logits = torch.zeros(cfg["L"], cfg["V"], device="cuda")
        eng.forward_window(logits)
        torch.cuda.synchronize()
        got.append(logits.cpu())
        eng.close()
    assert torch.equal(got[0], got[1])


@pytest.mark.parametrize("plan", ["3:8,2:8,1:8,3:8", "9:8,32:8,16:8,32:8", "1:8,1,3:8,1:8", "7,3:8,5,11:8"])
def test_wide_groups_with_idle_waves_on_wide_models(orc, monkeypatch, plan):
    """As test_window_forward_wide_groups_with_idle_waves, on a model that is not
    narrow, so that every projection is a GEMM of its own: QKV 180 blocks, O and down
    34, gate|up 100, none a multiple of 8 (O, down and gate|up not of 6 either).
    Grids of more than 192 workgroups run eight wide (QKV at 9 splits, gate|up at 16),
    the smaller ones six; 17 k-steps, fewer than some splits."""
    cfg = model_config("tiny", weights_f32=False, n_layers=2, d_model=1088, n_heads=39, n_kv_heads=3, head_dim=128,
                       ffn_dim=1600, L=32, K=4, D=3, n_prompt=9)
    w, prompt = setup(cfg, wseed=71, pseed=72, device="cuda")
    dev = weights_device(w)
    got = []
    for pin in (plan, plan.replace(":8", "")):
        print(f"case {pin}", flush=True)
        monkeypatch.setenv("SJD_SPLITS", pin)
        eng = make_engine(cfg, dev)
        eng.prefill(prompt.cuda(), 7)
        logits = torch.empty(cfg["L"], cfg["V"], dtype=torch.float32, device="cuda")
        eng.forward_window(logits)
        torch.cuda.synchronize()
        got.append(logits.cpu())
        eng.close()
    assert torch.equal(got[0], got[1])  # the width does not change a result
    ref = oracle_first_window(orc, cfg, weights_numpy(w), prompt.numpy().astype(np.int32), 7)
    err = np.abs(got[0].numpy() - ref).max()
    print(f"max |logit error| = {err:.3e}, max |logit| = {np.abs(ref).max():.3f}", flush=True)
    assert err <= np.abs(ref).max() * 2.0 ** -11, err


@pytest.mark.parametrize("L,batch", [(1, 1), (32, 1), (33, 1), (20, 3), (32, 4)])
def test_narrow_models_with_a_wide_head_match_the_split_kernels_bitwise(monkeypatch, L, batch):
    """The LM head of a narrow model with many columns: eight blocks per workgroup,
    its row scale from the sums of squares of fours of columns; 1539 blocks, so that
    the last workgroup has idle waves; one to four row tiles. Against the split
    kernels (the LM head's row scale from chunk sums) under the same plan."""
    from paper_2603_18599_amd.sjd import SJD_AC, SJD_PD, SJD_TUNE
    monkeypatch.setenv("SJD_SPLITS", "3,2,4,5")
    base = model_config("tiny", weights_f32=False, n_layers=1, d_model=320, n_heads=5, n_kv_heads=5, ffn_dim=640,
                        vocab_size=49248, V=49248, L=L, K=1, D=0, n_prompt=40, batch=batch)
    w, prompt = setup(base, wseed=81, pseed=82, device="cuda")
    dev = weights_device(w)
    got = []
    for flags in (SJD_AC | SJD_PD, SJD_AC | SJD_PD | SJD_TUNE):
        print(f"L {L} batch {batch} flags {flags}", flush=True)
        eng = make_engine(dict(base, flags=flags), dev)
        assert eng.plan()[9] == 8
        for b in range(batch):
            eng.prefill_image(b, prompt[:len(prompt) - b].cuda(), 5 + b)
        logits = torch.zeros(32 * (batch - 1) + L, base["V"], device="cuda")
        eng.forward_window(logits)
        torch.cuda.synchronize()
        got.append(logits.cpu())
        eng.close()
    for b in range(batch):
        assert torch.isfinite(got[0][32 * b:32 * b + L]).all()
        assert torch.equal(got[0][32 * b:32 * b + L], got[1][32 * b:32 * b + L])
