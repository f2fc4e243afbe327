"""A GEMM workgroup whose K range is not a whole number of load rings pads it;
what a padded step multiplies must be finite whatever the activation buffers
hold. A row that is not finite (here: a token whose embedding is NaN) therefore
stays its own stream's affair: another image of the batch, and a later request of
the same context, get the bits that they get without it. The shape (d = 1088, 17
k-steps) is not narrow, and its plans leave padded steps in every projection."""
import pytest
import torch

from model_util import make_engine, setup, weights_device
from synth_inputs import model_config

pytestmark = pytest.mark.gpu

BAD = 7  # the token with a NaN embedding; used only where a test places it


def _model(**over):
    cfg = model_config("tiny", weights_f32=False, d_model=1088, n_heads=4, n_kv_heads=2, head_dim=128, ffn_dim=1600,
                       L=32, K=1, D=0, n_prompt=40, **over)
    w, prompt = setup(cfg, wseed=51, pseed=52, device="cuda")
    w["embed"][BAD] = float("nan")
    prompt[prompt == BAD] = BAD + 1
    return cfg, weights_device(w), prompt.cuda()


def _drafts(cfg, bad_at=None):
    g = torch.Generator().manual_seed(53)
    t = torch.randint(BAD + 1, cfg["V"], (cfg["L"],), generator=g, dtype=torch.int32)
    if bad_at is not None:
        t[bad_at] = BAD
    return t.cuda()


@pytest.mark.parametrize("images", [2, 4])
def test_a_nonfinite_row_of_one_image_leaves_the_others_alone(images):
    cfg, dev, prompt = _model(batch=images)
    L, got = cfg["L"], []
    for bad_at in (None, 5):  # draft 5 is fed at row 6 of image 0
        print(f"images {images}, bad row {bad_at}", flush=True)
        eng = make_engine(cfg, dev)
        for b in range(images):
            eng.prefill_image(b, prompt[:len(prompt) - 3 * b].contiguous(), 3)
            eng.set_drafts(_drafts(cfg, bad_at if b == 0 else None), image=b)
        logits = torch.zeros(32 * (images - 1) + L, cfg["V"], device="cuda")
        eng.forward_window(logits)
        torch.cuda.synchronize()
        got.append(logits.cpu())
        eng.close()
    assert torch.isfinite(got[0]).all() and torch.isnan(got[1][6]).any()  # (its own stream may see it anywhere)
    assert torch.equal(got[1][32:], got[0][32:])


@pytest.mark.parametrize("n_late", [2, 8, 20])
def test_a_nonfinite_row_does_not_reach_a_later_request(n_late):
    """The later prompt's windows have fewer rows than the window that held the
    row, and its positions lie below those that request cached."""
    cfg, dev, prompt = _model(max_seq=300)
    late = prompt[:n_late].contiguous()
    long = prompt.repeat(5)
    got = []
    for bad_at in (None, 24):  # fed at row 25, position 199 + 25
        print(f"later prompt of {n_late}, bad row {bad_at}", flush=True)
        eng = make_engine(cfg, dev)
        logits = torch.zeros(cfg["L"], cfg["V"], device="cuda")
        eng.prefill(long, 3)
        eng.set_drafts(_drafts(cfg, bad_at))
        eng.forward_window(logits)
        assert bad_at is None or torch.isnan(logits[25]).any()
        eng.prefill(late, 3)
        eng.set_drafts(_drafts(cfg))
        eng.forward_window(logits)
        torch.cuda.synchronize()
        got.append(logits.cpu())
        eng.close()
    assert torch.isfinite(got[0]).all()
    assert torch.equal(got[1], got[0])
