"""The forward at 1, 2 and 4 pixels per lane and on either side of the line
between its two forms of the update (selects on frames of few wavefronts, lane
masks on others).  Small frames take one pixel per lane by themselves, so the width
is set here; large ones take the others."""
import numpy as np
import pytest
import torch

import oracle
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

from paper_1702_05156_amd import dsgm

MODES = [(torch.float64, dsgm.ACC_F64), (torch.float32, dsgm.ACC_F64_IO32), (torch.bfloat16, dsgm.ACC_F64),
         (torch.float32, dsgm.ACC_F32), (torch.bfloat16, dsgm.ACC_F32)]
PLANES = ("mean_a", "var_a", "mean_c", "var_c", "age_a", "age_c")


@pytest.fixture
def width():
    yield lambda v: dsgm.dsgm_set_launch(0, v)
    dsgm.dsgm_set_launch(0, 0)


def _same(a, b, T, H, W, K=0, size=0):
    for k in a[0]:
        if k == "ckpt":
            assert torch.equal(G.ckpt_payload(a[0][k], T, H, W, K, size),
                               G.ckpt_payload(b[0][k], T, H, W, K, size))
        else:
            assert torch.equal(a[0][k], b[0][k]), k
    for x, y in zip(a[1].planes(), b[1].planes()):
        assert torch.equal(x, y)


@pytest.mark.parametrize("printed", [False, True])
@pytest.mark.parametrize("T", [1, 4, 11])
@pytest.mark.parametrize("in_dtype,acc", MODES)
def test_every_width_gives_the_same(in_dtype, acc, T, printed, width):
    """One-frame calls, exactly one batch of frames, and batches with a
    remainder; with and without bg and checkpoints.  FP64 state equals the oracle."""
    H, W, K, seed = 9, 40, 4, 61
    sd = dsgm.STATE_TORCH[acc]
    p = dsgm.dsgm_params_default(2.0, dsgm.MASK_PRINTED if printed else dsgm.MASK_VARIANCE)
    fr, st0 = G.device_case(seed, T, H, W, in_dtype, sd)
    for kw in (dict(), dict(bg=True), dict(bg=True, ckpt_every=K)):
        runs = []
        for v in (1, 2, 4):
            width(v)
            st = st0.clone()
            runs.append((dsgm.forward(fr, st, p, acc=acc, **kw), st))
        for r in runs[1:]:
            _same(r, runs[0], T, H, W, K, sd.itemsize)
    if acc != dsgm.ACC_F32:
        x, host = G.host_case(seed, T, H, W, in_dtype, sd)
        ref = oracle.forward(x, host, G.oracle_params(p))
        out, st = runs[2]
        G.assert_bit_exact("masks", G.flat(out["masks"]).astype(np.uint8), ref["masks"])
        G.assert_bit_exact("bg", out["bg"].cpu().numpy().reshape(T, -1),
                           ref["bg"].astype(np.float64 if acc == dsgm.ACC_F64 else np.float32))
        hs = G.state_to_host(st)
        for k in PLANES:
            G.assert_bit_exact(k, hs[k], ref[k])


@pytest.mark.parametrize("mr", [0, 1])
@pytest.mark.parametrize("T", [1, 3, 8, 21])
def test_u8_every_width_equals_the_oracle(T, mr, width):
    """The 8-bit model: one-frame calls and whole sequences (batches of eight frames
    and remainders), with and without decision codes."""
    H, W = 7, 52
    rng = np.random.default_rng(62)
    x = rng.integers(0, 256, (T, H, W)).astype(np.uint8)
    host = {k: rng.integers(0, 256, H * W).astype(np.uint8) for k in PLANES[:4]}
    host.update({k: rng.integers(1, 31, H * W).astype(np.uint8) for k in PLANES[4:]})
    p = dsgm.dsgm_params_default(255.0, mr)
    p.weight_rule = mr
    ref = oracle.forward_u8(x.reshape(T, -1), host, G.oracle_params(p))
    for v in (1, 2, 4):
        for codes in (False, True):
            width(v)
            st = dsgm.State(*(torch.as_tensor(host[k].reshape(H, W), device="cuda") for k in PLANES))
            out = dsgm.forward(torch.as_tensor(x, device="cuda"), st, p, codes=codes)
            G.assert_bit_exact("masks", G.flat(out["masks"]).astype(np.uint8), ref["masks"])
            if codes:
                G.assert_bit_exact("codes", G.flat(out["codes"]).astype(np.uint8), ref["codes"])
            for k in PLANES:
                G.assert_bit_exact(k, getattr(st, k).cpu().numpy().ravel(), ref[k].astype(np.uint8))


@pytest.mark.parametrize("H", [255, 257, 509, 513])
@pytest.mark.parametrize("in_dtype,acc", MODES)
def test_either_form_of_the_update(in_dtype, acc, H):
    """Frames of 257 columns just below and above 1,024 and 2,048 wavefronts, the
    lines of FP64 and FP32 state: the pixels of their first and last rows get what
    they get in a frame of those rows alone."""
    W, T, K, n = 257, 9, 4, 3
    sd = dsgm.STATE_TORCH[acc]
    p = dsgm.dsgm_params_default(2.0)
    fr, st = G.device_case(63, T, H, W, in_dtype, sd)
    for kw in (dict(codes=True, bg=True), dict(bg=True, ckpt_every=K), dict()):
        whole = st.clone()
        out = dsgm.forward(fr, whole, p, acc=acc, **kw)
        for rows in (slice(0, n), slice(H - n, H)):
            s = dsgm.State(*(t.reshape(H, W)[rows].clone() for t in st.planes()))
            o = dsgm.forward(fr[:, rows].contiguous(), s, p, acc=acc, **kw)
            for k in o:
                if k != "ckpt":
                    assert torch.equal(o[k], out[k][:, rows]), k
            for a, b in zip(s.planes(), whole.planes()):
                assert torch.equal(a, b.reshape(H, W)[rows])
            if "ckpt" in o:  # mean A before every K-th frame
                size = sd.itemsize
                pl = lambda c, px: c.view(-1, c.numel() // -(-T // K))[:, :px * size].contiguous().view(sd)
                assert torch.equal(pl(o["ckpt"], n * W),
                                   pl(out["ckpt"], H * W).reshape(-1, H, W)[:, rows].reshape(-1, n * W))


@pytest.mark.parametrize("printed", [False, True])
@pytest.mark.parametrize("H", [1023, 1024])
@pytest.mark.parametrize("in_dtype,acc", MODES + [(torch.bfloat16, dsgm.ACC_F64_IO32)])
def test_one_large_frame_at_every_width(in_dtype, acc, H, printed, width):
    """One frame just below and at 3 x 2^19 pixels, from which its request follows
    the table: every width gives what one pixel per lane gives, whose request never
    does."""
    W = 1536
    p = dsgm.dsgm_params_default(2.0, dsgm.MASK_PRINTED if printed else dsgm.MASK_VARIANCE)
    fr, st0 = G.device_case(64, 1, H, W, in_dtype, dsgm.STATE_TORCH[acc])
    for bg in (False, True):
        runs = []
        for v in (1, 2, 4):
            width(v)
            st = st0.clone()
            runs.append((dsgm.forward(fr, st, p, bg=bg, acc=acc), st))
        for r in runs[1:]:
            _same(r, runs[0], 1, H, W)
