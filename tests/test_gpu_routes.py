"""Inference over few and over many records takes different kernels; a record's
prediction must not depend on which.

Every accumulator sees the same products in the same order in all of them, so
the predictions of a batch and of its slices (of a few records, down to one) are
equal bit for bit: no tolerance.  (The slices are copied out: device buffers are
16-byte aligned.)
"""
import numpy as np
import pytest
import torch

import synthdata as sd

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def N():
    from paper_2106_12372_amd import nrc
    return nrc


# Records per 64-record tile and compute unit at which the kernels change.
def _lines(cus):
    return {("fp16", 64): 4 * 64 * cus, ("bf16", 64): 4 * 64 * cus, ("fp16", 128): 6 * 64 * cus,
            ("bf16", 128): 6 * 64 * cus, ("fp32", 64): 24 * 64 * cus}


SLICES = ((0, 1), (0, 63), (64, 1001), (5, 22))


@pytest.mark.parametrize("prec,width,n_hidden", [("fp16", 64, 5), ("bf16", 64, 5), ("fp16", 64, 1), ("bf16", 64, 8),
                                                 ("fp16", 128, 5), ("bf16", 128, 1), ("bf16", 128, 4),
                                                 ("fp32", 64, 5), ("fp32", 64, 1), ("fp32", 64, 6)])
@pytest.mark.parametrize("raw_form", [False, True])
@pytest.mark.parametrize("past", [0, 1, 64 * 300 + 37])
def test_batches_and_their_slices_agree(N, prec, width, n_hidden, raw_form, past):
    if raw_form and width == 128:
        pytest.skip("raw records feed the 64-wide network only")
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    n = _lines(cus)[(prec, width)] + past
    cfg = N.make_config(width=width, n_hidden=n_hidden, precision=prec, factorize=n_hidden % 2 == 1)
    c = N.Cache(cfg)
    c.set_weights(sd.glorot_weights(width, n_hidden, seed=3))
    raw = torch.from_numpy(sd.raw_records(n, 40 + n_hidden)).cuda()
    enc = N.nrc_encode(c, raw)
    whole = N.nrc_forward_raw(c, raw) if raw_form else N.nrc_forward(c, enc)
    assert bool(torch.isfinite(whole).all())
    for lo, hi in SLICES + ((n - 1000, n), (n - 1, n)):
        part = enc[lo:hi].clone()
        assert torch.equal(N.nrc_forward(c, part), whole[lo:hi]), (lo, hi)
        if width == 64:
            assert torch.equal(N.nrc_forward_raw(c, raw[lo:hi].clone()), whole[lo:hi]), (lo, hi)


@pytest.mark.parametrize("prec,width,n_hidden,ema", [("fp16", 64, 5, 0.0), ("bf16", 64, 8, 0.99), ("fp16", 128, 3, 0.9),
                                                     ("bf16", 128, 5, 0.0), ("fp32", 64, 2, 0.5),
                                                     ("fp32_valu", 64, 1, 0.0)])
def test_weights_from_the_device_equal_weights_from_the_host(N, prec, width, n_hidden, ema):
    """One launch sets what the host path sets with copies and fills: every byte of the
    workspace (weights, moments, step count, EMA set, fragment copies) is the same."""
    cfg = N.make_config(width=width, n_hidden=n_hidden, precision=prec, ema_alpha=ema)
    w = sd.glorot_weights(width, n_hidden, seed=5)
    caches = [N.Cache(cfg), N.Cache(cfg)]
    raw = sd.raw_records(130, 8)
    for c in caches:                                   # leave something in every field
        c.set_weights(sd.glorot_weights(width, n_hidden, seed=9))
        enc = N.nrc_encode(c, torch.from_numpy(raw).cuda())
        for _ in range(3):
            N.nrc_train_step(c, enc, torch.from_numpy(sd.targets(raw)).cuda())
    caches[0].set_weights(w)
    caches[1].set_weights_device(torch.from_numpy(w).cuda())
    torch.cuda.synchronize()
    assert torch.equal(caches[0].ws, caches[1].ws)


def test_calls_go_to_the_current_stream(N):
    """The handle the binding passes on is the current stream's, by whatever way it became
    current, and an explicit stream's own."""
    side = torch.cuda.Stream()
    external = torch.cuda.ExternalStream(torch.cuda.Stream().cuda_stream)
    for s in (torch.cuda.default_stream(), side, external):
        with torch.cuda.stream(s):
            assert N._stream(None) == torch.cuda.current_stream().cuda_stream == s.cuda_stream
    assert N._stream(None) == torch.cuda.current_stream().cuda_stream
    assert N._stream(side) == N._stream(side.cuda_stream) == side.cuda_stream


def test_device_weights_of_any_stride(N):
    """A strided vector is refused; a matrix of strided rows reaches the cache as its storage lies."""
    c = N.Cache(N.make_config())
    w = torch.rand(c.n_params, device="cuda")
    with pytest.raises(ValueError, match="contiguous"):
        c.set_weights_device(torch.rand(2 * c.n_params, device="cuda")[::2])
    with pytest.raises(ValueError, match="float32"):
        c.set_weights_device(w.double())
    with pytest.raises(ValueError, match="device tensor"):
        c.set_weights_device(w.cpu())
    c.set_weights_device(w.view(-1, 64).t())
    assert np.array_equal(c.get_weights(), w.cpu().numpy())


@pytest.mark.parametrize("n_hidden,past", [(5, 1), (5, 64 * 40 + 17), (6, 33), (1, 64), (2, 64 * 300 - 1)])
def test_fp32_forward_with_activations_over_many_tiles(N, n_hidden, past):
    """More tiles than compute units take another kernel: same predictions as in slices, and a
    buffer that gives the gradients of a recomputed forward pass, equal bit for bit."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    n = 64 * cus + past
    c = N.Cache(N.make_config(n_hidden=n_hidden, precision="fp32", factorize=n_hidden == 5))
    c.set_weights(sd.glorot_weights(64, n_hidden, seed=4))
    enc = torch.from_numpy(sd.uniform_features(n, 64, 21)).cuda()
    up = torch.rand(n, 3, device="cuda", generator=torch.Generator("cuda").manual_seed(2)) - 0.5
    act = torch.full((N.nrc_act_ws_bytes(c.cfg, n),), 0xff, dtype=torch.uint8, device="cuda")   # NaN where nothing is written
    rgb, act = N.nrc_forward_train(c, enc, act=act)
    assert torch.equal(rgb, N.nrc_forward(c, enc))
    for lo in range(0, n, 64 * cus):
        assert torch.equal(N.nrc_forward_train(c, enc[lo:lo + 64 * cus].clone())[0], rgb[lo:lo + 64 * cus])
    for got, ref in zip(N.nrc_backward(c, enc, up, act=act), N.nrc_backward(c, enc, up)):
        assert torch.equal(got, ref)


@pytest.mark.parametrize("prec", ["fp16", "bf16", "fp32"])
@pytest.mark.parametrize("preset,layout", [(0, 0), (1, 1), (2, 0), (3, 1), (0, 1), (3, 0)])
def test_a_row_is_encoded_alike_in_any_batch(N, prec, preset, layout):
    """Rows of ragged batches equal the same vertices' rows in one large batch bit for bit, and
    nothing is written past a batch's last row."""
    c = N.Cache(N.make_config(precision=prec, enc_preset=preset))
    raw = torch.from_numpy(sd.raw_records(64 * 700 + 5, 31, layout)).cuda()
    whole = N.nrc_encode(c, raw, layout)
    for lo, n in ((0, 1), (64, 63), (128, 64), (1000, 65), (63, 321), (64 * 650, 64 * 50 + 5)):
        out = torch.full((n + 2, 64), 7.0, dtype=c.enc_dtype, device="cuda")
        N.nrc_encode(c, raw[lo:lo + n].clone(), layout, enc=out[:n])
        assert torch.equal(out[:n], whole[lo:lo + n]) and bool((out[n:] == 7.0).all())


def _installed(N, cfg, src, upload):
    c = N.Cache(cfg)
    upload(c, src)
    torch.cuda.synchronize()
    return c.ws.clone()


@pytest.mark.parametrize("prec", ["fp32", "fp16", "bf16"])
def test_device_weights_that_a_kernel_may_not_reach(N, prec):
    """Weights in pinned host memory, or on another device, are copied to the cache first:
    every byte of its workspace is what the cache's own device's weights give."""
    cfg = N.make_config(n_hidden=3, precision=prec, ema_alpha=0.9)
    w = torch.from_numpy(sd.glorot_weights(64, 3, seed=5))
    want = _installed(N, cfg, w.cuda(), lambda c, t: c.set_weights_device(t))
    call = lambda c, t: N.check(N.lib.nrc_set_weights_device(c.handle, t.data_ptr(), t.numel(), N._stream(None)))
    assert torch.equal(_installed(N, cfg, w.pin_memory(), call), want)
    if torch.cuda.device_count() > 1:
        other = w.to("cuda:1")
        torch.cuda.synchronize(1)
        assert torch.equal(_installed(N, cfg, other, lambda c, t: c.set_weights_device(t)), want)


def test_device_weights_set_inside_a_graph(N):
    """The upload can be captured; every replay installs what the tensor holds then."""
    c, ref = (N.Cache(N.make_config(precision="fp16", ema_alpha=0.9)) for _ in range(2))
    w = torch.zeros(c.n_params, device="cuda")
    side = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        c.set_weights_device(w)
        torch.cuda.synchronize()
        with torch.cuda.graph(g, stream=side):
            c.set_weights_device(w)
    for seed in range(3):
        host = sd.glorot_weights(64, 5, seed=seed)
        w.copy_(torch.from_numpy(host))
        ref.set_weights(host)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(c.ws, ref.ws)


# tiles of the fullest compute unit and hidden layers: FP32 queries on either side of the
# lines between 16-query units and 64-query tiles (a last round full, or nearly so)
@pytest.mark.parametrize("n_hidden,r", [(1, 2), (1, 3), (2, 6), (2, 8), (5, 7), (5, 8), (5, 9), (5, 12), (5, 13),
                                        (3, 17), (3, 18), (6, 16), (6, 21), (4, 24), (4, 25)])
@pytest.mark.parametrize("raw_form", [False, True])
@pytest.mark.parametrize("rest", [0, -37])
def test_fp32_batches_of_units_and_of_tiles_agree(N, n_hidden, r, raw_form, rest):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    test_batches_and_their_slices_agree(N, "fp32", 64, n_hidden, raw_form, 64 * r * cus + rest - 24 * 64 * cus)


@pytest.mark.parametrize("preset,layout", [(0, 1), (1, 0), (2, 1), (3, 0), (3, 1)])
@pytest.mark.parametrize("r", [3, 8, 18])
def test_fp32_raw_batches_of_units_and_of_tiles_agree(N, preset, layout, r):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    n = 64 * r * cus - 5
    c = N.Cache(N.make_config(n_hidden=3, precision="fp32", enc_preset=preset, factorize=True))
    c.set_weights(sd.glorot_weights(64, 3, seed=3))
    raw = torch.from_numpy(sd.raw_records(n, 41, layout)).cuda()
    whole = N.nrc_forward_raw(c, raw, layout)
    assert torch.equal(N.nrc_forward(c, N.nrc_encode(c, raw, layout)), whole)
    for lo in (0, 64 * cus * (r - 1)):
        assert torch.equal(N.nrc_forward_raw(c, raw[lo:lo + 64 * cus].clone(), layout), whole[lo:lo + 64 * cus])
