"""The FP16/BF16 trainer over many tiles (weight gradients summed in registers).

A record's forward pass and deltas do not depend on its batch, so dL/d(input) of
a large batch equals that of its slices bit for bit.  The weight gradients are
FP32 sums of the same products in another order.  With non-negative weights,
inputs and upstream gradients every product is non-negative, so each sum's
relative error is at most its number of roundings times 2^-24: at most 64 per
tile that a workgroup takes and one per partial, on either side.
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


def _cus():
    return torch.cuda.get_device_properties(0).multi_processor_count


# tiles per compute unit, records past the last whole tile: one workgroup per CU
# with one or two tiles, two workgroups per CU, and ragged ends
SIZES = [(1, 1), (1, 64), (2, -63), (3, 5), (4, 0)]


@pytest.mark.parametrize("prec,width,n_hidden", [("fp16", 64, 5), ("bf16", 64, 5), ("fp16", 64, 1), ("bf16", 64, 2),
                                                 ("fp16", 64, 6), ("bf16", 64, 8), ("fp16", 128, 5), ("bf16", 128, 5),
                                                 ("fp16", 128, 1), ("bf16", 128, 3)])
@pytest.mark.parametrize("per_cu,rest", SIZES)
def test_gradients_of_a_large_batch_and_of_its_slices(N, prec, width, n_hidden, per_cu, rest):
    tiles = per_cu * _cus()
    n = 64 * tiles + rest
    fact = n_hidden in (2, 5)
    cfg = N.make_config(width=width, n_hidden=n_hidden, precision=prec, factorize=fact)
    c = N.Cache(cfg)
    c.set_weights(np.abs(sd.glorot_weights(width, n_hidden, seed=2)) / np.float32(width ** 0.5))
    enc = torch.from_numpy(sd.uniform_features(n, 64, 11)).cuda().to(c.enc_dtype)
    up = torch.rand(n, 3, device="cuda", generator=torch.Generator("cuda").manual_seed(4)) * 0.5 + 0.5
    rgb, act = N.nrc_forward_train(c, enc)
    got_w, got_x = N.nrc_backward(c, enc, up, act=act)
    again_w, again_x = N.nrc_backward(c, enc, up)           # the forward pass recomputed
    assert torch.equal(got_w, again_w) and torch.equal(got_x, again_x)
    only_w, none = N.nrc_backward(c, enc, up, want_grad_enc=False, act=act)
    assert none is None and torch.equal(only_w, got_w)
    ref_w = torch.zeros_like(got_w, dtype=torch.float64)
    step = 64 * (_cus() // 2) - 7
    for lo in range(0, n, step):
        e, u = enc[lo:lo + step].clone(), up[lo:lo + step].clone()
        assert torch.equal(N.nrc_forward_train(c, e)[0], rgb[lo:lo + step])
        w, x = N.nrc_backward(c, e, u)
        assert torch.equal(x, got_x[lo:lo + step]), lo
        ref_w += w.double()
    bound = 2 * (64 * (per_cu + 1) + 2 * _cus()) * 2.0 ** -24
    assert bool((ref_w >= 0).all())
    assert bool(((got_w.double() - ref_w).abs() <= bound * ref_w).all())


@pytest.mark.parametrize("prec,n_hidden", [("fp16", 5), ("bf16", 5), ("bf16", 8), ("fp16", 1)])
@pytest.mark.parametrize("preset,layout", [(0, 0), (1, 1), (2, 0), (3, 1)])
@pytest.mark.parametrize("past", [1, 64 * 300 + 9])
def test_raw_encoded_and_indexed_steps_agree(N, prec, n_hidden, preset, layout, past):
    """One step over a batch of more tiles than compute units: from raw records, from
    encoded rows and through an index list, equal bit for bit."""
    n = 64 * _cus() + past
    cfg = N.make_config(n_hidden=n_hidden, precision=prec, enc_preset=preset, ema_alpha=0.9)
    w = sd.glorot_weights(64, n_hidden, seed=6)
    raw_np = sd.raw_records(n, 77, layout)
    raw, y = torch.from_numpy(raw_np).cuda(), torch.from_numpy(sd.targets(raw_np)).cuda()
    res = []
    for form in ("raw", "encoded", "indexed"):
        c = N.Cache(cfg)
        c.set_weights(w)
        if form == "raw":
            loss, skipped = N.nrc_train_frame_raw(c, raw, y, layout, steps=1, batch=n, seed=5)
        elif form == "encoded":
            loss, skipped = N.nrc_train_frame(c, N.nrc_encode(c, raw, layout), y, steps=1, batch=n, seed=5)
        else:
            loss, skipped = N.nrc_train_step_indexed(c, N.nrc_encode(c, raw, layout), y, N.nrc_shuffle(n, 5))
        assert int(skipped.item()) == 0
        res.append((loss.clone(), c.ws.clone()))
    for loss, ws in res[1:]:
        assert torch.equal(loss, res[0][0]) and torch.equal(ws, res[0][1])


def test_a_non_finite_gradient_in_any_tile_skips_the_step(N):
    n = 64 * _cus() * 3 + 100
    for prec, width in (("fp16", 64), ("bf16", 128)):
        c = N.Cache(N.make_config(width=width, precision=prec))
        w = sd.glorot_weights(width, 5, seed=8)
        c.set_weights(w)
        raw = sd.raw_records(n, 13)
        enc, y = N.nrc_encode(c, torch.from_numpy(raw).cuda()), torch.from_numpy(sd.targets(raw)).cuda()
        for at in (0, 64 * _cus() + 70, n - 1):
            bad = y.clone()
            bad[at, 1] = float("nan")
            _, skipped = N.nrc_train_step(c, enc, bad)
            assert int(skipped.item()) == 1
            assert np.array_equal(c.get_weights(), w)


@pytest.mark.parametrize("n", [64 * 64, 64 * 65, 64 * 2048 - 1, 64 * 2049 + 3])
def test_the_loss_of_any_number_of_tiles(N, n):
    """The reduction adds the tiles' loss terms in rounds of 2,048: the loss of n records is
    the mean over its parts (compensated FP32 sums of non-negative terms, one rounding each)."""
    enc = torch.from_numpy(sd.uniform_features(n, 64, 3)).cuda().half()
    y = torch.rand(n, 3, device="cuda", generator=torch.Generator("cuda").manual_seed(1))

    def loss(lo, hi):
        c = N.Cache(N.make_config(precision="fp16", n_hidden=2))
        c.set_weights(sd.glorot_weights(64, 2, seed=3))
        return N.nrc_train_step(c, enc[lo:hi].clone(), y[lo:hi].clone())[0].item() * (hi - lo)

    parts = sum(loss(lo, min(lo + 4096, n)) for lo in range(0, n, 4096))
    # a tile's 64 terms are added in FP32 with compensation; scaling and its inverse round twice
    assert abs(loss(0, n) - parts) <= 8 * 2.0 ** -24 * parts


# ---------------------------------------------------------------------------
# Many tiles per workgroup
# ---------------------------------------------------------------------------
TILES = 129                                     # per workgroup, more than its sums are held for


@pytest.mark.parametrize("prec,width,wgs_per_cu", [("fp16", 64, 2), ("bf16", 64, 2), ("fp16", 128, 1), ("bf16", 128, 1)])
@pytest.mark.parametrize("n_hidden", [1, 3])
def test_small_gradients_after_large_ones_are_not_lost(N, prec, width, wgs_per_cu, n_hidden):
    """A weight gradient's terms, positive and equal but for a factor: the records of every
    workgroup's first tile weigh 2^24 times the others'.  A tile's term of 1 is half a unit in
    the last place of the 2^24 before it and vanishes in an FP32 sum that holds both.  A sum
    over at most 8 tiles loses at most 7 * 2^-24 of the gradient, one over all of them
    128 * 2^-24.  Every operand is a power of two, so products and exact sums are known;
    16 * 2^-24 leaves room for the sums' own roundings (two per tile)."""
    cus = _cus()
    wgs = cus * wgs_per_cu
    n = 64 * wgs * TILES
    c = N.Cache(N.make_config(width=width, n_hidden=n_hidden, precision=prec, loss_scale=1.0))
    w = np.concatenate([np.full(64 * width, 2.0 ** -6)] + [np.full(width * width, 1.0 / width)] * (n_hidden - 1) +
                       [np.full(3 * width, 0.25)]).astype(np.float32)
    c.set_weights(w)                            # every activation and prediction weight as below
    enc = torch.ones((n, 64), dtype=c.enc_dtype, device="cuda")
    up = torch.zeros((n, 3), device="cuda")
    up[:, 0] = 2.0 ** -12
    up[: 64 * wgs, 0] = 2.0 ** 12               # tile b is workgroup b's first
    grad, _ = N.nrc_backward(c, enc, up, want_grad_enc=False)
    total = 64 * wgs * (2.0 ** 12 + (TILES - 1) * 2.0 ** -12)
    want = np.full(w.shape, 0.25 * total)       # h_l = 1 and delta_l = dL/dy / 4 in every layer
    want[-3 * width:] = 0.0
    want[-3 * width:-2 * width] = total         # dL/dy is zero in two channels
    got = grad.cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got - want) <= 16 * 2.0 ** -24 * want)


# tiles per compute unit, records past the last whole tile: two launches, the second
# with one whole tile and a ragged one, or as many as the first less a record
@pytest.mark.parametrize("prec,width,n_hidden,per_cu,rest", [("fp16", 64, 2, 16, 69), ("bf16", 64, 5, 16, 69),
                                                             ("fp16", 64, 6, 8, 69), ("bf16", 64, 8, 8, 69),
                                                             ("fp16", 128, 5, 8, 69), ("bf16", 128, 3, 16, -1)])
def test_gradients_over_several_launches(N, prec, width, n_hidden, per_cu, rest):
    test_gradients_of_a_large_batch_and_of_its_slices(N, prec, width, n_hidden, per_cu, rest)


@pytest.mark.parametrize("prec,n_hidden,layout", [("fp16", 2, 0), ("bf16", 5, 1), ("fp16", 8, 1)])
@pytest.mark.parametrize("n", [64 * 8 * 512 + 64 + 5, 1 << 20])   # an index list; the orbit in the kernel
def test_steps_over_several_launches(N, prec, n_hidden, layout, n):
    """Raw, encoded and indexed steps as above, and a step on the rows as they lie equal to
    one through the list 0, 1, 2, ...; the loss is that of the same records in slices."""
    test_raw_encoded_and_indexed_steps_agree(N, prec, n_hidden, 1, layout, n - 64 * _cus())
    cfg = N.make_config(n_hidden=n_hidden, precision=prec, enc_preset=1)
    w = sd.glorot_weights(64, n_hidden, seed=6)
    raw = sd.raw_records(n, 78, layout)
    res = []
    for form in ("rows", "list"):
        c = N.Cache(cfg)
        c.set_weights(w)
        enc, y = N.nrc_encode(c, torch.from_numpy(raw).cuda(), layout), torch.from_numpy(sd.targets(raw)).cuda()
        if form == "rows":
            loss, skipped = N.nrc_train_step(c, enc, y)
        else:
            loss, skipped = N.nrc_train_step_indexed(c, enc, y, torch.arange(n, dtype=torch.int32, device="cuda"))
        assert int(skipped.item()) == 0
        res.append((loss.clone(), c.ws.clone()))
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])
    bad = y.clone()
    bad[n - 1, 2] = float("inf")                # in the last launch
    assert int(N.nrc_train_step(c, enc, bad)[1].item()) == 1


def test_the_loss_over_several_launches(N):
    test_the_loss_of_any_number_of_tiles(N, 64 * 8 * 512 + 64 * 70 + 1)


# ---------------------------------------------------------------------------
# Two workgroups per compute unit (width 64, up to depth 5, more than three tiles each)
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("prec,n_hidden", [("fp16", 5), ("bf16", 5), ("bf16", 2), ("fp16", 1)])
@pytest.mark.parametrize("preset,layout", [(p, la) for p in range(4) for la in range(2)])
def test_steps_of_two_workgroups_per_cu_agree(N, prec, n_hidden, preset, layout):
    test_raw_encoded_and_indexed_steps_agree(N, prec, n_hidden, preset, layout, 64 * (2 * _cus() + 5) + 9)


@pytest.mark.parametrize("prec,n_hidden", [("fp16", 5), ("bf16", 5), ("fp16", 1), ("bf16", 3)])
def test_the_weights_of_a_step_with_two_workgroups_per_cu(N, prec, n_hidden):
    """The first moment after one step is 0.1 times the gradient.  The gradient of four tiles
    per compute unit is the mean over its quarters, one tile and one workgroup per compute
    unit each: with the loss scale in proportion to the records their deltas are the same
    numbers.  Weights and inputs are non-negative and the targets zero, so every product is
    non-negative and the bound is that of the gradients above."""
    q = 64 * _cus()
    enc_np = sd.uniform_features(4 * q, 64, 17)
    w = np.abs(sd.glorot_weights(64, n_hidden, seed=2)) / np.float32(8.0)

    def step(lo, hi):
        c = N.Cache(N.make_config(n_hidden=n_hidden, precision=prec, loss_scale=2.0 ** 16 * (hi - lo) / q))
        c.set_weights(w)
        enc = torch.from_numpy(enc_np[lo:hi]).cuda().to(c.enc_dtype)
        loss, skipped = N.nrc_train_step(c, enc, torch.zeros((hi - lo, 3), device="cuda"))
        assert int(skipped.item()) == 0
        _, m, v, t = c.get_state()
        assert t == 1
        return loss.item(), m.astype(np.float64), c

    loss, m, c = step(0, 4 * q)
    parts = [step(i * q, (i + 1) * q) for i in range(4)]
    want = sum(p[1] for p in parts) / 4
    bound = 2 * (64 * (4 + 1) + 2 * _cus()) * 2.0 ** -24
    assert np.all(want >= 0) and np.count_nonzero(want) > want.size // 2
    assert np.all(np.abs(m - want) <= bound * want)
    assert abs(loss - sum(p[0] for p in parts) / 4) <= 8 * 2.0 ** -24 * loss
    # Adam's first step from there: w - lr * sign(g) but for eps, in every weight
    moved = w.astype(np.float64) - c.get_weights()
    assert np.any(want > 1e-6) and np.allclose(moved[want > 1e-6], 1e-2, rtol=1e-2)


@pytest.mark.parametrize("prec,width,n_hidden,per_cu", [("fp16", 128, 1, 1), ("bf16", 128, 2, 1), ("fp16", 128, 5, 1),
                                                        ("bf16", 64, 6, 1), ("fp16", 64, 5, 2), ("bf16", 64, 1, 2)])
def test_workgroups_beyond_those_a_cu_holds_are_not_launched(N, prec, width, n_hidden, per_cu):
    """A wave of the width-128 trainer takes 256 registers: one workgroup fills a compute
    unit whatever its LDS.  Each workgroup writes one partial of n_params floats, from the
    start of the scratch on."""
    cus = _cus()
    n = 64 * 4 * cus
    c = N.Cache(N.make_config(width=width, n_hidden=n_hidden, precision=prec))
    c.set_weights(sd.glorot_weights(width, n_hidden, seed=2))
    enc = torch.from_numpy(sd.uniform_features(n, 64, 11)).cuda().to(c.enc_dtype)
    sc = N._aligned_bytes(N.nrc_train_scratch_bytes(c.cfg, n), "cuda").fill_(0xff)   # NaN where nothing is written
    N.nrc_train_step(c, enc, torch.rand((n, 3), device="cuda"), scratch=sc)
    slots = sc[:4 * c.n_params * 4 * cus].view(torch.float32).view(4 * cus, c.n_params)
    written = ~slots.isnan().all(dim=1)
    assert int(written.sum()) == per_cu * cus and bool(written[:per_cu * cus].all())
