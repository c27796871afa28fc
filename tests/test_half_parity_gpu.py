"""The split kernels on two f16 terms (split_f16.h) against the oracle.

Tolerance.  An operand is off by at most 2^-23 of itself and a product misses another 2^-22, of random sign; the sums are rounded
once per 16 or 32 indices as on the bf16 terms.  Over 32 indices and more the operands' part is below a fifth of
2^-24 sqrt(K/16 + 32), the bound of test_split_parity_gpu.py, which holds here too.  Operands that the terms cannot hold come from
the bf16 terms, within the same bound, or, where those cannot either, from the fp32 matrix instructions, which round every second
index: 2^-24 sqrt(K/2 + 32).
"""
import re

import numpy as np
import pytest
import torch

import oracle
import paper_1810_02272_amd as conv
from oracle import OracleParams
from paper_1810_02272_amd import workloads
from parity_cases import FOLD_CASES, HALF_CASES, SPLIT_CASES, P
from parity_metric import nerr
from test_parity_gpu import TOL, check_filter_and_bias_in_one_pass, run_all
from test_split_parity_gpu import CORR, DEV, ODD, WGRAD, check_odd_values, names, norm_error

PASSES = ("fwd", "bwd_data", "bwd_filter")
MIXED = P(24, 128, 28, 28, 128, 3, 3, 1, 1, 1, 1)  # all three passes on f16 terms
PIXELS = P(4096, 1400, 1, 1, 1400, 1, 1)


def test_cases_select_every_instance():
    corr, wgrad = set(), set()
    for pd in HALF_CASES + SPLIT_CASES:
        n = names(pd)
        for which in PASSES[:2]:
            m = CORR.match(n[which])
            if m and "half" in n[which]:
                corr |= {(m[1], m[3] if m[2] == "p" else m[2]), (which, m[4], int(m[5]) > 1)}
        m = WGRAD.match(n["bwd_filter"])
        if m and "half" in n["bwd_filter"]:
            wgrad |= {(m[1], m[2]), m[3]}
    tiles = ["m32_128x128", "m32_64x256", "m32_64x128", "m32_96x128", "m32_32x256", "m32_32x128", "m16_48x256"]
    want = {(t, u) for t in tiles for u in ("34" if t.endswith("x256") else "234")}
    want |= {(t, f) for t in ("m32_128x128", "m32_64x128", "m32_96x128") for f in ("cols", "rows")}
    want |= {("fwd", "s", s) for s in (False, True)} | {("bwd_data", e, s) for e in "sr" for s in (False, True)}
    assert want - corr == set()
    assert {(t, u) for t in ("128x9", "128x8", "64x16", "32x28", "32x12", "96x8") for u in "234"} | {"1", "2"} <= wgrad


def test_folded_filter_gradients_select_every_instance():
    found = set()
    for pd in FOLD_CASES:
        m = re.match(r"splitwgrad_fold\d+_(\d+x\d+)x16\[p(\d),st(\d)", names(pd)["bwd_filter"])
        found |= {(m[1], "4" if m[2] == "4" else "3"), m[3]} if m else set()
    assert found >= {(t, u) for t in ("96x10", "128x9", "64x16", "32x12") for u in "34"} | {"1", "2"}


WIDE = P(130, 2064, 13, 13, 512, 3, 1, 1, 1, 1, 0)  # a grid that fills the chip, 129 chunks: one more than a slice's bits


def test_many_chunks_take_the_least_slices_that_hold_them():
    for c, slices in ((2048, 1), (2064, 2), (4096, 2), (4112, 3)):
        assert f"(S={slices},half" in names(dict(WIDE, c=c))["fwd"], c


@pytest.mark.gpu
@pytest.mark.parametrize("r", [0, 40])
def test_many_chunks_in_slices(r):
    """r: the last channel, the second slice's last, 2^-r of the others in half of the images"""
    d, n = conv.conv_desc_create(conv.ConvParams(**WIDE)), 4
    gen = torch.Generator(device=DEV).manual_seed(9904)
    x, w, b = (torch.randn(s, device=DEV, generator=gen) for s in ((130, 2064, 13, 13), (512, 2064, 3, 1), (512,)))
    x[::2, -1] *= 2.0 ** -r
    y = torch.full(conv.conv_desc_output_shape(d), float("nan"), device=DEV)
    ws = torch.full(((conv.conv_desc_workspace_bytes(d) + 7) // 8,), float("nan"), device=DEV, dtype=torch.float64)
    conv.conv_forward(d, x, w, b, y, ws)
    assert not torch.isnan(y).any()
    for first in (0, 126):
        cols = torch.nn.functional.unfold(x[first:first + n].double(), (3, 1), padding=(1, 0))
        ref = torch.matmul(w.double().view(512, -1), cols).view(n, 512, 13, 13) + b.double().view(1, -1, 1, 1)
        err = (y[first:first + n] - ref).flatten(1).norm(dim=1) / ref.flatten(1).norm(dim=1)
        assert float(err.max()) <= 2.0 ** -24 * np.sqrt(6192 / 16 + 32)


def test_short_sums_stay_on_the_bf16_terms():
    """The operands' error is below the sums' from about 620 indices on; slices count by themselves."""
    assert "half" not in names(P(64, 64, 28, 28, 128, 3, 3, 1, 1, 1, 1))["fwd"]
    assert "half" in names(P(64, 80, 28, 28, 128, 3, 3, 1, 1, 1, 1))["fwd"]
    for n, c, k in ((128, 9216, 4096), (300, 5000, 3000), (64, 2048, 2048), (900, 700, 900)):
        name = names(P(n, c, 1, 1, k, 1, 1))["fwd"]
        if "half" in name:
            assert c / int(re.search(r"S=(\d+)", name)[1]) > 600, name


def passes_of(pd, dev, host):
    """(name, kernel, result, reference, reduction length) of the three passes"""
    op, kernels, taps = OracleParams(**pd), names(pd), pd["kernel_h"] * pd["kernel_w"]
    ys = oracle.output_shape(op)
    y, dx, dw = dev
    return (("y", kernels["fwd"], y, oracle.forward(op, *host[:3]), pd["c"] // pd["group"] * taps),
            ("dx", kernels["bwd_data"], dx, oracle.backward_data(op, host[1], host[3]), pd["num_output"] // pd["group"] * taps),
            ("dw", kernels["bwd_filter"], dw, oracle.backward_filter(op, host[0], host[3]), ys[0] * ys[2] * ys[3]))


@pytest.mark.gpu
@pytest.mark.parametrize("i", range(len(HALF_CASES + FOLD_CASES)))
def test_half_full_compare(i):
    pd = (HALF_CASES + FOLD_CASES)[i]
    print("half case", i, pd, names(pd), flush=True)
    op = OracleParams(**pd)
    x, w, b, dy = workloads.random_inputs(oracle.x_shape(op), oracle.w_shape(op), oracle.output_shape(op), 9100 + 10 * i)
    d, ws, dev_in, (y, dx, dw, db) = run_all(pd, x, w, b, dy)
    host = (x.numpy(), w.numpy(), b.numpy(), dy.numpy())
    for name, kernel, got, ref, terms in passes_of(pd, (y, dx, dw), host):
        assert nerr(got, ref) <= TOL, (pd, name)
        if "split" in kernel:
            assert norm_error(got, ref) <= 2.0 ** -24 * np.sqrt(terms / 16 + 32), (pd, name, norm_error(got, ref))
    check_filter_and_bias_in_one_pass(pd, op, d, ws, dev_in, dw, oracle.backward_bias(op, host[3]), host)
    dw1 = dw.clone()  # beta = 1: dw + dw is exact
    conv.conv_backward_filter(d, dev_in[0], dev_in[3], dw1, 1.0, ws)
    torch.cuda.synchronize()
    assert torch.equal(dw1, dw + dw)


@pytest.mark.gpu
@pytest.mark.parametrize("pd", [MIXED, PIXELS], ids=["image", "rows"])
@pytest.mark.parametrize("case", ["tiny_images", "huge_image", "tiny_weights", "outliers", "zeros", "relu", "denormals"])
def test_ranges_beyond_f16(pd, case):
    """Images, weights and single values far from the sample's size: every image and every output channel keeps the bound by itself."""
    assert all("half" in names(pd)[p] for p in (PASSES[:2] if pd is PIXELS else PASSES))
    op = OracleParams(**pd)
    x, w, b, dy = workloads.random_inputs(oracle.x_shape(op), oracle.w_shape(op), oracle.output_shape(op), 9900)
    b = b * 0
    if case == "tiny_images":
        for t in (x, dy):
            t[3] *= 2.0 ** -20
            t[5] *= 2.0 ** -30
            t[6] *= 2.0 ** -70
    elif case == "huge_image":
        x[2] *= 2.0 ** 40
        dy[2] *= 2.0 ** 40
    elif case == "tiny_weights":
        w[7] *= 2.0 ** -40
        w[:, 16:32] *= 2.0 ** -28
    elif case == "outliers":
        for t in (x, dy, w):
            t.view(-1)[t.numel() // 3 + 5] = 1e9
    elif case == "zeros":
        x.zero_()
        w[:, 8:].zero_()
    elif case == "relu":
        x, dy = x.clamp(min=0), torch.where(dy > 0, dy, torch.zeros_like(dy))
    else:
        x, dy = x * 2.0 ** -130, dy * 2.0 ** -130
    d, ws, _, (y, dx, dw, db) = run_all(pd, x, w, b, dy)
    host = (x.numpy(), w.numpy(), b.numpy(), dy.numpy())
    for name, kernel, got, ref, terms in passes_of(pd, (y, dx, dw), host):
        if case == "denormals" and name == "dw":
            assert not got.any()  # products of 2^-260
            continue
        g, bound = got.cpu().double().numpy(), 2.0 ** -24 * np.sqrt(terms / 2 + 32)
        if case == "outliers":
            # one large term leaves every later partial sum at full size, and the roundings to it need not be of random sign; by
            # element, so that the large ones do not stand for the others
            mag = [np.abs(v) for v in host]
            size = {"y": lambda: oracle.forward(op, *mag[:3]), "dx": lambda: oracle.backward_data(op, mag[1], mag[3]),
                    "dw": lambda: oracle.backward_filter(op, mag[0], mag[3])}[name]()
            assert np.all(np.abs(g - ref) <= 2.0 ** -24 * (terms / 2 + 32) * size), (name, kernel)
            continue
        # both channels of dw; images of y and dx, and their channels (of one pixel each they may be single sums, which cancel)
        for axis in ((0,) if pd is PIXELS else (0, 1)):
            err = np.linalg.norm(np.moveaxis(g - ref, axis, 0).reshape(g.shape[axis], -1), axis=1)
            size = np.linalg.norm(np.moveaxis(ref, axis, 0).reshape(g.shape[axis], -1), axis=1)
            if case == "denormals":
                size = size + 2.0 ** -149 * 2 ** 24 * np.sqrt(g.size / g.shape[axis])  # results are denormal themselves
            assert np.all(err <= bound * size), (name, kernel, axis, np.max(err / np.maximum(size, 1e-300)) / bound)


RAGGED = P(40, 180, 20, 21, 204, 3, 3, 1, 1, 1, 1, g=2)  # 90 and 102 channels a group: the last eight of a group are not its own
FOLDED = FOLD_CASES[4]  # 1 x 4 taps to a channel of the fold: two of the image's channels in eight


def errors_by(axes, got, ref, terms, group=1):
    """Largest error of a slice along one of `axes`, in units of the slice's own bound; `group`: every group's channels of dw apart"""
    if group > 1:
        per = ref.shape[0] // group
        return max(errors_by(axes, got[i * per:(i + 1) * per], ref[i * per:(i + 1) * per], terms) for i in range(group))
    g, worst = got.cpu().double().numpy().reshape(ref.shape), 0.0
    for axis in axes:
        err = np.linalg.norm(np.moveaxis(g - ref, axis, 0).reshape(g.shape[axis], -1), axis=1)
        size = np.linalg.norm(np.moveaxis(ref, axis, 0).reshape(g.shape[axis], -1), axis=1)
        worst = max(worst, float(np.max(err / size)) / (2.0 ** -24 * np.sqrt(terms / 2 + 32)))
    return worst


@pytest.mark.gpu
@pytest.mark.parametrize("r", [22, 30, 44, 60])
@pytest.mark.parametrize("pd", [MIXED, RAGGED, FOLDED, PIXELS], ids=["image", "ragged", "folded", "rows"])
def test_dim_channels_of_the_filter_gradient(pd, r):
    """One channel of x and one of dy far below the others: their parts of dw are sums over them alone."""
    assert "half" in names(pd)["bwd_filter"] or pd is PIXELS
    op = OracleParams(**pd)
    x, w, b, dy = workloads.random_inputs(oracle.x_shape(op), oracle.w_shape(op), oracle.output_shape(op), 9901)
    x[:, pd["c"] // 2] *= 2.0 ** -r
    dy[:, 6] *= 2.0 ** -r
    _, _, _, (_, _, dw, _) = run_all(pd, x, w, b, dy)
    ys = oracle.output_shape(op)
    assert errors_by((0, 1), dw, oracle.backward_filter(op, x.numpy(), dy.numpy()), ys[0] * ys[2] * ys[3], pd["group"]) <= 1


@pytest.mark.gpu
@pytest.mark.parametrize("r", [22, 30, 44, 60])
@pytest.mark.parametrize("how", ["equalised", "hidden"])
@pytest.mark.parametrize("pd", [MIXED, RAGGED, PIXELS], ids=["image", "ragged", "rows"])
def test_channels_of_different_sizes_in_one_sum(pd, how, r):
    """Every eighth reduction channel 2^-r of the others with weights 2^r of theirs, which leaves the sums as they are; or the
    others 2^-r of every eighth, whose weights are zero."""
    assert all("half" in names(pd)[p] for p in PASSES[:2])
    op, taps = OracleParams(**pd), pd["kernel_h"] * pd["kernel_w"]
    for which in PASSES[:2]:
        x, w, b, dy = workloads.random_inputs(oracle.x_shape(op), oracle.w_shape(op), oracle.output_shape(op), 9902)
        b = b * 0
        blob, per_group = (x, pd["c"] // pd["group"]) if which == "fwd" else (dy, pd["num_output"] // pd["group"])
        eighth = torch.arange(per_group) % 8 == 3
        scale = torch.where(eighth == (how == "equalised"), 2.0 ** -r, 1.0)
        blob *= scale.repeat(pd["group"]).view(1, -1, 1, 1)
        by_w = 1 / scale if how == "equalised" else torch.where(eighth, 0.0, 1.0)
        w *= by_w.view(1, -1, 1, 1) if which == "fwd" else by_w.repeat(pd["group"]).view(-1, 1, 1, 1)
        _, _, _, (y, dx, _, _) = run_all(pd, x, w, b, dy)
        if which == "fwd":
            got, ref = y, oracle.forward(op, x.numpy(), w.numpy(), b.numpy())
        else:
            got, ref = dx, oracle.backward_data(op, w.numpy(), dy.numpy())
        assert errors_by((0,) if pd is PIXELS else (0, 1), got, ref, per_group * taps) <= 1, which


@pytest.mark.gpu
@pytest.mark.parametrize("pd", [P(64, 256, 13, 13, 384, 3, 3, 1, 1, 1, 1), P(32, 128, 56, 56, 128, 3, 3, 1, 1, 1, 1)], ids=["13x13", "56x56"])
def test_an_image_far_below_the_others_costs_little(pd):
    """1.0 to 1.2 times a pass, and 1.6 where the image is half of a slice of the filter gradient (made of NaN: 3 to 5 times)."""
    assert all("half" in names(pd)[p] for p in PASSES)
    d, op = conv.conv_desc_create(conv.ConvParams(**pd)), OracleParams(**pd)
    x, w, b, dy = (t.to(DEV) for t in workloads.random_inputs(oracle.x_shape(op), oracle.w_shape(op), oracle.output_shape(op), 9903))
    y, dx, dw, db = torch.empty_like(dy), torch.empty_like(x), torch.empty_like(w), torch.empty_like(b)
    ws = torch.empty((conv.conv_desc_workspace_bytes(d) + 7) // 8, device=DEV, dtype=torch.float64)
    x1, dy1 = x.clone(), dy.clone()
    for t in (x1, dy1):
        t[pd["n"] // 2] *= 2.0 ** -30

    def ms(call):
        best = float("inf")
        for _ in range(4):
            start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            start.record()
            for _ in range(5):
                call()
            end.record()
            torch.cuda.synchronize()
            best = min(best, start.elapsed_time(end))
        return best

    for which, call in (("fwd", lambda x, dy: conv.conv_forward(d, x, w, b, y, ws)),
                        ("bwd_data", lambda x, dy: conv.conv_backward_data(d, w, dy, dx, ws)),
                        ("bwd_filter", lambda x, dy: conv.conv_backward_filter_bias(d, x, dy, dw, db, 0.0, ws))):
        plain, uneven = ms(lambda: call(x, dy)), ms(lambda: call(x1, dy1))
        assert uneven < 2 * plain, (which, plain, uneven)


@pytest.mark.gpu
@ODD
def test_odd_values_in_the_folded_filter_gradient(odd):
    """Below and right of windows that do not have them too: 11 taps are rounded up to 12."""
    check_odd_values(P(60, 3, 147, 151, 128, 11, 11, 4, 4), odd, ("bwd_filter",), (15, 19, 4))
