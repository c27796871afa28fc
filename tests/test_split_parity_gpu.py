"""The kernels on three-way split bf16 operands (corr_split_kernel, wgrad_split_kernel) against the oracle.

Tolerance.  The split holds every bit of an operand, so the error is that of fp32 accumulation: the long sum of K terms is
rounded once per 16 of them (32 for the 16-row instruction), each rounding at most 2^-24 of a partial sum and of random sign,
so the 2-norm of the error is below 2^-24 sqrt(K/16 + 32) of the result's (the 32 stand for the split slices and the
partial products' own accumulator); element by element the suite's bar of 1e-4 applies.
"""
import re

import numpy as np
import pytest
import torch

import oracle
import paper_1810_02272_amd as conv
from oracle import OracleParams
from paper_1810_02272_amd import workloads
from parity_cases import SPLIT_CASES, SPLIT_PAD_CASES, P
from parity_metric import nerr
from test_ip_parity_gpu import run_case as run_ip_case
from test_parity_gpu import TOL, check_filter_and_bias_in_one_pass, run_all

DEV = "cuda:0"
CORR = re.compile(r"corrsplit_(m\d+_\d+x\d+)\[([a-z]+)(\d+),e(.)\]\(S=(\d+)")
WGRAD = re.compile(r"splitwgrad_(\d+x\d+)x16\[p(\d),st(\d)\]")


def names(pd):
    return dict(kv.split("=", 1) for kv in conv.conv_desc_kernel_names(conv.conv_desc_create(conv.ConvParams(**pd))).split(";"))


def test_cases_select_every_variant():
    corr, wgrad = set(), set()
    for pd in SPLIT_CASES:
        n = names(pd)
        for which in ("fwd", "bwd_data"):
            if m := CORR.match(n[which]):
                if m[2] == "p":
                    corr |= {(which, m[1]), (m[1], m[3]), (which, m[4], int(m[5]) > 1)}
                else:
                    corr |= {(which, m[2]), (m[2], m[1])}
        if m := WGRAD.match(n["bwd_filter"]):
            wgrad |= {(m[1], m[2]), m[3]}
    tiles = ["m32_128x128", "m32_64x256", "m32_64x128", "m32_96x128", "m32_32x256", "m32_32x128", "m16_48x256"]
    want = {(w, t) for w in ("fwd", "bwd_data") for t in tiles}
    want |= {(t, u) for t in tiles for u in ("34" if t.endswith("x256") else "234")}
    want |= {("fwd", "s", s) for s in (False, True)} | {("bwd_data", e, s) for e in "sr" for s in (False, True)}
    want |= {(f, t) for f in ("fold", "cols") for t in ("m32_128x128", "m32_64x128", "m32_96x128")} | {("fold", "m32_32x128")}
    want |= {("rows", t) for t in ("m32_128x128", "m32_64x128", "m32_96x128")}
    want |= {("fwd", "rows"), ("bwd_data", "rows"), ("fwd", "fold"), ("fwd", "cols"), ("bwd_data", "cols")}
    assert want - corr == set()
    assert {(t, u) for t in ("128x9", "128x8", "64x16", "32x28", "32x12", "96x8") for u in "234"} | {"1", "2"} <= wgrad


@pytest.mark.parametrize("h,w,split", [(1, 1, False), (1, 2, False), (1, 3, False), (1, 5, True), (2, 3, True),
                                       (1, 7, True), (5, 5, True)])
def test_filter_gradients_of_few_pixels(h, w, split):
    """Runs of eight pixels hold one image each: with up to three pixels they are mostly zeros (four are level)."""
    for n, c, k in ((128, 512, 512), (2048, 512, 512), (2048, 128, 256)):
        assert names(P(n, c, h, w, k, 3, 3, 1, 1, 1, 1))["bwd_filter"].startswith("splitwgrad") == split, (n, c, k)


def test_padding_of_runs_and_tiles_counts_together():
    """20 -> 320 channels pad rows and taps 1.75 times, 6 pixels the runs 1.33 times: 127 us fp32, 142 split."""
    assert names(P(6250, 20, 2, 3, 320, 5, 5, 1, 1, 2, 2))["bwd_filter"].startswith("wgrad")


def test_filter_gradients_that_the_fp32_kernel_is_faster_on():
    """2x2 and 1x3 taps leave half and more of the blocks of eight empty."""
    for pd in (P(48, 249, 15, 15, 266, 2, 2), P(1091, 50, 18, 18, 95, 1, 3), P(355, 744, 9, 9, 356, 2, 2, g=4)):
        assert names(pd)["bwd_filter"].startswith("wgrad"), pd


def test_many_weights_and_few_columns_stay():
    for pd in (P(1, 1024, 14, 14, 1024, 3, 3, 1, 1, 1, 1), P(2, 2048, 10, 10, 1024, 3, 3, 1, 1, 1, 1), P(1, 963, 14, 14, 878, 3, 3, 1, 1, 0, 1)):
        assert "split" not in names(pd)["fwd"], pd
    assert "split" not in names(P(2, 2048, 7, 7, 1024, 3, 3, 1, 1, 1, 1))["bwd_data"]
    # more columns for the same weights: 329 us fp32, 293 split
    assert "split" in names(P(4, 2048, 14, 14, 1024, 3, 3, 1, 1, 1, 1))["fwd"]


@pytest.mark.parametrize("m,k,o,split", [(512, 9216, 512, False), (1000, 4096, 500, False), (512, 9216, 900, True)])
def test_inner_products_of_few_outputs_stay(m, k, o, split):
    kernels = conv.ip_desc_kernel_names(conv.ip_desc_create(conv.IpParams(m=m, k=k, num_output=o, relu=1)))
    assert kernels.startswith("fwd=wgrad_on_corrsplit") == split, kernels


def norm_error(g, r):
    g = g.cpu().double().numpy().reshape(r.shape)
    return float(np.linalg.norm(g - r) / np.linalg.norm(r))


@pytest.mark.gpu
@pytest.mark.parametrize("i", range(len(SPLIT_CASES + SPLIT_PAD_CASES)))
def test_split_full_compare(i):
    pd = (SPLIT_CASES + SPLIT_PAD_CASES)[i]
    print("split case", i, pd, names(pd), flush=True)
    op = OracleParams(**pd)
    ys = oracle.output_shape(op)
    x, w, b, dy = workloads.random_inputs(oracle.x_shape(op), oracle.w_shape(op), ys, 6100 + 10 * i)
    d, ws, dev_in, (y, dx, dw, db) = run_all(pd, x, w, b, dy)
    host = (x.numpy(), w.numpy(), b.numpy(), dy.numpy())
    taps = pd["kernel_h"] * pd["kernel_w"]
    db_ref = oracle.backward_bias(op, host[3])
    kernels = names(pd)
    for name, which, got, ref, terms in (
            ("y", "fwd", y, oracle.forward(op, *host[:3]), pd["c"] // pd["group"] * taps),
            ("dx", "bwd_data", dx, oracle.backward_data(op, host[1], host[3]), pd["num_output"] // pd["group"] * taps),
            ("dw", "bwd_filter", dw, oracle.backward_filter(op, host[0], host[3]), ys[0] * ys[2] * ys[3])):
        assert nerr(got, ref) <= TOL, (pd, name)
        if "split" in kernels[which]:  # the bound is these kernels' own: the fp32 ones add a term per rounding
            assert norm_error(got, ref) <= 2.0 ** -24 * np.sqrt(terms / 16 + 32), (pd, name, norm_error(got, ref))
    check_filter_and_bias_in_one_pass(pd, op, d, ws, dev_in, dw, db_ref, host)
    # beta = 1: dw + dw is exact in fp32; the entry point without a workspace gives the same bits
    xd, _, _, dyd = dev_in
    dw1, dw2 = dw.clone(), torch.full_like(dw, float("nan"))
    conv.conv_backward_filter(d, xd, dyd, dw1, 1.0, ws)
    conv.conv_backward_filter_static(d, xd, dyd, dw2)
    torch.cuda.synchronize()
    assert torch.equal(dw1, dw + dw) and torch.equal(dw2, dw)


ODD = pytest.mark.parametrize("odd", [(float("inf"), float("-inf"), float("nan")), (3.4e38, -3.4028234e38)],
                              ids=["not_finite", "largest"])


@pytest.mark.gpu
@pytest.mark.parametrize("pd", [P(20, 48, 29, 30, 60, 5, 5), P(40, 48, 30, 31, 64, 3, 5)],
                         ids=["5x5", "3x5"])
@ODD
def test_infinities_nans_and_the_largest_floats(pd, odd):
    """An infinity or NaN spoils the split's differences and the largest floats round to a bf16 infinity: such sums are computed
    again, and must come out as plain fp32 arithmetic has them (no padding: a zero times an infinity is not the oracle's)."""
    check_odd_values(pd, odd, ("fwd", "bwd_data", "bwd_filter"))


@pytest.mark.gpu
@pytest.mark.parametrize("pd,passes", [
    (P(42, 3, 83, 87, 96, 11, 11, 4, 4), ("fwd",)), (P(8, 705, 39, 21, 284, 1, 1), ("fwd",)),
    (P(1200, 700, 1, 1, 2100, 1, 1), ("fwd", "bwd_data")), (P(24, 90, 29, 30, 90, 3, 5, g=2), ("fwd", "bwd_data", "bwd_filter"))],
    ids=["folded", "columns", "rows", "groups"])
@ODD
def test_odd_values_in_every_form(pd, passes, odd):
    """The same for the forms whose patch is not the image -- the folded one rounds 11x11 taps up to 12x12: the odd values sit
    right below and right of windows that do not have them -- and for channels of a chunk that are the next group's."""
    check_odd_values(pd, odd, passes, (15, 19, 4))


def check_odd_values(pd, odd, passes, at=None):
    """`at`: row and column of the first odd value of x, and the step to the next one's."""
    kernels = names(pd)
    assert all("split" in kernels[p] for p in passes), kernels
    op = OracleParams(**pd)
    x, w, b, dy = workloads.random_inputs(oracle.x_shape(op), oracle.w_shape(op), oracle.output_shape(op), 77)
    x_plain = x.clone()
    for i, v in enumerate(odd):
        r, c, step = at or (7 + i, 9, 0)
        x[i, 3 * i % x.shape[1], (r + i * step) % x.shape[2], (c + i * step) % x.shape[3]] = v
        dy[2 + i, 5 * i, 4 % dy.shape[2], (6 + 2 * i) % dy.shape[3]] = v
    d, ws, (_, _, bd, _), (y, dx, dw, db) = run_all(pd, x, w, b, dy)
    host = (x.numpy(), w.numpy(), b.numpy(), dy.numpy())
    # infinite and huge weights: forward only (the data gradient multiplies them with the zeros around dy, as any fp32
    # kernel does), on plain inputs
    w_inf = w.clone()
    w_inf[9, 3 % w.shape[1], 0, 2 % w.shape[3]] = float("inf")
    w_inf[7, 2, 1 % w.shape[2], 1 % w.shape[3]] = 3.4e38
    y_inf = torch.empty_like(y)
    conv.conv_forward(d, x_plain.to(DEV), w_inf.to(DEV), bd, y_inf, ws)
    torch.cuda.synchronize()
    mag = [np.abs(v) for v in host]
    results = []
    with np.errstate(all="ignore"):
        if "fwd" in passes:
            results += [("y", y, oracle.forward(op, *host[:3]), oracle.forward(op, *mag[:3])),
                        ("y, odd weights", y_inf, oracle.forward(op, x_plain.numpy(), w_inf.numpy(), host[2]),
                         oracle.forward(op, np.abs(x_plain.numpy()), np.abs(w_inf.numpy()), mag[2]))]
        if "bwd_data" in passes:
            results += [("dx", dx, oracle.backward_data(op, host[1], host[3]), oracle.backward_data(op, mag[1], mag[3]))]
        if "bwd_filter" in passes:
            results += [("dw", dw, oracle.backward_filter(op, host[0], host[3]), oracle.backward_filter(op, mag[0], mag[3]))]
    for name, got, ref, size in results:
        g = got.cpu().double().numpy().reshape(ref.shape)
        r = np.where(np.abs(ref) > 3.4028235e38, np.sign(ref) * np.inf, ref)  # what fp32 cannot hold
        close = np.isfinite(size) & (size > 1e38)  # terms at the edge of the range: fp32 may or may not overflow on the way
        with np.errstate(all="ignore"):
            same = (g == r) | (np.isnan(g) & np.isnan(r)) | close
            fine = np.isfinite(r) & np.isfinite(g) & (np.abs(g - r) <= TOL * np.maximum(size, 1.0))
        assert np.all(same | fine), (name, np.argwhere(~(same | fine))[:5])
        assert np.max(size[np.isfinite(size)]) > 1e30 or not np.isfinite(r).all()


@pytest.mark.gpu
@pytest.mark.parametrize("pd", [P(64, 256, 13, 13, 384, 3, 3, 1, 1, 1, 1), P(42, 3, 83, 87, 96, 11, 11, 4, 4),
                                P(1200, 700, 1, 1, 2100, 1, 1)], ids=["image", "folded", "rows"])
def test_recomputed_sums_cost_no_order_of_magnitude(pd):
    """All sums computed again take 1.1 to 3.9 times a pass (one value after the other: 40 to 95 times)."""
    d = conv.conv_desc_create(conv.ConvParams(**pd))
    op, kernels = OracleParams(**pd), names(pd)
    x, w, b, dy = (t.to(DEV) for t in workloads.random_inputs(oracle.x_shape(op), oracle.w_shape(op), oracle.output_shape(op), 79))
    y, dx, dw, db = torch.empty_like(dy), torch.empty_like(x), torch.empty_like(w), torch.empty_like(b)
    ws = torch.empty((conv.conv_desc_workspace_bytes(d) + 7) // 8, device=DEV, dtype=torch.float64)
    nan = float("nan")

    def ms(call):
        call()
        start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        start.record()
        for _ in range(5):
            call()
        end.record()
        torch.cuda.synchronize()
        return start.elapsed_time(end) / 5

    for which, call in (("fwd", lambda x, dy: conv.conv_forward(d, x, w, b, y, ws)),
                        ("bwd_data", lambda x, dy: conv.conv_backward_data(d, w, dy, dx, ws)),
                        ("bwd_filter", lambda x, dy: conv.conv_backward_filter_bias(d, x, dy, dw, db, 0.0, ws))):
        if "split" in kernels[which]:
            plain = ms(lambda: call(x, dy))
            spoilt = ms(lambda: call(torch.full_like(x, nan), torch.full_like(dy, nan)))
            assert spoilt < 10 * plain, (which, plain, spoilt)


@pytest.mark.gpu
@pytest.mark.parametrize("pd", [P(20, 48, 29, 30, 60, 5, 5), P(40, 48, 30, 31, 64, 3, 5), P(42, 3, 83, 87, 96, 11, 11, 4, 4),
                                P(8, 705, 39, 21, 284, 1, 1), P(1200, 700, 1, 1, 2100, 1, 1)],
                         ids=["5x5", "3x5", "folded", "columns", "rows"])
@pytest.mark.parametrize("ex,ew,edy", [(-118, 70, 70), (70, -118, 70), (70, 70, -118), (-136, 70, 70), (70, -136, 70), (70, 70, -136)])
def test_tiny_operands_keep_their_bits(pd, ex, ew, edy):
    """Operands down to fp32's denormals against large ones: the bound of ordinary operands holds, it does not
    know their size.  The filter gradient of two large blobs (2^140) and products of two tiny ones are left out."""
    op = OracleParams(**pd)
    x, w, b, dy = workloads.random_inputs(oracle.x_shape(op), oracle.w_shape(op), oracle.output_shape(op), 78)
    x, w, b, dy = x * 2.0 ** ex, w * 2.0 ** ew, b * 0, dy * 2.0 ** edy
    d, ws, _, (y, dx, dw, db) = run_all(pd, x, w, b, dy)
    kernels, ys = names(pd), oracle.output_shape(op)
    taps = pd["kernel_h"] * pd["kernel_w"]
    checked = 0
    for which, got, e, ref, terms in (
            ("fwd", y, ex + ew, lambda: oracle.forward(op, x.numpy(), w.numpy(), b.numpy()), pd["c"] * taps),
            ("bwd_data", dx, edy + ew, lambda: oracle.backward_data(op, w.numpy(), dy.numpy()), pd["num_output"] * taps),
            ("bwd_filter", dw, ex + edy, lambda: oracle.backward_filter(op, x.numpy(), dy.numpy()), ys[0] * ys[2] * ys[3])):
        if "split" in kernels[which] and -80 < e < 80:
            r = ref()
            assert norm_error(got, r) <= 2.0 ** -24 * np.sqrt(terms / 16 + 32), (which, norm_error(got, r))
            checked += 1
    assert checked or ew > 0


@pytest.mark.gpu
def test_split_passes_in_a_hip_graph():
    """Captured once after an eager step, replayed on other inputs: the eager step's bits each time."""
    pd = P(20, 48, 29, 30, 60, 5, 5)
    assert names(pd)["fwd"].endswith("L=3)") and "split" in names(pd)["bwd_data"] and "split" in names(pd)["bwd_filter"]
    op, d = OracleParams(**pd), conv.conv_desc_create(conv.ConvParams(**pd))
    shapes = (oracle.x_shape(op), oracle.w_shape(op), oracle.output_shape(op))
    x, w, b, dy = (t.to(DEV) for t in workloads.random_inputs(*shapes, 80))
    y, dx, dw, db = torch.empty_like(dy), torch.empty_like(x), torch.empty_like(w), torch.empty_like(b)
    ws = torch.empty((conv.conv_desc_workspace_bytes(d) + 7) // 8, device=DEV, dtype=torch.float64)

    def step():
        conv.conv_forward(d, x, w, b, y, ws)
        conv.conv_backward_data(d, w, dy, dx, ws)
        conv.conv_backward_filter_bias(d, x, dy, dw, db, 0.0, ws)

    step()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for rep in range(3):
        for to, t in zip((x, w, b, dy), workloads.random_inputs(*shapes, 81 + rep)):
            to.copy_(t)
        for t in (y, dx, dw, db):
            t.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        got = [t.clone() for t in (y, dx, dw, db)]
        step()
        torch.cuda.synchronize()
        assert all(torch.equal(a, e) for a, e in zip(got, (y, dx, dw, db)))


@pytest.mark.gpu
@pytest.mark.parametrize("beta", [0.0, 1.0])
@pytest.mark.parametrize("m,k,o", [(333, 1503, 2570), (4100, 333, 965), (999, 1503, 1501), (2500, 1300, 2500)])
def test_inner_product_on_the_column_form(m, k, o, beta):
    """Ragged rows, columns and channels, the forward pass in one slice (2500 rows) and in several, the filter gradient too,
    added to dw or written."""
    assert "corrsplit" in conv.ip_desc_kernel_names(conv.ip_desc_create(conv.IpParams(m=m, k=k, num_output=o, relu=1)))
    x, w, b, dy = workloads.ip_random_inputs(m, k, o, seed=8100 + m)
    dw0, db0 = workloads.draw((o, k), "normal", 8300 + m), workloads.draw((o,), "normal", 8301 + m)
    run_ip_case(m, k, o, True, 1, x, w, b, dy, beta=beta, dw0=dw0, db0=db0)
