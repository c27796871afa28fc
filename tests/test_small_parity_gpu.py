"""GPU parity of the one-launch kernels of small layers (corr_small_kernel, wgrad_small_kernel) in both base types, at sizes
that end inside a tile, a group of reduction indices, a run of four pixels and a slice, with every way of reading the weights.

Tolerances are those of the sweeps (test_parity_gpu.py, test_f64_parity_gpu.py): the same sums in another order."""
import re

import pytest
import torch

import paper_1810_02272_amd as conv
from paper_1810_02272_amd import workloads
import oracle
from oracle import OracleParams
from parity_cases import P
from test_f64_parity_gpu import check_full64, widen
from test_parity_gpu import check_full

DEV = "cuda:0"
NAN = float("nan")

CASES = [
    P(23, 180, 33, 29, 102, 1, 1, 1, 1, 0, 0, 1, 1, 3),
    P(23, 136, 5, 8, 58, 7, 7, 3, 1, 7, 0, 1, 1, 2),
    P(51, 8, 45, 49, 70, 3, 3, 3, 3, 2, 3, 1, 1, 2),
    P(7, 21, 48, 46, 93, 1, 1, 1, 1, 0, 0, 2, 2, 1),
    P(5, 12, 22, 23, 57, 7, 7, 1, 1, 0, 5, 1, 1, 3),
    P(20, 63, 10, 5, 90, 7, 5, 2, 2, 3, 0, 1, 1, 1),
    P(29, 68, 38, 40, 5, 1, 1, 1, 1, 0, 0, 1, 1, 1),
    P(5, 44, 36, 33, 53, 1, 1, 1, 1, 0, 1, 1, 1, 1),
    P(24, 4, 24, 20, 34, 5, 5, 1, 1, 3, 1, 2, 2, 2),
    P(2, 44, 9, 4, 18, 7, 7, 1, 1, 5, 7, 1, 1, 1),
    P(33, 9, 17, 22, 276, 1, 1, 1, 1, 0, 0, 1, 1, 3),
    P(33, 4, 23, 26, 92, 4, 4, 3, 3, 3, 2, 1, 1, 2),
    P(16, 6, 15, 20, 33, 4, 2, 1, 1, 2, 0, 1, 1, 1),
    P(29, 6, 26, 28, 7, 5, 2, 1, 1, 1, 1, 2, 2, 1),
    P(7, 2, 44, 48, 12, 7, 7, 1, 1, 5, 1, 2, 2, 2),
    P(1, 78, 39, 42, 49, 1, 1, 1, 1, 0, 0, 1, 1, 1),
    P(29, 36, 17, 12, 6, 7, 7, 2, 2, 4, 1, 1, 1, 2),
    P(10, 17, 48, 44, 37, 3, 1, 3, 3, 3, 1, 1, 1, 1),
    P(12, 39, 22, 18, 3, 4, 4, 1, 1, 1, 0, 2, 2, 1),
    P(11, 102, 5, 4, 6, 7, 7, 1, 1, 7, 7, 2, 2, 3),
    P(3, 33, 30, 32, 3, 4, 4, 1, 1, 1, 0, 1, 1, 1),
    P(23, 18, 9, 7, 348, 1, 1, 1, 1, 0, 0, 1, 1, 3),
    P(2, 57, 19, 18, 162, 1, 1, 1, 1, 1, 0, 1, 1, 3),
    P(39, 12, 33, 36, 1, 1, 3, 1, 1, 1, 3, 1, 1, 1),
    P(18, 33, 51, 53, 1, 3, 3, 3, 3, 2, 2, 1, 1, 1),
    P(31, 1, 24, 19, 145, 1, 1, 1, 2, 1, 1, 1, 1, 1),
    P(16, 1, 60, 65, 33, 1, 1, 2, 1, 1, 1, 1, 1, 1),
    P(51, 100, 7, 11, 4, 7, 7, 1, 1, 3, 1, 2, 2, 2),
    P(18, 34, 7, 12, 2, 7, 7, 1, 1, 3, 3, 2, 2, 1),
    P(1, 18, 5, 7, 270, 1, 2, 1, 1, 0, 1, 1, 1, 2),
    P(1, 1, 9, 8, 36, 3, 3, 1, 2, 1, 0, 1, 1, 1),
    P(2, 1, 4, 4, 82, 1, 1, 1, 1, 0, 0, 1, 1, 1),
    P(5, 2, 5, 4, 8, 5, 5, 2, 2, 0, 1, 1, 1, 1),
    P(4, 3, 8, 4, 1, 4, 4, 1, 1, 1, 2, 2, 2, 1),
    P(1, 7, 5, 8, 1, 1, 2, 1, 1, 1, 0, 1, 1, 1),
    P(2, 1, 8, 4, 1, 1, 1, 1, 1, 0, 0, 1, 1, 1),
    # without padding, and runs cut at the ends of rows
    P(38, 144, 27, 26, 118, 1, 1, 1, 1, 0, 0, 1, 1, 2),
    P(12, 5, 69, 69, 39, 3, 3, 1, 1, 0, 0, 1, 1, 1),
    P(7, 18, 40, 44, 249, 1, 5, 1, 1, 0, 0, 2, 2, 3),
    P(13, 76, 15, 17, 42, 7, 7, 2, 2, 0, 0, 1, 1, 1),
    P(13, 66, 7, 11, 142, 5, 5, 1, 1, 0, 0, 1, 1, 2),
    P(18, 210, 28, 25, 195, 1, 1, 3, 2, 0, 0, 1, 1, 3),
    P(3, 156, 28, 23, 80, 1, 2, 1, 1, 1, 1, 1, 1, 2),
    P(25, 134, 8, 9, 80, 4, 4, 3, 1, 0, 0, 1, 1, 2),
    P(31, 174, 5, 4, 57, 5, 5, 1, 1, 0, 5, 1, 1, 3),
    P(8, 54, 55, 55, 51, 1, 1, 1, 1, 1, 0, 1, 1, 3),
    P(2, 27, 26, 31, 123, 7, 7, 3, 3, 0, 0, 1, 1, 1),
    P(23, 177, 6, 5, 288, 2, 1, 1, 1, 0, 0, 1, 1, 3),
    P(16, 98, 23, 20, 52, 1, 1, 1, 1, 0, 0, 1, 1, 2),
    P(2, 26, 67, 68, 19, 5, 5, 3, 2, 0, 0, 1, 1, 1),
    P(51, 1, 50, 46, 61, 2, 1, 1, 1, 0, 0, 1, 1, 1),
    P(1, 68, 16, 20, 84, 5, 2, 1, 1, 0, 0, 1, 1, 1),
    P(3, 180, 6, 5, 57, 5, 5, 1, 1, 2, 3, 1, 1, 3),
    P(3, 69, 23, 24, 36, 1, 2, 1, 1, 1, 1, 2, 2, 1),
    P(5, 150, 13, 11, 78, 3, 3, 2, 2, 0, 0, 1, 1, 2),
    P(9, 234, 7, 11, 21, 5, 5, 1, 1, 0, 0, 1, 1, 3),
    P(3, 7, 46, 43, 95, 1, 2, 1, 1, 0, 0, 1, 1, 1),
    P(20, 18, 48, 46, 6, 1, 3, 2, 1, 0, 0, 1, 1, 1),
    P(1, 68, 38, 33, 34, 1, 2, 1, 1, 1, 1, 2, 2, 1),
    P(18, 42, 11, 8, 36, 7, 7, 2, 2, 3, 0, 1, 1, 2),
    P(2, 26, 53, 51, 3, 5, 2, 1, 1, 0, 0, 1, 1, 1),
    P(5, 201, 43, 44, 6, 2, 2, 2, 2, 0, 0, 1, 1, 3),
    P(5, 65, 53, 55, 1, 2, 2, 1, 1, 0, 0, 1, 1, 1),
    P(17, 3, 61, 62, 90, 1, 2, 2, 2, 0, 0, 1, 1, 3),
    P(32, 13, 20, 15, 1, 7, 7, 1, 2, 0, 5, 1, 1, 1),
    P(14, 1, 65, 64, 47, 1, 1, 1, 1, 1, 0, 1, 1, 1),
    P(1, 112, 9, 10, 4, 7, 7, 1, 1, 6, 6, 1, 1, 2),
    P(2, 1, 6, 4, 134, 1, 1, 1, 1, 0, 1, 1, 1, 1),
    P(2, 1, 4, 4, 63, 2, 1, 1, 1, 0, 1, 1, 1, 1),
    P(4, 73, 10, 5, 1, 1, 1, 3, 3, 0, 0, 1, 1, 1),
    P(1, 5, 4, 9, 4, 1, 1, 1, 1, 0, 1, 2, 2, 1),
    P(5, 1, 5, 10, 1, 1, 1, 2, 2, 0, 0, 1, 1, 1),
]


def small_variants(pd):
    d = conv.conv_desc_create(conv.ConvParams(**pd))
    out = set()
    for names in (conv.conv_desc_kernel_names(d), conv.conv_desc_kernel_names_f64(d)):
        for field in names.split(";"):
            which, v = field.split("=", 1)
            if "small" in v:
                name, rest = v.split("(", 1)
                out.add((name, not rest.startswith("S=1,")))
    return out


def test_cases_reach_every_variant():
    """Every tile x way of reading (forward w0; backward data w1 single loads, w2 with a test of the tap, w3 16-byte loads),
    the filter gradient with one slice and several, with single (v0) and 16-byte (v1) loads of x."""
    have = set().union(*(small_variants(pd) for pd in CASES))
    tiles = ["16x16x4", "16x16x8", "32x16x4", "16x32x4", "32x32x4", "48x16x4"]
    want = {(f"corrsmall{b}_{t}[w{m}]", False) for b in ("", "64") for t in tiles for m in range(4)}
    want |= {(f"corrsmall_48x32x4[w{m}]", False) for m in range(4)}
    for b, tiles in (("", ["16x16x8", "16x32x8", "32x16x8", "32x32x8", "32x32x4"]), ("64", ["16x16x8", "16x32x8", "32x16x8", "32x32x4"])):
        want |= {(f"smallwgrad{b}_{t}[v0]", s) for t in tiles for s in (False, True)}
        want |= {(f"smallwgrad{b}_16x16x8[v1]", s) for s in (False, True)} | {(f"smallwgrad{b}_{t}[v1]", True) for t in tiles if (b, t) != ("", "32x32x4")}
    want |= {(f"smallwgrad_{t}[v2]", s) for t in ("16x16x8", "16x32x8", "32x16x8", "32x32x8", "32x32x4") for s in (False, True)}
    assert want <= have, sorted(want - have)


def test_cases_reach_both_sides_of_padding():
    """Instances without bounds tests and with them (backward data of one tap has none, of two always)."""
    padded, plain = set(), set()
    for pd in CASES:
        for v in small_variants(pd):
            if "[w1]" in v[0]:
                (padded if pd["kernel_h"] * pd["kernel_w"] > 1 else plain).add(v)
            elif re.search(r"\[(w0|v0|v2)\]", v[0]):
                (padded if pd["pad_h"] or pd["pad_w"] else plain).add(v)
    # one tap a channel and eight waves a tile do not meet in backward data of floats; the same for one slice of this tile
    assert padded - plain <= {("corrsmall_16x16x8[w1]", False), ("smallwgrad_32x32x4[v2]", False)}, sorted(padded - plain)
    assert plain <= padded, sorted(plain - padded)


@pytest.mark.gpu
@pytest.mark.parametrize("i", range(len(CASES)))
def test_small_layers_against_the_oracle(i):
    pd = CASES[i]
    print("small case", i, pd, small_variants(pd), flush=True)
    check_full(pd, seed=91000 + 10 * i)
    op = OracleParams(**pd)
    x, w, b, dy = (widen(t, 92000 + 10 * i + j) for j, t in enumerate(
        workloads.random_inputs(oracle.x_shape(op), oracle.w_shape(op), oracle.output_shape(op), 91000 + 10 * i)))
    check_full64(pd, x, w, b, dy)


@pytest.mark.gpu
@pytest.mark.parametrize("pad", [1, 0])
@pytest.mark.parametrize("f64", [False, True])
def test_what_lies_behind_a_row_does_not_leak(f64, pad):
    """NaN in one output channel's weights, one input channel's, one channel of dy and of x: the wide loads run past a row's
    reduction, a channel's taps and an image's last pixels, and only the results that own a NaN may show it."""
    pd = P(3, 6, 15, 15, 40, 3, 3, 1, 1, pad, pad)  # 54 indices forward (10 past them), nine taps, rows of 15 or 13 pixels
    o = 13 + 2 * pad
    d = conv.conv_desc_create(conv.ConvParams(**pd))
    assert len(small_variants(pd)) >= 5 and ("smallwgrad_16x16x8[v2]", False) in small_variants(pd), small_variants(pd)
    dt = torch.float64 if f64 else torch.float32
    size = conv.conv_desc_workspace_bytes_f64(d) if f64 else conv.conv_desc_workspace_bytes(d)
    gen = torch.Generator().manual_seed(5)
    x, w, b, dy = (torch.randn(s, generator=gen, dtype=torch.float64).to(DEV, dt) for s in ((3, 6, 15, 15), (40, 6, 3, 3), (40,), (3, 40, o, o)))
    ws = torch.full((size // 8 + 1,), NAN, device=DEV, dtype=torch.float64)
    f, bd, bf = ((conv.conv_forward_f64, conv.conv_backward_data_f64, conv.conv_backward_filter_f64) if f64 else
                 (conv.conv_forward, conv.conv_backward_data, conv.conv_backward_filter))
    y, dx, dw, db = torch.empty_like(dy), torch.empty_like(x), torch.empty_like(w), torch.empty_like(b)
    bad = w.clone()
    bad[17] = NAN
    f(d, x, bad, b, y, ws)
    assert y[:, 17].isnan().all() and not y[:, [k for k in range(40) if k != 17]].isnan().any()
    bad = w.clone()
    bad[:, 3] = NAN
    bd(d, bad, dy, dx, ws)
    assert dx[:, 3].isnan().all() and not dx[:, [0, 1, 2, 4, 5]].isnan().any()
    bad = dy.clone()
    bad[:, 17] = NAN
    bf(d, x, bad, dw, 0.0, ws)
    assert dw[17].isnan().all() and not dw[[k for k in range(40) if k != 17]].isnan().any()
    if not f64:
        conv.conv_backward_filter_bias(d, x, bad, dw, db, 0.0, ws)
        assert db[17].isnan() and int(db.isnan().sum()) == 1
    bad = x.clone()
    bad[:, 3] = NAN
    bf(d, bad, dy, dw, 0.0, ws)
    assert dw[:, 3].isnan().all() and not dw[:, [0, 1, 2, 4, 5]].isnan().any()


@pytest.mark.gpu
def test_small_kernels_in_a_hip_graph():
    """Three passes of two layers captured, replayed with other work in between: every replay equals the eager results."""
    runs = []
    for j, pd in enumerate((P(4, 12, 14, 15, 24, 5, 5, 1, 1, 2, 2), P(9, 20, 17, 17, 18, 3, 3, 2, 2, 1, 1))):
        assert len(small_variants(pd)) >= 3, small_variants(pd)
        d = conv.conv_desc_create(conv.ConvParams(**pd))
        op = OracleParams(**pd)
        x, w, b, dy = (t.to(DEV) for t in workloads.random_inputs(oracle.x_shape(op), oracle.w_shape(op), oracle.output_shape(op), 93000 + j))
        ws = torch.zeros(conv.conv_desc_workspace_bytes(d) // 4 + 1, device=DEV)
        out = [torch.empty_like(t) for t in (dy, x, w, b)]

        def run(d=d, x=x, w=w, b=b, dy=dy, ws=ws, out=out):
            conv.conv_forward(d, x, w, b, out[0], ws)
            conv.conv_backward_data(d, w, dy, out[1], ws)
            conv.conv_backward_filter_bias(d, x, dy, out[2], out[3], 0.0, ws)

        run()
        torch.cuda.synchronize()
        runs.append((run, out, [t.clone() for t in out]))
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for run, _, _ in runs:
            run()
    for _ in range(4):
        for _, out, _ in runs:
            for t in out:
                t.fill_(NAN)
        g.replay()
        torch.cuda.synchronize()
        for _, out, ref in runs:
            assert all(torch.equal(a, r) for a, r in zip(out, ref))
        runs[0][0]()
        torch.cuda.synchronize()
