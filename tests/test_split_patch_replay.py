"""Every operand read of the split kernels' LDS patches, replayed on the CPU from the descriptors' kernel arguments
(split_patch_replay.cpp): inside the patch, and the position that the definition of the convolution names."""
import ctypes
import os
import random
import subprocess

import pytest

import oracle
import paper_1810_02272_amd as conv
from oracle import OracleParams
from parity_cases import SPLIT_CASES, SPLIT_PAD_CASES, P

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def replay(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("replay") / "split_patch_replay.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_1810_02272_amd", "csrc"), os.path.join(HERE, "split_patch_replay.cpp"), "-o", so],
                   check=True)
    lib = ctypes.CDLL(so)

    def run(pd):
        """pass -> (reads, reads outside the patch, wrong positions), for the passes on the split kernels"""
        d = conv.conv_desc_create(conv.ConvParams(**pd))
        h, found = ctypes.c_void_p(d.handle), {}
        for name, call in (("fwd", lambda o: lib.replay_corr(h, 0, o)), ("bwd_data", lambda o: lib.replay_corr(h, 1, o)),
                           ("bwd_filter", lambda o: lib.replay_wgrad(h, o))):
            out = (ctypes.c_int64 * 3)()
            if call(out) == 1:
                found[name] = tuple(out)
        return found

    return run


def draw(rng):
    """Layers that the rules may take, padding up to three windows (beyond the image and the window) included."""
    kh, kw = rng.choice((1, 2, 3, 3, 5, 7, 11)), rng.choice((1, 2, 3, 3, 5, 7, 11))
    dh, dw = (rng.choice((1, 1, 1, 2, 3)) for _ in range(2))
    group = rng.choice((1, 1, 1, 2))
    h, w = rng.randint(1, 60), rng.randint(1, 60)
    ph, pw = (rng.randint(0, rng.choice((1, 2, 3)) * (1 + d * (k - 1))) for k, d in ((kh, dh), (kw, dw)))
    return P(rng.randint(1, 64), group * rng.choice((3, 3, 16, 45, 64, 128, 256)), h, w, group * rng.choice((24, 32, 77, 96, 128, 384)), kh, kw,
             rng.choice((1, 1, 1, 2, 4)), rng.choice((1, 1, 1, 2, 4)), ph, pw, dh, dw, group)


def check(replay, pd):
    found = replay(pd)
    for name, (reads, out, wrong) in found.items():
        assert reads > 0 and out == 0 and wrong == 0, (pd, name, reads, out, wrong)
    return len(found)


@pytest.mark.parametrize("pd", SPLIT_PAD_CASES, ids=[str(i) for i in range(len(SPLIT_PAD_CASES))])
def test_padding_beyond_the_window(replay, pd):
    assert check(replay, pd) >= 2, "the case does not reach the split kernels"


def test_patches_of_the_parity_cases(replay):
    assert sum(check(replay, pd) for pd in SPLIT_CASES) >= 45


def test_patches_of_drawn_layers(replay):
    rng, passes, beyond = random.Random(5), 0, 0
    while passes < 400:
        pd = draw(rng)
        op = OracleParams(**pd)
        if min(oracle.out_size(pd["h"], pd["kernel_h"], pd["stride_h"], pd["pad_h"], pd["dilation_h"]),
               oracle.out_size(pd["w"], pd["kernel_w"], pd["stride_w"], pd["pad_w"], pd["dilation_w"])) < 1:
            continue
        if pd["n"] * op.c * pd["h"] * pd["w"] > 1 << 24:
            continue
        got = check(replay, pd)
        passes += got
        beyond += got > 0 and pd["pad_h"] > pd["dilation_h"] * (pd["kernel_h"] - 1) + 1
    assert beyond >= 20, beyond
