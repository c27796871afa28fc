"""Every patch read of the folded filter gradient, replayed on the CPU from the descriptors' arguments (split_fold_replay.cpp)."""
import ctypes
import os
import random
import subprocess

import paper_1810_02272_amd as conv
from parity_cases import FOLD_CASES, P

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def draw(rng):
    kh, g = rng.choice((4, 5, 7, 8, 11, 12)), rng.choice((1, 1, 2))
    return P(rng.randint(8, 128), g * rng.randint(1, 11), rng.randint(20, 227), rng.randint(20, 227), g * rng.randint(16, 200), kh,
             rng.choice((kh, 11, 8, 4)), rng.choice((4, 4, 1, 2, 3)), rng.choice((4, 4, 8)), rng.randint(0, 5), rng.choice((0, 4)), 1, 1, g)


def test_patches_of_folded_filter_gradients(tmp_path):
    so = str(tmp_path / "split_fold_replay.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_1810_02272_amd", "csrc"), os.path.join(HERE, "split_fold_replay.cpp"), "-o", so], check=True)
    lib, rng, passes, cases = ctypes.CDLL(so), random.Random(6), 0, list(FOLD_CASES)
    while passes < 120:
        pd = cases.pop() if cases else draw(rng)
        if pd["h"] + 2 * pd["pad_h"] < pd["kernel_h"] or pd["w"] + 2 * pd["pad_w"] < pd["kernel_w"]:
            continue
        d, out = conv.conv_desc_create(conv.ConvParams(**pd)), (ctypes.c_int64 * 3)()
        if lib.replay_fold(ctypes.c_void_p(d.handle), out) == 1:
            assert out[0] > 0 and out[1] == 0 and out[2] == 0, (pd, list(out))
            passes += 1
