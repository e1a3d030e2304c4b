"""The time-split rules (splits.h), compiled for the host: the scratch of a
run's partial images stays bounded however long the run is."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))

# N, channels, workgroups of one split, frames a workgroup images at once
SHAPES = [(16, 3, 3, 64), (32, 75, 75, 24), (64, 128, 128, 8), (64, 1, 1, 8), (64, 128, 128, 4), (128, 512, 512, 2),
          (128, 64, 64, 2), (256, 512, 2048, 2), (256, 64, 128, 1), (256, 1, 4, 2), (128, 5000, 5000, 2)]
LENGTHS = [1, 7, 250, 2000, 10 ** 4, 10 ** 5, 2 * 10 ** 5, 10 ** 6, 10 ** 8]


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("splits") / "splits_check")
    csrc = os.path.join(os.path.dirname(HERE), "paper_1603_02126_amd", "csrc")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I", csrc,
                    os.path.join(HERE, "host_splits", "splits_check.cpp"), "-o", exe], check=True, timeout=120)

    def run(cases):
        text = "\n".join(" ".join(str(v) for v in c) for c in cases)
        r = subprocess.run([exe], input=text, capture_output=True, text=True, check=True, timeout=60)
        out = [tuple(int(v) for v in line.split()) for line in r.stdout.splitlines()]
        assert len(out) == len(cases)
        return out
    run.exe = exe
    return run


@pytest.mark.parametrize("fused", [0, 1])
def test_partial_images_are_bounded(rule, fused):
    cases = [(*s, fused, 0.05, T) for s in SHAPES for T in LENGTHS]
    for c, (splits, size) in zip(cases, rule(cases)):
        n, f, units, slots, _, _, T = c
        assert 1 <= splits <= T
        # 12 rounds of 256 workgroups, each with its tile of the image
        assert size <= max(4 * n * n * f, -(-3072 // units) * 4 * n * n * f), c
        assert size <= 4 * n * n * (f + 3072), c
    # past the bound the run's length does not matter
    for s in SHAPES:
        a, b = rule([(*s, fused, 0.05, 10 ** 7), (*s, fused, 0.05, 10 ** 8)])
        assert a[1] <= 2 * b[1] + 4 * s[0] ** 2 * s[1] and b[1] <= 2 * a[1] + 4 * s[0] ** 2 * s[1]


def test_long_run_shapes(rule):
    """The shapes whose partial images had grown with the run: one million
    samples of the LWA shape, 2e5 of 512 channels at 128 x 128, 1e6 of 512
    channels at 256 x 256."""
    sizes = [b for _, b in rule([(64, 128, 128, 8, 1, 0.043, 10 ** 6), (128, 512, 512, 2, 0, 0, 2 * 10 ** 5),
                                 (256, 512, 2048, 2, 0, 0, 10 ** 6)])]
    assert sizes[0] <= 0.06e9 and sizes[1] <= 0.25e9 and sizes[2] <= 0.3e9


def test_short_runs_keep_the_rounding_of_the_image(rule):
    """Rounding of T frames in n FP32 accumulators per pixel, sqrt(T / 3) / n:
    no more than the rule by workgroups gave (16 splits at 256 x 256, one frame
    at a time; four of eight waves at 64 x 64), or half of one rounding."""
    (dense, _), (pair, _), (cls, _) = rule([(256, 64, 128, 1, 0, 0, 250), (64, 128, 128, 8, 0, 0, 2500),
                                            (128, 64, 64, 2, 0, 0, 250)])
    assert dense >= 16
    assert (2500 / 3) ** 0.5 / (8 * pair) <= (2500 / 3 / 32 ** 2 + 8 / 3 / 4) ** 0.5
    assert (250 / 3) ** 0.5 / (2 * cls) <= 0.5


@pytest.mark.parametrize("lengths,worked", [(1, 1), (2, 2), (8, 8), (9, 1000)])
def test_alternating_run_lengths_are_worked_out_once(rule, lengths, worked):
    r = subprocess.run([rule.exe, str(lengths)], capture_output=True, text=True, check=True, timeout=60)
    assert int(r.stdout) == worked
