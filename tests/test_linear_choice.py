"""The kernel that each test of a packed linear layer names in its comments is the one that the dispatch gives its size to: a refit of the
predicted times that moves a test off its tile fails here (wchoice.h on the host; no GPU)."""
import shutil

import pytest

import bench
import test_gpu_k_tails
import test_gpu_linear_epilogue
import test_gpu_linear_parts_choice
import test_gpu_linear_tiles
import test_gpu_ops
from linear_choice import WAVE, choices

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs the compiler")


def rows(test):
    return [tuple(r) for r in test.pytestmark[0].args[1]]


def check(layers, want):
    assert len(layers) == len(want)
    wrong = [(l, got, w) for l, (got, parts), w in zip(layers, choices(layers), want) if (got, parts) != (w, 1)]
    assert not wrong, wrong


def test_layers_of_few_stages():
    check(rows(test_gpu_k_tails.test_linear_of_few_stages),
          ["128x128/2"] * 2 + ["128x192"] * 3 + ["128x96"] + ["64x64"] * 6 + ["128x320"] * 3 + ["256x320", "128x128", WAVE])
    check([(m, c, c, "xa", text) for m, c, text in rows(test_gpu_k_tails.test_cross_attention_of_few_stages)],
          [WAVE] * 3 + ["128x128/2"] + ["128x128"] * 3 + ["64x128/2"] * 3)


def test_layers_of_the_less_common_tiles():
    check(rows(test_gpu_linear_tiles.test_linear_packed_more_tiles),
          ["64x96"] * 2 + ["128x160"] * 2 + ["256x256"] * 2 + ["128x96"] * 2 + ["128x192"] * 2 + ["128x128/2"] * 2)


def test_layers_with_the_epilogue_in_the_accumulators():
    check([(m, n, k, "ln_geglu" if ln else "geglu") for m, n, k, ln in rows(test_gpu_linear_epilogue.test_geglu_in_the_accumulators)],
          ["128x128"] + ["128x320"] * 2 + ["256x320"] * 2 + ["256x256"] + ["128x192"] * 3)


def test_layers_of_the_operation_tests():
    check([(m, n, k, v.replace("_far", "")) for m, n, k, v in rows(test_gpu_ops.test_linear_packed_tiles)],
          ["64x64", "128x96", "128x96", "128x96", "128x128/2", "128x128", "128x128", "64x64/2", "256x320", "128x320", "128x320"])
    check([(b * m, c, c, "xa", text) for b, m, c, text, *_ in rows(test_gpu_ops.test_cross_attn_packed)],
          [WAVE] * 4 + ["64x128/2", "128x128", "128x128", "128x128/2"])


def test_layers_whose_timelines_are_read():
    """`bench.py --timeline` reads stamps that only the wave-level kernel writes."""
    check(bench.TIMELINE_LAYERS, [WAVE] * len(bench.TIMELINE_LAYERS))


def test_parts_of_middle_sizes():
    """Token counts on either side of each change of the number of parts, with scratch for eight."""
    counts = test_gpu_linear_parts_choice.test_linear_packed_parts_of_middle_sizes.pytestmark[0].args[1]
    assert [n for _, n in choices([(m, 1280, 5120, "plain", 8) for m in counts])] == [8, 8, 1, 5, 5, 4, 1, 1, 1]


def test_layers_of_other_widths():
    """Layers that constants from 1280 x 5120 alone sent to a slower kernel or split in parts, and those that they were made for."""
    layers = [(1500, 640, 2560), (2400, 320, 1280), (3000, 320, 2560), (224, 1280, 3840), (288, 960, 3840), (640, 640, 5120),
              (768, 1280, 5120), (494, 1280, 5120), (1024, 1280, 5120)]
    assert choices([(*l, "plain", 8) for l in layers]) == [
        ("64x64", 1), ("64x64", 1), ("64x64", 1), (WAVE, 1), (WAVE, 1), ("128x128", 8), (WAVE, 1), ("128x128", 5), ("128x128", 3)]
    assert choices([(1224, 1280, 1280, "xa", n) for n in (20, 50, 77, 100)]) == [("64x128/2", 1), ("64x128/2", 1), (WAVE, 1), ("64x128/2", 1)]


def test_cross_attention_of_short_k_stays_off_the_deep_ring():
    """128 x 128 with a unit to itself (a ring of four) takes cross-attention only with a K of three stages of 64: the launcher refuses it
    below, and the dispatch never asks."""
    layers = [(m, c, c, "xa", n) for c in (64, 128) for m in (*range(64, 4096, 96), 10000, 40000, 200000) for n in (20, 77, 128)]
    assert "128x128" not in {tile for tile, _ in choices(layers)}
