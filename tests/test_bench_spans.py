"""What bench.py takes the stamped Top-K span to be: the whole iteration end where
the library pipelines it, else the worker compression alone."""
import os
import re

import pytest

from paper_2008_05823_amd import workloads as W

CSRC = os.path.join(os.path.dirname(os.path.abspath(W.__file__)), "csrc")


def _n_tiles(w, tile=2048):
    return sum(-(-int(n) // tile) for n in w.sizes)


@pytest.mark.parametrize("name,pipelined", [("flat64k", False), ("resnet56", False),
                                            ("resnet50", True), ("bert_base", True),
                                            ("flat256m", False)])
def test_span_of_a_workload(name, pipelined):
    w = W.get(name)
    assert W.topk_pipelined(w.L, _n_tiles(w), w.K) == pipelined
    b = W.topk_algorithmic_bytes_per_param(w.K, 0.05, 1)
    span = W.topk_span_bytes_per_param(w.K, 0.05, 1, pipelined)
    assert span == pytest.approx(b["worker"] + (b["server"] if pipelined else 0))
    mom = W.topk_span_bytes_per_param(w.K, 0.05, 1, pipelined, True)
    assert mom == pytest.approx(span + 8 * w.K)


def test_the_rule_is_the_library_s():
    text = open(os.path.join(CSRC, "saef_topk.h")).read()
    assert int(re.search(r"kTkSplitTiles = (\d+);", text).group(1)) == W.TOPK_SPLIT_TILES
    assert "#define SAEF_TILE_ELEMS 2048" in open(os.path.join(CSRC, "saef_internal.h")).read()


def test_bench_uses_it():
    root = os.path.dirname(os.path.dirname(CSRC))
    text = open(os.path.join(root, "bench.py")).read()
    assert "W.topk_pipelined(" in text and 'prof["aggregate"]' not in text
