"""Prefix sums of the one-launch kernel (two blocks per lane of one wave) at the edges of lanes and of the
range, with sums one below the limit of 2^62 and at it, the excess in the last block."""
import numpy as np
import pytest

from paper_2103_16063_amd import binding as B
from paper_2103_16063_amd import synth
from tests.gpu_util import assert_results_match

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1, 2, 3, 63, 64, 65, 127, 128])
def test_sums_at_the_edges(N):
    good = synth.random_small(900 + N, N, 4, 3, tight=50.0)
    below, at, negative = dict(good), dict(good), dict(good)
    below["param_bytes"] = good["param_bytes"].copy()
    below["param_bytes"][N - 1] = (1 << 62) - 1 - int(good["param_bytes"][:N - 1].sum())
    at["param_bytes"] = below["param_bytes"].copy()
    at["param_bytes"][N - 1] += 1
    negative["time_ns"] = good["time_ns"].copy()
    negative["time_ns"][N - 1] = -1
    with B.Session(synth.concat_batch([good, below, at, negative]), one_launch_small=2) as s:
        res = s.run()
    assert_results_match([good], {k: v[:1] for k, v in res.items()})
    assert list(res["status"]) == [B.PROBLEM_OK, B.PROBLEM_OK, B.PROBLEM_SUM_OVERFLOW, B.PROBLEM_NEGATIVE_INPUT]
    assert int(res["n_stages"][1]) == 0   # its last block fits nowhere
