"""Which kernels a batch takes, where the choice depends on how many searches there are: either side of each line,
with the oracle's results."""
import pytest

from paper_2103_16063_amd import binding as B
from paper_2103_16063_amd import synth
from tests.gpu_util import assert_results_match, oracle_solve_many

pytestmark = pytest.mark.gpu
WIDE = B.WIDE_RECOMPUTE_MAX_TOTAL_TIME


def _chains(Q, sizes, D, comm=False, S=3):
    probs = [synth.random_small(700 + q % 7, sizes[q % len(sizes)], D, S, tight=2.5) for q in range(Q)]
    return [synth.with_cut_bytes(p, q % 7, 1000) for q, p in enumerate(probs)] if comm else probs


def _run(probs, kernel_of, **kw):
    distinct = oracle_solve_many(probs[:7])  # (the chains repeat)
    with B.Session(synth.concat_batch(probs), **kw) as s:
        assert_results_match(probs, s.run(), oracle_results=[distinct[q % 7] for q in range(len(probs))])
        rc, info = B.rannc_dp_solve_info(s.h)
        assert rc == B.OK and kernel_of(info)


# One workgroup to a compute unit (64-bit values at 64 devices, or at 32 with the times recomputed) and more than 64
# blocks: one launch where its rounds are nearly full.
@pytest.mark.parametrize("Q,D,comm,one", [
    (256, 64, True, True), (257, 64, True, False), (479, 64, True, False), (480, 64, True, True),
    (191, 32, False, False), (192, 32, False, True), (300, 32, False, False), (512, 32, False, True),
])
def test_one_launch_of_many_searches_in_full_rounds(Q, D, comm, one):
    kernel = (B.KERNEL_ONE_LAUNCH if comm else B.KERNEL_ONE_LAUNCH_RECOMPUTE) if one else \
        (B.KERNEL_MERGE_TABLE if comm else B.KERNEL_MERGE_RECOMPUTE)
    cls = {32: 2, 64: 3}[D]
    _run(_chains(Q, [66, 65, 70, 68, 66, 67, 72], D, comm), lambda info: info.level_kernel[cls] == kernel,
         max_total_time_ns=WIDE)


# Fewer searches than make a batch: one launch where the launches per level would take longer, which they do with every
# further search (not beside another class).
@pytest.mark.parametrize("Q,N,D,beside,one", [
    (34, 128, 8, False, False), (35, 128, 8, False, True), (8, 80, 16, False, False), (16, 80, 16, False, True),
    (35, 128, 8, True, False),
])
def test_one_launch_of_some_tens_of_searches(Q, N, D, beside, one):
    probs = _chains(Q, [N, N - 1, N - 15, 66, N, 70, N], D, S=8)
    if beside:
        probs = probs[:7] * 5 + [synth.random_small(3, 40, 64, 8, tight=2.5)] * 40
    kernel = B.KERNEL_ONE_LAUNCH_RECOMPUTE if one else B.KERNEL_MERGE_RECOMPUTE
    cls = {8: 0, 16: 1}[D]
    if not beside:
        _run(probs, lambda info: info.level_kernel[cls] == kernel)
        return
    with B.Session(synth.concat_batch(probs)) as s:
        res = s.run()
        distinct = oracle_solve_many(probs[:7] + probs[-1:])
        assert_results_match(probs, res, oracle_results=[distinct[q % 7] for q in range(35)] + [distinct[7]] * 40)
        rc, info = B.rannc_dp_solve_info(s.h)
        assert rc == B.OK and info.level_kernel[cls] != B.KERNEL_ONE_LAUNCH_RECOMPUTE
