"""A tile's coordinates split over workgroups: every remainder of the batches in which the chunks' shares are summed, and the
comparators' predictions that come with the Gram matrices (at most sixteen runs, one segment) against those of their own kernel
(seventeen runs).  Against the float64 reference through the C ABI, tolerances as in the other parity tests."""
import re

import pytest

from paper_2603_12617_amd import workloads as WL
from test_gpu_parity import _check, _gpu

pytestmark = pytest.mark.gpu


# chunks: 2, 6, 7, 9 = 8 + 1, 11 = 8 + 3, 15, 20 = 16 + 4, 29 = 16 + 8 + 5; 19 tiles, 12 chunks each, which leave the runs' compute units; 128 chunks (a wavefront has four blocks)
@pytest.mark.parametrize("d,R,K,chunks", [
    (132, 16, 1, 2), (708, 1, 3, 6), (772, 17, 1, 7), (1056, 16, 2, 9), (1300, 2, 5, 11), (1804, 16, 1, 15), (2440, 17, 2, 20), (3588, 3, 5, 29),
    (1800, 19, 16, 12), (65536, 2, 8, 128),
])
@pytest.mark.parametrize("optimistic", [0, 1])
def test_any_number_of_chunks_matches_the_oracle(d, R, K, chunks, optimistic, capfd):
    wl = WL.make("c3", T=141, R=R, d=d, K=K, seg_len=141, optimistic=optimistic)
    data = WL.generate(wl)
    print("case split", d, R, K, "optimistic", optimistic, flush=True)
    capfd.readouterr()
    got = _gpu(wl, data, options=dict(window_resident=5, verbose=1))
    assert re.search(r"\b%d chunks of coordinates" % chunks, capfd.readouterr().err)
    _check(wl, data, got, runs=sorted({0, R // 2, R - 1}), label="split d=%d R=%d K=%d optimistic=%d" % (d, R, K, optimistic))
