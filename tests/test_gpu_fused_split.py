"""In-kernel consumer with the streams cut across lanes: draw counts around a
lane's segment, a chunk of 16 and a wavefront, stream counts at which one, four
or sixteen wavefronts share a stream and at which a lane keeps a whole stream;
sums, histograms and final states equal to the oracle's."""
import numpy as np
import pytest

from paper_1003_1898_amd import inputs
from paper_1003_1898_amd.generator import Generator

pytestmark = pytest.mark.gpu

KINDS = ["ggl", "xor128", "ranecu", "ranmar", "drand48", "rannyu"]
# stream count, draws of successive calls
CALLS = [(1, (1, 63, 64, 65, 1024, 16385, 100003)),
         (5, (2, 15, 16, 17, 1000, 1025, 70001)),
         (300, (31, 129, 2047, 5000)),
         (4099, (100, 4097)),
         (70001, (1, 50))]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n,calls", CALLS)
def test_fused_cut_streams(oracle, kind, n, calls):
    print(f"\n[fused cut] {kind} n={n}", flush=True)
    seeds = inputs.seed_words(kind, 5150, n)
    g = Generator(kind, n, seed_words=seeds)
    st = oracle.init(kind, seeds)
    for draws in calls:
        s, h = g.fused_sum_hist(draws)
        rs, rh = oracle.fused(kind, st, draws, threads=8)
        assert np.array_equal(s.cpu().numpy(), rs), f"draws {draws}"
        assert np.array_equal(h.cpu().numpy(), rh), f"draws {draws}"
        assert np.array_equal(g.state_words(), st), f"draws {draws}"
