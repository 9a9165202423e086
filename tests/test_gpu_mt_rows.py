"""MT19937 plain rows, one stream per wavefront and (fp64, and many long rows)
one per workgroup: draw counts around the block of 624 from every position the
calls before leave, stream counts that leave a workgroup ragged; bit-exact with
the oracle."""
import numpy as np
import pytest

from paper_1003_1898_amd import inputs
from paper_1003_1898_amd.generator import Generator

from mirror import bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 6, 131])
@pytest.mark.parametrize("dt", ["u32", "f32", "f32_paper", "f64"])
def test_mt_rows(oracle, n, dt):
    print(f"\n[mt rows] n={n} {dt}", flush=True)
    seeds = inputs.seed_words("mt19937", 624, n)
    g = Generator("mt19937", n, seed_words=seeds)
    st = oracle.init("mt19937", seeds)
    for count in (624, 1, 623, 625, 1248, 1247, 63, 64, 65, 1249, 5000):
        got = bits(g.generate(count, dt).cpu().numpy())
        assert np.array_equal(got, bits(oracle.generate("mt19937", st, count, dt, threads=8))), f"count={count}"
        assert np.array_equal(g.state_words(), st), f"state after count={count}"


def test_mt_long_rows_of_many_streams(oracle):
    print("\n[mt rows] many", flush=True)
    n = 32769
    seeds = inputs.seed_words("mt19937", 625, n)
    g = Generator("mt19937", n, seed_words=seeds)
    st = oracle.init("mt19937", seeds)
    for count in (700, 4097):  # per wavefront, then per workgroup
        got = g.generate(count, "f32").cpu().numpy()
        assert np.array_equal(bits(got), bits(oracle.generate("mt19937", st, count, "f32", threads=8))), count
        assert np.array_equal(g.state_words(), st), count
