"""RANMAR with one stream per wavefront (256 positions per emitted block, steps
of 64, a window kept in a ring of 512): draw counts around a step, a block, the
ring and the window of 97, stream counts that do not fill a workgroup, rows
that start at every alignment, every dtype; bit-exact with the oracle."""
import numpy as np
import pytest

from paper_1003_1898_amd import inputs
from paper_1003_1898_amd.generator import Generator

from mirror import bits

pytestmark = pytest.mark.gpu

COUNTS = [1, 2, 3, 33, 63, 64, 65, 96, 97, 98, 129, 130, 131, 191, 255, 256, 257, 319, 511, 512, 513, 767, 769,
          1023, 1025, 4099]


@pytest.mark.parametrize("n", [1, 6, 37])
@pytest.mark.parametrize("dt", ["u32", "f32", "f64", "f32_paper"])
def test_ranmar_rows(oracle, n, dt):
    print(f"\n[ranmar wave] n={n} {dt}", flush=True)
    seeds = inputs.seed_words("ranmar", 97, n)
    g = Generator("ranmar", n, seed_words=seeds)
    st = oracle.init("ranmar", seeds)
    for count in COUNTS:
        got = bits(g.generate(count, dt).cpu().numpy())
        assert np.array_equal(got, bits(oracle.generate("ranmar", st, count, dt))), f"count={count}"
        assert np.array_equal(g.state_words(), st), f"state after count={count}"


def test_ranmar_packed(oracle):
    print("\n[ranmar wave packed]", flush=True)
    n = 8
    seeds = inputs.seed_words("ranmar", 98, n)
    g = Generator("ranmar", n, seed_words=seeds)
    st = oracle.init("ranmar", seeds)
    for count in COUNTS:
        got = g.generate_packed4(count, "f32").cpu().numpy().transpose(0, 2, 1).reshape(n, count)
        assert np.array_equal(bits(got), bits(oracle.generate("ranmar", st, count, "f32"))), f"count={count}"
        assert np.array_equal(g.state_words(), st), f"state after count={count}"


@pytest.mark.parametrize("n", [4097, 49153])
def test_ranmar_many_streams(oracle, n):
    """Two streams per wavefront with a ragged last workgroup, and the lane kernel
    from three quarters of the SIMDs on."""
    print(f"\n[ranmar many] n={n}", flush=True)
    seeds = inputs.seed_words("ranmar", 99, n)
    g = Generator("ranmar", n, seed_words=seeds)
    st = oracle.init("ranmar", seeds)
    for count, dt in ((37, "u32"), (515, "f32")):
        got = bits(g.generate(count, dt).cpu().numpy())
        assert np.array_equal(got, bits(oracle.generate("ranmar", st, count, dt, threads=8))), f"count={count}"
        assert np.array_equal(g.state_words(), st), f"state after count={count}"
