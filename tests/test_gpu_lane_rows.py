"""Kernels that only many streams reach, at stream and draw counts that leave
wavefronts, chunks of 128 draws and blocks ragged, several calls in a row: RANMAR
by one lane per stream (plain and interleaved) and MT19937 rows of one workgroup
per stream, every dtype, and interleaved RANECU of a few draws; bit-exact with the oracle."""
import numpy as np
import pytest

from paper_1003_1898_amd import inputs
from paper_1003_1898_amd.generator import Generator

from mirror import bits

pytestmark = pytest.mark.gpu

N = 49156  # fills three quarters of the SIMDs, not a multiple of 64


def _new(oracle, kind, n):
    print(f"\n[lane rows] {kind} n={n}", flush=True)
    seeds = inputs.seed_words(kind, 80, n)
    return Generator(kind, n, seed_words=seeds), oracle.init(kind, seeds)


def test_ranmar_rows_of_lanes(oracle):
    g, st = _new(oracle, "ranmar", N)
    for count, dt in ((127, "f32_paper"), (65, "f64"), (129, "u32"), (128, "f64"), (255, "f32_paper"), (1, "f64")):
        got = bits(g.generate(count, dt).cpu().numpy())
        assert np.array_equal(got, bits(oracle.generate("ranmar", st, count, dt, threads=8))), f"{count} {dt}"
        assert np.array_equal(g.state_words(), st), f"state after {count} {dt}"


def test_ranmar_interleaved_rows_of_lanes(oracle):
    g, st = _new(oracle, "ranmar", N)
    for count, dt in ((127, "u32"), (129, "f32"), (128, "f32_paper"), (255, "f32_paper"), (1, "u32"), (256, "f32")):
        got = g.generate_packed4(count, dt).cpu().numpy().transpose(0, 2, 1).reshape(N, count)
        assert np.array_equal(bits(got), bits(oracle.generate("ranmar", st, count, dt, threads=8))), f"{count} {dt}"
        assert np.array_equal(g.state_words(), st), f"state after {count} {dt}"


@pytest.mark.parametrize("n", [57348, 65536])
def test_ranecu_interleaved_rows_of_few_draws(oracle, n):
    g, st = _new(oracle, "ranecu", n)
    for count, dt in ((16, "u32"), (55, "f32"), (24, "f32_paper"), (33, "f32"), (56, "u32")):
        got = g.generate_packed4(count, dt).cpu().numpy().transpose(0, 2, 1).reshape(n, count)
        assert np.array_equal(bits(got), bits(oracle.generate("ranecu", st, count, dt, threads=8))), f"{count} {dt}"
        assert np.array_equal(g.state_words(), st), f"state after {count} {dt}"


@pytest.mark.parametrize("dt", ["f32_paper", "u32"])
def test_mt_rows_of_workgroups(oracle, dt):
    n = 32769
    g, st = _new(oracle, "mt19937", n)
    for count in (4097, 4098):
        got = bits(g.generate(count, dt).cpu().numpy())
        assert np.array_equal(got, bits(oracle.generate("mt19937", st, count, dt, threads=8))), count
        assert np.array_equal(g.state_words(), st), count
