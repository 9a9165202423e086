"""Calls at the lines between two ways of running them: draw and stream counts
on both sides, bit-exact with the oracle."""
import numpy as np
import pytest

from paper_1003_1898_amd import inputs
from paper_1003_1898_amd.generator import Generator

from mirror import bits

pytestmark = pytest.mark.gpu


def _check_rows(oracle, kind, n, calls, p=223):
    print(f"\n[routes] {kind} n={n}", flush=True)
    seeds = inputs.seed_words(kind, 77, n)
    g = Generator(kind, n, seed_words=seeds, p=p)
    st = oracle.init(kind, seeds)
    for count, dt in calls:
        got = bits(g.generate(count, dt).cpu().numpy())
        assert np.array_equal(got, bits(oracle.generate(kind, st, count, dt, p=p, threads=8))), f"{count} {dt}"
        assert np.array_equal(g.state_words(), st), f"state after {count} {dt}"


@pytest.mark.parametrize("n,calls", [(1000, ((256, "f32"), (257, "u32"), (150, "f64"))),
                                     (16384, ((512, "u32"), (513, "f32"), (301, "f32"), (300, "u32"))),
                                     (8200, ((9200, "f32"), (4601, "f64"))),  # beyond the cache: long segments
                                     (24001, ((3200, "u32"),))])
def test_xor128_rows(oracle, n, calls):
    _check_rows(oracle, "xor128", n, calls)


@pytest.mark.parametrize("n,p,calls", [(70, 24, ((492, "u32"), (242, "f64"), (480, "f32"))),
                                       (300, 97, ((240, "f32"), (241, "u32"), (180, "f64"))),
                                       (130, 389, ((192, "u32"), (193, "f32"), (101, "f64"))),
                                       (16500, 97, ((520, "f32"), (470, "u32"))),
                                       (32800, 223, ((500, "f32"), (390, "u32"), (120, "f64")))])
def test_ranlux_rows(oracle, n, p, calls):
    _check_rows(oracle, "ranlux", n, calls, p)


@pytest.mark.parametrize("n,calls", [(40001, ((1001, "f32"), (1249, "u32"))), (24003, ((2100, "f32_paper"),)),
                                     (18002, ((3500, "u32"),))])
def test_mt_rows(oracle, n, calls):
    _check_rows(oracle, "mt19937", n, calls)


@pytest.mark.parametrize("n,calls", [(28675, ((128, "f32"), (64, "f64"), (128, "u32"), (127, "f32"))),
                                     (43009, ((4097, "u32"), (2049, "f64")))])
def test_ranmar_rows(oracle, n, calls):
    _check_rows(oracle, "ranmar", n, calls)


def _check_packed(oracle, kind, n, calls):
    print(f"\n[routes packed] {kind} n={n}", flush=True)
    seeds = inputs.seed_words(kind, 78, n)
    g = Generator(kind, n, seed_words=seeds)
    st = oracle.init(kind, seeds)
    for count, dt in calls:
        got = g.generate_packed4(count, dt).cpu().numpy().transpose(0, 2, 1).reshape(n, count)
        assert np.array_equal(bits(got), bits(oracle.generate(kind, st, count, dt, threads=8))), f"{count} {dt}"
        assert np.array_equal(g.state_words(), st), f"state after {count} {dt}"


@pytest.mark.parametrize("n,calls", [(40000, ((1, "f32"), (128, "u32"), (257, "f32_paper"), (900, "f32"), (256, "u32"))),
                                     (24004, ((128, "f32_paper"), (384, "f32"), (1, "u32")))])
def test_ranmar_interleaved_rows(oracle, n, calls):
    _check_packed(oracle, "ranmar", n, calls)


def _check_consumer(oracle, kind, n, calls):
    print(f"\n[routes consumer] {kind} n={n}", flush=True)
    seeds = inputs.seed_words(kind, 79, n)
    g = Generator(kind, n, seed_words=seeds)
    st = oracle.init(kind, seeds)
    for draws in calls:
        s, h = g.fused_sum_hist(draws)
        rs, rh = oracle.fused(kind, st, draws, threads=8)
        assert np.array_equal(s.cpu().numpy(), rs), f"draws {draws}"
        assert np.array_equal(h.cpu().numpy(), rh), f"draws {draws}"
        assert np.array_equal(g.state_words(), st), f"draws {draws}"


@pytest.mark.parametrize("n,calls", [(17001, (1, 128, 255, 257)), (24001, (0, 130, 512, 513))])
def test_ranmar_consumer(oracle, n, calls):
    _check_consumer(oracle, "ranmar", n, calls)


@pytest.mark.parametrize("kind", ["ggl", "ranecu", "drand48", "rannyu"])
def test_leap_interleaved_rows(oracle, kind):
    paper = "f32_paper" if kind in ("ggl", "ranecu") else "u32"
    _check_packed(oracle, kind, 57344, ((128, "u32"), (128, paper), (256, "f32"), (129, "f32"), (128, "f32")))


@pytest.mark.parametrize("kind", ["ggl", "xor128", "ranecu", "drand48", "rannyu"])
def test_consumer(oracle, kind):
    _check_consumer(oracle, kind, 10007, (1, 64, 300, 2500))
