"""Stream counts beyond one launch of a wavefront (2^26) or a workgroup (2^25)
per stream, and beyond the count from which interleaved rows and the consumer go
one lane per stream (2^25): the first streams, those around each range's end and
the last ones against the oracle, over two calls."""
import numpy as np
import pytest
import torch

from paper_1003_1898_amd.generator import Generator

from mirror import bits

pytestmark = pytest.mark.gpu

RANGE = 1 << 24  # launches start at multiples of this many streams


def _streams(kind, n):
    words = 2 if kind in ("ranecu", "ranmar") else 1
    seeds = np.empty((n, words), dtype=np.uint64)
    for j in range(words):
        seeds[:, j] = 1 + (np.arange(n, dtype=np.uint64) * np.uint64(7919 + j)) % np.uint64(30000)
    at = sorted({s for c in [0, n] + list(range(RANGE, n, RANGE)) for s in range(c - 3, c + 3) if 0 <= s < n})
    print(f"\n[many streams] {kind} n={n}", flush=True)
    return seeds, np.array(at)


@pytest.fixture(autouse=True)
def _give_memory_back():
    yield
    torch.cuda.empty_cache()


@pytest.mark.parametrize("kind,n,dt,counts", [("ggl", (1 << 26) + 5, "f32", (3, 2)),
                                              ("mt19937", (1 << 25) + 3, "f64", (1, 1))])
def test_rows(oracle, kind, n, dt, counts):
    seeds, at = _streams(kind, n)
    g = Generator(kind, n, seed_words=seeds)
    st = oracle.init(kind, seeds[at])
    for count in counts:
        got = g.generate(count, dt)[torch.from_numpy(at).cuda()].cpu().numpy()
        assert np.array_equal(bits(got), bits(oracle.generate(kind, st, count, dt)))


def test_interleaved_rows(oracle):
    n = (1 << 25) + 4
    seeds, at = _streams("ggl", n)
    g = Generator("ggl", n, seed_words=seeds)
    st = oracle.init("ggl", seeds[at])
    for count in (2, 3):
        out = g.generate_packed4(count, "f32")
        got = out[torch.from_numpy(at // 4).cuda(), :, torch.from_numpy(at % 4).cuda()].cpu().numpy()
        assert np.array_equal(bits(got), bits(oracle.generate("ggl", st, count, "f32")))


@pytest.mark.parametrize("kind", ["ggl", "ranmar"])
def test_consumer(oracle, kind):
    n = (1 << 25) + 4
    seeds, at = _streams(kind, n)
    g = Generator(kind, n, seed_words=seeds)
    st = oracle.init(kind, seeds[at])
    for draws in (40, 7):
        s, h = g.fused_sum_hist(draws)
        i = torch.from_numpy(at).cuda()
        rs, rh = oracle.fused(kind, st, draws)
        assert np.array_equal(s.view(torch.int64)[i].cpu().numpy().view(np.uint64), rs)
        assert np.array_equal(h.view(torch.int32)[i].cpu().numpy().view(np.uint32), rh)
