"""Interleaved rows of the multiplicative and affine generators: one, four or
sixteen wavefronts per row of four streams, draw counts around a wavefront's and
a workgroup's stride, several calls in a row; bit-exact with the oracle."""
import numpy as np
import pytest

from paper_1003_1898_amd import inputs
from paper_1003_1898_amd.generator import Generator

from mirror import bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["ggl", "ranecu", "drand48", "rannyu"])
@pytest.mark.parametrize("n,counts", [(4, (1, 64, 257, 1023, 1024, 1025, 5000)), (36, (63, 65, 3000)),
                                      (4100, (255, 256, 300)), (20004, (2, 130))])
def test_packed_leap(oracle, kind, n, counts):
    print(f"\n[packed leap] {kind} n={n}", flush=True)
    seeds = inputs.seed_words(kind, 44, n)
    g = Generator(kind, n, seed_words=seeds)
    st = oracle.init(kind, seeds)
    dts = ["u32", "f32"] + (["f32_paper"] if kind in ("ggl", "ranecu") else [])
    for i, count in enumerate(counts):
        dt = dts[i % len(dts)]
        got = g.generate_packed4(count, dt).cpu().numpy().transpose(0, 2, 1).reshape(n, count)
        assert np.array_equal(bits(got), bits(oracle.generate(kind, st, count, dt, threads=8))), f"{count} {dt}"
        assert np.array_equal(g.state_words(), st), f"state after {count} {dt}"
