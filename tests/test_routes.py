"""The dispatch rules of csrc/routes.h on the CPU: calls that one way of running
them was measured to be slower for take the other one, and every answer is one
that the kernels accept."""
import os
import random
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1003_1898_amd", "csrc")


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("routes") / "routes_check")
    subprocess.run(["g++", "-O1", "-std=c++20", "-I", CSRC, os.path.join(HERE, "routes_check.cpp"), "-o", exe],
                   check=True)

    def ask(rule, calls):
        """The rule's answers (lists of integers) to calls of three numbers."""
        text = "".join("%s %d %d %d\n" % (rule, *c) for c in calls)
        out = subprocess.run([exe], input=text, check=True, capture_output=True, text=True).stdout
        return [[int(v) for v in line.split()] for line in out.splitlines()]

    return ask


def _calls(seed, count, n_max, d_max, third):
    r = random.Random(seed)
    return [(int(2 ** r.uniform(0, n_max)), int(2 ** r.uniform(0, d_max)), r.choice(third)) for _ in range(count)]


# ------------------------------------------------------------------ XOR128 rows
@pytest.mark.parametrize("n,d", [(64, 256), (256, 200), (4096, 256), (10007, 160), (20011, 512), (28000, 384),
                                 (32000, 512)])
def test_xor128_short_calls_stay_uncut(routes, n, d):
    assert routes("xor128", [(n, d, 0)])[0][1] == 1


@pytest.mark.parametrize("n,d,K", [(256, 192, 2), (256, 384, 3), (4096, 512, 4), (4096, 4000, 32), (20011, 448, 4), (20011, 2048, 4),
                                   (1024, 32768, 128)])
def test_xor128_short_segments(routes, n, d, K):
    S, got = routes("xor128", [(n, d, 0)])[0]
    assert got == K and S & (S - 1) == 0


@pytest.mark.parametrize("n,d,K", [(12032, 8192, 4), (20011, 4000, 2), (28000, 3072, 1), (20032, 4096, 2), (24000, 16384, 8), (28000, 4096, 2),
                                   (32768, 1500, 1), (65536, 16384, 4)])
def test_xor128_output_beyond_the_cache_takes_long_segments(routes, n, d, K):
    assert routes("xor128", [(n, d, 0)])[0][1] == K


def test_xor128_cuts_are_whole(routes):
    calls = _calls(1, 4000, 20, 30, (0, 1))
    for (n, d, shared), (S, K) in zip(calls, routes("xor128", calls)):
        assert (K - 1) * S < d <= K * S, (n, d, shared)
        assert K == 1 or (S % 128 == 0 and K * ((n + 255) // 256) < 1 << 24), (n, d, shared)
        assert not shared or d >= 4096 or K == 1, (n, d)


# ------------------------------------------------------------------ RANLUX rows
@pytest.mark.parametrize("n,d,p", [(64, 192, 24), (4096, 256, 24), (256, 360, 24), (4096, 256, 97), (20011, 256, 97),
                                   (40000, 192, 223), (40000, 512, 97), (48000, 2304, 24), (40000, 3000, 97)])
def test_ranlux_short_calls_stay_uncut(routes, n, d, p):
    assert routes("lux", [(n, d, p)])[0][1] == 1


@pytest.mark.parametrize("n,d,p,K", [(4096, 576, 24, 6), (256, 224, 97, 2), (4096, 384, 97, 4), (64, 224, 389, 2),
                                     (20011, 1001, 97, 4), (40000, 512, 389, 2), (300, 5000, 97, 27),
                                     (24000, 3072, 24, 2), (65536, 16384, 223, 2)])
def test_ranlux_segments(routes, n, d, p, K):
    assert routes("lux", [(n, d, p)])[0][1] == K


@pytest.mark.parametrize("n,d,p,K", [(4096, 192, 24, 1), (4096, 384, 24, 4), (40000, 3000, 97, 2),
                                     (40000, 3000, 24, 1), (20011, 4000, 24, 4)])
def test_ranlux_f64_segments(routes, n, d, p, K):
    assert routes("lux_f64", [(n, d, p)])[0][1] == K


@pytest.mark.parametrize("rule", ["lux", "lux_f64", "lux_shared"])
def test_ranlux_cuts_are_whole(routes, rule):
    calls = _calls(2, 4000, 20, 30, (24, 48, 97, 223, 389, 800))
    for (n, d, p), (S, K) in zip(calls, routes(rule, calls)):
        assert (K - 1) * S < d <= K * S and 1 <= K <= 64, (n, d, p)
        assert K == 1 or (S % 96 == 0 and K * ((n + 255) // 256) < 1 << 24), (n, d, p)
        assert rule != "lux_shared" or K == 1 or d >= 3072, (n, d)


# --------------------------------------------------------------- MT19937 rows
@pytest.mark.parametrize("n,d,wave", [(256, 16384, 1), (14000, 16384, 1), (18000, 4096, 1), (19968, 8256, 0),
                                      (20011, 3072, 1), (24000, 3000, 0), (23516, 2503, 1), (28083, 8075, 1),
                                      (32768, 1248, 1), (40000, 1500, 0), (49152, 800, 0), (65536, 400, 1),
                                      (65536, 500, 0), (65536, 16384, 0), (96000, 64, 0), (131072, 800, 1),
                                      (131072, 2000, 0)])
def test_mt_rows(routes, n, d, wave):
    assert routes("mt19937", [(n, d, 0)]) == [[wave]]


# --------------------------------------------------------------------- RANMAR
@pytest.mark.parametrize("n,d,lane", [(40000, 128, 1), (16384, 128, 0), (40000, 256, 0), (44000, 4096, 1),
                                      (40000, 4096, 0), (49152, 1, 1), (65536, 16384, 1), (66048, 4096, 0),
                                      (81920, 128, 1), (81920, 2048, 0)])
def test_ranmar_rows(routes, n, d, lane):
    assert routes("ranmar", [(n, d, 0)]) == [[lane]]


@pytest.mark.parametrize("n,d,lane", [(40000, 1, 1), (40000, 256, 1), (40000, 512, 1), (40000, 1000, 0),
                                      (24000, 128, 1), (24000, 512, 0), (16384, 100, 0), (4096, 128, 0),
                                      (81920, 384, 1), (66048, 1000, 0), (48000, 2048, 1), (131072, 1, 1)])
def test_ranmar_interleaved_rows(routes, n, d, lane):
    assert routes("ranmar_packed", [(n, d, 0)]) == [[lane]]


@pytest.mark.parametrize("n,d,lane", [(20011, 16, 1), (20011, 512, 0), (32768, 512, 1), (32768, 1000, 0),
                                      (16384, 16, 0), (4096, 1 << 20, 0), (40000, 16, 0)])
def test_ranmar_consumer(routes, n, d, lane):
    assert routes("ranmar_consumer", [(n, d, 0)]) == [[lane]]


# ------------------------------------------ interleaved rows of the leap kinds
@pytest.mark.parametrize("n,d,ranecu,lane", [(65536, 128, 1, 1), (65536, 256, 1, 1), (65536, 512, 1, 1),
                                             (65536, 1024, 1, 0), (40000, 384, 1, 0), (16384, 256, 1, 0),
                                             (65536, 250, 1, 0), (65536, 128, 0, 1), (65536, 256, 0, 0),
                                             (16384, 128, 0, 0)])
def test_leap_interleaved_rows(routes, n, d, ranecu, lane):
    assert routes("leap_packed", [(n, d, ranecu)]) == [[lane]]


@pytest.mark.parametrize("n,d,ranecu,lane", [(65536, 24, 1, 1), (65536, 32, 1, 1), (131072, 24, 1, 1), (65500, 37, 1, 1),
                                             (54848, 35, 1, 1), (65536, 8, 1, 0), (65536, 64, 1, 0), (44032, 32, 1, 0),
                                             (98304, 32, 1, 0), (65536, 24, 0, 0)])
def test_leap_interleaved_rows_of_few_draws(routes, n, d, ranecu, lane):
    assert routes("leap_packed", [(n, d, ranecu)]) == [[lane]]


# ----------------------------------------------------------------- the consumer
GGL, XOR128, RANECU, DRAND48, RANNYU = 1, 2, 3, 7, 8


@pytest.mark.parametrize("kind,n,d,width", [(GGL, 20011, 256, 0), (GGL, 20011, 1000, 1), (GGL, 28000, 512, 0),
                                            (GGL, 50000, 1000, 1), (GGL, 65536, 16, 1), (GGL, 4096, 16, 1),
                                            (XOR128, 64, 512, 0), (XOR128, 10007, 2048, 0), (XOR128, 20011, 4096, 0),
                                            (XOR128, 4096, 4096, 1), (RANECU, 28000, 256, 0), (RANECU, 4096, 1 << 20, 1),
                                            (RANECU, 64, 1 << 20, 16), (DRAND48, 28000, 512, 0), (GGL, 1383, 28672, 4),
                                            (RANNYU, 20011, 4096, 1), (GGL, (1 << 25) + 4, 100, 0)])
def test_consumer_width(routes, kind, n, d, width):
    assert routes("consumer", [(n, d, kind)]) == [[width]]


def test_consumer_widths_fit_a_launch(routes):
    calls = _calls(3, 4000, 30, 30, (GGL, XOR128, RANECU, DRAND48, RANNYU)) + [(1, 0, XOR128), (100000, 0, RANECU)]
    for (n, d, kind), (w,) in zip(calls, routes("consumer", calls)):
        assert w in (0, 1, 4, 16) and n * max(w, 1) <= max(n, 1 << 25), (n, d, kind)


def test_stream_ranges_cover_every_stream_once(routes):
    for n, most in ((1, 8), (8, 8), (9, 8), (64, 8), (67, 12), ((1 << 26) + 5, 1 << 25)):
        (got,) = routes("ranges", [(n, most, 0)])
        first, count = got[0::2], got[1::2]
        assert first == list(range(0, n, most)) and sum(count) == n and max(count) <= most
        assert all(a + c == b for a, c, b in zip(first, count, first[1:] + [n]))
