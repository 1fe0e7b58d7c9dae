"""The binned form's fixed point and polynomial, emulated on the CPU.

The constants are read from the kernels' sources.  The fields of the packed
words must come back exactly for any number of pairs up to kBinMaxCount, also
where every pair of a bin has the same extreme coordinate; the nodes and the
Lagrange table are those of fit_bins.py; and the whole chain (powers rounded to
fixed point, sums, node weights) must reproduce the sum of sinc(q r) over a
bin's pairs."""
from __future__ import annotations

import importlib.util
import math
import os
import re

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1306_2258_amd", "csrc")
HPP = open(os.path.join(CSRC, "sas_bins.hpp")).read()
HIP = open(os.path.join(CSRC, "sas_bins.hip")).read()
_spec = importlib.util.spec_from_file_location("fit_bins", os.path.join(CSRC, "fit_bins.py"))
fit = importlib.util.module_from_spec(_spec)
_spec.loader.exec_module(fit)


def const(name):
    return re.search(r"\b" + name + r" = ([^,;]+)[,;]", HPP).group(1)


BITS = [0] + [int(const(f"kBinBits{k}")) for k in range(1, 6)]
SHIFT5, SHIFT4, CSHIFT = int(const("kBinShift5")), int(const("kBinShift4")), int(const("kBinCountShift"))
MAGIC = int(const("kBinMagicBits").rstrip("u"), 16)
BIAS4 = float.fromhex(const("kBinBias4"))
STEP = float(const("kBinStep"))
MAX_COUNT = (1 << 15) + 16 * 64 * 64
M32, M64 = (1 << 32) - 1, (1 << 64) - 1


def signed(v, bits):
    v &= (1 << bits) - 1
    return v - (1 << bits) if v >> (bits - 1) else v


def fields(u):
    """Integer values of the powers of u as the kernel rounds them (FP32)."""
    u = np.float32(u)
    u2 = u * u
    p = [u, u2, u2 * u, u2 * u2, u2 * u2 * u]
    return [int(np.rint(float(p[k]) * 2.0 ** BITS[k + 1])) for k in range(5)]


def words(f):
    b = [(MAGIC + v) & M32 for v in f]
    return (((1 << CSHIFT) << 32) + b[0], (((b[4] << SHIFT5) & M32) << 32) + b[1], (((b[3] << SHIFT4) & M32) << 32) + b[2])


def decode(wa, wb, wc):
    ka = (1 << (32 + CSHIFT)) + MAGIC
    kb = (((MAGIC << SHIFT5) & M32) << 32) + MAGIC
    kc = (((MAGIC << SHIFT4) & M32) << 32) + MAGIC
    cnt = int(float(wa) / float(ka) + 0.5)
    tb, tc = (wb - cnt * kb) & M64, (wc - cnt * kc) & M64
    low_b, low_c = 32 + SHIFT5, 32 + SHIFT4
    m2, m3 = signed(tb, low_b), signed(tc, low_c)
    return [cnt, signed(wa - cnt * ka, 64), m2, m3, signed(tc - m3, 64) >> low_c, signed(tb - m2, 64) >> low_b]


@pytest.mark.parametrize("count", [1, 2, 4096, 1 << 15, MAX_COUNT])
@pytest.mark.parametrize("u", [0.0, -1.001, -1.0, 1.001, 1.5, 0.37, -1e-3])
def test_fields_hold_a_full_bin(u, count):
    assert "(1 << 15)" not in const("kBinMaxCount") and const("kBinSpill") == "1 << 15"
    assert const("kBinMaxCount") == "kBinSpill + kBinWaves * kWave * 64"
    f = fields(u)
    assert all(abs(v) < 1 << 22 for v in f)  # (the low bits of the FP32 sum hold them)
    w = [(x * count) & M64 for x in words(f)]
    assert [x * count for x in words(f)][0] <= M64
    assert decode(*w) == [count] + [v * count for v in f]


def test_fields_of_mixed_pairs():
    rng = np.random.default_rng(5)
    for _ in range(20):
        fs = [fields(u) for u in rng.uniform(-1.0, 1.0, 3000)]
        w = [sum(words(f)[k] for f in fs) & M64 for k in range(3)]
        assert decode(*w) == [len(fs)] + [sum(f[k] for f in fs) for k in range(5)]


def test_nodes_and_table():
    v = fit.nodes()
    got = [float.fromhex(x) for x in re.findall(r"-?0x1\.[0-9a-f]+p[+-]\d+", HIP[HIP.index("double kBinNode["):HIP.index("double kBinL[")])]
    assert got == [float(x) for x in v]
    at = HIP.index("double kBinL[")
    rows = [float.fromhex(x) for x in re.findall(r"-?0x1\.[0-9a-f]+p[+-]\d+", HIP[at:HIP.index("}};", at)])]
    assert rows == [float(x) for row in fit.lagrange(v) for x in row]
    assert BIAS4 == pytest.approx(fit.rounding_mean(4, BITS[4]), rel=1e-9)


@pytest.mark.parametrize("b", [0, 1, 2, 7, 100, 6000])
def test_bin_reproduces_sinc(b):
    """Pairs spread over bin b at the largest q.  Per pair the polynomial is off
    by at most 3e-8 and the rounding of the powers by at most
    sum_k |c_k| 2^-(bits_k + 1), c_k the polynomial's coefficients; the roundings
    are independent, so the mean over n pairs keeps about 1/sqrt(n) of it."""
    rng = np.random.default_rng(b)
    n = 20000
    tc = b + 0.5
    s = rng.uniform(0.25 if b == 0 else b * b, (b + 1) ** 2, n)
    u = ((s - tc * tc) / tc).astype(np.float32)
    f = np.array([np.rint(p.astype(np.float64) * 2.0 ** BITS[k + 1]) for k, p in
                  enumerate([u, u * u, u * u * u, (u * u) * (u * u), (u * u) * (u * u) * u])])
    m = np.concatenate([[float(n)], f.sum(axis=1) / 2.0 ** np.array(BITS[1:])])
    m[4] -= BIAS4 * n
    scale, al = (4.0 / 3.0, -0.75) if b == 0 else (1.0, -0.25 / tc)
    for p in range(1, 6):
        for k in range(5, p - 1, -1):
            m[k] += al * m[k - 1]
    m *= scale ** np.arange(6)
    v = np.array([float(x) for x in fit.nodes()])
    lag = np.array([[float(x) for x in row] for row in fit.lagrange(fit.nodes())])
    radius = np.sqrt(0.375 + 0.375 * v if b == 0 else b * b + b + 0.25 + tc * v)
    for x in (1.0, 0.5, 0.1):  # q / qmax
        h = STEP * x
        got = float((m @ lag) @ np.sinc(h * radius / math.pi))
        ref = float(np.sinc(h * np.sqrt(np.maximum(s - 0.25, 0.0)) / math.pi).sum())
        size = float(np.abs(np.sinc(h * np.sqrt(np.maximum(s - 0.25, 0.0)) / math.pi)).max())
        coeff = np.abs(lag @ np.sinc(h * radius / math.pi)) * scale ** np.arange(6)
        rounding = float((coeff[1:] * 0.5 ** (np.array(BITS[1:]) + 1)).sum()) * 4.0 / math.sqrt(n)
        assert abs(got - ref) / n <= 3e-8 * x ** 6 * max(size, 1.0 / (h * max(tc, 1.0))) + rounding + 1e-12
