"""The ordering of a row's candidates by one histogram on a linear scale: spread rows whose candidates stay in registers, and bf16 rows of the calls
with one workgroup per row, against the oracle where bins are as full as may be, fuller, or hold equal values."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_19133_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ps():
    from paper_2603_19133_amd import binding
    return binding


@pytest.fixture(scope="module")
def pu():
    import parity_util
    return parity_util


def _rows(rng, pattern, R, V, dtype):
    z = rng.standard_normal((R, V)) * 3
    if pattern == "below_zero":
        z = z - 40
    elif pattern == "around_zero":                         # signed zeros and the values next to them among the largest
        z = np.where(z > 0, 0.0, z)
        z[:, ::7] = -0.0
        z[:, 5], z[:, 6] = 1e-30, -1e-30
    elif pattern == "even":                                # as many near the largest as at the threshold
        z = rng.random((R, V))
    elif pattern.startswith("equal"):                      # that many values that no bin tells apart, above the rest
        m = int(pattern[5:])
        at = rng.permutation(V)[:m]
        z = np.minimum(z, 9.0)
        z[:, at] = 10.0 if dtype == "f32" else 0.0
        if dtype == "bf16":                                # (equal bf16 values spread by id unless they are zero)
            z = np.minimum(z, 0.0)
    elif pattern == "outlier":
        z[:, V // 3] = 1e6
    elif pattern.startswith("far"):                        # that many values far above the others, in as many places, some in turn above the rest of them
        m = int(pattern[3:])
        z[:, 100:100 + (V // (m + 1)) * m:V // (m + 1)] = 300.0
        z[0, 100] = 1e6
    elif pattern.startswith("grid"):                       # values on a grid: bins of some ten to some hundred
        z = np.round(z * int(pattern[4:])) / int(pattern[4:])
    elif pattern == "steep":                               # a few far above, many close together
        z = np.sign(z) * np.abs(z) ** 4
    elif pattern == "late":                                # the largest ones in one workgroup's share: its list does not hold them
        z = z + 30.0 * ((np.arange(V) // 256) % 64 == 5)
    elif pattern == "masked":
        z = np.where(rng.random((R, V)) < 0.995, -np.inf, z)
    return z.astype(np.float32)


@pytest.mark.parametrize("pattern", ["normal", "below_zero", "around_zero", "even", "equal64", "equal65", "equal200", "equal256", "equal257", "outlier", "far1", "far2",
                                     "far9", "far40", "grid2", "grid4", "grid8", "grid16", "steep", "late", "masked"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("V,R,k,top_p", [(16384, 2, 1, 0.0), (33001, 3, 64, 0.0), (33001, 2, 777, 0.9), (151936, 2, 1024, 0.0), (100003, 2, 1700, 0.0),
                                         (65536, 2, 2049, 0.0)])      # (slots of all lists on either side of 4096)
def test_spread_rows(gpu, pu, ps, pattern, dtype, V, R, k, top_p):
    print("[case]", pattern, dtype, V, R, k, top_p, flush=True)
    z = _rows(np.random.default_rng(V + k), pattern, R, V, dtype)
    z = W.to_bf16_bits(z) if dtype == "bf16" else z
    o = oracle.compress(z, V, 0.9, k, top_p)
    g = ps.compress(pu.to_device(z, gpu), V, 0.9, k, top_p)
    pu.compare_compress(g, o, top_p)


@pytest.mark.parametrize("pattern", ["normal", "below_zero", "around_zero", "even", "equal64", "equal65", "equal200", "outlier", "steep"])
@pytest.mark.parametrize("V,k,top_p", [(32768, 10, 0.0), (33001, 777, 0.9), (152064, 2048, 0.0), (131072, 3000, 0.0)])
def test_rows_of_one_workgroup(gpu, pu, ps, pattern, V, k, top_p):
    print("[case]", pattern, V, k, top_p, flush=True)
    z = W.to_bf16_bits(_rows(np.random.default_rng(V + k), pattern, 2, V, "bf16"))
    o = oracle.compress(z, V, 1.0, k, top_p)
    t = pu.to_device(z, gpu)
    with pu.no_scratch():
        g = ps.compress(t, V, 1.0, k, top_p)
    pu.compare_compress(g, o, top_p)
