"""GPU parity of the products on pair rows (fp32 values as two f16 values with one exponent per row)
against the fp64 structured reference, at the sizes where they can go wrong: widths around the K
tile and the 64- and 128-wide tiles, ragged row counts, one output, one hidden layer, rows and
columns of very different magnitudes, rows of zeros.

Tolerance (Cauchy-Schwarz-normalised, worst case): a product of two pairs is off by at most
2^-24 per factor (23 significant bits) and 2^-22 (the dropped lo lo'), 4e-7 together; a sum over K
adds 3 K / 16 roundings of 2^-24, 3.4e-6 at K = 300 (flushed every 256 k in the contraction); the
cotangents of a depth-3 net pass two such products before the contraction's own and the Grams'
rounding: 4 x 3.8e-6 = 1.5e-5.
"""
import numpy as np
import pytest

import oracle
import workloads as wl
from tests.gpu_helpers import errors, gpu_ntk, report, scaled_errors, variant_of, variant_scale

pytestmark = pytest.mark.gpu
S = "fp32"
PAIR_TOL = 1.5e-5


def _check(name, spec, params, X1, X2, variant=("full", "full", 0)):
    print(f"[pair] {name} {variant}", flush=True)
    got = gpu_ntk(spec, params, X1, X2, variant=variant)
    ref = oracle.ntk_structured_fp64(spec, params, X1, X2, layer_storage=S)
    d1 = oracle.ntk_structured_diag_fp64(spec, params, X1, layer_storage=S)
    d2 = d1 if X2 is X1 else oracle.ntk_structured_diag_fp64(spec, params, X2, layer_storage=S)
    if variant == ("full", "full", 0):
        cs, nw = errors(got, ref, d1, d2)
    else:
        cs, nw = scaled_errors(got, variant_of(ref, *variant), variant_scale(d1, d2, *variant))
    report(name, cs, nw)
    assert cs <= PAIR_TOL and nw <= PAIR_TOL


CASES = [
    # widths, O, n1, n2, act, bias
    ("tile edges", [128, 129, 255], 10, 128, 103, "relu", False),
    ("ragged erf, biases", [161, 300, 257], 7, 150, 133, "erf", True),
    ("one output", [301, 130], 1, 1100, 515, "relu", True),
    ("one hidden layer", [131], 10, 300, 127, "relu", False),
    ("100 outputs, few samples", [200, 140], 100, 9, 8, "erf", False),
    ("stream-K tiles", [133, 160], 10, 300, 301, "relu", False),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_pair_rows_shapes(case):
    name, widths, O, n1, n2, act, bias = case
    spec = wl.fcn_spec("pair", 70, widths, O, act=act, bias=bias)
    params = wl.make_params(spec, 41, "2/fan_in" if act == "relu" else "1/fan_in")
    X1, X2 = wl.make_inputs(spec, n1, 42), wl.make_inputs(spec, n2, 43)
    _check(name, spec, params, X1, X2)
    _check(name + " aliased", spec, params, X1, X1)


@pytest.mark.parametrize("variant", [("trace", "full", 0), ("logit", "full", 3), ("full", "diagonal", 0),
                                     ("trace", "diagonal", 0)])
def test_pair_rows_variants(variant):
    spec = wl.fcn_spec("pairv", 60, [515, 389, 517], 6)
    params = wl.make_params(spec, 44, "2/fan_in")
    X1, X2 = wl.make_inputs(spec, 257, 45), wl.make_inputs(spec, 257, 46)
    _check("variants", spec, params, X1, X2, variant)


def test_pair_rows_magnitudes():
    """Units, outputs and layers whose weights differ by powers of two up to 2^40, and dead units
    (rows of zeros): every row has an exponent of its own."""
    spec = wl.fcn_spec("pairm", 64, [200, 170, 150], 10)
    params = wl.make_params(spec, 47, "2/fan_in")
    rng = np.random.default_rng(48)
    params[3] *= np.exp2(rng.integers(-20, 21, (10, 1))).astype(np.float32)     # outputs
    params[0] *= np.float32(2.0 ** 30)                                         # layers
    params[2] *= np.float32(2.0 ** -40)
    params[1][::7] = -np.abs(params[1][::7])                                   # dead units of layer 1
    params[1][5] = 0.0
    X1, X2 = wl.make_inputs(spec, 140, 49), wl.make_inputs(spec, 120, 50)
    _check("magnitudes", spec, params, X1, X2)
