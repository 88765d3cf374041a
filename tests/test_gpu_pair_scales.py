"""GPU parity of the products on pairs on networks whose units have very different weight scales.

Multiplying the incoming weights (and bias) of a hidden unit by s and its outgoing ones by 1/s leaves a
ReLU network's function, and with s a power of two every fp32 value but that unit's scale, as they were,
while the cotangents and weights of one layer then spread over many powers of two.

Tolerance: that of the pair tests at weights of one scale, with one difference.  Where a single unit
carries a Jacobian row, the row's norm is one cotangent, a sum of both signs, and some rows' happen to
cancel; the error of such a sum is set by its terms, which are alike for all outputs of a sample.  The
error of an entry is therefore taken relative to the largest row norms among the outputs of its two
samples.  (Relative to its own rows' norms the fp32 kernels reach 1.2e-4 as well.)
"""
import numpy as np
import pytest

import oracle
import workloads as wl
from tests.gpu_helpers import gpu_ntk, report, scaled_errors, variant_of, variant_scale

pytestmark = pytest.mark.gpu
S = "fp32"
PAIR_TOL = 1.5e-5


def scales(kind, n, rng):
    """Exponents of s, one per unit: "one k" (one unit), "many k" (every 16th), "normal k" (standard
    deviation k bits)."""
    k, e = int(kind.split()[1]), np.zeros(n)
    if kind.startswith("one"):
        e[rng.integers(n)] = k
    elif kind.startswith("many"):
        e[::16] = k
    else:
        e = np.round(rng.standard_normal(n) * k)
    return e


def rescale_fcn(spec, params, kind, seed):
    rng = np.random.default_rng(seed)
    step = 2 if spec["layers"][0]["bias"] else 1
    params = [p.copy() for p in params]
    for l in range(len(spec["layers"]) - 1):
        s = np.exp2(scales(kind, spec["layers"][l]["out"], rng)).astype(np.float32)
        for p in params[step * l:step * l + step]:
            p *= s.reshape((-1,) + (1,) * (p.ndim - 1))
        params[step * (l + 1)] /= s
    return params


def sample_scale(d1, d2):
    """sqrt of the largest Theta(x, x)[o, o] over o of both samples, for every entry [N1, N2, O, O]."""
    s = np.sqrt(d1.max(1)[:, None] * d2.max(1)[None, :])
    return np.broadcast_to(s[:, :, None, None], s.shape + (d1.shape[1],) * 2)


KINDS = ["one -8", "one -14", "one -24", "one 16", "many -16", "many 12", "normal 3", "normal 4", "normal 6"]


def _check(kind, widths, n1, n2, bias, variants):
    spec = wl.fcn_spec("pairu", 64, widths, 10, bias=bias)
    params = rescale_fcn(spec, wl.make_params(spec, 91, "2/fan_in"), kind, 92)
    X1, X2 = wl.make_inputs(spec, n1, 93), wl.make_inputs(spec, n2, 94)
    ref = oracle.ntk_structured_fp64(spec, params, X1, X2, layer_storage=S)
    d1, d2 = (oracle.ntk_structured_diag_fp64(spec, params, X, layer_storage=S) for X in (X1, X2))
    for variant in variants:
        print(f"[pair] unit scales {kind} {widths} {variant}", flush=True)
        prof = {}
        got = gpu_ntk(spec, params, X1, X2, variant=variant, profile=prof)
        assert "dense_bwd_pair" in prof
        scale = sample_scale(d1, d2) if variant[0] == "full" else variant_scale(d1, d2, *variant)
        cs, nw = scaled_errors(got, variant_of(ref, *variant), scale)
        report(f"unit scales {kind} {widths} {variant}", cs, nw)
        assert np.isfinite(got).all() and cs <= PAIR_TOL and nw <= PAIR_TOL


FULL, TRACE = ("full", "full", 0), ("trace", "full", 0)


@pytest.mark.parametrize("kind", KINDS)
def test_pair_rows_unit_scales(kind):
    # widths of whole 64- and 128-wide tiles and ragged ones with biases
    _check(kind, [512] * 4, 300, 256, False, (FULL, TRACE))
    _check(kind, [389, 260, 515], 80, 60, True, (FULL, TRACE))


@pytest.mark.parametrize("widths", [[2056, 8200], [2101, 9001]], ids=str)
def test_pair_rows_of_wide_layers(widths):
    """Rows of more than 2048 values (a workgroup each) and of more than its registers hold."""
    _check("normal 4", widths, 9, 8, False, (FULL,))
