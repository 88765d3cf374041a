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


# ---- convolutions ---------------------------------------------------------------------------------
C3, DW, PW, POOL, SC = "conv3x3", "dwconv3x3", "conv1x1", "avgpool2", "scale"
# as derived for the convolutions' pair tests: three backward products, a weight-space product, J1 J2^T
CONV_TOL = 3 * 6.8e-6 + 5.8e-6 + 1e-5
PLAIN = ((20, 20), [(C3, 64, "relu", True)] * 3, 13, 10)
STRUCT = ((24, 20), [(C3, 64, "relu", True), (DW, "relu", True), (PW, 64, "relu", True), (POOL,), (SC, "relu", True),
                     (C3, 64, "relu", True), (DW, "relu", False), (SC, "relu", False), (C3, 64, "relu", False)], 40, 21)
# padded channels, scalar loads
ODD = ((15, 15), [(C3, 20, "relu", False), (C3, 45, "relu", True), (SC, "relu", True), (C3, 37, "relu", False),
                  (C3, 17, "relu", False)], 24, 17)


def param_slots(spec):
    """(layer, index of its weight in params) of the layers with parameters."""
    out, i = [], 0
    for L in spec["layers"]:
        if L["kind"] in wl.PARAM_KINDS:
            out.append((L, i))
            i += 2 if L["bias"] else 1
    return out


def rescale_cnn(spec, params, kind, seed):
    rng = np.random.default_rng(seed)
    params = [p.copy() for p in params]
    slots = param_slots(spec)
    for (L, i), (_, j) in zip(slots, slots[1:]):
        s = np.exp2(scales(kind, L["out"], rng)).astype(np.float32)
        # outputs lead in a convolution's weights, channels come last in depthwise and scale weights
        if L["kind"] in (C3, PW):
            params[i] *= s.reshape((-1,) + (1,) * (params[i].ndim - 1))
        else:
            params[i] *= s
        if L["bias"]:
            params[i + 1] *= s
        params[j] /= s   # the inputs' axis is the last one of every kind
    return params


def _conv_check(name, net, change, hooks=("conv_bwd_pair", "conv_wgrad_pair"), act=None):
    hw, blocks, n1, n2 = net
    if act:
        blocks = [tuple(act if x == "relu" else x for x in b) for b in blocks]
    spec = wl.cnn_layers_spec("pairu", hw, 3, blocks, 10)
    params = change(spec, wl.make_params(spec, 95, "2/fan_in", bias_var=0.05))
    X1, X2 = wl.make_inputs(spec, n1, 96), wl.make_inputs(spec, n2, 97)
    print(f"[pair] {name} {hw}", flush=True)
    prof = {}
    got = gpu_ntk(spec, params, X1, X2, profile=prof)
    assert set(hooks) <= set(prof)
    ref, d1, d2 = oracle.ntk_jc_with_norms(spec, params, X1, X2, layer_storage=S)
    cs, nw = scaled_errors(got, ref, sample_scale(d1, d2))
    report(f"{name} {hw}", cs, nw)
    assert np.isfinite(got).all() and cs <= CONV_TOL and nw <= CONV_TOL


@pytest.mark.parametrize("net", [PLAIN, STRUCT, ODD], ids=["plain", "struct", "odd"])
@pytest.mark.parametrize("kind", KINDS)
def test_pair_conv_channel_scales(kind, net):
    _conv_check(f"channel scales {kind}", net, lambda spec, params: rescale_cnn(spec, params, kind, 98))


def test_pair_conv_outlier_channels():
    """Depthwise and scale layers each with one large channel, not the same one."""
    def change(spec, params):
        for n, (L, i) in enumerate(l for l in param_slots(spec) if l[0]["kind"] in (DW, SC)):
            params[i][..., 7 + 11 * n] *= np.float32(2.0 ** 24)
        return params
    _conv_check("outlier channels", STRUCT, change)


def test_pair_conv_saturated_act():
    """act' of the last layer near 2^-36 for every unit, readout weights that make up for it."""
    def change(spec, params):
        (_, i), (_, j) = param_slots(spec)[-2:]
        params[i] *= np.float32(0.02)
        params[i + 1][:] = 5.0
        params[j] *= np.float32(2.0 ** 44)
        return params
    # (enough images for the last layer's weight-space product to take pairs)
    _conv_check("saturated", PLAIN[:2] + (24, 16), change, act="erf")


def test_pair_conv_dead_channel():
    """A channel that no image activates has the largest readout weights by 2^32."""
    def change(spec, params):
        (_, i), (_, j) = param_slots(spec)[-2:]
        params[i + 1][5] = -100.0
        params[j][:, 5] *= np.float32(2.0 ** 32)
        return params
    _conv_check("dead channel", PLAIN, change)


# ---- what stays in fp32 -----------------------------------------------------------------------------
def _disjoint(params, X1, X2):
    """Every other unit answers to X1 alone and carries readout weights of 2^30: entries (x1, x2) come
    from the units between, below the precision of a pair row whose exponent is that of the first."""
    W, b, Wr = params[:3]
    b[::2] = -1e3
    W[::2] = 0.0
    W[(slice(None, None, 2),) + (1,) * (W.ndim - 2) + (0,)] = 1e3   # (the middle tap of a convolution)
    Wr[:, ::2] *= np.float32(2.0 ** 30)
    X1[..., 0], X2[..., 0] = 2.0, 0.0


def _entry_errors(got, ref):
    """Largest error relative to the entry itself, over entries that do not cancel."""
    m = np.abs(ref) > 1e-2 * np.abs(ref).max()
    assert m.mean() > 0.05
    return float(np.max(np.abs(got.astype(np.float64) - ref)[m] / np.abs(ref)[m]))


@pytest.mark.parametrize("call", ["jacobian", "static"])
def test_jacobian_baseline_and_static_calls_stay_in_fp32(call):
    import torch
    from paper_2206_08720_amd import _lib
    from paper_2206_08720_amd.ntk import compute_static
    from tests.gpu_helpers import to_dev
    if call == "jacobian":
        spec = wl.fcn_spec("disj", 96, [256], 10, bias=True)
        n1, n2 = 24, 16
    else:
        spec = wl.cnn_layers_spec("disj", (8, 8), 8, [(C3, 64, "relu", True), (POOL,)], 10)
        n1, n2 = 40, 24
    params = wl.make_params(spec, 81, "2/fan_in")
    X1, X2 = np.abs(wl.make_inputs(spec, n1, 82)), np.abs(wl.make_inputs(spec, n2, 83))
    _disjoint(params, X1, X2)
    ref = oracle.ntk_jc(spec, params, X1, X2, layer_storage=S)
    print(f"[pair] fp32 {call}", flush=True)
    if call == "jacobian":
        got = gpu_ntk(spec, params, X1, X2, options={_lib.NTK_OPT_METHOD: _lib.NTK_METHOD_JACOBIAN})
    else:
        got = compute_static(spec, to_dev(params), *to_dev([X1, X2]))
        torch.cuda.synchronize()
        got = got.cpu().numpy()
    err = _entry_errors(got, ref)
    print(f"[parity] fp32 {call}: entries {err:.3e}", flush=True)
    # fp32 partial sums of about 1000 columns: 1000 2^-24 at most
    assert err <= 6e-5


@pytest.mark.parametrize("kind", ["normal 0", "normal 4"])
def test_pair_conv_long_runs_of_block_diagonal_layers(kind):
    """Seven depthwise, scale and pool layers between two convolutions: the maxima are the images' own, however
    many layers lie between."""
    blocks = [(C3, 64, "relu", True), (DW, "relu", False), (SC, "relu", True), (DW, "relu", True), (SC, "relu", False),
              (POOL,), (DW, "relu", False), (SC, "relu", True), (C3, 64, "relu", False), (C3, 64, "relu", False)]
    _conv_check(f"long run {kind}", ((24, 20), blocks, 44, 30), lambda spec, params: rescale_cnn(spec, params, kind, 99))
