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
    prof = {}
    got = gpu_ntk(spec, params, X1, X2, variant=variant, profile=prof)
    # the case is here for the pair kernels: a retuned dispatch must not empty it
    assert "dense_bwd_pair" in prof and ("ntk_fcn_pair" in prof) == (variant == ("full", "full", 0))
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
    ("100 outputs, few samples", [200, 140], 100, 17, 13, "erf", False),
    ("stream-K tiles", [133, 160], 10, 300, 301, "relu", False),
    # from 512 tiles of 128 x 128 on; the Gram block of a tile does not fit in LDS beside the stages
    ("stream-K tiles, one output", [133, 160], 1, 2905, 2950, "relu", True),
    ("stream-K tiles, two outputs", [160, 130], 2, 1460, 1461, "erf", False),
    ("stream-K tiles, three outputs", [160, 130], 3, 970, 981, "relu", False),
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
    n = 640 if variant[0] == "logit" else 257   # one output's rows are few
    X1, X2 = wl.make_inputs(spec, n, 45), wl.make_inputs(spec, n, 46)
    _check("variants", spec, params, X1, X2, variant)


def test_pair_rows_magnitudes():
    """Outputs and whole layers whose weights differ by powers of two up to 2^40, and dead units (rows of
    zeros): every row has an exponent of its own.  (Units of different scales: test_gpu_pair_scales.py.)"""
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


# ---- convolutions: the cotangent backward and the weight-space products on pairs -----------------
# Tolerance as above: a backward product sums 9 Cout terms (576: 108 roundings of 2^-24, 6.4e-6, and
# 4e-7), at most three of them in a row, the weight-space product D terms (480 pixels: 5.4e-6), then
# J1 J2^T, on pairs as well or in fp32 (worst case K 2^-24 on sums of random sign; 1e-5 allowed here).
CONV_TOL = 3 * 6.8e-6 + 5.8e-6 + 1e-5


def _conv_check(name, spec, params, X1, X2, variant=("full", "full", 0), classes=("conv_bwd_pair", "conv_wgrad_pair")):
    print(f"[pair] {name} {variant}", flush=True)
    prof = {}
    got = gpu_ntk(spec, params, X1, X2, variant=variant, profile=prof)
    assert {k for k in prof if k in ("conv_bwd_pair", "conv_wgrad_pair")} == set(classes)
    ref, d1, d2 = oracle.ntk_jc_with_norms(spec, params, X1, X2, layer_storage=S)
    if variant == ("full", "full", 0):
        cs, nw = errors(got, ref, d1, d2)
    else:
        cs, nw = scaled_errors(got, variant_of(ref, *variant), variant_scale(d1, d2, *variant))
    report(name, cs, nw)
    assert cs <= CONV_TOL and nw <= CONV_TOL


C3 = "conv3x3"
CONV_CASES = [
    # odd image (rows of a tile straddle images, the halo is not whole tiles), biases
    ("21x19, 64 channels", (21, 19), 3, [(C3, 64, "relu", True), (C3, 64, "relu", True), (C3, 64, "relu", False)],
     10, 14, 9),
    # image rows that are whole K tiles; 96 and 36 channels (36: no pair backward behind it)
    ("12x32, 96 and 36 channels", (12, 32), 4, [(C3, 96, "erf", False), (C3, 36, "relu", True), (C3, 64, "relu", False)],
     9, 13, 9),
    # the widest image the halo holds, and one beyond it
    ("5x63", (5, 63), 8, [(C3, 64, "relu", False), (C3, 64, "relu", False), (C3, 64, "relu", True)], 10, 18, 13),
    ("6x66", (6, 66), 3, [(C3, 64, "relu", False), (C3, 64, "relu", False), (C3, 64, "relu", True)], 10, 40, 21),
    # bounds through depthwise, scale and pool layers, pointwise layers
    ("struct 24x20", (24, 20), 3, [(C3, 64, "relu", True), ("dwconv3x3", "erf", True), ("conv1x1", 64, "relu", True),
                                   ("avgpool2",), ("scale", "relu", True), (C3, 64, "relu", True),
                                   ("scale", "erf", False), (C3, 64, "relu", False)], 10, 40, 21),
    # channels that are no multiple of 32, 4 or anything, scalar loads in each operand's place
    ("30x26, 24, 47 and 33 channels", (30, 26), 1, [(C3, 24, "erf", True), (C3, 47, "erf", True), ("avgpool2",),
                                                    (C3, 33, "erf", True)], 7, 31, 18),
    ("15x15, 20, 45, 36 and pointwise 13", (15, 15), 5, [(C3, 20, "relu", False), (C3, 45, "relu", True),
                                                         (C3, 36, "relu", False), ("conv1x1", 13, "relu", True),
                                                         (C3, 17, "relu", False)], 6, 21, 14),
    # small images: many per tile
    ("3x3 images", (3, 3), 5, [(C3, 60, "relu", False), (C3, 60, "erf", True)] + [(C3, 60, "relu", False)] * 4,
     10, 90, 70),
]


@pytest.mark.parametrize("case", CONV_CASES, ids=[c[0] for c in CONV_CASES])
def test_pair_conv_shapes(case):
    name, hw, cin, blocks, O, n1, n2 = case
    spec = wl.cnn_layers_spec("pairc", hw, cin, blocks, O)
    params = wl.make_params(spec, 61, "2/fan_in", bias_var=0.05)
    X1, X2 = wl.make_inputs(spec, n1, 62), wl.make_inputs(spec, n2, 63)
    # an image wider than the halo: the fp32 backward, whose maxima the weight-space products use
    classes = ("conv_wgrad_pair",) if hw[1] > 63 else ("conv_bwd_pair", "conv_wgrad_pair")
    _conv_check(name, spec, params, X1, X2, classes=classes)
    if hw == (21, 19):
        _conv_check(name, spec, params, X1, X1)
        _conv_check(name, spec, params, X1, X2, ("trace", "full", 0))


def test_pair_conv_magnitudes():
    """Images, outputs and whole layers that differ by powers of two, an image of zeros.  (Channels of
    different scales: test_gpu_pair_scales.py.)"""
    spec = wl.cnn_layers_spec("paircm", (20, 20), 3, [(C3, 64, "relu", False)] * 3, 10)
    params = wl.make_params(spec, 64, "2/fan_in")
    rng = np.random.default_rng(65)
    params[3] *= np.exp2(rng.integers(-20, 21, (10, 1))).astype(np.float32)
    params[0] *= np.float32(2.0 ** 30)
    params[1] *= np.float32(2.0 ** -45)
    X1, X2 = wl.make_inputs(spec, 13, 66), wl.make_inputs(spec, 10, 67)
    X1 *= np.exp2(rng.integers(-15, 16, (13, 1, 1, 1))).astype(np.float32)
    X2[3] = 0.0
    _conv_check("conv magnitudes", spec, params, X1, X2)


@pytest.mark.parametrize("scaling", ["growing", "shrinking", "dead channels"])
@pytest.mark.parametrize("n1,n2", [(43, 27), (40, 40)])
def test_pair_splitk_row_exponents(scaling, n1, n2):
    """J1 J2^T on pairs, whose row exponents follow the columns: 5 x 9 x 91 weight and 91 bias columns
    (scalar loads, a ragged last K tile) whose channels differ by 2^45, or are zero at first."""
    spec = wl.cnn_layers_spec("pairs", (6, 6), 5, [(C3, 91, "relu", True), (C3, 40, "relu", False)], 13)
    params = wl.make_params(spec, 71, "2/fan_in", bias_var=0.05)
    f = np.exp2(np.arange(91) / 2).astype(np.float32)
    f = {"growing": f, "shrinking": f[::-1], "dead channels": (np.arange(91) > 50).astype(np.float32)}[scaling]
    params[2] *= f
    X1 = wl.make_inputs(spec, n1, 72)
    X2 = X1 if n1 == n2 else wl.make_inputs(spec, n2, 73)
    _conv_check("split-K " + scaling, spec, params, X1, X2, classes=())   # small: the other products in fp32


@pytest.mark.parametrize("case", ["layer groups", "stream-K", "trace", "convolutions"])
def test_pair_theta_of_one_batch_is_exactly_symmetric(case):
    """Theta(X, X) equals its transpose bit for bit, inside the diagonal's tiles too (the pair products
    of (r, s) and (s, r) round differently)."""
    variant = ("trace", "full", 0) if case == "trace" else ("full", "full", 0)
    if case == "convolutions":
        spec, n = wl.cnn_layers_spec("sym", (20, 20), 3, [(C3, 64, "relu", True)] * 2 + [("scale", "relu", False)], 10), 23
    else:
        spec, n = wl.fcn_spec("sym", 64, [389, 260, 515], 10, bias=True), {"layer groups": 90, "stream-K": 330, "trace": 400}[case]
    params = wl.make_params(spec, 51, "2/fan_in")
    X = wl.make_inputs(spec, n, 52)
    print(f"[pair] symmetric {case}", flush=True)
    prof = {}
    got = gpu_ntk(spec, params, X, X, variant=variant, profile=prof)
    assert any(k.endswith("_pair") for k in prof)
    assert np.array_equal(got, got.T if case == "trace" else got.transpose(1, 0, 3, 2))


def test_pair_calls_of_two_threads_with_different_outputs():
    """Two host threads, a handle and a stream each, whose contractions ask for different amounts of LDS
    (few outputs more than many): every call succeeds and repeats the result of a call alone."""
    import threading
    import torch
    from paper_2206_08720_amd.ntk import NTK
    from tests.gpu_helpers import to_dev
    jobs = []
    for O, n in ((3, 400), (3, 100), (10, 220), (10, 60)):
        spec = wl.fcn_spec("thr", 64, [389, 260], O)
        ps = to_dev(wl.make_params(spec, 53, "2/fan_in"))
        xs = to_dev([wl.make_inputs(spec, n, 54), wl.make_inputs(spec, n, 55)])
        jobs.append((spec, ps, xs, gpu_ntk(spec, [p.cpu().numpy() for p in ps], *[x.cpu().numpy() for x in xs])))
    errors = []

    def run(part):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                handles = [(NTK(spec, x1.shape[0], x2.shape[0]), ps, x1, x2, ref) for spec, ps, (x1, x2), ref in part]
                for _ in range(40):
                    for h, ps, x1, x2, ref in handles:
                        out = h.compute(ps, x1, x2)
                for h, ps, x1, x2, ref in handles:
                    out = h.compute(ps, x1, x2)
                    torch.cuda.current_stream().synchronize()
                    if not np.array_equal(out.cpu().numpy(), ref):
                        errors.append("results differ")
                    h.close()
        except Exception as e:   # reported by the test's own thread
            errors.append(repr(e))

    print("[pair] two threads", flush=True)
    threads = [threading.Thread(target=run, args=(part,)) for part in (jobs[:2], jobs[2:])]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    assert not errors, errors


def test_pair_buffers_are_planned_once_and_only_where_pairs_can_run():
    """Options allocate nothing, and a network that never takes the pair kernels (a layer below 128, or too
    small at the handle's largest batches) has no buffers for them: its workspace grows with the outputs by
    the fp32 cotangent rows alone."""
    import torch
    from paper_2206_08720_amd.ntk import NTK

    def handle(widths, O, n):
        return NTK(wl.fcn_spec("mem", 64, widths, O), n, n)

    h = handle([512, 512, 512], 100, 300)
    try:
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        for variant in (("trace", "full", 0), ("logit", "diagonal", 1), ("full", "diagonal", 0)):
            h.set_variant(*variant)
            assert torch.cuda.mem_get_info()[0] == free
    finally:
        h.close()
    for widths, n in (([256, 64, 256], 100), ([256, 128, 256], 2)):
        sizes = []
        for O in (100, 200):
            h = handle(widths, O, n)
            sizes.append(h.workspace_bytes())
            h.close()
        rows = 2 * n * 100 * sum(widths) * 4
        assert abs(sizes[1] - sizes[0] - rows) <= 4096, (widths, sizes, rows)   # (rounded to 256 bytes an array)


@pytest.mark.parametrize("variant", [("full", "full", 0), ("trace", "diagonal", 0)])
def test_pair_halves_on_two_streams_with_layers_of_different_widths(variant):
    """The two halves of the samples may be at different layers; with rows of different lengths they must not
    reach into each other's.  With per-kernel timing the forward runs on one stream: the same bits."""
    spec = wl.fcn_spec("halves", 64, [2304, 2048, 2560, 2112], 10)
    params = wl.make_params(spec, 56, "2/fan_in")
    X1, X2 = wl.make_inputs(spec, 500, 57), wl.make_inputs(spec, 500, 58)
    print(f"[pair] halves {variant}", flush=True)
    prof = {}
    ref = gpu_ntk(spec, params, X1, X2, variant=variant, profile=prof)
    assert "dense_bwd_pair" in prof
    for _ in range(3):
        assert np.array_equal(gpu_ntk(spec, params, X1, X2, variant=variant), ref)
    sub = [0, 249, 250, 499]
    full = oracle.ntk_structured_fp64(spec, params, X1[sub], X2[sub], layer_storage=S)
    d1, d2 = (oracle.ntk_structured_diag_fp64(spec, params, X[sub], layer_storage=S) for X in (X1, X2))
    got = ref[sub] if variant[1] == "diagonal" else ref[np.ix_(sub, sub)]
    cs, nw = scaled_errors(got, variant_of(full, *variant), variant_scale(d1, d2, *variant))
    report(f"halves {variant}", cs, nw)
    assert cs <= PAIR_TOL and nw <= PAIR_TOL
