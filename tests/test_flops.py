"""The analytic operation counter against the paper's cost formulas (CPU only).

The paper counts a (M,K)x(K,P) product as M*K*P multiply-adds (appendix
"Experimental Details"); the counter reports 2*M*K*P flops.  The FCN terms are
those of Section 4.1 ("FCN SD cost": N O L W^2 + N^2 O^2 L W + N^2 O^3) and the CNN
terms those of the appendix "CNN NTK Complexity" / table "complexities_cnn".
"""
import pytest

import workloads as wl
from paper_2206_08720_amd.flops import cnn_flops, fcn_flops, ntk_entries, vp_flops


def test_fcn_terms_match_section_4_1():
    N, O, L, W = 16, 7, 5, 96
    spec = wl.fcn_spec("f", W, [W] * L, O)            # input size W as in Section 4.1
    f = fcn_flops(spec, N, N)
    # contraction: the N^2 O^2 L W term (one O x O product per layer and pair)
    assert f["contraction"] == 2 * N * N * O * O * L * W
    # backward: the (N1 + N2) O (L - 1) W^2 cotangent products (the N O L W^2 term)
    assert f["backward"] == 2 * (2 * N) * O * (L - 1) * W * W
    # forward: (N1 + N2) L W^2 (no readout: f itself is not needed)
    assert f["forward"] == 2 * (2 * N) * L * W * W
    assert f["gram"] == 2 * N * N * (L + 1) * W
    sym = fcn_flops(spec, N, N, symmetric=True)
    assert sym["forward"] == f["forward"] / 2 and sym["backward"] == f["backward"] / 2
    # the symmetric schedule contracts the N (N + 1) / 2 pairs n1 <= n2
    assert sym["contraction"] == 2 * (N * (N + 1) // 2) * O * O * L * W
    assert sym["gram"] == f["gram"]


def test_workload_totals():
    spec, _, X1, X2 = wl.make_workload("relu_mlp_d8_w2048")
    f = fcn_flops(spec, 512, 512)
    assert f["total"] == pytest.approx(1.5435e12, rel=1e-4)
    assert f["contraction"] == pytest.approx(8.59e11, rel=1e-3)
    assert ntk_entries(spec, 512, 512) == 512 * 512 * 100
    spec, _, _, _ = wl.make_workload("cnn4_c64_32x32")
    c = cnn_flops(spec, 64, 64)
    assert c["total"] == pytest.approx(5.89e11, rel=1e-3)


def test_cnn_terms_match_complexities_cnn():
    N, O, D, W, Fs = 4, 5, 36, 8, 9
    spec = wl.cnn_spec("c", (6, 6), W, [W, W], O)
    oi = cnn_flops(spec, N, N, order="outside_in", fold=False)
    io = cnn_flops(spec, N, N, order="inside_out")
    # outside-in: N^2 O^2 F W^2 per layer for J1 J2^T, plus N O D F W^2 to form J
    assert oi["contraction"] == 2 * (N * O) * (N * O) * 2 * Fs * W * W
    assert oi["wgrad"] == 2 * (2 * N) * O * W * Fs * W * D * 2
    # the library's schedule folds the last convolution (its cotangent is the readout's through
    # the global pool): O-free rows A [2N, W, F W], per-channel Grams of the N^2 pairs and their
    # O x O sums over the W channels, and no J columns of that layer
    fo = cnn_flops(spec, N, N, order="outside_in")
    assert fo["wgrad"] == 2 * (2 * N) * O * W * Fs * W * D + 2 * (2 * N) * W * Fs * W * D
    assert fo["contraction"] == 2 * (N * O) * (N * O) * Fs * W * W
    assert fo["gram"] == 2 * N * N * W + 2 * N * N * W * Fs * W + 3 * N * N * O * O * W
    assert fo["forward"] == oi["forward"] and fo["backward"] == oi["backward"]
    # inside-out: N^2 (D^2 F W + O D^2 W + O^2 D W) multiply-adds per layer in the paper's table;
    # here the patch-pair Gram comes from the pixel Gram (D^2 W) and F D^2 tap sums; no J columns
    assert io["pairsum"] == 2 * N * N * (2 * D * D * W + Fs * D * D + 2 * O * D * D * W + 2 * O * O * D * W)
    assert io["contraction"] == 0 and "wgrad" not in io


def test_auto_order_is_the_cost_model():
    """order="auto" mirrors the library's per-layer choice: on 4x4 images the 64->64
    convolutions go inside-out (several times cheaper than outside-in), except the last one,
    whose fold (its O outputs out of its weight-space product) is cheaper still; the 3-channel
    one stays outside-in; on 32x32 images every layer stays outside-in."""
    spec, _, _, _ = wl.make_workload("cnn4_c64_4x4")
    N, O, D, W = 64, 10, 16, 64
    io1 = N * N * (2 * D * D * W + 9 * D * D + 2 * O * D * D * W + 2 * O * O * D * W)
    plain = cnn_flops(spec, N, N, order="auto", fold=False)
    assert plain["pairsum"] == 3 * io1
    assert plain["contraction"] == 2 * N * N * O * O * 9 * 3 * W
    assert plain["wgrad"] == 2 * (2 * N) * O * W * 9 * 3 * D
    oi = cnn_flops(spec, N, N, order="outside_in", fold=False)
    assert oi["contraction"] + oi["wgrad"] > 8 * (plain["pairsum"] + plain["contraction"] + plain["wgrad"])
    a = cnn_flops(spec, N, N, order="auto")
    assert a["pairsum"] == 2 * io1
    assert a["contraction"] == 2 * N * N * O * O * 9 * 3 * W
    assert a["wgrad"] == 2 * (2 * N) * O * W * 9 * 3 * D + 2 * (2 * N) * W * 9 * W * D
    assert a["gram"] == 2 * N * N * W + 2 * N * N * W * 9 * W + 3 * N * N * O * O * W
    # the fold's cost (multiply-adds) against the last layer's inside-out cost
    assert 2 * N * D * 9 * W * W + N * N * (9 * W * W + O * O * W) < io1 / 2
    spec, _, _, _ = wl.make_workload("cnn4_c64_32x32")
    assert cnn_flops(spec, 64, 64, order="auto") == cnn_flops(spec, 64, 64, order="outside_in")


def test_variant_counts():
    N, O, L, W = 16, 7, 5, 96
    spec = wl.fcn_spec("f", W, [W] * L, O)
    full = fcn_flops(spec, N, N)
    tr = fcn_flops(spec, N, N, output="trace")
    lg = fcn_flops(spec, N, N, output="logit")
    dg = fcn_flops(spec, N, N, batch="diagonal")
    assert tr["contraction"] == full["contraction"] / O and tr["backward"] == full["backward"]
    assert lg["contraction"] == full["contraction"] / O ** 2 and lg["backward"] == full["backward"] / O
    assert dg["contraction"] == full["contraction"] / N and dg["gram"] == full["gram"] / N
    assert ntk_entries(spec, N, N, "trace") == N * N and ntk_entries(spec, N, N, "full", "diagonal") == N * O * O
    cs = wl.cnn_spec("c", (4, 4), 3, [8, 8], O)
    cf, cl = cnn_flops(cs, N, N, fold=False), cnn_flops(cs, N, N, output="logit")
    assert cl["wgrad"] == cf["wgrad"] / O and cl["contraction"] == cf["contraction"] / O ** 2
    # one logit: nothing to fold (its backward has one output already)
    assert cnn_flops(cs, N, N, output="logit", fold=False) == cl
    # the trace folds the last convolution like the full output, with one weighted sum per pair
    ct = cnn_flops(cs, N, N, output="trace")
    ctu = cnn_flops(cs, N, N, output="trace", fold=False)
    M, D, F, cin, cout = 2 * N, 16, 9, 8, 8
    assert ctu["wgrad"] - ct["wgrad"] == 2 * M * (O - 1) * cout * F * cin * D
    assert ct["gram"] - ctu["gram"] == 2 * N * N * cout * F * cin + 2 * O * cout + 2 * N * N * cout
    assert ctu["contraction"] - ct["contraction"] == 2 * N * N * O * F * cin * cout
    # and on the batch diagonal: the per-channel Grams of the N pairs (n, n) only
    cd = cnn_flops(cs, N, N, batch="diagonal")
    cdu = cnn_flops(cs, N, N, batch="diagonal", fold=False)
    assert cdu["wgrad"] - cd["wgrad"] == 2 * M * (O - 1) * cout * F * cin * D
    assert cd["gram"] - cdu["gram"] == 2 * N * cout * F * cin + 3 * N * O * O * cout


def test_jacobian_contraction_count_is_the_papers_n2_o2_p():
    import oracle
    from paper_2206_08720_amd.flops import ntk_flops, param_total
    for name in ("relu_mlp_d8_w2048", "cnn4_c64_32x32", "tiny_relu_mlp"):
        spec, params, X1, X2 = wl.make_workload(name)
        assert param_total(spec) == oracle.param_count(spec)
        n1, n2, O = X1.shape[0], X2.shape[0], spec["layers"][-1]["out"]
        jc = ntk_flops(spec, n1, n2, method="jacobian")
        assert jc["contraction"] == 2 * n1 * n2 * O * O * oracle.param_count(spec)
    spec, _, _, _ = wl.make_workload("relu_mlp_d8_w2048")
    assert ntk_flops(spec, 512, 512, method="jacobian")["contraction"] == pytest.approx(1.87e15, rel=1e-2)


def test_structured_layer_kinds_counts():
    import oracle
    from paper_2206_08720_amd.flops import ntk_flops, param_total
    N, O = 3, 4
    spec = wl.cnn_layers_spec("s", (4, 6), 2, [("conv3x3", 8, "relu", True), ("avgpool2",),
                                               ("dwconv3x3", "erf", True), ("scale", "none", False)], O)
    f = cnn_flops(spec, N, N)
    M, D0, D1 = 2 * N, 24, 6
    # the conv (with its bias in the epilogue), then the pool, depthwise (+ bias) and scale
    assert f["forward"] == 2 * M * D0 * 9 * 2 * 8 + M * D0 * 8
    assert f["struct_forward"] == M * D0 * 8 + 2 * M * D1 * 9 * 8 + M * D1 * 8 + M * D1 * 8
    assert f["backward"] == 0
    assert f["struct_backward"] == M * O * D0 * 8 + 2 * M * O * D1 * 9 * 8 + M * O * D1 * 8
    assert f["wgrad"] == 2 * M * O * 8 * 9 * 2 * D0
    assert f["struct_wgrad"] == M * O * D0 * 8 + 2 * M * O * D1 * 9 * 8 + M * O * D1 * 8 \
        + 2 * M * O * D1 * 8
    # J columns: 9 Cin Cout + Cout (conv and its bias), 9 C + C (depthwise and bias), C (scale)
    assert f["contraction"] == 2 * N * N * O * O * (9 * 2 * 8 + 8 + 9 * 8 + 8 + 8)
    assert param_total(spec) == oracle.param_count(spec) == 9 * 2 * 8 + 8 + 9 * 8 + 8 + 8 + 8 * O
    jc = ntk_flops(spec, N, N, method="jacobian")
    assert jc["contraction"] == 2 * N * N * O * O * oracle.param_count(spec)


def test_pointwise_counts():
    import oracle
    from paper_2206_08720_amd.flops import param_total
    N, O = 2, 3
    spec = wl.cnn_layers_spec("pw", (2, 4), 3, [("conv1x1", 6, "relu", True), ("dwconv3x3", "relu", False),
                                               ("conv1x1", 5, "erf", False)], O)
    f = cnn_flops(spec, N, N, fold=False)
    M, D = 2 * N, 8
    assert f["forward"] == 2 * M * D * 3 * 6 + M * D * 6 + 2 * M * D * 6 * 5
    assert f["backward"] == 2 * M * O * D * 5 * 6
    assert f["wgrad"] == 2 * M * O * 6 * 3 * D + 2 * M * O * 5 * 6 * D
    assert f["contraction"] == 2 * N * N * O * O * (3 * 6 + 6 + 9 * 6 + 6 * 5)
    # folded last pointwise convolution (5 channels of 6 inputs): O-free rows, no J columns
    g = cnn_flops(spec, N, N)
    assert g["wgrad"] == 2 * M * O * 6 * 3 * D + 2 * M * 5 * 6 * D
    assert g["contraction"] == 2 * N * N * O * O * (3 * 6 + 6 + 9 * 6)
    assert g["gram"] == 2 * N * N * 5 + 2 * N * N * 5 * 6 + 3 * N * N * O * O * 5
    assert param_total(spec) == oracle.param_count(spec)


def test_vector_product_counts_the_cheaper_form():
    """One hidden layer of 8 -> 6 -> 2: through the Grams for 2 + 3 samples, through the weights for 50 + 60."""
    spec = wl.fcn_spec("vp", 8, [6], 2)
    tangents = {n1: 2.0 * n1 * 6 * 2 for n1 in (2, 50)}
    assert vp_flops(spec, 2, 3)["gram_products"] == 2.0 * 2 * 3 * (8 + 6 + 6 + 2) + tangents[2]
    assert vp_flops(spec, 50, 60)["gram_products"] == 2.0 * 110 * (8 * 6 + 6 * 2) + tangents[50]
