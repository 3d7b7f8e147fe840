"""The kernel that each layer call launches, by the library's own query (host
only): which calls run the wide kernel and which their other kernel, and that
layers whose outputs are promised equal bit for bit (the quantized output and
the bf16 one; a convolution and the linear layer on its im2col matrix, when
nothing is split) add the groups of an output in the same order."""
import ctypes
import math
import random

import pytest

import paper_2509_26436_amd as q

GS = (8, 16, 32, 64)


def _order(k):
    """Order of an output's group sum: ascending, by teams, or by a split of its own."""
    return ("split", k["kernel"]) if k["split"] else k["teams"]


def _shapes(seed, count, K_unit=64):
    rng = random.Random(seed)
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    for _ in range(count):
        M, K = log(1, 18432), K_unit * log(1, 12288 // K_unit)
        N = 64 * log(1, 192)
        yield M, N, K, rng.choice(GS), rng.randint(0, 1), rng.random() < 0.5


def test_full_size_layers_run_the_wide_kernel():
    for layer, M, K, N in (("linear", 4608, 3072, 9216), ("linear", 4608, 12288, 3072), ("asym", 4608, 3072, 3072),
                           ("static", 4608, 3072, 12288), ("quantize", 18432, 3072, 12288)):
        k = q.layer_kernel(M, N, K, layer=layer, epilogue=int(layer in ("static", "quantize")))
        assert k["kernel"] == "wide" and k["cols"] == 256 and k["teams"] == 1 and not k["split"], (layer, k)
    k = q.layer_kernel(256, 1152, 1152)
    assert (k["rows"], k["cols"], k["teams"]) == (64, 64, 4)


def test_other_kernel_follows_its_schedule():
    for M, N, K, gs, epi, split in _shapes(1, 400):
        for layer, tiles in (("linear", 0), ("static", 0), ("asym", 0)):
            k = q.layer_kernel(M, N, K, gs, layer, epi, split)
            if k["kernel"] == "wide":
                assert k["teams"] * k["cols"] == 256 and k["rows"] <= k["cols"] and not k["split"]
                continue
            s, _ = q.linear_schedule(M, N, K, 256, split, tiles)
            assert k == {"kernel": "linear", "rows": 128, "cols": 256, "teams": 1, "split": s["split"] == 1}
    for M, N, K, gs, epi, split in _shapes(2, 400, 576):
        for layer in ("conv3x3", "conv3x3_static"):
            k = q.layer_kernel(M, N, K, gs, layer, epi, split)
            if k["kernel"] != "wide":
                s, _ = q.linear_schedule(M, N, K, 256, split, 1)
                assert k == {"kernel": "gemm", "rows": 256, "cols": 128, "teams": 1, "split": s["split"] == 1}


@pytest.mark.parametrize("seed,K_unit", [(3, 64), (4, 576)])
def test_quantized_output_adds_in_the_order_of_the_bf16_one(seed, K_unit):
    for M, N, K, gs, epi, split in _shapes(seed, 2000, K_unit):
        a, b = (q.layer_kernel(M, N, K, gs, layer, epi, split) for layer in ("linear", "quantize"))
        assert _order(a) == _order(b), (M, N, K, gs, epi, split, a, b)


def test_unsplit_convolution_adds_in_the_order_of_the_linear_layer():
    """(The static setting's sums are exact integers in any order up to K = 21376.)"""
    for M, N, K, gs, epi, split in _shapes(5, 2000, 576):
        splits = any(q.linear_schedule(M, N, K, 256, split, t)[0]["split"] for t in (0, 1))
        if splits:
            continue
        a, b = (q.layer_kernel(M, N, K, gs, layer, epi, split) for layer in ("linear", "conv3x3"))
        assert _order(a) == _order(b), (M, N, K, gs, epi, split, a, b)


def test_arguments():
    out = (ctypes.c_int32 * 5)()
    call = lambda *a: q.quartz_w4a4_layer_kernel(*a, ctypes.addressof(out))
    assert call(256, 256, 576, 16, 0, 4, 1, 256) == 0
    for bad, status in (((0, 256, 576, 16, 0, 0, 1, 256), 2), ((256, 256, 100, 16, 0, 0, 1, 256), 2),
                        ((256, 256, 576, 16, 0, 0, 1, 0), 2), ((256, 100, 576, 16, 0, 1, 1, 256), 2),
                        ((256, 256, 640, 16, 0, 4, 1, 256), 2), ((256, 256, 576, 4, 0, 0, 1, 256), 3),
                        ((256, 256, 576, 16, 2, 0, 1, 256), 3), ((256, 256, 576, 16, 0, 6, 1, 256), 3)):
        assert call(*bad) == status, bad
    assert q.quartz_w4a4_layer_kernel(256, 256, 576, 16, 0, 0, 1, 256, None) == 1


# (layer, M, N, K, G_s, epilogue, workspace): calls that w4a4_linear runs 5 to 10 % faster than the
# wide kernel's best tile does
@pytest.mark.parametrize("case", [
    ("asym", 7107, 6667, 2432, 8, 1, True), ("asym", 8534, 10432, 3072, 16, 1, True),
    ("asym", 3722, 2560, 10752, 8, 0, True),
    ("asym", 2806, 2368, 2688, 8, 1, True), ("asym", 4042, 2027, 2752, 16, 1, True),
    ("static", 16716, 461, 11648, 8, 0, True), ("static", 3367, 1703, 1088, 8, 0, True),
    ("static", 16190, 380, 1280, 8, 0, True), ("static", 571, 12203, 1216, 8, 0, False),
], ids=lambda c: "-".join(map(str, c)))
def test_calls_that_the_other_kernel_runs_faster(case):
    layer, M, N, K, gs, epi, split = case
    assert q.layer_kernel(M, N, K, gs, layer, epi, split)["kernel"] != "wide"


# the same where the wide kernel would win for the bf16 output alone
@pytest.mark.parametrize("case", [
    (5823, 704, 4608, 16, 0, True), (3965, 5824, 11200, 8, 0, True), (14894, 1088, 5376, 8, 1, True),
    (648, 5696, 1152, 8, 0, True), (700, 11264, 6912, 16, 0, True), (15199, 1472, 11264, 8, 0, True),
    (12882, 320, 704, 64, 0, False),
], ids=lambda c: "-".join(map(str, c)))
def test_quantized_outputs_that_the_other_kernel_runs_faster(case):
    M, N, K, gs, epi, split = case
    for layer in ("linear", "quantize"):
        k = q.layer_kernel(M, N, K, gs, layer, epi, split)
        assert k["kernel"] != "wide" or (layer == "linear" and k["teams"] == 1), (layer, k)


# (layer, M, N, K, G_s, epilogue, workspace): convolutions that w4a4_gemm runs 15 to 24 % faster
# than the tile the linear layer would take
@pytest.mark.parametrize("case", [
    (8932, 120, 11520, 8, 1, True), (12540, 560, 2880, 32, 0, False), (17548, 896, 1728, 32, 0, True),
    (8588, 848, 2880, 16, 0, True), (12006, 640, 2880, 16, 0, True), (13824, 600, 8640, 16, 0, True),
    (17776, 320, 8640, 32, 0, True), (6765, 1136, 5760, 64, 0, True),
], ids=lambda c: "-".join(map(str, c)))
def test_convolutions_that_w4a4_gemm_runs_faster(case):
    M, N, K, gs, epi, split = case
    assert q.layer_kernel(M, N, K, gs, "conv3x3", epi, split)["kernel"] == "gemm"


def test_unsplit_static_convolution_past_the_exact_sums():
    """K > 21376: the static setting's fp32 sums may round, and a convolution
    and the linear layer on its im2col matrix add them in one order."""
    for M, N, K, gs, epi, split in _shapes(6, 4000, 576):
        K += 21888                               # (a multiple of 576)
        if any(q.linear_schedule(M, N, K, 256, split, t)[0]["split"] for t in (0, 1)):
            continue
        a, b = (q.layer_kernel(M, N, K, gs, layer, epi, split) for layer in ("static", "conv3x3_static"))
        assert _order(a) == _order(b), (M, N, K, gs, epi, split, a, b)
