"""GPU parity of the kernels that layer calls run where the wide kernel does not:
w4a4_linear and, for convolutions, w4a4_gemm, with whole tiles, with tiles cut
along K among fewer tiles than workgroups, and with only the last rounds of
more tiles cut.  Every mode, ragged M and N, every G_s, GELU, no bias, strided
outputs.  Each case first asserts, through the library's query, that its call
launches the kernel and the split it is meant for (on 256 compute units).
Sampled rows and columns against the oracle within the tolerance of
tests/helpers.py; nothing outside y written; a second call and one whose
workspace slots hold NaNs give the same bits, and the counters are zero again;
the allocation-free entry point gives the workspace one's bits, and the
quantized output those of quantizing the bf16 one."""
import numpy as np
import pytest

import oracle
from helpers import bf16_bits_to_f64, to_host_u16, y_tolerance

pytestmark = pytest.mark.gpu


def _q():
    import paper_2509_26436_amd as q
    return q


def _inputs(seed, M, Cin, N, K, outliers=6):
    """Heavy-tailed activations with outlier channels, weights, bias (bf16)."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    x = rnd(M, Cin) / torch.sqrt((rnd(M, Cin) ** 2 + rnd(M, Cin) ** 2 + rnd(M, Cin) ** 2) / 3) * 0.05
    x[:, torch.randperm(Cin, generator=g, device="cuda")[:outliers]] *= 30.0
    return x.bfloat16(), (rnd(N, K) * 0.02).bfloat16(), (rnd(N) * 0.02).bfloat16()


def _sample(n, tile, seed):
    """Both ends, both sides of the first and last tile boundaries, random ones."""
    last = n // tile * tile
    fixed = {0, 1, n - 1, n - 2, tile - 1, tile, last - 1, last, 31, 32, 63, 64}
    rest = np.random.Generator(np.random.PCG64(seed)).choice(n, size=min(n, 24), replace=False)
    return np.array(sorted({i for i in fixed if 0 <= i < n} | set(int(i) for i in rest)), np.int64)


def _host(t):
    return to_host_u16(t.contiguous())


def _assert_kernel(layer, M, N, K, gs, epi, use_ws, kernel, split, over):
    import torch
    q = _q()
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        return
    k = q.layer_kernel(M, N, K, gs, layer, epi, use_ws)
    assert (k["kernel"], k["split"]) == (kernel, split), f"the case no longer reaches {kernel}: {k}"
    s, _ = q.linear_schedule(M, N, K, 256, use_ws, 0 if kernel == "linear" else 1)
    assert not split or (s["sk_first"] + s["sk_tiles"] > 256) == over


def _counters_zero(ws, M, N, K, tiles):
    import torch
    s, _ = _q().linear_schedule(M, N, K, torch.cuda.get_device_properties(0).multi_processor_count, True, tiles)
    n = -(-s["sk_tiles"] * 8 * 4 // 256) * 256
    return n, not bool(ws[:n].any())


# (layer, split, more tiles than workgroups, M, N, K, gs, epilogue, bias, extra columns)
CASES = [
    ("linear", True, False, 995, 1080, 8768, 8, 0, True, 0),
    ("linear", True, False, 836, 1166, 9600, 16, 1, True, 6),
    ("linear", True, False, 367, 2734, 9536, 32, 0, False, 0),
    ("linear", True, False, 740, 1773, 11392, 64, 1, True, 3),
    ("linear", True, True, 4769, 3449, 7232, 8, 0, True, 0),
    ("linear", False, False, 5789, 1074, 2752, 8, 1, True, 0),
    ("linear", False, False, 3052, 2193, 5184, 16, 0, True, 7),
    ("linear", False, False, 2824, 2406, 3904, 32, 0, False, 2),
    ("linear", False, False, 3303, 1833, 6336, 64, 1, True, 0),
    ("quantize", True, False, 359, 2816, 8128, 8, 0, True, 0),
    ("quantize", True, False, 333, 3008, 11712, 16, 1, True, 0),
    ("quantize", True, False, 4582, 256, 8896, 32, 0, False, 0),
    ("quantize", True, False, 396, 2496, 11968, 64, 0, True, 0),
    ("quantize", True, True, 4744, 3456, 5376, 8, 1, True, 0),
    ("quantize", False, False, 2145, 2176, 1728, 8, 0, True, 0),
    ("quantize", False, False, 2029, 2752, 3392, 16, 0, True, 0),
    ("quantize", False, False, 3163, 1344, 3136, 32, 0, False, 0),
    ("quantize", False, False, 2458, 1792, 3392, 64, 0, True, 0),
    ("static", True, False, 654, 1686, 12096, 8, 1, True, 5),
    ("static", True, False, 878, 1223, 12032, 16, 0, True, 0),
    ("static", True, False, 471, 2097, 11072, 64, 0, False, 0),
    ("static", False, False, 1050, 4036, 3008, 8, 0, True, 4),
    ("static", False, False, 4183, 1493, 4672, 16, 0, True, 0),
    ("static", False, False, 5179, 1361, 4032, 32, 1, False, 0),
    ("static", False, False, 4093, 1294, 4160, 64, 0, True, 0),
    ("asym", True, False, 631, 1836, 8576, 8, 0, True, 0),
    ("asym", True, False, 4753, 217, 8896, 16, 1, True, 1),
    ("asym", True, False, 726, 1506, 8128, 32, 0, False, 0),
    ("asym", True, False, 2073, 473, 8320, 64, 1, True, 0),
    ("asym", True, True, 2326, 3544, 8000, 64, 0, True, 0),
    ("asym", True, True, 5161, 3096, 4288, 16, 0, True, 0),
    ("asym", False, False, 2700, 2222, 4160, 8, 1, True, 0),
    ("asym", False, False, 4180, 1518, 7104, 16, 1, False, 2),
    ("asym", False, False, 1866, 3693, 4416, 32, 1, True, 0),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}-{'over' if c[2] else 'split' if c[1] else 'whole'}-"
                         f"{c[3]}x{c[4]}x{c[5]}-gs{c[6]}")
def test_linear_kernel(case):
    import torch
    q = _q()
    layer, split, over, M, N, K, gs, epi, with_bias, pad = case
    print(f"linear kernel {case}", flush=True)
    _assert_kernel(layer, M, N, K, gs, epi, True, "linear", split, over)
    if layer == "quantize" and split:            # so does the bf16 output it is compared with
        _assert_kernel("linear", M, N, K, gs, epi, True, "linear", split, over)
    x, w, bias = _inputs(M + N + K, M, K, N, K)
    bias = bias if with_bias else None
    rows, cols = _sample(M, 128, M), _sample(N, 256, N)
    xr, wc = _host(x[rows.tolist()]), _host(w[cols.tolist()])
    bc = None if bias is None else _host(bias[cols.tolist()])
    ws = q.gemm_workspace(M, N, K, "cuda")
    assert not split or ws is not None
    if layer == "static":
        s = float(np.float32(float(x.abs().max()) * 0.9 / 127))
        a, pw = q.quantize_act_static(x, s, gs), q.pack_weight_per_channel(w)
        call = lambda out: q.w4a4_linear_static(a, pw, s, bias, epi, out=out, workspace=ws)
        y64, S = oracle.linear_static_f64(oracle.quantize_act_static(xr, s, gs), s,
                                          *oracle.quantize_weight_per_channel(wc), bc, epi)
    elif layer == "asym":
        a, pw = q.quantize_act(x, gs, mode=q.MODE_ASYMMETRIC), q.pack_weight(w)
        sums = q.weight_group_sums(pw)
        call = lambda out: q.w4a4_linear_asym(a, pw, sums, bias, epi, out=out, workspace=ws)
        y64, S = oracle.linear_asym_f64(oracle.quantize_act_asym(xr, gs), *oracle.quantize_weight(wc), bc, epi)
    else:
        a, pw = q.quantize_act(x, gs), q.pack_weight(w)
        call = lambda out: q.w4a4_linear(a, pw, bias, epi, out=out, workspace=ws)
        y64, S = oracle.linear_f64(oracle.quantize_act(xr, gs), *oracle.quantize_weight(wc), bc, epi)
    buf = torch.full((M + 40, N + pad), 5.0, dtype=torch.bfloat16, device="cuda")
    out = buf[:M, :N]
    call(out)
    torch.cuda.synchronize()
    assert torch.all(buf[M:] == 5.0) and torch.all(buf[:M, N:] == 5.0), "wrote outside y"
    got = bf16_bits_to_f64(_host(out[rows.tolist()][:, cols.tolist()]))
    err, tol = np.abs(got - y64), y_tolerance(y64, S, K, gelu=epi == 1)
    assert (err <= tol).all(), f"{(err > tol).sum()} outputs out of tolerance; worst excess {(err - tol).max():.3e}"
    y = out.clone()
    if split:
        n, zero = _counters_zero(ws, M, N, K, 0)
        assert zero, "counters not zero after the call"
        ws[n:] = 0xFF                            # NaN slots
    call(out)
    torch.cuda.synchronize()
    assert torch.equal(out, y)
    if layer == "linear" and split:
        alone = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
        q.w4a4_linear_noalloc(a, pw, alone, bias, epi)
        torch.cuda.synchronize()
        assert torch.equal(alone, y)
    if layer == "quantize":
        want = q.quantize_act(y.contiguous(), 16)
        fields = ("codes", "flags", "scales")
        guarded = {f: torch.full((getattr(want, f).nbytes + 4096,), 0xA5, dtype=torch.uint8, device="cuda") for f in fields}
        h = q.QuantizedAct(**{f: b[:-4096].view(getattr(want, f).dtype).view(getattr(want, f).shape)
                              for f, b in guarded.items()}, zeros=None, M=M, K=N, lzs_group=16)
        for _ in range(2):
            q.w4a4_linear_quantize(a, pw, bias, epi, 16, out=h, workspace=ws)
            torch.cuda.synchronize()
            for f in fields:
                assert torch.equal(getattr(h, f), getattr(want, f)), f
                assert torch.all(guarded[f][-4096:] == 0xA5), f"wrote past {f}"


# (static, split, images, H, W, C, N, gs, epilogue, bias, extra columns)
CONVS = [
    (False, True, 2, 47, 44, 896, 209, 8, 0, True, 3),
    (False, True, 1, 35, 33, 896, 861, 16, 0, True, 0),
    (False, True, 1, 31, 47, 896, 710, 32, 1, False, 0),
    (False, True, 3, 27, 30, 960, 390, 64, 0, True, 2),
    (False, False, 1, 67, 72, 256, 1586, 8, 1, True, 0),
    (False, False, 1, 48, 47, 320, 1838, 16, 1, True, 2),
    (False, False, 2, 38, 41, 320, 1316, 32, 0, False, 0),
    (False, False, 1, 25, 107, 320, 1708, 64, 1, True, 4),
    (True, True, 1, 43, 33, 1152, 708, 8, 0, True, 0),
    (True, True, 1, 35, 34, 1152, 834, 32, 0, True, 6),
    (True, True, 1, 53, 27, 1216, 742, 64, 0, False, 0),
]


@pytest.mark.parametrize("case", CONVS, ids=lambda c: f"{'static' if c[0] else 'plain'}-{'split' if c[1] else 'whole'}-"
                         f"{c[2]}x{c[3]}x{c[4]}x{c[5]}-{c[6]}-gs{c[7]}")
def test_gemm_kernel_convolution(case):
    import torch
    import torch.nn.functional as F
    q = _q()
    static, split, B, H, Wd, C, N, gs, epi, with_bias, pad = case
    M, K = B * H * Wd, 9 * C
    print(f"conv {case} M={M} K={K}", flush=True)
    _assert_kernel("conv3x3_static" if static else "conv3x3", M, N, K, gs, epi, True, "gemm", split, False)
    x, w, bias = _inputs(M + N + C, M, C, N, K)
    bias = bias if with_bias else None
    padded = F.pad(x.view(B, H, Wd, C), (0, 0, 1, 1, 1, 1))
    im2col = torch.cat([padded[:, i:i + H, j:j + Wd] for i in range(3) for j in range(3)], 3).reshape(M, K)
    rows, cols = _sample(M, 256, M), _sample(N, 128, N)
    xr, wc = _host(im2col[rows.tolist()]), _host(w[cols.tolist()])
    bc = None if bias is None else _host(bias[cols.tolist()])
    ws = q.gemm_workspace(M, N, K, "cuda")
    if static:
        s = float(np.float32(float(x.abs().max()) * 0.9 / 127))
        a, pw = q.quantize_act_static(x, s, gs), q.pack_weight_per_channel(w)
        call = lambda out: q.w4a4_conv3x3_static(a, pw, s, B, H, Wd, bias, epi, out=out, workspace=ws)
        y64, S = oracle.linear_static_f64(oracle.quantize_act_static(xr, s, gs), s,
                                          *oracle.quantize_weight_per_channel(wc), bc, epi)
    else:
        a, pw = q.quantize_act(x, gs), q.pack_weight(w)
        call = lambda out: q.w4a4_conv3x3(a, pw, B, H, Wd, bias, epi, out=out, workspace=ws)
        y64, S = oracle.linear_f64(oracle.quantize_act(xr, gs), *oracle.quantize_weight(wc), bc, epi)
    buf = torch.full((M + 40, N + pad), 5.0, dtype=torch.bfloat16, device="cuda")
    out = buf[:M, :N]
    call(out)
    torch.cuda.synchronize()
    assert torch.all(buf[M:] == 5.0) and torch.all(buf[:M, N:] == 5.0), "wrote outside y"
    got = bf16_bits_to_f64(_host(out[rows.tolist()][:, cols.tolist()]))
    err, tol = np.abs(got - y64), y_tolerance(y64, S, K, gelu=epi == 1)
    assert (err <= tol).all(), f"{(err > tol).sum()} outputs out of tolerance; worst excess {(err - tol).max():.3e}"
    y = out.clone()
    if split:
        n, zero = _counters_zero(ws, M, N, K, 1)
        assert zero, "counters not zero after the call"
        ws[n:] = 0xFF
    call(out)
    torch.cuda.synchronize()
    assert torch.equal(out, y)
    if not split:                                # the linear layer adds in the same order: equal bit for bit
        want = q.w4a4_linear(q.quantize_act(im2col.contiguous(), gs), pw, bias, epi)
        whole = q.w4a4_conv3x3(a, pw, B, H, Wd, bias, epi)
        torch.cuda.synchronize()
        assert torch.equal(whole, want)
