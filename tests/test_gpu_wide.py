"""GPU parity of the wide kernel (tiles of 32 TR rows by 32 WN columns, whose
8 / WN teams of waves share the 64-groups) where it can go wrong: every tile, M
inside a row tile and inside a wave's 32 rows, N inside a wave's 32 columns and
inside a panel of 64, numbers of 64-groups that leave teams with one or two
groups past the last, one and several tiles per workgroup, every G_s, in every
mode.  The dispatch picks the tile from the shape; each case names the one it is
meant for and asserts, through the library's query, that its calls take it (on
256 compute units).  Sampled rows and columns against the oracle
within the tolerance of tests/helpers.py, every output of a larger buffer
outside y untouched, the quantized output equal to quantizing the bf16 one, the
convolutions equal to the linear layer on the im2col matrix, and infinite
scales kept to their own columns."""
import dataclasses

import numpy as np
import pytest

import oracle
import workloads as W
from helpers import bf16_bits_to_f64, to_dev_bf16, to_host_u16, y_tolerance

pytestmark = pytest.mark.gpu


def _q():
    import paper_2509_26436_amd as q
    return q


def _sample(n, tile, seed):
    """Both ends, both sides of the first and last tile boundaries, random ones."""
    last = n // tile * tile
    fixed = {0, 1, n - 1, n - 2, tile - 1, tile, last - 1, last, 31, 32, 63, 64}
    rest = np.random.Generator(np.random.PCG64(seed)).choice(n, size=min(n, 24), replace=False)
    return np.array(sorted({i for i in fixed if 0 <= i < n} | set(int(i) for i in rest)), np.int64)


def _assert_tile(layer, M, N, K, gs, epi, split, tr, wn):
    import torch
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        return
    k = _q().layer_kernel(M, N, K, gs, layer, epi, split)
    assert (k["kernel"], k["rows"], k["cols"]) == ("wide", 32 * tr, 32 * wn), f"the case no longer takes its tile: {k}"


CASES = [
    # (mode, TR, WN, M, N, K, gs, epilogue, bias, extra columns of the buffer)
    ("plain", 2, 2, 303, 546, 192, 16, 0, True, 6),    # 16-byte rows do not hold: element stores
    ("plain", 2, 4, 2403, 459, 128, 16, 0, True, 6),
    ("plain", 5, 8, 8242, 776, 448, 8, 1, True, 0),    # N % 32 == 8
    ("plain", 6, 8, 8286, 1046, 256, 32, 0, False, 2),
    ("plain", 7, 8, 8126, 1291, 320, 64, 0, True, 5),
    ("plain", 8, 8, 8131, 1541, 448, 16, 1, True, 3),
    ("plain", 7, 8, 9100, 3072, 192, 16, 0, True, 0),  # two tiles per workgroup, odd groups
    ("plain", 2, 2, 68, 60, 320, 16, 0, True, 4),      # 5 groups among 4 teams
    ("plain", 2, 2, 333, 1000, 2048, 8, 1, True, 0),
    ("plain", 2, 2, 129, 72, 832, 64, 0, False, 0),    # 13 groups
    ("plain", 2, 2, 62, 196, 64, 16, 0, True, 0),      # a single group: the other teams have none
    ("plain", 2, 4, 8575, 71, 64, 16, 0, True, 0),
    ("plain", 3, 4, 8295, 135, 320, 16, 1, True, 1),
    ("plain", 4, 4, 8296, 268, 192, 32, 0, True, 0),   # 3 groups; N % 32 == 12
    ("plain", 4, 4, 8853, 269, 64, 16, 0, True, 3),
    ("plain", 4, 8, 8475, 427, 64, 8, 0, True, 3),
    ("plain", 4, 8, 3167, 1392, 128, 32, 1, True, 0),
    ("plain", 2, 4, 774, 4655, 192, 16, 0, True, 0),   # two tiles per workgroup
    ("static", 2, 4, 379, 308, 256, 16, 0, True, 4),
    ("static", 5, 8, 8296, 783, 320, 8, 1, True, 1),
    ("static", 6, 8, 8189, 1050, 448, 32, 0, False, 6),
    ("static", 7, 8, 8110, 1314, 192, 64, 0, True, 6),
    ("static", 7, 8, 16300, 1600, 64, 16, 0, True, 0), # a single group
    ("static", 8, 8, 8123, 1562, 64, 16, 0, True, 6),
    ("static", 2, 2, 181, 64, 320, 8, 1, True, 0),
    ("static", 3, 4, 8846, 129, 64, 16, 0, True, 3),
    ("static", 4, 4, 8277, 264, 448, 64, 0, False, 0),
    ("static", 4, 4, 8341, 258, 64, 32, 0, True, 6),
    ("static", 4, 8, 5740, 683, 128, 16, 0, True, 1),
    ("asym", 2, 2, 424, 386, 320, 8, 0, True, 6),
    ("asym", 5, 8, 8301, 773, 320, 16, 1, True, 3),
    ("asym", 6, 8, 8205, 1030, 192, 32, 0, False, 2),
    ("asym", 7, 8, 8214, 1287, 256, 64, 0, True, 1),
    ("asym", 2, 2, 96, 63, 448, 16, 0, True, 1),
    ("asym", 2, 2, 65, 80, 64, 64, 1, True, 0),
    ("asym", 2, 4, 6455, 168, 128, 16, 0, True, 0),
    ("asym", 2, 4, 8225, 65, 64, 32, 1, True, 3),
    ("asym", 3, 4, 8210, 159, 192, 16, 0, True, 1),
    ("asym", 4, 4, 8208, 269, 192, 8, 0, False, 3),
    ("asym", 4, 4, 8186, 262, 64, 32, 0, True, 2),
    ("asym", 4, 8, 7874, 971, 64, 8, 1, True, 5),
    ("quantized", 2, 2, 408, 512, 256, 16, 0, True, 0),
    ("quantized", 2, 4, 1228, 832, 64, 8, 1, True, 0),
    ("quantized", 2, 4, 3167, 384, 128, 64, 0, False, 0),
    ("quantized", 5, 8, 8238, 832, 448, 8, 1, True, 0),
    ("quantized", 6, 8, 8319, 1088, 320, 32, 0, False, 0),
    ("quantized", 7, 8, 8069, 1344, 448, 64, 1, True, 0),
    ("quantized", 8, 8, 8253, 1600, 512, 16, 0, True, 0),
    ("quantized", 2, 2, 131, 64, 320, 8, 1, True, 0),
    ("quantized", 2, 2, 333, 1024, 2048, 16, 0, True, 0),
    ("quantized", 3, 4, 8196, 192, 64, 16, 1, True, 0),
    ("quantized", 4, 4, 8162, 320, 192, 32, 0, False, 0),
    ("quantized", 4, 4, 8166, 320, 64, 64, 0, True, 0),
    ("quantized", 4, 8, 8552, 448, 64, 16, 1, True, 0),
    ("quantized", 4, 8, 4702, 896, 128, 16, 0, True, 0),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}-{c[1]}x{c[2]}-{c[3]}x{c[4]}x{c[5]}-gs{c[6]}")
def test_wide_kernel_parity(case):
    import torch
    q = _q()
    mode, tr, wn, M, N, K, gs, epi, with_bias, pad = case
    print(f"wide {case}", flush=True)
    _assert_tile({"plain": "linear", "quantized": "quantize"}.get(mode, mode), M, N, K, gs, epi, True, tr, wn)
    xb = W.make_random_x(M + 3 * N + K, M, K, "t3", 0.05)
    wb = W.to_bf16_bits(np.random.Generator(np.random.PCG64(N + 5 * K)).normal(0, 0.02, (N, K)))
    bias_b = W.to_bf16_bits(np.random.Generator(np.random.PCG64(N)).normal(0, 0.02, N)) if with_bias else None
    bias = None if bias_b is None else to_dev_bf16(bias_b)
    x, w = to_dev_bf16(xb), to_dev_bf16(wb)
    buf = torch.full((M + 40, N + pad), 5.0, dtype=torch.bfloat16, device="cuda")
    out = buf[:M, :N]
    ws = q.gemm_workspace(M, N, K, "cuda")
    rows, cols = _sample(M, 32 * tr, M), _sample(N, 32 * wn, N)
    xr, wc = np.ascontiguousarray(xb[rows]), np.ascontiguousarray(wb[cols])
    bc = None if bias_b is None else np.ascontiguousarray(bias_b[cols])
    if mode == "static":
        s = float(np.abs(bf16_bits_to_f64(xb)).max() * 0.9 / 127)
        s = float(np.float32(s))
        q.w4a4_linear_static(q.quantize_act_static(x, s, gs), q.pack_weight_per_channel(w), s, bias, epi,
                             out=out, workspace=ws)
        wq, sw = oracle.quantize_weight_per_channel(wc)
        y64, S = oracle.linear_static_f64(oracle.quantize_act_static(xr, s, gs), s, wq, sw, bc, epi)
    elif mode == "asym":
        pw = q.pack_weight(w)
        q.w4a4_linear_asym(q.quantize_act(x, gs, mode=q.MODE_ASYMMETRIC), pw, q.weight_group_sums(pw), bias, epi,
                           out=out, workspace=ws)
        wq, sw = oracle.quantize_weight(wc)
        y64, S = oracle.linear_asym_f64(oracle.quantize_act_asym(xr, gs), wq, sw, bc, epi)
    else:
        qa, pw = q.quantize_act(x, gs), q.pack_weight(w)
        q.w4a4_linear(qa, pw, bias, epi, out=out, workspace=ws)
        wq, sw = oracle.quantize_weight(wc)
        y64, S = oracle.linear_f64(oracle.quantize_act(xr, gs), wq, sw, bc, epi)
    torch.cuda.synchronize()
    assert torch.all(buf[M:] == 5.0) and torch.all(buf[:M, N:] == 5.0), "wrote outside y"
    got = bf16_bits_to_f64(to_host_u16(out[rows.tolist()][:, cols.tolist()].contiguous()))
    err, tol = np.abs(got - y64), y_tolerance(y64, S, K, gelu=epi == 1)
    assert (err <= tol).all(), f"{(err > tol).sum()} outputs out of tolerance; worst excess {(err - tol).max():.3e}"
    if mode == "quantized":
        fused = q.w4a4_linear_quantize(qa, pw, bias, epi, 16, workspace=ws)
        plain = q.quantize_act(out.contiguous(), 16)
        torch.cuda.synchronize()
        for name in ("codes", "flags", "scales"):
            assert torch.equal(getattr(fused, name), getattr(plain, name)), name


@pytest.mark.parametrize("case", [
    # (static, TR, WN, batch, H, W, C, N, gs, epilogue, extra columns of the buffer)
    (False, 2, 2, 1, 9, 7, 64, 72, 16, 0, 0),          # 9 groups, an image inside one row tile
    (False, 2, 2, 3, 19, 5, 128, 700, 8, 1, 4),        # rows of a tile in two images
    (False, 2, 4, 1, 83, 99, 64, 67, 32, 1, 0),
    (False, 4, 8, 1, 45, 191, 64, 386, 8, 0, 0),       # odd groups, one team
    (False, 5, 8, 2, 65, 64, 128, 919, 64, 0, 1),
    (False, 6, 8, 2, 59, 59, 64, 1329, 8, 0, 0),
    (False, 7, 8, 1, 63, 129, 64, 1339, 32, 0, 2),
    (False, 8, 8, 2, 66, 65, 64, 1539, 16, 1, 0),
    (False, 3, 4, 1, 128, 65, 64, 135, 64, 0, 1),
    (False, 4, 4, 2, 64, 65, 128, 268, 16, 0, 0),
    (True, 2, 2, 2, 8, 11, 64, 60, 8, 1, 4),
    (True, 4, 4, 2, 64, 65, 64, 264, 16, 0, 0),
    (True, 4, 8, 1, 130, 126, 320, 320, 16, 0, 0),
    (True, 5, 8, 2, 65, 64, 64, 794, 64, 1, 0),
    (True, 6, 8, 1, 96, 96, 128, 1280, 32, 0, 0),
    (True, 7, 8, 1, 93, 90, 64, 1285, 32, 0, 3),
    (True, 8, 8, 1, 65, 129, 64, 1606, 8, 0, 0),
], ids=lambda c: f"{'static' if c[0] else 'plain'}-{c[1]}x{c[2]}-{c[3]}x{c[4]}x{c[5]}x{c[6]}-{c[7]}")
def test_wide_conv_is_the_linear_layer_on_im2col(case):
    import torch
    import torch.nn.functional as F
    q = _q()
    static, tr, wn, B, H, Wd, C, N, gs, epi, pad = case
    print(f"wide conv {case}", flush=True)
    M, K = B * H * Wd, 9 * C
    _assert_tile("conv3x3_static" if static else "conv3x3", M, N, K, gs, epi, False, tr, wn)
    x = to_dev_bf16(W.make_random_x(M + 3 * N + K, M, C, "t3", 0.05))
    g = torch.Generator(device="cuda").manual_seed(N + K)
    w = (torch.randn(N, K, generator=g, device="cuda") * 0.02).bfloat16()
    bias = torch.randn(N, generator=g, device="cuda").bfloat16()
    # (kh, kw, c), c fastest
    padded = F.pad(x.view(B, H, Wd, C), (0, 0, 1, 1, 1, 1))
    cols = torch.cat([padded[:, i:i + H, j:j + Wd] for i in range(3) for j in range(3)], 3).reshape(M, K).contiguous()
    buf = torch.full((M + 40, N + pad), 5.0, dtype=torch.bfloat16, device="cuda")
    out = buf[:M, :N]
    if static:
        s = float(np.float32(float(x.abs().max()) * 0.9 / 127))
        pw = q.pack_weight_per_channel(w)
        q.w4a4_conv3x3_static(q.quantize_act_static(x, s, gs), pw, s, B, H, Wd, bias, epi, out=out)
        want = q.w4a4_linear_static(q.quantize_act_static(cols, s, gs), pw, s, bias, epi)
    else:
        pw = q.pack_weight(w)
        q.w4a4_conv3x3(q.quantize_act(x, gs), pw, B, H, Wd, bias, epi, out=out)
        want = q.w4a4_linear(q.quantize_act(cols, gs), pw, bias, epi)
    torch.cuda.synchronize()
    assert torch.all(buf[M:] == 5.0) and torch.all(buf[:M, N:] == 5.0), "wrote outside y"
    assert torch.equal(out, want)
    # with a workspace: equal too where neither kernel of either call would split
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    if not static and any(q.linear_schedule(M, N, K, cus, True, t)[0]["split"] for t in (0, 1)):
        return
    ws = q.gemm_workspace(M, N, K, "cuda")
    ws = torch.zeros(256, dtype=torch.uint8, device="cuda") if ws is None else ws
    if static:
        q.w4a4_conv3x3_static(q.quantize_act_static(x, s, gs), pw, s, B, H, Wd, bias, epi, out=out, workspace=ws)
        want = q.w4a4_linear_static(q.quantize_act_static(cols, s, gs), pw, s, bias, epi, workspace=ws)
    else:
        q.w4a4_conv3x3(q.quantize_act(x, gs), pw, B, H, Wd, bias, epi, out=out, workspace=ws)
        want = q.w4a4_linear(q.quantize_act(cols, gs), pw, bias, epi, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(out, want)


@pytest.mark.parametrize("M,N,K,tr,wn", [(68, 192, 320, 2, 2), (2403, 459, 192, 2, 4), (8242, 776, 448, 5, 8)],
                         ids=["2x2", "2x4", "5x8"])
def test_infinite_scales_stay_in_their_columns(M, N, K, tr, wn):
    """The group after a panel's last one is the next panel's first: its scales
    are infinite here, and multiply nothing."""
    import torch
    q = _q()
    for layer in ("linear", "asym"):
        _assert_tile(layer, M, N, K, 16, 0, False, tr, wn)
    x = to_dev_bf16(W.make_random_x(M, M, K, "t3", 0.05))
    w = to_dev_bf16(W.to_bf16_bits(np.random.Generator(np.random.PCG64(N)).normal(0, 0.02, (N, K))))
    pw = q.pack_weight(w)
    sums = q.weight_group_sums(pw)
    # a chunk per panel of 64 columns and group: 2048 bytes of codes, 64 fp16 scales
    bad = dataclasses.replace(pw, data=pw.data.clone())
    bad.data.view(-1, K // 64, 2176)[1, :, 2048:].view(torch.int16).fill_(0x7C00)
    keep = [*range(64), *range(128, N)]
    for asym in (False, True):
        qa = q.quantize_act(x, 16, mode=q.MODE_ASYMMETRIC if asym else q.MODE_SYMMETRIC)
        y, z = (q.w4a4_linear_asym(qa, v, sums) if asym else q.w4a4_linear(qa, v) for v in (pw, bad))
        torch.cuda.synchronize()
        assert not torch.isfinite(z[:, 64:128]).any()
        assert torch.equal(y[:, keep], z[:, keep])
