"""GPU parity of the wide linear kernel (tiles of 32 TR rows by 256 columns)
where it can go wrong: every tile height, M inside a row tile and inside a
wave's 32 rows, N inside a wave's 32 columns and inside a panel of 64, an odd
number of 64-groups (a round's second group masked out), one and several tiles
per workgroup, every G_s, in every mode.  The dispatch picks the height from
the shape; the comment at each shape names the one it is meant for.  Sampled
rows and columns against the oracle within the tolerance of tests/helpers.py,
every output of a larger buffer outside y untouched, and the quantized output
equal to quantizing the bf16 one."""
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


CASES = [
    # (mode, TR, M, N, K, gs, epilogue, bias, extra columns of the buffer)
    ("plain", 4, 303, 546, 192, 16, 0, True, 6),       # 16-byte rows do not hold: element stores
    ("plain", 5, 8242, 776, 448, 8, 1, True, 0),       # N % 32 == 8
    ("plain", 6, 8286, 1046, 256, 32, 0, False, 2),
    ("plain", 7, 8126, 1291, 320, 64, 0, True, 5),
    ("plain", 8, 8131, 1541, 448, 16, 1, True, 3),
    ("plain", 7, 9100, 3072, 192, 16, 0, True, 0),     # two tiles per workgroup, odd groups
    ("static", 4, 379, 308, 256, 16, 0, True, 4),
    ("static", 5, 8296, 783, 320, 8, 1, True, 1),
    ("static", 6, 8189, 1050, 448, 32, 0, False, 6),
    ("static", 7, 8110, 1314, 192, 64, 0, True, 6),
    ("static", 8, 16300, 1600, 64, 16, 0, True, 0),    # a single group
    ("asym", 4, 424, 386, 320, 8, 0, True, 6),
    ("asym", 5, 8301, 773, 320, 16, 1, True, 3),
    ("asym", 6, 8205, 1030, 192, 32, 0, False, 2),
    ("asym", 7, 8214, 1287, 256, 64, 0, True, 1),
    ("quantized", 4, 408, 512, 256, 16, 0, True, 0),
    ("quantized", 5, 8238, 832, 448, 8, 1, True, 0),
    ("quantized", 6, 8319, 1088, 320, 32, 0, False, 0),
    ("quantized", 7, 8069, 1344, 448, 64, 1, True, 0),
    ("quantized", 8, 8253, 1600, 512, 16, 0, True, 0),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}-tr{c[1]}-{c[2]}x{c[3]}x{c[4]}-gs{c[5]}")
def test_wide_kernel_parity(case):
    import torch
    q = _q()
    mode, tr, M, N, K, gs, epi, with_bias, pad = case
    print(f"wide {case}", flush=True)
    xb = W.make_random_x(M + 3 * N + K, M, K, "t3", 0.05)
    wb = W.to_bf16_bits(np.random.Generator(np.random.PCG64(N + 5 * K)).normal(0, 0.02, (N, K)))
    bias_b = W.to_bf16_bits(np.random.Generator(np.random.PCG64(N)).normal(0, 0.02, N)) if with_bias else None
    bias = None if bias_b is None else to_dev_bf16(bias_b)
    x, w = to_dev_bf16(xb), to_dev_bf16(wb)
    buf = torch.full((M + 40, N + pad), 5.0, dtype=torch.bfloat16, device="cuda")
    out = buf[:M, :N]
    ws = q.gemm_workspace(M, N, K, "cuda")
    rows, cols = _sample(M, 32 * tr, M), _sample(N, 256, N)
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
