"""GPU parity of the fused attention's block shapes: whole rounds of unsplit
blocks, and what is left over split among two or four teams of waves that take
the 64-key chunks in turn.  The shapes give every one (on 256 compute units),
chunk counts that leave teams without a chunk in the last step, query blocks
that end inside a head, and scores whose maximum comes late and far above the
first tile's (the sums' reference moves).  Heads against the oracle, bounds as
in the attention tests: the bf16 rounding of the output, 2^-9 relative, and
1e-3 for the softmax codes that land on the other side of a rounding boundary."""
import numpy as np
import pytest

import oracle
import workloads as W
from helpers import bf16_bits_to_f64, to_dev_bf16, to_host_u16

pytestmark = pytest.mark.gpu

REL_BOUND = 2.0 ** -9 + 1e-3


def _rand(seed, shape, outliers=0, grow=1.0):
    rng = np.random.Generator(np.random.PCG64(seed))
    x = rng.normal(0, 1.0, shape)
    if outliers:
        x[:, rng.choice(shape[1], outliers, replace=False)] *= 20.0
    return W.to_bf16_bits(x * grow)


def _check(qb, kb, vb, heads, L, gs, which):
    import torch
    import paper_2509_26436_amd as q
    d = qb.shape[1]
    O = q.lzs_attention(to_dev_bf16(qb), to_dev_bf16(kb), to_dev_bf16(vb), heads, gs)
    torch.cuda.synchronize()
    for h in which:
        r = slice(h * L, (h + 1) * L)
        O64, _ = oracle.lzs_attention_f64(qb[r], kb[r], vb[r], gs)
        got = bf16_bits_to_f64(to_host_u16(O[:, h * d:(h + 1) * d].contiguous()))
        rel = np.linalg.norm(got - O64) / np.linalg.norm(O64)
        assert rel <= REL_BOUND, f"head {h}: relative error {rel:.2e}"


@pytest.mark.parametrize("heads,L,d,gs,which", [
    (3, 512, 128, 16, (0, 2)),          # four teams of two waves
    (2, 832, 64, 32, (0, 1)),           # the same, 13 chunks: three teams idle in the last step
    (3, 64, 128, 8, (0, 2)),            # two teams, one without any chunk
    (3, 448, 64, 64, (1,)),             # two teams, 7 chunks
    (44, 448, 128, 16, (0, 43)),        # two teams of four waves (176 blocks of 128 queries)
    (150, 320, 64, 16, (0, 149)),       # 450 blocks, unsplit, half of each head's last one past its end
    (95, 576, 128, 32, (0, 94)),        # 475 blocks
    (174, 320, 128, 16, (0, 170, 173)), # a whole round and 10 blocks over: two teams (L < 512)
    (105, 576, 64, 8, (0, 102, 104)),   # a round and 13 blocks: four teams
    (80, 640, 64, 16, (40, 79)),        # 400 blocks, unsplit
    (70, 640, 128, 64, (0, 69)),        # 350 blocks: two teams of two waves
])
def test_block_shapes(heads, L, d, gs, which):
    print(f"attention blocks {heads} x {L} x {d} gs {gs}", flush=True)
    n = heads * L
    qb, kb, vb = (_rand(700 + heads + i, (n, d), outliers=2) for i in range(3))
    _check(qb, kb, vb, heads, L, gs, which)


@pytest.mark.parametrize("heads,L,d", [(2, 576, 128), (3, 192, 64), (44, 448, 64)])
def test_late_maxima(heads, L, d):
    """The keys grow along the sequence, up to scores hundreds of powers of two
    above the first tile's."""
    print(f"attention late maxima {heads} x {L} x {d}", flush=True)
    n = heads * L
    grow = np.tile(np.linspace(0.05, 12.0, L), heads)[:, None]
    qb, kb, vb = _rand(800, (n, d)), _rand(801, (n, d), grow=grow), _rand(802, (n, d))
    _check(qb, kb, vb, heads, L, 16, (0, heads - 1))
