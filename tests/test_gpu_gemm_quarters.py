"""Products of launches with few output tiles, whose wavefronts share the K
slices of a tile, against the oracle, bit-exact: one slice in all and fewer
slices than wavefronts, K split over workgroups as well, tiles cut by M and N,
both rings, both protocols, three parties, and the dealer's one-segment
products (the triple's C)."""
import pytest
import torch

import oracle as O
from gpu_util import compare_cs, compare_layer, free, gpu_layers, oracle_run, say
from paper_2311_04406_amd.binding import RESULT_WORDS

pytestmark = pytest.mark.gpu
KEY = 31


class Spec:
    def __init__(self, M, K, N):
        self.M, self.K, self.N, self.seed, self.layer_id = M, K, N, 41, 3
        self.name = f"{M}x{K}x{N}"


# 1 to 4 slices, a ragged last one, about 8 a wavefront, K split over workgroups (64 x 2100 x 40, 40 x 4100 x 33)
SHAPES = [(1, 1, 9), (32, 32, 32), (33, 65, 17), (64, 96, 31), (65, 129, 97), (31, 1000, 64), (64, 2100, 40), (40, 4100, 33)]
CASES = ([(s, 1, 2, 64) for s in SHAPES] + [(s, 0, 2, 64) for s in SHAPES[2:7:2]] + [(s, 1, 2, 32) for s in SHAPES[1::2]] +
         [(s, 1, 3, 64) for s in SHAPES[2::3]])


@pytest.mark.parametrize("shape,mode,parties,kbits", CASES)
def test_products_with_shared_slices(shape, mode, parties, kbits):
    from paper_2311_04406_amd import Context
    spec = Spec(*shape)
    ctx = Context(device=0, key_seed=KEY, parties=parties, kbits=kbits)
    layers = gpu_layers(ctx, [spec])
    layers[0]["work"].fill_(0x3C3C3C3C3C3C3C3C)
    ctx.gen_triple_tags(layers)
    out = torch.zeros(RESULT_WORDS, dtype=torch.int64, device="cuda:0")
    say(f"[shared slices] {spec.name} mode={mode} p={parties} k={kbits}")
    ctx.tag_linear_check(mode, layers, out)
    torch.cuda.synchronize()
    ol = oracle_run(mode, spec, KEY, parties=parties, kbits=kbits)
    compare_layer(layers[0], ol, mode, dealt=True, what=spec.name)
    res = Context.decode_results(out, 1, parties)[0]
    compare_cs(res, ol, what=spec.name)
    assert res.accept
    ctx.close()
    free()
