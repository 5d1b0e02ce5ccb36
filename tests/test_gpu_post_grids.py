"""The pass over M x N of batches whose layers are compressed along M and along
N, with very different amounts of work on the two sides (each side's kernel has
a grid of its own size), against the oracle, bit-exact."""
import pytest
import torch

import oracle as O
from gpu_util import compare_cs, compare_layer, free, gpu_layers, oracle_run, say
from paper_2311_04406_amd.binding import COMPRESS_M, COMPRESS_N, RESULT_WORDS

pytestmark = pytest.mark.gpu
KEY = 5


class Spec:
    def __init__(self, M, K, N, compress, f, layer_id):
        self.M, self.K, self.N, self.seed, self.layer_id, self.compress, self.f = M, K, N, 77, layer_id, compress, f


SMALL_N, SMALL_M = (3, 5, 9, COMPRESS_N), (9, 7, 3, COMPRESS_M)
LARGE_N, LARGE_M = (700, 16, 1100, COMPRESS_N), (1500, 16, 600, COMPRESS_M)
BATCHES = {"n_large": [LARGE_N, SMALL_M], "m_large": [SMALL_N, LARGE_M], "n_only": [SMALL_N], "m_only": [SMALL_M],
           "mixed": [LARGE_M, SMALL_N, (513, 9, 1, COMPRESS_M), (1, 12, 513, COMPRESS_N), (33, 8, 65, COMPRESS_M)]}


@pytest.mark.parametrize("f", [0, 13])
@pytest.mark.parametrize("kbits", [64, 32])
@pytest.mark.parametrize("mode", [O.MODE_SPDZ2K, O.MODE_COMPACT])
@pytest.mark.parametrize("batch", sorted(BATCHES))
def test_grids_of_both_sides(batch, mode, kbits, f):
    from paper_2311_04406_amd import Context
    specs = [Spec(*s, f, i + 1) for i, s in enumerate(BATCHES[batch])]
    ctx = Context(device=0, key_seed=KEY, kbits=kbits)
    layers = gpu_layers(ctx, specs)
    ctx.gen_triple_tags(layers)
    out = torch.zeros(RESULT_WORDS * len(specs), dtype=torch.int64, device="cuda:0")
    say(f"[post grids] {batch} mode={mode} k={kbits} f={f}")
    ctx.tag_linear_check(mode, layers, out)
    torch.cuda.synchronize()
    for s, L, res in zip(specs, layers, Context.decode_results(out, len(specs))):
        ol = oracle_run(mode, s, KEY, kbits=kbits)
        compare_layer(L, ol, mode, dealt=False, what=f"{batch} {s.M}x{s.K}x{s.N}")
        compare_cs(res, ol, what=f"{batch} {s.M}x{s.K}x{s.N}")
        assert res.accept
    ctx.close()
    free()
