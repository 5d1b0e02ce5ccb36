"""The pass over M x K where the cut of a layer into work items changes (rows
shorter than, at and past one segment; few and many rows; row blocks with a
remainder when compressing along M) and the column sweeps, against the oracle,
bit-exact."""
import pytest
import torch

import oracle as O
from gpu_util import compare_cs, compare_layer, free, gpu_layers, oracle_run, say
from paper_2311_04406_amd.binding import RESULT_WORDS

pytestmark = pytest.mark.gpu
KEY = 23


class Spec:
    def __init__(self, M, K, N, compress=0):
        self.M, self.K, self.N, self.seed, self.layer_id, self.compress = M, K, N, 17, 6, compress
        self.name = f"{M}x{K}x{N}"


# along N: segments of 128 (few rows), 256 and 512 (around ROW_ITEMS = 512 items), 1024
ALONG_N = [(1, 127, 9), (3, 129, 1), (255, 257, 9), (256, 513, 2), (257, 300, 4), (511, 1025, 9), (513, 1000, 8)]
# along M: 2, 4 to 16 and 32 rows a wavefront, shared by workgroup or not (2051 x 4100 x 1, 1900 x 1100 x 5), a
# remainder of one row; column sweeps of several row groups per wavefront (K > 2048, M > 2048)
ALONG_M = [(3, 65, 9), (65, 513, 3), (517, 1025, 9), (1031, 515, 2), (2051, 770, 10), (8195, 260, 1), (8300, 65, 3),
           (2051, 4100, 1), (1900, 1100, 5), (33, 2500, 40), (2600, 40, 40)]
CASES = ([(Spec(*s), p) for s in ALONG_N for p in (2, 3)] + [(Spec(*s, compress=1), 2) for s in ALONG_M])


@pytest.mark.parametrize("spec,parties", CASES, ids=[f"{s.name}-c{s.compress}-p{p}" for s, p in CASES])
def test_row_pass_items(spec, parties):
    from paper_2311_04406_amd import Context
    ctx = Context(device=0, key_seed=KEY, parties=parties)
    layers = gpu_layers(ctx, [spec])
    ctx.gen_triple_tags(layers)
    out = torch.zeros(RESULT_WORDS, dtype=torch.int64, device="cuda:0")
    say(f"[row items] {spec.name} compress={spec.compress} p={parties}")
    ctx.tag_linear_check(O.MODE_COMPACT, layers, out)
    torch.cuda.synchronize()
    ol = oracle_run(O.MODE_COMPACT, spec, KEY, parties=parties)
    compare_layer(layers[0], ol, O.MODE_COMPACT, dealt=False, what=spec.name)
    res = Context.decode_results(out, 1, parties)[0]
    compare_cs(res, ol, what=spec.name)
    assert res.accept
    ctx.close()
    free()
