"""Device memory of the residue products (ct_set_scratch): what takes it and
what does not, how a caller declines or sizes it, and that the results are the
same without it."""
import pytest
import torch

import oracle as O
from gpu_util import free, gpu_layers, say
from paper_2311_04406_amd.binding import PATH_DIGITS, PATH_RESIDUES, PATH_ROW_PASS, RESULT_WORDS, SCRATCH_BYTES

pytestmark = pytest.mark.gpu
KEY = 11
OTHER = 256 << 20   # tables, the test's own copies, and what the runtime may take meanwhile


class Spec:
    def __init__(self, M, K, N, layer_id=4, compress=0, conv=None):
        self.M, self.K, self.N, self.seed, self.layer_id = M, K, N, 91, layer_id
        self.compress, self.conv = compress, conv


LARGE = Spec(512, 640, 512)   # its products go through residues
SMALL = Spec(64, 128, 32)


def context(**kw):
    from paper_2311_04406_amd import Context
    return Context(device=0, key_seed=KEY, **kw)


def results(n=1):
    return torch.zeros(n * RESULT_WORDS, dtype=torch.int64, device="cuda:0")


def outputs(layers, out):
    """Copies of everything that the call wrote."""
    torch.cuda.synchronize()
    got = {"result": out.clone()}
    for i, L in enumerate(layers):
        for n in ("E", "U", "D", "cvec"):
            got[f"{n}.{i}"] = L[n].clone()
        for n in ("Z", "tZ") + (("Zf", "tZf") if L.f else ()):
            for p in range(L.parties):
                got[f"{n}{p}.{i}"] = L[n][p].clone()
    return got


def same(a, b):
    assert a.keys() == b.keys()
    for n in a:
        assert torch.equal(a[n], b[n]), n


def free_bytes():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info(0)[0]


@pytest.fixture(scope="module", autouse=True)
def loaded():
    """One call of each kind, so that code objects and pools are on the device before anything is weighed."""
    ctx = context()
    layers = gpu_layers(ctx, [LARGE])
    ctx.gen_triple_tags(layers)
    out = results()
    ctx.tag_linear_check(O.MODE_COMPACT, layers, out)
    ctx.mac_check_device(O.MODE_COMPACT, layers, out)
    torch.cuda.synchronize()
    ctx.close()
    free()


@pytest.mark.parametrize("parties", [2, 5])
def test_only_residue_products_take_the_scratch(parties):
    say(f"[scratch] parties={parties}")
    before = free_bytes()
    ctx = context(parties=parties)
    assert before - free_bytes() < OTHER, "at creation"
    layers, small, out = gpu_layers(ctx, [LARGE]), gpu_layers(ctx, [SMALL]), results()
    before = free_bytes()
    ctx.gen_triple_tags(layers)
    ctx.gen_triple_tags(small)
    ctx.mac_check_device(O.MODE_COMPACT, layers, out)
    ctx.tag_linear_check(O.MODE_COMPACT, small, out)
    ctx.tag_linear_check_static(O.MODE_COMPACT, small, out)
    ctx.tag_linear_check_static(O.MODE_COMPACT, layers, out)   # allocates nothing: digits
    by_digits = outputs(layers, out)
    assert before - free_bytes() < OTHER, "calls without residue products"
    if ctx.product_paths(O.MODE_COMPACT, layers) == [PATH_RESIDUES]:
        ctx.tag_linear_check(O.MODE_COMPACT, layers, out)
        same(by_digits, outputs(layers, out))
        assert abs(before - free_bytes() - SCRATCH_BYTES) < OTHER, "the first call with residue products"
        ctx.tag_linear(O.MODE_COMPACT, layers)
        ctx.tag_linear_check_static(O.MODE_COMPACT, layers, out)   # now by residues
        same(by_digits, outputs(layers, out))
        assert abs(before - free_bytes() - SCRATCH_BYTES) < OTHER, "once"
    else:
        assert parties > 2
    ctx.close()
    del layers, small
    free()


def test_sizes_that_calls_refuse_have_no_path():
    from paper_2311_04406_amd import CtError
    ctx = context(max_layers=2)
    layers = gpu_layers(ctx, [SMALL] * 2)
    assert ctx.product_paths(O.MODE_COMPACT, layers) == [PATH_DIGITS] * 2
    with pytest.raises(CtError):
        ctx.product_paths(O.MODE_COMPACT, layers + layers)
    for M, K, N in ((0, 1, 1), (1 << 31, 1, 1), (9, 1 << 21, 9), (9, 9, 1 << 22)):
        layers[1].M, layers[1].K, layers[1].N = M, K, N
        with pytest.raises(CtError):
            ctx.product_paths(O.MODE_COMPACT, layers)
    ctx.close()


def test_declined_sized_and_taken_ahead():
    from paper_2311_04406_amd import CtError
    ctx = context()
    layers, out = gpu_layers(ctx, [LARGE, Spec(300, 100, 5, 7)]), results(2)
    ctx.gen_triple_tags(layers)
    before = free_bytes()

    def run(paths):
        """One call; its outputs and what the free memory fell by."""
        assert ctx.product_paths(O.MODE_COMPACT, layers) == paths
        ctx.set_timing(True)
        ctx.stage_times()
        ctx.tag_linear_check(O.MODE_COMPACT, layers, out)
        torch.cuda.synchronize()
        st = ctx.stage_times()
        ctx.set_timing(False)
        assert ("rns_gemm" in st) == (PATH_RESIDUES in paths), st
        taken = before - free_bytes()
        return outputs(layers, out), taken

    ctx.set_scratch(0)
    want, taken = run([PATH_DIGITS, PATH_ROW_PASS])
    assert taken < OTHER
    plan = ctx.plan(O.MODE_COMPACT, layers, out)   # by digits too
    out.zero_()
    plan.launch()
    same(want, outputs(layers, out))
    plan.close()
    size = 512 << 20
    ctx.set_scratch(size)
    got, taken = run([PATH_RESIDUES, PATH_ROW_PASS])
    same(want, got)
    assert abs(taken - size) < OTHER
    ctx.set_scratch(1 << 20)   # not enough for any chunk
    got, taken = run([PATH_DIGITS, PATH_ROW_PASS])
    same(want, got)
    assert taken < OTHER
    ctx.set_scratch(size, now=True)
    assert abs(before - free_bytes() - size) < OTHER
    same(want, run([PATH_RESIDUES, PATH_ROW_PASS])[0])
    with pytest.raises(CtError):
        ctx.set_scratch(-1)
    same(want, run([PATH_RESIDUES, PATH_ROW_PASS])[0])
    with pytest.raises(CtError) as e:   # more than the card has: digits from then on
        ctx.set_scratch(1 << 42, now=True)
    assert "CT_ENOMEM" in str(e.value)
    same(want, run([PATH_DIGITS, PATH_ROW_PASS])[0])
    ctx.close()
    del layers
    free()

