"""Residue products under a small scratch (ct_set_scratch): layers cut into
chunks of K, against the oracle, bit-exact; and batches cut into groups that
share the scratch, on two streams and on one, captured, and against the
products by digits."""
import pytest
import torch

import oracle as O
from gpu_util import compare_cs, compare_layer, free, gpu_layers, oracle_run, say
from paper_2311_04406_amd.binding import PATH_DIGITS, PATH_RESIDUES, RESULT_WORDS

pytestmark = pytest.mark.gpu
KEY = 11
MODULI = 36


class Spec:
    def __init__(self, M, K, N, f=0, compress=0, conv=None, layer_id=4):
        self.M, self.K, self.N, self.seed, self.layer_id = M, K, N, 91, layer_id
        self.f, self.compress, self.conv = f, compress, conv
        self.name = f"{M}x{K}x{N}"


def scratch_bytes(s, parties, mode, chunks):
    """What a layer needs with K in this many chunks: its operands' planes of a chunk and its outputs' residues."""
    blocks = lambda major: -(-major // 32)
    kc = -(-(-(-s.K // chunks)) // 64) * 64
    assert (chunks - 1) * kc < s.K
    nops, outs = (parties + 1, parties) if mode == O.MODE_COMPACT else (2 * parties + 1, 2 * parties)
    return MODULI * 1024 * (outs * blocks(s.M) * blocks(s.N) + nops * (blocks(s.M) + blocks(s.N)) * (kc // 32))


# the paths into the planes: opened with them (two parties), converted (along M,
# convolutions, more parties; an odd number of parties has products of one
# kind and of the other); last chunks shorter than the others
CASES = [(Spec(449, 1025, 481), 2, 1, 2), (Spec(449, 1025, 481), 2, 1, 9), (Spec(415, 1100, 415), 2, 0, 3),
         (Spec(833, 1100, 801, f=13, compress=1), 2, 1, 2), (Spec(833, 1100, 801, compress=1), 2, 0, 2),
         (Spec(385, 1152, 784, conv=(128, 28, 28, 3, 1, 1)), 2, 1, 4), (Spec(641, 900, 610), 3, 1, 2),
         (Spec(353, 900, 448), 4, 0, 3), (Spec(577, 700, 610), 5, 1, 2)]


@pytest.mark.parametrize("spec,parties,mode,chunks", CASES,
                         ids=[f"{s.name}-p{p}-m{m}-c{c}" for s, p, m, c in CASES])
def test_chunks_of_k_bit_exact(spec, parties, mode, chunks):
    from paper_2311_04406_amd import Context
    ctx = Context(device=0, key_seed=KEY, parties=parties)
    ctx.set_scratch(scratch_bytes(spec, parties, mode, chunks))
    layers = gpu_layers(ctx, [spec])
    layers[0]["work"].fill_(0x5A5A5A5A5A5A5A5A)
    ctx.gen_triple_tags(layers)
    out = torch.zeros(RESULT_WORDS, dtype=torch.int64, device="cuda:0")
    say(f"[chunks] {spec.name} p={parties} mode={mode} chunks={chunks}")
    ctx.set_timing(True)
    ctx.stage_times()
    ctx.tag_linear_check(mode, layers, out)
    torch.cuda.synchronize()
    st = ctx.stage_times()
    ctx.set_timing(False)
    kinds = 2 if parties % 2 else 1   # problems of two products, and of one
    assert st["rns_gemm"][1] == chunks * kinds and "ring_gemm" not in st, st
    ol = oracle_run(mode, spec, KEY, parties=parties)
    compare_layer(layers[0], ol, mode, dealt=False, what=spec.name)
    res = Context.decode_results(out, 1, parties)[0]
    compare_cs(res, ol, what=spec.name)
    assert res.accept
    ctx.close()
    free()


# what the batch needs is above 1 GiB, where groups take the halves of the scratch in turn
BATCH = [Spec(512, 2048, 512, layer_id=1), Spec(449, 2000, 600, layer_id=2), Spec(700, 1500, 481, layer_id=3),
         Spec(512, 1024, 1024, layer_id=4), Spec(385, 1152, 784, conv=(128, 28, 28, 3, 1, 1), layer_id=5),
         Spec(833, 1100, 801, f=13, compress=1, layer_id=6), Spec(600, 2300, 512, layer_id=7),
         Spec(1024, 1024, 512, layer_id=8)]


def outputs(layers, out):
    torch.cuda.synchronize()
    got = {"result": out.clone()}
    for i, L in enumerate(layers):
        for n in ("E", "U", "D", "cvec"):
            got[f"{n}.{i}"] = L[n].clone()
        for n in ("Z", "tZ") + (("Zf", "tZf") if L.f else ()):
            for p in range(L.parties):
                got[f"{n}{p}.{i}"] = L[n][p].clone()
    return got


@pytest.mark.parametrize("mode", [O.MODE_SPDZ2K, O.MODE_COMPACT])
# groups on halves; half as much, with a layer or two on the whole scratch; about one layer at a time, some in chunks
@pytest.mark.parametrize("mib", [1024, 512, 160])
def test_groups_on_one_and_two_streams(mode, mib):
    from paper_2311_04406_amd import Context
    ctx = Context(device=0, key_seed=KEY)
    layers = gpu_layers(ctx, BATCH)
    ctx.gen_triple_tags(layers)
    out = torch.zeros(RESULT_WORDS * len(BATCH), dtype=torch.int64, device="cuda:0")

    def call():
        for L in layers:   # nothing of the call before is taken for this one's
            for t in [L["E"], L["U"], L["D"], L["work"], *L["Z"], *L["tZ"]]:
                t.fill_(-1)
        out.fill_(-1)
        ctx.tag_linear_check(mode, layers, out)
        return outputs(layers, out)

    def same(a, b, what):
        for n in a:
            assert torch.equal(a[n], b[n]), (what, n)

    say(f"[groups] mode={mode} {mib} MiB")
    ctx.set_scratch(0)
    assert ctx.product_paths(mode, layers) == [PATH_DIGITS] * len(BATCH)
    want = call()
    assert all(r.accept for r in Context.decode_results(out, len(BATCH)))
    ctx.set_scratch(mib << 20)
    assert PATH_RESIDUES in ctx.product_paths(mode, layers)
    for _ in range(3):
        same(want, call(), "two streams")
    ctx.set_overlap(False)
    same(want, call(), "one stream")
    ctx.set_overlap(True)
    plan = ctx.plan(mode, layers, out)
    for _ in range(3):
        call()
        out.fill_(-1)
        for L in layers:
            L["Z"][0].fill_(-1)
        plan.launch()
        same(want, outputs(layers, out), "captured")
    plan.close()
    ctx.close()
    del layers, want
    free()
