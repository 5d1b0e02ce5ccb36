"""Performance cases of the linear-layer hot path.

A case is one call of the public Python binding on one batch of layers:

  call "check"   ``Context.tag_linear_check``: the online phase with the
                 verification fused in, as one eager call
  call "online"  ``Context.tag_linear``: the online phase alone, eager
  call "plan"    ``Plan.launch``: the fused step as a captured graph, the way
                 a program runs the same batch shape again and again
  call "verify"  ``Context.mac_check_device``: the standalone verification
  call "deal"    ``Context.gen_triple_tags``: the dealer (preprocessing)

``layers`` holds one ``MxKxN`` per layer, or ``MxKxN/C.H.W.k.s.p`` for a
convolution whose im2col matrix is left implicit.  ``prepare`` holds what a
program has before the call: a context, the layers' shares, tags and triple
(dealt from the seed), its result records and, for "plan", the plan.
"""
import math

import torch

from paper_2311_04406_amd import MODE_COMPACT, MODE_SPDZ2K, RESULT_WORDS, Context, workloads

MODES = {"compact": MODE_COMPACT, "spdz2k": MODE_SPDZ2K}
MK_OUT, KN_OUT, MN_OUT = ("E",), ("U",), ("D", "Z", "tZ", "Zf", "tZf")
OUTPUTS = MK_OUT + KN_OUT + MN_OUT + ("cvec",)
DEALT = ("X", "tX", "A", "tA", "Y", "tY", "B", "tB", "C", "tC", "R", "tR", "Rf", "tRf")


def text(specs, implicit=False):
    return " ".join("%dx%dx%d" % (s.M, s.K, s.N) + ("/" + ".".join(map(str, s.conv)) if implicit and s.conv else "")
                    for s in specs)


def parse(layers):
    out = []
    for item in layers.split():
        dims, _, conv = item.partition("/")
        out.append(tuple(int(v) for v in dims.split("x")) + (tuple(int(v) for v in conv.split(".")) if conv else None,))
    return out


def case(call, layers, mode="compact", kbits=64, parties=2, f=0, compress=0, **more):
    return dict(more, call=call, mode=mode, kbits=kbits, parties=parties, f=f, compress=compress, layers=layers)


def listed():
    enc = workloads.transformer(1)
    odd = "33x65x17 7x129x40 250x999x301 1x64x63 129x31x257 513x77x9 64x1000x3 31x2051x100"
    return [
        # one small fully connected layer, tagged and verified: latency and launches
        case("check", text(workloads.fc_small()), name="fc_small"),
        # one small convolutional layer on the benchmark's deepest feature map
        case("check", text(workloads.cnn()[3:4], True), compress=2, name="conv_deep"),
        # odd and ragged sizes, fixed-point outputs (f = 13), the compressed dimension by the operation count
        case("check", odd, f=13, compress=2, name="ragged_f13"),
        # the products of one encoder at sequence 128, captured
        case("plan", text(enc), name="encoder"),
        # the same encoder under the baseline protocol
        case("plan", text(enc), mode="spdz2k", name="encoder_spdz2k"),
        # twelve encoders: the weights (K x N) dominate
        case("plan", text(workloads.transformer(12)), name="encoders_12"),
        # VGG convolutions (implicit im2col) and the 25088 -> 4096 classifier at batch 1
        case("plan", text(workloads.cnn(), True), name="cnn"),
        # 64 uneven layers tagged and verified together: the headline batch
        case("plan", text(workloads.batched()), name="batched_64"),
        # the same batch over the smaller parameter set k = s = 32
        case("plan", text(workloads.batched()), kbits=32, name="batched_64_k32"),
        # the products of a training step of two encoders: forward, dX and dW
        case("plan", text(workloads.training(2)), name="training_2"),
        # three parties on one encoder, online phase and verification
        case("check", text(enc), parties=3, name="encoder_p3"),
        # preprocessing of one encoder: triple, masks, inputs and their tags
        case("deal", text(enc), name="deal_encoder"),
    ]


def log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """A batch of 1 to 64 layers with M, K, N log-uniform in [9, 4096] (a
    quarter of them rounded to multiples of 64, now and then a matrix-vector
    layer or a convolution), sum M K N at most 4e9, under any of the calls."""
    call = rng.choice(("check", "check", "plan", "plan", "online", "verify", "deal"))
    parties = rng.choice((2, 2, 2, 2, 3, 5))
    kbits = rng.choice((64, 64, 64, 32))
    f = rng.choice((0, 0, 0, 13))
    compress = rng.choice((0, 0, 2)) if parties == 2 else 0
    count, budget = log_int(rng, 1, 64), 4e9 / (2 if kbits == 64 and parties > 2 else 1)
    items, mkn, elems = [], 0.0, 0
    for _ in range(count):
        M, K, N = (log_int(rng, 9, 4096) for _ in range(3))
        if rng.random() < 0.25:
            M, K, N = (max(64, v // 64 * 64) for v in (M, K, N))
        conv = ""
        kind = rng.random()
        if kind < 0.08:
            N = rng.randint(1, 8)
        elif kind < 0.16 and parties == 2:
            c, hw, kk = log_int(rng, 3, 256), rng.randint(5, 40), rng.choice((1, 3))
            K, N, conv = c * kk * kk, hw * hw, "/%d.%d.%d.%d.1.%d" % (c, hw, hw, kk, kk // 2)
        size = M * K + K * N + M * N
        if items and (mkn + M * K * N > budget or elems + size > 6e7):
            continue
        while M * K * N > budget:
            M = (M + 1) // 2
        items.append("%dx%dx%d%s" % (M, K, N, conv))
        mkn += M * K * N
        elems += size
    return case(call, " ".join(items), mode=rng.choice(("compact", "compact", "compact", "spdz2k")), kbits=kbits,
                parties=parties, f=f, compress=compress)


def flat_outputs(layers, names):
    """Rebinds the named arrays of the layers to consecutive parts of one
    buffer per array (and party); returns the buffers."""
    out = {}
    for n in names:
        have = [l.t[n] for l in layers if n in l.t]
        if not have:
            continue
        per = len(have[0]) if isinstance(have[0], list) else 0
        for p in range(max(per, 1)):
            parts = [h[p] if per else h for h in have]
            rows = [t.numel() // t.shape[-1] for t in parts]
            buf = torch.zeros((sum(r + r % 2 for r in rows), parts[0].shape[-1]), dtype=torch.int64,
                              device=parts[0].device)
            at = 0
            for l, t, r in zip([l for l in layers if n in l.t], parts, rows):
                view = buf[at: at + r].view(t.shape)
                if per:
                    l.t[n][p] = view
                else:
                    l.t[n] = view
                at += r + r % 2  # 16-byte alignment of 8-byte elements
            out["%s%s" % (n, p if per else "")] = buf
    return out


def prepare(case, seed):
    ctx = Context(device=0, key_seed=(seed * 1000003 + 7) & 0xFFFFFFFF, kbits=case["kbits"], parties=case["parties"])
    layers = [ctx.layer(M, K, N, (seed << 20) + 4000 + i, i + 1, f=case["f"], compress=case["compress"], conv=conv)
              for i, (M, K, N, conv) in enumerate(parse(case["layers"]))]
    mode = MODES[case["mode"]]
    s = {"call": case["call"], "ctx": ctx, "layers": layers, "mode": mode}
    s["out"] = flat_outputs(layers, DEALT if case["call"] == "deal" else OUTPUTS)
    if case["call"] != "deal":
        ctx.gen_triple_tags(layers)
        if case["call"] != "online":
            s["out"]["result"] = torch.zeros(len(layers) * RESULT_WORDS, dtype=torch.int64, device=ctx.torch_device)
        if case["call"] == "verify":
            ctx.tag_linear(mode, layers)
            s["out"] = {"result": s["out"]["result"]}
        elif case["call"] == "plan":
            s["plan"] = ctx.plan(mode, layers, s["out"]["result"])
        if mode == MODE_SPDZ2K or case["call"] == "verify":
            s["out"].pop("cvec", None)  # compact-tag vectors: not written by these calls
    return s


def run(s):
    call = s["call"]
    if call == "check":
        s["ctx"].tag_linear_check(s["mode"], s["layers"], s["out"]["result"])
    elif call == "plan":
        s["plan"].launch()
    elif call == "online":
        s["ctx"].tag_linear(s["mode"], s["layers"])
    elif call == "verify":
        s["ctx"].mac_check_device(s["mode"], s["layers"], s["out"]["result"])
    else:
        s["ctx"].gen_triple_tags(s["layers"])
    return s["out"]


def work(case):
    """Bytes: every array of shares and tags that the call reads once and
    every array it writes once (all parties run on the one GPU).  Operations:
    a product of two 128-bit (64-bit) elements mod 2^128 (2^64) takes at
    least 31 (15) products of 8-bit digits, the bilinear rank of the
    truncated product of 16 (8) digits."""
    p, elem = case["parties"], case["kbits"] // 4
    compact, call = case["mode"] == "compact", case["call"]
    size = ops = 0
    for M, K, N, conv in parse(case["layers"]):
        right = conv[0] * conv[1] * conv[2] if conv else K * N
        if call == "deal":  # X, tX, A, tA; Y, tY, B, tB; C, tC, R, tR (f > 0: Rf, tRf)
            size += 4 * p * (M * K + right) + (6 if case["f"] else 4) * p * M * N
            products = 1
        elif call == "verify":  # E and U checked (SPDZ2k: D too); the compact check reads vectors only
            size += (2 * p + 1) * (M * K + right) + (0 if compact else (2 * p + 1) * M * N)
            products = 0
        else:  # X, A, tX, tA read, E written; Y, B, tY, tB read, U written; C, R, tC, tR read, D, Z, tZ written
            size += (4 * p + 1) * (M * K + right) + (6 * p + 1 + (4 * p if case["f"] else 0)) * M * N
            products = (2 if compact else 4) * p
        ops += products * M * K * N
    return {"bytes": size * elem, "flops": 2 * ops * (31 if case["kbits"] == 64 else 15)}


def exact(case, seed):
    """Every output is a whole number mod 2^128 or 2^64 (limbs in int64): it
    has one right value, and no nearer or further one in floating point."""
    return None
