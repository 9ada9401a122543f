"""Performance cases of one recurrent layer's online prefill and of the steps around it.

``listed()`` names the calls that a serving program makes of this library per
recurrent layer, from the smallest (a decode step of a few requests) to the
largest (the transition fold of four 32K contexts); ``draw()`` gives more of
the same kinds over the same ranges.  Each case goes through the binding in
``paper_2608_11231_amd.lkv`` as a user's program does; ``exact()`` evaluates the
recurrences token by token in fp64 with plain torch.

Gates: layers of trained models mix heads of short and long memory, so the mean
log-gate varies over the heads from the slow to the fast end of the laws that
the repository's workloads use (Gated DeltaNet x ~ N(-9..-4, 1); Mamba-2 dt ~
softplus(N(-6..-3, 1)) with A in -[1, 16]).
"""
import math
import random

import torch

from paper_2608_11231_amd import lkv

_IO = {"bf16": torch.bfloat16, "f32": torch.float32}


# ---------------------------------------------------------------- cases
def _case(name, op, **kw):
    c = dict(name=name, op=op, fam="gdn", n_req=1, hqk=32, hv=32, dk=128, dv=128, chunk=64, io="bf16", gate="bf16",
             pool="f32", tok_lo=0, tok_hi=0, blk_per=0, blk_lo=0, blk_hi=0, pieces=0, layout=1)
    c.update(kw)
    if c["fam"] == "ssd":
        c["gate"] = "f32"
    return c


def listed():
    ssd = dict(fam="ssd", hqk=1, hv=64, dk=128, dv=64)
    return [
        # the smallest layer the library takes, fp32 tokens in 16-token chunks: block summaries,
        # composition and scan of one short request, a call chain that is all launches
        _case("tiny_gdn_f32", "prefill", hqk=1, hv=1, dk=16, dv=16, chunk=16, io="f32", gate="f32",
              blk_per=2, blk_lo=64, blk_hi=64, tok_lo=32, tok_hi=32),
        # decoding after the prefill, one token for each of four requests: latency
        _case("decode_gdn_4", "decode", n_req=4),
        # decoding at a full serving batch: state traffic
        _case("decode_ssd_256", "decode", n_req=256, **ssd),
        # LinearKV's path for one 8K request: the scan straight from a bf16 cached state
        _case("pool_gdn_8k", "pool_scan", pool="bf16", blk_per=8, tok_lo=1536, tok_hi=1536),
        # the same request on the sequence-parallel scan, which short batches are served with
        _case("sp_gdn_8k", "sp_scan", pieces=4, tok_lo=1536, tok_hi=1536),
        # exact composition of one 8K request: transitions of 7 of its 8 blocks folded, then composed
        _case("exact_gdn_8k", "exact", blk_per=8, blk_lo=1024, blk_hi=1024),
        # the recompute step of four 32K requests: selected rows gathered from the context, then scanned
        _case("recompute_gdn_32k", "recompute", n_req=4, blk_per=32, blk_lo=1024, blk_hi=1024,
              tok_lo=4096, tok_hi=4096),
        # a ragged batch of 16 requests with grouped query heads
        _case("scan_gdn_ragged", "scan", n_req=16, hqk=16, tok_lo=512, tok_hi=3072),
        # the transitions of four 32K contexts of ragged cached blocks: the largest call
        _case("fold_gdn_32k", "fold", n_req=4, blk_per=32, blk_lo=512, blk_hi=1536),
        # composing four requests' 32 cached blocks each, whose transitions are at hand
        _case("compose_gdn_32k", "compose", n_req=4, blk_per=32),
        # Mamba-2: one 8K request, sequence parallel
        _case("sp_ssd_8k", "sp_scan", pieces=4, tok_lo=1536, tok_hi=1536, **ssd),
        # Mamba-2: fold, composition from a bf16 pool and scan of a ragged batch
        _case("exact_ssd_ragged", "prefill_pool", n_req=16, pool="bf16", blk_per=8, blk_lo=256, blk_hi=2048,
              tok_lo=512, tok_hi=3072, **ssd),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost(case):
    w = work(case)
    return max(w["bytes"] / 5e12, w["flops"] / (0.5e15 if case["io"] == "bf16" else 0.25e15))


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        c = _draw(rng)
        if _cost(c) <= 0.7 * most:
            return c


def _draw(rng):
    op = rng.choice(["decode", "pool_scan", "sp_scan", "exact", "recompute", "scan", "fold", "compose", "prefill_pool",
                     "prefill"])
    fam = "ssd" if op == "prefill_pool" else rng.choice(["gdn", "gdn", "ssd"])
    layout = rng.randrange(1, 1 << 20)
    if fam == "ssd":
        hqk = rng.choice([1, 1, 2, 8])
        hv = hqk * rng.choice([8, 16, 24, 40, 64][:5 if hqk == 1 else 2])
        geo = dict(fam="ssd", hqk=hqk, hv=hv, dk=rng.choice([64, 128, 128]), dv=rng.choice([64, 64, 128]))
    else:
        hqk = rng.choice([4, 8, 15, 16, 30, 32])
        geo = dict(hqk=hqk, hv=hqk * rng.choice([1, 1, 2] if hqk <= 16 else [1]), dk=rng.choice([64, 128, 128]),
                   dv=rng.choice([64, 128, 128, 192, 256]))
    # fp32 tokens are taken up to a key dim of 64
    if geo["dk"] == 64 and rng.random() < 0.3:
        geo.update(io="f32", gate=rng.choice(["bf16", "f32"]))
    if op == "prefill":
        geo.update(dk=rng.choice([16, 32, 64]), dv=rng.choice([16, 32, 48, 64]), chunk=rng.choice([16, 64]))
        geo["hqk"], geo["hv"] = 1, rng.choice([1, 2, 4])
        return _case("", op, n_req=rng.randint(1, 3), layout=layout, blk_per=rng.randint(1, 4), blk_lo=16, blk_hi=200,
                     tok_lo=1, tok_hi=_log_int(rng, 8, 300), **geo)
    if op == "decode":
        return _case("", op, n_req=_log_int(rng, 1, 256), layout=layout, **geo)
    # requests and tokens such that no draw is larger than the listed 32K fold
    n_req = _log_int(rng, 1, 16)
    hi = _log_int(rng, 200, 4096 if n_req <= 4 else 3072)
    tok = dict(tok_lo=max(1, hi // rng.choice([1, 2, 6])), tok_hi=hi)
    heads = geo["hv"] * max(1, geo["dv"] // 128) * (geo["dk"] // 64) / 64.0
    if op in ("fold", "exact", "prefill_pool"):
        per = max(1, min(32, int(64 / (n_req * max(heads, 0.5)))))
        b_hi = _log_int(rng, 300, 1536)
        blk = dict(blk_per=rng.randint(1, per), blk_lo=max(1, b_hi // 3), blk_hi=b_hi)
    elif op == "recompute":
        per = max(1, min(32, 64 // n_req))
        blk = dict(blk_per=rng.randint(1, per), blk_lo=512, blk_hi=1024)
    else:
        blk = dict(blk_per=rng.randint(1, max(1, min(32, 128 // n_req))))
    if op == "sp_scan":
        tok = dict(tok_lo=max(1, hi // 2), tok_hi=hi)
        return _case("", op, n_req=rng.choice([1, 1, 2]), pieces=rng.choice([2, 3, 4, 8]), layout=layout, **tok, **geo)
    if op in ("fold", "exact", "compose"):
        tok = {}
    if op == "recompute":
        tok = dict(tok_lo=max(1, min(hi, 512 * blk["blk_per"]) // 2), tok_hi=min(hi, 512 * blk["blk_per"]))
    pool = rng.choice(["f32", "bf16"])
    return _case("", op, n_req=n_req, layout=layout, pool=pool, **blk, **tok, **geo)


# ---------------------------------------------------------------- layout (from the case alone)
def _lens(case, what, n):
    rng = random.Random("%d %s" % (case["layout"], what))
    return [rng.randint(case[what + "_lo"], case[what + "_hi"]) for _ in range(n)]


def _cum(lens):
    out = [0]
    for x in lens:
        out.append(out[-1] + x)
    return out


def _blocks(case):
    """Lengths of the cached blocks, in context order, request after request."""
    return _lens(case, "blk", case["n_req"] * case["blk_per"])


def _fold_lens(case):
    """Block lengths as the transition fold reads them: no composition reads the
    transition of a request's first block, so those are empty segments."""
    return [0 if i % case["blk_per"] == 0 else x for i, x in enumerate(_blocks(case))]


# ---------------------------------------------------------------- inputs
def _tokens(case, gen, n, with_q=True, with_v=True):
    d = dict(device="cuda", generator=gen)
    io = _IO[case["io"]]
    hqk, hv, dk, dv = case["hqk"], case["hv"], case["dk"], case["dv"]

    def unit():
        x = torch.randn((n, hqk, dk), **d)
        return x.div_(x.norm(dim=-1, keepdim=True)).to(io)

    t = dict(q=unit() if with_q else None, k=unit(), v=torch.randn((n, hv, dv), **d).to(io) if with_v else None)
    lin = torch.linspace(0.0, 1.0, hv, device="cuda")
    if case["fam"] == "gdn":
        gate = _IO[case["gate"]]
        t["g"] = (-torch.nn.functional.softplus(torch.randn((n, hv), **d) - 9.0 + 5.0 * lin)).to(gate)
        t["beta"] = torch.sigmoid(torch.randn((n, hv), **d)).to(gate)
        t["A"] = None
    else:
        t["g"] = torch.nn.functional.softplus(torch.randn((n, hv), **d) - 6.0 + 3.0 * lin)
        t["beta"] = None
        t["A"] = -torch.exp(torch.rand((hv,), **d) * math.log(16.0))
    return t


def _struct(t, cu, n):
    return lkv.make_tokens(cu, n, t["q"], t["k"], t["v"], t["g"], t["beta"], t["A"])


def _i32(x):
    return torch.tensor(x, dtype=torch.int32, device="cuda")


def _inputs(case, seed):
    """Every tensor that the call reads, from the seed."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    op, n_req, per = case["op"], case["n_req"], case["blk_per"]
    hv, dk, dv = case["hv"], case["dk"], case["dv"]
    state = (hv, dv, dk)
    x = {}

    def states(n, scale=0.3):
        return scale * torch.randn((n,) + state, device="cuda", generator=gen)

    if op == "decode":
        x["on"] = _tokens(case, gen, n_req)
        x["S0"] = states(n_req)
        return x
    n_blk = n_req * per
    if op in ("fold", "exact", "prefill_pool"):
        lens = _fold_lens(case)
        x["blk_cu_tok"] = _cum(lens)
        x["blk"] = _tokens(case, gen, sum(lens), with_q=False, with_v=False)
    if op == "prefill":
        lens = _blocks(case)
        x["blk_cu_tok"] = _cum(lens)
        x["blk"] = _tokens(case, gen, sum(lens), with_q=False)
    if op in ("exact", "compose", "prefill_pool", "pool_scan", "recompute"):
        x["B"] = states(n_blk).to(_IO[case["pool"]])
    if op == "compose":
        if case["fam"] == "gdn":
            # contractions, as folded blocks are: a spectral radius of 0.9
            x["M"] = torch.randn((n_blk, hv, dk, dk), device="cuda", generator=gen).mul_(0.9 / math.sqrt(dk))
        else:
            x["M"] = -2.0 * torch.rand((n_blk, hv), device="cuda", generator=gen)
    if op == "recompute":
        ctx = _blocks(case)
        x["ctx_cu"] = [sum(ctx[:r * per]) for r in range(n_req + 1)]
        x["ctx"] = _tokens(case, gen, sum(ctx))
        sel = _lens(case, "tok", n_req)
        x["sel_cu"] = _cum(sel)
        pos = []
        for r in range(n_req):
            n = x["ctx_cu"][r + 1] - x["ctx_cu"][r]
            pos.append(torch.randperm(n, device="cuda", generator=gen)[:sel[r]].sort().values.to(torch.int32))
        x["pos"] = torch.cat(pos)
    if op in ("pool_scan", "sp_scan", "scan", "prefill_pool", "prefill"):
        lens = _lens(case, "tok", n_req)
        x["on_cu"] = _cum(lens)
        x["on"] = _tokens(case, gen, sum(lens))
    if op in ("sp_scan", "scan"):
        x["S0"] = states(n_req)
    return x


def prepare(case, seed):
    x = _inputs(case, seed)
    op, n_req, per = case["op"], case["n_req"], case["blk_per"]
    hv, dk, dv, io = case["hv"], case["dk"], case["dv"], _IO[case["io"]]
    gdn = case["fam"] == "gdn"
    n_blk = n_req * per
    s = dict(x, case=case, n_blk=n_blk)
    s["layer"] = lkv.make_layer(lkv.GDN if gdn else lkv.SSD, case["hqk"], hv, dk, dv, case["chunk"], io,
                                _IO[case["gate"]])
    s["scale"] = dk ** -0.5

    def f32(*shape):
        return torch.empty(shape, device="cuda", dtype=torch.float32)

    s["S"] = f32(n_req, hv, dv, dk)
    if op == "decode":
        s["S"] = x["S0"]
        s["o"] = torch.empty((n_req, hv, dv), device="cuda", dtype=io)
        return s
    if "blk" in x:
        s["cu_b"] = _i32(x["blk_cu_tok"])
        s["blocks"] = _struct(x["blk"], s["cu_b"], x["blk_cu_tok"][-1])
        s["M"] = f32(n_blk, hv, dk, dk) if gdn else f32(n_blk, hv)
    if op == "prefill":
        s["B"] = f32(n_blk, hv, dv, dk)
    s["blk_ids"] = _i32(list(range(n_blk)))
    s["blk_cu"] = _i32([r * per for r in range(n_req + 1)])
    s["last"] = _i32([r * per + per - 1 for r in range(n_req)])
    s["S_exact"] = f32(n_req, hv, dv, dk)
    if op == "recompute":
        t = x["ctx"]
        s["cu_c"], s["cu_s"] = _i32(x["ctx_cu"]), _i32(x["sel_cu"])
        s["ctx_t"] = _struct(t, s["cu_c"], x["ctx_cu"][-1])
        n = s["n_on"] = x["sel_cu"][-1]
        s["on"] = {a: None if t[a] is None else torch.empty((n,) + tuple(t[a].shape[1:]), device="cuda", dtype=t[a].dtype)
                   for a in ("q", "k", "v", "g", "beta")}
        s["on"]["A"] = t["A"]
        s["online"] = _struct(s["on"], s["cu_s"], n)
    elif "on" in x:
        s["cu_o"] = _i32(x["on_cu"])
        n = s["n_on"] = x["on_cu"][-1]
        s["online"] = _struct(x["on"], s["cu_o"], n)
    if "online" in s:
        s["o"] = torch.empty((n, hv, dv), device="cuda", dtype=io)
    if op == "sp_scan":
        s["ws"] = torch.empty(lkv.chunk_scan_sp_workspace(s["layer"], n_req, case["pieces"]), dtype=torch.uint8,
                              device="cuda")
    return s


# ---------------------------------------------------------------- one pass
def _scan(s, S0):
    if s["case"]["fam"] == "gdn":
        lkv.gdn_chunk_scan(s["layer"], s["online"], s["scale"], S0, s["o"], s["S"])
    else:
        lkv.ssd_chunk_scan(s["layer"], s["online"], S0, s["o"], s["S"])


def _compose(s):
    f = lkv.init_compose_bf16 if s["B"].dtype == torch.bfloat16 else lkv.init_compose
    f(s["layer"], s["n_blk"], s["B"], s["M"], s["blk_ids"], s["blk_cu"], s["n_blk"], s["S_exact"])


def run(s):
    op, layer = s["case"]["op"], s["layer"]
    if op == "decode":
        t = s["on"]
        if s["case"]["fam"] == "gdn":
            lkv.gdn_decode(layer, t["q"], t["k"], t["v"], t["g"], t["beta"], s["scale"], s["S"], s["o"])
        else:
            lkv.ssd_decode(layer, t["q"], t["k"], t["v"], t["g"], t["A"], s["S"], s["o"])
        return s["o"], s["S"]
    if op == "scan":
        _scan(s, s["S0"])
        return s["o"], s["S"]
    if op == "pool_scan":
        lkv.chunk_scan_from_pool(layer, s["online"], s["scale"], s["B"], s["n_blk"], s["last"], s["o"], s["S"])
        return s["o"], s["S"]
    if op == "sp_scan":
        lkv.chunk_scan_sp(layer, s["online"], s["scale"], s["S0"], s["o"], s["S"], s["case"]["pieces"], s["ws"])
        return s["o"], s["S"]
    if op == "recompute":
        t = s["on"]
        lkv.gather_selected(layer, s["ctx_t"], s["pos"], s["cu_s"], s["n_on"], t["q"], t["k"], t["v"], t["g"], t["beta"])
        lkv.chunk_scan_from_pool(layer, s["online"], s["scale"], s["B"], s["n_blk"], s["last"], s["o"], s["S"])
        return {"o": s["o"], "S": s["S"], "rows": [t[a] for a in ("q", "k", "v", "g", "beta") if t[a] is not None]}
    if op == "compose":
        _compose(s)
        return s["S_exact"]
    if op == "prefill":
        lkv.block_summary(layer, s["blocks"], s["B"], s["M"])
        _compose(s)
        _scan(s, s["S_exact"])
        return {"B": s["B"], "M": s["M"], "S_exact": s["S_exact"], "o": s["o"], "S": s["S"]}
    # fold, exact, prefill_pool: the transitions of blocks 2..K first
    lkv.block_summary(layer, s["blocks"], None, s["M"])
    if op == "fold":
        return s["M"]
    _compose(s)
    if op == "exact":
        return s["M"], s["S_exact"]
    _scan(s, s["S_exact"])
    return {"M": s["M"], "S_exact": s["S_exact"], "o": s["o"], "S": s["S"]}


# ---------------------------------------------------------------- work
def _chunks(lens, c):
    for n in lens:
        for a in range(0, n, c):
            yield min(c, n - a)


def work(case):
    """Every input read once, every output written once; flops of the chunkwise form at
    the chunks' real token counts (the token recurrence's for decoding)."""
    op, n_req, per = case["op"], case["n_req"], case["blk_per"]
    hqk, hv, dk, dv, C = case["hqk"], case["hv"], case["dk"], case["dv"], case["chunk"]
    io, gb = (2 if case["io"] == "bf16" else 4), (2 if case["gate"] == "bf16" else 4)
    gdn = case["fam"] == "gdn"
    state, n_blk = hv * dk * dv * 4, n_req * per
    pool = n_blk * hv * dk * dv * (2 if case["pool"] == "bf16" else 4)
    trans = n_blk * hv * (dk * dk if gdn else 1) * 4
    read_trans = n_req * max(per - 1, 0) * hv * (dk * dk if gdn else 1) * 4
    gates = hv * gb * (2 if gdn else 1)

    def scan(lens, q=True):
        nb = sum(lens) * ((2 if q else 1) * hqk * dk * io + (2 if q else 1) * hv * dv * io + gates) + n_req * 2 * state
        if gdn:
            fl = sum((5 if q else 2) * 2 * n * n * dk + (3 if q else 2) * 2 * n * dk * dv + n ** 3 / 3
                     for n in _chunks(lens, C)) * hv
        else:
            fl = sum((2 * n * n * (dk + dv) if q else 0) + (2 if q else 1) * 2 * n * dk * dv
                     for n in _chunks(lens, C)) * hv
        return nb, fl

    def fold(lens):
        if not gdn:
            return sum(lens) * hv * 4 + trans, sum(lens) * hv
        return (sum(lens) * (hqk * dk * io + gates) + trans,
                sum(4 * n * n * dk + n ** 3 / 3 + 4 * n * dk * dk for n in _chunks(lens, C)) * hv)

    def compose():
        return pool + read_trans + n_req * state, n_req * max(per - 1, 0) * hv * 2 * dv * dk * (dk if gdn else 1)

    def add(*xs):
        return {"bytes": sum(x[0] for x in xs), "flops": sum(x[1] for x in xs)}

    if op == "decode":
        return {"bytes": n_req * (2 * state + 2 * hqk * dk * io + 2 * hv * dv * io + gates),
                "flops": n_req * hv * dk * dv * (8 if gdn else 5)}
    if op == "fold":
        return add(fold(_fold_lens(case)))
    if op == "compose":
        return add(compose())
    if op == "exact":
        return add(fold(_fold_lens(case)), compose())
    on = _lens(case, "tok", n_req)
    if op == "prefill":
        blk = _blocks(case)
        nb, fl = scan(blk, q=False)
        nb += (n_blk - 2 * n_req) * state + trans  # the summaries start from zero and write every block's state
        return add((nb, fl + fold(blk)[1]), compose(), scan(on))
    if op == "prefill_pool":
        return add(fold(_fold_lens(case)), compose(), scan(on))
    if op == "recompute":
        row = 2 * hqk * dk * io + hv * dv * io + gates
        return add((2 * sum(on) * row, 0), scan(on))
    return add(scan(on))  # scan, pool_scan, sp_scan


# ---------------------------------------------------------------- tolerance
def tolerance(case):
    # fp32 states come from sums whose fp32 operands are split in two bf16 parts (16
    # significant bits): about 1e-5 after thousands of tokens.  Outputs in bf16 carry its
    # rounding and that of the bf16 operands of the output products
    if case["op"] in ("fold", "exact", "compose") or case["io"] == "f32":
        return {"rel": 4e-5, "max": 4e-3}
    return {"rel": 1e-2, "max": 6e-2}


# ---------------------------------------------------------------- 64-bit reference
def _recur(case, t, cu, S, scale=1.0, want_o=True, transition=False):
    """The recurrences token by token in fp64, all (segment, head) states at once.  S
    [n_seq, hv, rows, dk] is advanced in place; returns the outputs [n_tok, hv, dv].
    transition: rows of the transition itself (no values)."""
    gdn, hv, dv = case["fam"] == "gdn", case["hv"], case["dv"]
    rep = hv // case["hqk"]
    n_seq, n_tok = len(cu) - 1, cu[-1]
    starts = torch.tensor(cu[:-1], device="cuda")
    lens = torch.tensor([cu[i + 1] - cu[i] for i in range(n_seq)], device="cuda")
    o = torch.zeros((n_tok, hv, dv), device="cuda", dtype=torch.float64) if want_o else None
    for i in range(max([cu[j + 1] - cu[j] for j in range(n_seq)], default=0)):
        live = (lens > i).nonzero().flatten()
        rows = starts[live] + i
        whole = live.numel() == n_seq
        s = S if whole else S[live]
        k = t["k"][rows].double().repeat_interleave(rep, 1)[:, :, None, :]
        g = t["g"][rows].double()
        if gdn:
            a, b = torch.exp(g)[:, :, None, None], t["beta"][rows].double()[:, :, None, None]
            s.mul_(a)
            d = torch.matmul(s, k.transpose(2, 3)).neg_()
            if not transition:
                d += t["v"][rows].double()[:, :, :, None]
            s.addcmul_(b * d, k.expand(-1, -1, s.shape[2], -1))
        else:
            s.mul_(torch.exp(g * t["A"].double())[:, :, None, None])
            s.addcmul_((g[:, :, None] * t["v"][rows].double())[:, :, :, None], k.expand(-1, -1, s.shape[2], -1))
        if want_o:
            q = t["q"][rows].double().repeat_interleave(rep, 1)[:, :, :, None]
            o[rows] = scale * torch.matmul(s, q)[..., 0]
        if not whole:
            S[live] = s
    return o


def _transitions(case, t, cu):
    n, hv, dk = len(cu) - 1, case["hv"], case["dk"]
    if case["fam"] == "ssd":
        g = t["g"].double() * t["A"].double()
        return torch.stack([g[cu[i]:cu[i + 1]].sum(0) for i in range(n)])
    M = torch.eye(dk, device="cuda", dtype=torch.float64).repeat(n, hv, 1, 1)
    _recur(case, t, cu, M, want_o=False, transition=True)
    return M


def _composed(case, B, M):
    per, out = case["blk_per"], []
    for r in range(case["n_req"]):
        S = B[r * per].double()
        for j in range(r * per + 1, (r + 1) * per):
            S = (S @ M[j] if case["fam"] == "gdn" else torch.exp(M[j])[:, None, None] * S) + B[j].double()
        out.append(S)
    return torch.stack(out)


def exact(case, seed):
    x = _inputs(case, seed)
    op, n_req, per = case["op"], case["n_req"], case["blk_per"]
    scale = case["dk"] ** -0.5 if case["fam"] == "gdn" else 1.0
    if op in ("decode", "scan", "sp_scan"):
        S = x["S0"].double()
        o = _recur(case, x["on"], x.get("on_cu") or list(range(n_req + 1)), S, scale)
        return o, S
    last = [r * per + per - 1 for r in range(n_req)]
    if op == "pool_scan":
        S = x["B"][last].double()
        return _recur(case, x["on"], x["on_cu"], S, scale), S
    if op == "recompute":
        rows = torch.cat([x["ctx_cu"][r] + x["pos"][x["sel_cu"][r]:x["sel_cu"][r + 1]].long() for r in range(n_req)])
        on = {a: v if v is None or a == "A" else v[rows] for a, v in x["ctx"].items()}
        S = x["B"][last].double()
        o = _recur(case, on, x["sel_cu"], S, scale)
        return {"o": o, "S": S, "rows": [on[a].double() for a in ("q", "k", "v", "g", "beta") if on[a] is not None]}
    if op == "compose":
        return _composed(case, x["B"], x["M"].double())
    M = _transitions(case, x["blk"], x["blk_cu_tok"])
    if op == "fold":
        return M
    if op == "prefill":
        B = torch.zeros((n_req * per, case["hv"], case["dv"], case["dk"]), device="cuda", dtype=torch.float64)
        _recur(case, x["blk"], x["blk_cu_tok"], B, want_o=False)
    else:
        B = x["B"]
    S0 = _composed(case, B, M)
    if op == "exact":
        return M, S0
    S = S0.clone()
    o = _recur(case, x["on"], x["on_cu"], S, scale)
    out = {"M": M, "S_exact": S0, "o": o, "S": S}
    return dict(out, B=B) if op == "prefill" else out
