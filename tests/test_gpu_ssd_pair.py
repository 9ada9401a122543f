"""The Mamba-2 kernel that takes two adjacent 64-row units per workgroup, against
the shared chunk kernel: the same products in the same order, so scans, block
summaries (B and Lambda), pool starts and state-only calls must agree bit for
bit.  Sizes: two heads of 64 rows, two tiles of one head, pairs that straddle
nothing (grouped heads), ragged, empty, one-token and chunk-multiple segments; and
batches on both sides of the rule that chooses between the two from the
segments' lengths."""
import numpy as np
import pytest

from paper_2608_11231_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2608_11231_amd import gpu_io, lkv  # noqa: E402

CASES = [
    # (N, P, G, H, blocks, online)
    (128, 64, 1, 4, ((130, 64), (1, 70), (0,)), (150, 64, 0)),
    (128, 64, 2, 4, ((100, 0, 65),), (129,)),
    (128, 128, 1, 3, ((64, 128), (3,)), (0, 191)),
    (128, 192, 2, 4, ((65,), (200,), (7,)), (63, 1, 256)),
    (128, 256, 3, 3, ((65, 2),), (320,)),
]


def _bits(t):
    return t.view(torch.int16) if t.dtype == torch.bfloat16 else t.view(torch.int32)


def _same(a, b):
    na, nb = a.isnan(), b.isnan()
    return torch.equal(na, nb) and torch.equal(_bits(a.masked_fill(na, 0)), _bits(b.masked_fill(nb, 0)))


@pytest.mark.parametrize("case", CASES, ids=[f"ssd{c[:4]}" for c in CASES])
def test_pairs_match_chunk_kernel(case, monkeypatch):
    dk, dv, hq, hv, blocks, online = case
    layer = I.Layer(I.SSD, hq, hv, dk, dv, 64, "bf16", "f32")
    law = I.GateLaw(dt_mu=-3.0, dt_bias=-1.0, a_lo=1.0, a_hi=4.0)
    w = I.build_workload("pair", layer, [list(b) for b in blocks], list(online), law, 31)
    G = gpu_io.GpuWorkload(w)
    S0 = torch.from_numpy((0.5 * np.random.default_rng(4).standard_normal(tuple(G.S_final.shape)))
                          .astype(np.float32)).cuda()
    # a cached row, the zero state (-1), an id outside the pool (NaN state)
    src = torch.tensor([w.n_blk - 1, -1, w.n_blk + 5][:w.n_req], dtype=torch.int32, device="cuda")

    def passes():
        res = []
        for t in (G.B_pool, G.M_pool, G.out, G.S_final):
            t.fill_(7.0)
        G.block_summary()
        res += [G.B_pool.clone(), G.M_pool.clone()]
        G.block_summary(M=False)
        res += [G.B_pool.clone()]
        G.scan(S0)
        res += [G.out.clone(), G.S_final.clone()]
        for pool in (G.B_pool, G.B_pool.to(torch.bfloat16)):
            lkv.chunk_scan_from_pool(G.layer, G.online.struct, 1.0, pool, w.n_blk, src, G.out, G.S_final)
            res += [G.out.clone(), G.S_final.clone()]
        lkv.ssd_chunk_scan(G.layer, G.online.struct, S0, None, G.S_final)  # state only
        lkv.ssd_chunk_scan(G.layer, G.online.struct, None, G.out, None)    # outputs only, zero start
        res += [G.S_final.clone(), G.out.clone()]
        torch.cuda.synchronize()
        return res

    monkeypatch.setenv("LKV_SSD_PAIR", "0")
    ref = passes()
    monkeypatch.setenv("LKV_SSD_PAIR", "1")
    got = passes()
    for i, (a, b) in enumerate(zip(got, ref)):
        assert _same(a, b), i


# segments x heads on either side of the dispatch's lines: one round of the chunk
# kernel, ssd_scan_kernel (96 units of dk 128), pairs (more than 256 units of one group),
# more segments than are ranked by length, an odd number of units per group
@pytest.mark.parametrize("n_seq,hq,hv,dv", [(1, 1, 64, 64), (4, 1, 24, 64), (5, 1, 64, 64), (70, 1, 8, 64),
                                            (9, 15, 15, 192)])
def test_dispatch_keeps_bits(n_seq, hq, hv, dv, monkeypatch):
    layer = I.Layer(I.SSD, hq, hv, 128, dv, 64, "bf16", "f32")
    law = I.GateLaw(dt_mu=-3.0, dt_bias=-1.0, a_lo=1.0, a_hi=4.0)
    lens = [(37 * i) % 150 for i in range(n_seq)]
    w = I.build_workload("rule", layer, [[] for _ in lens], lens, law, 5)
    G = gpu_io.GpuWorkload(w, with_cached=False)
    S0 = 0.5 * torch.randn(G.S_final.shape, device="cuda", generator=torch.Generator("cuda").manual_seed(2))
    G.scan(S0)
    out, S = G.out.clone(), G.S_final.clone()
    monkeypatch.setenv("LKV_SSD_PAIR", "0")
    G.out.fill_(7.0)
    G.scan(S0)
    torch.cuda.synchronize()
    assert _same(out, G.out) and _same(S, G.S_final)


def _batch(hq, hv, dv, lens, seed):
    layer = I.Layer(I.SSD, hq, hv, 128, dv, 64, "bf16", "f32")
    law = I.GateLaw(dt_mu=-3.0, dt_bias=-1.0, a_lo=1.0, a_hi=4.0)
    return gpu_io.GpuWorkload(I.build_workload("len", layer, [[] for _ in lens], list(lens), law, seed),
                              with_cached=False)


# Where pairs or the eight-wave kernel may take a batch, two launches follow each other and exactly one works, as the
# lengths have it: random batches whose longest chain is short, about the line, and long
@pytest.mark.parametrize("hq,hv,dv,n_seq", [(1, 64, 64, 5), (1, 24, 64, 13), (1, 40, 128, 10), (8, 64, 64, 13),
                                            (5, 10, 128, 40), (1, 16, 64, 70), (1, 64, 64, 16),
                                            (1, 8, 64, 9), (2, 16, 128, 3), (1, 2, 64, 70)])
def test_lengths_choose_one_launch(hq, hv, dv, n_seq, monkeypatch):
    units = n_seq * hv * dv // 64
    # pairs, or (a second round of the chunk kernel's small units) the eight-wave kernel
    assert units > (256 if hq == 1 and hv * dv // 64 >= 24 else 768) or 64 < units < 240
    rng = np.random.default_rng(units)
    for draw in range(6):
        lens = rng.integers(0, (65, 130, 65)[draw % 3], n_seq)
        if draw % 3:
            lens[rng.integers(n_seq)] = (200, 900)[draw % 3 - 1]
        if draw == 3:
            lens[:] = 64
        G = _batch(hq, hv, dv, [int(x) for x in lens], draw)
        S0 = 0.5 * torch.randn(G.S_final.shape, device="cuda", generator=torch.Generator("cuda").manual_seed(draw))
        T = G.online.struct
        res = []
        for pair in (None, "0"):
            if pair:
                monkeypatch.setenv("LKV_SSD_PAIR", pair)
            for t in (G.out, G.S_final):
                t.fill_(float("nan"))
            B = torch.full_like(G.S_final, float("nan"))
            M = torch.full((n_seq, hv), float("nan"), device="cuda")
            G.scan(S0)
            lkv.block_summary(G.layer, T, B, M)
            torch.cuda.synchronize()
            res.append([x.clone() for x in (G.out, G.S_final, B, M)])
            monkeypatch.delenv("LKV_SSD_PAIR", raising=False)
        for a, b in zip(*res):
            assert torch.equal(_bits(a), _bits(b)) and not bool(a.isnan().any()), (draw, list(lens))
