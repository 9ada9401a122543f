"""The Gated DeltaNet scan with 128 state rows per workgroup (two row tiles per
state wave) against the 64-row form, which computes the same products in the
same order: bit for bit, on tails, empty and one-token segments, grouped heads,
pool starts and state-only calls; and where the segments' lengths choose the form.
And the longest-first order of a ragged batch's segments against the segments
one at a time."""
import numpy as np
import pytest

from paper_2608_11231_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2608_11231_amd import gpu_io, lkv  # noqa: E402


def _work(dv, hq, hv, online, seed=11):
    layer = I.Layer(I.GDN, hq, hv, 128, dv, 64)
    return I.build_workload("rows", layer, [[] for _ in online], list(online), I.GateLaw(), seed, scale=0.5)


def _rand(shape, seed):
    return 0.5 * torch.randn(shape, device="cuda", generator=torch.Generator("cuda").manual_seed(seed))


@pytest.mark.parametrize("dv,hq,hv,online", [(128, 2, 2, (150, 64, 0, 1)), (256, 1, 2, (63, 200)), (512, 1, 1, (129,)),
                                             (384, 3, 3, (64, 320))])
def test_128_rows_match_64(dv, hq, hv, online, monkeypatch):
    w = _work(dv, hq, hv, online)
    G = gpu_io.GpuWorkload(w, with_cached=False)
    S0 = _rand(G.S_final.shape, 3)
    src = torch.tensor([1, -1, 7, 0][:w.n_req], dtype=torch.int32, device="cuda")  # 7: outside the pool

    def passes():
        res = []
        for t in (G.out, G.S_final):
            t.fill_(7.0)
        G.scan(S0)
        res += [G.out.clone(), G.S_final.clone()]
        for pool in (S0, S0.to(torch.bfloat16)):
            lkv.chunk_scan_from_pool(G.layer, G.online.struct, 0.5, pool, w.n_req, src, G.out, G.S_final)
            res += [G.out.clone(), G.S_final.clone()]
        lkv.gdn_chunk_scan(G.layer, G.online.struct, 0.5, S0, None, G.S_final)
        lkv.gdn_chunk_scan(G.layer, G.online.struct, 0.5, None, G.out, None)
        res += [G.S_final.clone(), G.out.clone()]
        torch.cuda.synchronize()
        return res

    monkeypatch.setenv("LKV_SCAN_NB", "4")
    ref = passes()
    monkeypatch.setenv("LKV_SCAN_NB", "8")
    for i, (a, b) in enumerate(zip(passes(), ref)):
        assert torch.equal(a.isnan(), b.isnan()) and torch.equal(a.nan_to_num(), b.nan_to_num()), i


def _ranked(fam, n_seq, hq, units, n_tok):
    """Whether the library takes a batch's segments longest first."""
    return units >= 384 and 1 < n_seq <= 64 and n_tok >= 640 * n_seq and (fam == I.SSD or hq % 8 == 0)


# Gated DeltaNet with 64 (nb 4) and 128 (nb 8) state rows per workgroup; Mamba-2 pairs, of
# which up to 512 are mirrored; 65 segments and 4 heads are not ranked
@pytest.mark.parametrize("fam,n_seq,hq,hv,dv,nb,units,ranked", [
    (I.GDN, 17, 8, 16, 128, 4, 544, True), (I.GDN, 17, 8, 16, 256, 8, 544, True), (I.GDN, 64, 8, 8, 128, 8, 512, True),
    (I.GDN, 65, 8, 8, 128, 8, 520, False), (I.GDN, 64, 4, 8, 128, 8, 512, False),
    (I.SSD, 25, 1, 32, 64, 4, 400, True), (I.SSD, 33, 2, 32, 64, 4, 528, True), (I.SSD, 64, 1, 16, 64, 4, 512, True),
    (I.SSD, 65, 1, 16, 64, 4, 520, False)])
@pytest.mark.parametrize("summary", [False, True])
def test_ranked_segments_match_one_at_a_time(fam, n_seq, hq, hv, dv, nb, units, ranked, summary, monkeypatch):
    rows = 128 if fam == I.SSD else 16 * nb
    assert n_seq * hv * dv // rows == units
    rng = np.random.default_rng(n_seq)
    lens = [int(x) for x in rng.integers(500, 1400, n_seq)]
    lens[3] = lens[5] = 900  # equal lengths
    lens[7], lens[11] = 0, 1
    layer = I.Layer(fam, hq, hv, 128, dv, 64, "bf16", "bf16" if fam == I.GDN else "f32")
    n = sum(lens)
    assert _ranked(fam, n_seq, hq, units, n) == ranked
    g = torch.Generator("cuda").manual_seed(n_seq)
    unit = lambda x: (x / x.norm(dim=-1, keepdim=True)).to(torch.bfloat16)
    q, k = (unit(torch.randn((n, hq, 128), device="cuda", generator=g)) for _ in range(2))
    v = torch.randn((n, hv, dv), device="cuda", generator=g).to(torch.bfloat16)
    if fam == I.GDN:
        gate = (-0.05 * torch.rand((n, hv), device="cuda", generator=g)).to(torch.bfloat16)
        beta, A = torch.rand((n, hv), device="cuda", generator=g).to(torch.bfloat16), None
    else:
        gate, beta = 0.05 * torch.rand((n, hv), device="cuda", generator=g), None
        A = -1.0 - torch.rand((hv,), device="cuda", generator=g)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    L = gpu_io.layer_struct(layer)

    def run(a, b):
        t0, t1 = int(cu[a]), int(cu[b])
        c = torch.from_numpy(cu[a:b + 1] - cu[a]).cuda()
        part = [None if x is None else x[t0:t1].contiguous() for x in (q, k, v, gate, beta)]
        T = lkv.make_tokens(c, t1 - t0, *part, A)
        S = torch.full((b - a, hv, dv, 128), 7.0, device="cuda")
        if summary:
            M = torch.full((b - a, hv, 128, 128) if fam == I.GDN else (b - a, hv), 7.0, device="cuda")
            lkv.block_summary(L, T, S, M)
            return [S, M]
        out = torch.full((t1 - t0, hv, dv), 7.0, device="cuda", dtype=torch.bfloat16)
        if fam == I.GDN:
            lkv.gdn_chunk_scan(L, T, 0.3, None, out, S)
        else:
            lkv.ssd_chunk_scan(L, T, None, out, S)
        return [S, out]

    def pin(fam):
        if fam == I.GDN:
            monkeypatch.setenv("LKV_SCAN_NB", str(nb))
        else:
            monkeypatch.setenv("LKV_SSD_PAIR", "1")

    pin(fam)
    S, x = run(0, n_seq)
    for s in range(n_seq):  # one segment alone is never ranked
        S1, x1 = run(s, s + 1)
        assert torch.equal(S[s], S1[0]), s
        assert torch.equal(x[s] if summary else x[cu[s]:cu[s + 1]], x1[0] if summary else x1), s


# q/k heads, value heads, dv, lengths, whether the lengths allow 128 rows: one long request
# among short ones, equal ones, longest last, more than a wave's 64 segments, uneven heads
@pytest.mark.parametrize("hq,hv,dv,lens", [
    (8, 32, 128, [70] * 4 + [1500] + [70] * 3), (8, 32, 128, [200] * 8), (16, 16, 256, [65] * 9 + [1, 0, 900]),
    (8, 8, 128, [40 + i for i in range(70)]), (8, 8, 128, [30] * 69 + [1300]), (15, 30, 128, [150] * 9),
    (15, 30, 128, [20] * 8 + [600]), (8, 32, 128, [0] * 8)])
def test_rows_chosen_by_lengths_keep_bits(hq, hv, dv, lens, monkeypatch):
    assert len(lens) * hv * dv // 128 >= 240  # the batch gets the kernel that holds both forms
    w = _work(dv, hq, hv, lens)
    G = gpu_io.GpuWorkload(w, with_cached=False)
    S0 = _rand(G.S_final.shape, 3)
    res = []
    for nb in (None, "4"):
        if nb:
            monkeypatch.setenv("LKV_SCAN_NB", nb)
        for t in (G.out, G.S_final):
            t.fill_(7.0)
        G.scan(S0)
        torch.cuda.synchronize()
        res.append((G.out.clone(), G.S_final.clone()))
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])
