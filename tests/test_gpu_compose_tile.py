"""The composition with one 16-row tile per workgroup, against fp64: request
lengths around its two-step rounds (0 to 7 blocks and a long one), invalid ids
at every position, reused rows, fp32 and bf16 pools, both key dims; and the
same inputs through the 64-row form."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2608_11231_amd import lkv  # noqa: E402


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("dk,dv,h", [(128, 128, 2), (64, 48, 3), (128, 16, 1)])
def test_tiles_match_fp64(dk, dv, h, bf16, monkeypatch):
    rng = np.random.default_rng(dk + dv)
    n_blk = 9
    B = torch.from_numpy(rng.standard_normal((n_blk, h, dv, dk)).astype(np.float32)).cuda()
    if bf16:
        B = B.to(torch.bfloat16)
    M = torch.from_numpy((0.9 / np.sqrt(dk) * rng.standard_normal((n_blk, h, dk, dk))).astype(np.float32)).cuda()
    Ks = [0, 1, 2, 3, 4, 5, 6, 7, 33]
    ids = [rng.integers(0, n_blk, K).astype(np.int32) for K in Ks]
    bad = []
    for K in (1, 2, 3, 5, 6):  # an id outside the pool at every position
        for j in range(K):
            x = rng.integers(0, n_blk, K).astype(np.int32)
            x[j] = -1 if j % 2 else n_blk
            bad.append(len(ids))
            ids.append(x)
    cu = np.concatenate([[0], np.cumsum([len(x) for x in ids])]).astype(np.int32)
    flat = np.concatenate(ids).astype(np.int32)
    L = lkv.make_layer(lkv.GDN, h, h, dk, dv, 64)
    d_ids, d_cu = torch.from_numpy(flat).cuda(), torch.from_numpy(cu).cuda()

    def compose(tile):
        monkeypatch.setenv("LKV_COMPOSE_TILE", tile)
        S = torch.full((len(ids), h, dv, dk), 7.0, device="cuda")
        (lkv.init_compose_bf16 if bf16 else lkv.init_compose)(L, n_blk, B, M, d_ids, d_cu, len(flat), S)
        torch.cuda.synchronize()
        return S

    S, S64 = compose("1"), compose("0")
    Bd, Md = B.double(), M.double()
    for r, x in enumerate(ids):
        if r in bad:
            assert S[r].isnan().all() and S64[r].isnan().all(), r
            continue
        ref = torch.zeros((h, dv, dk), device="cuda", dtype=torch.float64)
        for j, b in enumerate(x):
            ref = Bd[b] if j == 0 else ref @ Md[b] + Bd[b]
        # 16 significant bits per split operand, a contraction per step: the state bar, 1e-4
        for got in (S, S64):
            assert (got[r].double() - ref).abs().max() <= 1e-4 * ref.abs().max().clamp(min=1e-30), (r, len(x))


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("dk,dv", [(128, 64), (64, 128)])
def test_tiles_keep_the_wide_forms_bits(dk, dv, bf16, monkeypatch):
    """Same split products in the same order in both forms: which one the sizes choose must not show."""
    g = torch.Generator("cuda").manual_seed(dk + dv)
    n_blk, h, Ks = 12, 3, [1, 2, 3, 8, 17]
    B = torch.randn((n_blk, h, dv, dk), device="cuda", generator=g)
    B = B.to(torch.bfloat16) if bf16 else B
    M = 0.9 / dk ** 0.5 * torch.randn((n_blk, h, dk, dk), device="cuda", generator=g)
    ids = torch.randint(0, n_blk, (sum(Ks),), device="cuda", generator=g).to(torch.int32)
    cu = torch.from_numpy(np.concatenate([[0], np.cumsum(Ks)]).astype(np.int32)).cuda()
    L = lkv.make_layer(lkv.GDN, h, h, dk, dv, 64)
    got = []
    for tile in "01":
        monkeypatch.setenv("LKV_COMPOSE_TILE", tile)
        S = torch.full((len(Ks), h, dv, dk), 7.0, device="cuda")
        (lkv.init_compose_bf16 if bf16 else lkv.init_compose)(L, n_blk, B, M, ids, cu, sum(Ks), S)
        got.append(S)
    torch.cuda.synchronize()
    assert torch.equal(got[0].view(torch.int32), got[1].view(torch.int32))


def test_sequence_parallel_scan_keeps_bits(monkeypatch):
    """The pieces' start states are the composition's running states: outputs alike in both forms."""
    g = torch.Generator("cuda").manual_seed(9)
    n, h, d = 700, 2, 128
    unit = lambda x: (x / x.norm(dim=-1, keepdim=True)).to(torch.bfloat16)
    q, k = (unit(torch.randn((n, h, d), device="cuda", generator=g)) for _ in range(2))
    v = torch.randn((n, h, d), device="cuda", generator=g).to(torch.bfloat16)
    gate = (-0.05 * torch.rand((n, h), device="cuda", generator=g)).to(torch.bfloat16)
    beta = torch.rand((n, h), device="cuda", generator=g).to(torch.bfloat16)
    S0 = torch.randn((2, h, d, d), device="cuda", generator=g)
    L = lkv.make_layer(lkv.GDN, h, h, d, d, 64)
    T = lkv.make_tokens(torch.tensor([0, 500, n], dtype=torch.int32, device="cuda"), n, q, k, v, gate, beta)
    ws = torch.empty(lkv.chunk_scan_sp_workspace(L, 2, 4), dtype=torch.uint8, device="cuda")
    got = []
    for tile in "01":
        monkeypatch.setenv("LKV_COMPOSE_TILE", tile)
        out, S = torch.full_like(v, 7.0), torch.full_like(S0, 7.0)
        lkv.chunk_scan_sp(L, T, 0.09, S0, out, S, 4, ws)
        got.append((out, S))
    torch.cuda.synchronize()
    assert torch.equal(got[0][0].view(torch.int16), got[1][0].view(torch.int16))
    assert torch.equal(got[0][1].view(torch.int32), got[1][1].view(torch.int32))
