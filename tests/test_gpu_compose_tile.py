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
