"""The Mamba-2 composition and log-decay fold against fp64: request lengths around
the composition's groups of four blocks, an id outside the pool at every
position, state sizes on both sides of its workgroup multiple, fp32 and bf16
pools; block lengths around the fold's 256-row passes and head counts around
its 64-lane groups."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2608_11231_amd import lkv  # noqa: E402


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("dk,dv,h", [(128, 64, 3), (16, 64, 2), (64, 16, 5), (32, 48, 1), (32, 64, 2)])
def test_compose_matches_fp64(dk, dv, h, bf16):
    rng = np.random.default_rng(dk * dv)
    n_blk = 7
    B = torch.from_numpy(rng.standard_normal((n_blk, h, dv, dk)).astype(np.float32)).cuda()
    if bf16:
        B = B.to(torch.bfloat16)
    Lam = torch.from_numpy(-rng.uniform(0, 1.5, (n_blk, h)).astype(np.float32)).cuda()
    ids = [rng.integers(0, n_blk, K).astype(np.int32) for K in (0, 1, 3, 4, 5, 8, 9, 31)]
    bad = []
    for K in (1, 4, 6):
        for j in range(K):
            x = rng.integers(0, n_blk, K).astype(np.int32)
            x[j] = -1 if j % 2 else n_blk
            bad.append(len(ids))
            ids.append(x)
    cu = np.concatenate([[0], np.cumsum([len(x) for x in ids])]).astype(np.int32)
    flat = np.concatenate(ids).astype(np.int32)
    L = lkv.make_layer(lkv.SSD, 1, h, dk, dv, 64, torch.bfloat16, torch.float32)
    S = torch.full((len(ids), h, dv, dk), 7.0, device="cuda")
    (lkv.init_compose_bf16 if bf16 else lkv.init_compose)(L, n_blk, B, Lam, torch.from_numpy(flat).cuda(),
                                                          torch.from_numpy(cu).cuda(), len(flat), S)
    torch.cuda.synchronize()
    for r, x in enumerate(ids):
        if r in bad:
            assert S[r].isnan().all(), r
            continue
        ref = torch.zeros((h, dv, dk), device="cuda", dtype=torch.float64)
        for j, b in enumerate(x):
            f = torch.exp(Lam[b].double())[:, None, None]
            ref = B[b].double() if j == 0 else f * ref + B[b].double()
        # an fp32 exp (a few ulp), a product and a sum per block, errors decaying with the state
        assert (S[r].double() - ref).abs().max() <= 2e-6 * max(1.0, float(ref.abs().max())), (r, len(x))


@pytest.mark.parametrize("h", [1, 63, 64, 130])
def test_lambda_matches_fp64(h):
    lens = [0, 1, 15, 16, 255, 256, 257, 700, 1]
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    n = int(cu[-1])
    g = torch.Generator("cuda").manual_seed(h)
    dt = torch.rand((n, h), device="cuda", generator=g) * 0.1
    A = -1.0 - torch.rand((h,), device="cuda", generator=g)
    L = lkv.make_layer(lkv.SSD, 1, h, 64, 64, 64, torch.bfloat16, torch.float32)
    M = torch.full((len(lens), h), 7.0, device="cuda")
    lkv.block_summary(L, lkv.make_tokens(torch.from_numpy(cu).cuda(), n, None, None, None, dt, None, A), None, M)
    torch.cuda.synchronize()
    for s in range(len(lens)):
        ref = A.double() * dt[cu[s]:cu[s + 1]].double().sum(0)
        # a sum of at most 700 fp32 terms of one sign over 256 partial sums
        assert ((M[s].double() - ref).abs() <= 4e-6 * ref.abs() + 1e-30).all(), s


def _fold_order(x):
    """The fold's fp32 sum of one block's rows [n, h]: 16 token lanes, each with four sums over
    whole groups of four of its rows and the rest on the first, lanes added in order."""
    x = x.astype(np.float32)
    total = np.zeros(x.shape[1], np.float32)
    for lane in range(16):
        rows = x[lane::16]
        acc, full = np.zeros((4, x.shape[1]), np.float32), len(rows) // 4 * 4
        for k, r in enumerate(rows):
            acc[k % 4 if k < full else 0] += r
        total += (acc[0] + acc[1]) + (acc[2] + acc[3])
    return total


@pytest.mark.parametrize("h", [1, 8, 65])
def test_lambda_order_of_the_sum(h):
    """Every remainder of the fold's loops (eight rows of a lane, then four, then single ones), bit for bit."""
    lens = [*range(0, 40), 127, 128, 129, 191, 192, 193, 255, 257, 319, 320, 450, 1000]
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    rng = np.random.default_rng(h)
    dt = rng.uniform(0, 0.2, (int(cu[-1]), h)).astype(np.float32)
    A = -rng.uniform(1, 16, h).astype(np.float32)
    L = lkv.make_layer(lkv.SSD, 1, h, 64, 64, 64, torch.bfloat16, torch.float32)
    M = torch.full((len(lens), h), 7.0, device="cuda")
    T = lkv.make_tokens(torch.from_numpy(cu).cuda(), int(cu[-1]), None, None, None, torch.from_numpy(dt).cuda(), None,
                        torch.from_numpy(A).cuda())
    lkv.block_summary(L, T, None, M)
    ref = np.stack([A * _fold_order(dt[cu[s]:cu[s + 1]]) for s in range(len(lens))])
    assert np.array_equal(M.cpu().numpy(), ref)


def test_lambda_rows_past_32_bit_offsets():
    """128 dt rows of 2^23 heads are 2^32 bytes: eight rows of a lane span more than 32-bit offsets hold."""
    h, n = 1 << 23, 130
    dt = (torch.arange(n, device="cuda") % 8 / 8.0).to(torch.float32)[:, None].expand(n, h).contiguous()
    A = torch.full((h,), -2.0, device="cuda")
    L = lkv.make_layer(lkv.SSD, 1, h, 16, 16, 16, torch.bfloat16, torch.float32)
    M = torch.full((1, h), 7.0, device="cuda")
    cu = torch.tensor([0, n], dtype=torch.int32, device="cuda")
    lkv.block_summary(L, lkv.make_tokens(cu, n, None, None, None, dt, None, A), None, M)
    assert bool((M == -2.0 * float((np.arange(n) % 8 / 8.0).sum())).all())
