"""Calls that a form chosen for other sizes once slowed down by 40% and more: each
timed against the call or the form that it must keep up with, in turn, medians
of several runs.  The bounds leave 20% for noise; both sides measured are given."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2608_11231_amd import lkv  # noqa: E402


def _times(calls, reps=10, rounds=9):
    """Median microseconds of each of several calls, timed in turn."""
    e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    got = [[] for _ in calls]
    for r in range(rounds + 1):
        for i, call in enumerate(calls):
            e[0].record()
            for _ in range(reps):
                call()
            e[1].record()
            e[1].synchronize()
            if r:  # the first round warms up
                got[i].append(e[0].elapsed_time(e[1]) * 1e3 / reps)
    return [sorted(g)[rounds // 2] for g in got]


def test_composition_of_one_block_is_a_copy():
    """Mamba-2 requests of one cached block: 64 x 64 heads of 64 x 128 fp32, 40.5 us against the
    copy's 45.0 (67.2 us when a group's missing blocks are read as the first one again)."""
    n, h, dv, dk = 64, 64, 64, 128
    L = lkv.make_layer(lkv.SSD, 1, h, dk, dv, 64, torch.bfloat16, torch.float32)
    B = torch.randn((n, h, dv, dk), device="cuda")
    Lam = -torch.rand((n, h), device="cuda")
    ids = torch.arange(n, dtype=torch.int32, device="cuda")
    cu = torch.arange(n + 1, dtype=torch.int32, device="cuda")
    S, C = torch.empty_like(B), torch.empty_like(B)
    t, copy = _times([lambda: lkv.init_compose(L, n, B, Lam, ids, cu, n, S), lambda: lkv.init_single(L, n, B, ids, C)])
    assert torch.equal(S, B) and torch.equal(C, B)
    assert t <= 1.2 * copy, (t, copy)


def _gdn(lens, h, d=128):
    """One Gated DeltaNet layer's scan of requests of these lengths, as a call."""
    n = sum(lens)
    g = torch.Generator("cuda").manual_seed(n)
    unit = lambda x: (x / x.norm(dim=-1, keepdim=True)).to(torch.bfloat16)
    q, k = (unit(torch.randn((n, h, d), device="cuda", generator=g)) for _ in range(2))
    v = torch.randn((n, h, d), device="cuda", generator=g).to(torch.bfloat16)
    gate = (-0.05 * torch.rand((n, h), device="cuda", generator=g)).to(torch.bfloat16)
    beta = torch.rand((n, h), device="cuda", generator=g).to(torch.bfloat16)
    cu = torch.tensor([0, *torch.tensor(lens).cumsum(0).tolist()], dtype=torch.int32, device="cuda")
    L = lkv.make_layer(lkv.GDN, h, h, d, d, 64)
    T = lkv.make_tokens(cu, n, q, k, v, gate, beta)
    out, S = torch.empty_like(v), torch.empty((len(lens), h, d, d), device="cuda")
    return lambda: lkv.gdn_chunk_scan(L, T, 0.09, None, out, S)


@pytest.mark.parametrize("lens", [[4096] + [512] * 7, [256] * 8 + [4096] + [256] * 7])
def test_one_long_request_among_short_ones(lens, monkeypatch):
    """The longest request's chain decides: 181 us with 64 state rows per workgroup, 256 us with 128
    (4096 and seven of 512 tokens, 32 heads).  The call must not take the latter."""
    scan = _gdn(lens, 32)

    def pinned(nb):
        def call():
            monkeypatch.setenv("LKV_SCAN_NB", nb)
            scan()
            monkeypatch.delenv("LKV_SCAN_NB")
        return call

    t, narrow = _times([scan, pinned("4")])
    assert t <= 1.2 * narrow, (t, narrow)


def _ssd(lens, h, dk=128, dv=64):
    """One Mamba-2 layer's scan of requests of these lengths, as a call."""
    n = sum(lens)
    g = torch.Generator("cuda").manual_seed(n)
    C, B = (torch.randn((n, 1, dk), device="cuda", generator=g).to(torch.bfloat16) for _ in range(2))
    x = torch.randn((n, h, dv), device="cuda", generator=g).to(torch.bfloat16)
    dt = 0.05 * torch.rand((n, h), device="cuda", generator=g)
    A = -1.0 - torch.rand((h,), device="cuda", generator=g)
    cu = torch.tensor([0, *torch.tensor(lens).cumsum(0).tolist()], dtype=torch.int32, device="cuda")
    L = lkv.make_layer(lkv.SSD, 1, h, dk, dv, 64, torch.bfloat16, torch.float32)
    T = lkv.make_tokens(cu, n, C, B, x, dt, None, A)
    y, S = torch.empty_like(x), torch.empty((len(lens), h, dv, dk), device="cuda")
    return lambda: lkv.ssd_chunk_scan(L, T, None, y, S)


@pytest.mark.parametrize("lens,h", [([256] * 6 + [4096] + [256] * 5, 24), ([256] * 18 + [4096] + [256] * 17, 8)])
def test_one_long_request_among_short_ones_ssd(lens, h, monkeypatch):
    """The same with pairs of heads: the chunk kernel takes 142 us, pairs 211 (24 heads; 8: 140 and 209)."""
    scan = _ssd(lens, h)

    def chunk():
        monkeypatch.setenv("LKV_SSD_PAIR", "0")
        scan()
        monkeypatch.delenv("LKV_SSD_PAIR")

    t, other = _times([scan, chunk])
    assert t <= 1.2 * other, (t, other)
