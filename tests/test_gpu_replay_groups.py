"""Selection from registers and the four-position sparse attention at the edges
of their tiles, against torch in double on the CPU."""
import numpy as np
import pytest
import torch

from paper_2607_28979_amd import binding as mb

pytestmark = pytest.mark.gpu


def _select(A, S):
    """Top-S key sets by a stable sort: larger first, ties to the lower position."""
    B, T, _ = A.shape
    out = torch.full((B, T, S), -1, dtype=torch.int32)
    for b in range(B):
        for u in range(T):
            row = A[b, u, :u + 1]
            got = torch.sort(row, descending=True, stable=True).indices[:S].sort().values
            out[b, u, :len(got)] = got.int()
    return out


def _attend(q, k, v, idx):
    """o[b][u][h] over the entries of idx[b][u] in 0..u as listed (duplicates count)."""
    B, T, H, D = q.shape
    G = H // k.shape[2]
    q, k, v = q.double(), k.double(), v.double()
    o = torch.zeros(B, T, H, D, dtype=torch.float64)
    for b in range(B):
        for u in range(T):
            n = idx[b, u][(idx[b, u] >= 0) & (idx[b, u] <= u)].long()
            if len(n) == 0:
                continue
            kk, vv = (x[b, n].repeat_interleave(G, 1) for x in (k, v))
            p = torch.softmax(torch.einsum("hd,nhd->hn", q[b, u], kk) / D ** 0.5, -1)
            o[b, u] = torch.einsum("hn,nhd->hd", p, vv)
    return o


# T around the pieces (1024 positions) and their 16-byte alignment, S above and
# below 256 (the lower bound), S = 1, and rows longer than the registers hold
@pytest.mark.parametrize("T,S", [(1030, 32), (1029, 300), (2051, 256), (1100, 1), (8196, 64), (16388, 32)])
def test_select_edges(T, S):
    _check_select(T, S, {S, S + 1, 1023, 1024, 1025, T // 2, T - 2, T - 1})


# a map at the last length of each form (one piece of one or of four values per thread,
# two, four, eight and sixteen pieces) and at the first of the next, with rows on both
# sides of the length from which a lower bound is looked for (3072), S to 256 and past it
# (rows much longer than S: at a boundary of 0 the zeros' signs would count)
@pytest.mark.parametrize("T,S", [(2, 1), (255, 16), (256, 255), (257, 16), (1024, 90), (1025, 300), (2048, 256), (2049, 64),
                                 (3080, 256), (3080, 257), (4096, 32), (4097, 128), (8192, 256), (8193, 1), (16384, 64),
                                 (16385, 256)])
def test_select_forms(T, S):
    _check_select(T, S, {S, T // 3, 2047, 3070, 3071, 3072, T - 2, T - 1})


def _check_select(T, S, us):
    print("case", T, S, flush=True)
    g = torch.Generator().manual_seed(T)
    rows = sorted(us & set(range(T)))
    A = torch.zeros(1, T, T, device="cuda")
    want = {}
    for i, u in enumerate(rows):
        r = torch.randn(T, generator=g)
        if i % 4 == 1:
            r = torch.round(r * 4) / 4                       # heavy ties
        if i % 4 == 2:
            r[torch.randperm(T, generator=g)[:T // 2]] = -torch.inf
            r[5] = torch.inf
        if i % 4 == 3:
            r = torch.where(r > 0, r * 1e-30, torch.finfo(torch.float32).min)   # lowest values, tiny ones
        r[u + 1:] = 7.0                                      # never chosen
        A[0, u] = r
        want[u] = torch.sort(r[:u + 1], descending=True, stable=True).indices[:S].sort().values.int()
    idx = torch.full((1, T, S), -9, dtype=torch.int32, device="cuda")
    mb.topS_select(A, idx, 1, T, S)
    torch.cuda.synchronize()
    for u, w in want.items():
        got = idx[0, u].cpu()
        assert torch.equal(got[:len(w)], w) and (got[len(w):] == -1).all(), u


@pytest.mark.parametrize("T,off", [(1032, 1), (1032, 2), (8200, 3), (1032, 4)])
def test_select_unaligned_base(T, off):
    """A 4-byte aligned map at any offset from a 16-byte boundary (rows of T % 4 == 0
    are fetched in 16-byte pieces only where they start on one)."""
    S = 64
    print("case", T, off, flush=True)
    g = torch.Generator().manual_seed(off)
    buf = torch.zeros(T * T + off, device="cuda")
    A = buf[off:].view(1, T, T)
    assert buf.data_ptr() % 16 == 0 and A.data_ptr() % 16 == 4 * off % 16
    want = {}
    for u in (S, 1023, 1026, T - 2, T - 1):
        r = torch.randn(T, generator=g)
        r[u + 1:] = 7.0
        A[0, u] = r
        want[u] = torch.sort(r[:u + 1], descending=True, stable=True).indices[:S].sort().values.int()
    idx = torch.full((1, T, S), -9, dtype=torch.int32, device="cuda")
    mb.topS_select(A, idx, 1, T, S)
    torch.cuda.synchronize()
    for u, w in want.items():
        assert torch.equal(idx[0, u].cpu(), w), u


# KV heads 1, 2, 3, 4 and 8 in short calls (up to four: one position per workgroup), 1 to 8
# query heads per KV head, every T mod 4, head-major K and V, sets past 128, and lists that
# are unordered, repeat keys or hold none; then contexts of several times the set, so that
# every set is full and a group's list runs to hundreds of keys
ATTN = [(1, 37, 7, 1, 128, 32, 0), (2, 38, 4, 2, 64, 64, 1), (1, 39, 24, 3, 128, 96, 0), (1, 90, 28, 4, 128, 160, 1),
        (3, 41, 8, 8, 64, 256, 0), (1, 1, 4, 4, 128, 32, 0), (9, 230, 7, 1, 128, 32, 0), (7, 237, 4, 2, 64, 64, 1),
        (3, 1, 16, 2, 128, 32, 0), (5, 215, 3, 3, 64, 32, 1), (5, 220, 16, 2, 64, 32, 0),
        (3, 701, 12, 2, 128, 128, 0), (3, 700, 14, 2, 128, 192, 1), (3, 703, 14, 2, 64, 256, 0),
        (1, 702, 28, 4, 128, 192, 1), (1, 701, 32, 8, 64, 256, 0)]
# the four-position kernel: five to eight KV heads (waves with one head and with two), every
# T mod 4; two groups of two waves per workgroup, one of them idle or not, and an odd number
# of groups; one group of four waves, two of them idle or one; the largest sets of each head
# width with both
ATTN += [(1, 37, 35, 5, 128, 32, 0), (2, 38, 12, 6, 64, 64, 1), (1, 39, 56, 7, 128, 96, 0), (1, 90, 40, 5, 128, 160, 1),
         (1, 1, 8, 8, 128, 32, 0), (21, 230, 7, 1, 128, 32, 0), (12, 237, 4, 2, 64, 64, 1), (5, 516, 14, 2, 64, 96, 1),
         (12, 220, 16, 2, 64, 32, 0), (4, 703, 14, 2, 64, 256, 0), (2, 600, 6, 2, 128, 64, 0)]


@pytest.mark.parametrize("case", ATTN, ids=lambda c: "x".join(map(str, c)))
@pytest.mark.parametrize("kind", ["selected", "listed"])
def test_attention_groups(case, kind):
    B, T, Hq, Hkv, D, S, lay = case
    print("case", case, kind, flush=True)
    g = torch.Generator().manual_seed(S + T)
    q, k, v = (torch.randn(B, T, h, D, generator=g).bfloat16() for h in (Hq, Hkv, Hkv))
    if kind == "selected":
        idx = _select(torch.randn(B, T, T, generator=g), S)
    else:   # any order, repeats, entries past u, -1 anywhere; some positions with nothing
        idx = torch.randint(-2, T + 3, (B, T, S), generator=g).int()
        idx[:, ::5] = -1
    dev = [x.transpose(1, 2).contiguous().cuda() if lay and i else x.cuda() for i, x in enumerate((q, k, v))]
    o = torch.full((B, T, Hq, D), -3.75, dtype=torch.bfloat16, device="cuda")
    mb.replay_attention(*dev, idx.cuda(), o, B, T, Hq, Hkv, D, S=S, kv_layout=lay)
    torch.cuda.synchronize()
    ref = _attend(q, k, v, idx)
    d = (o.cpu().double() - ref)
    # bf16 probabilities and outputs: 2^-9 of the row's scale each
    assert d.norm() <= 2.0 ** -7 * ref.norm()
    assert d.abs().max() <= 2.0 ** -6 * max(1.0, ref.abs().max().item())
    if kind == "listed":
        assert (o[:, ::5] == 0).all()
    again = torch.empty_like(o)
    mb.replay_attention(*dev, idx.cuda(), again, B, T, Hq, Hkv, D, S=S, kv_layout=lay)
    assert torch.equal(o, again)


@pytest.mark.parametrize("D,Hq,Hkv", [(128, 40, 8), (128, 28, 4), (64, 24, 8)])
def test_attention_large_scores(D, Hq, Hkv):
    """Scores near 2^23 (whole numbers, exact in fp32) that differ by a few units and grow
    along the sets: the blocks of a set keep their weights against each other."""
    T, S = 200, 128
    g = torch.Generator().manual_seed(D)
    q, k = torch.full((1, T, Hq, D), 256.0), torch.full((1, T, Hkv, D), 256.0 * 128 // D)
    q[..., 0] = torch.randint(1, 4, (1, T, Hq), generator=g).float()
    k[..., 0] = torch.randint(0, 9, (1, T, Hkv), generator=g) + (torch.arange(T) // 4)[None, :, None].float()
    q, k, v = (x.bfloat16() for x in (q, k, torch.randn(1, T, Hkv, D, generator=g)))
    idx = _select(torch.randn(1, T, T, generator=g), S)
    o = torch.empty(1, T, Hq, D, dtype=torch.bfloat16, device="cuda")
    mb.replay_attention(q.cuda(), k.cuda(), v.cuda(), idx.cuda(), o, 1, T, Hq, Hkv, D, S=S)
    ref = _attend(q, k, v, idx)
    d = o.cpu().double() - ref
    assert d.norm() <= 2.0 ** -7 * ref.norm()
    assert d.abs().max() <= 2.0 ** -6 * max(1.0, ref.abs().max().item())


@pytest.mark.parametrize("H,Hkv", [(16, 8), (8, 4)])
def test_attention_value_rows_that_are_not_finite(H, Hkv):
    """NaN and infinite value rows reach exactly the positions that attend them; their
    group's other positions come out as without them."""
    T, S, D = 64, 32, 128
    g = torch.Generator().manual_seed(3)
    q, k, v = (torch.randn(1, T, h, D, generator=g).bfloat16() for h in (H, Hkv, Hkv))
    idx = _select(torch.randn(1, T, T, generator=g), S)
    idx[idx == 20] = 19          # (a repeat where 19 is in the set as well)
    idx[idx == 40] = 39
    idx[0, 33, 0], idx[0, 50, 1] = 20, 40
    outs = []
    for poke in (False, True):
        w = v.clone()
        if poke:
            w[0, 20, 0], w[0, 40, 1, 7] = float("nan"), float("inf")
        o = torch.empty(1, T, H, D, dtype=torch.bfloat16, device="cuda")
        mb.replay_attention(q.cuda(), k.cuda(), w.cuda(), idx.cuda(), o, 1, T, H, Hkv, D, S=S)
        outs.append(o.cpu().float()[0])
    clean, got = outs
    assert torch.isnan(got[33, :2]).all()                                # KV head 0's query heads
    assert torch.isposinf(got[50, 2:4, 7]).all()
    same = torch.ones(T, H, D, dtype=torch.bool)
    same[33, :2], same[50, 2:4, 7] = False, False
    # repeats make both runs walk the sets as listed, or one by one: the same sums
    # in another order
    assert (clean - got)[same].abs().max() <= 2.0 ** -7 * max(1.0, clean.abs().max().item())


# tiles of a batch row: 3 of many heads; 8, 4 and 9, where the whole batch takes pairs of
# tiles (36, 448 and 48 heads) and one row of it single ones; 3, 7 and 17 in single tiles, with
# heads that share rows of tiles unevenly among the XCDs; one tile
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("B,T,Hq,Hkv", [(36, 261, 32, 4), (3, 1000, 12, 2), (16, 500, 28, 4), (6, 1153, 8, 8), (3, 300, 5, 1),
                                        (2, 870, 6, 3), (2, 2050, 4, 4), (5, 101, 3, 1)])
def test_causal_tile_orders_agree(D, B, T, Hq, Hkv):
    """A short and a long tile per workgroup or one tile each, in any order: the same bits."""
    print("case", D, B, T, Hq, Hkv, flush=True)
    g = torch.Generator().manual_seed(9)
    q, k, v = (torch.randn(B, T, h, D, generator=g).bfloat16().cuda() for h in (Hq, Hkv, Hkv))
    whole = torch.full((B, T, Hq, D), -3.75, dtype=torch.bfloat16, device="cuda")
    mb.replay_attention(q, k, v, None, whole, B, T, Hq, Hkv, D)
    for b in (0, B // 2, B - 1):
        one = torch.full((1, T, Hq, D), -3.75, dtype=torch.bfloat16, device="cuda")
        mb.replay_attention(q[b:b + 1], k[b:b + 1], v[b:b + 1], None, one, 1, T, Hq, Hkv, D)
        assert torch.equal(whole[b], one[0])
    ref = torch.nn.functional.scaled_dot_product_attention(
        *(x[:1].cpu().double().transpose(1, 2).repeat_interleave(Hq // x.shape[2], 1) for x in (q, k, v)),
        is_causal=True).transpose(1, 2)
    d = whole[:1].cpu().double() - ref
    assert d.norm() <= 2.0 ** -7 * ref.norm()
