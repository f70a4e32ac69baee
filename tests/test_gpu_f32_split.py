"""The fp32 path's split products (k_f32_split.hip) at the edges of its tiles and
K steps, and with operands outside the split's range, against numpy in double."""
import numpy as np
import pytest
from math import erf

from paper_2607_28979_amd import binding as mb

pytestmark = pytest.mark.gpu


def _reference(z, w1, b1, w2, b2, wr, br):
    """One unit in double: z [n][d_in] -> [n][d_out], dense mixture."""
    with np.errstate(all="ignore"):
        z, w1, b1, w2, b2, wr, br = (x.astype(np.float64) for x in (z, w1, b1, w2, b2, wr, br))
        lg = z @ wr.T + br
        g = np.exp(lg - lg.max(-1, keepdims=True))
        g /= g.sum(-1, keepdims=True)
        out = g @ b2
        for m in range(len(w1)):
            s = z @ w1[m].T + b1[m]
            h = s * 0.5 * (1 + np.vectorize(erf)(s * np.sqrt(0.5)))
            out = out + (g[:, m:m + 1] * h) @ w2[m].T
        return out


def _run(B, T, H_src, D_src, H_tgt, D_tgt, E, hidden, L=1, layout=0, seed=0, poke=None):
    """GPU result and reference, [L][2][n][d_out]; poke(d) edits the inputs."""
    import torch
    rng = np.random.default_rng(seed)
    di, do = H_src * D_src, H_tgt * D_tgt
    d = {"z": rng.standard_normal((2, L, B, T, H_src, D_src)), "w1": rng.standard_normal((L, 2, E, hidden, di)) / di ** .5,
         "b1": rng.standard_normal((L, 2, E, hidden)), "w2": rng.standard_normal((L, 2, E, do, hidden)) / hidden ** .5,
         "b2": rng.standard_normal((L, 2, E, do)), "wr": rng.standard_normal((L, 2, E, di)) / di ** .5,
         "br": rng.standard_normal((L, 2, E))}
    d = {k: v.astype(np.float32) for k, v in d.items()}
    if poke:
        poke(d)
    dev = {k: torch.from_numpy(v).cuda() for k, v in d.items()}
    src = [x.transpose(2, 3).contiguous() if layout else x.contiguous() for x in dev["z"]]
    shape = (L, B, H_tgt, T, D_tgt) if layout else (L, B, T, H_tgt, D_tgt)
    dst = [torch.full(shape, -3.75, device="cuda") for _ in range(2)]
    sh = mb.Shapes(L, L, B, T, H_src, D_src, H_tgt, D_tgt, E, hidden, dtype=mb.MOT_F32, src_layout=layout,
                   dst_layout=layout)
    mb.translate(*src, list(range(L)), dev["w1"], dev["b1"], dev["w2"], dev["b2"], dev["wr"], dev["br"], *dst, sh)
    torch.cuda.synchronize()
    got = np.stack([(x.transpose(2, 3) if layout else x).reshape(L, B * T, do).cpu().numpy() for x in dst], 1)
    ref = np.stack([[_reference(d["z"][x, j].reshape(B * T, di), *(d[k][j, x] for k in ("w1", "b1", "w2", "b2", "wr", "br")))
                     for x in range(2)] for j in range(L)])
    return got.astype(np.float64), ref


# one token; partial 64-wide tiles of tokens and outputs; one K step and an odd
# number; d_in % 32 == 16; BHTD heads of 20 and 32; many units and tokens (the
# 128-row tiles, ragged); E = 16
SHAPES = [(1, 1, 1, 16, 1, 4, 1, 64), (1, 65, 3, 16, 3, 20, 2, 64), (2, 33, 4, 20, 5, 12, 3, 64, 1, 1),
          (2, 31, 3, 32, 2, 36, 2, 192, 1, 1), (1, 700, 2, 48, 1, 132, 4, 192, 12), (2, 450, 4, 40, 1, 260, 2, 320, 12, 1),
          (1, 130, 1, 64, 2, 64, 16, 64)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_split_products(shape):
    print("case", shape, flush=True)
    got, ref = _run(*shape)
    err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    print("  rel %.2e" % err, flush=True)
    # products to 2^-33 and fp32 sums of up to 1024 terms: below 1e-6
    assert err < 1e-6
    assert np.abs(got - ref).max() < 2e-5 * np.sqrt(np.mean(ref ** 2))


@pytest.mark.parametrize("T", [40, 900])
def test_operands_outside_the_split(T):
    """A value above bf16's largest, infinities and NaN: the rows they reach come
    out as in plain fp32, every other row as without them."""
    def poke(d):
        d["z"][0, :, 0, 3, 0, 5] = 3.4e38     # finite in fp32, rounds to infinity in bf16
        d["wr"][:] = 0                         # so that the router stays finite
        d["w1"][:, 1, 0, 7] = 0                # values: one weight of one hidden unit
        d["w1"][:, 1, 0, 7, 9] = np.inf
        d["z"][1, :, 0, 11, 0, 9] = 0          # inf * 0 = NaN in that row
    L = 12 if T > 64 else 1
    got, ref = _run(1, T, 2, 32, 1, 64, 2, 128, L, poke=poke)
    for j in range(L):
        k, v = got[j], ref[j]
        err = np.abs(k[0] - v[0]) / np.sqrt(np.mean(v[0] ** 2, -1, keepdims=True))
        assert np.isfinite(k[0]).all() and err.max() < 2e-5
        assert np.array_equal(np.isnan(k[1]), np.isnan(v[1]))
        inf = np.isinf(v[1])
        assert inf.any() and np.array_equal(k[1][inf], v[1][inf])
        assert np.isnan(v[1][11]).all()


@pytest.mark.parametrize("heads", [(2, 32, 0), (3, 32, 1), (4, 20, 1)], ids=["bthd", "bhtd", "bhtd-20"])
def test_infinite_source_value(heads):
    """An infinite source value makes its token's row NaN and no other (the others of its
    blocks are computed again from rows in either layout)."""
    def poke(d):
        d["z"][:, :, 0, 5, 0, 1] = np.inf
    got, ref = _run(1, 40, heads[0], heads[1], 1, 64, 2, 128, layout=heads[2], poke=poke)
    assert np.isnan(got[:, :, 5]).all() and np.isnan(ref[:, :, 5]).all()
    rest = np.arange(40) != 5
    assert np.abs(got[:, :, rest] - ref[:, :, rest]).max() < 2e-5 * np.sqrt(np.mean(ref[:, :, rest] ** 2))


def _linear(z, w1, w2):
    """W2 (W1 z) of every unit (identity activation, one translator, whose gate is 1): z
    [2][L][T][d_in], w1 [L][2][hidden][d_in], w2 [L][2][d_out][hidden]; [L][2][T][d_out]."""
    import torch
    _, L, T, di = z.shape
    hidden, do = w1.shape[2], w2.shape[2]
    dev = [torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).cuda() for x in (*z, w1, w2)]
    dst = [torch.full((L, 1, T, 1, do), -3.75, device="cuda") for _ in range(2)]
    sh = mb.Shapes(L, L, 1, T, 1, di, 1, do, 1, hidden, dtype=mb.MOT_F32, act=mb.ACT_IDENTITY)
    mb.translate(dev[0], dev[1], list(range(L)), dev[2], None, dev[3], None, torch.zeros(L, 2, 1, di, device="cuda"), None,
                 *dst, sh)
    torch.cuda.synchronize()
    return np.stack([x.reshape(L, T, do).cpu().numpy() for x in dst], 1).astype(np.float64)


# exponents of the weights and of the values: ordinary; parts of one operand below
# bf16's least value; subnormal operands; products of ordinary operands whose small
# parts fall below fp32's least value; both operands small
EXPONENTS = [(0, 0), (-120, 100), (100, -124), (-126, 120), (-140, 120), (-60, -50), (-45, -70), (-110, 0)]


@pytest.mark.parametrize("T", [40, 900])
@pytest.mark.parametrize("exps", EXPONENTS, ids=lambda e: "%d,%d" % e)
@pytest.mark.parametrize("layer", [1, 2])
def test_single_products(T, exps, layer):
    """Rows with one value that is not zero: every output is one fp32 product, rounded once."""
    print("case", T, exps, layer, flush=True)
    n, L = 64, 12 if T > 64 else 1
    rng = np.random.default_rng(T + 7 * layer)

    def draw(e, *shape):
        return ((1 + rng.random(shape)) * rng.choice([-1, 1], shape) * 2.0 ** e).astype(np.float32)

    z = np.zeros((2, L, T, n), np.float32)
    t = np.arange(T)
    z[:, :, t, (5 * t) % n] = draw(exps[1], 2, L, T)
    w = draw(exps[0], L, 2, n, n)
    eye = np.broadcast_to(np.eye(n, dtype=np.float32), w.shape)
    got = _linear(z, w, eye) if layer == 1 else _linear(z, eye, w)
    want = np.einsum("xltk,lxok->lxto", z.astype(np.float64), w.astype(np.float64))
    # half a unit in the last place (the dropped term is 2^-33 of the product), of the
    # least normal value where a product lies below it
    bound = 2.0 ** -24 * np.maximum(np.abs(want) * 1.01, 2.0 ** -126)
    err = np.abs(got - want)
    print("  worst %.2e of the product" % (err / np.abs(want)).max(), flush=True)
    assert (err <= bound).all()


@pytest.mark.parametrize("T", [40, 900])
def test_small_products_that_count(T):
    """A tiny weight times a huge value beside ordinary terms of the same size, and sums
    of tiny weights only: as near 64 bits as sums of ordinary values."""
    n, L = 64, 12 if T > 64 else 1
    rng = np.random.default_rng(T)
    z, w = rng.standard_normal((2, L, T, n)), rng.standard_normal((L, 2, n, n))
    z[..., 0] *= 2.0 ** 110
    w[..., 0] *= 2.0 ** -118
    z[..., 1:] *= 2.0 ** -8
    z[:, :, 7] = 0                          # a row of zeros
    w[:, :, 9] = rng.standard_normal((L, 2, n)) * 2.0 ** -117
    z, w = z.astype(np.float32), w.astype(np.float32)
    eye = np.broadcast_to(np.eye(n, dtype=np.float32), w.shape)
    got = _linear(z, w, eye)
    want = np.einsum("xltk,lxok->lxto", z.astype(np.float64), w.astype(np.float64))
    mass = np.einsum("xltk,lxok->lxto", np.abs(z).astype(np.float64), np.abs(w).astype(np.float64))
    # fp32 sums of 64 terms: below 64 roundings of half a unit of the terms' total
    assert (np.abs(got - want) <= 64 * 2.0 ** -24 * mass).all()
    assert (got[:, :, 7] == 0).all()
