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
    # exact products up to 2^-25 and fp32 sums of up to 1024 terms: below 1e-6
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


def test_infinite_source_value():
    """An infinite source value makes its token's row NaN and no other."""
    def poke(d):
        d["z"][:, :, 0, 5, 0, 1] = np.inf
    got, ref = _run(1, 40, 2, 32, 1, 64, 2, 128, poke=poke)
    assert np.isnan(got[:, :, 5]).all() and np.isnan(ref[:, :, 5]).all()
    rest = np.arange(40) != 5
    assert np.abs(got[:, :, rest] - ref[:, :, rest]).max() < 2e-5 * np.sqrt(np.mean(ref[:, :, rest] ** 2))
