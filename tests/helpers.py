"""Shared test plumbing: device upload, GPU calls through the C ABI, oracle
calls, and the per-unit relative Frobenius error."""
from __future__ import annotations

import numpy as np

from paper_2607_28979_amd import binding as mb
from paper_2607_28979_amd.inputs import Inputs, bf16_bits

SENTINEL = -3.75   # exactly representable in bf16 and fp32

TOL = {"f32": 1e-5, "bf16": 2e-2}


def to_dev(a: np.ndarray, dtype: str):
    import torch
    if dtype == "f32":
        return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
    bits = bf16_bits(a)
    return torch.from_numpy(bits.view(np.int16)).cuda().view(torch.bfloat16)


def dst_shape(w):
    if w.dst_layout == 0:
        return (w.L_tgt, w.B, w.T, w.H_tgt, w.D_tgt)
    return (w.L_tgt, w.B, w.H_tgt, w.T, w.D_tgt)


def run_gpu(w, inp: Inputs, layer_map, algo=mb.ALGO_AUTO, act=mb.ACT_GELU, with_bias=True,
            dev=None, **kw):
    """Translate on the GPU through the C ABI; returns (dst_k, dst_v) as
    float64 numpy arrays in the dst layout (unmapped layers hold SENTINEL);
    kw: further arguments of translate."""
    import torch
    d = dev or {}
    if not d:
        for name in ("src_k", "src_v", "w1", "b1", "w2", "b2", "wr", "br"):
            d[name] = to_dev(getattr(inp, name), w.dtype)
    tdt = torch.float32 if w.dtype == "f32" else torch.bfloat16
    dk = torch.full(dst_shape(w), SENTINEL, dtype=tdt, device="cuda")
    dv = torch.full(dst_shape(w), SENTINEL, dtype=tdt, device="cuda")
    shapes = mb.Shapes.from_workload(w, algo=algo, act=act)
    mb.translate(d["src_k"], d["src_v"], layer_map, d["w1"], d["b1"] if with_bias else None,
                 d["w2"], d["b2"] if with_bias else None, d["wr"], d["br"] if with_bias else None,
                 dk, dv, shapes, **kw)
    torch.cuda.synchronize()
    return dk.float().cpu().numpy().astype(np.float64), dv.float().cpu().numpy().astype(np.float64)


def oracle_dims(w, act=0):
    from oracle import OracleDims
    return OracleDims(L_src=w.L_src, L_tgt=w.L_tgt, B=w.B, T=w.T, H_src=w.H_src, D_src=w.D_src,
                      H_tgt=w.H_tgt, D_tgt=w.D_tgt, E=w.E, hidden=w.hidden,
                      src_layout=w.src_layout, dst_layout=w.dst_layout, act=act,
                      top_k=w.top_k, streams=w.streams)


def unit_rows(dst, w, j):
    """Target layer j of a dst array as [B*T][d_out] (layout-aware)."""
    a = dst[j]
    if w.dst_layout == 1:
        a = a.transpose(0, 2, 1, 3)
    return a.reshape(w.B * w.T, w.d_out)


def rel_frob(got: np.ndarray, ref: np.ndarray) -> float:
    num = np.linalg.norm((got - ref).ravel())
    den = np.linalg.norm(ref.ravel())
    return float(num / den) if den > 0 else float(num)


def max_unit_error(gpu_k, gpu_v, ref_k, ref_v, w, layer_map):
    worst = 0.0
    for j in range(w.L_tgt):
        if layer_map[j] < 0:
            continue
        for g, r in ((gpu_k, ref_k), (gpu_v, ref_v)):
            worst = max(worst, rel_frob(unit_rows(g, w, j), unit_rows(r, w, j)))
    return worst


# Per-row bound: the relative L2 error of every single token row of a unit.
# In bf16 a row's error comes from the bf16 hidden activation (~1.7e-3 of the
# row), the tanh-form GELU (~2e-4) and the output rounding (~1.1e-3); its
# spread over rows is small (hundreds of independent terms per row), so the
# unit bar also holds row by row.  A defect confined to a few rows or a part
# of a row fails it even when the unit's Frobenius norm hides it.
ROW_TOL = {"f32": 1e-5, "bf16": 2e-2}


def row_errors(got: np.ndarray, ref: np.ndarray) -> np.ndarray:
    """Relative L2 error of each row (last axis)."""
    num = np.linalg.norm(got - ref, axis=-1)
    den = np.linalg.norm(ref, axis=-1)
    return num / np.where(den > 0, den, 1.0)


def src_rows(w, inp: Inputs, x: int, i: int) -> np.ndarray:
    """Source layer i of K (x = 0) or V (x = 1) as [B*T][d_in] float64."""
    a = (inp.src_k, inp.src_v)[x][i].astype(np.float64)
    if w.src_layout == 1:
        a = a.transpose(0, 2, 1, 3)
    return a.reshape(w.B * w.T, w.d_in)


def unit_logits(w, inp: Inputs, lm, j: int, x: int, rows=None) -> np.ndarray:
    """Router logits of unit (j, x) in float64, [rows][E]."""
    z = src_rows(w, inp, x, lm[j])
    if rows is not None:
        z = z[rows]
    return z @ inp.wr[j, x].astype(np.float64).T + inp.br[j, x].astype(np.float64)


def topk_margin(logits: np.ndarray, K: int) -> np.ndarray:
    """Per row: relative gap between the K-th and the (K+1)-th softmax score
    (1 when K = E).  Where it is below the fp32 resolution of the scores, fp32
    and the oracle's double may pick different, equally valid sets."""
    E = logits.shape[-1]
    if K >= E:
        return np.ones(logits.shape[0])
    g = np.exp(logits - logits.max(axis=1, keepdims=True))
    g /= g.sum(axis=1, keepdims=True)
    gs = -np.sort(-g, axis=1)
    return (gs[:, K - 1] - gs[:, K]) / gs[:, K - 1]


def admissible_sets(logit_row: np.ndarray, K: int, rel: float = 1e-3):
    """The Top-K sets a near-tie row may select (paper Sec. 3, Definition
    "Mixture-of-Translators"): translators whose softmax score lies within
    `rel` of the K-th largest form the boundary group; every set made of the
    translators clearly above the group plus any choice of the remaining
    count from the group is admissible."""
    import itertools
    g = np.exp(logit_row - logit_row.max())
    g /= g.sum()
    gk = -np.sort(-g)[K - 1]
    group = [m for m in range(g.size) if abs(g[m] - gk) <= rel * gk]
    certain = [m for m in range(g.size) if g[m] > gk and m not in group]
    need = K - len(certain)
    return [tuple(sorted(certain + list(c))) for c in itertools.combinations(group, need)]


def forced_set_router_bias(inp: Inputs, logit_row: np.ndarray, j: int, x: int, chosen, K: int,
                           rel: float = 1e-3, delta: float = 1e-4) -> np.ndarray:
    """A copy of the router bias that makes one row select `chosen` without
    ambiguity: the chosen translators keep their logits, and the others of
    the boundary group are moved to delta below the lowest chosen one.  The
    renormalised gates of the chosen set depend only on the chosen logits, so
    the forced row is the mixture over `chosen` with the row's own gates."""
    g = np.exp(logit_row - logit_row.max())
    g /= g.sum()
    gk = -np.sort(-g)[K - 1]
    group = [m for m in range(g.size) if abs(g[m] - gk) <= rel * gk]
    inside = [m for m in group if m in chosen]
    floor = min(logit_row[inside]) if inside else max(logit_row[group])
    br = inp.br.copy()
    for m in group:
        if m not in chosen:
            br[j, x, m] = np.float32(float(br[j, x, m]) + (floor - delta - logit_row[m]))
    return br


def near_tie_references(w, inp: Inputs, lm, j: int, x: int, row: int, act: int = 0):
    """Oracle rows of token `row` of unit (j, x), one per admissible Top-K
    set of that row (the oracle's own choice included)."""
    from oracle import oracle_rows
    K = w.top_k
    lg = unit_logits(w, inp, lm, j, x, rows=[row])[0]
    refs = []
    for chosen in admissible_sets(lg, K):
        br = forced_set_router_bias(inp, lg, j, x, chosen, K)
        refs.append(oracle_rows(oracle_dims(w, act), inp.src_k, inp.src_v, lm, inp.w1, inp.b1, inp.w2,
                                inp.b2, inp.wr, br, units=[(j, x)], rows=[row])[0][0])
    return refs


def check_topk_rows(w, inp: Inputs, lm, j: int, x: int, got: np.ndarray, ref: np.ndarray, rows=None,
                    act: int = 0):
    """Compare the token rows of one unit under Top-K routing.  Rows with a
    clear Top-K set are returned for the unit's Frobenius bar and must meet
    the per-row bar.  A near-tie row (K-th and (K+1)-th scores within 1e-3)
    must match the oracle row of one of its admissible sets within the
    per-row bar.  Returns (keep mask, worst row error, number of near-tie
    rows)."""
    lg = unit_logits(w, inp, lm, j, x, rows=rows)
    keep = topk_margin(lg, w.top_k) >= 1e-3
    worst = float(row_errors(got[keep], ref[keep]).max()) if keep.any() else 0.0
    assert worst <= ROW_TOL[w.dtype], ("row", j, x, worst)
    for r in np.nonzero(~keep)[0]:
        row = int(rows[r]) if rows is not None else int(r)
        cands = near_tie_references(w, inp, lm, j, x, row, act)
        errs = [float(row_errors(got[r], c)) for c in cands]
        assert min(errs) <= ROW_TOL[w.dtype], ("near-tie row", j, x, row, errs)
        worst = max(worst, min(errs))
    return keep, worst, int((~keep).sum())
