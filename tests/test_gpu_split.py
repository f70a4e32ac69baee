"""The fused kernel's split tiles (mot_translate_scratch): the last tiles of a
launch cut along E*hidden over several workgroups, fp32 partial rows summed by
a second kernel, against the same call unsplit and the CPU oracle."""
import ctypes

import numpy as np
import pytest

from paper_2607_28979_amd import binding as mb
from paper_2607_28979_amd.configs import WORKLOADS, small_variant
from paper_2607_28979_amd.inputs import generate

from helpers import TOL, dst_shape, max_unit_error, oracle_dims, to_dev


def _scratch_bytes(w, lm):
    lm = np.ascontiguousarray(lm, dtype=np.int32)
    c = mb.Shapes.from_workload(w).c()
    return mb.load_library().mot_translate_scratch_bytes(ctypes.byref(c), lm.ctypes.data)


def test_scratch_rule():
    """Bytes are whole fp32 tiles; no split when the tiles fill the chip, on the
    other paths, or for invalid arguments."""
    head = WORKLOADS[3]
    one = _scratch_bytes(head.with_(B=1, T=37), range(28))
    assert one > 0 and one % (56 * 128 * 512 * 4) == 0
    assert _scratch_bytes(head, range(28)) == 0                          # 56 full rounds
    assert _scratch_bytes(head.with_(B=1, T=37, top_k=1), range(28)) == 0
    assert _scratch_bytes(WORKLOADS[2].with_(B=1, T=37), range(28)) == 0   # two-GEMM shape
    assert _scratch_bytes(head.with_(T=-1), range(28)) == 0
    assert _scratch_bytes(head.with_(B=1, T=37), [-1] * 28) == 0
    lib, c = mb.load_library(), mb.Shapes.from_workload(head.with_(B=1, T=37)).c()
    assert lib.mot_translate_scratch_bytes(ctypes.byref(c), None) == 0


@pytest.mark.parametrize("d_in,d_out,slots,rows", [(128, 128, 512, 128), (256, 128, 256, 128), (128, 256, 256, 128),
                                                   (512, 128, 256, 128), (512, 512, 256, 96)])
def test_tail_past_full_rounds(d_in, d_out, slots, rows):
    """Only the tiles past the last round that the chip holds are split: one workgroup
    per CU, two of 128 -> 128 (256 -> 128 has the LDS for two but not the registers)."""
    units, ntx = 20, slots // 20 + 2
    tail = units * ntx % slots
    sh = mb.Shapes(10, 10, 1, ntx * rows, 1, d_in, 1, d_out, 4, 4096)
    n = mb.translate_scratch_bytes(sh, range(10))
    parts, rest = divmod(n, tail * rows * d_out * 4)
    assert 0 < tail < 64 and 2 <= parts <= 16 and rest == 0


def test_no_split_where_one_workgroup_per_cu_is_faster():
    """128 -> 128, 24 layers, E * hidden 2048 and 240 tiles: unsplit 50.5 us, in two
    parts 57.3 (each CU then runs two workgroups)."""
    w = WORKLOADS[1].with_(B=1)
    assert (w.d_in, w.d_out, w.E * w.hidden, w.units()) == (128, 128, 2048, 48)
    for T, split in ((37, True), (200, True), (391, False), (600, False), (1501, True)):
        assert (_scratch_bytes(w.with_(T=T), range(24)) > 0) == split, T


# (workload, variant): one token, a partial tile of each row count (128 and 96),
# several parts that do not divide the walk, full tiles ahead of the split ones
# (one workgroup per CU, and two), usage, an unmapped layer, BHTD
CASES = {
    "one-token": (3, dict(L_src=2, L_tgt=2, B=1, T=1), {}),
    "odd-parts": (3, dict(L_src=1, L_tgt=3, B=3, T=45, hidden=192), dict(E=3)),
    "bhtd": (3, dict(L_src=2, L_tgt=2, B=2, T=37), dict(dst_layout=1, src_layout=1)),
    "tile-of-96": (4, dict(L_src=2, L_tgt=2, B=1, T=97), {}),
    "full-and-tail": (4, dict(L_src=1, L_tgt=3, B=1, T=6337, hidden=256), dict(E=4)),
    "two-per-cu": (1, dict(L_src=1, L_tgt=2, B=1, T=16777), {}),
    "masked-top2": (3, dict(L_src=2, L_tgt=3, B=1, T=65), dict(top_k=2)),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(CASES))
def test_split_matches_unsplit(name, oracle_built):
    import torch
    from oracle import oracle_translate
    base, var, kw = CASES[name]
    w = small_variant(WORKLOADS[base], **var).with_(**kw)
    lm = np.arange(w.L_tgt, dtype=np.int32) % w.L_src
    if w.L_tgt == 3:
        lm[1] = -1
    inp = generate(w)
    d = {n: to_dev(getattr(inp, n), w.dtype) for n in ("src_k", "src_v", "w1", "b1", "w2", "b2", "wr", "br")}
    sh = mb.Shapes.from_workload(w, algo=mb.ALGO_FUSED)
    c = sh.c()
    lib = mb.load_library()
    n = lib.mot_translate_scratch_bytes(ctypes.byref(c), lm.ctypes.data)
    print("case", name, "scratch", n, flush=True)
    assert n > 0
    got = {}
    for mode in ("split", "whole"):
        out = [torch.full(dst_shape(w), -3.75, dtype=torch.bfloat16, device="cuda") for _ in range(2)]
        use = torch.zeros((w.L_tgt, 2, w.E), dtype=torch.int32, device="cuda")
        args = (d["src_k"], d["src_v"], lm, d["w1"], d["b1"], d["w2"], d["b2"], d["wr"], d["br"], *out, sh)
        (mb.translate if mode == "split" else mb.translate_raw)(*args, usage=use)
        torch.cuda.synchronize()
        got[mode] = [x.float().cpu().numpy().astype(np.float64) for x in out] + [use.cpu().numpy()]
    assert np.array_equal(got["split"][2], got["whole"][2])
    for a, b in zip(got["split"][:2], got["whole"][:2]):
        # the same bf16 value, or its neighbour where the two fp32 sums fall on
        # either side of a rounding boundary (sums of hundreds of terms: 1e-5 of
        # the row's rms covers them where terms cancel)
        assert np.all(np.abs(a - b) <= 2.0 ** -7 * np.abs(b) + 1e-5 * np.sqrt(np.mean(b * b)))
        assert np.mean(a != b) < 0.01
    if w.n_tok <= 256:
        ref = oracle_translate(oracle_dims(w), inp.src_k, inp.src_v, lm, inp.w1, inp.b1, inp.w2, inp.b2, inp.wr,
                               inp.br)
        assert max_unit_error(*got["split"][:2], *ref, w, lm) <= TOL["bf16"]


@pytest.mark.gpu
def test_split_under_graph_capture():
    """The scratch of a captured call belongs to the graph: replays between
    eager calls give the eager result."""
    import torch
    w = small_variant(WORKLOADS[3], L_src=2, L_tgt=2, B=1, T=37)
    inp = generate(w)
    d = {n: to_dev(getattr(inp, n), w.dtype) for n in ("src_k", "src_v", "w1", "b1", "w2", "b2", "wr", "br")}
    out = [[torch.zeros(dst_shape(w), dtype=torch.bfloat16, device="cuda") for _ in range(2)] for _ in range(2)]
    sh = mb.Shapes.from_workload(w)

    def call(o):
        mb.translate(d["src_k"], d["src_v"], [0, 1], d["w1"], d["b1"], d["w2"], d["b2"], d["wr"], d["br"], *o, sh)

    call(out[0])
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(out[1])
    for _ in range(3):
        for o in out[1]:
            o.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(*out))
        call(out[0])
        torch.cuda.synchronize()


def _small(T, **kw):
    """A headline-like call of few layers, its arguments on the GPU and its map."""
    w = small_variant(WORKLOADS[3], L_src=2, L_tgt=2, B=1, T=T, **kw)
    inp = generate(w)
    d = {n: to_dev(getattr(inp, n), w.dtype) for n in ("src_k", "src_v", "w1", "b1", "w2", "b2", "wr", "br")}
    return w, d


def _translate(w, d, **kw):
    import torch
    out = [torch.full(dst_shape(w), -3.75, dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    mb.translate(d["src_k"], d["src_v"], [0, 1], d["w1"], d["b1"], d["w2"], d["b2"], d["wr"], d["br"], *out,
                 mb.Shapes.from_workload(w), **kw)
    torch.cuda.synchronize()
    return out


@pytest.mark.gpu
def test_scratch_argument():
    """The caller's scratch gives the bits of the allocated one and nothing is allocated;
    one byte too few, False and mot_translate give those of the unsplit call."""
    import torch
    w, d = _small(37)
    sh = mb.Shapes.from_workload(w)
    n = mb.translate_scratch_bytes(sh, [0, 1])
    assert n > 0 and n == _scratch_bytes(w, [0, 1])
    own, whole = _translate(w, d), _translate(w, d, scratch=False)
    buf = torch.full((n,), 0x5A, dtype=torch.uint8, device="cuda")
    assert not all(torch.equal(a, b) for a, b in zip(own, whole))        # (they differ in a last bit somewhere)
    out = [torch.empty_like(x) for x in own]
    args = (d["src_k"], d["src_v"], [0, 1], d["w1"], d["b1"], d["w2"], d["b2"], d["wr"], d["br"], *out, sh)
    for kw, want in ((dict(scratch=buf), own), (dict(scratch=buf[:n - 1]), whole), (dict(scratch=buf[1:n]), whole),
                     (dict(scratch=False), whole)):
        for x in out:
            x.fill_(-3.75)
        torch.cuda.reset_peak_memory_stats()
        before = torch.cuda.memory_allocated()
        mb.translate(*args, **kw)
        torch.cuda.synchronize()
        assert torch.cuda.max_memory_allocated() == before
        assert all(torch.equal(a, b) for a, b in zip(out, want)), kw.keys()
    mb.translate_raw(*args)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(out, whole))
    with pytest.raises(mb.MotError) as e:
        mb.translate(*args, scratch=torch.empty(n + 16, dtype=torch.uint8, device="cuda")[8:])
    assert e.value.name == "MOT_ERR_MISALIGNED"


@pytest.mark.gpu
def test_rows_of_a_sub_batch():
    """Without a split a token's rows keep their bits whatever else the call holds; with
    one they may move to the neighbouring bf16 value."""
    import torch
    w, d = _small(600)
    part = w.with_(T=512)
    sub = dict(d, src_k=d["src_k"][:, :, :512].contiguous(), src_v=d["src_v"][:, :, :512].contiguous())
    assert _scratch_bytes(w, [0, 1]) != _scratch_bytes(part, [0, 1])
    for a, b in zip(_translate(w, d, scratch=False), _translate(part, sub, scratch=False)):
        assert torch.equal(a[:, :, :512], b)
    for a, b in zip(_translate(w, d), _translate(part, sub)):
        a, b = a[:, :, :512].double(), b.double()
        # neighbours, or sums of cancelling terms apart by their fp32 rounding
        assert ((a - b).abs() <= 2.0 ** -7 * b.abs() + 1e-5 * b.square().mean().sqrt()).all()


@pytest.mark.gpu
def test_capture_begun_outside_torch():
    """A graph captured through the HIP runtime: the call takes no memory that torch's
    allocator would hand out again, and replays give the unsplit result."""
    import torch
    path, = mb._hip_runtimes()
    hip = ctypes.CDLL(path)
    w, d = _small(37)
    want = _translate(w, d, scratch=False)
    out = [torch.zeros_like(x) for x in want]
    args = (d["src_k"], d["src_v"], [0, 1], d["w1"], d["b1"], d["w2"], d["b2"], d["wr"], d["br"], *out,
            mb.Shapes.from_workload(w))
    torch.empty(1, dtype=torch.uint8, device="cuda")          # (its block is kept by the allocator)
    stream = torch.cuda.Stream()
    st, graph, ex = ctypes.c_void_p(stream.cuda_stream), ctypes.c_void_p(), ctypes.c_void_p()
    torch.cuda.synchronize()
    torch.cuda.reset_peak_memory_stats()
    before = torch.cuda.memory_allocated()
    with torch.cuda.stream(stream):
        assert hip.hipStreamBeginCapture(st, 2) == 0           # relaxed mode
        try:
            mb.translate(*args)
        finally:
            rc = hip.hipStreamEndCapture(st, ctypes.byref(graph))
    assert rc == 0 and torch.cuda.max_memory_allocated() - before < 4096
    assert hip.hipGraphInstantiate(ctypes.byref(ex), graph, None, None, ctypes.c_size_t(0)) == 0
    for _ in range(3):
        for x in out:
            x.zero_()
        torch.cuda.synchronize()
        assert hip.hipGraphLaunch(ex, st) == 0
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out, want))
        _translate(w, d)
    assert hip.hipGraphExecDestroy(ex) == 0 and hip.hipGraphDestroy(graph) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("workload", [1, 3, 4])
@pytest.mark.parametrize("top_k", [0, 1])
def test_rows_of_short_tiles(workload, top_k):
    """A tile's last rows, at every remainder of the groups of eight that it stores: the
    bits they have in a longer call (a routed tile holds other rows there)."""
    import torch
    w = small_variant(WORKLOADS[workload], L_src=2, L_tgt=2, B=1, T=260)
    w = w.with_(top_k=top_k or w.E)
    d = {n: to_dev(getattr(generate(w), n), w.dtype) for n in ("src_k", "src_v", "w1", "b1", "w2", "b2", "wr", "br")}
    long = _translate(w, d, scratch=False)
    for T in (1, 2, 7, 8, 9, 15, 17, 31, 33, 95, 96, 97, 127, 129, 200):
        print("case", workload, top_k, T, flush=True)
        sub = dict(d, src_k=d["src_k"][:, :, :T].contiguous(), src_v=d["src_v"][:, :, :T].contiguous())
        for a, b in zip(long, _translate(w.with_(T=T), sub, scratch=False)):
            assert torch.equal(a[:, :, :T], b)
