"""The prefill GEMMs' 256 x 256 tiles and the long-chunk attention, at the
shapes where their edges lie: last token tile of one to all rows, hidden sizes
and column counts that end inside a k-tile and inside an output tile, one and
several split-K slices. The reference is the layer in float64 (plain torch on
the same device); bars as in the oracle's prefill tests.
"""
import ctypes
import math

import pytest
import torch

from paper_2607_07046_amd import pack
from paper_2607_07046_amd import voltron as vt
from tests.common import FLOOR, NORM_TOL, REL_TOL

pytestmark = pytest.mark.gpu
BOTH = vt.VT_ATTN | vt.VT_FFN
EPS, BASE = 1e-5, 10000.0


def shared_blocks(T, heads, d, ctx, window=0):
    """Whether the chunk's attention shares key blocks between 128 queries."""
    return bool(vt.load_library().vt_test_long_attention(T, heads, d, ctx, window))


def gemm_plan(T, hidden, heads, kv, d, F):
    """Tile edge and slices of the QKV, O, gate/up and down GEMMs."""
    n = ctypes.c_int()
    tile = lambda N, K, residual: (vt.load_library().vt_test_prefill_tile(T, N, K, residual, ctypes.byref(n)), n.value)
    return [tile((heads + 2 * kv) * d, hidden, 0), tile(hidden, heads * d, 1), tile((F + 63) // 64 * 128, hidden, 0),
            tile(hidden, F, 1)]


def _normal(g, shape, sigma, mean=0.0):
    return torch.empty(shape, dtype=torch.float16, device="cuda").normal_(mean, sigma, generator=g)


def _rotate(v, pos0):
    T, _, d = v.shape
    i = torch.arange(d // 2, dtype=torch.float64, device=v.device)
    a = torch.arange(pos0, pos0 + T, dtype=torch.float64, device=v.device)[:, None] * BASE ** (-2.0 * i / d)
    c, s = torch.cos(a)[:, None], torch.sin(a)[:, None]
    e, o = v[..., 0::2], v[..., 1::2]
    return torch.stack((e * c - o * s, e * s + o * c), -1).reshape(v.shape)


def _rms(x, g):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS) * g.double()


def _layer(w, kc, vc, x, pa, pf, heads, kv, d, F, pos, window, h_dev):
    """h_dev: the h the FFN reads, as the boundary defines it (fp16)."""
    T = x.shape[0]
    u = _rms(x.double(), w["g_attn"])
    q = _rotate((u @ w["wq"].double().T).reshape(T, heads, d), pos)
    k = _rotate((u @ w["wk"].double().T).reshape(T, kv, d), pos)
    v = (u @ w["wv"].double().T).reshape(T, kv, d)
    tok = torch.arange(pos, pos + T, device=x.device)[:, None]
    key = torch.arange(pos + T, device=x.device)[None]
    hidden = key > tok
    if window:
        hidden |= key <= tok - window
    o = torch.empty((T, heads, d), dtype=torch.float64, device=x.device)
    for j in range(heads):
        g = j // (heads // kv)
        K, V = torch.cat((kc[g, :pos].double(), k[:, g])), torch.cat((vc[g, :pos].double(), v[:, g]))
        sc = (q[:, j] @ K.T / math.sqrt(d)).masked_fill_(hidden, -math.inf)
        o[:, j] = torch.softmax(sc, -1) @ V
    p = o.reshape(T, -1) @ w["wo"].double().T
    h = x.double() + p + pa.double()
    u = _rms(h_dev.double(), w["g_ffn"])
    gate = u @ w["wg"].double().T
    f = (gate * torch.sigmoid(gate) * (u @ w["wu"].double().T)) @ w["wd"][:, :F].double().T
    return {"p_attn": p, "h": h, "p_ffn": f, "y": h_dev.double() + f + pf.double(), "k": k.transpose(0, 1),
            "v": v.transpose(0, 1)}


def _close(got, ref, what):
    got = got.double()
    assert torch.isfinite(got).all(), what
    err = (got - ref).abs()
    floor = FLOOR * ref.square().mean(-1, keepdim=True).sqrt()  # of the row: rows differ in size
    rel = float((err / torch.maximum(ref.abs(), floor)).max())
    norm = float(err.norm() / ref.norm())
    print(f"[tiles] {what}: element-wise {rel:.4f}, normwise {norm:.6f}")
    assert rel <= REL_TOL and norm <= NORM_TOL, (what, rel, norm)


def run_layer(T, hidden, heads, kv, d, F, ctx, window=0, seed=0):
    return run_chunks([T], hidden, heads, kv, d, F, ctx, window, seed)[0]


def run_chunks(chunks, hidden, heads, kv, d, F, ctx, window=0, seed=0, scale=1.0, phases=(BOTH,), peers=True, y=True,
               pad=0, replays=0):
    """Runs the chunks one after the other, the phases of each in turn; returns the outputs
    and the float64 layer's. pad: elements of NaN after every matrix row. replays: the same calls
    as a graph, replayed between eager runs, each with the eager run's bits."""
    T = sum(chunks)
    g = torch.Generator(device="cuda").manual_seed(100 + seed)
    dims = vt.vt_layer_dims(hidden=hidden, n_heads=heads, n_kv_heads=kv, head_dim=d, ffn=F, rms_eps=EPS,
                            rope_base=BASE, window=window)
    spec = vt.vt_shard_spec_create(dims, [1.0], [1.0], 0)
    dims, info = vt.vt_shard_spec_query(spec)
    s = scale / math.sqrt(hidden)
    w, full = {"g_attn": _normal(g, (hidden,), 0.1, 1.0), "g_ffn": _normal(g, (hidden,), 0.1, 1.0)}, {}
    for n, rows, cols in (("wq", heads * d, hidden), ("wk", kv * d, hidden), ("wv", kv * d, hidden),
                          ("wo", hidden, heads * d), ("wg", F, hidden), ("wu", F, hidden), ("wd", hidden, F)):
        full[n] = torch.full((rows, pack.round_up(cols, 8) + pad), math.nan, dtype=torch.float16, device="cuda")
        w[n] = full[n][:, :cols]  # row padding: never read
        w[n].copy_(_normal(g, (rows, cols), s))
    weights = pack.struct_of({**w, **full}, dims, info, full["wd"].shape[1])
    for n in "qkvogud":
        setattr(weights, "ld_" + n, full["w" + n].shape[1])
    cap = ctx + T + 2
    kc, vc = _normal(g, (kv, cap, d), 1.0), _normal(g, (kv, cap, d), 1.0)
    k0, v0 = kc.clone(), vc.clone()
    x, pa, pf = (_normal(g, (T, hidden), 1.0) for _ in range(3))
    out = {n: torch.full((T + 1, hidden), 7.0, dtype=torch.float16, device="cuda")
           for n in ("p_attn", "h", "p_ffn", "y")}
    ws = torch.zeros(vt.vt_workspace_size(spec, T, cap), dtype=torch.uint8, device="cuda")
    view = vt.vt_kv_view(k=kc.data_ptr(), v=vc.data_ptr(), capacity=cap, n_kv_heads=kv, head_dim=d, len=ctx)

    def launch():
        t0, view.len = 0, ctx
        for n in chunks:
            io = vt.vt_layer_io(x=x[t0:].data_ptr(), peer_attn=pa[t0:].data_ptr() if peers else None,
                                peer_ffn=pf[t0:].data_ptr() if peers else None,
                                attn_partial=out["p_attn"][t0:].data_ptr(), h=out["h"][t0:].data_ptr(),
                                ffn_partial=out["p_ffn"][t0:].data_ptr(), y=out["y"][t0:].data_ptr() if y else None)
            for phase in phases:
                vt.vt_layer_prefill_chunk(spec, weights, view, io, n, ctx + t0, phase, ws.data_ptr(), ws.numel(),
                                          torch.cuda.current_stream().cuda_stream)
            t0 += n

    launch()
    if replays:
        torch.cuda.synchronize()
        eager = {n: t.clone() for n, t in out.items()}
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            launch()
        for _ in range(replays):
            for t in out.values():
                t.fill_(7.0)
            graph.replay()
            torch.cuda.synchronize()
            assert all(torch.equal(out[n], t) for n, t in eager.items())
            launch()
            torch.cuda.synchronize()
            assert all(torch.equal(out[n], t) for n, t in eager.items())
    if not peers:
        pa, pf = pa * 0, pf * 0
    torch.cuda.synchronize()
    assert int(ws[vt.VT_WS_ERROR_WORD:vt.VT_WS_ERROR_WORD + 4].view(torch.int32)) == 0
    ref = _layer(w, k0, v0, x, pa, pf, heads, kv, d, F, ctx, window, out["h"][:T])
    for n in ("p_attn", "h", "p_ffn", "y"):
        assert (out[n][T] == 7.0).all(), n  # nothing past the chunk's rows
        if n == "y" and not y:
            assert (out[n] == 7.0).all()
            continue
        _close(out[n][:T], ref[n], n)
    _close(kc[:, ctx:ctx + T], ref["k"], "keys")
    _close(vc[:, ctx:ctx + T], ref["v"], "values")
    for c, c0 in ((kc, k0), (vc, v0)):
        assert torch.equal(c[:, :ctx], c0[:, :ctx]) and torch.equal(c[:, ctx + T:], c0[:, ctx + T:])
    return out, ref


# tokens, hidden, heads, KV heads, head_dim, FFN columns, context; the tile edge and slices
# of each GEMM: every epilogue of the 256 tile whole and in each number of slices
GEMM_EDGES = [
    # QKV, O, down unsplit; K ends 8 and 3 into a k-tile
    ((2305, 4104, 24, 24, 64, 4099, 5), [(256, 1), (256, 1), (128, 1), (256, 1)]),
    # gate/up and down in 2 slices, the second with the partial k-tile
    ((777, 8192, 24, 3, 128, 10609, 130), [(128, 2), (128, 1), (256, 2), (256, 2)]),
    ((4090, 4096, 16, 16, 128, 1031, 0), [(256, 1), (256, 1), (256, 1), (128, 1)]),
    ((900, 8192, 64, 8, 128, 520, 33), [(256, 3), (256, 2), (128, 3), (128, 1)]),
    ((1290, 3080, 64, 8, 128, 520, 2), [(256, 1), (256, 3), (128, 2), (128, 1)]),
    ((777, 3080, 64, 8, 128, 520, 0), [(256, 1), (256, 4), (128, 4), (128, 1)]),
    # QKV in 2 slices, the second with a k-tile of 8
    ((579, 5128, 26, 26, 128, 520, 70), [(256, 2), (128, 2), (128, 4), (128, 1)]),
    ((900, 8192, 8, 8, 128, 520, 1), [(256, 4), (128, 1), (128, 3), (128, 1)]),
    # one row of token tiles, its second half of 12 tokens
    ((140, 8192, 8, 1, 128, 17003, 9), [(128, 4), (128, 2), (256, 3), (128, 4)]),
    ((385, 8192, 8, 1, 128, 2700, 0), [(128, 4), (128, 1), (256, 4), (128, 1)]),
    ((1290, 3080, 8, 1, 128, 5504, 3), [(128, 2), (128, 1), (128, 1), (256, 3)]),
    # down in 4 slices, the last with a k-tile of 7
    ((579, 3080, 8, 1, 128, 9351, 3), [(128, 4), (128, 2), (256, 1), (256, 4)]),
]


@pytest.mark.parametrize("shape,plan", GEMM_EDGES, ids=[f"T{s[0]}-H{s[1]}-F{s[5]}" for s, _ in GEMM_EDGES])
def test_gemm_tile_edges(shape, plan):
    assert gemm_plan(*shape[:6]) == plan
    run_layer(*shape)


@pytest.mark.parametrize("shape,plan", [GEMM_EDGES[i] for i in (0, 1, 2)], ids=["down", "gate-up-split", "O"])
def test_gemm_tile_phases_apart(shape, plan):
    """The phases as calls of their own (no gain and no sums of squares between them), no
    peers, no y, and rows of every matrix with padding."""
    assert gemm_plan(*shape[:6]) == plan
    run_chunks([shape[0]], *shape[1:], seed=3, phases=(vt.VT_ATTN, vt.VT_FFN), peers=False, y=False, pad=24)


@pytest.mark.parametrize("i", [2, 11])
def test_gemm_tiles_repeat_is_bitwise(i):
    a, b = run_layer(*GEMM_EDGES[i][0]), run_layer(*GEMM_EDGES[i][0])
    for n in a:
        assert torch.equal(a[n], b[n]), n


def test_gemm_split_repeat_is_bitwise():
    """The slices' sums are added in slice order, whichever arrives last."""
    a = run_layer(*GEMM_EDGES[1][0])
    b = run_layer(*GEMM_EDGES[1][0])
    for n in a:
        assert torch.equal(a[n], b[n]), n


def test_gemm_tile_graph_replays():
    """Two chunks, split on the 256 tile and with the shared-block attention, as one graph."""
    shape = (4104, 40, 8, 128, 6001)
    assert [p[0] for p in gemm_plan(1290, *shape)] == [256, 256, 128, 256] and shared_blocks(1290, 40, 128, 50)
    run_chunks([1290, 900], *shape, 50, seed=4, replays=3)


# attention with 128 queries per workgroup: enough heads and tokens for it, the
# last block of one query and of all, contexts that end inside a key block,
# fewer keys than queries, sliding windows inside and across blocks, GQA groups
ATTN_EDGES = [
    (3585, 512, 8, 8, 64, 64, 0, 0),
    (897, 512, 32, 8, 128, 64, 31, 0),
    (1793, 1024, 16, 2, 128, 64, 1000, 0),
    (1411, 512, 20, 4, 64, 64, 77, 33),
    (1665, 512, 18, 18, 128, 64, 500, 128),
    (1542, 512, 20, 20, 64, 64, 7, 1),
    (1792, 512, 16, 16, 128, 64, 40, 0),
    (3585, 512, 16, 16, 64, 64, 0, 0),
    (1792, 512, 24, 24, 128, 64, 40, 0),
]
SEPARATE = [ATTN_EDGES[0], ATTN_EDGES[6]]  # the 32-query kernel's, the others the shared blocks'


@pytest.mark.parametrize("shape", ATTN_EDGES, ids=[f"T{s[0]}-q{s[2]}-d{s[4]}-w{s[7]}" for s in ATTN_EDGES])
def test_long_attention_edges(shape):
    T, _, heads, _, d, _, ctx, window = shape
    assert shared_blocks(T, heads, d, ctx, window) == (shape not in SEPARATE)
    run_layer(*shape, seed=1)


@pytest.mark.parametrize("seed", [1, 2])
@pytest.mark.parametrize("shape", [(512, 16, 16, 128, 64, 768), (512, 32, 8, 64, 64, 33)], ids=["d128", "d64"])
def test_long_attention_error(shape, seed):
    """The shared-block attention is no further from float64 than the 32-query
    one, which the same tokens take in four chunks (0.4% of the error was lost with one
    exact weight per group of waves; 1e-3 is for the GEMMs' other order of sums)."""
    err = []
    _, heads, _, d, _, ctx = shape
    assert shared_blocks(1792, heads, d, ctx)
    assert not any(shared_blocks(448, heads, d, ctx + t) for t in range(0, 1792, 448))
    for chunks in ([1792], [448] * 4):
        out, ref = run_chunks(chunks, *shape, seed=seed, scale=1.28)
        err.append(float((out["p_attn"][:1792].double() - ref["p_attn"]).norm() / ref["p_attn"].norm()))
    print(f"[tiles] p_attn error: shared blocks {err[0]:.4e}, 32 queries {err[1]:.4e}")
    assert err[0] <= err[1] * (1 + 1e-3), err


def test_long_attention_large_scores():
    """Scores of 2^17 and an eighth more from key block to key block, exact in fp32:
    every block moves the running maximum. The values tell the last eight blocks
    from the others, so a weight that changes with the rescales shows."""
    T, H, heads, d, ctx = 1793, 64, 32, 64, 2048
    assert shared_blocks(T, heads, d, ctx)
    g = torch.Generator(device="cuda").manual_seed(5)
    dims = vt.vt_layer_dims(hidden=H, n_heads=heads, n_kv_heads=heads, head_dim=d, ffn=64, rms_eps=1e-6,
                            rope_base=1e30, window=0)
    spec = vt.vt_shard_spec_create(dims, [1.0], [1.0], 0)
    dims, info = vt.vt_shard_spec_query(spec)
    x = torch.sign(_normal(g, (T, H), 1.0))
    x[x == 0] = 1.0
    x[:, 0] = 1.0  # the norm of +-1 rows is 1: u = x to the bit
    one = lambda n: torch.ones(n, dtype=torch.float16, device="cuda")
    w = {"g_attn": one(H), "g_ffn": one(H)}
    for n, rows in (("wq", heads * d), ("wk", heads * d), ("wv", heads * d)):
        w[n] = torch.zeros((rows, H), dtype=torch.float16, device="cuda")
    w["wq"][62::d, 0], w["wq"][63::d, 0] = 2048.0, 1.0  # the last pair does not rotate at this base
    w["wo"] = _normal(g, (H, heads * d), 1.0 / math.sqrt(heads * d))
    w["wg"], w["wu"], w["wd"] = (_normal(g, (64, 64), 0.1) for _ in range(3))
    kc = torch.zeros((heads, ctx + T, d), dtype=torch.float16, device="cuda")
    vc = torch.zeros_like(kc)
    block = torch.arange(ctx, device="cuda") // 32
    kc[:, :ctx, 62], kc[:, :ctx, 63] = 512.0, block.half()
    sign = torch.where(block < 56, 1.0, -1.0)
    vc[:, :ctx] = (sign[None, :, None] * (1.0 + 0.25 * torch.rand((heads, 1, d), generator=g, device="cuda"))).half()
    ws = torch.zeros(vt.vt_workspace_size(spec, T, ctx + T), dtype=torch.uint8, device="cuda")
    out = {n: torch.empty((T, H), dtype=torch.float16, device="cuda") for n in ("p", "h")}
    io = vt.vt_layer_io(x=x.data_ptr(), attn_partial=out["p"].data_ptr(), h=out["h"].data_ptr())
    view = vt.vt_kv_view(k=kc.data_ptr(), v=vc.data_ptr(), capacity=ctx + T, n_kv_heads=heads, head_dim=d, len=ctx)
    vt.vt_layer_prefill_chunk(spec, pack.struct_of(w, dims, info, 64), view, io, T, ctx, vt.VT_ATTN, ws.data_ptr(),
                              ws.numel(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    # the chunk's own keys are zero: 1.3e5 below the others, weight 0
    assert not kc[:, ctx:].any()
    p = torch.softmax((2048.0 * 512.0 + block.double()) / 8.0, 0)
    o = (p[None, :, None] * vc[:, :ctx].double()).sum(1).reshape(1, -1)
    _close(out["p"], (o @ w["wo"].double().T).expand(T, H), "p_attn")


@pytest.mark.parametrize("d", [64, 128])
def test_long_attention_infinite_value_after_the_queries(d):
    """A token whose value overflows to infinity leaves the queries of the 32-token
    groups before its own as they are, though it shares their last key block."""
    T, H, heads, F, ctx, bad = 1793, 512, 32, 64, 5, 32 * 9
    assert shared_blocks(T, heads, d, ctx)
    g = torch.Generator(device="cuda").manual_seed(7)
    dims = vt.vt_layer_dims(hidden=H, n_heads=heads, n_kv_heads=heads, head_dim=d, ffn=F, rms_eps=EPS,
                            rope_base=BASE, window=0)
    spec = vt.vt_shard_spec_create(dims, [1.0], [1.0], 0)
    dims, info = vt.vt_shard_spec_query(spec)
    s = 1.0 / math.sqrt(H)
    w = {n: _normal(g, shape, s) for n, shape in
         (("wq", (heads * d, H)), ("wk", (heads * d, H)), ("wv", (heads * d, H)), ("wo", (H, heads * d)),
          ("wg", (F, H)), ("wu", (F, H)), ("wd", (H, F)))}
    w["g_attn"], w["g_ffn"] = _normal(g, (H,), 0.1, 1.0), _normal(g, (H,), 0.1, 1.0)
    w["wv"][:, 0] = 3e4
    x = _normal(g, (T, H), 1.0)
    x[:, 0] = 0.0
    outs = []
    for big in (False, True):
        if big:
            x[bad] = 0.0
            x[bad, 0] = 1.0  # normalised to sqrt(H) = 22.6: a value of 6.8e5
        kc = torch.zeros((heads, ctx + T, d), dtype=torch.float16, device="cuda")
        vc = torch.zeros_like(kc)
        kc[:, :ctx], vc[:, :ctx] = 0.5, 1.0
        ws = torch.zeros(vt.vt_workspace_size(spec, T, ctx + T), dtype=torch.uint8, device="cuda")
        out = {n: torch.empty((T, H), dtype=torch.float16, device="cuda") for n in ("p", "h")}
        io = vt.vt_layer_io(x=x.data_ptr(), attn_partial=out["p"].data_ptr(), h=out["h"].data_ptr())
        view = vt.vt_kv_view(k=kc.data_ptr(), v=vc.data_ptr(), capacity=ctx + T, n_kv_heads=heads, head_dim=d, len=ctx)
        vt.vt_layer_prefill_chunk(spec, pack.struct_of(w, dims, info, F), view, io, T, ctx, vt.VT_ATTN, ws.data_ptr(),
                                  ws.numel(), torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert bool(torch.isinf(vc[:, ctx + bad]).all()) == big
        outs.append(out["p"])
    assert torch.isfinite(outs[0]).all()
    assert torch.equal(outs[0][:bad], outs[1][:bad])
