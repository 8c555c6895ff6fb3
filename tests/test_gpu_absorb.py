"""The value-absorbed fused path (kvd_fused_recompute_attn in automatic mode, bf16,
head_dim 256, sizes that kvd_fused_keys_only names) against the fp64 oracle and the
tiled engines, at the edges of its tiles: ragged token tiles and 32-token steps, a
last half column slice, one and several ranges per sequence, packed and split
query-head rows, one and two passes over a KV head's query heads and over d_model
(W_v product), every kind of stored tail, each score tile.

Tolerance: as the tiled engines', 2e-2 of the largest value; the 2-norm error
against the oracle is besides no larger than the tiled engine's (keys and values
are rounded there and not here) plus a tenth."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2603_19664_amd import configs as C
from paper_2603_19664_amd import kvd

from gpu_cases import empty_kv, err, f64, gpu_fused, gpu_project, gpu_recompute, make_layer, note, oracle_decode

pytestmark = pytest.mark.gpu
TOL = 2e-2


@pytest.fixture(autouse=True)
def _announce(request):
    note(f"[gpu] {request.node.nodeid}")
    yield
    torch.cuda.synchronize()
    kvd.kvd_set_fused_tokens(0)


def _bits(t):
    return t.view(torch.int16)


def _layer(B, T, d=1024, n_q=8, n_kv=4, **kw):
    return make_layer(C.GEMMA3_4B, B=B, T=T, seed=B + T + d, d_model=d, n_q=n_q, n_kv=n_kv,
                      pos0=[(37 * b) % 1000 for b in range(B)], **kw)


def _rel(x, ref):
    x = f64(x) if isinstance(x, torch.Tensor) else x
    return float(np.linalg.norm(x - ref) / np.linalg.norm(ref))


def _counters(ws, L):
    s = L.shape
    n = -(-L.B * s.n_kv_heads * 8 // 256) * 256 + -(-L.B * s.n_kv_heads * 4 * 8 // 256) * 256
    return int(torch.count_nonzero(ws[:n]))


@pytest.mark.parametrize("packed", [False, True, "gamma"])
@pytest.mark.parametrize("B,T,d,n_q,n_kv", [
    (28, 450, 1024, 8, 4),     # ragged tiles, one range, 2 query heads per KV head
    (28, 449, 1088, 8, 4),     # a last half column slice, one token past a tile
    (14, 449, 1024, 16, 8),    # 16 query heads: two-part rows
    (28, 512, 1024, 9, 3),     # 768 K rows: 256-row tiles only
    (60, 1000, 1024, 5, 1),    # one KV head
    (24, 700, 1024, 12, 1),    # its query heads in two passes of the score epilogue
    (24, 700, 1024, 16, 1),
    (4, 1700, 3584, 16, 8),    # two passes of the W_v product over d_model
    (1, 4133, 2560, 8, 4),     # several ranges, a ragged last step
    (12, 1025, 1216, 16, 4)])  # several ranges, 16 query heads, half slice
def test_absorbed_vs_oracle(B, T, d, n_q, n_kv, packed):
    L = _layer(B, T, d, n_q, n_kv, packed=packed)
    assert kvd.kvd_fused_keys_only(L.shape, B, T, 1)
    q, _, out, _ = gpu_fused(L)
    sel = sorted({0, B // 2, B - 1})
    ref = oracle_decode(L, b_sel=sel)
    e = err(f64(out[sel]), ref)
    kvd.kvd_set_fused_tokens(64)
    _, _, tiled, _ = gpu_fused(L, q=q)
    r, rt = _rel(out[sel], ref), _rel(tiled[sel], ref)
    note(f"    err {e:.3e}, 2-norm {r:.3e} (tiled {rt:.3e})")
    assert e < TOL and r <= 1.1 * rt
    assert not torch.equal(_bits(out), _bits(tiled))  # the absorbed path ran
    assert err(f64(out), f64(tiled)) < TOL


@pytest.mark.parametrize("B,T,d,n_q,n_kv,T_tail,t_cap,t_off", [
    (28, 450, 1024, 8, 4, *t) for t in [(0, 1, 0), (1, 1, 0), (4, 7, 5), (5, 9, 2), (64, 64, 63), (68, 100, 60),
                                        (70, 80, 33), (200, 211, 150)]] + [
    (12, 1025, 1216, 16, 4, 200, 211, 150),   # several ranges per sequence
    (24, 700, 1024, 16, 1, 90, 90, 77)])      # 16 query heads per KV head
def test_absorbed_stored_tail(B, T, d, n_q, n_kv, T_tail, t_cap, t_off):
    # a ring of t_cap slots read from slot t_off, wrapping: rows T .. T + T_tail - 1
    L = _layer(B, T + T_tail, d, n_q, n_kv)
    assert kvd.kvd_fused_keys_only(L.shape, B, T, T_tail)
    s = L.shape
    K, V = gpu_recompute(L)
    rk, rv = empty_kv(L, t_cap)
    for i in range(T_tail):
        rk[:, :, (t_off + i) % t_cap] = K[:, :, T + i]
        rv[:, :, (t_off + i) % t_cap] = V[:, :, T + i]
    q = gpu_project(L)

    def run(mode):
        kvd.kvd_set_fused_tokens(mode)
        ws = kvd.workspace(s, kvd.KVD_OP_FUSED, B, T, T_tail)
        outs = []
        for _ in range(2):
            o = torch.empty_like(q)
            kvd.kvd_fused_recompute_attn(s, q, L.h, T, L.gamma, L.lw_k, L.lw_v, L.pos0, o, ws,
                                         rk if T_tail else None, rv if T_tail else None, T_tail, t_off)
            outs.append(o)
        assert torch.equal(_bits(outs[0]), _bits(outs[1])) and _counters(ws, L) == 0
        return outs[0]

    out, tiled = run(0), run(64)
    sel = [0, B - 1]
    pos = f64(L.pos0)[sel][:, None] + np.arange(T)[None, :]
    ref = O.kv_direct_decode(f64(q)[sel], f64(L.h[sel, :T]), f64(L.gamma), f64(L.w_k), f64(L.w_v), pos,
                             f64(K[sel, :, T:]) if T_tail else None, f64(V[sel, :, T:]) if T_tail else None,
                             s.n_kv_heads, s.head_dim, s.rms_eps, s.rope_theta)
    e, r, rt = err(f64(out[sel]), ref), _rel(out[sel], ref), _rel(tiled[sel], ref)
    note(f"    err {e:.3e}, 2-norm {r:.3e} (tiled {rt:.3e})")
    assert e < TOL and r <= 1.1 * rt and not torch.equal(_bits(out), _bits(tiled))


@pytest.mark.parametrize("B,T,n_q,n_kv,packed", [(16, 1000, 8, 4, True), (16, 1000, 8, 4, False),
                                                 (9, 2048, 8, 8, True), (5, 1500, 6, 3, True), (2, 3000, 8, 4, "gamma"),
                                                 (18, 448, 8, 4, False), (16, 640, 6, 3, "gamma")])
def test_absorbed_score_tiles(B, T, n_q, n_kv, packed):
    # grids on both sides of the score tiles' rule (512 x 64, 256 x 128, 256 x 64; the
    # last two: 512 x 64 of row-major and 256 x 128 of folded weights), and the call
    # without a workspace argument
    L = _layer(B, T, 1024, n_q, n_kv, packed=packed)
    s = L.shape
    q, (tk, tv), out, _ = gpu_fused(L)
    na = torch.empty_like(out)
    kvd.kvd_fused_recompute_attn_noalloc(s, q, L.h, T, L.gamma, L.lw_k, L.lw_v, L.pos0, na, tk, tv, 1)
    assert torch.equal(_bits(out), _bits(na))
    kvd.kvd_set_fused_tokens(64)
    _, _, tiled, _ = gpu_fused(L, q=q)
    ref = oracle_decode(L, b_sel=[B - 1])
    e, r, rt = err(f64(out), f64(tiled)), _rel(out[B - 1:], ref), _rel(tiled[B - 1:], ref)
    note(f"    vs tiled {e:.3e}, 2-norm vs oracle {r:.3e} (tiled {rt:.3e})")
    assert e < TOL and r <= 1.1 * rt and not torch.equal(_bits(out), _bits(tiled))


def test_absorbed_window_and_longer_store():
    # a window over a longer checkpoint store (row stride h_ld > T), positions from 0
    B, T, W = 28, 900, 451
    L = _layer(B, T, 1024)
    s = L.shape
    q = torch.empty((B, s.n_q_heads, s.head_dim), dtype=s.torch_dtype, device="cuda")
    tk, tv = empty_kv(L, 1)
    pos = torch.full((B,), W - 1, dtype=torch.int32, device="cuda")
    kvd.kvd_project_qkv(s, L.h_new, L.gamma, L.lw_q, L.lw_k, L.lw_v, pos, q, tk, tv, 0)
    out = torch.empty_like(q)
    ws = kvd.workspace(s, kvd.KVD_OP_FUSED, B, W - 1, 1)
    kvd.kvd_fused_window_attn(s, q, L.h, T, L.gamma, L.lw_k, L.lw_v, W, out, ws, tk, tv, 1)
    assert kvd.kvd_fused_keys_only(s, B, W - 1, 1)
    tiled = torch.empty_like(q)
    kvd.kvd_set_fused_tokens(64)
    kvd.kvd_fused_window_attn(s, q, L.h, T, L.gamma, L.lw_k, L.lw_v, W, tiled, ws, tk, tv, 1)
    assert not torch.equal(_bits(out), _bits(tiled))  # the absorbed path ran
    sel = [0, B - 1]
    ref = O.sliding_window_decode(f64(L.h_new[sel]), f64(L.h[sel, :T]), f64(L.gamma), f64(L.w_q), f64(L.w_k),
                                  f64(L.w_v), W, s.n_q_heads, s.n_kv_heads, s.head_dim, s.rms_eps, s.rope_theta)
    assert err(f64(out[sel]), ref) < TOL


@pytest.mark.parametrize("B,T,d", [(28, 450, 1024), (1, 4133, 2560), (4, 4096, 1024)])
def test_workspace_size_and_path(B, T, d):
    # the documented size and any larger one give the same bits (the ranges of a
    # sequence do not follow the buffer); a smaller workspace that holds the tiled
    # engine's splits was accepted before and still is, and runs that engine
    L = _layer(B, T, d)
    s = L.shape
    q, (tk, tv), ref, _ = gpu_fused(L)
    up = lambda x: -(-x // 256) * 256  # noqa: E731
    S = kvd.kvd_num_splits(s, kvd.KVD_OP_FUSED, B, T, 1)
    doc = kvd.kvd_workspace_bytes(s, kvd.KVD_OP_FUSED, B, T, 1)
    least = (up(B * s.n_kv_heads * 8) + up(B * s.n_kv_heads * 32) + up(B * s.n_q_heads * S * s.head_dim * 4)
             + up(B * s.n_q_heads * S * 8))
    assert least < doc
    out = {}
    for n in (least, doc - 256, doc, doc + 256, 4 * doc):
        ws = torch.zeros(n, dtype=torch.uint8, device="cuda")
        out[n] = torch.empty_like(q)
        kvd.kvd_fused_recompute_attn(s, q, L.h, T, L.gamma, L.lw_k, L.lw_v, L.pos0, out[n], ws, tk, tv, 1)
        assert _counters(ws, L) == 0
    kvd.kvd_set_fused_tokens(64 if S == -(-T // 64) else 128)
    assert kvd.kvd_num_splits(s, kvd.KVD_OP_FUSED, B, T, 1) == S
    _, _, tiled, _ = gpu_fused(L, q=q)
    assert not torch.equal(_bits(ref), _bits(tiled))
    for n, o in out.items():
        assert torch.equal(_bits(o), _bits(tiled if n < doc else ref)), n


def test_absorbed_scratch_larger_than_the_workspace():
    # B = 16 x 512 tokens at d 2560: the residual sums alone outgrow the documented
    # workspace, so the call runs the tiled engine its sizes give
    L = _layer(16, 512, 2560)
    s = L.shape
    q, _, out, _ = gpu_fused(L)
    S = kvd.kvd_num_splits(s, kvd.KVD_OP_FUSED, 16, 512, 1)
    kvd.kvd_set_fused_tokens(512 // S)
    assert kvd.kvd_num_splits(s, kvd.KVD_OP_FUSED, 16, 512, 1) == S
    _, _, tiled, _ = gpu_fused(L, q=q)
    assert torch.equal(_bits(out), _bits(tiled))


@pytest.mark.parametrize("T,noalloc", [(16000, True), (36000, False)])
def test_absorbed_beyond_the_static_scratch(T, noalloc):
    # sizes whose workspace is larger than the static scratch: where the call without
    # a workspace takes them it gives the same bits, and beyond the path is the same
    L = _layer(16, T)
    s = L.shape
    assert kvd.kvd_workspace_bytes(s, kvd.KVD_OP_FUSED, 16, T, 1) > 32 << 20 and kvd.kvd_fused_keys_only(s, 16, T, 1)
    q, (tk, tv), out, _ = gpu_fused(L)
    na = torch.empty_like(out)

    def call():
        kvd.kvd_fused_recompute_attn_noalloc(s, q, L.h, T, L.gamma, L.lw_k, L.lw_v, L.pos0, na, tk, tv, 1)

    if noalloc:
        call()
        assert torch.equal(_bits(out), _bits(na))
    else:
        with pytest.raises(kvd.KvdError):
            call()
    kvd.kvd_set_fused_tokens(128)
    _, _, tiled, _ = gpu_fused(L, q=q)
    ref = oracle_decode(L, b_sel=[15])
    r, rt = _rel(out[15:], ref), _rel(tiled[15:], ref)
    note(f"    2-norm vs oracle {r:.3e} (tiled {rt:.3e})")
    assert err(f64(out), f64(tiled)) < TOL and r <= 1.1 * rt and not torch.equal(_bits(out), _bits(tiled))


def test_absorbed_under_capture():
    L = _layer(1, 4133, 2560)
    s = L.shape
    q, (tk, tv), ref, _ = gpu_fused(L)
    ws = kvd.workspace(s, kvd.KVD_OP_FUSED, 1, L.T, 1)
    out = torch.empty_like(q)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        kvd.kvd_fused_recompute_attn(s, q, L.h, L.T, L.gamma, L.lw_k, L.lw_v, L.pos0, out, ws, tk, tv, 1)
    for _ in range(4):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(_bits(out), _bits(ref))


@pytest.mark.parametrize("B,T,d,n_q,n_kv", [(1, 4133, 2560, 8, 4), (12, 1025, 1216, 16, 4),
                                              (2, 6200, 2560, 8, 2)])
def test_workspace_with_only_the_split_counters_zero(B, T, d, n_q, n_kv):
    # kvd.h asks for zero split counters and nothing else: calls of several ranges on
    # a workspace whose other bytes hold anything equal the call on a zeroed one,
    # the first time and again
    L = _layer(B, T, d, n_q, n_kv)
    s = L.shape
    q, (tk, tv), ref, _ = gpu_fused(L)
    ws = kvd.workspace(s, kvd.KVD_OP_FUSED, B, T, 1)
    n = -(-B * n_kv * 8 // 256) * 256
    for fill in (0xFF, 0x01, 0x03):
        ws[n:] = fill
        for _ in range(2):
            out = torch.empty_like(q)
            kvd.kvd_fused_recompute_attn(s, q, L.h, T, L.gamma, L.lw_k, L.lw_v, L.pos0, out, ws, tk, tv, 1)
            assert torch.equal(_bits(out), _bits(ref))
        assert int(torch.count_nonzero(ws[:n])) == 0
