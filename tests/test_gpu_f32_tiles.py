"""The fp32 engines at the edges of their tiles: the one-wave and the staged
projection, and the fused call with the K and V rows of a tile in two workgroups
(at most 128 tiles) or in one.  K/V of every producer are bit-identical; fused
attention in both forms equals the stored-K/V attention bit for bit where they
share 64-key chunks; all against the fp64 oracle to 1e-5 of the largest value."""
import pytest
import torch

from paper_2603_19664_amd import configs as C
from paper_2603_19664_amd import kvd

from gpu_cases import err, f64, gpu_fused, gpu_recompute, gpu_unfused, make_layer, note, oracle_decode, oracle_kv

pytestmark = pytest.mark.gpu
TOL = 1e-5


@pytest.fixture(autouse=True)
def _announce(request):
    note(f"[gpu] {request.node.nodeid}")
    yield
    torch.cuda.synchronize()


def _bits(t):
    return t.view(torch.int32)


# d 64: one K-step; 576: an odd number of K-steps; hd 256: two row blocks per wave
@pytest.mark.parametrize("d,n_q,n_kv,hd", [(64, 3, 3, 64), (576, 9, 3, 64), (320, 4, 2, 128), (128, 2, 1, 256)])
@pytest.mark.parametrize("B,T", [(1, 1), (1, 17), (2, 64), (3, 129), (2, 700)])
def test_f32_producers_agree(d, n_q, n_kv, hd, B, T):
    L = make_layer(C.SMOLLM_FP32, B=B, T=T, seed=d + T, d_model=d, n_q=n_q, n_kv=n_kv, head_dim=hd,
                   pos0=[11 * b for b in range(B)])
    K, V = gpu_recompute(L)
    ok, ov = oracle_kv(L)
    assert err(f64(K), ok) < TOL and err(f64(V), ov) < TOL
    # the same rows recomputed a few at a time (the one-wave form)
    n = min(T, 5)
    sub = make_layer(C.SMOLLM_FP32, B=B, T=T, seed=d + T, d_model=d, n_q=n_q, n_kv=n_kv, head_dim=hd,
                     pos0=[11 * b for b in range(B)])
    sub.T = n
    Ks, Vs = gpu_recompute(sub)
    assert torch.equal(_bits(Ks), _bits(K[:, :, :n])) and torch.equal(_bits(Vs), _bits(V[:, :, :n]))
    # the fused kernel's own K/V, and its attention
    q, _, out, (dk, dv) = gpu_fused(L, kv_debug=True)
    assert torch.equal(_bits(dk), _bits(K)) and torch.equal(_bits(dv), _bits(V))
    e = err(f64(out), oracle_decode(L))
    note(f"    B={B} T={T} d={d} hd={hd}: err {e:.2e}")
    assert e < TOL
    _, _, again, _ = gpu_fused(L, q=q)
    assert torch.equal(_bits(out), _bits(again))


@pytest.mark.parametrize("B,T", [(2, 256), (20, 256)])
def test_f32_fused_equals_stored_attention(B, T):
    # 3 KV heads x B x 4 tiles: 24 (K and V in two workgroups) and 240 (in one); no
    # tail, so both calls chunk the keys alike
    L = make_layer(C.SMOLLM_FP32, B=B, T=T, seed=5, pos0=[7 * b for b in range(B)])
    s = L.shape
    q, K, V, _ = gpu_unfused(L)
    ref, out = torch.empty_like(q), torch.empty_like(q)
    ws = kvd.workspace(s, kvd.KVD_OP_DECODE_ATTN, B, T)
    kvd.kvd_decode_attn(s, q, K, V, T, ref, ws)
    ws = kvd.workspace(s, kvd.KVD_OP_FUSED, B, T)
    for _ in range(2):
        kvd.kvd_fused_recompute_attn(s, q, L.h, T, L.gamma, L.lw_k, L.lw_v, L.pos0, out, ws)
        assert torch.equal(_bits(out), _bits(ref))
    n = -(-B * s.n_kv_heads * 8 // 256) * 256 + -(-B * s.n_kv_heads * 32 // 256) * 256
    assert int(torch.count_nonzero(ws[:n])) == 0  # counters and completion words


# one KV head x 40 and 41 chunks: more than the counter's high half has flags for; a
# stored tail of 70 rows beside the roles; 240 tiles: both halves in one workgroup
@pytest.mark.parametrize("B,T,n_q,n_kv,n_tail", [(1, 256, 9, 3, 1), (2, 300, 9, 3, 70), (1, 2560, 3, 1, 1),
                                                 (3, 2600, 2, 1, 0), (20, 256, 9, 3, 1)])
def test_f32_workspace_with_only_the_split_counters_zero(B, T, n_q, n_kv, n_tail):
    # kvd.h asks for zero split counters and nothing else: on a workspace whose other
    # bytes hold anything (a completion flag set, a count reached) the call gives the
    # zeroed workspace's bits, the first time and again
    L = make_layer(C.SMOLLM_FP32, B=B, T=T + n_tail, seed=T, n_q=n_q, n_kv=n_kv, pos0=[5 * b for b in range(B)])
    s = L.shape
    K, V = gpu_recompute(L)
    q = torch.randn((B, n_q, s.head_dim), device="cuda")
    n = B * n_kv * 8  # the counters alone, without their block's padding

    def call(ws, out):
        kvd.kvd_fused_recompute_attn(s, q, L.h, T, L.gamma, L.lw_k, L.lw_v, L.pos0, out, ws, K if n_tail else None,
                                     V if n_tail else None, n_tail, T if n_tail else 0)

    ws = kvd.workspace(s, kvd.KVD_OP_FUSED, B, T, n_tail)
    ref = torch.empty_like(q)
    call(ws, ref)
    for fill in (0xFF, 0x01):
        ws[n:] = fill
        for _ in range(2):
            out = torch.empty_like(q)
            call(ws, out)
            assert torch.equal(_bits(out), _bits(ref))
        assert int(torch.count_nonzero(ws[:n])) == 0
    # partials only: the counters may hold anything and are not touched
    ws[:] = 0xFF
    call(ws, None)
    assert bool((ws[:n] == 0xFF).all())
    out = torch.empty_like(q)
    kvd.kvd_combine(s, B, kvd.kvd_num_splits(s, kvd.KVD_OP_FUSED, B, T, n_tail), ws, out)
    assert torch.equal(_bits(out), _bits(ref))
