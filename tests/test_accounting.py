"""Closed-form accounting against the numbers the paper prints (Section 3.4 worked
example; Table tab:models).  Runs on the CPU."""
import json
import os

import pytest

from paper_2603_19664_amd import accounting as acc


@pytest.fixture(scope="module")
def golden(golden_dir):
    with open(os.path.join(golden_dir, "paper_memory.json")) as f:
        return json.load(f)


def test_worked_example(golden):
    w = golden["worked_example"]
    assert acc.kv_bytes_per_token(w["L"], w["n_kv"], w["head_dim"], w["b"]) == w["kv_bytes"]
    assert acc.residual_bytes_per_token(w["d_hidden"], w["b"]) == w["res_bytes"]
    assert round(acc.compression_ratio(w["L"], w["n_kv"], w["head_dim"], w["d_hidden"]), 1) == w["rho"]
    assert round(w["kv_bytes"] / 1024) == w["kv_kb_approx"]


def test_model_table(golden):
    for m in golden["models"]:
        kv = acc.kv_bytes_per_token(m["L"], m["n_kv"], m["head_dim"], 2) / 1024
        res = acc.residual_bytes_per_token(m["d"], 2) / 1024
        rho = acc.compression_ratio(m["L"], m["n_kv"], m["head_dim"], m["d"])
        assert round(kv, 1) == m["kv_kb"], m["model"]
        assert round(res, 1) == m["res_kb"], m["model"]
        assert round(rho, 1) == m["rho"], m["model"]
        assert round(100 * (1 - 1 / rho)) == m["saving_pct"], m["model"]


def test_rho_range(golden):
    rhos = {m["model"]: acc.compression_ratio(m["L"], m["n_kv"], m["head_dim"], m["d"]) for m in golden["models"]}
    r = golden["rho_range"]
    assert round(min(rhos.values()), 1) == r["min"] and min(rhos, key=rhos.get) == r["min_model"]
    assert round(max(rhos.values()), 1) == r["max"] and max(rhos, key=rhos.get) == r["max_model"]


def test_recompute_vs_read_intensity():
    # Eq. recomp_flops / Eq. read_bytes = d_hidden flop per byte at b = 2 (Section 3.4).
    for d, n_kv, hd in [(2560, 4, 256), (1536, 2, 128), (576, 3, 64)]:
        assert acc.recompute_flops(7, n_kv, d, hd) / acc.read_bytes(7, n_kv, hd, 2) == d


def test_total_memory_limits():
    L, n_kv, hd, d, b = 34, 4, 256, 2560, 2
    T = 1000
    # budget = T: the plain KV cache; budget = 0: residuals only (Eq. total_mem).
    assert acc.total_memory(T, T, L, n_kv, hd, d, b) == T * acc.kv_bytes_per_token(L, n_kv, hd, b)
    assert acc.total_memory(T, 0, L, n_kv, hd, d, b) == T * acc.residual_bytes_per_token(d, b)
    # growth rate in T at fixed budget is d*b per token
    assert acc.total_memory(T + 1, 64, L, n_kv, hd, d, b) - acc.total_memory(T, 64, L, n_kv, hd, d, b) == d * b


def test_fused_flops_follow_the_path_a_call_takes():
    kvd = pytest.importorskip("paper_2603_19664_amd.kvd")
    s = kvd.Shape(2560, 8, 4, 256, 1e-6, 1e4, kvd.KVD_BF16, kvd.KVD_W_PACKED)
    B, d, hd, n_q, n_kv = 16, 2560, 256, 8, 4

    def flops(T):
        return acc.fused_flops(B, T, 1, n_q, n_kv, d, hd, kvd.kvd_fused_keys_only(s, B, T, 1))

    full = lambda T: 4 * B * T * n_kv * d * hd + 4 * B * (T + 1) * n_q * hd  # noqa: E731
    # a conversation's first turn: the residual sums outgrow the workspace, K and V are recomputed
    assert not kvd.kvd_fused_keys_only(s, B, 256, 1) and flops(256) == full(256)
    # half way through: keys only
    assert kvd.kvd_fused_keys_only(s, B, 2560, 1)
    assert flops(2560) == (2 * B * 2560 * n_kv * d * hd + 2 * B * 2560 * n_q * (hd + d) + 2 * B * n_q * hd * d
                           + 4 * B * n_q * hd)
    # the largest calls too, whose scratch is more than the workspace-less call's 32 MiB
    assert kvd.kvd_fused_keys_only(s, 64, 14336, 1) and kvd.kvd_fused_keys_only(s, B, 57344, 1)
    # other head sizes, dtypes, long stored tails and forced engines recompute values too
    import dataclasses as dc
    for other in (dc.replace(s, head_dim=128), dc.replace(s, dtype=kvd.KVD_F32, w_layout=0)):
        assert not kvd.kvd_fused_keys_only(other, B, 2560, 1)
    assert not kvd.kvd_fused_keys_only(s, B, 2560, 64 * 200) and not kvd.kvd_fused_keys_only(s, 0, 2560, 1)
    try:
        kvd.kvd_set_fused_tokens(64)
        assert not kvd.kvd_fused_keys_only(s, B, 2560, 1)
    finally:
        kvd.kvd_set_fused_tokens(0)


# (d_model, query heads, KV heads, layout, B, T): measured slower with the value
# projection absorbed than on the tiled engine, then at least 10% faster
@pytest.mark.parametrize("sizes", [(1152, 4, 1, 1, 16, 2048), (1024, 4, 1, 1, 16, 1024), (2560, 4, 1, 1, 16, 4096),
                                   (1024, 8, 2, 1, 16, 1024), (1024, 8, 4, 1, 1, 4096), (1024, 16, 8, 1, 1, 2048),
                                   (1536, 6, 3, 1, 4, 1024), (2048, 8, 2, 1, 4, 1536), (1152, 4, 1, 0, 16, 1024)])
def test_calls_that_lose_by_absorption_recompute_values(sizes):
    kvd = pytest.importorskip("paper_2603_19664_amd.kvd")
    d, n_q, n_kv, layout, B, T = sizes
    assert not kvd.kvd_fused_keys_only(kvd.Shape(d, n_q, n_kv, 256, 1e-6, 1e4, kvd.KVD_BF16, layout), B, T, 1)


@pytest.mark.parametrize("sizes", [(2560, 8, 4, 1, 1, 4096), (2560, 8, 4, 1, 16, 2560), (2560, 8, 4, 0, 1, 3072),
                                   (1024, 8, 4, 1, 16, 1024), (2560, 16, 8, 1, 1, 8192), (2048, 8, 1, 1, 16, 4096),
                                   (2560, 8, 2, 1, 1, 16384), (5376, 16, 8, 1, 1, 2048)])
def test_calls_that_gain_by_absorption_recompute_keys_only(sizes):
    kvd = pytest.importorskip("paper_2603_19664_amd.kvd")
    d, n_q, n_kv, layout, B, T = sizes
    assert kvd.kvd_fused_keys_only(kvd.Shape(d, n_q, n_kv, 256, 1e-6, 1e4, kvd.KVD_BF16, layout), B, T, 1)
