"""Rank-64 decode of several requests: its splits follow the requests' lengths.
Against the oracle for lengths on the tile edges, empty and uneven requests, the
smallest and largest batch that balances and one more; paged (block table in
LDS, and the form for tables too long for it) against contiguous; and, through
the C ABI, with no more workspace than the call insists on."""
import ctypes
import re

import pytest
import torch

import paper_2609_34054_amd as prc
from paper_2609_34054_amd import binding
from gpu_cases import ATOL_MAX, ATOL_MEAN, LSE_ATOL, attn_errors, gpu_attention, lse_error, oracle_attention, to_dev
from test_gpu_paged import block_table, mk_cfg, to_pool
from workload import attention_case

pytestmark = pytest.mark.gpu

# id, n_q, n_kv, kv_lens, s_cap, block
CASES = [
    ("two_uneven", 8, 2, [8192, 1], 8192, 64),
    ("eight_edges", 16, 8, [4096, 31, 32, 33, 2047, 1, 4095, 1000], 32768, 64),
    ("ten_heads", 10, 10, [700, 5000, 64], 16384, 128),
    ("batch_64", 4, 1, [1 + (i * 613) % 2900 for i in range(64)], 3072, 64),
    ("batch_65", 4, 1, [1 + (i * 211) % 640 for i in range(65)], 640, 64),
    ("long_tables", 4, 1, [33, 131100], 131136, 64),  # 2049 blocks
    # Paged calls in the contiguous calls' form (V by direct loads): full
    # workgroups of eight KV heads and splits of more than 24 tiles.
    ("two_uneven_direct", 8, 8, [49200, 1], 49216, 64),
    ("sixteen_heads_direct", 16, 16, [700, 16300, 64], 16384, 128),
    ("batch_64_direct", 8, 8, [1 + (i * 613) % 2900 for i in range(64)], 3072, 64),
]
SAME_FORM = ("eight_edges", "two_uneven_direct", "sixteen_heads_direct", "batch_64_direct")


def _paged(g, c, cfg, blk, **kw):
    B, s_cap = c["K_base"].shape[:2]
    mb = s_cap // blk
    tbl = block_table(B, mb, B * mb + 2, 23)
    p = {k: to_pool(c[k], tbl, blk, B * mb + 2).cuda() for k in ("K_base", "V_base", "L_k", "L_v")}
    return prc.lr_shared_attention_paged(g["Q"], p["K_base"], p["V_base"], p["L_k"], p["L_v"], g["B_k"], g["B_v"],
                                         g["positions"], g["kv_len"], tbl.cuda(), rope_theta=cfg.theta, want_lse=True,
                                         **kw)


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_balanced_decode(case):
    cid, n_q, n_kv, kv_lens, s_cap, blk = case
    print(f"balanced {cid}", flush=True)
    cfg = mk_cfg(60 + len(cid), n_q, n_kv, 128, 64)
    c = attention_case(cfg, batch=len(kv_lens), n_tok=1, kv_len=kv_lens, positions=[[k - 1] for k in kv_lens],
                       s_cap=s_cap, seed_base=7 * len(cid), poison_tail=True)
    g = to_dev(c)
    Oref, lref = oracle_attention(c, cfg.theta)
    # A request of one or two keys has outputs above unit scale; their bf16
    # rounding (2^-9 of the value) scales with them.
    scale = max(1.0, float(abs(Oref).max()) / 2)
    O, lse = gpu_attention(g, cfg.theta)
    Op, lp = _paged(g, c, cfg, blk)
    torch.cuda.synchronize()
    for o, l in ((O, lse), (Op, lp)):
        mx, mean = attn_errors(o, Oref)
        assert mx <= ATOL_MAX * scale and mean <= ATOL_MEAN * scale, (mx, mean)
        assert lse_error(l, lref) <= LSE_ATOL
    if cid in SAME_FORM:  # the same kernel on the same splits
        assert torch.equal(O, Op) and torch.equal(lse, lp)


def test_balanced_empty_requests():
    """Requests without a visible key, alone and beside a long one, over stale partials."""
    cfg = mk_cfg(91, 8, 2, 128, 64)
    c = attention_case(cfg, batch=3, n_tok=1, kv_len=[8000, 7000, 16], positions=[[7999], [6999], [15]], s_cap=8192)
    g = to_dev(c)
    dims = prc.make_dims(g["Q"], g["K_base"], g["L_k"], g["L_v"], g["B_k"], g["B_v"], cfg.theta)
    ws = torch.full((prc.workspace_size(dims),), 255, dtype=torch.uint8, device="cuda")
    call = lambda kvl, pos, w: prc.lr_shared_attention(  # noqa: E731
        g["Q"], g["K_base"], g["V_base"], g["L_k"], g["L_v"], g["B_k"], g["B_v"], pos, kvl, rope_theta=cfg.theta,
        want_lse=True, workspace=w)
    call(g["kv_len"], g["positions"], ws)
    for kvl, pos in (([0, 7000, 0], [[0], [6999], [0]]), ([0, 0, 0], [[0], [0], [0]])):
        kvl, pos = (torch.tensor(t, dtype=torch.int32, device="cuda") for t in (kvl, pos))
        O, lse = call(kvl, pos, ws)
        O2, lse2 = call(kvl, pos, torch.zeros_like(ws))
        torch.cuda.synchronize()
        assert torch.equal(O, O2) and torch.equal(lse, lse2)
        for b in range(3):
            if int(kvl[b]) == 0:
                assert not O[b].any() and torch.isneginf(lse[b]).all()
            else:
                assert torch.isfinite(O[b].float()).all() and O[b].any()


# id, r, n_q, n_kv, kv_lens, s_cap, layout: calls that are taken with less than
# the workspace query recommends, and then cut even splits or take the other
# kernel (a short shared base: the shared one at rank 16, each by itself at 64).
SMALL_WORKSPACE = [
    ("even_splits", 64, 16, 8, [4096, 31, 32, 33, 2047, 1, 4095, 1000], 32768, "own"),
    ("even_splits_paged", 64, 16, 8, [4096, 31, 32, 33, 2047, 1, 4095, 1000], 12288, "paged"),
    ("short_base_r16", 16, 32, 8, [700, 1, 33, 64, 500, 699, 31, 32, 200], 704, "shared"),
    ("short_base_r64", 64, 4, 1, [2000 - 121 * i for i in range(16)], 2047, "shared"),
]


@pytest.mark.parametrize("case", SMALL_WORKSPACE, ids=[c[0] for c in SMALL_WORKSPACE])
def test_least_workspace(case):
    cid, r, n_q, n_kv, kv_lens, s_cap, layout = case
    print(f"least workspace {cid}", flush=True)
    B = len(kv_lens)
    cfg = mk_cfg(80 + len(cid), n_q, n_kv, 128, r)
    c = attention_case(cfg, batch=B, n_tok=1, kv_len=kv_lens, positions=[[k - 1] for k in kv_lens], s_cap=s_cap,
                       seed_base=11 * len(cid))
    if layout == "shared":
        for name in ("K_base", "V_base"):
            c[name] = c[name][:1].contiguous()
    g = to_dev(c)
    L = prc.lib()
    dims = prc.make_dims(g["Q"], g["K_base"], g["L_k"], g["L_v"], g["B_k"], g["B_v"], cfg.theta)
    O, lse = torch.empty_like(g["Q"]), torch.empty((B, 1, n_q), dtype=torch.float32, device="cuda")
    p = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    if layout == "paged":
        blk, mb = 64, s_cap // 64
        tbl = block_table(B, mb, B * mb + 2, 29)
        caches = {k: to_pool(c[k], tbl, blk, B * mb + 2).cuda() for k in ("K_base", "V_base", "L_k", "L_v")}
        tbl = tbl.cuda()
        dims.kv_req_stride = dims.l_req_stride = 0
        paging = binding.LrsaPaging(kv_block_table=tbl.data_ptr(), lr_block_table=None, block_size=blk, max_blocks=mb,
                                    n_kv_blocks=B * mb + 2, n_lr_blocks=B * mb + 2)
        fn, head, query = L.lr_shared_attention_paged, (ctypes.byref(dims), ctypes.byref(paging)), prc.paged_workspace_size
    else:
        caches, fn, head, query = g, L.lr_shared_attention, (ctypes.byref(dims),), prc.workspace_size

    def call(ws, n):
        return fn(*head, p(g["Q"]), *(p(caches[k]) for k in ("K_base", "V_base", "L_k", "L_v")), p(g["B_k"]), p(g["B_v"]),
                  p(g["positions"]), p(g["kv_len"]), p(O), p(lse), p(ws), n,
                  ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    ws = torch.full((query(dims) + 256,), 123, dtype=torch.uint8, device="cuda")
    assert call(ws, 0) == 5
    need = int(re.search(r"(\d+) needed", L.prc_last_error().decode()).group(1))
    assert 0 < need < query(dims)
    assert call(ws, need - 1) == 5
    Oref, lref = oracle_attention(c, cfg.theta)
    scale = max(1.0, float(abs(Oref).max()) / 2)
    for n in (query(dims), need):
        ws.fill_(123)
        O.fill_(9.0)
        assert call(ws, n) == 0
        torch.cuda.synchronize()
        assert bool((ws[n:] == 123).all())  # nothing past the bytes it was given
        mx, mean = attn_errors(O, Oref)
        assert mx <= ATOL_MAX * scale and mean <= ATOL_MEAN * scale, (n, mx, mean)
        assert lse_error(lse, lref) <= LSE_ATOL
