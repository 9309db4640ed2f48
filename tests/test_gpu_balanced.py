"""Rank-64 decode of several requests: its splits follow the requests' lengths.
Against the oracle for lengths on the tile edges, empty and uneven requests, the
smallest and largest batch that balances and one more; paged (block table in
LDS, and the form for tables too long for it) against contiguous; and with no
more workspace than the call insists on."""
import pytest
import torch

import paper_2609_34054_amd as prc
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
]


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
    # A workspace with room for even splits alone (half of the recommended one).
    dims = prc.make_dims(g["Q"], g["K_base"], g["L_k"], g["L_v"], g["B_k"], g["B_v"], cfg.theta)
    small = torch.empty(prc.workspace_size(dims) // 2 + 256, dtype=torch.uint8, device="cuda")
    Os, ls = gpu_attention(g, cfg.theta, workspace=small) if cid == "eight_edges" else (O, lse)
    torch.cuda.synchronize()
    for o, l in ((O, lse), (Op, lp), (Os, ls)):
        mx, mean = attn_errors(o, Oref)
        assert mx <= ATOL_MAX * scale and mean <= ATOL_MEAN * scale, (mx, mean)
        assert lse_error(l, lref) <= LSE_ATOL
    if cid != "long_tables":  # the same kernel on the same splits
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
