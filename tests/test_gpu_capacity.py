"""Caches reserved far beyond the keys in use: decode and prefill splits divide
the keys in use, so a request's splits depend on its own kv_len and position.
Lengths sit on the edges of the 32-token decode tiles and 64-token prefill
tiles, and include requests that see no key; every row past a length is NaN."""
import pytest
import torch

import paper_2609_34054_amd as prc
from gpu_cases import ATOL_MAX, ATOL_MEAN, LSE_ATOL, attn_errors, gpu_attention, lse_error, oracle_attention, to_dev
from test_gpu_paged import block_table, mk_cfg, to_pool
from workload import attention_case

pytestmark = pytest.mark.gpu

# id, d, r, n_q, n_kv, n_tok, kv_lens, s_cap, lr, layout
CASES = [
    ("decode_edges", 128, 16, 8, 2, 1, [1, 31, 32, 33, 2049, 4096], 8192, "kv", "own"),
    ("decode_one_of_many_tiles", 128, 16, 32, 8, 1, [1500], 32768, "kv", "own"),
    ("decode_r64", 128, 64, 10, 2, 1, [700, 65], 8192, "kv", "own"),
    # 21 splits over up to 22 tiles: one or two tiles each.
    ("decode_one_round", 128, 8, 8, 8, 1, [704, 703, 673, 672, 641, 1, 32, 33, 350, 700, 64, 65], 704, "kv", "own"),
    ("decode_d64_r8", 64, 8, 4, 4, 1, [333], 16384, "v", "own"),
    ("decode_paged_r64", 128, 64, 10, 2, 1, [700, 65, 2048], 8192, "kv", "paged"),
    ("decode_shared_two_groups", 128, 16, 8, 2, 1, [900, 33, 1, 64, 65, 31, 899, 5, 700], 8192, "kv", "shared"),
    ("decode_shared_r64", 128, 64, 8, 2, 1, [500, 499, 100, 1, 64], 4096, "kv", "shared"),
    # Shared base: 4, 3 and 2 requests per 16 columns, one and two groups per
    # workgroup, request slots and columns left over.
    ("decode_shared_g5_r64", 128, 64, 10, 2, 1, [200, 17, 16, 15, 1, 199, 64], 2048, "kv", "shared"),
    ("decode_shared_g8_r16", 128, 16, 16, 2, 1, [300, 31, 33, 299, 16], 2080, "kv", "shared"),
    ("decode_shared_g1_d64_r8", 64, 8, 2, 2, 1, [130, 129, 1, 16, 15, 64, 65, 100, 128], 2049, "kv", "shared"),
    # Two full groups of 4, and of 2 with three of them over two workgroups.
    ("decode_shared_eight", 128, 16, 8, 2, 1, [300, 299, 17, 1, 64, 33, 200, 16], 2048, "kv", "shared"),
    ("decode_shared_g5_seven", 128, 8, 10, 2, 1, [310, 32, 17, 1, 64, 33, 200], 2048, "v", "shared"),
    ("decode_shared_short", 128, 16, 8, 2, 1, [130, 129, 1, 33], 2047, "kv", "shared"),  # each request by itself
    ("decode_shared_g3_qv_r32", 128, 32, 6, 2, 1, [500, 480, 17], 2500, "v", "shared"),
    ("prefill_split", 128, 16, 8, 2, 40, [300, 64, 65], 8192, "kv", "own"),
    ("prefill_split_r8", 128, 8, 8, 2, 16, [1040], 16384, "kv", "own"),
    # More units than CUs and a cache four times the keys: fewer splits than planned.
    ("prefill_split_many_units", 64, 8, 64, 16, 1100, [1300], 5200, "kv", "own"),
    ("prefill_split_paged", 128, 32, 8, 2, 20, [129, 700], 8192, "kv", "paged"),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_splits_follow_the_keys_in_use(case):
    cid, d, r, n_q, n_kv, n_tok, kv_lens, s_cap, lr, layout = case
    print(f"capacity {cid}", flush=True)
    B = len(kv_lens)
    cfg = mk_cfg(40 + len(cid), n_q, n_kv, d, r)
    c = attention_case(cfg, batch=B, n_tok=n_tok, kv_len=kv_lens,
                       positions=[list(range(k - n_tok, k)) for k in kv_lens], s_cap=s_cap, seed_base=3 * len(cid),
                       lr_k=lr == "kv", poison_tail=layout != "shared")
    if layout == "shared":
        for name in ("K_base", "V_base"):
            c[name] = c[name][:1].clone()
            c[name][0, max(kv_lens):] = float("nan")
        for name in ("L_k", "L_v"):
            for b in range(B if c[name] is not None else 0):
                c[name][b, kv_lens[b]:] = float("nan")
    g = to_dev(c)
    if layout == "paged":
        blk = 64
        mb = s_cap // blk
        tbl = block_table(B, mb, B * mb + 3, 17)
        pools = {k: None if c[k] is None else to_pool(c[k], tbl, blk, B * mb + 3).cuda()
                 for k in ("K_base", "V_base", "L_k", "L_v")}
        O, lse = prc.lr_shared_attention_paged(g["Q"], pools["K_base"], pools["V_base"], pools["L_k"], pools["L_v"],
                                               g["B_k"], g["B_v"], g["positions"], g["kv_len"], tbl.cuda(),
                                               rope_theta=cfg.theta, want_lse=True)
        torch.cuda.synchronize()
    else:
        O, lse = gpu_attention(g, cfg.theta)
    Oref, lref = oracle_attention(c, cfg.theta)
    mx, mean = attn_errors(O, Oref)
    # kv_len = 1 .. 33 leaves outputs of unit scale and above: their bf16
    # rounding alone is 2^-9 of the value, so the bound scales with the output.
    scale = max(1.0, float(abs(Oref).max()) / 2)
    assert mx <= ATOL_MAX * scale and mean <= ATOL_MEAN, (mx, mean)
    assert lse_error(lse, lref) <= LSE_ATOL


def test_unwritten_splits_are_not_merged():
    """A request without keys, and stale partials of an earlier longer call in the same workspace."""
    cfg = mk_cfg(90, 8, 2, 128, 16)
    c = attention_case(cfg, batch=2, n_tok=1, kv_len=[8000, 4000], positions=[[7999], [3999]], s_cap=8192)
    g = to_dev(c)
    ws = torch.full((prc.workspace_size(prc.make_dims(g["Q"], g["K_base"], g["L_k"], g["L_v"], g["B_k"], g["B_v"],
                                                      cfg.theta)),), 255, dtype=torch.uint8, device="cuda")
    call = lambda kvl, pos, w: prc.lr_shared_attention(  # noqa: E731
        g["Q"], g["K_base"], g["V_base"], g["L_k"], g["L_v"], g["B_k"], g["B_v"], pos, kvl, rope_theta=cfg.theta,
        want_lse=True, workspace=w)
    call(g["kv_len"], g["positions"], ws)
    kvl = torch.tensor([0, 70], dtype=torch.int32, device="cuda")
    pos = torch.tensor([[0], [69]], dtype=torch.int32, device="cuda")
    O, lse = call(kvl, pos, ws)
    O2, lse2 = call(kvl, pos, torch.zeros_like(ws))
    torch.cuda.synchronize()
    assert torch.equal(O, O2) and torch.equal(lse, lse2)
    assert not O[0].any() and torch.isneginf(lse[0]).all()
    assert torch.isfinite(O[1].float()).all() and O[1].any()
