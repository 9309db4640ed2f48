"""Chunks of a few query tokens (tokens x GQA group <= 16) run as a decode over
split keys: against the oracle, paged against contiguous bit for bit, and with
no workspace at all (the call then runs as a prefill and must still be taken)."""
import ctypes

import pytest
import torch

import paper_2609_34054_amd as prc
from gpu_cases import ATOL_MAX, ATOL_MEAN, LSE_ATOL, attn_errors, gpu_attention, lse_error, oracle_attention, to_dev
from test_gpu_paged import block_table, mk_cfg, to_pool
from workload import attention_case

pytestmark = pytest.mark.gpu

# id, d, r, n_q, n_kv, n_tok, kv_lens, s_cap, lr ("kv"|"v"|"k"|"none"), positions ("end"|"mid"|"mixed")
CASES = [
    ("g1_16_tokens", 64, 8, 4, 4, 16, [528], 576, "kv", "end"),
    ("g4_4_tokens", 128, 16, 8, 2, 4, [300, 64, 5], 512, "kv", "end"),
    ("g4_3_tokens_long", 128, 16, 32, 8, 3, [5000], 8192, "kv", "end"),
    ("g8_2_tokens", 128, 32, 16, 2, 2, [333, 34, 2], 576, "kv", "mid"),
    ("g5_3_tokens_r64", 128, 64, 10, 2, 3, [700, 65], 704, "kv", "end"),
    ("g3_5_tokens_mixed", 128, 16, 6, 2, 5, [200, 129], 512, "kv", "mixed"),
    ("g2_7_tokens_qv", 64, 32, 4, 2, 7, [97], 640, "v", "end"),
    ("g1_9_tokens_k_only", 64, 8, 9, 9, 9, [130], 512, "k", "end"),
    ("g4_4_tokens_below", 128, 16, 8, 2, 4, [300, 5], 448, "kv", "end"),  # short caches stay a prefill
    # 16 splits, merged by a workgroup per row up to 2048 rows, by a wave above.
    ("g4_4_tokens_2048_rows", 64, 16, 64, 16, 4, [512, 300, 64, 33, 32, 31, 5, 480], 512, "kv", "end"),
    ("g4_4_tokens_2304_rows", 64, 16, 64, 16, 4, [512, 300, 64, 33, 32, 31, 5, 480, 100], 512, "kv", "end"),
    ("g4_2_tokens_plain", 128, 16, 8, 2, 2, [2000, 31], 2048, "none", "end"),
]


def _positions(k, n, mode):
    if mode == "mixed":  # any order, down to the first key
        return [(k - 1) * ((3 * i) % n) // max(1, n - 1) for i in range(n)]
    end = k if mode == "end" else max(n, k // 2)
    return list(range(end - n, end))


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_chunk_as_decode(case):
    cid, d, r, n_q, n_kv, n_tok, kv_lens, s_cap, lr, mode = case
    print(f"chunk {cid}", flush=True)
    B = len(kv_lens)
    cfg = mk_cfg(50 + len(cid), n_q, n_kv, d, r)
    c = attention_case(cfg, batch=B, n_tok=n_tok, kv_len=kv_lens,
                       positions=[_positions(k, n_tok, mode) for k in kv_lens], s_cap=s_cap, seed_base=5 * len(cid),
                       lr_k=lr in ("kv", "k"), lr_v=lr in ("kv", "v"))
    g = to_dev(c)
    O, lse = gpu_attention(g, cfg.theta)
    Oref, lref = oracle_attention(c, cfg.theta)
    # A query that sees one or two keys has outputs above unit scale; their
    # bf16 rounding (2^-9 of the value) and the rebuilt values' scale with them.
    scale = max(1.0, float(abs(Oref).max()) / 2)
    mx, mean = attn_errors(O, Oref)
    assert mx <= ATOL_MAX * scale and mean <= ATOL_MEAN * scale, (mx, mean)
    assert lse_error(lse, lref) <= LSE_ATOL
    # Paged, blocks in random order: the same bits.
    blk = 64
    mb = s_cap // blk
    tbl = block_table(B, mb, B * mb + 2, 23)
    p = {k: None if c[k] is None else to_pool(c[k], tbl, blk, B * mb + 2).cuda()
         for k in ("K_base", "V_base", "L_k", "L_v")}
    Op, lsep = prc.lr_shared_attention_paged(g["Q"], p["K_base"], p["V_base"], p["L_k"], p["L_v"], g["B_k"], g["B_v"],
                                             g["positions"], g["kv_len"], tbl.cuda(), rope_theta=cfg.theta,
                                             want_lse=True)
    torch.cuda.synchronize()
    assert torch.equal(O, Op) and torch.equal(lse, lsep)


def test_chunk_without_workspace_is_still_taken():
    cfg = mk_cfg(91, 8, 2, 128, 16)
    c = attention_case(cfg, batch=2, n_tok=3, kv_len=[300, 64], positions=[[297, 298, 299], [61, 62, 63]], s_cap=576)
    g = to_dev(c)
    dims = prc.make_dims(g["Q"], g["K_base"], g["L_k"], g["L_v"], g["B_k"], g["B_v"], cfg.theta)
    assert prc.workspace_size(dims) > 0
    O = torch.full_like(g["Q"], 9.0)
    p = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    st = prc.lib().lr_shared_attention(ctypes.byref(dims), p(g["Q"]), p(g["K_base"]), p(g["V_base"]), p(g["L_k"]),
                                       p(g["L_v"]), p(g["B_k"]), p(g["B_v"]), p(g["positions"]), p(g["kv_len"]), p(O),
                                       None, None, 0, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st == 0
    On = torch.empty_like(O)
    prc.lr_shared_attention_noalloc(g["Q"], g["K_base"], g["V_base"], g["L_k"], g["L_v"], g["B_k"], g["B_v"],
                                    g["positions"], g["kv_len"], rope_theta=cfg.theta, O=On)
    torch.cuda.synchronize()
    Oref, _ = oracle_attention(c, cfg.theta)
    for out in (O, On):
        mx, mean = attn_errors(out, Oref)
        assert mx <= ATOL_MAX and mean <= ATOL_MEAN, (mx, mean)


def test_noalloc_chunk_without_partials_stays_a_prefill():
    """A chunk whose prefill needs no partials does not touch the static array of
    the call that allocates nothing (only calls that do have to be ordered): the
    bits of the call without any workspace, not those of the split decode."""
    cfg = mk_cfg(92, 8, 2, 128, 16)
    c = attention_case(cfg, batch=2, n_tok=3, kv_len=[570, 264], positions=[[567, 568, 569], [261, 262, 263]], s_cap=576)
    g = to_dev(c)
    dims = prc.make_dims(g["Q"], g["K_base"], g["L_k"], g["L_v"], g["B_k"], g["B_v"], cfg.theta)
    O, On = torch.empty_like(g["Q"]), torch.empty_like(g["Q"])
    p = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    st = prc.lib().lr_shared_attention(ctypes.byref(dims), p(g["Q"]), p(g["K_base"]), p(g["V_base"]), p(g["L_k"]),
                                       p(g["L_v"]), p(g["B_k"]), p(g["B_v"]), p(g["positions"]), p(g["kv_len"]), p(O),
                                       None, None, 0, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert st == 0  # no partials needed
    prc.lr_shared_attention_noalloc(g["Q"], g["K_base"], g["V_base"], g["L_k"], g["L_v"], g["B_k"], g["B_v"],
                                    g["positions"], g["kv_len"], rope_theta=cfg.theta, O=On)
    Od, _ = gpu_attention(g, cfg.theta)
    torch.cuda.synchronize()
    assert torch.equal(O, On) and not torch.equal(O, Od)
