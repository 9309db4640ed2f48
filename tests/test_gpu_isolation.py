"""Shared-base decode: the heads of several requests share one MFMA result, and
what is infinite or NaN for one request must stay out of the others.  Every case
compares, bit for bit, with the same call on finite rows."""
import pytest
import torch

import paper_2609_34054_amd as prc
from gpu_cases import to_dev
from test_gpu_paged import mk_cfg
from workload import attention_case

pytestmark = pytest.mark.gpu

# d, r, n_q, n_kv, kv_lens: 3 + 2, 2 + 2, 2 + 1, 4 + 3 and 3 requests per result,
# one and two groups per workgroup, L_v tiles of their own (ranks 8, 16) and in
# turn (32, 64).
CASES = [
    (128, 16, 8, 2, [2000, 700, 33, 1500, 90]),
    (128, 64, 10, 2, [1900, 40, 600, 1200]),
    (64, 8, 16, 2, [1000, 20, 900]),
    (128, 16, 8, 2, [2000, 700, 33, 1500, 90, 1200, 1]),
    (128, 32, 6, 2, [2100, 64, 65]),
]


def _case(case):
    d, r, n_q, n_kv, kv_lens = case
    cfg = mk_cfg(70 + r, n_q, n_kv, d, r)
    c = attention_case(cfg, batch=len(kv_lens), n_tok=1, kv_len=kv_lens, positions=[[k - 1] for k in kv_lens],
                       s_cap=2112, seed_base=r)
    for name in ("K_base", "V_base"):
        c[name] = c[name][:1].contiguous()
    return cfg, to_dev(c)


def _run(cfg, g):
    O, lse = prc.lr_shared_attention(g["Q"], g["K_base"], g["V_base"], g["L_k"], g["L_v"], g["B_k"], g["B_v"],
                                     g["positions"], g["kv_len"], rope_theta=cfg.theta, want_lse=True)
    torch.cuda.synchronize()
    return O, lse


@pytest.mark.parametrize("name", ["L_v", "L_k"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"d{c[0]}r{c[1]}g{c[2] // c[3]}b{len(c[4])}")
def test_one_agents_rows_stay_its_own(case, name):
    print(f"isolation {name} {case}", flush=True)
    cfg, g = _case(case)
    O, lse = _run(cfg, g)
    assert torch.isfinite(O.float()).all()
    for bad in (0, 1):
        p = dict(g, **{name: g[name].clone()})
        p[name][bad, 3, 2] = float("inf")
        p[name][bad, 17] = float("nan")
        Op, lp = _run(cfg, p)
        rest = [b for b in range(O.shape[0]) if b != bad]
        assert not torch.isfinite(Op[bad].float()).all()
        assert torch.equal(Op[rest], O[rest]) and torch.equal(lp[rest], lse[rest])


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"d{c[0]}r{c[1]}g{c[2] // c[3]}b{len(c[4])}")
def test_base_rows_of_the_longest_request_alone(case):
    """Base rows that only the longest request sees (a 16-token sub-block and
    more past the others' ends)."""
    print(f"isolation base {case}", flush=True)
    cfg, g = _case(case)
    O, lse = _run(cfg, g)
    end = case[4][0]
    p = dict(g, V_base=g["V_base"].clone())
    p["V_base"][0, end - 10:end - 5] = float("inf")
    p["V_base"][0, end - 5] = float("nan")
    Op, lp = _run(cfg, p)
    assert not torch.isfinite(Op[0].float()).all()
    assert torch.equal(Op[1:], O[1:]) and torch.equal(lp[1:], lse[1:])
