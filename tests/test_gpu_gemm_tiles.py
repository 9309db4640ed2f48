"""The projection and precompute GEMMs at the edges of their tile choices: tails
of k (d_in below one step, below one step per wave, not a multiple of 32),
partial token and column tiles, contiguous and paged rows, against the fp64
oracle.  Tolerances: relative 2-norm 1e-2 as everywhere; each element within
2^-7 of its size (bf16 rounding is 2^-9) plus 2e-2 of unit-scale outputs."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2609_34054_amd as prc
from gpu_cases import PRE_REL, f64
from test_gpu_paged import block_table
from workload.gen import normal_bf16

pytestmark = pytest.mark.gpu

# id, T, d_in, n_kv, d, n_proj, N, r, tok_offset, block size (0: contiguous)
CASES = [
    # LR rows alone, small tiles (16 tokens x 32 columns, k over eight waves).
    ("small_one_chunk", 5, 8, 0, 64, 1, 1, 8, 0, 0),
    ("small_k_tail", 17, 264, 0, 64, 2, 3, 8, 7, 0),
    ("small_k_24", 16, 24, 0, 64, 1, 5, 8, 1, 0),
    ("small_paged", 33, 520, 0, 64, 2, 2, 16, 60, 64),
    ("small_most_tiles", 512, 320, 0, 64, 2, 4, 32, 3, 0),
    ("one_tile_too_many", 513, 96, 0, 64, 2, 4, 32, 3, 0),
    # Matrix-vector rows into paged caches.
    ("gemv_paged", 3, 264, 2, 64, 2, 2, 16, 126, 128),
    ("gemv_paged_lr", 1, 512, 0, 64, 2, 3, 64, 64, 64),
    # 64- and 128-wide tiles: few token tiles over all XCDs, odd tile counts.
    ("tiles_one_token_tile", 6, 72, 8, 128, 2, 3, 8, 250, 0),
    ("tiles_three_paged", 150, 136, 4, 128, 2, 3, 16, 50, 128),
    ("tiles_128_ragged", 500, 264, 8, 128, 2, 8, 16, 5, 0),
    # 256-token tiles of 96, 128 and 160 columns: one, two and five stages of k
    # with tails, last token and column tiles partial, both head dims.
    ("wide_96_one_stage", 2100, 40, 8, 128, 2, 8, 16, 1, 0),
    ("wide_96_d64_paged", 2100, 264, 9, 64, 1, 5, 8, 100, 64),
    ("wide_128_d64", 3000, 72, 19, 64, 1, 25, 8, 60000, 0),
    ("wide_128_paged", 2100, 264, 12, 128, 2, 4, 64, 7, 256),
    ("wide_160", 4097, 72, 8, 128, 2, 8, 16, 0, 0),
    ("tiles_d64", 700, 104, 6, 64, 1, 3, 64, 0, 64),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_gemm_edges(case):
    cid, T, d_in, n_kv, d, n_proj, N, r, off, blk = case
    print(f"gemm {cid}", flush=True)
    theta, g, sentinel = 5e5, 7000 + 10 * len(cid), -7.0
    X = normal_bf16((T, d_in), 1.0, g + 1)
    W = normal_bf16((d_in, 2 * n_kv * d), 1.0 / math.sqrt(d_in), g + 2)
    A = normal_bf16((d_in, n_proj * N * r), 1.0 / math.sqrt(d_in), g + 3)
    rows = np.arange(off, off + T)
    full = lambda *shape: torch.full(shape, sentinel, dtype=torch.bfloat16, device="cuda")  # noqa: E731
    if blk:
        mb = -(-(off + T) // blk)
        tbl = block_table(1, mb, mb + 2, 5)[0]
        L = full(n_proj, N, mb + 2, blk, r)
        K = full(mb + 2, blk, n_kv, d) if n_kv else None
        V = full(mb + 2, blk, n_kv, d) if n_kv else None
        prc.project_kv_and_lr_cache_paged(X.cuda(), W.cuda() if n_kv else None, A.cuda(), n_kv, d, n_proj, N, r, K, V,
                                          L, tbl.cuda(), rope_theta=theta, tok_offset=off)
        at = tbl.numpy()[rows // blk].astype(np.int64) * blk + rows % blk
    else:
        s_cap = off + T + 3
        L = full(n_proj, N, s_cap, r)
        K, V = (full(s_cap, n_kv, d), full(s_cap, n_kv, d)) if n_kv else (None, None)
        if n_kv:
            prc.project_kv_and_lr_cache(X.cuda(), W.cuda(), A.cuda(), n_kv, d, n_proj, N, r, K, V, L,
                                        rope_theta=theta, tok_offset=off)
        else:
            prc.precompute_lr_cache(X.cuda(), A.cuda(), n_proj, N, r, L, tok_offset=off)
        at = rows
    torch.cuda.synchronize()
    outs = [("L", f64(L).reshape(n_proj, N, -1, r), oracle.precompute_lr_cache(f64(X), f64(A), n_proj, N, r), 2)]
    if n_kv:
        Wn = f64(W)
        Kr, Vr, _ = oracle.project_kv_and_lr(f64(X), Wn[:, :n_kv * d], Wn[:, n_kv * d:], f64(A), n_kv, n_proj, N, r,
                                             rows, theta)
        outs += [("K", f64(K).reshape(-1, n_kv, d), Kr, 0), ("V", f64(V).reshape(-1, n_kv, d), Vr, 0)]
    for name, got, ref, axis in outs:
        mine = np.take(got, at, axis=axis)
        assert np.linalg.norm(mine - ref) / np.linalg.norm(ref) <= PRE_REL, name
        assert np.max(np.abs(mine - ref) - 2 ** -7 * np.abs(ref)) <= 2e-2, name
        rest = np.delete(got, at, axis=axis)
        assert (rest == sentinel).all(), name  # rows outside the segment are untouched


@pytest.mark.parametrize("ld_x", [2 ** 22 - 8, 2 ** 22, 2 ** 23 - 8])
def test_rows_far_apart(ld_x):
    """Row strides at the edge of the 256-token tiles' byte offsets and at the
    largest accepted one, with a tail of k; whatever lies between the rows is NaN."""
    T, d_in, n_kv, d, n_proj, N, r = 300, 72, 1, 64, 2, 64, 64
    print(f"gemm ld_x {ld_x}", flush=True)
    X = normal_bf16((T, d_in), 1.0, 7901)
    W = normal_bf16((d_in, 2 * n_kv * d), 1.0 / math.sqrt(d_in), 7902)
    A = normal_bf16((d_in, n_proj * N * r), 1.0 / math.sqrt(d_in), 7903)
    room = torch.full(((T - 1) * ld_x + d_in,), float("nan"), dtype=torch.bfloat16, device="cuda")
    Xs = room.as_strided((T, d_in), (ld_x, 1))
    Xs.copy_(X)
    z = lambda *shape: torch.zeros(shape, dtype=torch.bfloat16, device="cuda")  # noqa: E731
    K, V, L = prc.project_kv_and_lr_cache(Xs, W.cuda(), A.cuda(), n_kv, d, n_proj, N, r, z(T, n_kv, d), z(T, n_kv, d),
                                          z(n_proj, N, T, r), rope_theta=1e4)
    torch.cuda.synchronize()
    Wn = f64(W)
    Kr, Vr, Lr = oracle.project_kv_and_lr(f64(X), Wn[:, :n_kv * d], Wn[:, n_kv * d:], f64(A), n_kv, n_proj, N, r,
                                          np.arange(T), 1e4)
    for name, got, ref in (("K", K, Kr), ("V", V, Vr), ("L", L, Lr)):
        got = f64(got)
        assert np.isfinite(got).all() and np.linalg.norm(got - ref) / np.linalg.norm(ref) <= PRE_REL, name


def test_key_angles_do_not_depend_on_the_tile():
    """Every token's angle is reduced in fp64 by itself.  Keys with one weight of
    1 in the lower half of a head and none in the upper are x cos and x sin, one
    product each: a long call (256-token tiles) and short ones give equal bits."""
    T, d_in, n_kv, d, N, r, off = 2100, 40, 8, 128, 8, 16, 60000
    X = normal_bf16((T, d_in), 1.0, 7911).cuda()
    W = torch.zeros((d_in, 2 * n_kv * d), dtype=torch.bfloat16, device="cuda")
    for h in range(n_kv):
        for j in range(d // 2):
            W[(5 * h + j) % d_in, h * d + j] = 1.0
    A = normal_bf16((d_in, 2 * N * r), 1.0 / math.sqrt(d_in), 7912).cuda()
    out = []
    for step in (T, 300):
        K = torch.zeros((off + T, n_kv, d), dtype=torch.bfloat16, device="cuda")
        V, L = torch.zeros_like(K), torch.zeros((2, N, off + T, r), dtype=torch.bfloat16, device="cuda")
        for t in range(0, T, step):
            prc.project_kv_and_lr_cache(X[t:t + step], W, A, n_kv, d, 2, N, r, K, V, L, rope_theta=5e5, tok_offset=off + t)
        out.append(K)
    torch.cuda.synchronize()
    assert out[0][off:].any()
    assert torch.equal(out[0], out[1]), int((out[0] != out[1]).sum())
