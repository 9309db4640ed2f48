"""The native argument marshalling against the Python one: the same bits for
valid calls in every entry point and layout it takes, and the same error, type
and message, for calls it must not take."""
import pytest
import torch

import paper_2609_34054_amd as prc
from paper_2609_34054_amd import binding
from gpu_cases import to_dev
from test_gpu_paged import block_table, mk_cfg, to_pool
from workload import attention_case
from workload.gen import normal_bf16

pytestmark = pytest.mark.gpu


def _case(n_tok=1, B=2):
    cfg = mk_cfg(95, 8, 2, 128, 16)
    return cfg, attention_case(cfg, batch=B, n_tok=n_tok, kv_len=[120, 77][:B],
                               positions=[list(range(k - n_tok, k)) for k in [120, 77][:B]], s_cap=128)


def _attention(g, **kw):
    a = dict(g)
    a.update({k: v for k, v in kw.items() if k in a})
    rest = {k: v for k, v in kw.items() if k not in a}
    return prc.lr_shared_attention(a["Q"], a["K_base"], a["V_base"], a["L_k"], a["L_v"], a["B_k"], a["B_v"],
                                   a["positions"], a["kv_len"], rope_theta=1e4, want_lse=True, **rest)


class _Spy:
    """The native module's functions, and the kind of each one's last answer."""

    def __init__(self, m):
        self.last = None
        for name in ("attention", "paged", "project", "project_paged"):
            setattr(self, name, self._watch(getattr(m, name)))

    def _watch(self, f):
        def g(*a):
            r = f(*a)
            self.last = type(r)
            return r
        return g


def _both(call, monkeypatch, answer=int):
    """The call through the native module and through the Python checks.
    ``answer``: the type of what the module returns, ``int`` for a call that it
    makes itself (whatever the status), NoneType for one it leaves to Python."""
    got = []
    for native in (True, False):
        with monkeypatch.context() as m:
            spy = _Spy(binding._native().m)
            m.setattr(binding._native(), "m", spy)
            if not native:
                m.setattr(binding, "_on_gpu", lambda t: False)
            try:
                out = call()
                torch.cuda.synchronize()
                got.append([t.clone() for t in out if t is not None])
            except Exception as e:  # noqa: BLE001
                got.append((type(e), str(e)))
            assert spy.last is (answer if native else None), (native, spy.last)
    return got


NOT_TAKEN = type(None)


@pytest.mark.parametrize("n_tok", [1, 3, 40])
def test_attention_calls_agree(n_tok, monkeypatch):
    cfg, c = _case(n_tok)
    g = to_dev(c)
    one = {k: (v[:1].contiguous() if k in ("K_base", "V_base", "B_k", "B_v") else v) for k, v in g.items()}
    wide = torch.empty((2, 160, 2, 128), dtype=torch.bfloat16, device="cuda")
    strided = dict(g, K_base=wide[:, :128], V_base=wide.clone()[:, :128])
    strided["K_base"].copy_(g["K_base"])
    strided["V_base"].copy_(g["V_base"])
    for name, call in (("plain", lambda: _attention(g)), ("shared", lambda: _attention(one)),
                       ("strided", lambda: _attention(strided)),
                       ("values only", lambda: _attention(g, L_k=None, B_k=None)),
                       ("no LR", lambda: _attention(g, L_k=None, B_k=None, L_v=None, B_v=None)),
                       ("no cache", lambda: _attention(g, tile_cache=False)),
                       ("scale", lambda: _attention(g, softmax_scale=0.2))):
        a, b = _both(call, monkeypatch)
        assert len(a) == len(b) == 2 and all(torch.equal(x, y) for x, y in zip(a, b)), name
    tbl = block_table(2, 2, 6, 3)
    pl = {k: to_pool(c[k], tbl, 64, 6).cuda() for k in ("K_base", "V_base", "L_k", "L_v")}
    a, b = _both(lambda: prc.lr_shared_attention_paged(
        g["Q"], pl["K_base"], pl["V_base"], pl["L_k"], pl["L_v"], g["B_k"], g["B_v"], g["positions"], g["kv_len"],
        tbl.cuda(), rope_theta=1e4, want_lse=True), monkeypatch)
    assert all(torch.equal(x, y) for x, y in zip(a, b))
    # O holds a sentinel before each leg: the second must not see the first's.
    a, b = _both(lambda: prc.lr_shared_attention_noalloc(
        g["Q"], g["K_base"], g["V_base"], g["L_k"], g["L_v"], g["B_k"], g["B_v"], g["positions"], g["kv_len"],
        rope_theta=1e4, O=torch.full_like(g["Q"], 9.0)), monkeypatch)
    assert torch.equal(a[0], b[0]) and not (a[0] == 9.0).all()


def test_refusals_agree(monkeypatch):
    _, c = _case()
    g = to_dev(c)
    bad = [dict(Q=g["Q"].float()), dict(K_base=g["K_base"][:, :100]), dict(L_k=g["L_k"][:, :64]),
           dict(positions=g["positions"].long()), dict(kv_len=g["kv_len"][:1]), dict(B_k=g["B_k"][:, :8]),
           dict(L_k=None), dict(Q=g["Q"].transpose(1, 2)), dict(rope_theta=-1.0), dict(Q=g["Q"][0]),
           dict(L_v=g["L_v"].transpose(1, 2)), dict(kv_len=None), dict(Q=g["Q"][:, :, :7])]
    # Refused by the library (missing L_k, RoPE base, head count); a Q of three
    # dims does not reach the module.
    answers = {6: int, 8: int, 9: None, 12: int}
    for i, kw in enumerate(bad):
        def call(kw=kw):
            a = dict(g, rope_theta=1e4)
            a.update(kw)
            return prc.lr_shared_attention(a["Q"], a["K_base"], a["V_base"], a["L_k"], a["L_v"], a["B_k"], a["B_v"],
                                           a["positions"], a["kv_len"], rope_theta=a["rope_theta"])
        a, b = _both(call, monkeypatch, answers.get(i, NOT_TAKEN))
        assert isinstance(a, tuple) and a == b, (kw.keys(), a, b)


def test_projection_calls_agree(monkeypatch):
    T, d_in, n_kv, d, N, r = 6, 64, 2, 64, 2, 8
    X = normal_bf16((T, d_in + 8), 1.0, 1).cuda()[:, :d_in]
    W, A = normal_bf16((d_in, 2 * n_kv * d), 0.1, 2).cuda(), normal_bf16((d_in, 2 * N * r), 0.1, 3).cuda()
    z = lambda *s: torch.zeros(s, dtype=torch.bfloat16, device="cuda")  # noqa: E731
    tbl = torch.tensor([2, 0], dtype=torch.int32, device="cuda")
    calls = [
        lambda: (prc.precompute_lr_cache(X, A, 2, N, r, z(2, N, 16, r), 3),),
        lambda: prc.project_kv_and_lr_cache(X, W, A, n_kv, d, 2, N, r, z(16, n_kv, d), z(16, n_kv, d), z(2, N, 16, r),
                                            rope_theta=1e4, tok_offset=5),
        lambda: prc.project_kv_and_lr_cache_paged(X, W, A, n_kv, d, 2, N, r, z(3, 64, n_kv, d), z(3, 64, n_kv, d),
                                                  z(2, N, 3, 64, r), tbl, rope_theta=1e4, tok_offset=60),
    ]
    for call in calls:
        a, b = _both(call, monkeypatch)
        assert all(torch.equal(x, y) for x, y in zip(a, b)) and any(x.any() for x in a)
    bad = [lambda: (prc.precompute_lr_cache(X, A, 2, N, r, z(2, N, 16, r), 11),),   # rows past s_cap
           lambda: (prc.precompute_lr_cache(X, A[:, :8], 2, N, r, z(2, N, 16, r)),),
           lambda: (prc.precompute_lr_cache(X.float(), A, 2, N, r, z(2, N, 16, r)),),
           lambda: prc.project_kv_and_lr_cache(X, W[:, :8], A, n_kv, d, 2, N, r, z(16, n_kv, d), z(16, n_kv, d),
                                               z(2, N, 16, r), rope_theta=1e4),
           lambda: prc.project_kv_and_lr_cache_paged(X, W, A, n_kv, d, 2, N, r, z(3, 64, n_kv, d), z(3, 64, n_kv, d),
                                                     z(2, N, 3, 64, r), tbl.long(), rope_theta=1e4)]
    for i, call in enumerate(bad):
        a, b = _both(call, monkeypatch, int if i == 0 else NOT_TAKEN)
        assert isinstance(a, tuple) and a == b, (a, b)


def test_nested_tensors_are_refused(monkeypatch):
    """Tensors without sizes or strides: asking them for either throws."""
    _, c = _case()
    g = to_dev(c)
    nest = lambda t: torch.nested.nested_tensor(list(t.unbind(0)))  # noqa: E731
    z = torch.zeros((8, 8), dtype=torch.bfloat16, device="cuda")
    L = torch.zeros((1, 1, 8, 8), dtype=torch.bfloat16, device="cuda")
    tbl = torch.zeros((2, 2), dtype=torch.int32, device="cuda")
    pool = torch.zeros((2, 64, 2, 128), dtype=torch.bfloat16, device="cuda")

    def attention(**kw):
        a = dict(g, **kw)
        return prc.lr_shared_attention(a["Q"], a["K_base"], a["V_base"], a["L_k"], a["L_v"], a["B_k"], a["B_v"],
                                       a["positions"], a["kv_len"], rope_theta=1e4)
    for call in (lambda: attention(Q=nest(g["Q"])), lambda: attention(K_base=nest(g["K_base"])),
                 lambda: attention(kv_len=nest(g["positions"])),
                 lambda: prc.lr_shared_attention_paged(nest(g["Q"]), pool, pool, None, None, None, None, g["positions"],
                                                       g["kv_len"], tbl, rope_theta=1e4),
                 lambda: prc.precompute_lr_cache(nest(z), z, 1, 1, 8, L),
                 lambda: prc.project_kv_and_lr_cache_paged(nest(z), z, z, 1, 64, 1, 1, 8, pool, pool, L, tbl[0],
                                                           rope_theta=1e4)):
        a, b = _both(call, monkeypatch, NOT_TAKEN)
        assert isinstance(a, tuple) and a == b, (a, b)
