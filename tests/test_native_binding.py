"""The binding's native marshalling takes the plain case of a call only, and then does what the steps in Python do."""
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest
import torch

from paper_2501_09767_amd import lemo

NAMES = ("score_segments", "select_topk", "kept_attention", "gather_gemm", "gather_gemm_add", "gather_gemm_dx", "gather_gemm_dw", "scatter_grad")


class Refusing:
    """In the place of the native module: always the long way."""
    def __getattr__(self, name):
        return lambda *a: None


def test_what_is_not_plain_is_left_to_python():
    t = torch.ones(4, 4)
    for name in NAMES:
        f = getattr(lemo._native, name)
        for args in ((), (t,) * 3, (t,) * 4, (t,) * 5, (t,) * 6, (t,) * 7, (t,) * 9, (None,) * 9, (1, "x", 2.5, None)):  # (no GPU tensor among them)
            assert f(*args) is None
    with pytest.raises(ValueError, match="GPU"):
        lemo.lemo_gather_gemm(t, None, t, Y=t)
    with pytest.raises(TypeError):
        lemo._native.set_stream_source(1)


@pytest.mark.parametrize("native", ["missing", "no library", "of another torch"])
def test_binding_without_its_native_part(tmp_path, native):
    """The steps in Python need the HIP library and nothing else: where the native part cannot be used, they are taken."""
    home = os.path.dirname(lemo.__file__)
    package = tmp_path / "paper_2501_09767_amd"
    package.mkdir()
    for name in ("__init__.py", "lemo.py", "liblemo_hip.so", "lemo_native.so"):
        shutil.copy(os.path.join(home, name), package / name)
    if native == "missing":
        (package / "lemo_native.so").unlink()
    elif native == "no library":
        (package / "lemo_native.so").write_bytes(b"not an object file")
    code = """
import warnings
import torch
if %r: torch.__version__ = type(torch.__version__)("1.13.1+cu117")
with warnings.catch_warnings(record=True) as said:
    warnings.simplefilter("always")
    from paper_2501_09767_amd import lemo
assert any("lemo_native.so" in str(w.message) for w in said), said
assert lemo._native.gather_gemm(None, None, None, None, None, None) is None
assert lemo.lemo_kept_count(1000, 128, 64) == 500
t = torch.ones(8, 8)
for f in (lambda: lemo.lemo_gather_gemm(t, None, t, Y=t), lambda: lemo.lemo_score_segments(t, t, 8), lambda: lemo.lemo_select_topk(t, 8, 4), lambda: lemo.lemo_scatter_grad(t, t, t),
          lambda: lemo.lemo_gather_gemm_add(t, None, t, t, None), lambda: lemo.lemo_gather_gemm_dx(t, t, t, None), lambda: lemo.lemo_gather_gemm_dw(t, t, None)):
    try:
        f()
    except ValueError as e:
        assert "GPU" in str(e), e
    else:
        raise AssertionError("not refused")
""" % (native == "of another torch")
    r = subprocess.run([sys.executable, "-c", code], cwd=tmp_path, capture_output=True, text=True, env={**os.environ, "PYTHONPATH": str(tmp_path)})
    assert r.returncode == 0, r.stderr


def calls():
    gen = torch.Generator(device="cuda").manual_seed(3)
    S, H, Hkv, d, C, N, L = 300, 4, 2, 64, 64, 96, 128
    bf = lambda *s: torch.randn(s, generator=gen, device="cuda").bfloat16()
    Q, K, V = bf(S, H, d), bf(S, Hkv, d), bf(S, Hkv, d)
    k = lemo.lemo_keep_k(L, 0.5)
    M = lemo.lemo_kept_count(S, L, k)
    kept = torch.randperm(S, generator=gen, device="cuda")[:M].sort().values.int()
    X, W, b, G, dY = bf(S, C), bf(N, C), bf(N), bf(M, C), bf(M, N)
    ws = torch.empty(1 << 22, dtype=torch.uint8, device="cuda")
    R = bf(S, N)
    scores = torch.rand(S, generator=gen, device="cuda")
    new = lambda *s, dtype=torch.bfloat16: torch.zeros(s, dtype=dtype, device="cuda")
    return {
        "score_segments": lambda: lemo.lemo_score_segments(Q, K, L, 3, 0.1, new(S, dtype=torch.float32), new(H, S, dtype=torch.float32), new(H, S, dtype=torch.float32), ws),
        "select_topk": lambda: lemo.lemo_select_topk(scores, L, k, new(M, dtype=torch.int32)),
        "kept_attention": lambda: lemo.lemo_kept_attention(Q, K, V, kept, 1, 0.0, new(M, H, d), ws),
        "gather_gemm": lambda: lemo.lemo_gather_gemm(X, kept, W, b, new(M, N + 8)[:, :N]),
        "gather_gemm_M": lambda: lemo.lemo_gather_gemm(X, None, W, None, new(S, N), 77),
        "gather_gemm_add": lambda: lemo.lemo_gather_gemm_add(X, kept, W, R.clone(), kept, b),
        "gather_gemm_dx": lambda: lemo.lemo_gather_gemm_dx(dY, W, new(S, C), kept),
        "gather_gemm_dw": lambda: lemo.lemo_gather_gemm_dw(dY, X, kept, new(N, C)),
        "gather_gemm_dw_f32": lambda: lemo.lemo_gather_gemm_dw(dY.float(), X.float(), kept, new(N, C, dtype=torch.float32), ws),
        "scatter_grad": lambda: lemo.lemo_scatter_grad(G, kept, new(S, C, dtype=torch.float32), lemo.SCATTER_ZERO_PAD),
    }, dict(X=X, W=W, kept=kept, G=G, Q=Q, K=K, ws=ws, S=S, M=M, C=C, N=N)


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["score_segments", "select_topk", "kept_attention", "gather_gemm", "gather_gemm_M", "gather_gemm_add", "gather_gemm_dx",
                                  "gather_gemm_dw", "gather_gemm_dw_f32", "scatter_grad"])
def test_same_bits_either_way(monkeypatch, name):
    f = calls()[0][name]
    taken = []
    real = lemo._native

    class Watching:
        def __getattr__(self, n):
            def g(*a):
                taken.append(getattr(real, n)(*a))
                return taken[-1]
            return g
    monkeypatch.setattr(lemo, "_native", Watching())
    fast = f()
    assert taken == [0]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):  # on the current stream
        other = f()
    torch.cuda.current_stream().wait_stream(side)
    monkeypatch.setattr(lemo, "_native", Refusing())
    slow = f()
    torch.cuda.synchronize()
    assert taken == [0, 0] and torch.equal(fast, slow) and torch.equal(other, slow)


def more_rows_than_listed(o):
    """M beyond the end of the list of rows, with room for the result (and so for the reads, if a call went through)."""
    listed = torch.zeros(o["S"], dtype=torch.int32, device="cuda")[:o["M"]]
    M, new = o["M"] + 1, lambda *s: torch.zeros(*s, dtype=torch.bfloat16, device="cuda")
    H, d = o["Q"].shape[1:]
    return [lambda: lemo.lemo_gather_gemm(o["X"], listed, o["W"], None, new(M, o["N"]), M), lambda: lemo.lemo_gather_gemm(o["X"], listed, o["W"], M=M),
            lambda: lemo.lemo_gather_gemm_add(o["X"], listed, o["W"], new(o["S"], o["N"]), None, None, M),
            lambda: lemo.lemo_kept_attention(o["Q"], o["K"], o["K"], listed, 1, 0.0, new(M, H, d), o["ws"], M), lambda: lemo.lemo_kept_attention(o["Q"], o["K"], o["K"], listed, M=M)]


@pytest.mark.gpu
@pytest.mark.parametrize("native", [True, False])
def test_more_rows_than_listed_are_refused(monkeypatch, native):
    _, o = calls()
    if not native:
        monkeypatch.setattr(lemo, "_native", Refusing())
    for f in more_rows_than_listed(o):
        with pytest.raises(ValueError, match="shorter than M"):
            f()


@pytest.mark.gpu
def test_same_refusals_either_way(monkeypatch):
    _, o = calls()
    X, W, kept, G, S, M, C, N = (o[n] for n in ("X", "W", "kept", "G", "S", "M", "C", "N"))
    Y, dX = torch.empty(M, N, dtype=torch.bfloat16, device="cuda"), torch.zeros(S, C, dtype=torch.bfloat16, device="cuda")
    short = torch.empty(16, dtype=torch.uint8, device="cuda")
    scores = torch.empty(S, device="cuda")
    bad = [lambda: lemo.lemo_gather_gemm(X.float(), kept, W, Y=Y), lambda: lemo.lemo_gather_gemm(X[:, :60], kept, W[:, :60], Y=Y), lambda: lemo.lemo_gather_gemm(X, kept.long(), W, Y=Y),
           lambda: lemo.lemo_gather_gemm(X.t(), kept, W, Y=Y), lambda: lemo.lemo_gather_gemm(X, kept.cpu(), W, Y=Y), lambda: lemo.lemo_gather_gemm(X, None, W, Y=Y, M=S + 1),
           lambda: lemo.lemo_scatter_grad(G, kept, dX, 7), lambda: lemo.lemo_scatter_grad(G[:5], kept, dX), lambda: lemo.lemo_scatter_grad(G.half(), kept, dX),
           lambda: lemo.lemo_score_segments(o["Q"], o["K"], 128, scores=scores, workspace=short), lambda: lemo.lemo_score_segments(o["Q"], o["K"], 0, scores=scores, workspace=o["ws"]),
           lambda: lemo.lemo_score_segments(o["Q"], o["K"], 128, 64, scores=scores, workspace=o["ws"]), lambda: lemo.lemo_select_topk(scores, 128, 200, kept),
           lambda: torch.vmap(lambda g: lemo.lemo_scatter_grad(g, kept, dX))(torch.stack([G, G])),
           lambda: lemo.lemo_gather_gemm_add(X, kept, W, torch.empty(S, N, device="cuda"), kept)]
    seen = []
    for native in (lemo._native, Refusing()):
        monkeypatch.setattr(lemo, "_native", native)
        seen.append([])
        for f in bad:
            with pytest.raises(Exception) as e:
                f()
            seen[-1].append((type(e.value), str(e.value)))
    assert seen[0] == seen[1]
    # values that are no plain Python numbers go the long way and do the same
    want = lemo.lemo_scatter_grad(G, kept, dX.clone(), lemo.SCATTER_ACCUMULATE)
    assert torch.equal(lemo.lemo_scatter_grad(G, kept, dX.clone(), np.int64(0)), want)
    empty = torch.empty(0, dtype=torch.int32, device="cuda")
    assert lemo.lemo_gather_gemm(X, empty, W).shape == (0, N)
