"""The extension that calls the hot entry points: what it takes it computes as the general path does, and it leaves everything
else to that path, with its results and its errors."""
import os
import shutil
import subprocess
import sys
import threading

import numpy as np
import pytest
import torch

import paper_2502_04507_amd as sta
from paper_2502_04507_amd import binding

GRID, TILE, H, D = (2, 16, 24), (2, 8, 8), 3, 64
WINDOWS = [(1, 1, 3), (1, 3, 1), (2, 1, 1)]


def tensors(n, device, dtype=torch.bfloat16):
    g = torch.Generator().manual_seed(n)
    return [torch.randn((2, H, 768, D), generator=g).to(dtype).to(device) for _ in range(n)]


def test_leaves_what_it_does_not_know_to_the_general_path():
    fast = binding._fast()
    a, b, c, d = tensors(4, "cpu")                                     # host tensors are refused by the general path
    lse = torch.zeros((2, H, 768))
    assert fast.tile_permute(a, b, GRID, TILE) is None and fast.untile(a, b, GRID, TILE) is None
    assert fast.forward(a, b, c, d, GRID, TILE, WINDOWS, 0.0, None) is None
    assert fast.forward_lse(a, b, c, d, lse, GRID, TILE, WINDOWS, 0.0) is None
    assert fast.backward(*[a] * 5, lse, *[a] * 3, GRID, TILE, WINDOWS, lse, 0.0) is None
    for args in ((), (a,), (a, b, GRID), (a, b, GRID, TILE, None), (None, b, GRID, TILE), (np.zeros(4), b, GRID, TILE)):
        assert fast.tile_permute(*args) is None
    for call in (lambda: sta.sta_tile_permute(a, b, GRID, TILE), lambda: sta.sta_forward(a, b, c, d, GRID, TILE, WINDOWS)):
        with pytest.raises(ValueError, match="must live in device memory"):
            call()


def test_the_library_alone_suffices(tmp_path):
    """A copy of the package without the extension: host-side helpers work silently, a hot entry point warns once and behaves."""
    home = os.path.dirname(sta.__file__)
    copy = tmp_path / os.path.basename(home)
    copy.mkdir()
    for name in os.listdir(home):
        if name.endswith(".py") or name == "libsta.so":
            shutil.copy(os.path.join(home, name), copy / name)
    program = '''
import warnings
with warnings.catch_warnings():
    warnings.simplefilter("error")
    import paper_2502_04507_amd as sta
    assert sta.sta_version() >= 100 and sta.sta_strerror(0)
    assert sta.sta_kept_flops(1, 2, 64, (1, 16, 16), (1, 8, 8), [(1, 1, 1)] * 2) > 0
import torch
a, b = torch.zeros(1, 2, 256, 64, dtype=torch.bfloat16), torch.zeros(1, 2, 256, 64, dtype=torch.bfloat16)
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    for _ in range(2):
        try:
            sta.sta_tile_permute(a, b, (1, 16, 16), (1, 8, 8))
        except ValueError as e:
            assert "must live in device memory" in str(e)
        else:
            raise AssertionError
assert [w.category for w in seen] == [RuntimeWarning], seen
print("ok")
'''
    r = subprocess.run([sys.executable, "-c", program], cwd=tmp_path, capture_output=True, text=True,
                       env=dict(os.environ, PYTHONPATH=str(tmp_path)))
    assert r.stdout.strip().endswith("ok"), r.stdout + r.stderr


def test_a_build_without_a_host_compiler_says_so(monkeypatch, tmp_path):
    from paper_2502_04507_amd import build_lib
    stale = tmp_path / "sta_fastcall.so"
    stale.write_bytes(b"old")
    monkeypatch.setattr(build_lib, "FASTCALL_OUT", str(stale))
    monkeypatch.setenv("CXX", str(tmp_path / "no-such-compiler"))
    assert "no-such-compiler" in build_lib._build_fastcall()
    assert not stale.exists()


def test_first_use_by_several_threads(monkeypatch):
    monkeypatch.setattr(binding, "_FAST", None)
    monkeypatch.setattr(binding, "_LIB", None)
    a = tensors(2, "cpu")
    got = []
    threads = [threading.Thread(target=lambda: got.append(binding._fast().tile_permute(*a, GRID, TILE))) for _ in range(16)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert got == [None] * 16


def general(monkeypatch, call):
    """The call through ctypes."""
    class Nothing:
        def __getattr__(self, name):
            return lambda *a: None
    with monkeypatch.context() as m:
        m.setattr(binding, "_fast", lambda: Nothing())
        return call()


@pytest.mark.gpu
@pytest.mark.parametrize("spell", [lambda x: x, list, lambda x: [np.int64(v) if np.isscalar(v) else tuple(v) for v in x]])
def test_same_results_by_both_ways(spell, monkeypatch):
    q, k, v, do = tensors(4, "cuda:0")
    ws = torch.empty(max(16, sta.sta_backward_workspace_bytes(2, H, GRID)), dtype=torch.uint8, device="cuda:0")

    def everything():
        t, back, o, o2 = (torch.full_like(q, float("nan")) for _ in range(4))
        f = torch.empty(q.shape, dtype=torch.float32, device="cuda:0")
        lse = torch.empty(q.shape[:3], dtype=torch.float32, device="cuda:0")
        d = [torch.full_like(q, float("nan")) for _ in range(3)]
        grid, tile, windows = spell(GRID), spell(TILE), spell(WINDOWS)
        assert sta.sta_tile_permute(q, t, grid, tile) is t and sta.sta_untile(t, back, grid, tile) is back
        sta.sta_untile(t, f, grid, tile)
        assert sta.sta_forward(q, k, v, o, grid, tile, windows, workspace=ws) is o
        sta.sta_forward(q, k, v, o2, grid, tile, windows, 0.3)
        assert sta.sta_forward_lse(q, k, v, o, lse, grid, tile, windows)[1] is lse
        assert sta.sta_backward(q, k, v, o, do, lse, *d, grid, tile, windows, ws)[2] is d[2]
        return t, back, f, o, o2, lse, *d

    want = general(monkeypatch, everything)
    for got, ref in zip(everything(), want):
        assert torch.equal(got, ref)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):                                      # on whatever stream is current
        again = everything()
    side.synchronize()
    for got, ref in zip(again, want):
        assert torch.equal(got, ref)


@pytest.mark.gpu
def test_same_errors_by_both_ways(monkeypatch):
    q, k, v, o = tensors(4, "cuda:0")
    half, f32 = q.half(), q.float()
    lse = torch.empty(q.shape[:3], dtype=torch.float32, device="cuda:0")
    strided = torch.empty((2, H, D, 768), dtype=torch.bfloat16, device="cuda:0").transpose(2, 3)
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda:0")
    calls = [
        lambda: sta.sta_tile_permute(q, q, GRID, TILE), lambda: sta.sta_tile_permute(q, half, GRID, TILE),
        lambda: sta.sta_tile_permute(q, o, (2, 16, 25), TILE), lambda: sta.sta_untile(q, o, GRID, (2, 5, 8)),
        lambda: sta.sta_untile(q, strided, GRID, TILE), lambda: sta.sta_tile_permute(q, o[:1], GRID, TILE),
        lambda: sta.sta_tile_permute(q, o, GRID[:2], TILE), lambda: sta.sta_tile_permute(q.cpu(), o, GRID, TILE),
        lambda: sta.sta_forward(q, k, v, q, GRID, TILE, WINDOWS), lambda: sta.sta_forward(q, k, f32, o, GRID, TILE, WINDOWS),
        lambda: sta.sta_forward(q, k, v, o, GRID, TILE, WINDOWS[:2]), lambda: sta.sta_forward(q, k, v, o, GRID, TILE, [(0, 1, 1)] * H),
        lambda: sta.sta_forward(q, k, v, o, GRID, (1, 1, 8), WINDOWS), lambda: sta.sta_forward(q, k, v, o, GRID, TILE, None),
        lambda: sta.sta_forward(q, k, v, o, GRID, TILE, WINDOWS, workspace=ws[1:]),
        lambda: sta.sta_forward_lse(q, k, v, o, lse[:1], GRID, TILE, WINDOWS), lambda: sta.sta_forward_lse(q, k, v, o, q, GRID, TILE, WINDOWS),
        lambda: sta.sta_backward(q, k, v, o, o, lse, q, f32, f32, GRID, TILE, WINDOWS, ws),
        lambda: sta.sta_backward(q, k, v, o, o, lse, *tensors(3, "cuda:0"), GRID, TILE, WINDOWS, ws[:64]),
    ]
    for i, call in enumerate(calls):
        with pytest.raises(Exception) as slow:
            general(monkeypatch, call)
        with pytest.raises(type(slow.value)) as fast:
            call()
        assert str(fast.value) == str(slow.value) and getattr(fast.value, "status", None) == getattr(slow.value, "status", None), i
