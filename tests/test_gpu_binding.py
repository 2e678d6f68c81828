"""The native device calls of the binding against its general path: the same
bytes for every form that they take, and the same error for what is refused."""
import sys

import numpy as np
import pytest
import torch

from paper_2507_08523_amd import ilpc


def make(device, Hq=4, Hkv=2, D=64, lens=(40, 17), new=(9, 17), shared=0):
    g = torch.Generator().manual_seed(Hq * 100 + D)
    B, mb = len(lens), -(-max(lens) // 16)
    rnd = lambda *s: torch.randn(*s, generator=g).to(torch.bfloat16).to(device)  # noqa: E731
    ints = lambda a: torch.tensor(np.asarray(a, np.int32)).to(device)  # noqa: E731
    bt = np.arange(B * mb, dtype=np.int32).reshape(B, mb)
    bt[:, :shared // 16] = bt[0, :shared // 16]
    total = sum(new)
    return dict(
        q=rnd(total, Hq, D), k=rnd(total, Hkv, D), v=rnd(total, Hkv, D), kp=rnd(B * mb, Hkv, 16, D),
        vp=rnd(B * mb, Hkv, D, 16), bt=ints(bt), cu=ints(np.concatenate([[0], np.cumsum(new)])),
        sp=ints(np.subtract(lens, new)), L=ints(lens), max_new=max(new), shared=shared,
        freq=(10000.0 ** (-torch.arange(D // 2) / (D // 2))).to(device), out=rnd(total, Hq, D),
        ws=torch.zeros(ilpc.attn_cascade_workspace_bytes(B, max(new), Hq, Hkv, D), dtype=torch.uint8, device=device))


def append(m, **kw):
    ilpc.kv_append(m["k"], m["v"], m["kp"], m["vp"], m["bt"], m["cu"], m["sp"], m["max_new"], **kw)


def rope(m, **kw):
    ilpc.rope_kv_append(m["q"], m["q"], m["k"], m["v"], m["kp"], m["vp"], m["bt"], m["cu"], m["sp"], m["max_new"],
                        m["freq"], **kw)


def rope_k(m, **kw):
    ilpc.rope_kv_append(None, None, m["k"], m["v"], m["kp"], m["vp"], m["bt"], m["cu"], m["sp"], m["max_new"],
                        m["freq"], **kw)


def attend(m, **kw):
    ilpc.paged_prefill_attn(m["q"], m["kp"], m["vp"], m["bt"], m["cu"], m["L"], m["max_new"], 0.125, m["out"], **kw)


def attend_ws(m, **kw):
    attend(m, workspace=m["ws"], **kw)


def cascade(m, **kw):
    ilpc.paged_prefill_attn_cascade(m["q"], m["kp"], m["vp"], m["bt"], m["cu"], m["L"], m["max_new"], m["shared"],
                                    0.125, m["out"], m["ws"], **kw)


CALLS = [append, rope, rope_k, attend, attend_ws, cascade]


@pytest.mark.gpu
@pytest.mark.parametrize("own_stream", [False, True])
@pytest.mark.parametrize("shape", [dict(), dict(Hq=8, Hkv=1, D=128, lens=(33,), new=(1,)),
                                   dict(lens=(70, 64, 49), new=(22, 16, 1), shared=48)])
@pytest.mark.parametrize("call", CALLS)
def test_native_calls_equal_the_general_path(call, shape, own_stream, monkeypatch):
    print(call.__name__, shape, own_stream, flush=True)
    taken = []

    class Spy:
        def __getattr__(self, name):
            return lambda *a: taken.append(getattr(native, name)(*a)) or taken[-1]

    native = ilpc._native()
    assert not isinstance(native, ilpc._NoNative)
    stream = torch.cuda.Stream() if own_stream else None
    got = []
    for stand_in in (ilpc._NoNative(), Spy()):
        monkeypatch.setattr(ilpc, "_binding", stand_in)
        m = make("cuda:0", **shape)
        torch.cuda.synchronize()
        for _ in range(2):  # (the second call finds the kept workspace)
            call(m, stream=stream)
        torch.cuda.synchronize()
        got.append(m)
    assert taken[-1] == 0  # the call was made natively
    for name in ("q", "kp", "vp", "out"):
        assert torch.equal(got[0][name].view(torch.int16), got[1][name].view(torch.int16)), name


def wrong(m):
    """One wrong argument at a time: (name, value), on the device of the batch."""
    yield "k", m["k"].float()
    yield "v", m["v"][:-1]
    yield "k", m["k"][..., :32]
    yield "kp", m["kp"].transpose(2, 3)
    yield "vp", m["vp"].transpose(2, 3).contiguous()
    yield "bt", m["bt"][:1]
    yield "bt", m["bt"].long()
    yield "cu", m["cu"][:0]
    yield "sp", m["sp"][:-1]
    yield "L", m["L"][None]
    yield "q", m["q"][..., 0]
    yield "q", m["q"][..., ::2]
    yield "out", m["out"].cpu()
    yield "out", m["out"][:-1]
    yield "ws", m["ws"][:16]
    yield "ws", m["ws"].view(torch.int32)
    yield "freq", m["freq"].half()
    yield "freq", m["freq"][:-1]
    yield "max_new", -1
    yield "max_new", "17"
    yield "shared", 7


def refusals(device, monkeypatch):
    seen = []
    for stand_in in (ilpc._NoNative(), None):
        monkeypatch.setattr(ilpc, "_binding", stand_in)
        said = []
        for call in CALLS:
            m = make(device)
            for name, value in wrong(m):
                try:
                    call(dict(m, **{name: value}))
                    said.append((call.__name__, name, None))
                except Exception as e:  # noqa: BLE001
                    said.append((call.__name__, name, type(e), str(e)))
        seen.append(said)
    assert seen[0] == seen[1]
    return seen[0]


def test_refusals_on_the_cpu_equal_the_general_path(monkeypatch):
    said = refusals("cpu", monkeypatch)
    assert all(s[2] is not None for s in said)  # (no tensor is on a GPU)


def test_without_the_native_binding_calls_go_through_ctypes(monkeypatch):
    # not built, or built against another torch: a warning, and the general path's answer
    monkeypatch.setattr(ilpc, "_binding", None)
    monkeypatch.setitem(sys.modules, "paper_2507_08523_amd._binding", None)  # (importing it raises ImportError)
    monkeypatch.delattr("paper_2507_08523_amd._binding", raising=False)
    monkeypatch.setattr(torch.version, "hip", "7")
    with pytest.warns(RuntimeWarning, match="native binding"):
        with pytest.raises(ilpc.ILPCError, match="must be a CUDA/HIP torch tensor"):
            append(make("cpu"))
    assert isinstance(ilpc._binding, ilpc._NoNative)


def test_build_without_a_host_compiler_keeps_the_library(monkeypatch, tmp_path, capsys):
    from paper_2507_08523_amd import build

    stale = tmp_path / "_binding.so"
    stale.write_bytes(b"old")
    monkeypatch.setattr(build, "LIB", str(tmp_path / "libilpc.so"))
    monkeypatch.setattr(build, "BINDING", str(stale))

    def run(cmd, **kw):
        if cmd[0] == "g++":
            raise FileNotFoundError("g++")
        (tmp_path / "libilpc.so.tmp").write_bytes(b"lib")
        return build.subprocess.CompletedProcess(cmd, 0, "", "")

    monkeypatch.setattr(build.subprocess, "run", run)
    monkeypatch.setattr(torch.version, "hip", "7")
    assert build.build() == str(tmp_path / "libilpc.so")
    assert not stale.exists() and "no native binding" in capsys.readouterr().err


@pytest.mark.gpu
def test_refusals_equal_the_general_path(monkeypatch):
    # every wrong argument here is found by a check of shapes, types or sizes on
    # the host; what a call does not look at stays valid and is accepted both ways
    said = refusals("cuda:0", monkeypatch)
    torch.cuda.synchronize()
    refused = {(s[0], s[1]) for s in said if s[2] is not None}
    assert {("append", "k"), ("rope", "freq"), ("attend", "q"), ("attend_ws", "ws"), ("cascade", "shared")} <= refused
