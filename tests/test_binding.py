"""The extension module of the op calls (csrc/pk_call.cpp) against the ctypes conversions of pk.py: same status for every single changed
argument, and None, nothing done, for arguments that are not plain ints, tensors or names; without the module all through ctypes.  Needs no GPU, and runs only where there
is none: the pointers are made up, and a call that passes the library's checks ends at its launch."""
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest
import torch

from paper_2511_13940_amd import pk

pytestmark = pytest.mark.skipif(torch.cuda.device_count() > 0, reason="made-up pointers")

HEAD = dict(P=2, rank=0, M=256, N=256, K=512, dtype="bf16", A=0x1000, B=0x2000, scale_a=None, scale_b=None)
SLOTS = dict(partials=0x3000, outgoing=0x4000, flags_in=0x5000, flags_out=0x6000)
TAIL = dict(status=0x7000, timeout_us=0, stream=0, comm_cus=0)
ROWS = dict(HEAD, chunk_flags=0x5000, epoch=1, C_local=0x3000, **TAIL, act="none")
OPS = {
    "pk_gemm_rs": dict(HEAD, **SLOTS, epoch=1, out_shard=0x8000, phases=3, **TAIL, partial_dtype="f32", workspace=None, b_layout="kn"),
    "pk_gemm_rs_cols": dict(HEAD, **SLOTS, epoch=1, out_shard=0x8000, phases=3, **TAIL, partial_dtype="f32"),
    "pk_gemm_ar": dict(HEAD, **SLOTS, out_full=0x8000, bcast_out=0x9000, ar_flags_in=0xA000, ar_flags_out=0xB000, epoch=1, phases=7, **TAIL,
                       partial_dtype="f32"),
    "pk_ag_gemm": dict(ROWS, workspace=None, b_layout="kn"),
    "pk_ag_gemm_static": ROWS,
    "pk_ag_gemm_k": ROWS,
}
CHANGES = {"P": [3, 0, -1], "rank": [1, 2, -1], "M": [255, 0], "N": [252, 0], "K": [514, 0, -512], "dtype": ["fp8", 1, 7],
           "A": [None, 0, 0x1008], "B": [None, 0x2008], "scale_a": [0x100], "scale_b": [0x100], "epoch": [-1, 2 ** 31, 2 ** 32 - 1],
           "phases": [0, 1, 2, 8, 16, 11], "timeout_us": [2 ** 40], "comm_cus": [-8, 8, 10 ** 6], "partial_dtype": ["bf16", 1, 5],
           "act": ["silu", "gelu_tanh", "relu", 3, 9], "b_layout": ["nk", 1, 0]}
POINTERS = ["partials", "outgoing", "flags_in", "flags_out", "out_shard", "status", "chunk_flags", "C_local", "out_full", "bcast_out",
            "ar_flags_in", "ar_flags_out"]


def _status(call, args):
    try:
        call(*args.values())
        return pk.OK
    except pk.PkError as e:
        return e.code


def _through_ctypes(op, args, monkeypatch):
    with monkeypatch.context() as m:
        m.setattr(pk, "_calls", type("Nothing", (), {op: staticmethod(lambda *a: None)})())
        return _status(getattr(pk, op), args)


@pytest.mark.parametrize("op", OPS)
def test_same_status_for_every_changed_argument(op, monkeypatch):
    base, seen = OPS[op], set()
    variants = [{}] + [{k: v} for k in base for v in CHANGES.get(k, [])] + [{k: v} for k in POINTERS if k in base for v in (None, 0x3008)]
    for change in variants:
        args = dict(base, **change)
        st = getattr(pk._calls, op)(*args.values())
        assert st is not None, change
        assert st == _through_ctypes(op, args, monkeypatch), change
        seen.add(st)
    assert {pk.ERR_SHAPE, pk.ERR_DTYPE, pk.ERR_HIP} <= seen             # (the static one looks for its scratch array first)


class _Sub(torch.Tensor):
    pass


@pytest.mark.parametrize("op", OPS)
def test_other_kinds_of_arguments_are_left_to_ctypes(op):
    call = getattr(pk._calls, op)
    cpu = torch.zeros(8)
    odd = {"P": [2.0, True, np.int64(2), 2 ** 31], "M": [2 ** 70], "dtype": ["fp16", None, 1.0],
           "A": [cpu, cpu.as_subclass(_Sub), "x", -1, True, torch.zeros(8, device="meta")], "epoch": [1.0], "timeout_us": [-1],
           "stream": ["x", cpu], "partial_dtype": ["f16"], "act": ["tanh"], "b_layout": ["tn", 2], "workspace": [0x1000, cpu]}
    for k, values in odd.items():
        for v in values if k in OPS[op] else []:
            assert call(*dict(OPS[op], **{k: v}).values()) is None, (k, v)
    assert call(*list(OPS[op].values())[:-1]) is None                       # an argument too few
    with pytest.raises(ValueError):
        getattr(pk, op)(*dict(OPS[op], A=cpu).values())


@pytest.mark.parametrize("content", [None, "no shared object"])
def test_without_the_module_the_ops_go_through_ctypes(content, monkeypatch, tmp_path):
    path = tmp_path / "_pk_call.so"
    if content is not None:
        path.write_text(content)
    monkeypatch.setattr(pk, "CALL_PATH", str(path))
    monkeypatch.setattr(pk, "_calls", pk._Calls())
    with pytest.warns(RuntimeWarning, match="ctypes"):
        first = _status(pk.pk_gemm_rs, dict(OPS["pk_gemm_rs"], M=255))
    assert first == pk.ERR_SHAPE
    for op in OPS:
        assert _status(getattr(pk, op), OPS[op]) == _through_ctypes(op, OPS[op], monkeypatch)


def test_a_module_built_for_something_else_is_not_used(monkeypatch, tmp_path):
    built = open(pk.CALL_PATH, "rb").read()
    for name, old in (("interface", pk.load_binding().built_for.split()[0].encode()), ("torch", b" torch " + torch.__version__.encode())):
        assert old in built
        path = tmp_path / name / "_pk_call.so"
        path.parent.mkdir()
        path.write_bytes(built.replace(old, old[:-1] + b"?"))
        monkeypatch.setattr(pk, "CALL_PATH", str(path))
        with pytest.raises(RuntimeError, match="was built for"):
            pk.load_binding()
        monkeypatch.setattr(pk, "_calls", pk._Calls())
        with pytest.warns(RuntimeWarning, match="was built for"):
            assert _status(pk.pk_gemm_rs, dict(OPS["pk_gemm_rs"], M=255)) == pk.ERR_SHAPE


def test_the_module_calls_the_library_that_pk_has_loaded(tmp_path):
    shutil.copy(pk.LIB_PATH, tmp_path / "libpk.so")                         # another one, where the loader would look first
    code = ("from paper_2511_13940_amd import pk; pk.load_binding(); "
            "print({l.split()[-1] for l in open('/proc/self/maps') if 'libpk.so' in l} == {pk.LIB_PATH})")
    env = dict(os.environ, LD_LIBRARY_PATH=os.pathsep.join([str(tmp_path), os.environ.get("LD_LIBRARY_PATH", "")]))
    run = subprocess.run([sys.executable, "-c", code], env=env, cwd=os.path.dirname(os.path.dirname(pk.LIB_PATH)), capture_output=True, text=True)
    assert run.stdout.strip() == "True", run
