"""The Python binding's per-step calls on both of their routes, the C argument converter (csrc/pycall.cpp) and ctypes,
and the converter's build (no GPU: every call here fails at its checks or at the first HIP call, so the module is
skipped where a GPU is visible)."""
import ctypes
import importlib.machinery
import os
import warnings

import numpy as np
import pytest
import torch

from paper_2606_01483_amd import _build
from paper_2606_01483_amd import murmur as M

pytestmark = pytest.mark.skipif(torch.cuda.device_count() > 0, reason="host-only checks run where no GPU is visible")


@pytest.fixture(scope="module", autouse=True)
def _lib():
    if not os.path.exists(M.LIB_PATH):
        _build.build()
    M.lib()


# ---- the converter's build ---------------------------------------------------------------------------------------

def fake_build(monkeypatch, tmp_path, fail):
    """_build.build() into tmp_path with its commands replaced: each creates its output, the converter's fails."""
    def run(cmd):
        if fail and any(str(c).endswith("pycall.cpp") for c in cmd):
            raise RuntimeError("build step failed (1): Python.h: No such file or directory")
        with open(cmd[cmd.index("-o") + 1], "w") as f:
            f.write("built")
    monkeypatch.setattr(_build, "_run", run)
    monkeypatch.setattr(_build, "PKG", str(tmp_path))
    monkeypatch.setattr(_build, "BUILD_DIR", str(tmp_path))
    monkeypatch.setattr(_build, "LIB", str(tmp_path / "libmurmur.so"))
    monkeypatch.setattr(_build, "PYCALL", str(tmp_path / os.path.basename(_build.PYCALL)))


def test_build_without_the_converter(monkeypatch, tmp_path):
    """Where the converter does not compile (no Python headers) the library is built all the same, and no converter
    of an earlier build stays beside it, whose calls might be laid out for another library."""
    fake_build(monkeypatch, tmp_path, fail=True)
    (tmp_path / os.path.basename(_build.PYCALL)).write_text("old")
    (tmp_path / "_pycall.so").write_text("older")
    with pytest.warns(UserWarning, match="Python.h"):
        assert _build.build() == str(tmp_path / "libmurmur.so")
    assert (tmp_path / "libmurmur.so").read_text() == "built"
    assert [f for f in os.listdir(tmp_path) if "pycall" in f] == []
    fake_build(monkeypatch, tmp_path, fail=False)
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        _build.build()
    assert (tmp_path / os.path.basename(_build.PYCALL)).read_text() == "built"


def test_the_converter_is_for_one_interpreter():
    """Its file carries this interpreter's tag, so another Python version does not load it and goes through ctypes."""
    name = os.path.basename(_build.PYCALL)
    suffixes = importlib.machinery.EXTENSION_SUFFIXES
    assert name == "_pycall" + suffixes[0]
    assert suffixes[0] not in (".so", ".abi3.so")


# ---- the two routes ----------------------------------------------------------------------------------------------

FAKE = 0x100000  # never dereferenced: every call fails its checks, or with no GPU its first HIP call


def kv():
    return M.murmur_kv(FAKE, FAKE, 1, 4096, 4096 * 128 * 4, 4096 * 128 * 4, 4096 * 128, 128)


def ring():
    return M.murmur_ring(64, FAKE, FAKE)


class Buffer:
    """Stands for a device tensor."""
    def data_ptr(self):
        return FAKE


# (wrapper, its arguments by name, in order)
ATTN = dict(max_keep=850, B=12, Hq=28, Hkv=4, D=128, scale=1.0, split_len=0, out_dev=FAKE,
            out_dtype=M.MURMUR_DTYPE_BF16, lse_dev=None)
WS = dict(ws_dev=FAKE, ws_bytes=1 << 30)
SEG = dict(seg_dev=Buffer(), pol_dev=FAKE, pol_per_seq=1)
SETS = dict(idx_dev=FAKE, count_dev=FAKE, ranges_dev=None)
PAGED = dict(block_table_dev=FAKE, max_blocks=64, block_size=16)
CALLS = {
    "murmur_evict_compact": dict(**SEG, B=12, idx_dev=FAKE, max_keep=850, count_dev=FAKE, ranges_dev=None, stream=0),
    "murmur_evict_compact_paged": dict(**SEG, B=12, **PAGED, idx_dev=FAKE, max_keep=850, count_dev=FAKE,
                                       ranges_dev=None, stream=0),
    "murmur_decode_attn": dict(q_dev=FAKE, kv=kv(), idx_dev=FAKE, ranges_dev=None, count_dev=Buffer(), **ATTN, **WS,
                               stream=0),
    "murmur_decode_step": dict(**SEG, q_dev=FAKE, kv=kv(), **SETS, **ATTN, **WS, stream=0),
    "murmur_decode_step_static": dict(**SEG, q_dev=FAKE, kv=kv(), **SETS, **ATTN, stream=0),
    "murmur_decode_step_ring": dict(**SEG, ring=ring(), q_dev=FAKE, kv=kv(), **SETS, **ATTN, **WS, stream=0),
    "murmur_paged_step": dict(**SEG, B=12, **PAGED, free_stack_dev=FAKE, free_top_dev=FAKE, capacity=64,
                              full_scan=False, pool=kv(), Hkv=4, k_new_dev=FAKE, v_new_dev=FAKE, stream=0),
}


def outcome(name, **over):
    """What the call raises: the C status and message, or the Python error's kind."""
    try:
        getattr(M, name)(**{**CALLS[name], **over})
    except M.MurmurError as e:
        return e.code, M.murmur_last_error()
    except (TypeError, AttributeError, OverflowError, ctypes.ArgumentError):
        return "refused"
    return "returned"


@pytest.fixture(params=["converter", "ctypes"])
def route(request, monkeypatch):
    lib = M.lib()
    if request.param == "converter":
        if M._pycall is None:
            pytest.skip("built without the converter")
        assert all(convert is not None for _, _, convert in lib.per_step.values())
    else:
        monkeypatch.setattr(lib, "per_step", {n: (fn, at, None) for n, (fn, at, _) in lib.per_step.items()})
    return request.param


def test_every_per_step_call_is_here():
    assert sorted(CALLS) == sorted("murmur_" + n for n in M._PER_STEP)


@pytest.mark.parametrize("name", sorted(CALLS))
def test_the_call_arrives(route, name):
    """With valid arguments the call passes every check and fails where it needs a GPU; ints may be numpy's or of any
    type with __index__, the scale an int or a numpy float, a buffer a tensor, an address or None."""
    assert outcome(name)[0] == M.MURMUR_EHIP
    for arg, value in CALLS[name].items():
        if type(value) is int and not arg.endswith("_dev") and arg != "stream":
            for same in (np.int64(value), np.int32(value % 2**31)):
                if int(same) == value:
                    assert outcome(name, **{arg: same})[0] == M.MURMUR_EHIP, arg
        if arg == "scale":
            for same in (1, np.float32(1), np.float64(1), "1.0", True):
                assert outcome(name, scale=same)[0] == M.MURMUR_EHIP, same
        if arg.endswith("_dev") and value is FAKE:
            assert outcome(name, **{arg: Buffer()})[0] == M.MURMUR_EHIP, arg


@pytest.mark.parametrize("name", sorted(CALLS))
def test_every_argument_reaches_its_place(route, name, monkeypatch):
    """Each argument in turn replaced by a value its check refuses gives the message of that check."""
    bad = dict(seg_dev=FAKE + 2, pol_dev=FAKE + 2, idx_dev=FAKE + 2, count_dev=FAKE + 2, ranges_dev=FAKE + 2,
               pol_per_seq=9, B=0, max_keep=0, q_dev=FAKE + 8, Hq=27, Hkv=5, D=64, scale=float("nan"), split_len=31,
               out_dev=FAKE + 8, out_dtype=7, lse_dev=FAKE + 2, ws_dev=FAKE + 64, ws_bytes=1, block_table_dev=FAKE + 2,
               max_blocks=0, block_size=12, free_stack_dev=FAKE + 2, free_top_dev=FAKE + 2, capacity=0,
               k_new_dev=FAKE + 8, v_new_dev=FAKE + 8, kv=M.murmur_kv(), pool=M.murmur_kv(), ring=M.murmur_ring())
    convert_off = {n: (fn, at, None) for n, (fn, at, _) in M.lib().per_step.items()}
    for arg in CALLS[name]:
        if arg not in bad or (name == "murmur_decode_attn" and arg == "ranges_dev"):
            continue
        bad["Hkv"] = 0 if name == "murmur_paged_step" else 5
        got = outcome(name, **{arg: bad[arg]})
        assert got[0] in (M.MURMUR_EINVAL, M.MURMUR_EUNSUPPORTED, M.MURMUR_ENOSPACE), arg
        with monkeypatch.context() as m:
            m.setattr(M.lib(), "per_step", convert_off)
            assert outcome(name, **{arg: bad[arg]}) == got, arg


class Other(ctypes.Structure):
    """Of murmur_kv's size and of another type."""
    _fields_ = [("x", ctypes.c_uint8 * ctypes.sizeof(M.murmur_kv))]


class OtherRing(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint8 * ctypes.sizeof(M.murmur_ring))]


class OwnKv(M.murmur_kv):
    pass


@pytest.mark.parametrize("name,arg", [(n, a) for n in sorted(CALLS) for a in ("kv", "pool", "ring") if a in CALLS[n]])
def test_only_the_structure_itself(route, name, arg):
    """A structure argument is the structure or a subclass of it, not something else of its size."""
    size = ctypes.sizeof(CALLS[name][arg])
    other = OtherRing() if arg == "ring" else Other()
    assert ctypes.sizeof(other) == size
    for x in (bytes(size), bytearray(size), np.zeros(size, dtype=np.uint8), other, M.murmur_seg(), 0, FAKE, "kv"):
        assert outcome(name, **{arg: x}) == "refused", type(x)
    if arg != "ring":
        k = kv()
        own = OwnKv(*[getattr(k, f) for f, _ in M.murmur_kv._fields_])
        assert outcome(name, **{arg: own})[0] == M.MURMUR_EHIP
    if arg == "pool":
        assert outcome(name, pool=None)[0] == M.MURMUR_EHIP


@pytest.mark.parametrize("name", sorted(CALLS))
def test_other_types_are_refused(route, name):
    for arg, value in CALLS[name].items():
        if arg.endswith("_dev"):
            assert outcome(name, **{arg: object()}) == "refused", arg
        elif type(value) is int and arg != "stream":
            for x in (1.5, "1", None, object()):
                assert outcome(name, **{arg: x}) == "refused", (arg, x)
        elif arg == "scale":
            assert outcome(name, scale=None) == "refused" and outcome(name, scale=object()) == "refused"
