"""The native argument marshalling (csrc/oqm_binding.cpp) takes and refuses what the ctypes
prototypes of the same functions do.  No GPU: every call ends in the library's validation."""
import ctypes as C
import os
import subprocess
import sys
import sysconfig

import numpy as np
import pytest
import torch


@pytest.fixture()
def store():
    from paper_2510_18269_amd import oqm
    h = oqm.tom_oqm_create(oqm.make_config(2, 2, 4, 64, 4, 32, 8))
    oqm.tom_oqm_bind(h, 0x1000, 0x1000, 0x1000)
    yield oqm, h
    oqm.tom_oqm_destroy(h)


class FakeTensor:
    """What the binding reads of a tensor: its place, its strides, its size."""
    def __init__(self, strides=(), is_cuda=True, numel=0):
        self.strides, self.is_cuda, self.n = strides, is_cuda, numel
    def data_ptr(self): return 0x1000
    def dim(self): return len(self.strides)
    def stride(self): return self.strides
    def numel(self): return self.n
    def element_size(self): return 1


def test_arguments_that_ctypes_refuses(store):
    oqm, h = store
    for bad in (1.0, "1", None):
        with pytest.raises(C.ArgumentError):
            oqm.tom_oqm_topk(0x1000, 8, bad, 0, 1, 0x1000)
        with pytest.raises(C.ArgumentError):
            oqm.tom_oqm_set_num_groups(h, bad)
    with pytest.raises(AssertionError, match="device tensor"):
        oqm.tom_oqm_topk(torch.zeros(8), 8, 1, 8, 1, 0x1000)
    with pytest.raises(AttributeError):
        oqm.tom_oqm_topk(object(), 8, 1, 8, 1, 0x1000)
    with pytest.raises(AttributeError):
        oqm.tom_oqm_retrieve(h, 0, 2, 0x1000, 1, 1, 0x1000, 8, 0x1000, 0x1000, 0x1000, 0x1000, q_dtype=oqm.TOM_F32)


def test_integers_are_truncated_like_c_int32(store):
    oqm, h = store
    oqm.tom_oqm_set_num_groups(h, (1 << 32) + 3)
    assert oqm.tom_oqm_num_groups(h) == 3
    with pytest.raises(oqm.TomError) as e:
        oqm.tom_oqm_set_num_groups(h, -1)
    assert e.value.status == oqm.TOM_ERR_INVALID_ARG and "n = -1" in str(e.value)
    assert oqm.tom_oqm_topk(0, 8, 0, 8, 3, 0) == 3        # no rows: nothing launched, k_eff returned
    with pytest.raises(oqm.TomError, match="handle is NULL"):
        oqm.tom_oqm_set_num_groups(None, 0)


class AsParameter:
    def __init__(self, value): self._as_parameter_ = value


class Index:
    def __init__(self, value): self.value = value
    def __index__(self): return self.value


def test_integers_of_other_types(store):
    """Whatever has __index__, and the ctypes integer of the parameter's own type; no floats."""
    oqm, h = store
    kinds = (np.int32, np.int64, np.uint8, np.array, torch.tensor, Index, lambda v: torch.tensor([v]))
    for kind in (*kinds, C.c_int32, lambda v: AsParameter(v), lambda v: AsParameter(C.c_int32(v))):
        oqm.tom_oqm_set_num_groups(h, kind(5))
        assert oqm.tom_oqm_num_groups(h) == 5
        assert oqm.tom_oqm_topk(0, 8, 0, 8, kind(3), 0) == 3
        assert oqm.tom_oqm_quantize_append(h, kind(0), kind(2), kind(0), 0x1000, 0x1000, strides=(1, 1, 1, 64)) == 5
    for kind in (*kinds, C.c_int64):      # the 64-bit stride of the scores
        with pytest.raises(oqm.TomError, match="score_stride < n_groups"):
            oqm.tom_oqm_topk(0, kind(7), 0, 8, 3, 0)
        assert oqm.tom_oqm_topk(0, kind(8), 0, 8, 3, 0) == 3
    oqm.tom_oqm_set_num_groups(h, Index((1 << 32) + 2))
    assert oqm.tom_oqm_num_groups(h) == 2
    need = oqm.tom_oqm_score_workspace_bytes(h, 2, 1)
    short = FakeTensor(numel=np.int64(need - 1))
    with pytest.raises(oqm.TomError, match=f"{need} bytes needed, {need - 1} given"):
        oqm.tom_oqm_score_groups(h, 0, np.int32(2), 0x1000, np.int64(1), 0x1000, 8, workspace=short, q_dtype=np.int8(0))
    for bad in (np.float32(3), torch.tensor(3.0), C.c_int64(3), AsParameter(3.0), object()):
        with pytest.raises(C.ArgumentError):
            oqm.tom_oqm_topk(0, 8, 0, 8, bad, 0)
    for bad in (3.0, np.float64(8), C.c_int32(8)):
        with pytest.raises(C.ArgumentError):
            oqm.tom_oqm_topk(0, bad, 0, 8, 3, 0)


def test_handles_are_those_of_c_void_p(store):
    """Of a NULL-able pointer argument ctypes takes an int, None and its own pointer objects; nothing that merely
    has an address: a tensor's memory must never be taken for a handle."""
    oqm, h = store
    calls = (lambda x, **kw: oqm.tom_oqm_set_num_groups(x, 3),
             lambda x, **kw: oqm.tom_oqm_quantize_append(x, 0, 2, 0, 0x1000, 0x1000, strides=(1, 1, 1, 64), **kw),
             lambda x, **kw: oqm.tom_oqm_score_groups(x, 0, 0, 0x1000, 1, 0x1000, 8, q_dtype=oqm.TOM_F32, **kw),
             lambda x, **kw: oqm.tom_oqm_dequant_gather(x, 0, 0, 0x1000, 1, 1, 0x1000, 0x1000, **kw),
             lambda x, **kw: oqm.tom_oqm_assemble_active(x, 0, 0, 0x1000, 1, 1, 0, None, None, 0x1000, 0x1000, **kw),
             lambda x, **kw: oqm.tom_oqm_retrieve(x, 0, 0, 0x1000, 1, 1, 0x1000, 8, 0x1000, 0x1000, 0x1000, None,
                                                  q_dtype=oqm.TOM_F32, **kw),
             lambda x, **kw: oqm.tom_oqm_retrieve_noalloc(x, 0, 0, 0x1000, 1, 1, 0x1000, 8, 0x1000, 0x1000, 0x1000,
                                                          q_dtype=oqm.TOM_F32, **kw))
    stand_in = FakeTensor()
    stand_in.data_ptr = lambda: h      # were it read, it would be a valid handle
    for call in calls:
        for good in (h, C.c_void_p(h), C.cast(h, C.POINTER(C.c_char)), AsParameter(h), AsParameter(C.c_void_p(h))):
            call(good)
        for null in (None, C.c_void_p()):
            with pytest.raises(oqm.TomError, match="handle is NULL"):
                call(null)
        for bad in (stand_in, torch.tensor(h), 1.0, C.c_int64(h), object(), AsParameter(stand_in)):
            with pytest.raises(C.ArgumentError):
                call(bad)
    for call in calls[1:]:             # the same holds of the stream's address
        for stream in (0, None, C.c_void_p(), AsParameter(0)):
            call(h, stream=type("Stream", (), {"cuda_stream": stream}))
        with pytest.raises(C.ArgumentError):
            call(h, stream=type("Stream", (), {"cuda_stream": 1.0}))


def test_strides_of_tensors_and_of_raw_pointers(store):
    oqm, h = store
    good = (2 * 2 * 4 * 64, 2 * 4 * 64, 4 * 64, 64, 1)
    with pytest.raises(AssertionError, match="contiguous channel"):
        oqm.tom_oqm_quantize_append(h, 0, 2, 1, FakeTensor(good[1:]), FakeTensor(good[1:]))
    with pytest.raises(AssertionError, match="contiguous channel"):
        oqm.tom_oqm_quantize_append(h, 0, 2, 1, FakeTensor(good[:4] + (2,)), FakeTensor(good[:4] + (2,)))
    with pytest.raises(AssertionError):
        oqm.tom_oqm_quantize_append(h, 0, 2, 1, FakeTensor(good), FakeTensor((4,) + good[1:]))
    with pytest.raises(oqm.TomError, match="strides"):    # an odd frame stride, from the tensor and as given
        oqm.tom_oqm_quantize_append(h, 0, 2, 1, FakeTensor((3,) + good[1:]), FakeTensor((3,) + good[1:]))
    with pytest.raises(oqm.TomError, match=r"strides\[0\] = 3"):
        oqm.tom_oqm_quantize_append(h, 0, 2, 1, 0x1000, 0x1000, strides=[3, 1024, 256, 64])
    with pytest.raises(oqm.TomError, match="token stride 0"):   # fewer than four: the rest are 0, as in a C array
        oqm.tom_oqm_quantize_append(h, 0, 2, 1, 0x1000, 0x1000, strides=(2048, 1024, 256))
    with pytest.raises(IndexError):
        oqm.tom_oqm_quantize_append(h, 0, 2, 1, 0x1000, 0x1000, strides=(1, 2, 3, 4, 5))
    assert oqm.tom_oqm_quantize_append(h, 0, 2, 0, FakeTensor(good), FakeTensor(good)) == 0
    as_list = [np.int64(s) for s in good]
    assert oqm.tom_oqm_quantize_append(h, 0, 2, 0, FakeTensor(as_list), FakeTensor(good)) == 0


def test_workspace_size_is_that_of_the_tensor(store):
    oqm, h = store
    oqm.tom_oqm_set_num_groups(h, 4)
    need = oqm.tom_oqm_score_workspace_bytes(h, 2, 1)
    with pytest.raises(oqm.TomError, match=f"{need} bytes needed, {need - 1} given"):
        oqm.tom_oqm_score_groups(h, 0, 2, 0x1000, 1, 0x1000, 8, workspace=FakeTensor(numel=need - 1), q_dtype=oqm.TOM_F32)
    with pytest.raises(oqm.TomError, match="0 given"):
        oqm.tom_oqm_score_groups(h, 0, 2, 0x1000, 1, 0x1000, 8, q_dtype=oqm.TOM_F32)


def test_calls_reach_the_library_beside_the_binding(tmp_path):
    """Another libtom_oqm.so on the loader's path is not the one that the handles come from."""
    calls = ("set_num_groups", "quantize_append", "score_groups", "topk", "dequant_gather", "assemble_active", "retrieve",
             "retrieve_noalloc")
    (tmp_path / "other.c").write_text("".join(f"int tom_oqm_{c}() {{ return 42; }}\n" for c in calls))
    subprocess.run(["gcc", "-w", "-shared", "-fPIC", str(tmp_path / "other.c"), "-o", str(tmp_path / "libtom_oqm.so")], check=True)
    code = ("from paper_2510_18269_amd import oqm\n"
            "h = oqm.tom_oqm_create(oqm.make_config(2, 2, 4, 64, 4, 32, 8))\n"
            "oqm.tom_oqm_set_num_groups(h, 3)\n"
            "print(oqm.tom_oqm_num_groups(h))")
    path = os.pathsep.join([str(tmp_path), *filter(None, [os.environ.get("LD_LIBRARY_PATH")])])
    r = subprocess.run([sys.executable, "-c", code], env=dict(os.environ, LD_LIBRARY_PATH=path), capture_output=True, text=True,
                       cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    assert r.stdout.strip() == "3", r.stderr


def test_binding_is_built_for_this_interpreter(store):
    """CPython's headers fix the binding's layout: a file without the interpreter's tag would be loaded by any."""
    oqm, _ = store
    assert os.path.basename(oqm._native.__file__) == "_oqm_binding" + sysconfig.get_config_var("EXT_SUFFIX")
