"""The native marshalling declines what is not a well-formed call, and the
Python code then says what is wrong with it (no GPU needed: host tensors are
never well-formed arguments, and nothing is launched)."""
import pytest
import torch

from paper_2607_29221_amd import mosaic as m
from paper_2607_29221_amd.mosaic import Digits


def _i32(*shape):
    return torch.zeros(shape, dtype=torch.int32)


def _dig(rows, cols):
    return Digits.empty(rows, cols, device="cpu")


CALLS = {
    "sample": lambda: m.mosaic_sample(m.rng(1, 2, 3, m.DIST_UNIFORM), 4, 8, out=_i32(4, 8)),
    "mask": lambda: m.mosaic_mask(_i32(4, 8), None, None, 4, 8, out=_i32(4, 8)),
    "masked_matmul": lambda: m.mosaic_masked_matmul(_dig(2, 64), _dig(3, 64), 2, 3, 64, _i32(2, 3)),
    "integrity_check": lambda: m.mosaic_integrity_check(_dig(2, 64), _dig(3, 64), _dig(2, 64), _i32(3, 64), 2, 3, 64,
                                                        64, _i32(2, 3), torch.zeros(1, dtype=torch.int64)),
    "unmask": lambda: m.mosaic_unmask(_i32(2, 3), None, _dig(2, 64), _dig(3, 64), 2, 3, 64, y=_i32(2, 3)),
    "unmask_words": lambda: m.mosaic_unmask_words(_i32(2, 3), None, _i32(2, 64), _dig(3, 64), 2, 3, 64, y=_i32(2, 3)),
    "rotate_quantize_mask": lambda: m.mosaic_rotate_quantize_mask(torch.zeros(2, 1024), 127, _dig(2, 1024),
                                                                  scale=torch.zeros(2)),
    "hadamard_rotate": lambda: m.mosaic_hadamard_rotate(torch.zeros(2, 64), torch.zeros(2, 64)),
    "quantize_rows": lambda: m.mosaic_quantize_rows(torch.zeros(2, 64), 127, q=_i32(2, 64)),
    "stream_gather": lambda: m.mosaic_sparse_stream_gather_rows(m.rng(1, 2, 3, m.DIST_SPARSE), 2, 8, _i32(8, 4), 4,
                                                                _i32(2, 4)),
    "stream_terms": lambda: m.mosaic_sparse_stream_gather_rows_terms([(m.rng(1, 2, 3, m.DIST_SPARSE), 8, _i32(8, 4))],
                                                                     2, 4, _i32(2, 4)),
}


@pytest.mark.parametrize("name", list(CALLS))
def test_host_tensors_are_refused(name):
    with pytest.raises(ValueError):
        CALLS[name]()


def test_native_functions_decline():
    b = m._native()
    r = m.rng(1, 2, 3, m.DIST_UNIFORM)
    assert b.sample(r, 4, 8, _i32(4, 8), None) is None              # host memory
    assert b.sample(b"short", 4, 8, None, None) is None             # not an rng
    assert b.sample(r, 0, 8, None, None) is None                    # empty
    assert b.sample(r, 4.0, 8, None, None) is None                  # not a size
    assert b.sample(r, 1 << 70, 8, None, None) is None              # does not fit
    assert b.sample(r, 4, 8) is None                                # too few arguments
    assert b.masked_matmul(None, None, 2, 3, 64, None) is None
    assert b.masked_matmul(object(), 5, 2, 3, 64, "c") is None
    assert b.stream_terms([], 2, 4, None, False) is None
    with pytest.raises(TypeError):
        b.bind((1, 2), None, None, m._lib.MosaicRng)


def test_only_generators_are_taken_for_generators(monkeypatch):
    """Any other object of the struct's size raises, as ctypes has it."""
    import ctypes

    import numpy as np
    b = m._native()
    args = [tuple(ctypes.cast(getattr(m._lib.load(), n), ctypes.c_void_p).value for n in m._BOUND),
            lambda: 0, lambda device: 0, m._lib.MosaicRng]
    monkeypatch.setattr(m, "_stream", lambda: 0)
    b.bind(*args)                       # a current stream without a GPU; the library refuses calls without an output
    try:
        r = m.rng(1, 2, 3, m.DIST_UNIFORM)
        size = ctypes.sizeof(r)
        assert isinstance(b.sample(r, 4, 8, None, None), int)
        for o in (bytes(size), bytearray(size), np.zeros(size, np.uint8), (ctypes.c_char * size)()):
            assert b.sample(o, 4, 8, None, None) is None
            assert b.mask(None, None, o, 4, 8, None, None, False) is None
            assert b.stream_terms([(o, 8, None)], 2, 4, None, False) is None
            with pytest.raises((TypeError, ctypes.ArgumentError)):
                m.mosaic_sample(o, 4, 8)
    finally:
        b.bind(args[0], torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream, m._lib.MosaicRng)


def test_binding_of_another_torch_or_python_is_refused(monkeypatch, tmp_path):
    """_binding.so reads tensors by the layout of the torch it was compiled
    against: it is not loaded into another one, nor without its stamp."""
    import shutil
    from paper_2607_29221_amd import build
    assert m._lib.binding_stale_reason() is None
    monkeypatch.setattr(m, "_b", None)
    with monkeypatch.context() as c:
        c.setattr(torch, "__version__", "0.0.1")
        with pytest.raises(RuntimeError, match="run `python -m"):
            m._native()
    for name in ("BINDING", "BINDING_STAMP"):
        with monkeypatch.context() as c:
            c.setattr(build, name, str(tmp_path / name))
            with pytest.raises(RuntimeError, match="is missing"):
                m._native()
    with monkeypatch.context() as c:
        shutil.copytree(build.CSRC, tmp_path / "csrc")
        (tmp_path / "csrc" / "binding.cpp").write_text("// edited")
        c.setattr(build, "CSRC", str(tmp_path / "csrc"))
        assert "changed" in m._lib.binding_stale_reason()
    assert m._native() is not None


class _Recorder:
    """Stands in for the native marshalling (declines) and for the library (records)."""

    def __init__(self):
        self.ldd = None

    def cols_terms(self, *args):
        return None

    def mosaic_sparse_gather_cols_terms(self, terms, n, *args):
        self.ldd = [terms[i].ldd for i in range(n)]
        return 0


class _DeviceLike:
    """A host tensor that answers the shape checks as a device tensor would."""

    def __init__(self, t):
        self.t, self.is_cuda, self.dtype, self.shape = t, True, t.dtype, t.shape
        self.dim, self.stride, self.data_ptr, self.numel = t.dim, t.stride, t.data_ptr, t.numel


@pytest.mark.parametrize("stride", [0, 5, 64, 70])
def test_gather_cols_terms_passes_the_row_stride(monkeypatch, stride):
    """Rows of d that share memory (an expanded view) keep their stride: a longer
    one would read past the view's storage."""
    rec = _Recorder()
    monkeypatch.setattr(m, "_b", rec)
    monkeypatch.setattr(m._lib, "load", lambda: rec)
    monkeypatch.setattr(m, "_stream", lambda: 0)
    d = _DeviceLike(torch.zeros(1024, dtype=torch.int32).as_strided((8, 64), (stride, 1)))
    p = m.SparseRows(_i32(4).long(), _i32(4), _i32(4), 3, 64)
    m.mosaic_sparse_gather_cols_terms([(p, d)], 8, _DeviceLike(_i32(8, 3)))
    assert rec.ldd == [stride]


@pytest.mark.gpu
def test_flag_without_truth_value_is_refused():
    """A flag whose truth value raises is left to the Python code, which raises
    the same error as before."""
    x = torch.zeros(2, 64, device="cuda")
    with pytest.raises(RuntimeError, match="ambiguous"):
        m.mosaic_hadamard_rotate(x, torch.empty_like(x), inverse=torch.zeros(2))
