"""The binding's marshalling where no GPU is needed: what it makes of missing
tensors and of host tensors.  The library is loaded, nothing is launched."""
import os

import pytest
import torch

from paper_2104_05588_amd import _lib as L
from paper_2104_05588_amd import build as B

F32 = (torch.float32,)


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(L.LIB_PATH):
        B.build()
    return L.load()


def test_missing_tensors_are_null_pointers(lib):
    """None in a list is the null pointer: the C entry points take it for an empty
    call and refuse it with DASO_EINVAL otherwise."""
    arr = L._ptr_array([None, None], F32, 0, "grads")
    assert len(arr) == 2 and arr[0] is None and arr[1] is None
    assert lib.daso_local_avg(arr, 2, None, 0, None) == L.DASO_OK
    assert lib.daso_local_avg(arr, 2, 0x1000, 8, None) == L.DASO_EINVAL
    assert lib.daso_global_merge(None, arr, 2, L.bucket_table([]), 0, None, 0, None) == L.DASO_OK


@pytest.mark.parametrize("what,call", [
    (r"grads\[0\]", lambda t: L.local_avg([t], t)),
    (r"stale\[0\]", lambda t: L.global_merge(t, [t.to(torch.bfloat16)], [(0, 8, 1)])),
    ("src", lambda t: L.pack_bf16(t, t)),
    ("params", lambda t: L.global_merge(t, [], [(0, 8, 1)])),
])
def test_host_tensors_are_refused_as_such(lib, what, call):
    """A host tensor is named in a ValueError, with or without a GPU in the machine."""
    with pytest.raises(ValueError, match=what + " must be a device tensor"):
        call(torch.zeros(8))


@pytest.mark.gpu
def test_device_tensors_are_checked_one_by_one(lib):
    """Every wrong tensor of a list or on its own is named with what is wrong, wherever it stands;
    missing ones are null pointers between device tensors."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ok, host = torch.zeros(8, device="cuda"), torch.zeros(8)
    wide, short, strided = ok.double(), ok[:4], torch.zeros(16, device="cuda")[::2]
    arr = L._ptr_array([None, ok, None, ok], F32, 8, "grads")
    assert [arr[0], arr[1], arr[2], arr[3]] == [None, ok.data_ptr(), None, ok.data_ptr()]
    for bad, why in ((host, "must be a device tensor"), (wide, "must have dtype"), (short, "contiguous with 8"),
                     (strided, "contiguous with 8")):
        for lst, at in (([bad, ok], 0), ([ok, bad], 1), ([None, bad], 1), ([host if bad is host else ok, ok, bad], 0 if bad is host else 2)):
            with pytest.raises(ValueError, match=rf"grads\[{at}\] .*{why}"):
                L._ptr_array(lst, F32, 8, "grads")
        with pytest.raises(ValueError, match=f"out .*{why}"):
            L._ptr(bad, F32, 8, "out")
    assert L._ptr(ok, F32, 8, "out") == ok.data_ptr() and L._ptr(None, F32, 8, "out") is None


@pytest.mark.parametrize("nb", [0, 1, 2, 64, 257])
def test_bucket_table_holds_what_it_is_given(nb):
    buckets = [(7 * i + (1 << 40), 3 * i, i % 5) for i in range(nb)]
    arr = L.bucket_table(numpy_rows(buckets))
    assert len(arr) == max(nb, 1)
    assert [(b.start, b.numel, b.S, b.reserved) for b in arr] == [(*b, 0) for b in buckets or [(0, 0, 0)]]


def numpy_rows(buckets):
    """The same rows as lists of numpy integers, as a caller may have them."""
    import numpy as np
    return [list(np.asarray(b, dtype=np.int64)) for b in buckets]
