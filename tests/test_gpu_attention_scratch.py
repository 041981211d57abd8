"""The bf16 decode attention keeps its registers: an instance that spills makes every launch set up scratch memory
(0.5 us of a layer's 10)."""
import ctypes

import pytest
import torch

from paper_2403_18647_amd import binding as B

pytestmark = pytest.mark.gpu


class _Attributes(ctypes.Structure):   # hipFuncAttributes
    _fields_ = [("binaryVersion", ctypes.c_int), ("cacheModeCA", ctypes.c_int), ("constSizeBytes", ctypes.c_size_t),
                ("localSizeBytes", ctypes.c_size_t), ("maxDynamicSharedSizeBytes", ctypes.c_int),
                ("maxThreadsPerBlock", ctypes.c_int), ("numRegs", ctypes.c_int), ("preferredShmemCarveout", ctypes.c_int),
                ("ptxVersion", ctypes.c_int), ("sharedSizeBytes", ctypes.c_size_t)]


@pytest.mark.parametrize("dh,cols", [(128, 1), (128, 2), (128, 4), (128, 8), (64, 1), (64, 2), (64, 4)])
def test_no_scratch(dh, cols):
    torch.cuda.init()
    L = B.lib()
    kernel = ctypes.c_void_p.in_dll(L, f"_ZN5sdsat11attn_kernelItLi{dh}ELi{cols}EEEvNS_8AttnArgsE")
    a = _Attributes()
    assert L.hipFuncGetAttributes(ctypes.byref(a), ctypes.c_void_p(ctypes.addressof(kernel))) == 0
    assert a.numRegs > 0 and a.localSizeBytes == 0, (a.numRegs, a.localSizeBytes)
