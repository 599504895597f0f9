"""Door onto bcs_windows.hip: rows in device memory against their definition by windows."""
import ctypes
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SRC = os.path.join(HERE, "bcs_windows.hip")
LIB = os.path.join(HERE, "libbcs_windows.so")

_lib = None


def build():
    from paper_2205_10072_amd import build as b
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + b.FLAGS +
                   ["-I", os.path.join(ROOT, "paper_2205_10072_amd", "csrc"), "-o", LIB, SRC], check=True)
    return LIB


def lib():
    global _lib
    if _lib is None:
        if not os.path.exists(LIB):
            build()
        L = ctypes.CDLL(LIB)
        L.bw_check.argtypes = [ctypes.c_int32] * 4 + [ctypes.c_void_p] * 2
        L.bw_result.restype = ctypes.c_int64
        _lib = L
    return _lib


def check(p, root, r0, r1, recv, send=None):
    """Enqueues the check of the rows of ranks [r0, r1) (tensors of r1 - r0 rows, made on the default stream)."""
    for t in (recv, send):
        assert t is None or (t.is_cuda and t.is_contiguous() and t.numel() == (r1 - r0) * (p - 1).bit_length())
    assert lib().bw_check(p, root, r0, r1, None if recv is None else recv.data_ptr(),
                          None if send is None else send.data_ptr()) == 0


def differences():
    """Entries that differed in the checks since the last call."""
    n = lib().bw_result()
    assert n >= 0
    return n
