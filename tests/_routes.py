"""The kernel a GEMM of given sizes takes (fp8q_gemm_route of the library, a
host function), by name, so that a test can hold its shapes to the path that
it is about."""
import ctypes

import paper_2609_22870_amd as fp8q

NAMES = ("large", "mid", "eight waves", "small", "two K groups", "thin", "split-K")
FORMS = {"tensor": 0, "row": 1, "block": 2, "blockk": 3, "pow2": 4, "quantized": 5, "splitk tensor": 6,
         "splitk row": 7, "splitk block": 8, "splitk blockk": 9}


def route(form, M, K, N):
    fn = fp8q.lib().fp8q_gemm_route
    fn.argtypes = [ctypes.c_int] + [ctypes.c_int64] * 3
    fn.restype = ctypes.c_int
    return NAMES[fn(FORMS[form], M, N, K)]


def few_rows(rows, cols):
    """Whether 1x128 quantization (plain layout) takes two rows a thread."""
    fn = fp8q.lib().fp8q_quantize_few_rows
    fn.argtypes = [ctypes.c_int64] * 2
    fn.restype = ctypes.c_int
    return bool(fn(rows, cols))
