"""arithmetic.hip, built in place: the searches' arithmetic as the kernels have it."""
import ctypes as C
import os

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(HERE, "libarithmetic.so")


def build():
    from paper_2305_12356_amd import build as b
    return b.build_library(os.path.join(HERE, "arithmetic.hip"), LIB)


def load():
    if not os.path.exists(LIB):
        build()
    lib = C.CDLL(LIB)
    u32, i32, f32, vp = C.c_uint32, C.c_int, C.c_float, C.c_void_p
    lib.arithmetic_patterns.argtypes, lib.arithmetic_patterns.restype = [i32, vp, i32, f32, f32, i32, vp], None
    lib.arithmetic_quotients.argtypes, lib.arithmetic_quotients.restype = [i32, u32, u32], u32
    lib.arithmetic_reciprocals.argtypes, lib.arithmetic_reciprocals.restype = [u32, u32, vp, vp], i32
    return lib
