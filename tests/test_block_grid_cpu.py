"""Which grids the block kernel takes, asked of the library's own rule (host code:
runs without a GPU)."""
import ctypes as C
import os

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2009_04619_amd", "libwave.so")
pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libwave.so not built")


class SweepArgs(C.Structure):
    """wave::SweepArgs of wave_internal.h."""
    _fields_ = [("cur", C.c_void_p), ("nxt", C.c_void_p), ("vp", C.c_void_p), ("eta", C.c_void_p),
                ("etab", C.c_void_p), ("etq", C.c_void_p), ("dt", C.c_double), ("phi", C.c_void_p),
                ("nx", C.c_int32), ("ny", C.c_int32), ("nz", C.c_int32), ("w", C.c_int32),
                ("pitch", C.c_int32), ("plane", C.c_int64), ("c", C.c_float * 13), ("ce", C.c_float),
                ("q", C.c_float * 3), ("damping", C.c_int32), ("step", C.c_int32)]


F32, BF16, F16, BF16SR = 0, 1, 2, 3


@pytest.fixture(scope="module")
def lib():
    lib = C.CDLL(LIB)
    lib.supported = lib._ZN4wave22block_config_supportedEiiRKNS_9SweepArgsEi
    lib.supported.restype = C.c_bool
    lib.default = lib._ZN4wave13block_defaultERKNS_9SweepArgsEiPiS3_
    lib.default.restype = None
    return lib


def args(nx, ny, nz, w=0):
    pitch = (nx + 8 + 63) // 64 * 64
    return SweepArgs(nx=nx, ny=ny, nz=nz, w=w, pitch=pitch, plane=(ny + 8) * pitch, damping=int(w > 0))


def default(lib, a, storage):
    ty, zc = C.c_int(-1), C.c_int(-1)
    lib.default(C.byref(a), storage, C.byref(ty), C.byref(zc))
    return ty.value, zc.value


def threads(nx, ny, nz, tw, ty, zc, per_block):
    up = lambda a, b: -(-a // b)
    return up(nx, tw) * up(ny, ty) * up(nz, zc) * per_block


@pytest.mark.parametrize("nx,ny,nz", [(65, 32768, 32768), (100, 32768, 32768), (1, 32768, 32768), (64, 32760, 16384),
                                      (120, 20000, 20000)])
def test_grids_of_more_threads_than_a_launch_holds(lib, nx, ny, nz):
    a = args(nx, ny, nz)
    tw = 32 if -(-nx // 32) in (1, 3, 5) else 64
    for ty, zc, n in ((4, 4, threads(nx, ny, nz, tw, 256 // tw, 4, 256)), (8, 8, threads(nx, ny, nz, 64, 8, 8, 512)),
                      (8, 4, threads(nx, ny, nz, 64, 8, 4, 256))):
        if n >= 1 << 32:
            assert not lib.supported(ty, zc, C.byref(a), BF16), (ty, zc)
        elif n < 1 << 31:
            assert lib.supported(ty, zc, C.byref(a), BF16), (ty, zc)
    for storage in (F32, BF16, F16):
        ty, zc = default(lib, a, storage)
        assert ty == 0 or threads(nx, ny, nz, 64, ty, zc, 64 * ty) < 1 << 32, storage


@pytest.mark.parametrize("shape,storage,want", [
    ((64, 64, 64, 16), F32, (4, 4)), ((256, 256, 256, 20), F32, (4, 4)), ((288, 288, 288, 20), F32, (0, 0)),
    ((256, 256, 256, 20), BF16, (8, 4)), ((64, 64, 64, 16), F16, (4, 4)), ((256, 240, 256, 20), BF16SR, (4, 4)),
    ((512, 512, 512, 20), BF16, (0, 0)), ((512, 512, 512, 0), F32, (8, 8)), ((512, 512, 512, 0), BF16SR, (0, 0)),
    ((2529, 1756, 9, 0), F32, (0, 0)), ((2529, 1756, 13, 0), F32, (8, 8)), ((1840, 1278, 17, 0), F32, (0, 0)),
    ((990, 688, 33, 0), F32, (8, 8)), ((1321, 917, 33, 0), F32, (0, 0)), ((1185, 823, 41, 0), F32, (8, 8)),
    ((3098, 2151, 9, 0), BF16, (0, 0)), ((2254, 1565, 17, 0), BF16, (8, 8)), ((5692, 3952, 1, 0), F32, (8, 8)),
    ((7589, 5270, 1, 0), F32, (0, 0))])      # 16 planes of it exceed the index window
def test_default_block(lib, shape, storage, want):
    assert default(lib, args(*shape), storage) == want
