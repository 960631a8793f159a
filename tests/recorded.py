"""The library's host code on the recording runtime of hip_recorder.c: allocations and launches are
lines of a log.  Run as a program (torch brings the real runtime with it, so the library has to be
loaded in a process of its own): ``python recorded.py RECORDER LIBRARY`` executes the Python on its
standard input with the names of this module."""
import collections
import ctypes as C
import sys

F32, BF16, F16 = 0, 1, 2
Launch = collections.namedtuple("Launch", "kernel x y z threads lds device")


class Info(C.Structure):
    _fields_ = [("d", C.c_int64), ("k", C.c_int64)] + [(f, C.c_int32) for f in (
        "Bc Br kappa s M a b a_inv").split()] + [("key0", C.c_uint32), ("key1", C.c_uint32), ("scale", C.c_float)] + [
        (f, C.c_int32) for f in "kind variant last_variant last_mode last_hip_error".split()] + [
        ("workspace_bytes", C.c_uint64), ("last_kernel", C.c_char * 64)]


def _load(recorder, library):
    rec = C.CDLL(recorder, mode=C.RTLD_GLOBAL)
    rec.rec_log.restype = C.c_char_p
    rec.rec_live.restype = C.c_size_t
    rec.rec_budget.argtypes = [C.c_size_t]
    return rec, C.CDLL(library)


def lines(word=None):
    """The log so far, split; with `word`, the entries of that kind without it."""
    out = [ln.split() for ln in rec.rec_log().decode().splitlines()]
    return out if word is None else [ln[1:] for ln in out if ln[0] == word]


def launches():
    return [Launch(ln[0], *map(int, ln[1:])) for ln in lines("launch")]


STREAM = C.c_void_p(64)   # any handle but that of the default stream, which cannot be captured


class Sketch:
    def __init__(self, d, k, Bc=1, Br=1, kappa=1, s=1, kind=0, seed=0):
        self.h, self.d, self.k = C.c_void_p(), d, k
        self.status = lib.fs_sketch_create_kind(C.byref(self.h), kind, C.c_int64(d), C.c_int64(k), Bc, Br, kappa, s,
                                                C.c_uint64(seed))

    def apply(self, n, dtype=F32, ld=None, first=0, ldo=None, stream=None):
        esz = 4 if dtype == F32 else 2
        return lib.fs_sketch_apply_ld(self.h, C.c_void_p((1 << 44) + first * esz), C.c_int64(ld or n), C.c_int64(n),
                                      C.c_void_p(1 << 45), C.c_int64(ldo or n), dtype, stream)

    def apply_static(self, n, dtype=F32):
        return lib.fs_sketch_apply_static(self.h, C.c_void_p(1 << 44), C.c_int64(n), C.c_int64(n), C.c_void_p(1 << 45),
                                          C.c_int64(n), dtype, None)

    def apply_rows(self, n, dtype=F32, ld=None, stream=None):
        return lib.fs_sketch_apply_rows(self.h, C.c_void_p(1 << 44), C.c_int64(ld or self.d), C.c_int64(n),
                                        C.c_void_p(1 << 45), C.c_int64(self.k), dtype, stream)

    def attach(self, address, size):
        return lib.fs_sketch_set_workspace(self.h, C.c_void_p(address), C.c_size_t(size))

    def info(self):
        out = Info()
        assert lib.fs_sketch_info(self.h, C.byref(out)) == 0
        return out

    def kernel(self):
        return self.info().last_kernel.decode()

    def destroy(self):
        return lib.fs_sketch_destroy(self.h)


if __name__ == "__main__":
    rec, lib = _load(sys.argv[1], sys.argv[2])
    exec(compile(sys.stdin.read(), "<test>", "exec"), globals())
