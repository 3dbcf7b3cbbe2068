"""The many-row product's arguments as its launcher takes them, and the tile shapes it is built for."""
import ctypes as C

from paper_2407_09722_amd import binding as mb

vp, i32, f32, size_t = C.c_void_p, C.c_int32, C.c_float, C.c_size_t
STORE, RESID, SWIGLU, QKV = range(4)
# (strips per wave, groups of 64 rows (0: one of 32), wave groups side by side)
TILES = [(A, B, 0) for A in (4, 5, 6, 7, 8) for B in range(5) if A > 4 or B < 2] + [(A, B, 1) for A in (5, 6, 7, 8) for B in (3, 4)]


class KvView(C.Structure):
    _fields_ = [("k", vp), ("v", vp), ("page_table", vp), ("len", vp)] + [(n, i32) for n in ("page_size", "max_pages", "n_pages", "n_kv_heads", "head_dim")] + \
               [("layer_stride", C.c_int64)]


class GemmArgs(C.Structure):
    _fields_ = [("W", vp), ("X", vp)] + [(n, i32) for n in ("R", "N", "K", "ncg", "row0")] + [("ssq", vp), ("NP", i32), ("eps", f32), ("Y", vp), ("ldy", i32),
               ("accumulate", i32), ("lse_part", vp), ("h", vp), ("g_next", vp), ("planes_out", vp), ("ssq_out", vp), ("act_out", vp), ("q_out", vp), ("rope", vp),
               ("slot", vp), ("kv", KvView), ("layer", i32), ("Rseq", i32), ("n_heads", i32), ("status", vp), ("part", vp), ("counters", vp),
               ("part_floats", size_t), ("counters_n", i32), ("xfrag", vp), ("xfrag_elems", size_t)]


def _call(args, epi, tile, run, stream):
    fn = mb.lib().mtad_test_gemm_tiles
    fn.argtypes, fn.restype = [vp, size_t, C.c_int, C.POINTER(C.c_int * 4), C.c_int, vp], C.c_int
    t = (C.c_int * 4)(*tile)
    return fn(C.byref(args), C.sizeof(args), epi, C.byref(t), run, stream), tuple(t)


def launch(args, epi, tile, ranges, stream=None, lds=1):
    """The product on the given tile (lds: on a device with that many bytes per compute unit); 0, or the entry point's error."""
    return _call(args, epi, (*tile, ranges), lds, stream)[0]


def planned(R, N, K, epi=STORE, part_floats=256 ** 3):
    """(strips, row groups, side by side, ranges) the launcher would take, for 256 compute units where there is no device."""
    a = GemmArgs(R=R, N=N, K=K, ncg=(R + 7) // 8, ldy=N, part=vp(256) if part_floats else None, part_floats=part_floats)
    status, t = _call(a, epi, (0, 0, 0, 0), 0, None)
    assert status == 0
    return t


def many_rows(R, N, K, part_floats=256 ** 3):
    """Whether a product with activations in fragment order goes to the many-row kernel."""
    fn = mb.lib().mtad_test_gemm_many_rows
    fn.argtypes, fn.restype = [vp, size_t], C.c_int
    a = GemmArgs(R=R, N=N, K=K, ncg=(R + 7) // 8, part=vp(256) if part_floats else None, part_floats=part_floats)
    return bool(fn(C.byref(a), C.sizeof(a)))
