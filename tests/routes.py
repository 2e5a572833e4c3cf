"""The library's own choice between its routes, asked on the host: its C++ functions by their mangled names."""
import ctypes as C

import paper_2511_13732_amd as pcg
from paper_2511_13732_amd.binding import PreparedInfo, _GroupsStruct


class CsrShape(C.Structure):
    _fields_ = [(n, C.c_int32) for n in ("width", "nchunks", "chunk_groups", "ntiles", "tile_len")]


def _function(name, result, *arguments):
    f = pcg.lib()[name]
    f.restype, f.argtypes = result, list(arguments)
    return f


def csr_shape(V, G, nnz, rows, max_chunks):
    shape = CsrShape()            # larger than two registers: returned where the hidden first argument points
    _function("_ZN3pcg9csr_shapeEiilll", None, C.c_void_p, C.c_int32, C.c_int32, C.c_int64, C.c_int64, C.c_int64)(
        C.addressof(shape), V, G, nnz, rows, max_chunks)
    return shape


def _groups(V, G, nnz, weighted, info=None):
    some = 4096                   # an address: nothing is read through it
    return _GroupsStruct(V, G, nnz, some, some, some, some if info else None, C.pointer(info) if info else None, None, None,
                         some if weighted else None, None)


def _csr_is_faster(V, G, nnz, weighted, shape):
    f = _function("_ZN3pcg13csr_is_fasterERK10pcg_groupsRKNS_8CsrShapeE", C.c_bool, C.c_void_p, C.c_void_p)
    g = _groups(V, G, nnz, weighted)
    return f(C.addressof(g), C.addressof(shape))


def rows_from_csr(V, G, nnz, weighted, rows):
    """Whether pcg_group_probs gathers so many rows of a prepared membership from the CSR."""
    return _csr_is_faster(V, G, nnz, weighted, csr_shape(V, G, nnz, rows, 256))


def step_from_csr(V, G, nnz, weighted, B, K):
    """Whether the four launches of pcg_verify do."""
    room = max((G + 4095) // 4096, (2 * K + 1) * ((V + 2047) // 2048) * 2)
    return _csr_is_faster(V, G, nnz, weighted, csr_shape(V, G, nnz, B, room))


def step_launches(V, G, nnz, weighted, B, K, nchunks, slots):
    """Launches of a pcg_verify step on a prepared membership of one tile, whose layout has so many slots."""
    f = _function("_ZN3pcg10step_shapeERK10pcg_groupsii", C.c_int, C.c_void_p, C.c_int32, C.c_int32)
    info = PreparedInfo(V=V, G=G, ntiles=1, tile_len=V, nchunks=nchunks, off_data=0, off_weights=2 * slots if weighted else 0,
                        bytes=(6 if weighted else 2) * slots)
    g = _groups(V, G, nnz, weighted, info)
    return {0: 1, 1: 2, 2: 4}[f(C.addressof(g), B, K)]


def csr_step_launches(V, G, nnz, weighted, B, K):
    """Launches of a pcg_verify step from the CSR."""
    f = _function("_ZN3pcg10step_shapeERK10pcg_groupsii", C.c_int, C.c_void_p, C.c_int32, C.c_int32)
    g = _groups(V, G, nnz, weighted)
    return {0: 1, 1: 2, 2: 4}[f(C.addressof(g), B, K)]


class GatherMap(C.Structure):
    _fields_ = [("row_shift", C.c_int32), ("chunks_each", C.c_int32)]


def gather_map(nrows, nchunks, row_bytes, chunk_bytes, csr, weighted):
    return _function("_ZN3pcg10gather_mapEiillbb", GatherMap, C.c_int32, C.c_int32, C.c_int64, C.c_int64, C.c_bool, C.c_bool)(
        nrows, nchunks, row_bytes, chunk_bytes, csr, weighted)
