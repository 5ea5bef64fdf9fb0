"""Runs calls of librapidgnn.so over tests/recording_runtime.cpp, in a process of its own, and returns what the program printed.
The program sees `lib`, `rt` (the recording runtime), the helpers below, and addresses that nothing ever reads."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.environ.get("RG_HOST_CALLS_LIB", os.path.join(os.path.dirname(HERE), "paper_2505_10806_amd", "librapidgnn.so"))

_PRELUDE = r'''
import ctypes, sys
from ctypes import POINTER, Structure, byref, c_char_p, c_int, c_int32 as i32, c_int64 as i64, c_size_t, c_uint32 as u32, c_uint64 as u64, c_void_p as p
rt = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)           # found before the real runtime
lib = ctypes.CDLL(sys.argv[2])
rt.recorded.restype, rt.memory_held.restype = c_char_p, c_size_t
rt.limit_memory.argtypes, rt.begin_capture.argtypes = [c_size_t], [p]
lib.rg_last_error.restype, lib.rg_last_error.argtypes = c_char_p, [p]
OK, OOM, ASCENDING, FIRST_SEEN = 0, 3, 0, 1

class Csr(Structure):
    _fields_ = [("num_nodes", i64), ("num_edges", i64), ("row_ptr", p), ("bits", i32), ("col_idx", p)]
class Blocks(Structure):
    _fields_ = [("nodes", p), ("nodes_cap", i64), ("tier_off", p), ("indptr", POINTER(p)), ("indptr_cap", POINTER(i64)),
                ("nbr", POINTER(p)), ("nbr_local", POINTER(p)), ("nbr_cap", POINTER(i64)), ("num_edges", p)]
class Cache(Structure):
    _fields_ = [("cache_ids", p), ("cache_rows", p), ("capacity_rows", i64), ("row_stride", i64), ("loc", p), ("num_cached", p),
                ("filled", p), ("mirror_rows", i64), ("home", p)]

_next = [0x500000000000]
def address(bytes=1 << 36):
    _next[0] += (bytes + 4095) // 4096 * 4096
    return _next[0] - (bytes + 4095) // 4096 * 4096

def context():
    c = p()
    assert lib.rg_create(0, byref(c)) == OK
    return c

def log(prefix=""):
    lines = [x for x in rt.recorded().decode().splitlines() if x.startswith(prefix)]
    rt.forget()
    return lines

def kernels():
    return [x.split()[1] for x in log("launch")]

def sample(c, n, nnz, seeds, fanouts, order=ASCENDING, stream=0, local=True):
    """rg_sample_blocks_group of len(seeds) batches on a graph of n nodes and nnz edges."""
    H, g = len(fanouts), len(seeds)
    csr, outs, keep = Csr(n, nnz, address(), 64, address()), (Blocks * g)(), []
    fo = (i32 * H)(*fanouts)
    for j, k in enumerate(seeds):
        fub, eub = (i64 * (H + 1))(), (i64 * H)()
        assert lib.rg_blocks_bounds(i64(n), i64(nnz), i64(k), fo, H, fub, eub) == OK
        arrays = [(p * H)(*[address() for _ in range(H)]) for _ in range(3)]
        caps = (i64 * H)(*[fub[h] + 1 for h in range(H)]), (i64 * H)(*eub)
        keep += arrays + list(caps)
        outs[j] = Blocks(address(), fub[H], address(), arrays[0], caps[0], arrays[1], arrays[2] if local else None, caps[1], address())
    return lib.rg_sample_blocks_group(c, byref(csr), g, (p * g)(*[address() for _ in seeds]), (i32 * g)(*seeds), fo, H, u64(7), u32(1),
                                      order, outs, p(stream))

def gather(c, rows, dim, hit=0, miss=None, static=False):
    cache = Cache(address(), address(), 1000, dim, address(), address(), address(), 0, None)
    call = lib.rg_gather_features_static if static else lib.rg_gather_features
    return call(c, p(address()), i64(rows), None, byref(cache), p(address()), i64(dim), p(address()), i64(dim), i32(dim), p(address()),
                i64(dim), p(address()), p(hit), p(miss))

def histogram(c, n, batches, hops, first=True, stream=0, stride=1 << 24, seeds=100):
    return lib.rg_access_histogram_epoch(c, p(address()), i64(stride), p(address()), i32(batches), i32(hops), i32(seeds), p(address()),
                                         p(address()) if first else None, i64(n), p(stream))
'''

_runtime = None


def run(program):
    global _runtime
    if _runtime is None:
        import atexit
        import shutil
        import tempfile
        folder = tempfile.mkdtemp()
        atexit.register(shutil.rmtree, folder, ignore_errors=True)
        _runtime = os.path.join(folder, "recording_runtime.so")
        subprocess.run(["g++", "-O1", "-std=c++17", "-Wno-format-security", "-shared", "-fPIC", "-o", _runtime, os.path.join(HERE, "recording_runtime.cpp")],
                       check=True)
    r = subprocess.run([sys.executable, "-c", _PRELUDE + program, _runtime, LIB], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout
