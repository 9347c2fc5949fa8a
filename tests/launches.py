"""What libqg would launch, without a GPU: the library on tests/hip_stub.c in a process of its own."""
import ctypes
import json
import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


class CodesArgs(ctypes.Structure):
    """Arguments of the raw-code product kernel (QgCodesArgs)."""
    _fields_ = [(n, ctypes.c_void_p) for n in ("codes", "scales", "zeros", "Xop", "Y", "partial", "arrived")] + \
        [(n, ctypes.c_int32) for n in ("M", "N", "tiles", "tile_codes", "tile_scales", "tile_zeros", "steps_padded",
                                       "group_magic", "zshift", "units", "ranges", "quota", "total", "fused", "kw", "zblocks", "per_die",
                                       "self", "K")] + [("X", ctypes.c_void_p)]


class RowsI8Args(ctypes.Structure):
    """Arguments of the product on int8 digits (QgRowsI8Args)."""
    _fields_ = [(n, ctypes.c_void_p) for n in ("codes", "scales", "zeros", "Aop", "inverse", "out")] + \
        [(n, ctypes.c_int32) for n in ("M", "N", "tiles", "ngroups", "zwords", "units", "units_padded", "per_wave")]


class GemvProblem(ctypes.Structure):
    """One problem of a GEMV launch, up to the meeting slots and the cuts of K."""
    _fields_ = [(n, ctypes.c_void_p) for n in ("codes", "scales", "zeros", "x", "y", "slots")] + \
        [(n, ctypes.c_int32) for n in ("N", "K", "tiles", "steps", "ngroups", "zwords", "group", "chunks", "chunk_shift", "team", "inv_team",
                                       "team_full", "tiles_per_block", "steps_per_wave")] + [("rest", ctypes.c_ubyte * 152)]


class GemvArgs(ctypes.Structure):
    _fields_ = [("count", ctypes.c_int32), ("block_begin", ctypes.c_int32 * 31), ("p", GemvProblem * 16)]


WORKSPACE = 1 << 32


class GemvDesc(ctypes.Structure):
    """qg_gemv_desc"""
    _fields_ = [("packed", ctypes.c_void_p), ("N", ctypes.c_int64), ("K", ctypes.c_int64), ("bits", ctypes.c_int32), ("group", ctypes.c_int32),
                ("x", ctypes.c_void_p), ("y", ctypes.c_void_p)]


SLOTS_PER_TILE = 33 * 64 * 4           # bytes of meeting slots per tile of 64 outputs


def _run(stub_path, lib_path, calls):
    stub = ctypes.CDLL(stub_path, mode=ctypes.RTLD_GLOBAL)
    L = ctypes.CDLL(lib_path)
    stub.stub_name.restype = ctypes.c_char_p
    stub.stub_args.restype = ctypes.c_void_p
    i64, i32, vp = ctypes.c_int64, ctypes.c_int, ctypes.c_void_p
    L.qg_workspace_bytes.restype = ctypes.c_size_t
    L.qg_workspace_bytes.argtypes = [i64, i64, i32, i32, i32]
    L.qg_gemm_autotune.argtypes = [ctypes.POINTER(vp), i32, i64, i64, i32, i32, vp, i32, vp, vp, ctypes.c_size_t, vp, i32, vp, vp, vp]
    L.qg_gemm_small.argtypes = [vp, i64, i64, i32, i32, vp, i32, vp, vp, ctypes.c_size_t, vp]
    L.qg_gemv_grouped.argtypes = [vp, i32, vp, ctypes.c_size_t, vp]
    out = []
    for c in calls:
        stub.stub_clear()
        stub.stub_device(c.get("device", 0))
        if "grouped" in c:
            d = (GemvDesc * len(c["grouped"]))(*[GemvDesc(1 << 20, N, K, bits, group, 1 << 20, 1 << 20) for N, K, bits, group in c["grouped"]])
            status = L.qg_gemv_grouped(d, len(d), WORKSPACE, 1 << 40, None)
            problems = [p for i in range(stub.stub_launches()) for a in [GemvArgs.from_address(stub.stub_args(i))] for p in a.p[:a.count]]
            out.append({"status": status, "cuts": [(p.N, p.K, p.team, p.chunks, p.steps_per_wave) for p in problems]})
            continue
        N, K, bits, group, M = c["problem"]
        assert L.qg_set_gemm_tuning(c.get("splits", 0), c.get("shape", 0)) == 0
        size = c.get("size") or L.qg_workspace_bytes(N, K, bits, group, M)
        if c.get("search"):
            blobs, us, timed = (vp * 1)(1 << 20), (ctypes.c_float * 120)(), (ctypes.c_int * 2)()
            status = L.qg_gemm_autotune(blobs, 1, N, K, bits, group, 1 << 20, M, 1 << 20, 1 << 20, size, None, 1, None, None, None)
            L.qg_gemm_autotune_report(us, 120, timed, None)
            L.qg_clear_tuning()
            out.append({"status": status, "us": list(us)})
            continue
        status = L.qg_gemm_small(1 << 20, N, K, bits, group, 1 << 20, M, 1 << 20, WORKSPACE, size, None)
        kernels = []
        for i in range(stub.stub_launches()):
            shape = (ctypes.c_uint32 * 5)()
            stub.stub_shape(i, shape)
            mangled = stub.stub_name(i).decode()
            # _ZN12_GLOBAL__N_1<length><name>I...: the length says where the name ends
            length, rest = re.match(r"_ZN12_GLOBAL__N_1(\d\d?)(\D.*)", mangled).groups()
            name, tail = rest[:int(length)], rest[int(length):]
            k = {"name": name, "template": [int(v) for v in re.findall(r"L[ib](\d+)E", tail)], "grid": list(shape[:3]),
                 "block": shape[3], "lds": shape[4]}
            if name == "gemm_codes":
                a = CodesArgs.from_address(stub.stub_args(i))
                k["args"] = {f: getattr(a, f) for f, _ in CodesArgs._fields_}
            # what a launch writes into the workspace, and the meeting slots it expects empty: [from, to) in it
            if name == "gemm_rows_i8":
                a = RowsI8Args.from_address(stub.stub_args(i))
                blocks = (a.M + 7) // 8
                writes = [(a.Aop, blocks * a.units * 4096), (a.inverse, blocks * a.units * 32)]
                if shape[1] > 1:
                    writes.append((a.out, shape[1] * a.M * a.N * 4))
                k["writes"] = [(p - WORKSPACE, p - WORKSPACE + n) for p, n in writes]
            if name.startswith("gemv_"):
                a = GemvArgs.from_address(stub.stub_args(i))
                k["slots"] = [(p.slots - WORKSPACE, p.slots - WORKSPACE + p.tiles * SLOTS_PER_TILE) for p in a.p[:a.count] if p.chunks > 1]
            kernels.append(k)
        out.append({"status": status, "kernels": kernels, "limits": stub.stub_limits(), "size": size})
    return out


def launches(tmp_path, calls):
    """calls: dicts with problem = (N, K, bits, group, M) of qg_gemm_small and, optionally, splits and shape
    (qg_set_gemm_tuning), device and the workspace's size, or search = True for qg_gemm_autotune; or grouped = [(N, K, bits, group), ...] of qg_gemv_grouped, which
    returns (N, K, wavefronts of a team, cuts of K over workgroups, steps of a wavefront) per problem.  Returns per call its status and
    the kernels it launches, or the times of the search's candidates (-1: not timed)."""
    from paper_2307_03738_amd import build
    stub = os.path.join(str(tmp_path), "hip_stub.so")
    subprocess.run(["gcc", "-O1", "-w", "-shared", "-fPIC", os.path.join(HERE, "hip_stub.c"), "-o", stub], check=True)
    done = subprocess.run([sys.executable, os.path.abspath(__file__), stub, os.environ.get("QG_LIBRARY", build.OUT)],
                          input=json.dumps(calls), capture_output=True, text=True, timeout=120)
    assert done.returncode == 0, done.stderr
    return json.loads(done.stdout)


if __name__ == "__main__":
    json.dump(_run(sys.argv[1], sys.argv[2], json.load(sys.stdin)), sys.stdout)
