"""The library's host code over the device-less runtime of tests/cpu/hip_stub.c:
run as a program with that runtime preloaded, it makes the calls of a scenario
(JSON: a list of contexts, each a workspace cap and its calls) and prints each
call's status, the memory held and what the stub counted."""

import ctypes
import json
import sys

GEOM = ("L", "r_min", "r_max", "n_phi", "shift_max", "mirror", "precision", "normalize", "rescore_rows")
PREC = {"fp32": 0, "bf16": 1, "fp16": 2}
P = 4096  # any device address: nothing is read


class Geom(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in GEOM]


class Result(ctypes.Structure):
    _fields_ = [(n, ctypes.c_void_p) for n in ("ref", "shift_x", "shift_y", "psi", "mirror", "cc", "cc2", "flat_index",
                                               "psi_frac")]


class Stack(ctypes.Structure):
    _fields_ = [("refset_id", ctypes.c_int32), ("parts", ctypes.c_void_p), ("N", ctypes.c_int64),
                ("shift_max", ctypes.c_int32), ("out", Result)]


def geom(g):
    return Geom(g["L"], 1, g["r"], 256, g["T"], 1, PREC[g["prec"]], 0, 0 if g["prec"] == "fp32" else 4)


def result(cc2=False):
    return Result(P, P, P, P, P, P, P if cc2 else None, P, None)


def main(path, scenario):
    lib = ctypes.CDLL(path)
    stub = ctypes.CDLL(None)
    for n in ("held", "most_items", "launches", "bad_frees"):
        getattr(stub, "stub_" + n).restype = ctypes.c_uint64
    vp, i32, i64 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64
    lib.mra_create.argtypes = [ctypes.POINTER(vp), ctypes.c_int, vp, ctypes.c_uint64]
    lib.mra_load_refs.argtypes = [vp, i32, vp, i32, ctypes.POINTER(Geom)]
    lib.mra_align.argtypes = lib.mra_align_noalloc.argtypes = [vp, i32, vp, i64, ctypes.POINTER(Result)]
    lib.mra_update_averages.argtypes = [vp, i32, vp, i64, ctypes.POINTER(Result), vp, vp]
    lib.mra_align_batch.argtypes = [vp, ctypes.POINTER(Stack), i32]
    lib.mra_classify.argtypes = [vp, i32, ctypes.POINTER(Geom), vp, i64, vp, i32, i32, ctypes.c_double,
                                 ctypes.POINTER(Result), vp, ctypes.POINTER(i32), ctypes.POINTER(i64)]
    lib.mra_last_error.argtypes, lib.mra_last_error.restype = [vp], ctypes.c_char_p
    lib.mra_destroy.argtypes = [vp]
    out = []
    for c in scenario:
        stub.stub_reset()
        h = vp()
        assert lib.mra_create(ctypes.byref(h), 0, None, c["cap"]) == 0
        codes, errors = [], []
        for call in c["calls"]:
            kind, a = call[0], call[1]
            if kind == "load":
                rc = lib.mra_load_refs(h, a.get("id", 0), P, a["K"], ctypes.byref(geom(a)))
            elif kind in ("align", "align_noalloc"):
                rc = getattr(lib, "mra_" + kind)(h, a.get("id", 0), P, a["N"], ctypes.byref(result(a.get("cc2"))))
            elif kind == "averages":
                rc = lib.mra_update_averages(h, a.get("id", 0), P, a["N"], ctypes.byref(result()), P, P)
            elif kind == "classify":
                n, ch = i32(), (i64 * 8)()
                rc = lib.mra_classify(h, 0, ctypes.byref(geom(a)), P, a["N"], P, a["K"], 3, 0.0,
                                      ctypes.byref(result()), P, ctypes.byref(n), ch)
            elif kind == "batch":
                st = (Stack * len(a["stacks"]))(*[Stack(i, P, N, -1, result()) for i, N in a["stacks"]])
                rc = lib.mra_align_batch(h, st, len(a["stacks"]))
            elif kind == "fail_sync":
                stub.stub_fail_sync(a["n"])
                rc = 0
            codes.append(rc)
            errors.append(lib.mra_last_error(h).decode() if rc else "")
        held = stub.stub_held()
        lib.mra_destroy(h)
        out.append(dict(codes=codes, errors=errors, held=held, left=stub.stub_held(), most_items=stub.stub_most_items(),
                        launches=stub.stub_launches(), bad_frees=stub.stub_bad_frees()))
    print(json.dumps(out))


if __name__ == "__main__":
    main(sys.argv[1], json.load(sys.stdin))
