"""Runs calls of libtensair's host side against stand-ins of the HIP runtime (hip_trace.c) and prints what each of them
enqueued, as JSON.  A process of its own, without torch, whose own HIP runtime would come first:

    python launch_trace.py LIBRARY STAND_INS < calls.json

calls.json: {"model": {...fields of tensair_config...}, "tokens": T, "counts": unigram counts (64 words once if absent),
"calls": [[name, ...], ...]} with the calls
    ["grad", begin, n, epoch, output...] (optional outputs: "negatives", "offsets_in", "offsets_out")   ["step", begin, n, epoch, peers]   ["step_packed", begin, n, epoch, peers, rows_out of each]   ["prefetch", begin, n, epoch]   ["rebind", worker]
    ["apply", rows_in, rows_out, peers]   ["capture", 0 | 1]   ["profile", level]
Every pointer is made up: nothing reads or writes them."""
import ctypes as C
import json
import sys

FIELDS = [("vocab", C.c_int64), ("dim", C.c_int32), ("row_stride", C.c_int32), ("dtype", C.c_int32), ("window", C.c_int32),
          ("negatives", C.c_int32), ("max_centers", C.c_int32), ("max_peers", C.c_int32), ("worker_id", C.c_uint32),
          ("seed", C.c_uint64), ("flags", C.c_uint32)]


class Config(C.Structure):
    _fields_ = FIELDS


class Rows(C.Structure):
    _fields_ = [("capacity", C.c_int64), ("n_rows", C.c_void_p), ("row_ids", C.c_void_p), ("row_grads", C.c_void_p)]


class Grad(C.Structure):
    _fields_ = [("in_", Rows), ("out", Rows)]


def main():
    hip = C.CDLL(sys.argv[2], mode=C.RTLD_GLOBAL)
    lib = C.CDLL(sys.argv[1])
    hip.hip_trace_take.restype = C.c_char_p
    vp, i32, i64 = C.c_void_p, C.c_int32, C.c_int64
    lib.tensair_workspace_bytes.restype = C.c_size_t
    lib.tensair_capacity_in.restype = lib.tensair_capacity_out.restype = i64
    job = json.load(sys.stdin)
    cfg = Config(**job["model"])
    need = lib.tensair_workspace_bytes(C.byref(cfg))
    assert need > 0
    at = [1 << 44]

    def pointer(n=1):
        at[0] += (1 << 36) * n
        return at[0]

    counts = (C.c_uint64 * cfg.vocab)()      # zeros, and a few words of the noise distribution
    for i, n in enumerate(job.get("counts") or [1] * min(cfg.vocab, 64)):
        counts[i] = n
    h = vp()
    workspace, stream, T = pointer(64), None, job["tokens"]
    rc = lib.tensair_model_init(C.byref(h), C.byref(cfg), vp(pointer()), vp(pointer()), 0, counts, vp(workspace),
                                C.c_size_t(need), stream)
    assert rc == 0, rc
    del counts
    hip.hip_trace_take()
    tokens = pointer()

    def grad(rows_in, rows_out):
        return Grad(Rows(rows_in, pointer(), pointer(), pointer()), Rows(rows_out, pointer(), pointer(), pointer()))

    own = grad(lib.tensair_capacity_in(C.byref(cfg), cfg.max_centers), lib.tensair_capacity_out(C.byref(cfg), cfg.max_centers))
    out = []
    for name, *a in job["calls"]:
        if name == "capture":
            hip.hip_trace_capture(a[0])
            continue
        if name == "rebind":
            rc = lib.tensair_model_rebind(h, vp(pointer()), vp(pointer()), C.c_uint32(a[0]))
        elif name == "profile":
            rc = lib.tensair_profile(h, a[0])
        elif name == "apply":
            src = (Grad * (a[2] + 1))(*[grad(a[0], a[1]) for _ in range(a[2] + 1)])
            rc = lib.tensair_dasgd_apply(h, C.byref(src[0]), C.byref(src, C.sizeof(Grad)), i32(a[2]), C.c_float(0.1), stream)
        else:
            batch = (h, vp(tokens), i64(T), i64(a[0]), i32(a[1]), C.c_uint32(a[2]))
            if name == "prefetch":
                rc = lib.tensair_prefetch(*batch, stream)
            elif name == "grad":
                dbg = [vp(pointer()) if o in a[3:] else None for o in ("negatives", "offsets_in", "offsets_out")]
                rc = lib.tensair_sgns_grad(*batch, C.byref(own), None, *dbg, stream)
            elif name == "step_packed":
                peers = (Grad * max(a[3], 1))(*[grad(own.in_.capacity, a[4]) for _ in range(a[3])])
                rc = lib.tensair_step_packed(*batch, peers, i32(a[3]), C.c_float(0.1), C.byref(own), None, None, stream)
            else:
                peers = (Grad * max(a[3], 1))(*[grad(own.in_.capacity, own.out.capacity) for _ in range(a[3])])
                rc = lib.tensair_step(*batch, peers, i32(a[3]), C.c_float(0.1), C.byref(own), None, stream)
        out.append({"call": [name] + a, "rc": rc,
                    "did": [line.split() for line in hip.hip_trace_take().decode().splitlines()]})
    print(json.dumps(out))


main()
