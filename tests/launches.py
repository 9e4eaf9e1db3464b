"""Which kernels a call launches, without a GPU.  ``run(steps)`` makes the calls in a process of its own, in which
hip_recorder.cpp stands in for the HIP runtime (256 compute units, one block of a resident kernel on each); nothing runs.

A step is a list: an operation and its keywords.  What comes back for each step is its status and its launches
(kernel, blocks, threads, wait limit in 100 MHz ticks of those that wait for other blocks), or the value asked for."""
import ctypes
import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
PKG = os.path.join(ROOT, "paper_2502_01068_amd")


def run(steps, tmp_path):
    if not os.path.exists(os.path.join(PKG, "libfastkv_select.so")):
        from paper_2502_01068_amd import build
        build.build()
    recorder = os.path.join(str(tmp_path), "hip_recorder.so")
    if not os.path.exists(recorder):
        subprocess.run([os.environ.get("CXX", "g++"), "-O1", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wno-attributes", "-D__HIP_PLATFORM_AMD__=1",
                        "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(PKG, "csrc"), "-isystem", "/opt/rocm/include",
                        os.path.join(HERE, "hip_recorder.cpp"), "-o", recorder], check=True)
    out = subprocess.run([sys.executable, os.path.abspath(__file__), recorder], input=json.dumps(steps), check=True, stdout=subprocess.PIPE, text=True)
    return json.loads(out.stdout)


def kernels(result):
    """The kernels of one step, without namespaces and argument types."""
    return [l["kernel"].replace("void ", "").replace("fkv::", "") for l in result["launches"]]


class _Shape(ctypes.Structure):
    _fields_ = [("n_seq", ctypes.c_int32), ("cu_seqlens", ctypes.POINTER(ctypes.c_int32))] + [
        (n, ctypes.c_int32) for n in ("L", "n_q_heads", "n_kv_heads", "head_dim", "window", "pool_kernel", "pool_mode")] + [
        ("softmax_scale", ctypes.c_float), ("causal", ctypes.c_int32)]


def _i32(values):
    return (ctypes.c_int32 * len(values))(*values)


class _Calls:
    """Device pointers are made up: the library looks at their alignment only."""

    def __init__(self, lib):
        self.lib, self.ctx, self.ptr = lib, [], ctypes.c_void_p(1 << 20)

    def create(self, tokens=140000, seqs=64):
        handle = ctypes.c_void_p()
        rc = self.lib.fkv_create(ctypes.byref(handle), 0, ctypes.c_int64(tokens), seqs)
        self.ctx.append(handle)
        return rc

    def destroy(self):
        return self.lib.fkv_destroy(self.ctx.pop())

    def _shape(self, lengths, hq=32, hkv=8, window=8, pool_kernel=7, **_):
        cu = [0]
        for n in lengths:
            cu.append(cu[-1] + n)
        keep = _i32(cu)
        return ctypes.byref(_Shape(len(lengths), keep, 0, hq, hkv, 128, window, pool_kernel, 0, 0.0, 1)), keep

    def set(self, what, value):
        return getattr(self.lib, "fkv_" + what)(self.ctx[0], ctypes.c_int64(value) if what == "set_wait_limit" else value)

    def clear_error(self):
        return self.lib.fkv_clear_error(self.ctx[0])

    def query_error(self):
        flag = ctypes.c_int32(-1)
        assert self.lib.fkv_query_error(self.ctx[0], ctypes.byref(flag)) == 0
        return flag.value

    def workspace_bytes(self, tokens, seqs):
        self.lib.fkv_workspace_bytes.restype = ctypes.c_size_t
        return self.lib.fkv_workspace_bytes(ctypes.c_int64(tokens), seqs)

    def score(self, lengths, mean=True, heads=False, **kw):
        s, _keep = self._shape(lengths, **kw)
        p = self.ptr
        if heads:
            return self.lib.fkv_score_heads(self.ctx[0], s, p, p, p, None)
        return self.lib.fkv_score_window(self.ctx[0], s, p, p, p, p if mean else None, None)

    def window_output(self, lengths, scores=True, **kw):
        s, _keep = self._shape(lengths, **kw)
        p = self.ptr
        if scores:
            return self.lib.fkv_score_window_output(self.ctx[0], s, p, p, p, p, p, p, None)
        return self.lib.fkv_window_output(self.ctx[0], s, p, p, p, p, None)

    def select(self, lengths, rows, counts, **kw):
        s, _keep = self._shape(lengths, **kw)
        return self.lib.fkv_select_topk(self.ctx[0], s, self.ptr, rows, _i32(counts), self.ptr, None)

    def compress(self, lengths, budgets, k_tsp=None, hidden=4096, paged=False, **kw):
        s, _keep = self._shape(lengths, **kw)
        p = self.ptr
        if paged:
            return self.lib.fkv_compress_kv_paged(self.ctx[0], s, p, p, p, _i32(budgets), p, max(budgets), 4, ctypes.c_int64(sum(budgets)), p, p, p, None)
        tsp = k_tsp is not None
        return self.lib.fkv_compress_kv(self.ctx[0], s, p, p, p, _i32(budgets), p, p, p, p if tsp else None, ctypes.c_size_t(2 * hidden),
                                        _i32(k_tsp) if tsp else None, p if tsp else None, p if tsp else None, None)


def _main():
    rec = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)  # ahead of the library, whose runtime calls find it first
    rec.recorder_kernel.restype = ctypes.c_char_p
    rec.recorder_wait_ticks.restype = ctypes.c_ulonglong
    calls = _Calls(ctypes.CDLL(os.path.join(PKG, "libfastkv_select.so")))
    results = []
    for op, kw in json.load(sys.stdin):
        refuse = kw.pop("refuse_launch", -1)
        rec.recorder_reset(refuse)
        value = getattr(calls, op)(**kw)
        results.append({"value": value, "launches": [
            {"kernel": rec.recorder_kernel(i).decode(), "blocks": rec.recorder_blocks(i), "threads": rec.recorder_threads(i),
             "wait_ticks": rec.recorder_wait_ticks(i)} for i in range(rec.recorder_launches())]})
    json.dump(results, sys.stdout)


if __name__ == "__main__":
    _main()
