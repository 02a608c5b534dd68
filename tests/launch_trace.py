"""The host side of library calls without a GPU: which kernels a call launches, and what it returns.

`trace(calls)` runs the calls in a child process in which the HIP runtime's symbols are those of host_launches.c (a launch
records the kernel's name and grid and does nothing).  Buffers are addresses that nobody reads; workspace and ctx sizes are
exactly what the library's own queries say.  A call is a dict: `op` (linear, linear_norm, prefill, ffn, hp_int8, decode) and the
fields of its descriptor; for the linears also `workspace_bytes`, another size than the query's.  The result is one dict per call: `rc`, `error`, `launches`, a list of [kernel, template
arguments, grid], and `symbols`, the launches' mangled kernel names."""
import ctypes as C
import json
import os
import re
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2602_22592_amd", "libpquant.so")

# template arguments of the GEMM kernels, in order (operand kinds: 0 KC16, 1 KS16, 2 KC8, 3 BITS8, 4 BITS16; -1: no second contraction)
MFMA = ("bm", "bn", "wgm", "wgn", "kb", "whole_tiles", "partial_steps", "int8", "a", "b", "a2", "b2", "paired")


def trace(calls):
    with tempfile.TemporaryDirectory() as tmp:
        shim = os.path.join(tmp, "libhost_launches.so")
        subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", shim, os.path.join(HERE, "host_launches.c")], check=True)
        res = subprocess.run([sys.executable, os.path.abspath(__file__), shim, LIB], input=json.dumps(calls), text=True, capture_output=True,
                             check=False)
    assert res.returncode == 0, res.stderr
    return json.loads(res.stdout)


def kernels(result, name):
    """The launches of kernel `name`: (template arguments, grid)."""
    return [(args, grid) for n, args, grid in result["launches"] if n == name]


def gemms(result):
    """The launches of the 256x256 kernels as dicts of their template arguments, with their grid."""
    return [dict(zip(MFMA, args), grid=grid) for args, grid in kernels(result, "mfma_gemm_kernel")]


def _demangle(mangled):
    m = re.match(r"_ZN12_GLOBAL__N_1(\d+)", mangled) or re.match(r"_Z(\d+)", mangled)
    if not m:
        return mangled, []
    end = m.end() + int(m.group(1))
    name, rest, args = mangled[m.end():end], mangled[end:], []
    if rest.startswith("I"):
        rest = rest[1:]
        while (a := re.match(r"L[ibj](n?\d+)E|([a-z])", rest)):
            args.append(int(a.group(1).replace("n", "-")) if a.group(1) else a.group(2))
            rest = rest[a.end():]
    return name, args


def _child(shim_path, lib_path):
    shim = C.CDLL(shim_path, mode=C.RTLD_GLOBAL)
    shim.trace_name.restype = C.c_char_p
    lib = C.CDLL(lib_path)
    lib.pq_last_error_string.restype = C.c_char_p
    size = C.c_size_t

    def query(name, *a):
        f = getattr(lib, name)
        f.restype = size
        return f(*a)

    class Linear(C.Structure):
        _fields_ = [(n, C.c_float if n in ("ste_tau", "alpha", "beta") else C.c_int32) for n in (
            "tokens", "d_in", "d_out", "hp_rank", "n_experts", "top_k", "io_dtype", "w_kind", "ste_mode", "ste_tau", "alpha", "beta", "hp_kind")]

    class FFN(C.Structure):
        _fields_ = [(n, C.c_float if n in ("alpha", "beta") else C.c_int32) for n in (
            "tokens", "d_model", "d_ffn", "hp_rank", "n_experts", "top_k", "io_dtype", "alpha", "beta", "hp_kind")]

    class Decode(C.Structure):
        _fields_ = [(n, C.c_float if n == "alpha" else C.c_int32) for n in (
            "batch", "d_in", "d_out", "hp_rank", "n_experts", "top_k", "n_layers", "packed_layout", "alpha")]

    def buf(i):                                       # distinct aligned addresses, far apart
        return C.c_void_p((i + 1) << 44)

    def run(c):
        c = dict(c)
        op = c.pop("op")
        if op == "hp_int8":
            T, K, N, r = (c[n] for n in ("tokens", "d_in", "d_out", "hp_rank"))
            nc, nw = query("pq_hp_int8_ctx_bytes", T, K, N, r), query("pq_hp_int8_workspace_bytes", T, K, N, r)
            return (lib.pq_hp_int8_fwd(buf(0), buf(1), buf(2), buf(3), 1, T, K, N, r, C.c_float(1.5), buf(4), 1, buf(5), size(nc), buf(6), size(nw), None)
                    or lib.pq_hp_int8_bwd(buf(4), buf(0), 1, T, K, N, r, C.c_float(1.5), buf(5), size(nc), buf(7), 1, buf(8), buf(9), buf(6), size(nw), None))
        if op == "ffn":
            d = FFN(**{**dict(n_experts=1, top_k=1, io_dtype=1, alpha=2.0, beta=0.2, hp_kind=0), **c})
            p = C.byref(d)
            nc, nw = query("pq_ffn_ctx_bytes", p), query("pq_ffn_workspace_bytes", p)
            return (lib.pq_ffn_fwd(p, *map(buf, range(9)), buf(9), size(nc), buf(10), size(nw), None)
                    or lib.pq_ffn_bwd(p, buf(11), buf(0), buf(4), buf(5), buf(6), buf(7), buf(9), size(nc), *map(buf, range(12, 21)), buf(10), size(nw), None))
        if op == "decode":
            i8 = c.pop("int8", False)
            d = Decode(**{**dict(n_layers=1, packed_layout=1, alpha=2.0), **c})
            p = C.byref(d)
            nw = query("pq_decode_workspace_bytes", p)
            if i8:
                return lib.pq_decode_gemv_int8(p, *map(buf, range(9)), None, buf(9), size(nw), None)
            return lib.pq_decode_gemv(p, *map(buf, range(7)), None, buf(9), size(nw), None)
        given = c.pop("workspace_bytes", 0)
        d = Linear(**{**dict(hp_rank=0, n_experts=1, top_k=1, io_dtype=1, w_kind=1 if op == "prefill" else 0, alpha=2.0, beta=0.2), **c})
        p = C.byref(d)
        kind = "pq_linear_norm" if op == "linear_norm" else "pq_linear"
        nc, nw = query(kind + "_ctx_bytes", p), given or query(kind + "_workspace_bytes", p)
        hp = [buf(2), buf(3), buf(4)] if d.hp_rank else [None, None, None]
        dhp = [buf(5), buf(6), buf(7)] if d.hp_rank else [None, None, None]
        if op == "prefill":
            return lib.pq_linear_fwd(p, buf(0), buf(1), buf(8), *hp, buf(9), None, size(0), buf(11), size(nw), None)
        if op == "linear_norm":
            return (lib.pq_linear_norm_fwd(p, buf(0), buf(8), C.c_float(1e-6), buf(1), *hp, buf(9), buf(10), size(nc), buf(11), size(nw), None)
                    or lib.pq_linear_norm_bwd(p, buf(12), buf(0), buf(8), buf(1), *hp, buf(10), size(nc), buf(13), buf(14), buf(15), *dhp, buf(16), buf(11),
                                              size(nw), None))
        return (lib.pq_linear_fwd(p, buf(0), buf(1), None, *hp, buf(9), buf(10), size(nc), buf(11), size(nw), None)
                or lib.pq_linear_bwd(p, buf(12), buf(0), buf(1), *hp, buf(10), size(nc), buf(13), buf(15), *dhp, buf(16), buf(11), size(nw), None))

    out = []
    for c in json.load(sys.stdin):
        shim.trace_reset()
        rc = run(c)
        symbols = [shim.trace_name(i).decode() for i in range(shim.trace_count())]
        out.append(dict(rc=rc, error=lib.pq_last_error_string().decode() if rc else "", symbols=symbols,
                        launches=[[*_demangle(s), [shim.trace_grid(i, a) for a in range(3)]] for i, s in enumerate(symbols)]))
    json.dump(out, sys.stdout)


if __name__ == "__main__":
    _child(sys.argv[1], sys.argv[2])
