"""What the compiler made of the kernels that carry the large products: none of those that whole-step calls of the 1.3B shapes
launch keeps a value in scratch memory (a spilled register of a kernel with one wavefront per SIMD is a wait that nothing hides).
Read from the metadata that the build wrote into the library."""
import os
import struct

import pytest

from launch_trace import trace
from paper_2602_22592_amd import binding as pq

msgpack = pytest.importorskip("msgpack")


def kernel_metadata(path):
    """{mangled kernel name: its metadata} of every gfx950 code object in the library."""
    data = open(path, "rb").read()
    out = {}
    at = data.find(b"\x7fELF", 1)
    while at >= 0:
        if struct.unpack_from("<H", data, at + 18)[0] == 224:          # EM_AMDGPU
            shoff, = struct.unpack_from("<Q", data, at + 40)
            shentsize, shnum = struct.unpack_from("<HH", data, at + 58)
            for i in range(shnum):
                _, kind, _, _, off, size = struct.unpack_from("<IIQQQQ", data, at + shoff + i * shentsize)
                if kind == 7:                                          # SHT_NOTE
                    _note(data[at + off:at + off + size], out)
        at = data.find(b"\x7fELF", at + 1)
    return out


def _note(blob, out):
    pos = 0
    while pos + 12 <= len(blob):
        namesz, descsz, kind = struct.unpack_from("<III", blob, pos)
        desc = pos + 12 + (namesz + 3) // 4 * 4
        if kind == 32:                                                 # NT_AMDGPU_METADATA
            for k in msgpack.unpackb(blob[desc:desc + descsz])["amdhsa.kernels"]:
                out[k[".name"]] = k
        pos = desc + (descsz + 3) // 4 * 4


@pytest.fixture(scope="module")
def metadata():
    if not os.path.exists(pq.LIB_PATH):
        from paper_2602_22592_amd.build import build
        build(verbose=False)
    return kernel_metadata(pq.LIB_PATH)


@pytest.mark.parametrize("call", [dict(op="linear", tokens=8192, d_in=2048, d_out=2048, hp_rank=128),
                                  dict(op="linear", tokens=16384, d_in=2048, d_out=2048),
                                  dict(op="linear", tokens=8192, d_in=2048, d_out=2048, hp_rank=128, hp_kind=1),
                                  dict(op="ffn", tokens=8192, d_model=2048, d_ffn=5504, n_experts=8, hp_rank=32),
                                  dict(op="prefill", tokens=4096, d_in=4096, d_out=11008, hp_rank=128)])
def test_whole_step_products_keep_nothing_in_scratch(metadata, call):
    result = trace([call])[0]
    assert result["rc"] == 0, result["error"]
    names = {n for n in result["symbols"] if "gemm" in n}
    assert names, result["launches"]
    spilled = {n: metadata[n][".private_segment_fixed_size"] for n in names if metadata[n][".private_segment_fixed_size"]}
    assert not spilled


@pytest.mark.parametrize("call,kernels", [(dict(op="linear", tokens=2048, d_in=2048, d_out=2048, hp_rank=128, io_dtype=0), {"fixed_gemm_kernel"}),
                                          (dict(op="linear", tokens=1531, d_in=1056, d_out=3104, hp_rank=24, n_experts=4, top_k=2), {"tile_set_kernel"}),
                                          (dict(op="linear", tokens=393, d_in=5216, d_out=800), {"tile_set_kernel"}),
                                          (dict(op="ffn", tokens=304, d_model=2368, d_ffn=68, n_experts=8, hp_rank=128, top_k=2), {"tile_set_kernel"}),
                                          (dict(op="linear", tokens=600, d_in=1056, d_out=1088, hp_rank=264), {"tile64_grads_kernel"}),
                                          (dict(op="linear", tokens=130, d_in=768, d_out=800, hp_rank=40), {"tile64_grads_kernel"}),
                                          (dict(op="linear", tokens=1779, d_in=2208, d_out=800, hp_rank=64), {"tile64_grads_kernel"})])
def test_digit_products_and_shared_launches_keep_nothing_in_scratch(metadata, call, kernels):
    """... the digit products with 224 accumulators and two sets of operands in 512 registers above all."""
    result = trace([call])[0]
    assert result["rc"] == 0, result["error"]
    for kernel in kernels:
        names = {n for n in result["symbols"] if kernel in n}
        assert names, result["launches"]
        for n in names:
            m = metadata[n]
            assert (m[".private_segment_fixed_size"], m[".vgpr_spill_count"]) == (0, 0), n
