"""Registers of the built kernels, from the metadata the compiler leaves in libfvan.so: the number of waves a SIMD
holds follows from them (512 / VGPRs rounded up to 8), and a kernel that needs four loses a quarter of its loads in
flight to a single register too many."""
import struct

import msgpack
import pytest

import paper_2606_22984_amd as fv


def _code_objects(blob):
    """The gfx950 ELF images of the offload bundles in a shared library."""
    at = blob.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        count, = struct.unpack_from("<Q", blob, at + 24)
        entry = at + 32
        for _ in range(count):
            offset, size, name = struct.unpack_from("<QQQ", blob, entry)
            triple = blob[entry + 24:entry + 24 + name]
            entry += 24 + name
            if b"gfx950" in triple and size:
                yield blob[at + offset:at + offset + size]
        at = blob.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)


def _kernels(elf):
    """The kernels of a code object: its AMDGPU metadata note (type 32) is a msgpack map."""
    start, = struct.unpack_from("<Q", elf, 40)
    size, count = struct.unpack_from("<HH", elf, 58)
    for k in range(count):
        kind, = struct.unpack_from("<I", elf, start + k * size + 4)
        at, length = struct.unpack_from("<QQ", elf, start + k * size + 24)
        end = at + length if kind == 7 else at
        while at < end:
            name, desc, note = struct.unpack_from("<III", elf, at)
            body = at + 12 + (name + 3) // 4 * 4
            if note == 32:
                yield from msgpack.unpackb(elf[body:body + desc])["amdhsa.kernels"]
            at = body + (desc + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    fv.lib()
    with open(fv.LIB_PATH, "rb") as f:
        blob = f.read()
    return {k[".name"]: k for elf in _code_objects(blob) for k in _kernels(elf)}


def _template(name, *args):
    """Start of the mangled name of fvan::name<args...>."""
    return f"_ZN4fvan{len(name)}{name}I" + "".join(f"Li{a}E" for a in args) + "E"


@pytest.mark.parametrize("name,args,waves", [
    # QKV projection of many rows, d = 64: four workgroups of four waves a compute unit
    ("gemm_rows_staged_kernel", (0, 64, 192, 0, 2), 4),
    ("gemm_rows_staged_kernel", (2, 64, 192, 0, 2), 4),
    # feed-forward backward of many rows, FP32: two workgroups of eight waves
    ("ffn_bwd_fused_kernel", (0, 32, 8), 4),
    ("ffn_bwd_fused_kernel", (0, 64, 8), 4),
])
def test_waves_per_simd(kernels, name, args, waves):
    found = [k for n, k in kernels.items() if n.startswith(_template(name, *args))]
    assert len(found) == 1
    vgprs = found[0][".vgpr_count"]
    assert 512 // ((vgprs + 7) // 8 * 8) >= waves, f"{vgprs} VGPRs"
    assert found[0][".vgpr_spill_count"] == 0


@pytest.mark.parametrize("name", ["colsum_slices_kernel", "colsum_final_kernel"])
def test_column_sums_fit_beside_the_weight_gradients(kernels, name):
    """The LayerNorm column sums run on the caller's stream while the side stream fills the chip with the W2 gradient
    (two 8-wave workgroups a compute unit): they need no more registers than these leave, or wait for one to end."""
    wgrad, = (k for n, k in kernels.items() if n.startswith(_template("wgrad_kernel", 2, 128, 176)))
    kernel, = (k for n, k in kernels.items() if n.startswith(f"_ZN4fvan{len(name)}{name}E"))
    rounded = [(k[".vgpr_count"] + 7) // 8 * 8 for k in (wgrad, kernel)]
    assert rounded[1] <= 512 - 4 * rounded[0]
