"""What the compiler gave the kernels of the built library, read from its code objects' own metadata: registers that the launch rules
count on, and no scratch memory in the kernels of the main path."""
import os
import struct
import subprocess

import pytest

from paper_2501_08192_amd import build

msgpack = pytest.importorskip("msgpack")


def _code_objects(data):
    """The gfx950 images of every offload bundle in the library."""
    at = data.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        count, = struct.unpack_from("<Q", data, at + 24)
        p = at + 32
        for _ in range(count if count < 16 else 0):
            off, size, n = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + n]:
                yield data[at + off:at + off + size]
            p += 24 + n
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 1)


def _notes(elf):
    table, = struct.unpack_from("<Q", elf, 40)
    size, count = struct.unpack_from("<HH", elf, 58)
    for k in range(count):
        _, kind, _, _, at, length = struct.unpack_from("<IIQQQQ", elf, table + k * size)
        end = at + length if kind == 7 else 0
        while at < end:
            name, desc, tag = struct.unpack_from("<III", elf, at)
            d = at + 12 + (name + 3) // 4 * 4
            if tag == 32:
                yield elf[d:d + desc]
            at = d + (desc + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    found = {}
    for image in _code_objects(open(build.LIB if os.path.exists(build.LIB) else build.build(), "rb").read()):
        for note in _notes(image):
            for k in msgpack.unpackb(note)["amdhsa.kernels"]:
                found[k[".name"]] = k
    names = list(found)
    text = subprocess.run(["c++filt"], input="\n".join(names), text=True, capture_output=True, check=True).stdout.split("\n")
    return {t.split("(")[0].removeprefix("void ").removeprefix("psv::"): found[n] for t, n in zip(text, names)}


def test_no_projection_kernel_that_nothing_launches(kernels):
    """k_gemv<batch, rows a pass, loads a row, pair, prologue, ...>: pairs are normalised (prologue 1), and two sequences have normalised
    rows of one load only."""
    for n in _group(kernels, "k_gemv"):
        batch, _, loads, pair, prologue = n[len("k_gemv<"):-1].split(", ")[:5]
        assert not (pair == "true" and prologue != "1") and not (batch == "2" and loads == "2" and prologue == "1"), n


def _group(kernels, name):
    some = {n: k for n, k in kernels.items() if n == name or n.startswith(name + "<")}
    assert some, name
    return some


@pytest.mark.parametrize("name", ["k_attn", "k_attn_q8"])
def test_two_attention_workgroups_a_compute_unit(kernels, name):
    """The split fills the chip with two workgroups of four waves a compute unit: 512 registers a lane and SIMD, 160 KiB of LDS."""
    for n, k in _group(kernels, name).items():
        assert k[".vgpr_count"] <= 256 and k[".group_segment_fixed_size"] <= 80 * 1024, n


@pytest.mark.parametrize("name", ["k_attn", "k_attn_q8", "k_attn_merge", "k_attn_prep", "k_gemm_sk", "k_gemm_sk_i8", "k_gemv", "k_resid_sum", "k_sk_reduce"])
def test_no_scratch_in_the_kernels_of_an_operator(kernels, name):
    for n, k in _group(kernels, name).items():
        assert k[".private_segment_fixed_size"] == 0 and k[".vgpr_spill_count"] == 0, n
