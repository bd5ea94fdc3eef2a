"""Registers, scratch and code size of the built kernels, read from the library's own code objects."""
import os
import re
import struct

import msgpack
import pytest

import paper_2509_06980_amd as rl


def _code_objects(path):
    """The gfx950 ELF images in the offload bundles of a shared library."""
    with open(path, "rb") as f:
        blob = f.read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = blob.find(magic)
    while at >= 0:
        entries, p = struct.unpack_from("<Q", blob, at + 24)[0], at + 32
        for _ in range(entries):
            offset, size, n = struct.unpack_from("<QQQ", blob, p)
            if b"gfx950" in blob[p + 24:p + 24 + n]:
                yield blob[at + offset:at + offset + size]
            p += 24 + n
        at = blob.find(magic, at + 24)


def _kernels(path):
    """(name, integer template arguments) -> metadata of the kernel, with its code size as "code"; kernels with type
    arguments or none have () there."""
    found = {}
    for elf in _code_objects(path):
        at, = struct.unpack_from("<Q", elf, 40)
        size, count = struct.unpack_from("<HH", elf, 58)
        sections = [struct.unpack_from("<IIQQQQIIQQ", elf, at + i * size) for i in range(count)]
        code, kernels = {}, []
        for _, kind, _, _, offset, length, link, _, _, _ in sections:
            if kind == 2 or kind == 11:                        # symbols
                for q in range(offset, offset + length, 24):
                    name, info, _, _, _, n = struct.unpack_from("<IBBHQQ", elf, q)
                    s = sections[link][4] + name
                    if info & 15 == 2:
                        code[elf[s:elf.index(b"\0", s)].decode()] = n
            elif kind == 7:                                    # notes
                owner, n, tag = struct.unpack_from("<III", elf, offset)
                if tag == 32:
                    q = offset + 12 + -(-owner // 4) * 4
                    kernels += msgpack.unpackb(elf[q:q + n])["amdhsa.kernels"]
        for k in kernels:
            name = re.match(r"_ZN?(?:12_GLOBAL__N_1)?(\d+)(.*)", k[".name"])
            n = int(name[1])
            args = re.match(r"I((?:L[a-z]+\d+E)+)E", name[2][n:])
            key = name[2][:n], tuple(map(int, re.findall(r"\d+", args[1]))) if args else ()
            found.setdefault(key, []).append(dict(k, code=code[k[".name"]]))
    return found


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(rl.LIB_PATH):
        from paper_2509_06980_amd import build
        build.build()
    return _kernels(rl.LIB_PATH)


def test_forms_that_divide_no_rows_hold_no_code_for_it(kernels):
    # products and norms whose rows arrive divided by their rms (most passes) must not pay for those that divide themselves
    def one(name, *args):
        k, = kernels[name, args]
        return k
    swiglu = 2
    for (name, args), (k,) in [(key, k) for key, k in kernels.items() if key[0] in ("gemm_mfma_kernel", "gemm_decode_kernel")]:
        if args[0] != swiglu:
            assert not args[-1]
        elif not args[-1]:
            divides = one(name, *args[:-1], 1)
            assert divides["code"] - k["code"] > 500
    for fp8 in (0, 1):
        plain, divides = one("qkrope128_kernel", fp8, 0), one("qkrope128_kernel", fp8, 1)
        assert divides["code"] - plain["code"] > 500
        for k in (plain, divides):                             # 512 registers a SIMD lane in steps of 8: five waves
            assert k[".vgpr_count"] <= 96


def test_no_kernel_keeps_registers_in_scratch_memory(kernels):
    spills = {(key, k[".private_segment_fixed_size"]) for key, ks in kernels.items() for k in ks if k[".private_segment_fixed_size"]}
    assert not spills


def test_rows_in_one_workgroup_of_the_sampler_come_in_the_forms_that_are_launched(kernels):
    # (threads, 16-byte reads): rows that cannot be read in 16-byte pieces stop at the 4096 logits of 256 threads
    assert {args for name, args in kernels if name == "sample_row_kernel"} == {(256, 0), (256, 1), (512, 1), (1024, 1)}
