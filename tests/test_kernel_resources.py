"""The built library's GPU code, read on the CPU (nothing is launched): LDS of the split kernels against
what a gfx950 CU holds, the static part from the metadata of the code objects, the dynamic part from
the functions that the launches use; and what the append's barrier stands between."""
import ctypes
import os
import re
import struct
import subprocess

import msgpack
import pytest

from paper_2504_15930_amd import build, sl

LDS_PER_CU = 160 * 1024
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
KINDS = [(64, "bf16"), (128, "bf16"), (64, "e4m3"), (128, "e4m3")]


def _code_objects(data):
    """The gfx950 ELF images of the fat binaries in a library file."""
    at = data.find(MAGIC)
    while at >= 0:
        pos = at + len(MAGIC)
        n, = struct.unpack_from("<Q", data, pos)
        pos += 8
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + length]
            pos += 24 + length
            if name.endswith(build.ARCH.encode()):
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, at + 1)


def _kernels(elf):
    """The kernel records of a code object's AMDGPU metadata note."""
    phoff, = struct.unpack_from("<Q", elf, 32)
    phsize, phnum = struct.unpack_from("<HH", elf, 54)
    for i in range(phnum):
        kind, _, off, _, _, size = struct.unpack_from("<IIQQQQ", elf, phoff + i * phsize)
        if kind != 4:   # PT_NOTE
            continue
        end = off + size
        while off < end:
            namesz, descsz, note = struct.unpack_from("<III", elf, off)
            name = elf[off + 12:off + 12 + namesz]
            desc = off + 12 + (namesz + 3) // 4 * 4
            if note == 32 and name.startswith(b"AMDGPU"):
                yield from msgpack.unpackb(elf[desc:desc + descsz])["amdhsa.kernels"]
            off = desc + (descsz + 3) // 4 * 4


@pytest.fixture(scope="module")
def static_lds():
    """Static LDS bytes by mangled kernel name."""
    if not os.path.exists(sl.LIBRARY):
        build.build()
    data = open(sl.LIBRARY, "rb").read()
    return {k[".name"]: k[".group_segment_fixed_size"] for elf in _code_objects(data) for k in _kernels(elf)}


@pytest.fixture(scope="module")
def sizes(tmp_path_factory):
    """The launches' dynamic LDS functions, compiled for the host."""
    d = tmp_path_factory.mktemp("sizes")
    (d / "sizes.cpp").write_text(
        '#include "sl_internal.h"\n'
        'extern "C" size_t split_bytes(int b) { return sl::split_dynamic_lds(b); }\n'
        'extern "C" size_t prefix_bytes(int b, int ng, int g)\n'
        '{ return sl::prefix_dynamic_lds(b, sl::prefix_max_sub(b, ng, g)); }\n'
        'extern "C" int shared_workers(int own_tiles, int own_workers, int base, int most)\n'
        '{ return sl::effective_shared_workers(own_tiles, own_workers, base, most, 1, false); }\n'
        'extern "C" int max_batch(int prefix) { return prefix ? sl::kMaxPrefixBatch : sl::kMaxBatch; }\n')
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    out = str(d / "sizes.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-I",
                    os.path.join(rocm, "include"), "-I", build.CSRC, str(d / "sizes.cpp"), "-o", out], check=True)
    lib = ctypes.CDLL(out)
    lib.split_bytes.restype = lib.prefix_bytes.restype = ctypes.c_size_t
    return lib


def _kernel(static_lds, name, D, kv):
    hits = [v for k, v in static_lds.items() if f"{name}ILi{D}ELb{int(kv == 'e4m3')}E" in k]
    assert len(hits) == 1, (name, D, kv, sorted(static_lds))
    return hits[0]


@pytest.mark.parametrize("D,kv", KINDS)
def test_split_kernel_fits_the_largest_batch(static_lds, sizes, D, kv):
    lds = _kernel(static_lds, "split_kv_kernel", D, kv) + sizes.split_bytes(sizes.max_batch(0))
    assert lds <= LDS_PER_CU


# The grown sizes are those of a step of several tiles; a step of one tile (bf16, D = 128) holds one
# workgroup of the split kernel, as its output stage and K stage always did.
@pytest.mark.parametrize("D,kv,batch", [(64, "bf16", 512), (64, "e4m3", 1024), (128, "e4m3", 512)])
def test_two_split_workgroups_per_cu(static_lds, sizes, D, kv, batch):
    """A caller's own worker count above four per CU runs two workgroups on one."""
    assert 2 * (_kernel(static_lds, "split_kv_kernel", D, kv) + sizes.split_bytes(batch)) <= LDS_PER_CU


@pytest.mark.parametrize("D,kv", KINDS)
def test_prefix_kernel_fits_every_accepted_size(static_lds, sizes, D, kv):
    """Up to 4096 sequences in up to 4096 groups, 1 to 16 heads per KV head."""
    static, B = _kernel(static_lds, "prefix_split_kernel", D, kv), sizes.max_batch(1)
    worst = max(sizes.prefix_bytes(B, ng, g) for ng in range(B + 1) for g in (1, 4, 5, 16))
    assert static + worst <= LDS_PER_CU, (static, worst)


@pytest.mark.parametrize("D,kv", [k for k in KINDS if k != (128, "bf16")])
@pytest.mark.parametrize("batch,groups,group", [(1536, 768, 7), (3000, 2, 7), (2700, 1, 16), (1000, 1000, 1)])
def test_two_prefix_workgroups_per_cu(static_lds, sizes, D, kv, batch, groups, group):
    """The shared pages stream beside the own ones: two workgroups on a CU."""
    one = _kernel(static_lds, "prefix_split_kernel", D, kv) + sizes.prefix_bytes(batch, groups, group)
    assert 2 * one <= LDS_PER_CU


@pytest.mark.parametrize("own,base,most", [(1024, 256, 512), (1216, 304, 608), (64, 16, 32), (4, 1, 2), (9, 2, 4), (1, 1, 1)])
def test_shared_workgroups_of_a_launch(sizes, own, base, most):
    """Prefix sharing adds as many workgroups to the shared pages' as own ones are idle, if that gives most of the
    CUs two; a few more than one per CU would all end late. Never more than own and shared slots together."""
    slots, seen = (own + 3) // 4 + base, set()
    for tiles in range(0, 8 * own + 2):
        n = sizes.shared_workers(tiles, own, base, most)
        busy = (min(own, max(1, -(-tiles // 4))) + 3) // 4 if tiles else 0
        assert base <= n <= most and n + busy <= slots
        assert n == base or 4 * (n - base) >= 3 * base or n == most
        seen.add(n)
    assert base in seen and most in seen


@pytest.mark.parametrize("D", [64, 128])
def test_e4m3_append_loads_the_old_scale_before_its_barrier(tmp_path, D):
    """Four wavefronts re-encode a tile whose scale one of them overwrites after the barrier: nothing is
    loaded after it."""
    objdump = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
    if not os.path.exists(objdump):
        pytest.skip("no llvm-objdump under ROCm here")
    if not os.path.exists(sl.LIBRARY):
        build.build()
    found = 0
    for i, elf in enumerate(_code_objects(open(sl.LIBRARY, "rb").read())):
        path = tmp_path / f"{i}.elf"
        path.write_bytes(elf)
        text = subprocess.run([objdump, "-d", "--no-show-raw-insn", str(path)], capture_output=True, text=True,
                              check=True).stdout
        for name, body in re.findall(r"^[0-9a-f]+ <(\S+)>:\n(.*?)(?=^[0-9a-f]+ <|\Z)", text, re.S | re.M):
            if f"append_kernelILi{D}ELi2E" not in name:   # kAppendSpread
                continue
            found += 1
            before, _, after = body.partition("s_barrier")
            assert after, "the barrier"
            assert not re.findall(r"\b(?:s|s_buffer|global|flat|buffer)_load\S*.*", after)
    assert found == 1
