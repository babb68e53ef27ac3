"""What the built library's GPU code says of its kernels (the AMDGPU metadata note of its code objects; no GPU)."""
import os
import re
import struct
import subprocess

import msgpack
import pytest

import paper_2401_05031_amd as otas

BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"
NT_AMDGPU_METADATA = 32


def _kernels_of_elf(elf):
    phoff, = struct.unpack_from("<Q", elf, 32)
    size, count = struct.unpack_from("<HH", elf, 54)
    for i in range(count):
        kind, _, at, _, _, length = struct.unpack_from("<IIQQQQ", elf, phoff + i * size)
        end = at + length
        while kind == 4 and at < end:                              # PT_NOTE
            name, desc, note = struct.unpack_from("<III", elf, at)
            body = at + 12 + (name + 3) // 4 * 4
            if note == NT_AMDGPU_METADATA:
                return msgpack.unpackb(elf[body:body + desc])["amdhsa.kernels"]
            at = body + (desc + 3) // 4 * 4
    return []


def _code_objects():
    """Every gfx950 ELF in the library."""
    if not os.path.exists(otas.lib_path()):
        from paper_2401_05031_amd import build
        build.build(verbose=False)
    with open(otas.lib_path(), "rb") as f:
        data = f.read()
    out, at = [], data.find(BUNDLE)
    while at >= 0:
        entries, = struct.unpack_from("<Q", data, at + len(BUNDLE))
        p = at + len(BUNDLE) + 8
        for _ in range(entries):
            first, size, name = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + name]:
                out.append(data[at + first:at + first + size])
            p += 24 + name
        at = data.find(BUNDLE, at + 1)
    return out


def built_kernels():
    """Metadata of every gfx950 kernel in the library."""
    return [k for elf in _code_objects() for k in _kernels_of_elf(elf)]


@pytest.fixture(scope="module")
def kernels():
    found = built_kernels()
    assert len(found) > 100
    return found


def test_kernel_arguments_stay_within_what_hip_promises(kernels):
    """4 KB, the implicit arguments among them: kernels that carry a plan in their arguments come close."""
    sizes = {k[".name"]: k[".kernarg_segment_size"] for k in kernels}
    assert max(sizes.values()) > 3840                              # the plan's 960 entries are among them
    assert {n: s for n, s in sizes.items() if s > 4096} == {}


def test_every_kernel_has_its_place_in_the_traffic_figures(kernels, tmp_path):
    """The per-family HBM figures are counted by kernel name: no kernel of the library is outside the families and the
    named rest, every product (bf16 and fp32) counts as one, and an unknown kernel stops the tool."""
    from paper_2401_05031_amd import traffic
    names = [k[".name"] for k in kernels]
    assert {n for n in names if traffic.family(n) is None} == set()
    assert {n for n in names if "gemm" in n and traffic.family(n) != "gemm"} == set()
    assert {traffic.family(n) for n in names} == set(traffic.FAMILIES) | {""}
    csv = tmp_path / "fetch.csv"
    rows = ["Kernel_Name,Counter_Name,Counter_Value", "__amd_rocclr_copyBuffer,FETCH_SIZE,262144",
            "void otas::gemm_f32_kernel<float>,FETCH_SIZE,8", "void otas::gemm_mfma64_kernel<0>,FETCH_SIZE,4"]
    csv.write_text("\n".join(rows))
    per, cal = traffic._load(str(csv), "FETCH_SIZE")
    assert per["gemm"] == [2, 12.0] and cal == 262144
    csv.write_text("\n".join(rows + ["void otas::renamed_kernel,FETCH_SIZE,4"]))
    with pytest.raises(ValueError, match="renamed_kernel"):
        traffic._load(str(csv), "FETCH_SIZE")


def reads_in_flight_at_barriers(lines):
    """Names of the functions in a disassembly that reach an s_barrier with an LDS read of their own not waited for."""
    name, out, found, barriers = "", 0, set(), 0
    for line in lines:
        if line.endswith(">:\n"):
            name, out = line[line.index("<") + 1:-3], 0
            continue
        op = line.split(None, 1)[0] if line.strip() else ""
        if op.startswith("ds_read") or op.startswith("ds_load"):
            out += 1
        elif op == "s_waitcnt":
            count = re.search(r"lgkmcnt\((\d+)\)", line)
            out = min(out, int(count.group(1))) if count else out
        elif op == "s_barrier":
            barriers += 1
            if out:
                found.add(name)
    return found, barriers


def test_no_lds_read_is_under_way_at_a_barrier(tmp_path):
    """What a wave reads from LDS before a barrier may be overwritten after it, by loads or by another wave's stores, and the
    barrier itself waits for nothing: every kernel of the library has its reads back before it.  (In the order of the
    code: loops and branches are not followed.)"""
    objdump = "/opt/rocm/llvm/bin/llvm-objdump"
    if not os.path.exists(objdump):
        pytest.skip("no disassembler for the AMD GPU")
    lines = ["0 <planted>:\n", "\tds_read_b128 v[0:3], v4\n", "\ts_waitcnt lgkmcnt(1)\n", "\ts_barrier\n",
             "0 <sound>:\n", "\tds_read_b128 v[0:3], v4\n", "\ts_waitcnt vmcnt(0) lgkmcnt(0)\n", "\ts_barrier\n"]
    assert reads_in_flight_at_barriers(lines) == ({"planted"}, 2)
    total = 0
    for i, elf in enumerate(_code_objects()):
        path = tmp_path / f"{i}.elf"
        path.write_bytes(elf)
        with subprocess.Popen([objdump, "-d", "--no-show-raw-insn", str(path)], stdout=subprocess.PIPE, text=True) as p:
            found, barriers = reads_in_flight_at_barriers(p.stdout)
        assert p.returncode == 0 and not found, found
        total += barriers
    assert total > 300
