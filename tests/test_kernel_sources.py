"""Host checks on the kernel sources and on what they compile to: rules that a run of the kernels does not reliably
show when they are broken."""
import glob
import os
import re
import subprocess

import pytest

from paper_2011_09208_amd import buildlib

READELF = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")
CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2011_09208_amd", "csrc")


def asm_statements(text):
    """(template, outputs) of every inline-assembly statement."""
    for m in re.finditer(r"asm\s+volatile\s*\(", text):
        depth, i, quoted = 1, m.end(), False
        while depth:
            c = text[i]
            if c == '"' and text[i - 1] != "\\":
                quoted = not quoted
            depth += 0 if quoted else (c == "(") - (c == ")")
            i += 1
        body = text[m.end():i - 1]
        strings = re.match(r'\s*((?:"(?:[^"\\]|\\.)*"\s*)+)', body)
        rest = body[strings.end():]
        outputs = rest.split(":")[1].strip() if ":" in rest else ""
        yield strings.group(1), outputs


def test_asm_statements_are_found():
    got = list(asm_statements('asm volatile("a %0\\n" "b" : "=v"(x), "+v"(y) : "s"(f(z)) : "memory"); asm volatile("c" ::: "memory");'))
    assert [o for _, o in got] == ['"=v"(x), "+v"(y)', ""]


@pytest.mark.parametrize("path", sorted(glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(CSRC, "*.hip"))),
                         ids=os.path.basename)
def test_no_load_in_flight_has_an_output_register(path):
    """The compiler takes an output of inline assembly as written when the statement ends.  A load that is still in
    flight then may overwrite whatever the register holds by the time its data arrives."""
    for template, outputs in asm_statements(open(path).read()):
        if re.search(r"\b(buffer|global|flat|scratch|ds|s)_load|\bds_read", template) and outputs:
            assert "s_waitcnt" in template.rsplit("load", 1)[1], (os.path.basename(path), template)


def kernel_notes(lib, tmp_path):
    """{kernel: {field: value}} from the metadata of the gfx950 code objects inside the built library."""
    data, out, n = open(lib, "rb").read(), {}, 0
    at = data.find(b"\x7fELF", 4)
    while at >= 0:
        if int.from_bytes(data[at + 18:at + 20], "little") == 224:                  # EM_AMDGPU
            nxt = data.find(b"__CLANG_OFFLOAD_BUNDLE__", at)
            part = tmp_path / f"{n}.co"
            part.write_bytes(data[at:nxt if nxt > 0 else len(data)])
            text = subprocess.run([READELF, "--notes", str(part)], check=True, capture_output=True, text=True).stdout
            for kernel in text.split("- .agpr_count:")[1:]:
                fields = dict(re.findall(r"^\s+\.(\w+):\s+(\S+)$", kernel, re.M))
                out[fields["symbol"]] = fields
            n += 1
        at = data.find(b"\x7fELF", at + 4)
    return out


def test_no_kernel_spills_registers(tmp_path):
    """A spilled register that is reloaded inside a main loop makes the wave wait for all of its loads in flight."""
    if buildlib.is_stale():
        buildlib.build()
    kernels = kernel_notes(buildlib.LIB, tmp_path)
    assert len(kernels) > 30 and sum("bwd_dw_stream" in k for k in kernels) >= 4
    spilling = {k: v["vgpr_spill_count"] for k, v in kernels.items()
                if v["vgpr_spill_count"] != "0" or v["sgpr_spill_count"] != "0" or v["private_segment_fixed_size"] != "0"}
    assert not spilling, spilling


OBJDUMP = os.path.join(os.path.dirname(READELF), "llvm-objdump")


def test_stores_without_effect_are_not_merged(tmp_path):
    """The list kernels' first waits count 16 stores per wave that are issued to be counted.  They are alike; merged into fewer, the
    waits would let loads of the first tile pass for them and its first k-steps be read before they have arrived."""
    if buildlib.is_stale():
        buildlib.build()
    kernel_notes(buildlib.LIB, tmp_path)                                            # writes the code objects
    text = "".join(subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(p)], check=True, capture_output=True, text=True).stdout
                   for p in tmp_path.glob("*.co"))
    count = {}
    for body in re.split(r"^[0-9a-f]+ <", text, flags=re.M)[1:]:
        name = body.split(">", 1)[0]
        if "bwd_dz_list" in name:
            count[name] = len(re.findall(r"\bbuffer_store_dword ", body))
    assert count and all(n == 16 for n in count.values()), count
