"""What the compiler made of the kernels, read from the code objects in the library.  No kernel but the two layouts below spills vector registers or has any
scratch memory: what is spilled, every workgroup (and of a sum every member) stores and loads, and the loads are counted by the counter that its direct loads into LDS are
waited for with.  And how dot_mid_kernel stores its outputs."""
import os
import re
import subprocess

import pytest

import paper_2105_04663_amd as g

# dot_mfma_kernel through registers (STAGED) with a K-major lhs and 128 accumulators a lane: 8 to 11 of them, around its loop
SPILLS = {"dot_mfma_kernelI%sLi%dELb1E" % (out, layout): 11 for out in "ft" for layout in (1, 3)}
READELF, OBJDUMP = "/opt/rocm/llvm/bin/llvm-readelf", "/opt/rocm/llvm/bin/llvm-objdump"


def _code_objects(tmp_path):
    """Files with the library's gfx950 code objects."""
    with open(g.library_path(), "rb") as f:
        image = f.read()
    for i, at in enumerate(m.start() for m in re.finditer(rb"\x7fELF\x02\x01\x01\x40", image)):      # (0x40: the AMDGPU HSA ABI)
        path = str(tmp_path / f"code_{i}.o")
        with open(path, "wb") as f:
            f.write(image[at:])
        yield path
        os.remove(path)


def _kernels(tmp_path):
    """{name: (spilled vector registers, bytes of scratch per lane)} of every kernel of the library."""
    found = {}
    for path in _code_objects(tmp_path):
        notes = subprocess.run([READELF, "--notes", path], capture_output=True, text=True).stdout
        for entry in re.split(r"\n  - \.agpr_count", notes)[1:]:
            field = lambda key: re.search(r"\n    \.%s: +(\S+)" % key, entry).group(1)
            found[field("name")] = int(field("vgpr_spill_count")), int(field("private_segment_fixed_size"))
    return found


def test_no_kernel_spills(tmp_path):
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    kernels = _kernels(tmp_path)
    for kind in ("dot_mfma_kernel", "dot_mid_kernel", "dot_pair_kernel", "dot_split_kernel", "dot_f32_kernel"):
        assert sum(kind in name for name in kernels) >= 8, kind
    for name, (spilled, scratch) in kernels.items():
        most = max((n for kernel, n in SPILLS.items() if kernel in name), default=0)
        assert spilled <= most and scratch <= 4 * (most + 1), (name, spilled, scratch)


def test_how_dot_mid_kernel_stores_whole_tiles(tmp_path):
    """bf16 outputs: a store for each case, past the caches where a launch's outputs are more than these hold, else through to the memory side, where an einsum that
    reads them finds them (that one took up to 18 % longer with all of them past the caches), and rows that are not whole lines with neither hint; float32 outputs and staged tiles, whose lines
    may be stored in two parts: neither."""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    seen = {}
    for path in _code_objects(tmp_path):
        with open(path, "rb") as f:
            if b"dot_mid_kernel" not in f.read()[:1 << 16]:
                continue
        listing = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", path], capture_output=True, text=True).stdout
        for name, body in re.findall(r"^<(\S*dot_mid_kernel\S*)>:\n(.*?)(?=^<|\Z)", listing, re.S | re.M):
            stores = re.findall(r"global_store_dwordx4 [^\n]*", body)
            seen[name] = tuple(sum(bool(re.search(hint, x)) for x in stores) for hint in (r"\bnt\b", r"\bsc1\b", r"^(?!.*\b(nt|sc1)\b)"))
    assert len(seen) >= 40
    for name, (past, through, plain) in seen.items():
        out, chain, staged = re.search(r"dot_mid_kernelI(\w)Li\dELb(\d)ELi\dELb(\d)E", name).groups()
        hinted = out == "t" and staged == "0"
        assert (past, through) == ((8, 8) if hinted else (0, 0)), (name, past, through)
        assert not hinted or plain >= 16, (name, plain)          # eight of whole tiles, eight at edges
