"""Registers, scratch and memory instructions of the built kernels, read from
the code objects (no GPU needed).  The launch rules count on so many waves of
a kernel fitting on a SIMD (512 VGPRs, in blocks of 8), the streaming kernels
on buffer accesses with their cache policy; a change that costs either shows
here, while results stay the same."""
import re
import struct
import subprocess
from pathlib import Path

import pytest

TOOLS = Path("/opt/rocm/llvm/bin")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(fat):
    """The gfx950 code objects of a .hip_fatbin section (a chain of offload bundles)."""
    at = fat.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", fat, at + 24)
        pos = at + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", fat, pos)
            pos += 24
            if size and b"gfx950" in fat[pos:pos + length]:
                yield fat[at + off:at + off + size]
            pos += length
        at = fat.find(MAGIC, at + 1)


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """The library's code objects as files."""
    if not (TOOLS / "llvm-readelf").exists() or not (TOOLS / "llvm-objcopy").exists():
        pytest.skip("no LLVM tools")
    import paper_2510_20171_amd as xr
    if not xr._lib.LIB_PATH.exists():
        from paper_2510_20171_amd import build
        build.build()
    tmp = tmp_path_factory.mktemp("code")
    subprocess.run([TOOLS / "llvm-objcopy", f"--dump-section=.hip_fatbin={tmp / 'fat'}",
                    xr._lib.LIB_PATH, tmp / "copy"], check=True, timeout=100)
    paths = []
    for i, code in enumerate(_code_objects((tmp / "fat").read_bytes())):
        paths.append(tmp / f"{i}.co")
        paths[-1].write_bytes(code)
    return paths


@pytest.fixture(scope="module")
def kernels(code_objects):
    """{mangled name: (VGPRs, bytes of scratch per lane)}"""
    found = {}
    for path in code_objects:
        notes = subprocess.run([TOOLS / "llvm-readelf", "--notes", path], check=True, timeout=100,
                               capture_output=True, text=True).stdout
        for block in notes.split("\n  - .agpr_count:")[1:]:
            def field(key):
                return re.search(rf"\.{key}:\s+(\S+)", block).group(1)  # noqa: B023
            found[field("name")] = (int(field("vgpr_count")),
                                    int(field("private_segment_fixed_size")))
    assert len(found) > 1000
    return found


FUSED = re.compile(r"reduce_vec_kernelINS_\d+T(\w+?)ENS_\d+Op(\w+?)ELi(n?\d+)ELi\d+ELi(\d)ELi(\d+)"
                   r"ELb([01])E")


def _fused(kernels):
    """(type, op, sources, vectors a thread, threads, output off the grid?, VGPRs, scratch)"""
    out = []
    for name, (vgprs, scratch) in kernels.items():
        m = FUSED.search(name)
        if m:
            t, op, np_, u, b, off = m.groups()
            out.append((t, op, int(np_.replace("n", "-")), int(u), int(b), off == "1", vgprs,
                        scratch))
    assert len(out) > 1000
    return out


def _waves(vgprs):
    return 512 // max(8, -(-vgprs // 8) * 8)


def test_outputs_on_the_grid_do_not_pay_for_the_others(kernels):
    """Up to 8 sources and one vector a thread leave room for 7 waves per SIMD
    in every type and op, and no count of sources needs scratch."""
    bad = [k for k in _fused(kernels) if not k[5]
           and (k[7] or (1 <= k[2] <= 8 and k[3] == 1 and _waves(k[6]) < 7))]
    assert not bad, bad


def test_outputs_off_the_grid_fold_as_they_load(kernels):
    """Groups of sources are folded while later ones load there too: 64 sources
    stay within 128 VGPRs (4 waves per SIMD, more than their launches' cap)."""
    bad = [k for k in _fused(kernels) if k[5] and k[2] in (16, 32, 64) and _waves(k[6]) < 4]
    assert not bad, bad


def test_counts_known_at_launch_keep_their_waves(kernels):
    """Counts above 8 without a kernel of their own (0): the uncapped 512-thread
    shape counts on 8 waves per SIMD (16 values a vector: 3).  With the next
    group in flight (-1) they stay within the few waves such launches have."""
    byte = ("E4M3", "E5M2", "I8", "U8")
    got = [k for k in _fused(kernels) if k[2] in (0, -1)]
    assert any(k[2] == -1 for k in got)
    bad = [k for k in got if k[7] or _waves(k[6]) < (
        3 if k[0] in byte or k[2] == -1 else 8 if k[4] == 512 else 6)]
    assert not bad, bad


def test_two_vectors_a_thread_leave_two_workgroups_per_cu(kernels):
    """Two vectors of each source a thread: two 512-thread workgroups of every
    type fit on a CU (4 waves per SIMD), without scratch."""
    bad = [k for k in _fused(kernels) if k[3] == 2 and (k[7] or _waves(k[6]) < 4)]
    assert not bad, bad


def test_steps_of_wide_types_use_buffer_accesses(code_objects, kernels):
    """Closing casts and FINAL steps of 4- and 8-byte types store whole vectors
    at device scope, and plain steps load theirs, through buffer descriptors:
    per-lane tests and ordinary stores took 4 to 30 % more."""
    wide = r"NS_\d+T(F32|I32|U32|F64|I64|U64)E"
    stores = [n for n in kernels if re.search(rf"(acc_cast_kernelI{wide}|step_kernelI{wide}"
                                              r"NS_\d+OpSumELj[23]E)", n)]
    loads = [n for n in kernels if re.search(rf"step_kernelI{wide}NS_\d+OpSumELj0E", n)]
    assert len(stores) == 18 and len(loads) == 6, (stores, loads)
    text = ""
    for path in code_objects:
        text += subprocess.run([TOOLS / "llvm-objdump", "-d", "--disassemble-symbols="
                                + ",".join(stores + loads), path], check=True, timeout=100,
                               capture_output=True, text=True).stdout
    body = dict(re.findall(r"<(\w+)>:\n(.*?)(?=\n[0-9a-f]+ <|\Z)", text, re.S))
    for n in stores:
        assert len(re.findall(r"buffer_store_dwordx4 .* sc1", body[n])) >= 2, n
        assert "global_store_dwordx4" not in body[n] and "flat_store_dwordx4" not in body[n], n
    for n in loads:      # the input's two vectors and the accumulator's
        assert len(re.findall(r"buffer_load_dwordx4", body[n])) >= 4, n


def test_batched_tiles_do_not_read_sources_an_item_lacks(code_objects, kernels):
    """In the batched kernels a source's loads stand behind a test of the item's
    source count (7 in a first group that is not whole, 8 in later groups):
    loads of empty ranges made batches of few sources up to 40 % slower."""
    names = [n for n in kernels
             if re.search(r"batched_(rr_|table_|runs_|queue_)?kernelINS_\d+TBF16ENS_\d+OpSumE", n)]
    assert len(names) >= 5, names
    text = ""
    for path in code_objects:
        text += subprocess.run([TOOLS / "llvm-objdump", "-d", "--disassemble-symbols="
                                + ",".join(names), path], check=True, timeout=100,
                               capture_output=True, text=True).stdout
    body = dict(re.findall(r"<(\w+)>:\n(.*?)(?=\n[0-9a-f]+ <|\Z)", text, re.S))
    for n in names:
        blocks = [b for b in body[n].split("s_cbranch") if "buffer_load_dwordx4" in b]
        assert len(blocks) >= 15, (n, len(blocks))
