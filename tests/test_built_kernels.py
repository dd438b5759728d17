"""The instructions of the built library's kernels.  A buffer store of more than 8 bytes per lane whose offset is partly in a scalar
register, followed at once by an instruction that overwrites its data registers, has stored the new values on gfx950, and the
compiler inserts no wait there: no kernel may have such a store.  (Whether a wait is there depends on what follows the store, and
that changes with any edit; with the whole offset in a vector register the compiler waits where it has to.)

And what else is to be seen there: a kernel that writes device memory only does not write its caches back to the system."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2508_19263_amd import zc

LLVM = "/opt/rocm/llvm/bin"
STORE = re.compile(r"^\s*buffer_store_(?:dwordx[34]|format_xyzw?) ([^/]*)")


def wide_scalar_offset_stores(listing):
    """Lines of a listing that hold a store as described: data, vector offset, resource, then the scalar offset."""
    hits = []
    for line in listing:
        m = STORE.match(line)
        if m:
            soffset = m.group(1).split(", ")[3].split()[0]
            if not re.fullmatch(r"0|0x0|null", soffset):
                hits.append(line.strip())
    return hits


def test_the_pattern_finds_what_it_looks_for():
    assert wide_scalar_offset_stores(["\tbuffer_store_dwordx4 v[2:5], v9, s[4:7], s20 offen nt  // 00001234: E07E1000"])
    assert wide_scalar_offset_stores(["\tbuffer_store_dwordx4 v[2:5], off, s[4:7], m0  // 0"])
    assert not wide_scalar_offset_stores(["\tbuffer_store_dwordx4 v[2:5], v9, s[4:7], 0 offen offset:1024 nt  // 00001234: E07E1000",
                                          "\tbuffer_store_dwordx2 v[2:3], v9, s[4:7], s20 offen  // 0", "\tbuffer_load_dwordx4 v[2:5], v9, s[4:7], s20 offen"])


def test_no_wide_store_with_a_scalar_offset(tmp_path):
    if not os.path.exists(LLVM + "/llvm-objdump"):
        pytest.skip("llvm-objdump not found")
    zc.lib()                                                   # (fails if the library is not built)
    shutil.copy(os.path.join(os.path.dirname(zc.__file__), "libzc.so"), str(tmp_path))
    subprocess.run([LLVM + "/llvm-objdump", "--offloading", "libzc.so"], cwd=str(tmp_path), check=True, capture_output=True)
    objects = [f for f in os.listdir(str(tmp_path)) if f.endswith("gfx950")]
    assert objects
    stores, hits = 0, []
    for f in objects:
        listing = subprocess.run([LLVM + "/llvm-objdump", "-d", f], cwd=str(tmp_path), check=True, capture_output=True, text=True).stdout.splitlines()
        stores += sum(1 for line in listing if STORE.match(line))
        hits += wide_scalar_offset_stores(listing)
    assert stores > 100 and not hits, (stores, len(hits), hits[:5])


def listing_of(tmp_path, symbol):
    """The instructions of the kernel whose symbol starts like that (of all files of the library's: the one that has it)."""
    shutil.copy(os.path.join(os.path.dirname(zc.__file__), "libzc.so"), str(tmp_path))
    subprocess.run([LLVM + "/llvm-objdump", "--offloading", "libzc.so"], cwd=str(tmp_path), check=True, capture_output=True)
    for f in sorted(f for f in os.listdir(str(tmp_path)) if f.endswith("gfx950")):
        names = subprocess.run([LLVM + "/llvm-readelf", "-s", "--wide", f], cwd=str(tmp_path), check=True, capture_output=True, text=True).stdout.split()
        found = [n for n in names if n.startswith(symbol) and "." not in n]
        if found:
            return subprocess.run([LLVM + "/llvm-objdump", "-d", "--no-show-raw-insn", "--disassemble-symbols=" + found[0], f], cwd=str(tmp_path), check=True,
                                  capture_output=True, text=True).stdout
    return ""


@pytest.mark.parametrize("to_host", [False, True])
def test_only_what_the_host_reads_is_written_back_to_the_system(tmp_path, to_host):
    if not os.path.exists(LLVM + "/llvm-objdump"):
        pytest.skip("llvm-objdump not found")
    zc.lib()
    listing = listing_of(tmp_path, "_ZN2zc11k_hand_overILb%d" % to_host)
    assert "global_store" in listing and ("buffer_wbl2" in listing) == to_host


def waits_before_barrier(listing):
    """For every barrier of a listing: is the last instruction in front of it that concerns memory a wait for all of the wavefront's stores?"""
    lines = [line.split("//")[0].split() for line in listing.split("\n")]
    barriers, ok = [i for i, w in enumerate(lines) if w and w[0] == "s_barrier"], []
    for i in barriers:
        before = [" ".join(w) for w in lines[:i] if w and re.match(r"s_waitcnt|global_|buffer_|flat_", w[0])]
        ok.append(bool(before) and re.match(r"s_waitcnt.*vmcnt\(0\)", before[-1]) is not None)
    return ok


def test_the_waits_are_found():
    assert waits_before_barrier("\tglobal_store_dword v0, v1, s[0:1]  // 0\n\ts_waitcnt vmcnt(0)  // 4\n\ts_mov_b32 s0, 0  // 8\n\ts_barrier  // c") == [True]
    assert waits_before_barrier("\ts_waitcnt vmcnt(0)  // 0\n\tglobal_store_dword v0, v1, s[0:1]  // 4\n\ts_waitcnt lgkmcnt(0)  // 8\n\ts_barrier  // c") == [False]
    assert waits_before_barrier("\ts_barrier  // 0") == [False]


def test_what_the_host_is_told_of_has_been_stored(tmp_path):
    """One thread tells the host that the workgroup's bytes are there: every wavefront has waited for its stores in front of the barrier before that."""
    if not os.path.exists(LLVM + "/llvm-objdump"):
        pytest.skip("llvm-objdump not found")
    zc.lib()
    assert waits_before_barrier(listing_of(tmp_path, "_ZN2zc11k_hand_overILb1")) == [True]


def test_registers_of_the_decoder_whose_workgroups_share_a_compute_unit(tmp_path):
    """BF16 deltas with short rings: seven wavefronts per SIMD (85 registers and five of them made sets of small deltas 5 - 15 % slower)."""
    if not os.path.exists(LLVM + "/llvm-objdump"):
        pytest.skip("llvm-objdump not found")
    zc.lib()
    listing_of(tmp_path, "_ZN2zc14k_decode_pairsILi1ELb1E")    # (leaves the files' code objects there)
    counts = []
    for f in sorted(f for f in os.listdir(str(tmp_path)) if f.endswith("gfx950")):
        notes = subprocess.run([LLVM + "/llvm-readelf", "--notes", f], cwd=str(tmp_path), check=True, capture_output=True, text=True).stdout
        for kernel in notes.split("- .agpr_count")[1:]:
            if re.search(r"\.name: +_ZN2zc14k_decode_pairsILi1ELb1ELNS_6LaunchE2E", kernel):
                counts.append(int(re.search(r"\.vgpr_count: +(\d+)", kernel).group(1)))
    assert counts and max(counts) <= 72, counts
