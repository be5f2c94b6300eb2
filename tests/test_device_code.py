"""What the compiler makes of device code where times depend on it and results do not."""
import os
import re
import subprocess

import pytest

from paper_2602_06183_amd import build


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """source file -> {kernel's mangled name: its assembly}"""
    out = tmp_path_factory.mktemp("device")
    known = {}

    def compiled(source):
        if source not in known:
            path = str(out / (source + ".s"))
            subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, source), "-o", path],
                           check=True, stderr=subprocess.DEVNULL)
            known[source] = {m.group(1): m.group(2) for m in re.finditer(r"^(_Z\w+):\s*;.*?\n(.*?)^\.Lfunc_end", open(path).read(), re.M | re.S)}
        return known[source]
    return compiled


def test_rings_are_filled_without_loads_that_the_compiler_counts(kernels):
    """The ring's loads go past the compiler's count of what is in flight: it answers a load of its own among them by waiting for all, one stage after the other."""
    units = {name: code for name, code in kernels("gemm_vnm8.hip").items() if "Vnm8Unit" in name}
    assert len(units) >= 8
    for name, code in units.items():
        before = code[:code.index("v_smfmac")]
        assert "global_load_lds_dwordx4" in before and not re.search(r"\t(global|flat|buffer)_load_(?!lds)", before), name


def test_row_major_contractions_keep_their_registers(kernels):
    """A register that goes to scratch and comes back shares the counter of the ring's loads: waiting for it drains them."""
    units = {name: code for name, code in kernels("gemm_v2_row.hip").items() if "GemmV2Unit" in name}
    assert len(units) >= 12
    assert [name for name, code in units.items() if re.search(r"\tscratch_(load|store)", code)] == []


def router_epilogues(kernels):
    units = {name: code for name, code in kernels("gemm_v2.hip").items() if re.search(r"unit_kernelINS_10GemmV2UnitILb1ELb1ELi[34]E", name)}
    assert len(units) >= 4
    return units


def test_packed_rows_of_the_router_leave_in_one_group(kernels):
    """A branch per store keeps the LDS reads of the next sweep behind it."""
    for name, code in router_epilogues(kernels).items():
        groups = re.findall(r"(?:\tglobal_store_dword v[^\n]* nt\n(?:\t(?!s_cbranch|s_branch|ds_read)[^\n]*\n)*){16}", code)
        assert groups, name


def test_router_keeps_y1_for_eq_4_by_the_rule_of_the_launch(kernels):
    """What the epilogue of eq. (1) leaves for later launches has an ordinary store for every non-temporal one."""
    for name, code in router_epilogues(kernels).items():
        if "Li3E" in name.split("GemmV2Unit")[1][:30]:
            wide = re.findall(r"\tglobal_store_dwordx4 [^\n]*", code)
            assert len(wide) >= 32 and sum(" nt" in w for w in wide) * 2 == len(wide), name


def test_sums_of_the_other_splits_are_read_behind_the_count(tmp_path):
    """Counting in and the loads of the sums are relaxed atomics of different addresses, which a compiler may reorder; before any optimisation a barrier for it stands between them."""
    path = str(tmp_path / "vnm8.ll")
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *build.FLAGS, "--cuda-device-only", "-S", "-emit-llvm", "-Xclang", "-disable-llvm-passes", os.path.join(build.CSRC, "gemm_vnm8.hip"), "-o", path],
                   check=True, stderr=subprocess.DEVNULL)
    body = re.search(r"^define [^\n]*split_join4[^\n]*\{\n(.*?)^\}", open(path).read(), re.M | re.S).group(1)
    counted = body.index("atomicrmw add")
    barrier, sums = body.find('asm sideeffect "", "~{memory}"', counted), re.compile(r"call [^\n]*split_join4[^\n]*ENKUl").search(body, counted)
    assert sums and counted < barrier < sums.start()


def test_activations_are_stored_the_ordinary_way(kernels):
    """The next kernel reads them.  Results of eqs. (1), (4) by themselves and of the compression have a non-temporal form for sizes of the last-level cache, those of eqs. (3), (7) for those of the L2s;
    tiles of few tokens and shared contractions have none."""
    plain = re.compile(r"\tglobal_store_dwordx4 [^\n]*(?<! nt)\n")
    past = re.compile(r"\tglobal_store_dwordx4 [^\n]* nt\n")
    for source, pattern, few in (("gemm_vnm8.hip", "Vnm8Unit", "VTileILi1ELi1E"), ("gemm_gather.hip", "Gather", "GTileILi1E")):
        units = {name: code for name, code in kernels(source).items() if pattern in name}
        assert len(units) >= 3 and any(few in name for name in units)
        for name, code in units.items():
            assert len(plain.findall(code)) > 0 and len(past.findall(code)) == (0 if few in name else len(plain.findall(code))), name
    rows = {name: code for name, code in kernels("gemm_v2_row.hip").items() if "GemmV2UnitILb1ELb1ELi0E" in name}
    assert rows and all(len(plain.findall(code)) == len(past.findall(code)) > 0 for code in rows.values()), rows.keys()
    compress = {name: code for name, code in kernels("vnm_general.hip").items() if "compress_m_kernelILi8E" in name}
    assert {("Lb1E" in name, bool(past.search(code)), bool(plain.search(code))) for name, code in compress.items()} == {(True, True, False), (False, False, True)}
