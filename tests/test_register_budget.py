"""CPU-side check of what the compiler made of the scoring kernels: registers, scratch and LDS.

The weights sweeps and the statistics sweeps beyond 128 rows are laid out for two wavefronts per SIMD
(a SIMD has 512 registers per lane): a kernel of four-wavefront workgroups that needs more than 256
registers still runs, one wavefront per SIMD, at a little over half the speed, and a spill inside the
tile loop puts scratch loads between the K loads.  Neither shows in a parity test, and both have happened
after changes that looked harmless, so the build's own metadata is read back here (from the
code objects inside the built library, with the ROCm LLVM tools; nothing is launched)."""
import os
import re
import subprocess
import tempfile

import pytest

import paper_2407_11550_amd.binding as B

LLVM = "/opt/rocm/llvm/bin"
TOOLS = [os.path.join(LLVM, t) for t in ("llvm-objcopy", "clang-offload-bundler", "llvm-readelf")]
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _kernel_metadata(lib_path):
    """{kernel symbol: {vgpr, agpr, scratch, lds}} over every gfx950 code object in the library."""
    out = {}
    with tempfile.TemporaryDirectory() as tmp:
        fat = os.path.join(tmp, "fat.bin")
        subprocess.run([TOOLS[0], "-O", "binary", "--only-section=.hip_fatbin", lib_path, fat], check=True)
        data = open(fat, "rb").read()
        starts = [m.start() for m in re.finditer(re.escape(MAGIC), data)] + [len(data)]
        for i in range(len(starts) - 1):
            piece, obj = os.path.join(tmp, f"b{i}.bin"), os.path.join(tmp, f"co{i}.o")
            open(piece, "wb").write(data[starts[i]:starts[i + 1]])
            r = subprocess.run([TOOLS[1], "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950",
                                f"--input={piece}", f"--output={obj}"], capture_output=True, text=True)
            if r.returncode != 0 or not os.path.exists(obj) or os.path.getsize(obj) == 0:
                continue
            notes = subprocess.run([TOOLS[2], "--notes", obj], capture_output=True, text=True, check=True).stdout
            for block in notes.split("  - .agpr_count:")[1:]:
                def field(name, block=block):
                    m = re.search(r"\." + name + r":\s+(\S+)", block)
                    return m.group(1) if m else None
                out[field("name")] = dict(agpr=int(block.split()[0]), vgpr=int(field("vgpr_count")),
                                          scratch=int(field("private_segment_fixed_size")),
                                          lds=int(field("group_segment_fixed_size")))
    return out


def _instantiations(meta, kernel):
    """Template arguments of the kernel (whole numbers and truth values) -> metadata, from the mangled names.  The
    pattern reads all arguments: kernels that differ in one it left out would replace each other here."""
    pat = re.compile(r"%s((?:L[ib]\d+E)+)E" % (kernel + "I"))
    out = {}
    for name, md in meta.items():
        if kernel not in (name or ""):
            continue
        m = pat.search(name)
        assert m, f"{name}: template arguments of another kind"
        key = tuple(int(x) for x in re.findall(r"L[ib](\d+)E", m.group(1)))
        assert key not in out, f"two kernels with the arguments {key}"
        out[key] = md
    return out


@pytest.fixture(scope="module")
def metadata(lib):
    if not all(os.path.exists(t) for t in TOOLS):
        pytest.skip("ROCm LLVM tools not installed")
    return _kernel_metadata(B._LIB_PATH)


@pytest.fixture(scope="module")
def score_kernels(metadata):
    """(d, mb, rs, kg, chunk, pass, f16, pool_rows, wide steps) -> metadata"""
    ks = _instantiations(metadata, "score_mfma_kernel")
    # types x (the statistics sweep of five row counts per d, and three weights sweeps of d = 128: ten layouts, 64: nine)
    assert len(ks) == 2 * (2 * 5 + 3 * (10 + 9))
    return ks


@pytest.fixture(scope="module")
def cut_kernels(metadata):
    """fp32 scoring with products of bf16 parts: (d, pass, wavefronts, combines the statistics) -> metadata"""
    ks = _instantiations(metadata, "score_cut_kernel")
    assert set(ks) == {(d,) + form for d in (64, 128) for form in ((1, 4, 0), (1, 8, 0), (2, 4, 0), (2, 4, 1))}
    return ks


def test_two_wavefronts_per_simd_where_the_layout_counts_on_them(score_kernels):
    """The 128-, 256- and 512-row kernels in both sweeps and both 16-bit types, and both row-pooling
    forms of their weights sweeps: at most 256 registers (vector plus accumulation registers).  (The
    statistics sweep of up to 128 rows at d = 128 has the compute unit to itself for its tiles in LDS,
    one wavefront per SIMD; what it needs beyond 256 would be moved into accumulation registers.)  The
    32- and 64-row forms are bound by memory with one wavefront per SIMD as well."""
    checked = 0
    for key, md in score_kernels.items():
        if key[1:4] not in ((2, 2, 2), (2, 4, 1), (2, 8, 1), (4, 4, 1)):
            continue
        assert md["vgpr"] + md["agpr"] <= 256, (key, md)
        checked += 1
    # types x (the statistics sweep of three row counts per d, and three weights sweeps x (d = 128: four chunk
    # lengths, 256 rows and 512 rows with two each; d = 64: the first six and 512 rows with one))
    assert checked == 2 * (2 * 3 + 3 * (8 + 7))


def test_the_statistics_sweep_is_built_once_per_row_count(score_kernels):
    """It does not depend on how many scores a workgroup of the weights sweep has room for."""
    kinds = [key[:4] + key[5:] for key in score_kernels if key[5] == 1]
    assert len(kinds) == len(set(kinds)) == 2 * 2 * 5


def test_two_workgroups_of_the_cut_kernels_fit_on_a_compute_unit(cut_kernels):
    """What the rule on the pool's place counts on: two wavefronts per SIMD and half of a compute unit's LDS (160 KiB).
    (The form with eight wavefronts has the unit to itself: as many wavefronts.)"""
    for key, md in cut_kernels.items():
        assert md["vgpr"] + md["agpr"] <= 256, (key, md)
        assert md["lds"] <= 80 * 1024, (key, md)


def test_no_scoring_kernel_spills(score_kernels, cut_kernels):
    """No scratch memory in any matrix-core scoring kernel."""
    for key, md in list(score_kernels.items()) + list(cut_kernels.items()):
        assert md["scratch"] == 0, (key, md)
