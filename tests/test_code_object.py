"""The device code as built: what the instruction listing and the metadata of
libmmas.so's gfx950 code objects must show."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")


def _run(*cmd, cwd=None):
    return subprocess.run(cmd, cwd=cwd, check=True, capture_output=True, text=True, timeout=300).stdout


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """Paths of the library's gfx950 code objects."""
    lib = os.path.join(ROOT, "paper_2003_11902_amd", "libmmas.so")
    if not os.path.exists(lib):
        from paper_2003_11902_amd import build
        build.build()
    if not os.path.exists(os.path.join(LLVM, "llvm-objdump")):
        pytest.skip("no llvm-objdump")
    d = tmp_path_factory.mktemp("code")
    shutil.copy(lib, d)
    _run(os.path.join(LLVM, "llvm-objdump"), "--offloading", "libmmas.so", cwd=d)
    out = sorted(str(p) for p in d.iterdir() if p.name.endswith("gfx950"))
    assert out
    return out


def _scalars(text):
    """Numbers of the scalar registers that an operand list names."""
    out = set()
    for a, b, one in re.findall(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b", text):
        out.update(range(int(a), int(b) + 1) if a else [int(one)])
    return out


def close_scalar_reads(listing):
    """(writer, reader) pairs of a vector instruction that reads a scalar
    register fewer than two wait states after v_readlane or v_readfirstlane
    wrote it. An instruction in between counts for one, s_nop k for k + 1."""
    found, recent = [], []  # recent: [register, writer, wait states since]
    for line in listing.splitlines():
        m = re.match(r"\s+([a-z]\w+)\s*(.*?)\s*(?://.*)?$", line)
        if not m:
            if line.endswith(">:"):
                recent = []
            continue
        op, args = m.groups()
        if op.startswith("v_"):
            first, _, rest = args.partition(",")
            # (a lane write reads its second operand, and keeps the first)
            read = _scalars(rest if op.startswith(("v_read", "v_writelane")) else args)
            found += [(w, line.strip()) for r, w, d in recent if d < 2 and r in read]
        states = int(args or 0, 0) + 1 if op == "s_nop" else 1
        recent = [[r, w, d + states] for r, w, d in recent if d + states < 2]
        if op.startswith(("v_readlane", "v_readfirstlane")):
            recent += [[r, line.strip(), 0] for r in _scalars(args.partition(",")[0])]
    return found


def test_the_reader_of_listings():
    bad = "\tv_readfirstlane_b32 s4, v2\n\tv_writelane_b32 v1, s4, 2\n"
    one = "\tv_readlane_b32 s4, v2, 3\n\ts_add_i32 s5, s4, 1\n\tv_add_u32_e32 v1, s4, v1  // 00: 00\n"
    assert len(close_scalar_reads(bad)) == 1 and len(close_scalar_reads(one)) == 1
    assert not close_scalar_reads(bad.replace("\n\tv_w", "\n\ts_nop 1\n\tv_w"))
    assert not close_scalar_reads(bad.replace("s4, 2", "s5, 2"))


def test_lane_reads_settle_before_vector_reads(code_objects):
    """A vector instruction may read a scalar register two wait states after a
    lane read wrote it at the earliest; the compiler sees to that, but not
    where an instruction hides in inline assembly."""
    found = []
    for path in code_objects:
        found += close_scalar_reads(_run(os.path.join(LLVM, "llvm-objdump"), "-d", "--no-show-raw-insn", path))
    assert not found, f"{len(found)} reads too early, the first: {found[:3]}"


def kernel_lds(notes):
    """{kernel: bytes of static LDS, where its dynamic LDS starts}."""
    out = {}
    for block in notes.split(".agpr_count:")[1:]:
        size = re.search(r"\.group_segment_fixed_size:\s*(\d+)", block)
        name = re.search(r"\.name:\s*(_Z\S+)", block)
        out[name.group(1)] = int(size.group(1))
    return out


def test_dynamic_lds_starts_at_16_bytes(code_objects):
    """The nearest-neighbour tour stores 16 bytes at a time into its dynamic LDS,
    and so do the constructions and the 2-opt: it has to start at a multiple
    of 16, behind whatever static LDS the kernel has."""
    lds = {}
    for path in code_objects:
        lds.update(kernel_lds(_run(os.path.join(LLVM, "llvm-readelf"), "--notes", path)))
    wide = {k: v for k, v in lds.items()
            if any(s in k for s in ("k_nn_tour", "11k_construct", "k_batch_construct", "k_two_opt", "k_mlp_train"))
            and "k_construct_team" not in k}  # (the team has no dynamic LDS)
    assert any("k_nn_tour" in k for k in wide) and len(wide) > 20
    assert not {k: v for k, v in wide.items() if v % 16}


def test_batched_construction_fits_eight_waves(code_objects):
    """Eight waves share a SIMD's 512 vector registers: 64 each (the functions a
    kernel calls count)."""
    regs = {}
    for path in code_objects:
        for block in _run(os.path.join(LLVM, "llvm-readelf"), "--notes", path).split(".agpr_count:")[1:]:
            name = re.search(r"\.name:\s*(_Z\S+)", block).group(1)
            if "k_batch_construct" in name:
                regs[name] = int(re.search(r"\.vgpr_count:\s*(\d+)", block).group(1))
    assert len(regs) == 24
    assert not {k: v for k, v in regs.items() if v > 64}


@pytest.mark.parametrize("name", ["mmas.hip", "prep.hip", "construct.hip", "update.hip", "two_opt.hip", "batch.hip",
                                  "learned.hip", "diag.hip"])
def test_sources_compile_without_a_warning(name):
    """Neither the device's nor the host's pass of the compiler warns."""
    from paper_2003_11902_amd import build
    assert name in build.SOURCES
    r = subprocess.run([build._hipcc(), *build.FLAGS, "-fsyntax-only", os.path.join(build.CSRC, name)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "warning" not in r.stderr, r.stderr[:2000]
