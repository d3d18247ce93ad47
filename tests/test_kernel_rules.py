"""CPU checks of rules the kernels rely on, on the code itself: small host functions compiled from the kernels' headers."""
import ctypes as C
import os
import re
import subprocess

import numpy as np
import pytest

from paper_2308_15949_amd import build as B


def hipcc(*args):
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *B.FLAGS, *args], check=True, capture_output=True, text=True)


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.hip").write_text('#include "laud_common.h"\n'
                                 'extern "C" void entries(const int* rho, int n, int rows, int ss, int* out) {\n'
                                 '  for (int i = 0; i < n; ++i) out[i] = laud::list_entry(rho[i], rows, 1.f / ss);\n}\n')
    hipcc("--cuda-host-only", "-shared", str(d / "rules.hip"), "-o", str(d / "rules.so"))
    return C.CDLL(str(d / "rules.so"))


@pytest.mark.parametrize("S", [1, 2, 3, 4, 7, 8, 14, 56])
@pytest.mark.parametrize("count", [1, 2, 3, 63, 64, 65, 1000, 18725])
def test_rows_past_the_end_of_an_index_list_stay_inside_it(rules, S, count):
    """A list of exactly `count` entries: the rows of the last tiles (up to 128 rows, one tile looked ahead) read none past it."""
    rows = min(count * S * S, 1 << 21) // (S * S) * S * S
    if rows == 0:
        pytest.skip("more rows than the kernels take")
    rho = np.unique(np.concatenate([np.arange(min(rows, 5000)), np.arange(max(rows - 5000, 0), rows + 256), np.arange(0, rows, 997)])).astype(np.int32)
    out = np.empty_like(rho)
    ptr = lambda a: a.ctypes.data_as(C.c_void_p)  # noqa: E731
    rules.entries(ptr(rho), len(rho), rows, S * S, ptr(out))
    assert np.array_equal(out, np.minimum(rho, rows - 1) // (S * S))


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    """Lines of a kernel source's generated code."""
    d, made = tmp_path_factory.mktemp("assembly"), {}

    def lines(name):
        if name not in made:
            hipcc("--cuda-device-only", "-S", os.path.join(B.CSRC, name), "-o", str(d / (name + ".s")))
            made[name] = (d / (name + ".s")).read_text().splitlines()
        return made[name]
    return lines


@pytest.mark.parametrize("name,least", [("laud_narrow.hip", 2 * 12), ("laud_first.hip", 17)])
def test_lds_reads_have_landed_at_the_barriers_of_the_64_wide_kernels(assembly, name, least):
    """LDS that a wave has read is refilled by another wave's LDS-direct loads right behind a barrier, so no wave may pass a barrier
    with LDS reads under way: in the generated code every ds_read is waited for (lgkmcnt counts down in order) before the next
    s_barrier."""
    barriers, pending = 0, []
    for line in assembly(name):
        op = line.split()[:1]
        if not op:
            continue
        if op[0].startswith("ds_read") or op[0].startswith("ds_load"):
            pending.append(line.strip())
        elif op[0] == "s_waitcnt" and "lgkmcnt(" in line:
            left = int(line.split("lgkmcnt(")[1].split(")")[0])
            pending = pending[-left:] if left else []
        elif op[0] == "s_barrier":
            barriers += 1
            assert not pending, f"barrier {barriers} is passed with {pending} under way"
    assert barriers >= least


def test_stores_behind_the_input_that_the_whole_block_kernel_waits_for(assembly):
    """The kernel of the static first block waits for the next but one rectangle's input with "all but sixteen": in the generated code of
    its loop six LDS-direct loads and, behind them, sixteen stores are all that counts, none of them on a branch."""
    loop, loops, header = [], {}, None
    for line in assembly("laud_first.hip"):  # the code of each loop, in the order it stands in
        at = re.search(r"(?:in Loop: |=>This Inner Loop )Header[:=] ?(?:(BB\w+) )?Depth=1", line)
        if at:
            header = at.group(1) or line.split(":")[0].strip(". ").lstrip("L")
        elif re.match(r"\.LBB|; %bb", line):
            header = None
        if header:
            loops.setdefault(header, []).append(line.strip())
    loop, = (v for v in loops.values() if any("vmcnt(16)" in t for t in v))
    wait, = (i for i, t in enumerate(loop) if "vmcnt(16)" in t)
    skipped, order = None, []
    for t in loop[wait + 1:] + loop[:wait]:
        branch = re.match(r"s_cbranch_\w+ \.L(BB\w+)", t)
        if re.match(r"\.LBB", t):
            skipped = None
        elif branch and "=>" not in t:
            skipped = branch.group(1)
        memory = re.match(r"(buffer_|global_|flat_|scratch_)\w+", t)
        if memory:
            assert skipped is None or skipped not in " ".join(loop), (t, skipped)
            order.append("load" if "lds" in t else "store" if "store" in t else t)
    assert order == ["load"] * 6 + ["store"] * 16, order


def test_pooling_loads_of_a_batch_are_under_way_together(assembly):
    """The channel masker's pooling: in the generated code eight (bf16) and four (float32) 16-byte loads follow each other without
    a wait."""
    most = {}
    for line in assembly("laud_chanmask.hip"):
        if re.match(r"_ZN.*k_gap_partial.*:", line):
            name, run = line.split(":")[0], 0
            most[name] = 0
        elif most and ("vmcnt(" in line or "s_endpgm" in line):
            run = 0
        elif most and line.split()[:1] == ["global_load_dwordx4"]:
            run += 1
            most[name] = max(most[name], run)
    assert len(most) == 2 and all(v >= (8 if "ItE" in k else 4) for k, v in most.items()), most


@pytest.mark.parametrize("name", ["laud_first.hip", "laud_tail.hip"])
def test_wide_buffer_stores_have_no_scalar_offset(assembly, name):
    """A buffer store of more than 8 bytes reads its data registers over several cycles.  The compiler keeps the next vector instruction
    from writing them too early, but not where the store has a scalar register for an offset: there the first register was found
    overwritten.  In the generated code of the kernels with buffer stores none has one."""
    stores = [t.split(",") for t in assembly(name) if re.match(r"\s*buffer_store_dwordx[34]\b", t)]
    assert all(re.match(r"\s*(0|off|-?\d+)\b(?! *:)", t[3]) for t in stores), [t for t in stores if re.match(r"\s*s\d", t[3])]
    named = "raw_buffer_store" in open(os.path.join(B.CSRC, name)).read()
    assert bool(stores) == named


def test_no_inline_assembly_load_writes_a_register():
    """The compiler takes an asm statement's outputs as written when it ends and may copy or re-use them while the load is still
    under way.  Loads into registers are builtins, whose waits it places itself; asm loads go to LDS (no output operand)."""
    for name in sorted(os.listdir(B.CSRC)):
        if not name.endswith((".h", ".hip")):
            continue
        with open(os.path.join(B.CSRC, name)) as f:
            text = f.read()
        for at in re.finditer(r"\basm\b[^;]*?\(", text):
            body = text[at.end():text.index(");", at.end())]
            outputs = body.split(":")[1] if ":" in body else ""
            assert not ("load" in body and "=" in outputs), (name, body)


def test_lds_direct_loads_meet_no_static_lds():
    """LDS-direct loads take offsets from the start of the workgroup's LDS, where the dynamic part begins only in a kernel that
    has no static one."""
    for name in sorted(os.listdir(B.CSRC)):
        if name.endswith((".h", ".hip")):
            with open(os.path.join(B.CSRC, name)) as f:
                text = re.sub(r"//.*", "", f.read())
            if re.search(r"\bdma(4|16)\(", text) and name not in ("laud_tile_util.h", "laud_static.hip"):
                assert not re.search(r"(?<!extern )__shared__", text), name


@pytest.mark.parametrize("mode,builds", [("M_SD1", True), ("M_DENSE1", False)])
def test_masker_projection_and_two_k_groups_do_not_build_together(tmp_path, mode, builds):
    """The exchange between two groups of waves that share the K steps lies over the partial sums of the masker projection, with no barrier
    between: the tiled kernel refuses the combination."""
    (tmp_path / "tile.hip").write_text('#include "laud_pipe.h"\n'
                                       f"template __global__ void laud::k_pipe<laud::{mode}, laud::bf16_t, 64, 128, 2, 2, 2, 6>(const laud::PipeArgs);\n")
    made = subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *B.FLAGS, "--cuda-device-only", "-fsyntax-only", str(tmp_path / "tile.hip")],
                          capture_output=True, text=True)
    assert (made.returncode == 0) == builds, made.stderr
    assert builds or "partial sums" in made.stderr, made.stderr
