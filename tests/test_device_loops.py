"""What the block loops of the persistent kernels hold, read from the gfx950 assembly of
kernels built here: work that a condition drops at one of the shapes shows as missing
instructions, and no call of one block per workgroup would notice.
"""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SF_SHAPES = [(64, 32), (128, 32), (128, 64)]  # (C, M) of the slice-state pass 2


@pytest.fixture(scope="module")
def sf_assembly(tmp_path_factory):
    """{(C, M): lines of k_deslice_sf<C, M>}"""
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    import importlib.util
    spec = importlib.util.spec_from_file_location("ts3_build", os.path.join(ROOT, "paper_2602_04940_amd", "build.py"))
    build = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(build)
    d = tmp_path_factory.mktemp("sf")
    src, out = d / "sf.hip", d / "sf.s"
    args = ("const bf16_t *, int64_t, const bf16_t *, const float *, const bf16_t *, const bf16_t *, const float *, "
            "bf16_t *")
    src.write_text(f'#include "{os.path.dirname(build.SRC)}/ts3_pass2sf.h"\nnamespace ts3 {{\n' + "".join(
        f"template __global__ void k_deslice_sf<{c}, {m}>({args});\n" for c, m in SF_SHAPES) + "}\n")
    flags = [f for f in build.HIP_FLAGS if f not in ("-shared", "-fPIC")]
    r = subprocess.run([hipcc, *flags, "--cuda-device-only", "-S", "-o", str(out), str(src)], capture_output=True,
                       text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    lines = out.read_text().split("\n")
    kernels = {}
    for c, m in SF_SHAPES:
        at = next(i for i, l in enumerate(lines) if re.match(rf"^_Z\w*k_deslice_sfILi{c}ELi{m}E\w*:", l))
        end = next(i for i in range(at, len(lines)) if lines[i].startswith(".Lfunc_end"))
        kernels[c, m] = lines[at:end]
    return kernels


def block_loop(lines, stores):
    """(first, last) line of the innermost loop with matrix products and at least `stores` stores of rows."""
    labels = {m.group(1): i for i, l in enumerate(lines) if (m := re.match(r"^(\.LBB\w+):", l))}
    loops = [(labels[m.group(1)], i) for i, l in enumerate(lines)
             if (m := re.search(r"s_c?branch\w*\s+(\.LBB\w+)", l)) and labels[m.group(1)] < i]
    fits = [(a, b) for a, b in loops if any("v_mfma" in l for l in lines[a:b]) and
            sum("global_store_dwordx4" in l for l in lines[a:b]) >= stores]
    return min(fits, key=lambda ab: ab[1] - ab[0])


@pytest.mark.parametrize("C,M", SF_SHAPES)
def test_slice_state_decoder_loads_the_next_blocks_rows(sf_assembly, C, M):
    """Per 32 points: C/16 fragments of x (two tiles of C/32 K steps), (C/32)(C/16) of W3^T, and C/16 stores."""
    lines = sf_assembly[C, M]
    a, b = block_loop(lines, C // 16)
    loads = sum("global_load_dwordx4" in l for l in lines[a:b])
    assert loads == (C // 32) * (C // 16) + C // 16


@pytest.mark.parametrize("C,M", SF_SHAPES)
def test_slice_state_decoder_waits_before_blocks_are_redone(sf_assembly, C, M):
    """Waves past the end of a ragged block write the last row as computed by the unshifted
    softmax; the wave that owns it may write it again only after them: a wait for the
    stores and a barrier lie between the block loop and the products of the redone blocks."""
    lines = sf_assembly[C, M]
    _, b = block_loop(lines, C // 16)
    redo = next(i for i in range(b, len(lines)) if "v_mfma" in lines[i])
    barrier = [i for i in range(b, redo) if "s_barrier" in lines[i]]
    assert barrier
    assert any("vmcnt(0)" in l for l in lines[b:barrier[0]])
