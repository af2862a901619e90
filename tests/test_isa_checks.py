"""Checks on the generated gfx950 code of the kernels that fill LDS from inline assembly (no GPU needed: hipcc
cross-compiles).  The buffer resource of such a load has to sit in scalar registers and the hot loops must not touch
scratch memory; a source change that looks harmless can lose either (a descriptor chosen by a run-time index ends up in
vector registers and in scratch), and nothing at run time reports it."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2108_01624_amd", "csrc")


def _hipcc():
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    return None


def _isa(src, tmp_path):
    hipcc = _hipcc()
    if hipcc is None:
        pytest.skip("hipcc not found")
    from paper_2108_01624_amd.build import HIPCC_FLAGS

    out = tmp_path / (src + ".s")
    flags = [f for f in HIPCC_FLAGS if f != "-fPIC"]
    r = subprocess.run([hipcc] + flags + ["--cuda-device-only", "-S", os.path.join(CSRC, src), "-o", str(out)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return out.read_text()


def _kernels(text):
    """name -> (body, metadata block) for every kernel of the translation unit."""
    out = {}
    for m in re.finditer(r"\.amdhsa_kernel (\S+)(.*?)\.end_amdhsa_kernel", text, re.S):
        name, meta = m.group(1), m.group(2)
        start = text.find("\n" + name + ":")
        end = text.find("s_endpgm", start)
        out[name] = (text[start:end], meta)
    return out


@pytest.mark.parametrize("src,hot", [("dp_gram.hip", ("gram_dma_kernel", "gram_units_kernel", "gram_small_dma_kernel")),
                                     ("dp_wgemm.hip", ("wgemm_dma16_kernel",))])
def test_lds_filling_kernels_keep_descriptors_scalar_and_use_no_scratch(src, hot, tmp_path):
    kernels = _kernels(_isa(src, tmp_path))
    seen = 0
    for name, (body, meta) in kernels.items():
        if not any(h in name for h in hot):
            continue
        seen += 1
        scratch = int(re.search(r"\.amdhsa_private_segment_fixed_size (\d+)", meta).group(1))
        assert scratch == 0, f"{name} uses {scratch} bytes of scratch per lane"
        assert "scratch_" not in body, f"{name} has scratch instructions"
        loads = re.findall(r"buffer_load_dwordx4 (\S+), (\S+), (\S+) offen(?: nt)? lds", body)
        assert loads, f"{name}: no LDS-filling loads found"
        for vaddr, rsrc, soff in loads:
            assert vaddr.startswith("v") and rsrc.startswith("s[") and soff.startswith("s"), (name, vaddr, rsrc, soff)
        assert "v_pk_mul_f32" not in body and "v_pk_fma_f32" not in body and "v_pk_add_f32" not in body, name
    assert seen >= len(hot) and all(any(h in name for name in kernels) for h in hot)


def test_range_checked_accesses_have_no_scalar_offset(tmp_path):
    """The grouping of the ids and the segment sums leave what lies past an array to the range check of its buffer resource, which
    covers the vector and the immediate offset of an access and not the scalar one."""
    kernels = _kernels(_isa("dp_rowwise.hip", tmp_path))
    for hot in ("group_ids_kernel", "segment_sums_kernel"):
        bodies = {name: body for name, (body, _) in kernels.items() if hot in name}
        assert bodies
        for name, body in bodies.items():
            accesses = re.findall(r"buffer_(?:load|store)_\w+ [^,]+, [^,]+, s\[\d+:\d+\], (\S+)", body)
            assert accesses and set(accesses) == {"0"}, (name, sorted(set(accesses)))


def test_stages_past_the_end_have_a_resource_without_bytes(tmp_path):
    """The eight-wave Gram kernel goes on issuing loads past its last stage: what keeps them from memory is a resource of no bytes, not a
    scalar offset past every tensor, which the range check does not cover."""
    kernels = _kernels(_isa("dp_gram.hip", tmp_path))
    bodies = {name: body for name, (body, _) in kernels.items() if "gram_dma_kernel" in name}
    assert bodies
    for name, body in bodies.items():
        assert not re.search(r"0x7ffffff0|0x7fffffff|\b2147483632\b", body), name
