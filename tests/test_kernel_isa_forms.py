"""The static checks of the persistent kernels' code on the kernels beside them
that loop over tiles or blocks: the escape-time sweep, the wide and fed n-body
kernels and the binomial payload's call form. Barriers only in loops with uniform
exits, no packed FP32, no scratch memory (CPU only: hipcc cross-compiles)."""
import os
import re
import subprocess

import pytest

from test_kernel_isa import CSRC, HIPCC, _blocks, _functions

# source file -> (kernel name fragment, number of instantiations)
FORMS = {"kernels.hip": (("k_sweep_escape", 1), ("k_wide", 4), ("k_feed", 4), ("k_bare", 7)),
         "binomial_call.hip": (("k_persistent", 1), ("k_bare", 1))}


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("isa")
    texts = {}
    for src in FORMS:
        out = d / (src + ".s")
        subprocess.run([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-ffp-contract=off", "-Xclang",
                        "-target-feature", "-Xclang", "-packed-fp32-ops", "--cuda-device-only", "-S", "-o", str(out),
                        os.path.join(CSRC, src)], check=True, capture_output=True)
        texts[src] = out.read_text()
    return texts


def _resources(text):
    """kernel name -> its code object directives that are numbers."""
    return {m.group(1): {k: int(v) for k, v in re.findall(r"\.amdhsa_(\w+) (\d+)$", m.group(2), flags=re.M)}
            for m in re.finditer(r"\.amdhsa_kernel (\S+)\n(.*?)\.end_amdhsa_kernel", text, flags=re.S)}


@pytest.mark.parametrize("src", sorted(FORMS))
def test_forms_have_uniform_exits_around_barriers(asm, src):
    for frag, count in FORMS[src]:
        funcs = {k: v for k, v in _functions(asm[src]).items() if frag in k}
        assert len(funcs) == count, (frag, sorted(funcs))
        for name, body in funcs.items():
            blocks = _blocks(body)
            barrier_loops = {hdr for _, hdr, lines in blocks if hdr and any(x.startswith("s_barrier") for x in lines)}
            for label, hdr, lines in blocks:
                if hdr in barrier_loops:
                    bad = re.search(r"s_andn2_b64 exec, exec, s\[\d+:\d+\]\s*\n\s*s_cbranch_execz", "\n".join(lines))
                    assert not bad, f"{name}: loop {hdr} holds a barrier and a per-lane exit in {label}"


@pytest.mark.parametrize("src", sorted(FORMS))
def test_forms_use_no_packed_fp32_and_no_scratch(asm, src):
    for name, body in _functions(asm[src]).items():
        for op in ("v_pk_fma_f32", "v_pk_mul_f32", "v_pk_add_f32", "scratch_store", "scratch_load"):
            assert op not in body, (name, op)
    private = {k: v["private_segment_fixed_size"] for k, v in _resources(asm[src]).items()}
    for frag, count in FORMS[src]:
        assert [v for k, v in private.items() if frag in k] == [0] * count, (frag, private)


def test_call_form_keeps_two_workgroups_per_compute_unit(asm):
    """256 registers and 80 KB of LDS at most: the two waves per SIMD that its
    measured rate needs."""
    call = next(v for k, v in _resources(asm["binomial_call.hip"]).items() if "k_persistent" in k)
    assert call["next_free_vgpr"] <= 256
    assert call["group_segment_fixed_size"] <= 80 * 1024
