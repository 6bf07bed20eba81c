"""The compiler options of the HIP sources, for every file: the attention
kernel finds masked scores that are not finite by the NaN they give, so none
may let the compiler assume that there is no NaN or infinity; and packed fp32
instructions stay out of device code."""
import importlib.util
import os
import re
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def _builder():
    path = os.path.join(os.path.dirname(HERE), "paper_2609_25869_amd", "build.py")
    spec = importlib.util.spec_from_file_location("_flags_of_build", path)
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def test_no_option_assumes_finite_numbers():
    b = _builder()
    for src in b.SOURCES:
        flags = b.common_flags() + b.EXTRA_FLAGS.get(src, [])
        for f in ("-ffast-math", "-Ofast", "-fno-honor-nans", "-fno-honor-infinities", "-ffinite-math-only"):
            assert f not in flags, (src, f)
        assert "-packed-fp32-ops" in flags, src


def test_attention_kernels_keep_their_state_in_registers(tmp_path):
    """No attention kernel uses scratch memory: what one spills it reads again
    in every tile that needs masking."""
    b = _builder()
    try:
        cc = b.hipcc()
    except RuntimeError:
        pytest.skip("hipcc not available")
    out = str(tmp_path / "attn.s")
    subprocess.check_call([cc] + b.common_flags() + b.EXTRA_FLAGS["attn_fwd.hip"] +
                          ["--offload-device-only", "-S", os.path.join(b.CSRC, "attn_fwd.hip"), "-o", out],
                          stderr=subprocess.DEVNULL)
    text = open(out).read()
    text = text[text.index("amdhsa.kernels:"):]
    names = re.findall(r"\.name:\s+(\S+)", text)
    sizes = [int(x) for x in re.findall(r"\.private_segment_fixed_size:\s+(\d+)", text)]
    kernels = [n for n in names if "kernel" in n]
    assert len(kernels) == len(sizes) and len(kernels) >= 13
    assert not any(sizes), dict(zip(kernels, sizes))
