"""The compiler options of the HIP sources, for every file: the attention
kernel finds masked scores that are not finite by the NaN they give, so none
may let the compiler assume that there is no NaN or infinity; and packed fp32
instructions stay out of device code."""
import importlib.util
import os

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
