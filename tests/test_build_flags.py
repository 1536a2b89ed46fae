"""How the library is compiled."""
from paper_1907_08467_amd import build_lib


def test_no_hidden_code_generation_options():
    """Only documented compiler options: -mllvm ones change the code generator in
    ways that nothing promises (one left wave-uniform branches wrong)."""
    assert "-mllvm" not in build_lib.FLAGS


def test_no_packed_f32():
    flags = " ".join(build_lib.FLAGS)
    assert "-Xclang -target-feature -Xclang -packed-fp32-ops" in flags
