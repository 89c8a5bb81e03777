"""Kernel names as rocprofv3 gives them, mangled or not, as bench.py's summaries print them: names with
digits, template arguments that are types, flags or both, and none."""
import importlib.util
from pathlib import Path

import pytest

spec = importlib.util.spec_from_file_location("bench", Path(__file__).resolve().parents[1] / "bench.py")
bench = importlib.util.module_from_spec(spec)
spec.loader.exec_module(bench)


@pytest.mark.parametrize("name, want", [
    ("_ZN6stitch12_GLOBAL__N_15k_pyrIDF16_Lb1EEEvPKNS_7PyrItemEiiNS_9FrameArgsE", "k_pyr<_Float16, true>"),
    ("_ZN6stitch12_GLOBAL__N_112k_expand_subIfEEvPKT_llPS2_lliiiiS4_lliiiiii", "k_expand_sub<float>"),
    ("_ZN12_GLOBAL__N_110k_vreduce0ILb0ELb1EEEvNS_11Reduce0ArgsE", "k_vreduce0<false, true>"),
    ("_ZN12_GLOBAL__N_16k_vdg0ILb1EEEvNS_7Dg0ArgsE", "k_vdg0<true>"),
    ("_ZN12_GLOBAL__N_17k_vsrcTILb0EEEvNS_7SrcArgsEPi", "k_vsrcT<false>"),
    ("_ZN12_GLOBAL__N_17k_vpanoENS_8PanoArgsE", "k_vpano"),
    ("void stitch::(anonymous namespace)::k_level0<_Float16, true>(void const*, long)", "k_level0<_Float16, true>"),
    ("void (anonymous namespace)::k_vsrcT<false>((anonymous namespace)::SrcArgs, int*)", "k_vsrcT<false>"),
])
def test_short_names(name, want):
    assert bench._short_kernel(name) == want
