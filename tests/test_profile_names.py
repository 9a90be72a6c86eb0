"""The indices of the profile's phases: each keeps the name that programs know it by."""
import paper_2602_02549_amd as oz

NAMES = ["init", "absmax_A", "absmax_B", "bar_A", "bar_B", "gemm_scale", "shifts", "residue_A",
         "residue_B", "gemm_residue", "crt", "plan", "batched", "scan", "residues"]


def test_profile_names():
    names = [oz.lib().ozaki2_profile_name(i).decode() for i in range(-1, len(NAMES) + 1)]
    assert names == [""] + NAMES + [""]
