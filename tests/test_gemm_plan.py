"""Which kernel a GEMM with about one or two 128x128 tiles per CU takes (256 CUs): the edges of the rule."""
import pytest

import paper_1905_12334_amd as mp8

S2, S4, WAVES, SMALL = "128x128x128s2", "128x128x128s4", "128x128x128p", "64x64x128s2"


@pytest.mark.parametrize("tiles,stages,layouts,kernel", [
    ((12, 16), 15, "all", S2), ((12, 16), 16, "all", S4), ((14, 16), 16, "all", S4), ((15, 15), 16, "all", S2),
    ((16, 16), 23, "all", S2), ((16, 16), 24, "all", S4), ((16, 16), 63, "all", S4), ((16, 16), 64, "all", WAVES),
    ((257, 1), 24, "all", S2), ((257, 1), 64, "all", S2), ((32, 16), 127, "all", S2), ((28, 16), 128, "bt", WAVES),
    ((28, 16), 128, "tn", S2), ((27, 16), 128, "all", S2),
    ((16, 8), 47, "tn", SMALL), ((16, 8), 48, "tn", S4), ((18, 8), 31, "tn", SMALL), ((18, 8), 32, "tn", S4),
    ((18, 8), 64, "tn", S4), ((18, 8), 65, "tn", WAVES), ((18, 8), 32, "bt", SMALL)])
def test_plan_of_one_and_two_rounds(tiles, stages, layouts, kernel):
    flags = {"all": (0, mp8.FLAG_B_CONTRACTION_MAJOR, mp8.FLAG_CONTRACTION_MAJOR), "tn": (mp8.FLAG_CONTRACTION_MAJOR,),
             "bt": (mp8.FLAG_B_CONTRACTION_MAJOR,)}[layouts]
    for f in flags:
        assert mp8.gemm_fp8_plan(mp8.FWD, 128 * tiles[0], 128 * tiles[1], 128 * stages, f) == (kernel, 1)


def test_workspace_query_covers_operands_of_any_alignment():
    """200 tiles of 64x64 and 64 whole stages: unsplit on aligned operands, two slices on others."""
    rows, cols, kc = 64 * 20, 64 * 10, 8192
    assert mp8.gemm_fp8_plan(mp8.FWD, rows, cols, kc)[1] == 1
    assert mp8.gemm_fp8_workspace_bytes(mp8.FWD, rows, cols, kc) >= 2 * 4 * rows * cols
