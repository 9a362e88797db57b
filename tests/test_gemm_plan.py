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


LARGE = "256x256x128s2"
LAYOUTS = (0, mp8.FLAG_B_CONTRACTION_MAJOR, mp8.FLAG_CONTRACTION_MAJOR)


# more 256x256 tiles than CUs: columns and rows that fill them, or are mostly not there; rounds of 512 tiles of 128x128 for a round of 256 of them
@pytest.mark.parametrize("rows,cols,stages,large", [
    (25088, 1024, 3, True), (25088, 960, 3, True), (25088, 912, 3, True), (25088, 896, 3, False), (25088, 832, 16, False), (25088, 784, 4, False),
    (25088, 1152, 7, True), (16384, 4096, 4, True), (65536, 272, 3, False), (50000, 336, 6, False), (40000, 512, 4, False), (131072, 64, 4, False),
    (131072, 16, 3, False), (100352, 64, 16, False), (64, 131072, 3, False), (83200, 1024, 3, True), (57584, 784, 4, True), (38272, 1024, 3, False),
    (38400, 1536, 3, True)])
def test_plan_of_many_large_tiles(rows, cols, stages, large):
    """The plan names the tile that a call for codes to nearest alone takes, and with FLAG_SATURATE that of every other call."""
    for f in LAYOUTS:
        assert (mp8.gemm_fp8_plan(mp8.FWD, rows, cols, 128 * stages, f)[0] == LARGE) == large
        assert mp8.gemm_fp8_plan(mp8.FWD, rows, cols, 128 * stages, f | mp8.FLAG_SATURATE)[0] != LARGE


@pytest.mark.gpu
@pytest.mark.parametrize("rows,cols,kc", [(25088, 1024, 384), (25088, 896, 384), (131072, 64, 512), (65536, 272, 384), (4096, 4096, 1024), (16384, 4096, 256),
                                          (38400, 1536, 256)])
@pytest.mark.parametrize("layout", LAYOUTS)
def test_the_plan_is_the_kernel(rows, cols, kc, layout):
    """The call without a tile and the call with the tile that the plan names launch the same kernel; one with statistics that of
    the plan with FLAG_SATURATE."""
    import torch

    from captured import launches
    u8 = lambda n: torch.empty(n, dtype=torch.uint8, device="cuda")
    a, b, out, stats = u8(rows * kc), u8(cols * kc), u8(rows * cols), mp8.new_stats()
    names = mp8.gemm_tile_configs()
    for flags, kw in ((layout, {}), (layout | mp8.FLAG_SATURATE, dict(stats=stats))):
        tile = 1 + names.index(mp8.gemm_fp8_plan(mp8.FWD, rows, cols, kc, flags)[0])
        call = lambda t: launches(lambda: mp8.gemm_fp8(mp8.FWD, rows, cols, kc, a, b, out8=out, flags=layout, tile_config=t, **kw))
        assert call(0) == call(tile)
