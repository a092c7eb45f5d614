"""The tuning key "panel" reaches every kernel whose tiles are dealt in column panels, the 64 x 128 tiles of few rows among them."""
import host_dispatch as D


def test_panel_reaches_the_64_x_128_tiles():
    L, whole = D.lib(), D.lib().lcma_split_group_scratch_bytes()
    try:
        for value, few, many in ((b"2", 2, 2), (b"", 8, 8)):
            assert L.lcma_set_tuning(b"panel", value) == 0
            assert D.gemm_nt_ws(500, 4096, 1024, "bf16", whole)[1][0].endswith(" deep=1")    # up to 1024 rows: launched with the few rows
            assert L.dispatch_panel() == few
            assert D.gemm_nt_ws(1025, 1400, 1088, "bf16", whole)[1][0].endswith(" dealt=5")  # the same tiles beyond
            assert L.dispatch_panel() == (many if value else 8)
    finally:
        L.lcma_set_tuning(b"panel", b"")
