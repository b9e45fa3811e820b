"""The calls that return to the automatic launches check their handle."""


def test_null_handles():
    from paper_1710_06423_amd import build, sacx
    import os
    if not os.path.exists(sacx.LIB_PATH):
        build.build()
    lib = sacx.load_library()
    assert lib.sacx_set_launch_auto(None) == sacx.EINVAL
    assert lib.sacx_batch_set_tiles_auto(None) == sacx.EINVAL
