"""CPU tests of the launch rules and of what a call is refused for: no call that
an earlier rule took may need a workspace it did not need, or exceed a grid."""
import ctypes
import os

import pytest


@pytest.fixture(scope="module")
def fx():
    import paper_2604_22242_amd as fx
    if not os.path.exists(fx.LIB_PATH):
        from paper_2604_22242_amd import build
        build.build()
    return fx


def test_thin_columns(fx):
    """One thread per column up to 64 bytes of it, and up to 32 rows where there
    are 16 columns per CU; a wave or more per column elsewhere."""
    def split(dt, rows, cols):
        return fx.fx_resolve_launch(fx.R_COLSUM, dt, (rows, cols))[3]

    elem = {fx.F32: 4, fx.F64: 8, fx.BF16: 2, fx.U32: 4}
    for dt, e in elem.items():
        assert split(dt, 64 // e, 10) == 0
        assert split(dt, 9, 1 << 20) == 0
        assert split(dt, 32, 1 << 12) == 0
        # a grid of a wave per column has no room for these
        for rows in (17, 32):
            assert split(dt, rows, (1 << 26) + 5) == 0
        assert split(dt, 33, 1 << 20) != 0
        assert split(dt, 64 // e + 1, 100) != 0
        assert fx.fx_workspace_bytes(fx.R_COLSUM, dt, (32, 1 << 20)) == 0


def test_column_chunks_of_the_caller(fx):
    """A split given alone is limited to a pass of the default block per chunk
    (512 threads, 256 for half storage, a vector each); the workspace covers a
    tape's 256 threads as well."""
    for dt, rows_per_pass, tape_pass in ((fx.F32, 2048, 1024), (fx.F64, 1024, 512), (fx.BF16, 2048, 2048)):
        for rows, chunks in ((100, 1), (rows_per_pass, 1), (rows_per_pass + 1, 2), (8 * rows_per_pass, 8),
                             (100 * rows_per_pass, 8)):
            cfg = (0, 0, 0, 8)
            assert fx.fx_resolve_launch(fx.R_COLSUM, dt, (rows, 1000), cfg)[3] == chunks, (dt, rows)
            most = min(8, -(-rows // tape_pass))
            need = 0 if most == 1 else 4096 + 1000 * most * 8
            assert fx.fx_workspace_bytes(fx.R_COLSUM, dt, (rows, 1000), cfg) == need, (dt, rows)
    # many columns, where a column alone takes fewer threads
    for rows in (305, 757):
        assert fx.fx_resolve_launch(fx.R_COLSUM, fx.F32, (rows, 5000), (0, 0, 0, 8))[3] == 1
        assert fx.fx_workspace_bytes(fx.R_COLSUM, fx.F32, (rows, 8158790), (0, 0, 0, 8)) == 0


def test_whole_columns(fx):
    """Columns are chunked where there are fewer than CUs and each is five passes
    of its block long (two of half storage and below 64 columns), or where half-storage columns are
    long and hardly more than one per CU; up to two per CU take 512 threads whole."""
    def launch(dt, rows, cols, cfg=(0, 0, 0, 0)):
        return fx.fx_resolve_launch(fx.R_COLSUM, dt, (rows, cols), cfg)

    for rows, cols in ((10000, 419), (20000, 400), (65536, 512), (65535, 256), (65536, 384)):
        assert launch(fx.BF16, rows, cols)[::3] == (512, 1), (rows, cols)
    # more columns, and the 256 threads that generated kernels start from
    for rows, cols in ((12000, 700), (16384, 700), (65536, 700)):
        assert launch(fx.BF16, rows, cols)[3] == 1, (rows, cols)
    for rows, cols in ((10000, 419), (65535, 300)):
        assert launch(fx.BF16, rows, cols, (256, 1, 0, 0))[3] == 1, (rows, cols)
    for rows, cols in ((65536, 256), (65536, 383), (65536, 255), (8192, 104)):
        assert launch(fx.BF16, rows, cols)[3] > 1, (rows, cols)
    for dt, passes in ((fx.F32, 512 * 4 * 2), (fx.F64, 512 * 2 * 2)):
        assert launch(dt, 5 * passes - 1, 104)[3] == 1
        assert launch(dt, 5 * passes, 104)[3] == 5
        assert launch(dt, 2 * passes - 1, 63)[3] == 1
        assert launch(dt, 2 * passes, 63)[3] > 1


FAKE = 0x10000
C2 = [("leaf", -1, -1, 0, 0.0), ("leaf", -1, -1, 1, 0.0), ("add", 0, 1, -1, 0.0)]


def test_static_scratch_takes_the_row_sums_it_took(fx):
    """64 chunks of 32767 rows and a counter per 256 of them fill 16 MiB; the finer
    counters that the tiles need do not count against it."""
    def refused(dt, rows, cols, cfg):
        # (a NULL input is found after the workspace: nothing is enqueued)
        L, tape = fx.lib(), fx.Tape(C2)
        arr = (ctypes.c_void_p * 2)(None, FAKE)
        c = ctypes.pointer(fx.Launch(*cfg)) if cfg else None
        return L.fx_tape_eval_static(tape.handle, dt, arr, 2, fx.Shape(rows, cols), fx.R_ROWSUM, FAKE, c,
                                     None) == 4 and "static scratch" in fx.fx_last_error()

    for dt in (fx.F32, fx.F64, fx.BF16):
        assert fx.fx_workspace_bytes(fx.R_ROWSUM, dt, (32767, 126)) == 16 << 20
        for cfg in (None, (256, 2, 0, 64), (256, 1, 8, 64)):
            assert not refused(dt, 32767, 126, cfg), (dt, cfg)
            assert refused(dt, 32768, 126, cfg), (dt, cfg)
