"""Index arithmetic of the fp32 attention path at the largest shapes a call can have.  It is plain integer code that the
kernel and its launch share with the host programs under tests/host/, so it is checked there, without a GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def run_host(name, tmp_path, link=(), args=()):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("hipcc not found")
    exe = str(tmp_path / name)
    for cmd in ([hipcc, "--offload-host-only", "-O1", "-std=c++17", "-I" + os.path.join(ROOT, "include"),
                 "-I" + os.path.join(ROOT, "paper_2605_23163_amd", "csrc"), "-x", "hip",
                 os.path.join(ROOT, "tests", "host", name + ".cpp"), "-o", exe, *link], [exe, *args]):
        p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        assert p.returncode == 0, " ".join(cmd) + "\n" + p.stdout[-4000:]
    return p.stdout


def test_key_tiles_are_cut_without_overflow(tmp_path):
    assert "key cut: ok" in run_host("key_cut_main", tmp_path)


def test_launch_stays_below_2_to_the_32_work_items(tmp_path):
    assert "launch grid: ok" in run_host("launch_grid_main", tmp_path)


def test_long_calls_of_one_row_tile_are_cut():
    # one or two row tiles and keys for up to 64 pieces, the most there are (L = 8100: exactly 64): such a call is never left whole
    import ctypes as C

    import paper_2605_23163_amd.binding as b
    lib = b.load_library()
    for Hq, Hkv, D in ((4, 1, 64), (2, 2, 128)):
        for L in list(range(4000, 17000, 57)) + [8100, 16200]:
            p = b.AttnParams()
            p.N, p.B, p.L, p.Hq, p.Hkv, p.D, p.dtype = 1, 8, L, Hq, Hkv, D, b.FDD_F32
            need = lib.fdd_block_attn_workspace(C.byref(p))
            assert need > 0, (L, Hq, Hkv, D)


def test_unusual_scales_take_the_32_row_tiles():
    # (which need less scratch; 0 is the usual scale)
    import ctypes as C

    import paper_2605_23163_amd.binding as b
    lib = b.load_library()
    p = b.AttnParams()
    p.N, p.B, p.L, p.Hq, p.Hkv, p.D, p.dtype = 8, 32, 4096, 28, 4, 128, b.FDD_F32

    def need(scale):
        p.scale = scale
        return lib.fdd_block_attn_workspace(C.byref(p))
    assert need(0.0) > 0
    for scale in (-1.0, 2.0 ** -30, 0.1, 1.0, 2.0 ** 10):
        assert need(scale) == need(0.0), scale
    for scale in (2.0 ** -31, 1e-40, 1025.0, 3e38, float("inf")):
        assert need(scale) == 0, scale


def test_tiles_of_16_rows_are_taken_up_to_128_workgroups_of_32():
    # (the partial results say which: 5 rows beyond whole tiles of 32 are padded to 16 or to 32)
    import ctypes as C

    import paper_2605_23163_amd.binding as b
    lib = b.load_library()
    up = lambda n: (n + 255) // 256 * 256
    for D in (64, 128):
        for tiles, splits in ((1, 2), (1, 64), (2, 64), (32, 4), (33, 4), (43, 3), (42, 3), (64, 2), (65, 2), (200, 2)):
            p = b.AttnParams()
            p.N, p.B, p.L, p.Hq, p.Hkv, p.D, p.dtype, p.splits = 1, 32 * (tiles - 1) + 5, 20000, 1, 1, D, b.FDD_F32, splits
            rows = tiles * 32 - (16 if tiles * splits <= 128 else 0)
            assert lib.fdd_block_attn_workspace(C.byref(p)) == up(rows * splits * D * 4) + up(rows * splits * 8), (tiles, splits, D)
