"""Rules of the launchers that change no bits, or that kernels of other last bits hang on: shapes that were timed on both
sides stay on the one that was faster."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("rules") / "rules.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC",
                    "-I", os.path.join(ROOT, "paper_2605_14877_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "launch_rules.cpp"), "-o", lib], check=True)
    return ctypes.CDLL(lib)


@pytest.mark.parametrize("d,n_scales,blocks,fit,per_unit", [
    # one scale: 32 pairs x 400 rows, 64 x 256, 256 x 144, 32 x 144
    (128, 1, 800, 4, 4), (128, 1, 1024, 4, 4), (128, 1, 2304, 4, 3), (128, 1, 288, 4, 3),
    # the same behind so many scales that four do not fit: 64 pairs x 225 rows, 80 x 169, 104 x 144; 48 x 225, 80 x 196
    (128, 1, 960, 3, 2), (128, 1, 880, 3, 2), (128, 1, 936, 3, 2), (128, 1, 720, 3, 3), (128, 1, 1040, 3, 3), (128, 1, 800, 3, 3),
    (128, 1, 801, 3, 2), (128, 1, 1025, 3, 3),
    # all scales in one call: 16 pairs up to 400 rows, 40 pairs up to 276 and up to 300; many short workgroups behind the long ones
    (128, 8, 960, 4, 3), (128, 7, 1720, 4, 3), (128, 6, 1760, 4, 3), (128, 7, 2000, 4, 4), (128, 7, 4472, 4, 4), (128, 5, 13312, 4, 4),
    (128, 20, 4472, 3, 3), (128, 2, 7 * 256, 4, 3), (128, 2, 7 * 256 + 1, 4, 4), (128, 20, 960, 3, 3),
    # d = 64: 48 pairs x 603 rows, 48 x 635, 64 x 491, 64 x 507, 48 x 683; all scales of 40 pairs up to 276, of 48 up to 625
    (64, 1, 1824, 7, 7), (64, 1, 1920, 7, 6), (64, 1, 1984, 7, 6), (64, 1, 2048, 7, 6), (64, 1, 2064, 7, 7), (64, 1, 1984, 6, 6),
    (64, 1, 1984, 4, 4), (64, 7, 1720, 7, 7), (64, 8, 1984, 7, 7),
])
def test_workgroups_of_the_fp32_calibration_per_compute_unit(rules, d, n_scales, blocks, fit, per_unit):
    assert rules.calibration_f32_per_unit(d, n_scales, blocks, fit) == per_unit


@pytest.mark.parametrize("d,attend,copies,tiles,copiers", [
    # short walks, bf16 rows
    (128, 96, 192, 4, True), (128, 128, 256, 4, False), (128, 192, 270, 10, True), (128, 256, 360, 10, False), (128, 256, 512, 4, False),
    # long walks, 8-bit rows
    (128, 256, 208, 10, True), (128, 256, 378, 20, True), (128, 200, 480, 23, True), (128, 240, 456, 23, True), (128, 224, 304, 15, True),
    (128, 256, 320, 14, False), (128, 256, 333, 15, False), (128, 256, 480, 20, False), (128, 240, 960, 23, False),
    # long walks, d = 64
    (64, 160, 200, 8, True), (64, 240, 188, 16, True), (64, 256, 288, 14, False), (64, 256, 336, 15, False), (64, 240, 678, 31, False),
    (64, 256, 640, 39, False),
    # no update; one tile
    (128, 256, 0, 14, True), (64, 192, 0, 7, True), (128, 32, 0, 1, False), (128, 16, 15, 1, False), (128, 32, 0, 2, True),
])
def test_wavefronts_that_only_copy(rules, d, attend, copies, tiles, copiers):
    assert rules.copying_wavefronts(d, attend, copies, tiles) == copiers


@pytest.mark.parametrize("attend,update,tiles,two", [
    (256, 0, 39, True), (256, 284, 39, True), (256, 256, 20, True), (256, 148, 14, True), (256, 196, 15, True), (240, 324, 31, True),
    (240, 192, 18, True), (180, 675, 29, True), (180, 810, 36, True), (224, 328, 23, True), (192, 576, 23, True), (192, 384, 12, True), (160, 512, 31, True),
    (256, 288, 14, False), (256, 336, 15, False), (256, 768, 23, False), (240, 640, 16, False), (240, 480, 18, False),
    (240, 248, 12, False), (224, 448, 14, False), (256, 128, 8, False), (192, 0, 7, False), (240, 0, 7, False), (160, 0, 8, False),
])
def test_two_key_streams_at_head_dimension_64(rules, attend, update, tiles, two):
    assert rules.two_key_streams(64, attend, update, tiles) == two
    assert rules.two_key_streams(128, attend, update, tiles)
