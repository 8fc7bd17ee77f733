"""Index and size rules of the launches (csrc/rules.h), checked by the host compiler: every
expression below is a constant expression, in which an overflow does not compile."""
import os
import re
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2108_02054_amd", "csrc")


def holds(lines, tmp_path):
    """None if every constant expression holds, else the compiler's first error."""
    src = tmp_path / "rules.cpp"
    src.write_text('#include "rules.h"\nusing namespace amgmi;\n'
                   + "\n".join(f"static_assert({x}, \"\");" for x in lines) + "\n")
    r = subprocess.run(["g++", "-std=c++17", "-fsyntax-only", "-I", CSRC, str(src)], capture_output=True, text=True)
    return None if r.returncode == 0 else r.stderr


def test_lane_rows_of_the_largest_systems(tmp_path):
    """The rows of a 7-point operator of 2^31 - 1 entries with eight lanes each, and of every
    number of lanes at the most rows whose threads a launch can count."""
    lines = []
    for lanes in (1, 4, 8, 16, 32, 64, 128, 256):
        most = min(2**31 - 257, (2**32 - 1024) // lanes)
        for row in {0, 1, 2**31 // 7 // lanes, 2**31 // lanes - 1, 2**31 // lanes, most - 1}:
            if row > most - 1:
                continue
            block, first = divmod(row, 256 // lanes)
            for lane in {0, lanes - 1}:
                lines.append(f"lane_row({block}, 256, {first * lanes + lane}, {lanes}) == {row}")
    lines.append(f"lane_row({(2**31 // 7) // 32}, 256, 255, 8) >= {2**31 // 7 - 32}")
    assert holds(lines, tmp_path) is None


def test_former_index_leaves_32_bits(tmp_path):
    """The check can fail: the thread's number in the whole grid does not fit."""
    row = 2**28
    assert holds([f"({row // 32} * 256 + 0) / 8 == {row}"], tmp_path) is not None


def test_rows_that_fit_one_launch(tmp_path):
    assert holds(["lanes_fit_grid(1ll << 28, 8)", "lanes_fit_grid((1ll << 29) - 128, 8)",
                  "!lanes_fit_grid(1ll << 29, 8)", "lanes_fit_grid(2147483647ll, 1)"], tmp_path) is None


def test_setup_kernels_use_the_rule():
    """No kernel of the setup divides the thread's number in the whole grid."""
    for name in ("kernels_setup.hip", "kernels_symbolic.hip"):
        text = open(os.path.join(CSRC, name)).read()
        assert not re.search(r"\*\s*\(?(int64_t\))?\s*TPB\s*\+\s*(\(int\))?threadIdx\.x\)\s*(/|>>)", text), name


def test_owner_form_fits_its_lds(tmp_path):
    """Rows of every width that the owner form takes (8 to 248 columns, padded to multiples of
    8), in FP64 and FP32: two workgroups fit a CU's 160 KiB."""
    lines = ["2 * OWN_SMEM_MAX <= 160 * 1024", "own_smem(64, 128, 8, 8) == 66048"]
    for w in range(8, 249, 8):
        lanes = next(g for g in (8, 16, 32, 64) if g >= w or g == 64)
        lines.append(f"own_entries({w}) == {8 if w <= 128 else 4}")  # four positions per lane: four entries
        for size in (4, 8):
            lines.append(f"own_smem({lanes}, {w}, own_entries({w}), {size}) <= OWN_SMEM_MAX")
    assert holds(lines, tmp_path) is None
    assert holds(["own_smem(64, 136, 8, 8) <= 65536"], tmp_path) is not None


def test_window_reads_half_above_the_caches(tmp_path):
    """27 diagonals: all read up to 51^3 rows in FP64 and 63^3 in FP32, half of a symmetric
    operator's from 52^3 and 65^3 on; the products leave 32 bits."""
    lines = []
    for bytes_, last, first in ((8, 51, 52), (4, 63, 65)):
        lines += [f"!window_reads_half({last**3}, 27, {bytes_})", f"window_reads_half({first**3}, 27, {bytes_})",
                  f"window_reads_half({2**31 // 27}, 27, {bytes_})"]
    lines += ["!window_reads_half(135926, 27, 8)", "window_reads_half(135927, 27, 8)"]
    assert holds(lines, tmp_path) is None
