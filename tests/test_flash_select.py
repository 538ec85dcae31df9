"""Which bf16 calls take which block sizes of the streaming kernels, on the host: the rules are plain C++ (csrc/flash_select.h)."""
import os
import shutil
import subprocess

from tests import test_gpu_long_blocks as G

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2601_22275_amd", "csrc")


def _holds(tmp_path, *conditions):
    src = tmp_path / "select.cpp"
    src.write_text('#include "flash_select.h"\nusing namespace vm;\n' +
                   "".join(f"static_assert({c}, \"\");\n" for c in conditions))
    cxx = shutil.which("g++") or shutil.which("amdclang++") or "/opt/rocm/bin/amdclang++"
    r = subprocess.run([cxx, "-std=c++17", "-fsyntax-only", f"-I{CSRC}", str(src)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr


def test_rules_follow_the_device(tmp_path):
    """A device of half the units takes the choices of one of twice as many at half the problems."""
    conditions = []
    for frames, b in ((100, 300), (130, 1456), (252, 2048), (64, 1000), (512, 900)):
        for d in (64, 128):
            for v in ("false", "true"):
                conditions.append(f"update_short_blocks({d}, {v}, {frames}, {b}, 256) == update_short_blocks({d}, {v}, {frames} / 2, {b}, 128)")
        conditions.append(f"backward_short_blocks({frames}, {b}, 256) == backward_short_blocks({frames} / 2, {b}, 128)")
    conditions += ["whole_frame_tokens(128, true, 256, 256) == 192", "whole_frame_tokens(128, true, 257, 256) == 128",
                   "whole_frame_tokens(128, true, 128, 128) == 192", "whole_frame_tokens(128, true, 129, 128) == 128"]
    _holds(tmp_path, *conditions)


def test_the_choice_has_no_step_in_the_frame(tmp_path):
    """Launches of two full groups a unit, in frames of 256, 512, ... tokens: short blocks up to a length, long ones from there on, and
    one token more or less than 900, or a frame more, does not turn a choice that the neighbouring sizes share."""
    conditions = []
    for rule in ("update_short_blocks(64, true, 256, {b}, 256)", "update_short_blocks(128, false, 256, {b}, 256)",
                 "update_short_blocks(128, true, 256, {b}, 256)", "backward_short_blocks(256, {b}, 256)"):
        at = [rule.format(b=256 * i) for i in range(1, 15)]
        conditions += [f"!({b}) || ({a})" for a, b in zip(at, at[1:])] + [at[0], f"!({at[-1]})"]
        conditions.append(f"{rule.format(b=900)} == {rule.format(b=901)}")
    _holds(tmp_path, *conditions)


def test_launches_of_the_block_size_tests(tmp_path):
    """The launches of test_gpu_long_blocks.py (and of the backward's test of long owner blocks) take the blocks that it says."""
    conditions = ["!backward_short_blocks(256, 1200, 256)"]
    for d in (64, 128):
        for v in ("false", "true"):
            conditions += [f"!update_short_blocks({d}, {v}, {frames}, {b}, 256)"
                           for b, frames in G.LONG_UPDATES[d, v == "true"] + [G.LONG_SPIKES[d, v == "true"]]]
            conditions.append(f"update_short_blocks({d}, {v}, {G.SHORT_SPIKES[1]}, {G.SHORT_SPIKES[0]}, 256)")
            conditions.append(f"whole_frame_tokens({d}, {v}, 1, 256) < {G.SHORT_SPIKES[0]}")
        conditions += [f"!exact_rows_short_blocks({h}, {rows}, {n}, 256)" for h, rows, n in G.LONG_ROWS]
        conditions += [f"exact_rows_short_blocks({h}, {rows}, {n}, 256)" for h, rows, n in G.SHORT_ROWS]
        (t, p), (ts, ps) = G.LONG_TEMPORAL, G.SHORT_TEMPORAL
        conditions += [f"!temporal_lse_short_blocks({d}, {p}, {t}, 256)", f"temporal_lse_short_blocks({d}, {ps}, {ts}, 256)",
                       *(f"temporal_product_short_blocks({d}, {last}, {ps}, {ts}, 256)" for last in ("false", "true"))]
    conditions += [f"!temporal_product_short_blocks(64, {last}, {G.LONG_TEMPORAL[1]}, {G.LONG_TEMPORAL[0]}, 256)" for last in ("false", "true")]
    conditions += [f"!temporal_product_short_blocks(128, true, {p}, {t}, 256)" for t, p in G.LONG_LAST]
    for rows in (G.LONG_ROWS, G.SHORT_ROWS):
        conditions += [f"exact_rows_ranges({rows[0][0]}, {rows[0][1]}, {rows[0][2]}, 256) == 1", f"exact_rows_ranges({rows[1][0]}, {rows[1][1]}, {rows[1][2]}, 256) > 1"]
    _holds(tmp_path, *conditions)
