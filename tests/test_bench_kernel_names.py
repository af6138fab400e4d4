"""bench.py names the dense step kernel that the library launches (CPU): from the
form that the autotuner left in its tile file, else by the rule that the library
falls back on."""
import pytest

import bench
import paper_2604_01050_amd as sb

NAMES = {1: "k_dense_step_fine", 2: "k_dense_step_fine", 3: "k_dense_step", 4: "k_dense_step_sk", 5: "k_dense_step_sk",
         6: "k_dense_step_sk", 7: "k_dense_step_sk"}


@pytest.mark.parametrize("path", sorted(bench._PATH_CODES))
def test_rule_without_a_timed_form(path):
    form = sb.lib._ZN4sbqa18default_dense_formENS_4PathEiii
    pad = 128 if path in ("dense_fp32", "dense_bf16x3") else 512
    for N in (300, 601, 1500, 4096, 6000, 16384):
        for R, runs in ((1, 1), (10, 6), (16, 8), (16, 16), (16, 40), (32, 32), (16, 65)):
            for tile in (64, 128, 256):
                cg = -(-R * runs // tile) * tile
                want = NAMES[form(bench._PATH_CODES[path], -(-N // pad) * pad, tile // 64, cg)]
                if want == "k_dense_step" and path == "dense_bf16x3" and tile == 128 and cg % 256 == 0:
                    want = "k_dense_step_cg2"
                info = {"N": N, "R": R, "runs": runs, "path": path, "tile_cols": tile}
                assert bench.dense_kernel_name(info) == want, (info, want)


def test_form_from_the_tile_file(tmp_path, monkeypatch):
    f = tmp_path / "tiles.txt"
    monkeypatch.setenv("SBQA_TUNE_CACHE", str(f))
    info = {"N": 6000, "R": 16, "runs": 16, "path": "dense_int8", "tile_cols": 128}
    assert bench.tuned_form(info) is None
    f.write_text("garbage\nsbqa-tile-v1 gfx950 256 4 256 8192 2\n"          # a served context's
                 "sbqa-tile-v1 gfx950 256 %d 256 6144 2\n" % (4 + 16 * 1)
                 + "sbqa-tile-v1 gfx950 256 %d 256 6144 4\n" % (4 + 16 * 5)   # another tile
                 + "sbqa-tile-v1 gfx950 256 %d 128 6144 2\n" % (4 + 16 * 5))  # other columns
    assert bench.tuned_form(info) == 1
    f.write_text(f.read_text() + "sbqa-tile-v1 gfx950 256 %d 256 6144 2\n" % (4 + 16 * 6))
    assert bench.tuned_form(info) == 6
    assert bench.tuned_form(info, given=True) is None
    f.write_text(f.read_text() + "sbqa-tile-v1 gfx950 256 %d 256 6144 2\n" % (4 + 16 * 3 + 256))
    assert bench.tuned_form(info) == 6 and bench.tuned_form(info, given=True) == 3
    assert [bench.dense_kernel_name(info, q) for q in range(1, 8)] == [NAMES[q] for q in range(1, 8)]
