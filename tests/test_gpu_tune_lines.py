"""Lines of a tune cache file: which of them a library reads that knows only the
shapes of hisq_tune_set."""
import pytest

from gpu_util import need_gpu
from test_gpu_wave_blocks import load_shape

pytestmark = pytest.mark.gpu

DIMS = (6, 8, 10, 12)


def saved(hisq, tmp_path):
    hisq.hisq_tune_save(tmp_path / "s.txt")
    return [ln for ln in (tmp_path / "s.txt").read_text().splitlines() if ln.startswith("hisq-tune")]


@pytest.mark.parametrize("shape,known", [((1, 1, 2, 128, 0, 0), True), ((1, 1, -2, 256, 0, 2), True),
                                         ((1, 1, -2, 64, 0, 0), False), ((1, 1, -42, 128, 0, 0), False),
                                         ((4, 1, 1, 256, 0, 1), True), ((2, 2, 1, 64, 0, 1), False)])
def test_lines_of_new_shapes_are_another_device_to_older_readers(tmp_path, shape, known):
    hisq = need_gpu()
    c = shape[0] * shape[1]
    load_shape(hisq, tmp_path, "single", 18, DIMS, c, [0], shape)
    try:
        rep = hisq.hisq_tune_report()
        line, = saved(hisq, tmp_path)
        assert line.startswith("hisq-tune 1 gfx950" + (" " if known else "/2 "))
        hisq.hisq_tune_clear()
        assert hisq.hisq_tune_load(tmp_path / "s.txt") == 1
        assert hisq.hisq_tune_report().split(" (")[0] == rep.split(" (")[0]
        # the same shape without the mark, as a file of before holds it, and another device's
        for arch, n in (("gfx950", 1), ("gfx000/2", 0), ("gfx950/3", 0)):
            f = line.split()
            (tmp_path / "o.txt").write_text(" ".join(f[:2] + [arch] + f[3:]) + "\n")
            assert hisq.hisq_tune_load(tmp_path / "o.txt") == n
    finally:
        hisq.hisq_tune_clear()


# links of 111, 80 and 255 MB: all directions of the first two fit the solver's share of the memory-side cache and
# three of the last, none of 1.0 GB; 17 MB are the tuner's choice
RULE = [((20, 20, 20, 24), "single", 18, -42), ((20, 20, 20, 24), "int30", 8, -42), ((24, 24, 24, 32), "single", 18, -32),
        ((32, 32, 32, 32), "double", 12, None), ((12, 10, 14, 18), "single", 18, None)]


@pytest.mark.parametrize("dims,name,recon,stage", RULE)
def test_stage_of_a_solver(tmp_path, dims, name, recon, stage):
    hisq = need_gpu()
    told = ", stage %s in a solver's iterations" % stage
    try:
        load_shape(hisq, tmp_path, name, recon, dims, 1, [0], (1, 1, -2, 128, 0, 0))     # timed: the tuner's
        rep = hisq.hisq_tune_report()
        assert (told in rep) if stage else ("solver" not in rep), rep
        line, = saved(hisq, tmp_path)
        assert float(line.split()[-1]) > 0 and hisq.hisq_tune_load(tmp_path / "s.txt") == 1
        assert hisq.hisq_tune_report() == rep
        # fixed by the program, here or in the process that saved it: as it is
        hisq.hisq_tune_set(name, dims, 1, 1, 1, -2, 128, 0, long_recon=recon)
        assert "stage -2 " in hisq.hisq_tune_report() and "solver" not in hisq.hisq_tune_report()
        line, = saved(hisq, tmp_path)
        hisq.hisq_tune_clear()
        assert float(line.split()[-1]) < 0 and hisq.hisq_tune_load(tmp_path / "s.txt") == 1
        assert "stage -2 " in hisq.hisq_tune_report() and "solver" not in hisq.hisq_tune_report()
    finally:
        hisq.hisq_tune_clear()
