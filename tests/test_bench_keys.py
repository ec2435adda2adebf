"""What the benchmark's line says of the step's form comes from the step."""
import pytest

import bench
from paper_1501_03857_amd import lbboil as L


def test_recorded_counters_cover_the_rule_for_the_form():
    """The counters of a one-launch step depend on its tiles or strips: their
    key covers the header that picks them, which no other source does."""
    assert bench.source_hash() == bench.source_hash("lbb_device.hpp", "lbb_step.hpp", "lbb_form.hpp")
    csrc = bench.os.path.join(bench.ROOT, "paper_1501_03857_amd", "csrc")
    found = [n for n in sorted(bench.os.listdir(csrc)) if "StepForm step_form(" in open(bench.os.path.join(csrc, n)).read()]
    assert found == ["lbb_form.hpp"]


@pytest.mark.gpu
@pytest.mark.parametrize("nx,ny,precision,tiles,launches", [
    (128, 64, L.FP64, None, 1), (128, 64, L.FP64, (0, 0), 2), (1200, 900, L.FP32, None, 2), (2050, 1500, L.FP32, None, 1)])
def test_launches_are_counted(nx, ny, precision, tiles, launches):
    print("[gpu-case] launches a step", nx, ny, precision, tiles, flush=True)
    d = L.Domain(L.Params(nx=nx, ny=ny, precision=precision, liquid_rows=ny // 2))
    if tiles:
        d.set_tiles(*tiles)
    assert bench.launches_per_step(d) == launches
    d.step(3)
    assert d.t == 3
