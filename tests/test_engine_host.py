"""Host-side checks of the engine: what it refuses and how it orders layers (no GPU)."""
import pytest

B = pytest.importorskip("paper_1805_08691_amd.binding")

from paper_1805_08691_amd import workloads as wl          # noqa: E402
from paper_1805_08691_amd.engine import Engine            # noqa: E402


@pytest.mark.parametrize("batches", [[], iter(())])
def test_calibration_without_a_batch_is_refused(batches):
    eng = Engine(wl.bottleneck_block(), 1, device="cpu")
    eng.set_factors({"x": 0.5})
    with pytest.raises(ValueError):
        eng.calibrate(batches)
    assert eng.q == {"x": 0.5}
