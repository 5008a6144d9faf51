import gc
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


_module = None


def pytest_runtest_setup(item):
    """What earlier modules' failed calls left in reference cycles (an expected error holds its frame and the
    frame's tensors) goes before the next module starts: a test that compares the memory in use around a call
    must not see it released in between."""
    global _module
    if item.module is not _module:
        _module = item.module
        gc.collect()


class _Tuning:
    """Kernel-choice overrides of include/osc_tuning.h for one test; everything is back to
    automatic when the test ends."""

    def __init__(self):
        import paper_2604_12782_amd as osc
        self.osc = osc

    def gemm(self, cfg):
        """cfg = "<tile>,<kernel id>" (0 staged, 1 DMA, 2 persistent, 3 skinny, 4 and 5 ring, 6 streaming, 7 flowing) or None;
        the tile is rows / 64, of kernel 7 one of its own.  A kernel that cannot serve a shape gives way to another:
        osc_tuning_last_gemm() tells."""
        tile, kern = (-1, -1) if cfg is None else map(int, cfg.split(","))
        self.osc.osc_tuning_set(self.osc.OSC_TUNE_GEMM_TILE, tile)
        self.osc.osc_tuning_set(self.osc.OSC_TUNE_GEMM_KERNEL, kern)

    def reset(self):
        for k in range(5):
            self.osc.osc_tuning_set(k, -1)


import pytest  # noqa: E402


@pytest.fixture
def tuning():
    t = _Tuning()
    yield t
    t.reset()
