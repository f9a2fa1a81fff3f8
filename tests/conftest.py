import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (runs the HIP library)")


_CONFIG = None


@pytest.hookimpl(trylast=True)
def pytest_sessionstart(session):
    global _CONFIG
    _CONFIG = session.config


def say(msg):
    """One line that names the GPU case about to run (test, shape, entry point) or reports what it measured,
    written past pytest's output capture and flushed, so that it is on the terminal before the GPU step starts."""
    line = f"[gpu-case] {msg}"
    pm = _CONFIG.pluginmanager if _CONFIG is not None else None
    tr = pm.get_plugin("terminalreporter") if pm is not None else None
    capman = pm.get_plugin("capturemanager") if pm is not None else None
    if tr is not None and capman is not None:
        with capman.global_and_fixture_disabled():
            tr.ensure_newline()
            tr.write_line(line)
            tr._tw.flush()
    else:
        print(line, file=sys.stderr, flush=True)


def kernels_of(call):
    """Names of this library's kernels that call() launches, in order: which path a shape takes is part of what some tests are about."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    found = [e for e in prof.events() if "::ll_" in e.name]
    return [e.name.replace("(anonymous namespace)::", "").removeprefix("void ") for e in sorted(found, key=lambda e: e.time_range.start)]
