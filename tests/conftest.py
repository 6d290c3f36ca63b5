import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (run through the HIP library)")
    config.addinivalue_line("markers", "slow: long-running CPU test")


@pytest.hookimpl(tryfirst=True)
def pytest_runtest_protocol(item, nextitem):   # (before the output of the test is captured)
    """Name every GPU test on the terminal before its first GPU step: an abort
    inside a GPU call then leaves its test's name as the last line printed."""
    terminal = item.config.pluginmanager.get_plugin("terminalreporter")
    if item.get_closest_marker("gpu") and terminal is not None and terminal.verbosity <= 0:
        terminal.write_line("gpu: " + item.nodeid)
        terminal.flush()
