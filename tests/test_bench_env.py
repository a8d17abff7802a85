"""bench.py's switch to the five passes for its small warm-up plan (no GPU): a
caller's own SE2N_NO_PAIR, or its absence, holds again afterwards."""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402


@pytest.mark.parametrize("own", [None, "1", "2"])
@pytest.mark.parametrize("fails", [False, True])
def test_five_passes_restores_the_setting(monkeypatch, own, fails):
    if own is None:
        monkeypatch.delenv("SE2N_NO_PAIR", raising=False)
    else:
        monkeypatch.setenv("SE2N_NO_PAIR", own)
    try:
        with bench.five_passes():
            assert os.environ["SE2N_NO_PAIR"] == "1"
            if fails:
                raise ValueError
    except ValueError:
        pass
    assert os.environ.get("SE2N_NO_PAIR") == own
