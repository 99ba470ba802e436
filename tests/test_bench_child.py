"""The bench's figures beside the headline come from a child process: what it makes of the child."""

import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

import bench


@pytest.mark.parametrize("code,expected", [
    ("print('noise'); print('{\"a\": 1}')", {"a": 1}),
    ("import os; print('{}'); os.abort()", {"extras_failed": -6}),
    ("raise SystemExit(3)", {"extras_failed": 3}),
    ("pass", {"extras_failed": 0}),
    ("import time; time.sleep(60)", {"extras_failed": "timeout"})])
def test_child_json(code, expected):
    assert bench.child_json([sys.executable, "-c", code], timeout=5) == expected
