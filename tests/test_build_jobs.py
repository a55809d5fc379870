"""The build script takes any MAX_JOBS: one that is no positive number counts as not given."""
import importlib.util
import os

import pytest

from conftest import ROOT


@pytest.mark.parametrize("value,jobs", [(None, 8), ("", 8), ("0", 8), ("-2", 8), ("all", 8), ("3", 3), (" 16 ", 16)])
def test_jobs(monkeypatch, value, jobs):
    spec = importlib.util.spec_from_file_location("_build", os.path.join(ROOT, "paper_1404_5253_amd", "build.py"))
    b = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(b)
    monkeypatch.delenv("MAX_JOBS", raising=False) if value is None else monkeypatch.setenv("MAX_JOBS", value)
    with b.ThreadPoolExecutor(b._jobs()) as pool:
        assert pool._max_workers == jobs
