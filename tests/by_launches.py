"""Fixture of the test files that repeat others' tests with a launch (or a few)
for each CG iteration: contexts are created with one-launch solves off.  These
kernels serve large meshes, meshes with free surfaces and every solve after a
launch that gave up; at the tests' sizes the one-launch solves would run."""
import pytest

from paper_2510_09812_amd import gspm


@pytest.fixture(autouse=True)
def by_launches(monkeypatch):
    create = gspm.gspm_create
    made = []

    def off(*args, **kw):
        ctx = create(*args, **kw)
        gspm.gspm_set_solve_path(ctx, gspm.GSPM_PATH_LAUNCHES)
        made.append(ctx)
        return ctx

    monkeypatch.setattr(gspm, "gspm_create", off)
    yield
    assert made, "the test created no context that this file could switch"
