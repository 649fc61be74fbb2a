"""CPU: the autotuner's persistent choices belong to the library that timed them.

A choice stored by another build of the kernels (a key without the library's
digest, or with another one) must not be applied; a choice of the same build is,
without timing."""
import ctypes
import json

import pytest
import torch

import workloads as W
from paper_2202_09421_amd import rte

STALE = {"line_units_per_wave": 1, "line_generic": 1, "node_tiles_per_block": 1, "line_waves_per_unit": 2,
         "line_global_tables": 0}


class FakeLib:
    def __init__(self):
        self.calls = []

    def rte_plan_set_schedule(self, h, sched):
        self.calls.append("set")
        return 0

    def rte_plan_autotune(self, h, a, b, ws, n, stream, chosen):
        self.calls.append("tune")
        ctypes.cast(chosen, ctypes.POINTER(rte.rte_schedule)).contents.node_tiles_per_block = 4
        return 0


@pytest.fixture
def setup(monkeypatch, tmp_path):
    fake = FakeLib()
    lib_file = tmp_path / "librte.so"
    lib_file.write_bytes(b"one build")
    monkeypatch.setattr(rte, "lib", lambda: fake)
    monkeypatch.setattr(rte, "LIB_PATH", str(lib_file))
    monkeypatch.setattr(rte, "_stream", lambda: None)
    plan = object.__new__(rte.Plan)
    plan.spec = W.small_problem(N=999, M=4, K=2, Ny=9)
    plan.dtype, plan.device, plan._h = torch.float64, torch.device("cpu"), None
    plan.Nq, plan.Np_x, plan.Np_y, plan.generation = 1, 1080, 36, 0
    plan.workspace = lambda adj: torch.empty(256, dtype=torch.uint8)
    return plan, fake, lib_file, str(tmp_path / "schedules.json")


def test_choice_without_a_digest_is_not_applied(setup):
    plan, fake, _, path = setup
    dev = torch.cuda.get_device_name(plan.device) if torch.cuda.is_available() else "none"
    with open(path, "w") as fh:
        json.dump({dev + "|f64|nx1000|ny10|M4|Nq1|Np1080,36": STALE}, fh)
    got = plan.autotune(plan.spec.mu_a, plan.spec.mu_s, cache=path)
    assert fake.calls == ["tune"] and got == dict(STALE, line_generic=0, node_tiles_per_block=4, cached=False,
                                                  line_units_per_wave=0, line_waves_per_unit=0)


def test_choice_of_another_build_is_not_applied(setup):
    plan, fake, lib_file, path = setup
    tune = lambda: plan.autotune(plan.spec.mu_a, plan.spec.mu_s, cache=path)["cached"]
    assert [tune(), tune()] == [False, True] and fake.calls == ["tune", "set"]
    lib_file.write_bytes(b"another build")
    assert [tune(), tune()] == [False, True] and fake.calls == ["tune", "set"] * 2
