"""A batched plan's cached schedule belongs to the kernels it was timed with: an
entry of another build of the library, or of one that did not say, is not used."""
import pytest
import torch

from paper_1611_09704_amd import binding as B
from paper_1611_09704_amd import build

pytestmark = pytest.mark.gpu


def test_schedules_of_other_kernels_are_timed_again(tmp_path, monkeypatch):
    path = tmp_path / "sched.txt"
    monkeypatch.setenv("SPD_TUNE_CACHE", str(path))
    planes = [torch.randn((4, 5000 + 100 * i), device="cuda") for i in range(3)]
    p = B.Params(list(range(1, 101)), 6.0)

    def tuned():
        plan = B.BatchPlan(planes, p)
        t = plan.describe()["tuned"]
        plan.close()
        return t

    print("case: tune cache", flush=True)
    assert tuned() == 1 and tuned() == 2
    key, rest = path.read_text().splitlines()[0].split(" ", 1)
    parts = key.split("|")
    strided = "8 4 0 1 0"
    for other in (["v3"] + parts[2:], parts[:1] + ["0" * 12] + parts[2:]):
        path.write_text("%s %s\n" % ("|".join(other), strided))
        assert tuned() == 1, "used a schedule of other kernels"
    assert parts[1] == build.source_id()
    path.write_text("%s %s\n" % (key, strided))
    assert tuned() == 2
