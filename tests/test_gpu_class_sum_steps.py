"""Class sums of one, two and four steps of sixteen rows a group: classes that end on a step's edge, begin in one step and end in
another, fill a group or several (the cases and criteria of test_gpu_class_sums.py)."""
import pytest

from test_gpu_class_sums import test_classes_of_copies as classes_of_copies

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps", [1, 2, 4])
@pytest.mark.parametrize("copies", [2, 16, 31, 33, 64, 300])
@pytest.mark.parametrize("hidden,precision", [(64, "fp32"), (128, "bf16"), (256, "bf16")])
def test_class_sum_steps(copies, hidden, precision, steps, monkeypatch):
    monkeypatch.setenv("XRL_SUM_STEPS", str(steps))
    classes_of_copies(copies, hidden, precision, monkeypatch)
