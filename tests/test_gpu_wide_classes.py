"""Class sums of so many pieces that the four waves of a block add them up together, on both sides of where that begins (the cases
and criteria of test_gpu_class_sums.py)."""
import pytest

from test_gpu_class_sums import test_classes_of_copies as classes_of_copies

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,precision,copies", [
    (64, "fp32", 1023), (64, "fp32", 1040), (128, "fp32", 511), (128, "fp32", 530), (128, "bf16", 1500), (256, "bf16", 255), (256, "bf16", 272),
    (256, "fp32", 1100), (64, "bf16", 2300)])
def test_classes_of_many_pieces(hidden, precision, copies, monkeypatch):
    monkeypatch.setenv("XRL_SUM_STEPS", "1")
    classes_of_copies(copies, hidden, precision, monkeypatch)
