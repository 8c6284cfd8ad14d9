"""Refinement of batches of up to 64 atoms on both sides of the number of poses from which
their two classes are launched one after the other; bit for bit against the oracle."""
import pytest

import test_gpu_refine_classes as classes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kpl,copies", [(3, 1), (4, 700), (4, 1100), (8, 520)])   # 24, 22 400, 35 200 and 33 280 poses
def test_two_classes_match_oracle(monkeypatch, kpl, copies):
    sizes = [(1, 0), (16, 4), (31, 9), (32, 14), (33, 0), (40, 3), (49, 5), (64, 18)]
    monkeypatch.setattr(classes, "SIZES", sizes)
    monkeypatch.setattr(classes, "STEPS", 8)
    classes.test_refined_classes_match_oracle(kpl, copies)
