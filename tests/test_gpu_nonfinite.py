"""Non-finite and extreme activations in every encoder.  A NaN coordinate is the
largest level-0 score and is returned bit for bit; whatever a row holds, the
rows beside it are what they would be without it.
"""
import numpy as np
import pytest
import torch

from paper_2607_20652_amd import binding as dpb
from paper_2607_20652_amd import inputs

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

# name: (d, level bits, children per parent, K per level)
PLANS = {
    "narrow": (256, (8, 12, 16), 16, (8, 8, 32)),
    "narrow16": (192, (8, 11, 15), 16, (16, 16, 48)),
    "wide": (512, (9, 14), 256, (16, 32)),
    "general": (200, (8, 10, 14), 40, (3, 70, 40)),
    "one_level": (300, (9,), 16, (20,)),
}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dpb.load()


def make_plan(name):
    d, nb, br, K = PLANS[name]
    return dpb.Plan(d, seed=0, level_bits=list(nb), branchings=[0] + [br] * (len(nb) - 1), active=list(K))


@pytest.mark.parametrize("name", list(PLANS))
def test_nan_coordinates_come_back_bit_for_bit(name):
    plan = make_plan(name)
    d = plan.d
    x = inputs.normal((9, d), 71, "f32")
    bits = x.view(torch.int32)
    bits[4, 7] = 0x7FFFFFFF                      # the largest NaN payload
    bits[4, d - 1] = 0xFFF00001 - (1 << 32)      # a negative NaN above the clamp of the sorts
    idx, coef = dpb.encode(plan, x.to(DEV))
    print(f"[nan bits] {name}", flush=True)
    got = coef.cpu().view(torch.int32)[4, :2].tolist()
    assert idx.cpu()[4, :2].tolist() == [7, d - 1]
    assert got == [0x7FFFFFFF, 0xFFF00001 - (1 << 32)]
