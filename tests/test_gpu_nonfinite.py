"""Non-finite and extreme activations in every encoder.  A NaN coordinate is the
largest level-0 score and is returned bit for bit; whatever a row holds, the
rows beside it are what they would be without it.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2607_20652_amd import binding as dpb
from paper_2607_20652_amd import inputs
from parity_util import TOL_F32, EncodeCheck, compare_encode, random_std_state

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


@pytest.mark.parametrize("std", [False, True])
@pytest.mark.parametrize("dt", ["bf16", "f32"])
@pytest.mark.parametrize("name", ["narrow", "narrow16", "wide", "general"])
def test_extreme_rows_beside_ordinary_ones(name, dt, std):
    """Rows of NaN, infinities, zeros and magnitudes near 1e-35 among ordinary
    ones: the ordinary rows are bit for bit what they are without them, no row
    lists an index twice, and the finite ones are the oracle's."""
    d, nb, br, K = PLANS[name]
    nb, K, dl = list(nb), list(K), [0] + [br] * (len(nb) - 1)
    plan = make_plan(name)
    print(f"[extreme rows] {name} {dt} std={std}", flush=True)
    x = inputs.normal((40, d), 72, dt)
    stats = mu = r = None
    if std:
        mu, _, r = random_std_state(1 << nb[-1], 73)
        stats = torch.from_numpy(np.stack([mu, r], axis=1)).contiguous().to(DEV)
    plain, plain_coef = dpb.encode(plan, x.to(DEV), stats=stats)
    nan, inf = float("nan"), float("inf")
    x[3, 5], x[4, :], x[9, 17], x[10, d - 1], x[17, 0], x[17, 1] = nan, nan, inf, -inf, inf, -inf
    x[21] = 0.0
    small = [26, 27]
    x[small] = (x[small].double() * 1e-35).to(x.dtype)
    idx, coef = dpb.encode(plan, x.to(DEV), stats=stats)
    idx, coef = idx.cpu(), coef.cpu()
    odd = [3, 4, 9, 10, 17, 21] + small
    rest = [t for t in range(40) if t not in odd]
    assert torch.equal(idx[rest], plain.cpu()[rest])
    assert torch.equal(coef[rest].view(torch.int32), plain_coef.cpu()[rest].view(torch.int32))
    base = np.concatenate([[0], np.cumsum(K)]).astype(int)
    for t in range(40):
        for l in range(len(K)):
            s = idx[t, base[l]:base[l + 1]].numpy()
            s = s[s >= 0]
            assert np.unique(s).size == s.size, (t, l)
            assert (s < (1 << nb[l])).all() and (l == 0 or (s >= (1 << nb[l - 1])).all()), (t, l)
    # the finite rows against the oracle: zeros (every score a tie or, standardized, the statistics alone), small ones
    m, gens = oracle.masks(d, nb[-1]), oracle.generators(nb, dl, 0)
    rows = ([21] + small) if std else small
    xd = x[rows].double().numpy()
    if std:
        o = oracle.encode_std(d, m, nb, K, dl, gens, xd, mu, r)
    else:
        o = oracle.encode(d, m, nb, K, dl, gens, xd)
        zi, zc = oracle.encode(d, m, nb, K, dl, gens, np.zeros((1, d)))[:2]
        assert np.array_equal(idx[21].numpy(), zi[0]) and (coef[21] == 0).all()
    compare_encode(K, idx[rows].numpy(), coef[rows].numpy(), *o, TOL_F32, ctx=EncodeCheck(d, m, gens, xd, mu, r))
