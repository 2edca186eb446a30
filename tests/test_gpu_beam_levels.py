"""The beam levels' selection of the narrow encoder where children repeat: index
ranges so small that a child of two parents is often among a token's largest
(its equal scores fill two of the lane maxima, and the threshold is taken again
from distinct ones), one with fewer distinct children than slots, and a width
whose list of candidates just fits the LDS.
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

# name: (d, level bits, children per parent, K per level, tokens)
PLANS = {
    "four_parents": (200, (8, 10, 12), 16, (4, 4, 8), 401),
    "four_parents_small": (64, (6, 7, 8), 16, (4, 4, 16), 401),
    "eight_parents": (64, (6, 7, 8, 9), 16, (8, 8, 8, 32), 401),
    "sixteen_parents": (128, (7, 8, 9, 10), 16, (16, 16, 16, 64), 301),
    "few_children": (40, (6, 7, 8), 8, (8, 16, 16), 201),          # few of them distinct
    "lds_limit": (3296, (12, 20, 29), 16, (2, 16, 16), 9),         # standardized fp32: 104 candidates a token
}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dpb.load()


@pytest.mark.parametrize("name", list(PLANS))
@pytest.mark.parametrize("dt", ["bf16", "f32"])
def test_beam_levels_with_repeated_children(name, dt):
    d, nb, br, K, T = PLANS[name]
    nb, K, dl = list(nb), list(K), [0] + [br] * (len(nb) - 1)
    print(f"[beam levels] {name} {dt}", flush=True)
    plan = dpb.Plan(d, seed=0, level_bits=nb, branchings=dl, active=K)
    m, gens = oracle.masks(d, nb[-1]), oracle.generators(nb, dl, 0)
    x = inputs.normal((T, d), 8100 + d, dt)
    xd = x.double().numpy()
    idx, coef = dpb.encode(plan, x.to(DEV))
    oi, oc, om, oo = oracle.encode(d, m, nb, K, dl, gens, xd)
    st = compare_encode(K, idx.cpu().numpy(), coef.cpu().numpy(), oi, oc, om, oo, TOL_F32, ctx=EncodeCheck(d, m, gens, xd))
    if nb[-1] > 20:
        if dt == "bf16":
            return   # 4 GiB of statistics: once, where the list is at the limit
        mu = np.zeros(1 << nb[-1], np.float32)
        r = np.ones(1 << nb[-1], np.float32)
    else:
        mu, _, r = random_std_state(1 << nb[-1], 8200)
    stats = torch.from_numpy(np.stack([mu, r], axis=1)).contiguous().to(DEV)
    sidx, scoef = dpb.encode(plan, x.to(DEV), stats=stats)
    si, sc, sm, so = oracle.encode_std(d, m, nb, K, dl, gens, xd, mu, r)
    st2 = compare_encode(K, sidx.cpu().numpy(), scoef.cpu().numpy(), si, sc, sm, so, TOL_F32,
                         ctx=EncodeCheck(d, m, gens, xd, mu, r))
    print(f"  {st}\n  {st2}", flush=True)
