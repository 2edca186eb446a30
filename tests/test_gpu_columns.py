"""GPU parity of the column decode and its backward (columns.hpp) where they
can go wrong: each number of parent columns per token, widths that fill no
coordinate step or no pair, parents that are basis features, several words of
summed slots, and codes the encoder does not produce (a slot that routes to no
parent, repeated indices, hashed indices on level 0, padding, indices drawn at
random).  `wide_code` has more slots than a mark byte holds and takes the
table decode instead.
"""
import sys

import numpy as np
import pytest
import torch

import oracle
from paper_2607_20652_amd import binding as dpb
from paper_2607_20652_amd import inputs
from parity_util import TOL_BF16, TOL_F32, compare_dense

pytestmark = pytest.mark.gpu

DEV = "cuda:0"

# name: (d, level bits, K per level[, children per parent, else 16])
PLANS = {
    "cpt8": (768, (10, 12, 15, 17, 20), (8, 8, 8, 8, 64)),
    "cpt4_d200": (200, (8, 10, 12), (4, 4, 8)),
    "cpt16": (1024, (10, 12, 15, 18, 21, 24), (16, 16, 16, 16, 16, 64)),
    "odd_d": (101, (7, 10, 13), (8, 8, 24)),
    "d_tail": (1000, (10, 13, 16, 18), (6, 5, 6, 20)),       # 6 parents of 8 columns, 5 summed slots
    "basis_parents": (256, (8, 12), (8, 32)),
    "one_step": (40, (6, 9, 12), (16, 16, 48)),              # dp = 64 < one step of 128 coordinates
    "many_words": (512, (9, 11, 13, 15, 17, 19, 21, 23), (12, 12, 12, 12, 12, 12, 9, 18)),
    "beam24": (384, (9, 12, 15, 18), (24, 24, 8, 32)),       # 24 summed slots: all six groups of word 0
    "wide_code": (768, (10, 14, 18), (16, 16, 256)),
    # no leaf columns: every hashed slot through the tables
    "table_2l": (1024, (10, 15), (16, 32), 256),
    "table_3l": (1024, (10, 15, 17), (16, 32, 64), 256),
    "table_d2048": (2048, (11, 15), (16, 32), 256),
    "table_d522": (522, (10, 13, 16), (8, 8, 16), 32),
    "table_d64": (64, (6, 9), (3, 5), 16),
    "table_odd": (333, (9, 13, 17), (16, 16, 16), 16),       # 32 slots: one full word
    "table_254": (512, (9, 13, 17), (16, 110, 128), 64),     # the widest code of marks
    "one_level": (300, (9,), (20,), 16),
    # four parents under a wide beam: rows of four tokens leave a CU one workgroup, so these go without columns
    "few_parents": (1024, (10, 13, 16, 20), (32, 32, 4, 12)),           # the backward
    "few_parents_d1500": (1500, (11, 14, 17, 20), (32, 32, 4, 12)),     # the decode too
    "few_parents_d2048": (2048, (11, 14, 17), (4, 4, 8)),
    "few_parents_d4096": (4096, (12, 14, 16), (4, 4, 8)),               # rows of four tokens do not fit
    "four_of_2048": (2048, (11, 14, 17), (4, 4, 32)),                   # columns save a word: kept
    "table_k0": (300, (9, 13), (100, 64), 64),               # up to 100 hashed indices on level 0
}


def branch(name):
    return PLANS[name][3] if len(PLANS[name]) > 3 else 16


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dpb.load()


def codes(name, T, seed):
    """Codes of random children (the layout of the encoder's), then one oddity per row."""
    d, nb, K = PLANS[name][:3]
    L, rng = len(nb), np.random.default_rng(seed)
    dl = [0] + [branch(name)] * (L - 1)
    gens = oracle.generators(list(nb), dl, 0)
    base = np.concatenate([[0], np.cumsum(K)]).astype(int)
    idx = np.full((T, sum(K)), -1, np.int32)
    for t in range(T):
        par = rng.choice(d, K[0], replace=False)
        idx[t, : K[0]] = par
        for l in range(1, L):
            g = np.asarray(gens[l], np.int64)
            child = rng.permutation(np.unique(par[:, None] ^ g[None, :]))[: K[l]]
            idx[t, base[l]:base[l] + len(child)] = child
            par = child
    coef = rng.standard_normal(idx.shape).astype(np.float32)
    coef[idx < 0] = 0.0
    k, N = sum(K), 1 << nb[-1]
    rand = lambda: int(rng.integers(d, N)) if d < N else 0
    odd = {
        1: lambda r: r.__setitem__(k - 1, rand()),                            # routes to no parent
        2: lambda r: r.__setitem__(1, r[0]),                                  # a basis slot twice
        3: lambda r: r.__setitem__(slice(base[L - 1], k), r[base[L - 1]]),    # one leaf in every leaf slot
        4: lambda r: r.__setitem__(0, r[k - 1]),                              # a hashed index on level 0
        5: lambda r: r.__setitem__(k - 1, r[0]),                              # a basis index among the leaves
        6: lambda r: r.__setitem__(base[max(L - 2, 0)], rand() if L > 2 else r[1]),   # another parent: its children route nowhere
        7: lambda r: r.__setitem__(slice(0, k), -1),                          # all padding
        8: lambda r: r.__setitem__(slice(0, k), rng.integers(0, N, k)),       # any indices
        9: lambda r: r.__setitem__(slice(base[max(L - 2, 0)], base[max(L - 2, 0)] + 2), -1),  # padding parents
        10: lambda r: r.__setitem__(slice(0, k), rng.integers(0, d, k)),      # basis indices everywhere, repeated
    }
    for t, f in odd.items():
        f(idx[t])
    coef[idx < 0] = 0.0
    return idx, coef


@pytest.mark.parametrize("name", list(PLANS))
def test_column_decode_and_bwd(name):
    d, nb, K = PLANS[name][:3]
    T = 23                                       # ragged last group for 2 and 4 tokens per wave
    print(f"[columns] {name} d={d} T={T}", flush=True)
    sys.stdout.flush()
    plan = dpb.Plan(d, seed=0, level_bits=list(nb), branchings=[0] + [branch(name)] * (len(nb) - 1), active=list(K))
    m = oracle.masks(d, nb[-1])
    idx, coef = codes(name, T, 9000 + d)
    di, dc = torch.from_numpy(idx).to(DEV), torch.from_numpy(coef).to(DEV)
    ref = oracle.decode(d, m, idx, coef.astype(np.float64))
    for dt, tol in ((torch.float32, TOL_F32), (torch.bfloat16, TOL_BF16)):
        y = dpb.decode(plan, di, dc, dt)
        compare_dense(y.float().cpu().numpy(), ref, tol)
    for dt in ("f32", "bf16"):
        g = inputs.normal((T, d), 9100 + d, dt)
        rgc, rgx = oracle.decode_bwd(d, m, idx, g.double().numpy())
        for xt, tol in ((torch.float32, TOL_F32), (torch.bfloat16, TOL_BF16)):
            gc, gx = dpb.decode_bwd(plan, di, g.to(DEV), gx_dtype=xt)
            compare_dense(gc.cpu().numpy(), rgc, TOL_F32)
            compare_dense(gx.float().cpu().numpy(), rgx, tol)
            # the extra term added in place (the layer's use): same rows plus add
            add = inputs.normal((T, d), 9200 + d, "f32").to(xt)
            buf = add.to(DEV)
            _, gx2 = dpb.decode_bwd_ex(plan, di, g.to(DEV), add_grad_x=buf, grad_x=buf)
            compare_dense(gx2.float().cpu().numpy(), rgx + add.double().numpy(), tol)


@pytest.mark.parametrize("name", ["cpt8", "cpt4_d200", "cpt16", "odd_d"])
def test_infinite_fp32_gradient_reaches_the_parents_signed(name):
    """An fp32 gradient that is infinite, or finite beyond the largest bf16, has
    no split into bf16 terms: the parents' coefficients are the signed infinity
    (or the finite sum), as the definition gives, and other rows stay within tolerance."""
    d, nb, K = PLANS[name][:3]
    T = 23
    print(f"[infinite gradient] {name}", flush=True)
    plan = dpb.Plan(d, seed=0, level_bits=list(nb), branchings=[0] + [branch(name)] * (len(nb) - 1), active=list(K))
    m = oracle.masks(d, nb[-1])
    idx, _ = codes(name, T, 9300 + d)
    di = torch.from_numpy(idx).to(DEV)
    g = inputs.normal((T, d), 9400 + d, "f32")
    g[12, 3] = float("inf")
    g[15, d - 1] = -float("inf")
    g[18] = 0.0
    g[18, 5] = 3.4e38
    rgc, _ = oracle.decode_bwd(d, m, idx, g.double().numpy())
    got, _ = dpb.decode_bwd(plan, di, g.to(DEV))
    got = got.cpu().numpy()
    parents = slice(sum(K[:-2]), sum(K[:-1]))
    for t in (12, 15):
        assert np.array_equal(got[t, parents], rgc[t, parents].astype(np.float32))
    compare_dense(got[18, parents][None], rgc[18, parents][None], TOL_F32)
    rest = [t for t in range(T) if t not in (12, 15, 18)]
    compare_dense(got[rest], rgc[rest], TOL_F32)


@pytest.mark.parametrize("name", ["cpt8", "cpt4_d200", "cpt16", "odd_d", "table_2l", "one_level"])
def test_repeated_slots_add_in_slot_order(name):
    """A coordinate, or a leaf, that several slots hold gets the fp32 sum of
    their coefficients in slot order: the values are chosen so that every other
    order gives another sum."""
    d, nb, K = PLANS[name][:3]
    L, base = len(nb), np.concatenate([[0], np.cumsum(K)]).astype(int)
    plan = dpb.Plan(d, seed=0, level_bits=list(nb), branchings=[0] + [branch(name)] * (L - 1), active=list(K))
    print(f"[repeated slots] {name}", flush=True)
    orders = [(1e8, 1.0, -1e8), (1e8, -1e8, 1.0), (1.0, 1e8, -1e8), (-1e8, 1e8, 1.0), (1.0, -1e8, 1e8), (-1e8, 1.0, 1e8)]
    idx = np.full((2 * len(orders), sum(K)), -1, np.int32)
    coef = np.zeros(idx.shape, np.float32)
    want = np.zeros((idx.shape[0], d), np.float32)
    leaf_gens = oracle.generators(list(nb), [0] + [branch(name)] * (L - 1), 0)[L - 1] if L > 1 else None
    m = oracle.masks(d, nb[-1])
    columns = L > 1 and len(PLANS[name]) == 3
    for t in range(idx.shape[0]):
        val = orders[t % len(orders)]
        total = np.float32(np.float32(np.float32(val[0]) + np.float32(val[1])) + np.float32(val[2]))
        if t < len(orders):   # a basis coordinate in three slots, the last two as far apart as the code is wide
            at = [0, 1, sum(K) - 1]
            idx[t, at], coef[t, at] = d - 1, val
            want[t, d - 1] = total
        elif columns:         # a child of the last parent slot in three leaf slots
            p = 5 % d
            idx[t, base[L - 1] - 1] = p
            at = [base[L - 1], base[L - 1] + 2, sum(K) - 1]
            c = int(p) ^ int(leaf_gens[3])
            idx[t, at], coef[t, at] = c, val
            want[t] = oracle.decode(d, m, np.array([[c]], np.int32), np.array([[float(total)]]))[0].astype(np.float32)
    y = dpb.decode(plan, torch.from_numpy(idx).to(DEV), torch.from_numpy(coef).to(DEV), torch.float32).cpu().numpy()
    assert np.array_equal(y == 0, want == 0)
    compare_dense(y, want, TOL_F32)


@pytest.mark.parametrize("name", ["cpt8", "cpt4_d200", "cpt16", "odd_d", "basis_parents", "one_step", "many_words",
                                  "table_2l", "table_k0"])
def test_unlisted_slots(name):
    """Any number of slots that fit neither a parent's column nor the plan's own
    tables (leaves without a listed parent, hashed indices on level 0), from one
    to all of them, next to tokens of the same wave that have none: at, below
    and above the count up to which they are added one by one."""
    d, nb, K = PLANS[name][:3]
    L, k, N = len(nb), sum(K), 1 << nb[-1]
    base = np.concatenate([[0], np.cumsum(K)]).astype(int)
    print(f"[unlisted] {name}", flush=True)
    plan = dpb.Plan(d, seed=0, level_bits=list(nb), branchings=[0] + [branch(name)] * (L - 1), active=list(K))
    m = oracle.masks(d, nb[-1])
    counts = [0, 1, 4, 15, 16, 17, 31, 32, 33, 63, 64, 65, k]
    idx, _ = codes(name, 4 * len(counts), 9500 + d)
    idx, rng = idx[-4 * len(counts):], np.random.default_rng(9600 + d)
    open_slots = np.r_[base[L - 1]:k, 0:(K[0] if L != 2 or len(PLANS[name]) > 3 else 0)]   # leaves, then level 0
    for t in range(idx.shape[0]):
        n = min(counts[t // 4], len(open_slots)) if t % 4 != 2 else 0
        idx[t, open_slots[:n]] = rng.integers(d, N, n)
        if t % 4 == 3:
            idx[t, (base[L - 2] if L > 1 else 0):base[L - 1]] = -1   # no parents: a code of leaves alone
    coef = rng.standard_normal(idx.shape).astype(np.float32)
    coef[idx < 0] = 0.0
    di, dc = torch.from_numpy(idx).to(DEV), torch.from_numpy(coef).to(DEV)
    ref = oracle.decode(d, m, idx, coef.astype(np.float64))
    for dt, tol in ((torch.float32, TOL_F32), (torch.bfloat16, TOL_BF16)):
        compare_dense(dpb.decode(plan, di, dc, dt).float().cpu().numpy(), ref, tol)
        g = inputs.normal(idx.shape[:1] + (d,), 9700 + d, "f32").to(dt)
        rgc, rgx = oracle.decode_bwd(d, m, idx, g.double().numpy())
        gc, gx = dpb.decode_bwd(plan, di, g.to(DEV), gx_dtype=torch.float32)
        compare_dense(gc.cpu().numpy(), rgc, TOL_F32)
        compare_dense(gx.cpu().numpy(), rgx, TOL_F32)


# enough rows that every wave of the persistent grids takes several groups
STREAMED = {"cpt4_d200": 60000, "odd_d": 40000, "cpt16": 24000, "many_words": 24000, "cpt8": 40000, "few_parents": 24000,
            "table_3l": 24000, "table_k0": 24000, "wide_code": 24000}


@pytest.mark.parametrize("name", list(STREAMED))
def test_streamed_groups_match_single_ones(name):
    """Codes of every kind, shuffled and repeated over so many groups that each
    wave goes on to further ones (the prefetched codes and gradient rows, the
    marks, tables and columns a group leaves behind): every copy of a row is
    within the bar of the oracle's, and all copies decode to the same bits,
    whichever tokens share their waves."""
    d, nb, K = PLANS[name][:3]
    T, n = STREAMED[name], 23
    print(f"[streamed] {name} T={T}", flush=True)
    plan = dpb.Plan(d, seed=0, level_bits=list(nb), branchings=[0] + [branch(name)] * (len(nb) - 1), active=list(K))
    idx, coef = codes(name, n, 9000 + d)
    pick = torch.from_numpy(np.random.default_rng(9900 + d).integers(0, n, T)).to(DEV)
    di, dc = torch.from_numpy(idx).to(DEV), torch.from_numpy(coef).to(DEV)
    bi, bc = di[pick].contiguous(), dc[pick].contiguous()
    m = oracle.masks(d, nb[-1])
    ref = torch.from_numpy(oracle.decode(d, m, idx, coef.astype(np.float64))).to(DEV)

    def check(got, want, tol):
        want = want.to(DEV)
        den = torch.maximum(want.abs(), want.square().mean(-1, keepdim=True).sqrt())
        den = torch.where(den == 0, torch.ones_like(den), den)
        for lo in range(0, T, 8192):
            p = pick[lo:lo + 8192]
            err = ((got[lo:lo + 8192].double() - want[p]).abs() / den[p]).max()
            assert err <= tol, (lo, float(err))

    for dt, tol in ((torch.float32, TOL_F32), (torch.bfloat16, TOL_BF16)):
        y = dpb.decode(plan, bi, bc, dt)
        check(y, ref, tol)
        first = torch.zeros(n, dtype=torch.long, device=DEV).scatter_(0, pick.flip(0), torch.arange(T - 1, -1, -1, device=DEV))
        assert torch.equal(y, y[first][pick])            # copies of a row agree wherever they stand
        g = inputs.normal((n, d), 9100 + d, "f32").to(dt)
        rgc, rgx = oracle.decode_bwd(d, m, idx, g.double().numpy())
        gc, gx = dpb.decode_bwd(plan, bi, g.to(DEV)[pick].contiguous(), gx_dtype=dt)
        check(gc, torch.from_numpy(rgc), TOL_F32)
        check(gx, torch.from_numpy(rgx), tol)


def _call_us(fn, reps=9, inner=4):
    for _ in range(3):
        fn()
    ev = [[torch.cuda.Event(enable_timing=True) for _ in range(2)] for _ in range(reps)]
    for a, b in ev:
        a.record()
        for _ in range(inner):
            fn()
        b.record()
    torch.cuda.synchronize()
    return sorted(a.elapsed_time(b) * 1000 / inner for a, b in ev)[reps // 2]


def test_codes_of_unlisted_leaves_keep_the_table_rate():
    """A code of leaves alone (parents taken off) decodes through tables as a
    whole code does: at 16,384 tokens of d 768, k 96 it takes 1.9 to 2.0 times
    the whole code's time.  Added one by one the 64 leaves took 6.4 times."""
    d, nb, K = PLANS["cpt8"][:3]
    plan = dpb.Plan(d, seed=0, level_bits=list(nb), branchings=[0] + [16] * (len(nb) - 1), active=list(K))
    x = inputs.normal((16384, d), 9800, "bf16").to(DEV)
    idx, coef = dpb.encode(plan, x)
    leaves, lc = idx.clone(), coef.clone()
    leaves[:, : sum(K[:-1])] = -1
    lc[:, : sum(K[:-1])] = 0
    whole = _call_us(lambda: dpb.decode(plan, idx, coef, torch.bfloat16))
    alone = _call_us(lambda: dpb.decode(plan, leaves, lc, torch.bfloat16))
    print(f"[leaf-only decode] whole {whole:.1f} us, leaves alone {alone:.1f} us", flush=True)
    assert alone < 3.5 * whole
