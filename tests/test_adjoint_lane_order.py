"""The adjoints' order of a footprint's pixels over the lanes, restated in FP32 numpy
(pixel_order and group_pixel of backward.hip): every pixel of every view comes exactly
once and padding nowhere, for batches of one view and batches over the views' ends,
column groups of ku, 2 ku and 4 ku, up to 32 columns and row classes per voxel, and
footprints of more than 2^22 pixels (whose quotients take the remainder step)."""
import random

import numpy as np
import pytest

F = np.float32


def _layout(w, h, pu, pv, siddon):
    ku = max(int(np.ceil(F(min(pu, 32.0)) - F(0.1))), 1)
    kv = max(int(np.ceil(F(min(pv, 32.0)) - F(0.1))), 1)
    hp = (h + kv - 1) // kv
    wide = (4 if hp <= 5 else 2) if not siddon and kv <= 2 and hp <= 16 else 1
    per = wide * ku * kv * hp
    return dict(w=w, h=h, ku=ku, kv=kv, hp=hp, wide=wide, per=per, rk=(65536 + wide * ku - 1) // (wide * ku),
                rcol=F(1) / F(per), rrow=F(1) / F(hp), n=(w + wide * ku - 1) // (wide * ku) * per)


def _pixel(g, p, large):
    def quotient(i, r, n):
        q = ((i.astype(F) + F(0.5)) * r).astype(np.int64)
        if large:
            rem = i - q * n
            q += np.where(rem >= n, 1, np.where(rem < 0, -1, 0))
        return q

    cg = quotient(p, g["rcol"], g["per"])
    r = p - cg * g["per"]
    ab = quotient(r, g["rrow"], g["hp"])
    r = r - ab * g["hp"]
    a = (ab * g["rk"]) >> 16
    b = ab - a * g["wide"] * g["ku"]
    du = cg * g["wide"] * g["ku"] + (b >> (g["wide"] >> 1)) + (b & (g["wide"] - 1)) * g["ku"]
    return du, a + g["kv"] * r


def _check(g, p, large):
    du, dv = _pixel(g, p, large)
    assert (du >= 0).all() and (dv >= 0).all()
    ok = (du < g["w"]) & (dv < g["h"])
    assert np.array_equal(np.sort(dv[ok] * g["w"] + du[ok]), np.arange(g["w"] * g["h"]))


@pytest.mark.parametrize("siddon", [True, False])
def test_every_pixel_once(siddon):
    rng = random.Random(3)
    for _ in range(1500):
        w, h = (rng.choice([1, 2, 5, 16, 17, rng.randint(1, 60), rng.randint(1, 300)]) for _ in range(2))
        pu, pv = (rng.choice([0.05, 1.0, 1.1, 1.11, 2.1, 2.11, 8.0, 15.0, 32.0, 50.0, rng.uniform(0.1, 40.0)]) for _ in range(2))
        g = _layout(w, h, pu, pv, siddon)
        # batches of one view: whole batches of 64, so indices run past n
        _check(g, np.arange((g["n"] + 63) // 64 * 64), False)
    for w, h, pu, pv in ((3000, 2500, 30.0, 31.0), (4000, 1500, 2.0, 1.5), (70, 65535, 1.0, 2.0), (65535, 70, 1.0, 30.0)):
        g = _layout(w, h, pu, pv, siddon)
        _check(g, np.arange(g["n"]), g["n"] > 1 << 22)


@pytest.mark.parametrize("gv", [16, 32])
def test_batches_over_the_views_ends(gv):
    rng = random.Random(gv)
    for _ in range(60):
        gs = [_layout(rng.randint(1, 20), rng.randint(1, 12), rng.uniform(0.05, 1.5), rng.uniform(0.05, 1.5), False) if rng.random() < 0.7 else None
              for _ in range(gv)]
        pre = np.concatenate([[0], np.cumsum([g["n"] if g else 0 for g in gs])])
        p = np.arange((pre[-1] + 63) // 64 * 64)
        view = np.zeros_like(p)
        st = gv // 2
        while st:
            view += np.where(p >= pre[view + st], st, 0)
            st //= 2
        inside = p < pre[-1]
        for k, g in enumerate(gs):
            mine = p[inside & (view == k)] - pre[k]
            assert len(mine) == (g["n"] if g else 0)
            if g:
                _check(g, mine, False)
