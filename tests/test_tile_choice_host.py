"""The form and cuts of a product in tiles: the library's search, which passes over candidates that cannot win, against the same model over all
of them.  (The model as the comment above tile_plan states it; without a GPU the library assumes 256 compute units.)"""
import math
import random

import pytest

from paper_2504_11816_amd import binding

FORMS = [(256, 256, 1.442, False), (256, 192, 1.23, False), (128, 256, 0.825, False), (192, 128, 0.7245, False), (128, 128, 0.5305, True),
         (96, 128, 0.416, True), (64, 128, 0.374, True), (64, 64, 0.2256, True), (32, 64, 0.164, True)]


def whole_search(m, n_out, n_in, workspace, n_cus=256):
    stages = (n_in + 63) // 64
    best = None
    for rows, cols, stage, shares_cu in FORMS:
        tiles = -(-m // rows) * -(-n_out // cols)
        for s in range(1, 9):
            if s > 1 and (stages // s < 4 or s * m * n_out * 4 > workspace):
                break
            q = tiles * s / n_cus
            whole = math.ceil(q)
            stage_us = 1.12 * stage if rows == 192 and n_in % 64 and q > 1 else stage
            rounds = 0.5 * (whole + max(1.0, q)) if shares_cu else whole
            shares_mb = s * m * n_out * 4 / 1e6 if s > 1 else 0.0
            t = 4.0 + n_out * n_in * 2 / 1e6 / 19.4 + rounds * (-(-stages // s)) * stage_us * (1.0 - 0.08 * (1.0 - min(1.0, q)))
            if s > 1:
                t += 2.8 + shares_mb / 4.7
                t = 1.01 * t + 0.3 * max(0.0, shares_mb - 134.0) + (0.045 * shares_mb if m <= 192 else 0.0)
            if best is None or t < best[0]:
                best = (t, rows, cols, s)
    return best[1:]


@pytest.mark.parametrize("lo,hi", [(9, 96), (97, 128), (129, 192), (193, 1024), (1025, 4096)])
def test_form_and_cuts(lo, hi):
    r = random.Random(lo)
    tiles = 0
    for _ in range(1500):
        m, n_out = r.randint(lo, hi), 16 * round(math.exp(r.uniform(0, math.log(2600))))
        n_in = 32 * round(math.exp(r.uniform(math.log(2), math.log(640))))
        workspace = r.choice([binding.okv_linear_workspace_bytes(m, n_out, n_in), r.randint(0, 8) * m * n_out * 4])
        plan = binding.okv_linear_plan(m, n_out, n_in, workspace)
        if plan[0] == 2:
            tiles += 1
            assert tuple(plan[1:]) == whole_search(m, n_out, n_in, workspace), (m, n_out, n_in, workspace)
    assert tiles > 150
