"""GPU parity: bs_logsoftmax_reuse_check against the oracle (oracle/logsoftmax.py).

Both sides run the test in fp64 on the same seeded logits and Philox draws; the trial means
and se of the four statistics must agree to 1e-9 of their size (fp64 sums in different orders).
The paper's configuration (eps = 0.1, 128 classes, 64 rows, 4096 trials) is also checked
against the closed forms within a few se.
"""
import numpy as np
import pytest
import torch

from oracle import logsoftmax as ls
from oracle import philox

pytestmark = pytest.mark.gpu


def inputs(rows, C, seed):
    g = torch.Generator().manual_seed(600 + seed)
    z = torch.randn(rows, C, generator=g, dtype=torch.float64) * 2.0
    y = torch.randint(0, C, (rows,), generator=g, dtype=torch.int32)
    return z, y


def run(lib, rows, C, K, eps, seed, calibrate=False):
    z, y = inputs(rows, C, seed)
    print(f"[lsm] rows={rows} C={C} K={K} eps={eps} calibrate={calibrate}", flush=True)
    got = lib.logsoftmax_reuse_check(z.cuda(), y.cuda(), eps=eps, K=K, seed=seed, store_id=1,
                                     calibrate=calibrate).cpu().numpy()
    return z, y, got


@pytest.mark.parametrize("rows,C,K,eps,calibrate", [(3, 8, 40, 0.1, False), (5, 132, 33, 0.35, True),
                                                    (1, 4, 1, 0.2, False), (7, 260, 70, 0.05, False),
                                                    (4, 16, 300, 0.1, False)])
def test_statistics_match_oracle(lib, rows, C, K, eps, calibrate):
    z, y, got = run(lib, rows, C, K, eps, seed=rows, calibrate=calibrate)
    ref = ls.check(z.numpy(), y.numpy(), eps=eps, K=K, seed=rows, store_id=1, calibrate=calibrate)
    for i, name in enumerate(ls.STATS):
        m, se = ref[name]
        scale = max(abs(m), se, 1e-300)
        assert abs(got[i, 0] - m) <= 1e-9 * scale, (name, got[i, 0], m)
        assert abs(got[i, 1] - se) <= 1e-9 * max(se, 1e-300) or (K == 1 and got[i, 1] == 0), (name, got[i, 1], se)


@pytest.mark.parametrize("rows,C,K", [
    (2100, 16, 20),     # 16 lanes per trial, 2 trials per lane, a ragged last chunk of trials
    (1030, 68, 70),     # 17 groups on 32 lanes, two trials side by side, 16 per lane
    (2050, 200, 17),    # 50 groups on 64 lanes, 8 trials per wave and one more
    (3, 516, 9),        # 256 threads per row in the preparation, one trial per wave
    (2100, 16, 140),    # 16 lanes per trial, 16 trials per lane, three waves
    (2050, 200, 41),    # 64 lanes, 16 trials per wave, three waves
    (2100, 132, 9),     # 4 trials per wave, the last wave with one
    (2100, 16, 3),      # fewer trials than lie side by side in a wave
    (2100, 516, 1),     # one trial: blocks of one wave
    (2, 4100, 5),       # 1024 threads per row, the lanes' last group ragged
    (1, 8, 4100),       # more than 4096 trials: 64 per block of the reduction
])
def test_lane_and_trial_splits_match_oracle(lib, rows, C, K):
    """The edges of the trial kernel's lane groups, its two trial counts and both reductions; the
    tolerance is that of test_statistics_match_oracle (fp64 sums in different orders)."""
    test_statistics_match_oracle(lib, rows, C, K, 0.1, False)


@pytest.mark.slow
def test_rows_past_one_launch(lib):
    """2^24 + 5 rows of one Philox group: more blocks than a launch's grid dimension holds threads for."""
    rows, C, eps, seed = (1 << 24) + 5, 4, 0.1, 9
    z, y, got = run(lib, rows, C, 1, eps, seed)
    total = dict.fromkeys(ls.STATS, 0.0)
    for r0 in range(0, rows, 1 << 20):
        zc, yc = z[r0:r0 + (1 << 20)].numpy(), y[r0:r0 + (1 << 20)].numpy()
        row = np.arange(r0, r0 + len(yc), dtype=np.uint64)
        draw = [np.stack(philox.philox4x32_10(row, np.uint64(0), np.uint64(1), np.uint64(256 + use), np.uint64(seed),
                                              np.uint64(0)), axis=1) for use in (0, 1)]
        r, rp = [np.where(w >= np.uint64(1 << 31), eps, -eps) for w in draw]
        for name, e in ls.entry_errors(ls.log_softmax(zc), yc, r, rp).items():
            total[name] += e.sum()
    for i, name in enumerate(ls.STATS):
        m = total[name] / (rows * C)
        assert abs(got[i, 0] - m) <= 1e-9 * abs(m) and got[i, 1] == 0, (name, got[i], m)


def test_targets_outside_the_classes_match_none(lib):
    """A target outside [0, C) makes the likelihood's h zero on that row, on both sides."""
    z, y = inputs(4, 12, 3)
    y[1], y[3] = -1, 12
    got = lib.logsoftmax_reuse_check(z.cuda(), y.cuda(), eps=0.1, K=50, seed=3, store_id=1).cpu().numpy()
    ref = ls.check(z.numpy(), y.numpy(), eps=0.1, K=50, seed=3, store_id=1)
    for i, name in enumerate(ls.STATS):
        m, se = ref[name]
        assert abs(got[i, 0] - m) <= 1e-9 * max(abs(m), se, 1e-300), (name, got[i, 0], m)


def test_papers_configuration_matches_closed_forms(lib):
    eps = 0.1
    _, _, got = run(lib, 64, 128, 4096, eps, seed=9)
    target = [np.cosh(eps) - 1, np.cosh(eps) - 1, -eps * np.sinh(eps), 0.0]
    for i, name in enumerate(ls.STATS):
        assert abs(got[i, 0] - target[i]) < 5 * got[i, 1], (name, got[i])
    assert abs(got[2, 0]) > 50 * got[2, 1]                 # reuse's effect is resolved
    _, _, cal = run(lib, 64, 128, 4096, eps, seed=9, calibrate=True)
    assert abs(cal[0, 0]) < 5 * cal[0, 1]                  # LS5a: the likelihood's error is removed
    assert abs(cal[2, 0] + eps * np.tanh(eps)) < 5 * cal[2, 1]   # LS5b: reuse's effect / cosh(eps)


def test_rejected_arguments(lib):
    z, y = inputs(2, 6, 0)
    with pytest.raises(lib.BspError):
        lib.logsoftmax_reuse_check(z.cuda(), y.cuda(), K=4, ws=torch.empty(1 << 16, dtype=torch.uint8, device="cuda"))
