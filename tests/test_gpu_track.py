"""GPU parity of the schedule-track calls against the oracle: reward and advantage of a step
(Algorithm 1, Eq. 6) and the adaptive-stopping elimination (Section 5).

Bars: advantages and rewards within 1e-6 of their oracle scale (|r| + |gamma V(s')| + |V(s)| for
the advantage, |r| for the reward) -- a handful of fp32 roundings; the exact variant bit-exact;
eliminations bit-exact against the oracle applied to the same fp32 advantages."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from synth import gen_track_step, get_config
from tests.gpu_util import assert_close_scaled, log, require_gpu

pytestmark = pytest.mark.gpu


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def gpu_advantage(step, gamma, eps):
    import torch
    from paper_2211_11172_amd import harl
    n = step["c_prev"].size
    d = {k: _dev(v) for k, v in step.items()}
    r = torch.full((max(n, 1),), np.nan, dtype=torch.float32, device="cuda")
    a = torch.full((max(n, 1),), np.nan, dtype=torch.float32, device="cuda")
    harl.harl_track_advantage(d["c_prev"], d["c_next"], d["v_prev"], d["v_next"], n, gamma, eps, r, a)
    torch.cuda.synchronize()
    return r.cpu().numpy()[:n], a.cpu().numpy()[:n]


def gpu_eliminate(adv, n_keep, rows=None, ws_fill=None):
    import torch
    from paper_2211_11172_amd import harl
    n = adv.size
    ad = _dev(adv.astype(np.float32))
    keep = torch.full((max(n_keep, 1),), -7, dtype=torch.int32, device="cuda")
    wsb = harl.harl_track_eliminate_workspace_size(n)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    if ws_fill is not None:
        ws.fill_(ws_fill)
    rows_d = rows_out = None
    row_bytes = 0
    if rows is not None:
        rows_d = _dev(rows)
        row_bytes = rows.shape[1] * rows.itemsize
        rows_out = torch.zeros((max(n_keep, 1), rows.shape[1]), dtype=rows_d.dtype, device="cuda")
    harl.harl_track_eliminate(ad, n, n_keep, keep, rows_d, row_bytes, rows_out, ws, wsb)
    torch.cuda.synchronize()
    out = keep.cpu().numpy()[:n_keep]
    return out, (rows_out.cpu().numpy()[:n_keep] if rows is not None else None)


@pytest.mark.parametrize("n", [1, 255, 256, 257, 4096, 100003])
def test_advantage_matches_oracle(n):
    require_gpu()
    cfg = get_config("standard")
    step = gen_track_step(cfg, n=n)
    step["c_prev"][::17] = 0.0                     # zero scores: the eps floor
    step["c_prev"][5::23] *= np.float32(1e-8)      # |C(s)| below eps
    log("track advantage parity: n=%d" % n)
    r, a = gpu_advantage(step, 0.9, 1e-6)
    want = oracle.track_advantage(step["c_prev"], step["c_next"], step["v_prev"], step["v_next"], gamma=0.9, eps=1e-6)
    assert_close_scaled(r, want["reward"], np.abs(want["reward"]) + 1e-30, 1e-6, "reward")
    assert_close_scaled(a, want["adv"], want["scale"] + 1e-30, 1e-6, "advantage")


def test_advantage_exact_variant_bitwise():
    require_gpu()
    step = gen_track_step(get_config("throughput", exact=True))
    r, a = gpu_advantage(step, 0.5, 1e-6)
    want = oracle.track_advantage(step["c_prev"], step["c_next"], step["v_prev"], step["v_next"], gamma=0.5, eps=1e-6)
    np.testing.assert_array_equal(r.astype(np.float64), want["reward"])
    np.testing.assert_array_equal(a.astype(np.float64), want["adv"])


def test_advantage_special_values():
    require_gpu()
    step = dict(c_prev=np.array([0.0, np.nan, 2.0, -2.0, 1.0], np.float32),
                c_next=np.array([0.5, 1.0, np.nan, -1.0, np.inf], np.float32),
                v_prev=np.array([0.0, 0.0, 0.0, np.nan, 0.0], np.float32),
                v_next=np.zeros(5, np.float32))
    r, a = gpu_advantage(step, 0.9, 0.25)
    assert r[0] == 2.0 and np.isnan(r[1]) and np.isnan(r[2]) and r[3] == 0.5 and np.isposinf(r[4])
    assert a[0] == 2.0 and np.isnan(a[1]) and np.isnan(a[2]) and np.isnan(a[3]) and np.isposinf(a[4])


def _adv_values(n, kind, seed):
    rng = np.random.default_rng(seed)
    if kind == "normal":
        return rng.standard_normal(n).astype(np.float32)
    if kind == "ties":
        pool = np.array([-1.5, -0.0, 0.0, 0.25, 0.5, 2.0, np.nan, np.inf, -np.inf], np.float32)
        return rng.choice(pool, n).astype(np.float32)
    if kind == "equal":
        return np.full(n, 0.75, np.float32)
    if kind == "quantised":   # few distinct values near each other: ties across every digit
        return (rng.integers(0, 40, n) * np.float32(1e-3)).astype(np.float32)
    raise ValueError(kind)


@pytest.mark.parametrize("n", [2, 3, 100, 4095, 4096, 4097, 16384, 16385, 40001, 65536, 65537, 100003])
@pytest.mark.parametrize("kind", ["normal", "ties", "quantised"])
def test_eliminate_matches_oracle(n, kind):
    require_gpu()
    adv = _adv_values(n, kind, seed=n)
    for n_keep in sorted({1, n // 2, n - n // 2, n - 1, n}):
        if n_keep < 1:
            continue
        log("track eliminate parity: n=%d kind=%s n_keep=%d" % (n, kind, n_keep))
        got, _ = gpu_eliminate(adv, n_keep, ws_fill=0xA5)
        np.testing.assert_array_equal(got, oracle.track_eliminate(adv, n_keep))


def test_eliminate_all_equal_and_large():
    require_gpu()
    adv = _adv_values(10000, "equal", 0)
    got, _ = gpu_eliminate(adv, 3333)
    np.testing.assert_array_equal(got, np.arange(3333))
    adv = _adv_values(1_048_576 + 77, "quantised", 1)
    n_keep = oracle.eliminate_count(adv.size)
    log("track eliminate parity: n=%d n_keep=%d" % (adv.size, n_keep))
    got, _ = gpu_eliminate(adv, n_keep)
    np.testing.assert_array_equal(got, oracle.track_eliminate(adv, n_keep))


@pytest.mark.parametrize("n", [16385, 20480, 20481, 258048, 262143, 262144, 262145])
@pytest.mark.parametrize("kind", ["normal", "few values", "infinities and NaN"])
def test_eliminate_around_the_launch_chains(n, kind):
    """Sizes around one workgroup's limit (16,384), block edges (4,096) and the largest size that picks
    its digits inside the passes (64 blocks), from a workspace of leftover bytes; exact."""
    require_gpu()
    rng = np.random.default_rng(n)
    adv = rng.standard_normal(n).astype(np.float32)
    if kind == "few values":
        adv = rng.choice(np.array([-1.0, -0.0, 0.0, 1.0, 1.0000001], np.float32), n)
    elif kind == "infinities and NaN":
        adv[rng.random(n) < 0.3] = np.inf
        adv[rng.random(n) < 0.3] = -np.inf
        adv[rng.random(n) < 0.3] = np.nan
    for n_keep in (1, n // 2, n - 1):
        got, _ = gpu_eliminate(adv, n_keep, ws_fill=0xFF)
        np.testing.assert_array_equal(got, oracle.track_eliminate(adv, n_keep))


@pytest.mark.parametrize("dtype,width", [(np.float32, 64), (np.uint16, 128), (np.uint8, 7), (np.float32, 3)])
def test_eliminate_gathers_rows(dtype, width):
    require_gpu()
    n = 5000
    adv = _adv_values(n, "ties", 3)
    rows = (np.arange(n * width) % 251).astype(dtype).reshape(n, width)
    n_keep = oracle.eliminate_count(n)
    got, rows_out = gpu_eliminate(adv, n_keep, rows=rows)
    want = oracle.track_eliminate(adv, n_keep)
    np.testing.assert_array_equal(got, want)
    np.testing.assert_array_equal(rows_out, rows[want])
    # keep everything: indices 0..n-1 and a copy of the rows
    got, rows_out = gpu_eliminate(adv, n, rows=rows)
    np.testing.assert_array_equal(got, np.arange(n))
    np.testing.assert_array_equal(rows_out, rows)


def test_advantage_then_eliminate_pipeline():
    """One elimination point of the adaptive-stopping search on the standard round's 4,096
    tracks: advantages on the GPU, elimination of the lower half on the GPU, survivors' states
    compacted."""
    require_gpu()
    cfg = get_config("standard")
    step = gen_track_step(cfg)
    _, a = gpu_advantage(step, 0.9, 1e-6)
    want = oracle.track_advantage(step["c_prev"], step["c_next"], step["v_prev"], step["v_next"])
    assert_close_scaled(a, want["adv"], want["scale"], 1e-6, "advantage")
    n_keep = oracle.eliminate_count(cfg.n_prog)
    states = np.random.default_rng(5).standard_normal((cfg.n_prog, cfg.pol_s)).astype(np.float32)
    keep, rows = gpu_eliminate(a, n_keep, rows=states)
    np.testing.assert_array_equal(keep, oracle.track_eliminate(a, n_keep))
    np.testing.assert_array_equal(rows, states[keep])
    # against the oracle's own fp64 advantages: a survivor may differ only at a near-tie
    ref = oracle.track_eliminate(want["adv"].astype(np.float32), n_keep)
    diff = np.setxor1d(keep, ref)
    if diff.size:
        cut = np.sort(want["adv"])[::-1][n_keep - 1]
        assert np.all(np.abs(want["adv"][diff] - cut) <= 2e-6 * (want["scale"][diff] + abs(cut)))
