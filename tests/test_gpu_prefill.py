"""GPU parity: bc_prefill_attn (beacon-masked prefill attention, forward) against the dense
masked-attention oracle, and against bc_decode_attn over the evicted cache (training-time
masking simulates the eviction).  bf16 inputs, fp32 accumulation: max-abs-error 2e-3."""
import numpy as np
import pytest

from oracle import attention as OA
from paper_2510_13797_amd import workloads as W

pytestmark = pytest.mark.gpu
TOL = 2e-3


@pytest.fixture(scope="module")
def dev():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch.device("cuda:0")


# every forward test runs through both entry points: bc_prefill_attn and, when FORM says so,
# bc_prefill_attn_ws (V copied to half precision in a workspace, weights in one half-precision part)
FORM = {"workspace": False}


@pytest.fixture(params=["plain", "workspace"])
def form(request):
    """Which forward entry point _run() goes through."""
    FORM["workspace"] = request.param == "workspace"
    yield request.param
    FORM["workspace"] = False


def _run(pw, dev, want_lse=True, qkv=None):
    from paper_2510_13797_amd import bc
    bc.load()
    qkv = [pw.qkv(b) for b in range(pw.B)] if qkv is None else qkv
    off = np.zeros(pw.B + 1, np.int64)
    off[1:] = np.cumsum(pw.S)
    q = bc.to_device(np.concatenate([x[0] for x in qkv]), "bf16", dev)
    k = bc.to_device(np.concatenate([x[1] for x in qkv]), "bf16", dev)
    v = bc.to_device(np.concatenate([x[2] for x in qkv]), "bf16", dev)
    out, lse = bc.prefill_attn(q, k, v, off, pw.P, pw.c, pw.Hq, pw.Hkv, pw.d, pw.scale, want_lse,
                               workspace=FORM["workspace"])
    return qkv, off, out.cpu().numpy(), None if lse is None else lse.cpu().numpy()


def _check_rows(pw, qkv, off, out, lse, b, rows):
    q, k, v = qkv[b]
    ref, ref_lse = OA.masked_prefill_attention(q, k, v, int(pw.P[b]), int(pw.c[b]), pw.scale, rows=rows)
    got = out[off[b] + np.asarray(rows)]
    err = float(np.abs(got - ref).max())
    assert err <= TOL, (b, err)
    if lse is not None:
        lerr = float(np.abs(lse[off[b] + np.asarray(rows)] - ref_lse).max())
        assert lerr <= 1e-3, (b, lerr)
    return err


@pytest.mark.parametrize("Hq,Hkv", [(12, 2), (4, 1), (8, 8), (2, 2), (7, 1), (8, 1), (5, 1), (3, 1), (4, 2)])
def test_prefill_small_ragged_all_rows(dev, Hq, Hkv, form):
    pw = W.PrefillWorkload("pf_small", 50 + Hq, 6, Hq, Hkv, 128, "bf16",
                           np.array([0, 5, 64, 70, 33, 200], np.int32),      # prompt rows
                           np.array([150, 64, 1, 130, 97, 0], np.int32),     # response tokens
                           np.array([16, 2, 4, 0, 1, 16], np.int32))         # c (0: plain causal)
    qkv, off, out, lse = _run(pw, dev)
    assert np.isfinite(out).all()
    for b in range(pw.B):
        _check_rows(pw, qkv, off, out, lse, b, list(range(int(pw.S[b]))))


@pytest.mark.parametrize("Hq,Hkv", [(12, 2), (4, 4), (8, 1), (7, 1), (5, 1), (2, 2)])
def test_prefill_head_dimension_64_all_rows(dev, Hq, Hkv, form):
    # rows of 128 bytes: eight rows per LDS-DMA instruction, two k-steps, four output blocks, the
    # swizzle of the 8-unit rows; ragged trajectories with and without prompt, several ratios
    pw = W.PrefillWorkload("pf_d64", 64 + Hq, 4, Hq, Hkv, 64, "bf16", np.array([37, 0, 129, 64], np.int32),
                           np.array([300, 190, 75, 0], np.int32), np.array([4, 16, 0, 3], np.int32))
    qkv, off, out, lse = _run(pw, dev)
    assert np.isfinite(out).all()
    for b in range(pw.B):
        _check_rows(pw, qkv, off, out, lse, b, list(range(int(pw.S[b]))))


def test_prefill_ratios_and_long_beacon_runs(dev, form):
    # many beacons (several gathered beacon tiles) and every ratio the paper uses
    pw = W.PrefillWorkload("pf_ratios", 61, 5, 12, 2, 128, "bf16", np.array([3, 40, 128, 7, 256], np.int32),
                           np.array([700, 900, 1000, 1100, 1200], np.int32),
                           np.array([2, 4, 8, 16, 32], np.int32))
    qkv, off, out, lse = _run(pw, dev)
    rng = np.random.default_rng(0)
    for b in range(pw.B):
        S = int(pw.S[b])
        rows = sorted(set([0, 1, S - 1, S - 2, int(pw.P[b]), max(int(pw.P[b]) - 1, 0)])
                      | set(int(x) for x in rng.integers(0, S, size=150)))
        _check_rows(pw, qkv, off, out, lse, b, rows)


def test_config5_full_size(dev, form):
    pw = W.prefill_train()
    assert int(pw.S[0]) == 8688
    qkv, off, out, lse = _run(pw, dev)
    assert np.isfinite(out).all()
    rng = np.random.default_rng(1)
    # a band of consecutive rows across tile and window borders, every beacon-tile border, and
    # random rows of every trajectory
    worst = _check_rows(pw, qkv, off, out, lse, 0, list(range(0, 400)) + list(range(8300, 8688)))
    for b in range(pw.B):
        rows = sorted(set(int(x) for x in rng.integers(0, 8688, size=120)))
        worst = max(worst, _check_rows(pw, qkv, off, out, lse, b, rows))
    # every row of four (trajectory, query head) slices: first and last trajectory, heads of both
    # KV heads, first and last head of a group
    g = pw.Hq // pw.Hkv
    for b, h in ((0, 0), (0, pw.Hq - 1), (pw.B - 1, g - 1), (7, g)):
        q, k, v = qkv[b]
        kvh = h // g
        ref, ref_lse = OA.masked_prefill_attention(q[:, h:h + 1], k[:, kvh:kvh + 1], v[:, kvh:kvh + 1],
                                                   int(pw.P[b]), int(pw.c[b]), pw.scale)
        got = out[off[b]:off[b + 1], h:h + 1]
        err = float(np.abs(got - ref).max())
        lerr = float(np.abs(lse[off[b]:off[b + 1], h:h + 1] - ref_lse).max())
        assert err <= TOL and lerr <= 1e-3, (b, h, err, lerr)
        worst = max(worst, err)
    print("config5 worst", worst)


@pytest.mark.parametrize("d", [128, 64])
def test_prefill_rows_equal_decode_over_evicted_cache(dev, d, form):
    # Sec. 3.2: masking simulates eviction.  Feed the same q/k/v through the decode path
    # (append, attend, beacon append at the tail, attend with the beacon's query, evict) and
    # compare every row with the prefill output.
    from paper_2510_13797_amd import bc
    P, c, R = 37, 8, 475
    pw = W.PrefillWorkload("pf_eq", 62, 2, 12, 2, d, "bf16", np.full(2, P, np.int32),
                           np.full(2, R, np.int32), np.full(2, c, np.int32))
    qkv, off, out, _ = _run(pw, dev, want_lse=False)
    S = int(pw.S[0])
    assert S == P + R + R // c
    B = pw.B
    q = np.stack([x[0] for x in qkv]); k = np.stack([x[1] for x in qkv]); v = np.stack([x[2] for x in qkv])
    cap = np.full(B, P + R // c + c + 1, np.int32)
    rt = bc.Runtime(B, pw.Hq, pw.Hkv, pw.d, "bf16", pw.scale, pw.P, pw.c, cap, dev)
    rt.cache_init([k[b, :P] for b in range(B)], [v[b, :P] for b in range(B)])
    worst = 0.0
    row = P
    for t in range(1, R + 1):
        rt.append_kv(k[:, row], v[:, row])
        o = rt.decode_attn(q[:, row]).cpu().numpy()
        for b in range(B):
            worst = max(worst, float(np.abs(o[b] - out[off[b] + row]).max()))
        row += 1
        if t % c == 0:                                   # beacon row
            rt.append_kv(k[:, row], v[:, row], kind=bc.BC_ROW_BEACON)
            o = rt.decode_attn(q[:, row]).cpu().numpy()
            for b in range(B):
                worst = max(worst, float(np.abs(o[b] - out[off[b] + row]).max()))
            rt.compress_evict()
            row += 1
    assert row == S
    assert rt.tables()[2] == 0
    assert worst <= TOL, worst
    print("prefill vs decode worst", worst)


def test_prefill_argument_errors(dev):
    from paper_2510_13797_amd import bc
    import ctypes as C
    import torch
    x = torch.zeros(64, dtype=torch.float32, device=dev)
    p = C.c_void_p(x.data_ptr())
    sh32 = bc.bc_shape(1, 4, 1, 128, bc.BC_F32, 0.1)
    assert bc.bc_prefill_attn(sh32, p, p, p, p, p, p, 4, p, None, None) == -2      # bf16 only
    sh = bc.bc_shape(1, 4, 1, 128, bc.BC_BF16, 0.1)
    assert bc.bc_prefill_attn(sh, None, p, p, p, p, p, 4, p, None, None) == -1
    assert bc.bc_prefill_attn(sh, p, p, p, p, p, p, 0, p, None, None) == -1


# ---------------------------------------------------------------------------
# backward (next row): gradients against the dense fp64 oracle
# ---------------------------------------------------------------------------
def _run_bwd(pw, dev, half_forward=False):
    from paper_2510_13797_amd import bc
    qkv = [pw.qkv(b) for b in range(pw.B)]
    dos = [pw.dout(b) for b in range(pw.B)]
    off = np.zeros(pw.B + 1, np.int64)
    off[1:] = np.cumsum(pw.S)
    q = bc.to_device(np.concatenate([x[0] for x in qkv]), "bf16", dev)
    k = bc.to_device(np.concatenate([x[1] for x in qkv]), "bf16", dev)
    v = bc.to_device(np.concatenate([x[2] for x in qkv]), "bf16", dev)
    do = bc.to_device(np.concatenate(dos), "bf16", dev)
    # (out and lse from bc_prefill_attn, or from bc_prefill_attn_ws when the caller says so)
    out, lse = bc.prefill_attn(q, k, v, off, pw.P, pw.c, pw.Hq, pw.Hkv, pw.d, pw.scale, True, workspace=half_forward)
    dq, dk, dv = bc.prefill_attn_bwd(q, k, v, out, lse, do, off, pw.P, pw.c, pw.Hq, pw.Hkv, pw.d, pw.scale)
    return qkv, dos, off, dq.cpu().numpy(), dk.cpu().numpy(), dv.cpu().numpy()


def _check_bwd(pw, qkv, dos, off, dq, dk, dv, b):
    q, k, v = qkv[b]
    rq, rk, rv = OA.masked_prefill_attention_bwd(q, k, v, dos[b], int(pw.P[b]), int(pw.c[b]), pw.scale)
    sl = slice(int(off[b]), int(off[b + 1]))
    errs = [float(np.abs(g[sl] - r).max()) for g, r in ((dq, rq), (dk, rk), (dv, rv))]
    assert max(errs) <= TOL, (b, errs)
    return errs


@pytest.mark.parametrize("Hq,Hkv", [(12, 2), (4, 1), (8, 8), (6, 2), (7, 1), (8, 1), (5, 1)])
def test_prefill_bwd_small_ragged(dev, Hq, Hkv):
    pw = W.PrefillWorkload("pf_bwd", 55 + Hq, 6, Hq, Hkv, 128, "bf16",
                           np.array([0, 5, 64, 70, 33, 200], np.int32),
                           np.array([150, 64, 1, 130, 97, 0], np.int32),
                           np.array([16, 2, 4, 0, 1, 16], np.int32))
    qkv, dos, off, dq, dk, dv = _run_bwd(pw, dev)
    assert np.isfinite(dq).all() and np.isfinite(dk).all() and np.isfinite(dv).all()   # every element written
    for b in range(pw.B):
        _check_bwd(pw, qkv, dos, off, dq, dk, dv, b)


@pytest.mark.parametrize("Hq,Hkv", [(12, 2), (4, 4), (8, 1), (7, 1), (5, 1)])
def test_prefill_bwd_head_dimension_64(dev, Hq, Hkv):
    # the gradients at d = 64: every element of dq, dk, dv of ragged trajectories (head splits of
    # the dense key blocks and the fixed-order reduction included) against the dense oracle
    pw = W.PrefillWorkload("pfb_d64", 164 + Hq, 4, Hq, Hkv, 64, "bf16", np.array([37, 0, 129, 64], np.int32),
                           np.array([300, 190, 75, 0], np.int32), np.array([4, 16, 0, 3], np.int32))
    qkv, dos, off, dq, dk, dv = _run_bwd(pw, dev)
    assert np.isfinite(dq).all() and np.isfinite(dk).all() and np.isfinite(dv).all()
    for b in range(pw.B):
        _check_bwd(pw, qkv, dos, off, dq, dk, dv, b)


def test_prefill_bwd_many_beacons(dev):
    pw = W.PrefillWorkload("pf_bwd2", 63, 3, 12, 2, 128, "bf16", np.array([3, 128, 256], np.int32),
                           np.array([900, 1300, 1000], np.int32), np.array([2, 8, 16], np.int32))
    qkv, dos, off, dq, dk, dv = _run_bwd(pw, dev)
    assert np.isfinite(dq).all() and np.isfinite(dk).all() and np.isfinite(dv).all()
    worst = [0, 0, 0]
    for b in range(pw.B):
        worst = [max(a, e) for a, e in zip(worst, _check_bwd(pw, qkv, dos, off, dq, dk, dv, b))]
    print("bwd worst dq/dk/dv", worst)


def test_config5_bwd_full_size(dev):
    # B = 2 trajectories of the config-5 shape (8688 rows each); the dense fp64 oracle is run
    # on the first one in full
    pw = W.prefill_train(B=2)
    qkv, dos, off, dq, dk, dv = _run_bwd(pw, dev)
    assert np.isfinite(dq).all() and np.isfinite(dk).all() and np.isfinite(dv).all()
    errs = _check_bwd(pw, qkv, dos, off, dq, dk, dv, 0)
    print("config5 bwd dq/dk/dv", errs)


@pytest.mark.parametrize("B,Hq,Hkv", [(8, 1, 1), (5, 8, 8), (3, 48, 16), (9, 14, 7), (67, 2, 1), (72, 1, 1), (65, 2, 2)])
def test_prefill_pairs_that_change_places_from_row_to_row(dev, B, Hq, Hkv, form):
    # numbers of (trajectory, KV head) pairs that fill rows of eight, one row to many, or are padded to them (63, 67): every row and
    # every gradient element of every pair
    rng = np.random.default_rng([20251013, 79, B, Hkv])
    P, R = rng.integers(1, 40, size=B).astype(np.int32), rng.integers(0, 150, size=B).astype(np.int32)
    pw = W.PrefillWorkload("pf_turn", 400 + B, B, Hq, Hkv, 64, "bf16", P, R, rng.choice([0, 2, 5, 16], size=B).astype(np.int32))
    qkv, off, out, lse = _run(pw, dev)
    _, dos, _, dq, dk, dv = _run_bwd(pw, dev)
    for b in range(pw.B):
        _check_rows(pw, qkv, off, out, lse, b, list(range(int(pw.S[b]))))
        _check_bwd(pw, qkv, dos, off, dq, dk, dv, b)


@pytest.mark.parametrize("case", range(8))
def test_prefill_randomised_forward_and_backward(dev, case, form):
    # seeded random trajectory counts, prompt and response lengths, ratios and head layouts;
    # every row of the forward and every gradient element against the oracle
    rng = np.random.default_rng([20251013, 78, case])
    Hq, Hkv = [(12, 2), (4, 4), (8, 1), (6, 2), (7, 1), (5, 5), (16, 2), (3, 1)][case]
    B = int(rng.integers(1, 6))
    P = rng.integers(0, 150, size=B).astype(np.int32)
    R = rng.integers(0, 260, size=B).astype(np.int32)
    R[(P == 0) & (R == 0)] = 1
    c = rng.choice([0, 1, 2, 3, 7, 16, 33], size=B).astype(np.int32)
    pw = W.PrefillWorkload("pf_rand%d" % case, 300 + case, B, Hq, Hkv, 128, "bf16", P, R, c)
    qkv, off, out, lse = _run(pw, dev)
    assert np.isfinite(out).all()
    for b in range(pw.B):
        _check_rows(pw, qkv, off, out, lse, b, list(range(int(pw.S[b]))))
    qkv, dos, off, dq, dk, dv = _run_bwd(pw, dev)
    assert np.isfinite(dq).all() and np.isfinite(dk).all() and np.isfinite(dv).all()
    for b in range(pw.B):
        _check_bwd(pw, qkv, dos, off, dq, dk, dv, b)


def test_prefill_long_trajectory(dev, form):
    # a 32k-token response (the longest generation the paper's setups allow) in one trajectory:
    # 2,048 beacons, 64 gathered beacon tiles per late query tile; sampled rows against the oracle
    pw = W.PrefillWorkload("pf_long", 64, 1, 12, 2, 128, "bf16", np.array([512], np.int32),
                           np.array([32768], np.int32), np.array([16], np.int32))
    S = int(pw.S[0])
    assert S == 512 + 32768 + 2048
    qkv, off, out, lse = _run(pw, dev)
    assert np.isfinite(out).all()
    rng = np.random.default_rng(4)
    rows = sorted(set([0, 511, 512, 528, 529, S - 1, S - 2, S - 17, S - 18])
                  | set(int(x) for x in rng.integers(0, S, size=160)))
    _check_rows(pw, qkv, off, out, lse, 0, rows)


class _PeakedKeys:
    """A PrefillWorkload whose keys have a wide range of magnitudes: every 64th key row is scaled
    by 4 and the last quarter of every trajectory by 2 (both exact in bf16), so that the softmax
    is dominated by few keys and its running reference has to move many times."""

    def __init__(self, pw):
        self._pw = pw

    def __getattr__(self, name):
        return getattr(self._pw, name)

    def qkv(self, b):
        q, k, v = self._pw.qkv(b)
        k = k.copy()
        k[63::64] *= 4.0
        k[3 * len(k) // 4:] *= 2.0
        return q, k, v


def test_prefill_peaked_keys_forward_and_backward(dev, form):
    pw = _PeakedKeys(W.PrefillWorkload("pf_peak", 65, 3, 12, 2, 128, "bf16", np.array([5, 100, 256], np.int32),
                                       np.array([600, 900, 300], np.int32), np.array([16, 4, 0], np.int32)))
    qkv, off, out, lse = _run(pw, dev)
    assert np.isfinite(out).all()
    for b in range(pw.B):
        _check_rows(pw, qkv, off, out, lse, b, list(range(int(pw.S[b]))))
    qkv, dos, off, dq, dk, dv = _run_bwd(pw, dev)
    assert np.isfinite(dq).all() and np.isfinite(dk).all() and np.isfinite(dv).all()
    for b in range(pw.B):
        _check_bwd(pw, qkv, dos, off, dq, dk, dv, b)


def test_prefill_ratio_whose_window_index_needs_more_than_32_bits(dev, form):
    # c = 65535: rows * (c + 1) passes 2^32 inside the third window, where a multiply-high
    # estimate of offset / (c + 1) is one too large unless it is corrected (offset 131071, the
    # second beacon, is the first such place).  Forward rows and gradients around both beacons
    # and in the short third window, against the oracle's per-place sums.
    P, c = 24, 65535
    R = 2 * c + 150
    pw = W.PrefillWorkload("pf_wide_ratio", 66, 1, 2, 1, 128, "bf16", np.array([P], np.int32),
                           np.array([R], np.int32), np.array([c], np.int32))
    S = int(pw.S[0])
    assert S == P + R + 2 and (S - P) * (c + 1) > 2 ** 32
    b1, b2 = P + c, P + 2 * c + 1                      # the two beacon rows
    assert OA.is_beacon_row(b1, P, c) and OA.is_beacon_row(b2, P, c)
    qkv, dos, off, dq, dk, dv = _run_bwd(pw, dev)
    _, _, out, lse = _run(pw, dev)
    assert np.isfinite(out).all() and np.isfinite(dq).all() and np.isfinite(dk).all() and np.isfinite(dv).all()
    rows = [0, P - 1, P, b1 - 1, b1, b1 + 1, b2 - 2, b2 - 1, b2, b2 + 1, b2 + 2, b2 + 77, S - 2, S - 1]
    _check_rows(pw, qkv, off, out, lse, 0, rows)
    # keys whose columns are short enough to sum on the CPU: the tail of the second window, its
    # beacon, the third window
    keys = [b2 - 3, b2 - 1, b2, b2 + 1, b2 + 40, S - 1]
    q, k, v = qkv[0]
    rq, rk, rv = OA.masked_prefill_attention_bwd_at(q, k, v, dos[0], P, c, pw.scale, rows, keys)
    errs = [float(np.abs(dq[rows] - rq).max()), float(np.abs(dk[keys] - rk).max()),
            float(np.abs(dv[keys] - rv).max())]
    assert max(errs) <= TOL, errs


def test_values_beyond_half_precision_take_the_two_part_form(dev):
    # one V entry of 1e5 (finite in bf16, beyond half precision): the workspace entry point must
    # notice it on the device and compute what the plain entry point computes - bit for bit; and a
    # V whose entries all fit gives the half-precision form, which differs in the last bits but
    # stays inside the tolerance (checked by every other test of this file)
    pw = W.PrefillWorkload("pf_range", 67, 2, 12, 2, 128, "bf16", np.array([40, 7], np.int32),
                           np.array([200, 90], np.int32), np.array([16, 4], np.int32))
    qkv = [list(pw.qkv(b)) for b in range(pw.B)]
    qkv[1][2] = qkv[1][2].copy()
    qkv[1][2][50, 1, 77] = np.float32(99840.0)            # exact in bf16
    keep = FORM["workspace"]
    try:
        FORM["workspace"] = False
        _, off, plain, lse_plain = _run(pw, dev, qkv=qkv)
        FORM["workspace"] = True
        _, _, withws, lse_ws = _run(pw, dev, qkv=qkv)
    finally:
        FORM["workspace"] = keep
    assert np.array_equal(plain, withws) and np.array_equal(lse_plain, lse_ws)
    for b in range(pw.B):
        q, k, v = qkv[b]
        rows = list(range(int(pw.S[b])))
        ref, _ = OA.masked_prefill_attention(q, k, v, int(pw.P[b]), int(pw.c[b]), pw.scale, rows=rows)
        got = plain[off[b] + np.asarray(rows)]
        assert np.abs(got - ref).max() <= TOL * max(1.0, float(np.abs(ref).max()))


def test_gradients_from_the_half_form_forward(dev):
    # out and lse of the workspace form (weights in one half-precision part: out within 2e-3, but
    # some 70 times further from the oracle than the two-part form) fed to the backward: on N(0,1)
    # trajectories the gradients stay inside the same absolute bound.  The error of out enters the
    # gradients through Delta = sum(dO * out), scaled by the size of dO and K: with keys scaled
    # up as in the peaked-keys test it reaches 2.8e-3, so where gradients must meet the bound
    # whatever the data, the forward to use is bc_prefill_attn (which every other backward test takes).
    pw = W.PrefillWorkload("pf_half_bwd", 68, 3, 12, 2, 128, "bf16", np.array([37, 0, 129], np.int32),
                           np.array([300, 190, 75], np.int32), np.array([4, 16, 0], np.int32))
    qkv, dos, off, dq, dk, dv = _run_bwd(pw, dev, half_forward=True)
    assert np.isfinite(dq).all() and np.isfinite(dk).all() and np.isfinite(dv).all()
    for b in range(pw.B):
        _check_bwd(pw, qkv, dos, off, dq, dk, dv, b)


@pytest.mark.parametrize("P", [31, 32, 33, 64, 65])
@pytest.mark.parametrize("R", [62, 63, 64, 65, 129])
def test_prefill_key_list_at_the_edges_of_its_tiles(dev, P, R, form):
    # a query tile's keys are full tiles of prompt rows and of beacons, then a tail of what is left of
    # both with the band behind it: prompt lengths and beacon counts (c = 1: one beacon per token) just
    # below, at and above whole tiles, trajectories that end inside the first or second 32-row block
    pw = W.PrefillWorkload("pf_edges", 69, 2, 2, 1, 128, "bf16", np.array([P, P], np.int32),
                           np.array([R, R + 32], np.int32), np.array([1, 2], np.int32))
    qkv, off, out, lse = _run(pw, dev)
    assert np.isfinite(out).all()
    for b in range(pw.B):
        _check_rows(pw, qkv, off, out, lse, b, list(range(int(pw.S[b]))))


@pytest.mark.parametrize("d", [128, 64])
def test_prefill_addresses_beyond_32_bits(dev, d):
    # max_rows is an upper bound the caller states; from 4 GB of K rows on the kernel with 64-bit
    # offsets is launched, which must compute the same, bit for bit, as the one with 32-bit offsets
    import ctypes as C
    import torch
    from paper_2510_13797_amd import bc
    pw = W.PrefillWorkload("pf_wide", 70, 2, 16, 8, d, "bf16", np.array([37, 70], np.int32),
                           np.array([300, 90], np.int32), np.array([4, 0], np.int32))
    qkv = [pw.qkv(b) for b in range(pw.B)]
    off = np.zeros(pw.B + 1, np.int64)
    off[1:] = np.cumsum(pw.S)
    q, k, v = (bc.to_device(np.concatenate([x[i] for x in qkv]), "bf16", dev) for i in range(3))
    shape = bc.bc_shape(pw.B, pw.Hq, pw.Hkv, d, bc.BC_BF16, pw.scale)
    tab = [torch.from_numpy(x).to(dev) for x in (off, pw.P, pw.c)]
    ptr = lambda t: C.c_void_p(t.data_ptr())
    most = (1 << 32) // (pw.Hkv * d * 2) + 7
    got = []
    for max_rows in (int(pw.S.max()), most):
        out = torch.full((int(off[-1]), pw.Hq, d), float("nan"), device=dev)
        assert bc.bc_prefill_attn(shape, ptr(q), ptr(k), ptr(v), *map(ptr, tab), max_rows, ptr(out), None, None) == 0
        torch.cuda.synchronize()
        got.append(out.cpu().numpy())
    assert np.isfinite(got[0]).all() and np.array_equal(got[0], got[1])


def test_rows_in_front_of_the_first_trajectory_have_no_gradient(dev):
    # row_offsets[0] > 0: those rows belong to no trajectory; every other row is written
    import torch
    from paper_2510_13797_amd import bc
    S, first, P = 70, 5, 20
    g = torch.Generator(device=dev).manual_seed(3)
    q, k, v, do = (torch.randn(first + S, h, 128, generator=g, device=dev).to(torch.bfloat16) for h in (4, 2, 2, 4))
    args = (np.array([first, first + S]), [P], [4], 4, 2, 128, 128 ** -0.5)
    out, lse = bc.prefill_attn(q, k, v, *args)
    grads = bc.prefill_attn_bwd(q, k, v, out, lse, do, *args)
    alone = bc.prefill_attn_bwd(q[first:].contiguous(), k[first:].contiguous(), v[first:].contiguous(), out[first:].contiguous(),
                                lse[first:].contiguous(), do[first:].contiguous(), np.array([0, S]), *args[1:])
    for x, y in zip(grads, alone):
        assert torch.isnan(x[:first]).all() and torch.equal(x[first:], y)


@pytest.mark.parametrize("P", [31, 33, 64, 65])
@pytest.mark.parametrize("R,Hq,Hkv,d", [(62, 2, 1, 128), (65, 5, 1, 128), (129, 3, 3, 128), (700, 6, 1, 64)])
def test_prefill_bwd_key_blocks_and_their_parts_at_the_edges(dev, P, R, Hq, Hkv, d):
    # 64 keys per block, 32 per pair of waves, tiles of 32 rows, dense blocks whole and in two to eight
    # parts, windows that end inside and behind a tile; results and workspace hold NaN before the call:
    # what is not written, or read before it is written, shows
    import torch
    from paper_2510_13797_amd import bc
    pw = W.PrefillWorkload("pfb_edges", 71, 3, Hq, Hkv, d, "bf16", np.array([P, P, 0], np.int32),
                           np.array([R, R + 32, 33], np.int32), np.array([1, 6, 16], np.int32))
    qkv = [pw.qkv(b) for b in range(pw.B)]
    dos = [pw.dout(b) for b in range(pw.B)]
    off = np.concatenate([[0], np.cumsum(pw.S)]).astype(np.int64)
    q, k, v, do = (bc.to_device(np.concatenate(x), "bf16", dev) for x in (*zip(*qkv), dos))
    out, lse = bc.prefill_attn(q, k, v, off, pw.P, pw.c, Hq, Hkv, d, pw.scale)
    total, most = int(off[-1]), int(pw.S.max())
    nan = lambda *shape: torch.full(shape, float("nan"), device=dev)
    dq, dk, dv = nan(total, Hq, d), nan(total, Hkv, d), nan(total, Hkv, d)
    shape = bc.bc_shape(pw.B, Hq, Hkv, d, bc.BC_BF16, pw.scale)
    ws = nan(bc.bc_prefill_bwd_workspace_bytes(shape, total) // 4)
    tables = [torch.from_numpy(x).to(dev) for x in (off, pw.P, pw.c)]
    p = lambda t: t.data_ptr()
    st = bc.bc_prefill_attn_bwd(shape, p(q), p(k), p(v), p(out), p(lse), p(do), *map(p, tables), most, total, p(dq), p(dk),
                                p(dv), p(ws), ws.numel() * 4, None)
    assert st == bc.BC_OK
    torch.cuda.synchronize()
    dq, dk, dv = (x.cpu().numpy() for x in (dq, dk, dv))
    for b in range(pw.B):
        _check_bwd(pw, qkv, dos, off, dq, dk, dv, b)


@pytest.mark.parametrize("P", [1, 64])
@pytest.mark.parametrize("R,Hq,Hkv,d", [(1, 12, 2, 128), (63, 7, 1, 128), (65, 8, 1, 64), (190, 18, 3, 64)])
def test_prefill_bwd_response_blocks_in_parts(dev, P, R, Hq, Hkv, d):
    # groups of six heads and more on a chip that is not full: response blocks in two to four parts too, every row summed
    test_prefill_bwd_key_blocks_and_their_parts_at_the_edges(dev, P, R, Hq, Hkv, d)


@pytest.mark.parametrize("P,R,c,Hq,Hkv,d", [(5, 900, 32, 12, 2, 128), (130, 500, 1, 6, 1, 128), (60, 640, 0, 6, 1, 64), (64, 1100, 300, 8, 1, 64),
                                             (5, 1900, 32, 7, 1, 64), (5, 1400, 16, 8, 1, 128)])
def test_prefill_bwd_as_many_parts_as_there_is_room_for(dev, P, R, c, Hq, Hkv, d):
    # one trajectory on an idle chip: few dense keys, two thirds and all of the rows dense, a last window that stays open, chains of 427 and 368
    # tiles (sixteen parts); workspace and results hold NaN before the call
    import torch
    from paper_2510_13797_amd import bc
    pw = W.PrefillWorkload("pfb_room", 73, 1, Hq, Hkv, d, "bf16", np.array([P], np.int32), np.array([R], np.int32), np.array([c], np.int32))
    qkv, dos = [pw.qkv(0)], [pw.dout(0)]
    off, total = np.array([0, pw.S[0]], np.int64), int(pw.S[0])
    q, k, v, do = (bc.to_device(x[0], "bf16", dev) for x in (*zip(*qkv), dos))
    out, lse = bc.prefill_attn(q, k, v, off, pw.P, pw.c, Hq, Hkv, d, pw.scale)
    dq, dk, dv = (torch.full(shape, float("nan"), device=dev) for shape in ((total, Hq, d), (total, Hkv, d), (total, Hkv, d)))
    shape = bc.bc_shape(1, Hq, Hkv, d, bc.BC_BF16, pw.scale)
    ws = torch.full((bc.bc_prefill_bwd_workspace_bytes(shape, total) // 4,), float("nan"), device=dev)
    tables = [torch.from_numpy(x).to(dev) for x in (off, pw.P, pw.c)]
    st = bc.bc_prefill_attn_bwd(shape, *(t.data_ptr() for t in (q, k, v, out, lse, do, *tables)), total, total,
                                *(t.data_ptr() for t in (dq, dk, dv, ws)), ws.numel() * 4, None)
    assert st == bc.BC_OK
    torch.cuda.synchronize()
    _check_bwd(pw, qkv, dos, off, dq.cpu().numpy(), dk.cpu().numpy(), dv.cpu().numpy(), 0)


@pytest.mark.parametrize("P,R,c,Hq,Hkv,d", [
    ([11, 11, 11, 11], [592] * 4, [16] * 4, 12, 2, 128), ([11, 11, 12, 11], [592] * 4, [16] * 4, 12, 2, 128),   # 10 x 24 workgroups of dq, 11 x 24
    ([80, 80, 80, 80], [1476] * 4, [3] * 4, 8, 1, 64), ([80, 81, 80, 80], [1476] * 4, [3] * 4, 8, 1, 64),       # four pairs: 64 x 8, 65 x 8
    ([1, 0, 700, 40], [0, 33, 3, 0], [5, 0, 2, 4], 7, 1, 64), ([31, 64, 1], [65, 32, 700], [1, 16, 300], 3, 3, 128)])
def test_prefill_bwd_in_one_launch_and_in_two(dev, P, R, c, Hq, Hkv, d):
    # both sides of the lines up to which the two kinds of workgroup are one launch, and trajectories of very different length in one;
    # workspace and results hold NaN before the call
    import torch
    from paper_2510_13797_amd import bc
    B, i32 = len(P), lambda x: np.array(x, np.int32)
    pw = W.PrefillWorkload("pfb_joined", 79, B, Hq, Hkv, d, "bf16", i32(P), i32(R), i32(c))
    qkv, dos = [pw.qkv(b) for b in range(B)], [pw.dout(b) for b in range(B)]
    off = np.concatenate([[0], np.cumsum(pw.S)]).astype(np.int64)
    total, most = int(off[-1]), int(pw.S.max())
    q, k, v, do = (bc.to_device(np.concatenate(x), "bf16", dev) for x in (*zip(*qkv), dos))
    out, lse = bc.prefill_attn(q, k, v, off, pw.P, pw.c, Hq, Hkv, d, pw.scale)
    dq, dk, dv = (torch.full((total, h, d), float("nan"), device=dev) for h in (Hq, Hkv, Hkv))
    shape = bc.bc_shape(B, Hq, Hkv, d, bc.BC_BF16, pw.scale)
    ws = torch.full((bc.bc_prefill_bwd_workspace_bytes(shape, total) // 4,), float("nan"), device=dev)
    tables = [torch.from_numpy(x).to(dev) for x in (off, pw.P, pw.c)]
    st = bc.bc_prefill_attn_bwd(shape, *(t.data_ptr() for t in (q, k, v, out, lse, do, *tables)), most, total,
                                *(t.data_ptr() for t in (dq, dk, dv, ws)), ws.numel() * 4, None)
    assert st == bc.BC_OK
    torch.cuda.synchronize()
    dq, dk, dv = (x.cpu().numpy() for x in (dq, dk, dv))
    for b in range(B):
        _check_bwd(pw, qkv, dos, off, dq, dk, dv, b)


@pytest.mark.parametrize("P,R,c,Hq,Hkv,d", [([60, 5], [2200, 40], [2, 0], 5, 5, 64), ([2100, 3], [300, 64], [16, 1], 5, 5, 128),
                                            ([7, 130], [0, 900], [4, 1], 6, 1, 64)])
def test_prefill_bwd_sums_of_parts_in_keys_and_slices(dev, P, R, c, Hq, Hkv, d):
    # the sums' waves: two and three slices of a key's heads, more items than waves; four keys a wave; response rows with and without beacons among them
    test_prefill_bwd_in_one_launch_and_in_two(dev, P, R, c, Hq, Hkv, d)


@pytest.mark.parametrize("Hq,Hkv,d,B,longest", [
    (14, 2, 64, 67, 300), (14, 2, 128, 16, 700), (7, 1, 128, 65, 200), (2, 1, 64, 130, 400), (9, 3, 128, 20, 700), (12, 4, 64, 13, 700), (25, 5, 64, 4, 1100),
    (20, 4, 128, 7, 700), (2, 2, 64, 100, 700), (24, 8, 64, 3, 1100), (16, 8, 128, 9, 900)])
def test_prefill_bwd_in_two_launches(dev, Hq, Hkv, d, B, longest):
    # batches beyond the line for one launch, every kind of group and padded numbers of pairs (67, 65, 130 and 100 trajectories): one long trajectory,
    # beside it one of no rows, of one and of 33, all others of up to a third; workspace and results hold NaN before the call
    import torch
    from paper_2510_13797_amd import bc
    from test_prefill_grid import in_one_launch
    r = np.random.default_rng([Hq, Hkv, d, B])
    P, R, c = r.integers(0, 40, B), r.integers(1, longest // 3, B), r.choice([0, 1, 3, 16], B)
    P[:2], R[:2], c[:2] = (17, 33), (longest, 0), (4, 5)
    if B > 3:
        P[2:4], R[2:4] = (0, 0), (0, 1)
        P[-1], R[-1], c[-1] = 40, 170, 16
    i32 = lambda x: x.astype(np.int32)
    pw = W.PrefillWorkload("pfb_two", 83, B, Hq, Hkv, d, "bf16", i32(P), i32(R), i32(c))
    qkv, dos = [pw.qkv(b) for b in range(B)], [pw.dout(b) for b in range(B)]
    off = np.concatenate([[0], np.cumsum(pw.S)]).astype(np.int64)
    total, most = int(off[-1]), int(pw.S.max())
    assert not in_one_launch(B, Hq, Hkv, total)
    q, k, v, do = (bc.to_device(np.concatenate(x), "bf16", dev) for x in (*zip(*qkv), dos))
    out, lse = bc.prefill_attn(q, k, v, off, pw.P, pw.c, Hq, Hkv, d, pw.scale)
    dq, dk, dv = (torch.full((total, h, d), float("nan"), device=dev) for h in (Hq, Hkv, Hkv))
    shape = bc.bc_shape(B, Hq, Hkv, d, bc.BC_BF16, pw.scale)
    ws = torch.full((bc.bc_prefill_bwd_workspace_bytes(shape, total) // 4,), float("nan"), device=dev)
    tables = [torch.from_numpy(x).to(dev) for x in (off, pw.P, pw.c)]
    st = bc.bc_prefill_attn_bwd(shape, *(t.data_ptr() for t in (q, k, v, out, lse, do, *tables)), most, total,
                                *(t.data_ptr() for t in (dq, dk, dv, ws)), ws.numel() * 4, None)
    assert st == bc.BC_OK
    torch.cuda.synchronize()
    dq, dk, dv = (x.cpu().numpy() for x in (dq, dk, dv))
    for b in range(B):
        if pw.S[b]:
            _check_bwd(pw, qkv, dos, off, dq, dk, dv, b)


@pytest.mark.parametrize("d", [128, 64])
def test_prefill_bwd_addresses_beyond_32_bits(dev, d):
    # as above for the gradients: 512 heads make rows of 128 or 64 KB, so a stated 4 GB of K rows needs
    # little workspace; the same bits as with 32-bit offsets
    import torch
    from paper_2510_13797_amd import bc
    H, S = 512, 150
    g = torch.Generator(device=dev).manual_seed(5)
    q, k, v, do = (torch.randn(S, H, d, generator=g, device=dev).to(torch.bfloat16) for _ in range(4))
    out, lse = bc.prefill_attn(q, k, v, [0, S], [37], [4], H, H, d, d ** -0.5)
    shape = bc.bc_shape(1, H, H, d, bc.BC_BF16, d ** -0.5)
    tab = [torch.from_numpy(x).to(dev) for x in (np.array([0, S]), np.array([37], np.int32), np.array([4], np.int32))]
    p = lambda t: t.data_ptr()
    got = []
    for rows in (S, (1 << 32) // (H * d * 2) + 7):
        grads = [torch.full((S, H, d), float("nan"), device=dev) for _ in range(3)]
        ws = torch.empty(bc.bc_prefill_bwd_workspace_bytes(shape, rows), dtype=torch.uint8, device=dev)
        assert bc.bc_prefill_attn_bwd(shape, p(q), p(k), p(v), p(out), p(lse), p(do), *map(p, tab), rows, rows,
                                      *map(p, grads), p(ws), ws.numel(), None) == bc.BC_OK
        torch.cuda.synchronize()
        got.append(grads)
    for x, y in zip(*got):
        assert torch.isfinite(x).all() and torch.equal(x, y)


@pytest.mark.parametrize("Hq,Hkv,d", [(8, 8, 64), (16, 8, 128)])
def test_prefill_bwd_parts_follow_the_dense_keys_of_a_trajectory(dev, Hq, Hkv, d):
    # uncompressed trajectories (every key dense: blocks whole, or in two parts for groups of two) beside
    # compressed ones (few dense blocks, in parts) in one call; workspace and results hold NaN before it
    import torch
    from paper_2510_13797_amd import bc
    B = 12
    pw = W.PrefillWorkload("pfb_parts", 72, B, Hq, Hkv, d, "bf16", np.full(B, 30, np.int32), np.full(B, 490, np.int32),
                           np.resize(np.array([0, 6, 0, 16], np.int32), B))
    qkv = [pw.qkv(b) for b in range(B)]
    dos = [pw.dout(b) for b in range(B)]
    off = np.concatenate([[0], np.cumsum(pw.S)]).astype(np.int64)
    q, k, v, do = (bc.to_device(np.concatenate(x), "bf16", dev) for x in (*zip(*qkv), dos))
    out, lse = bc.prefill_attn(q, k, v, off, pw.P, pw.c, Hq, Hkv, d, pw.scale)
    total = int(off[-1])
    nan = lambda *shape: torch.full(shape, float("nan"), device=dev)
    dq, dk, dv = nan(total, Hq, d), nan(total, Hkv, d), nan(total, Hkv, d)
    shape = bc.bc_shape(B, Hq, Hkv, d, bc.BC_BF16, pw.scale)
    need = bc.bc_prefill_bwd_workspace_bytes(shape, total)
    assert (need - total * Hq * 8) // (2 * total * Hkv * d * 4) >= 2          # there is room for two parts
    ws = nan(need // 4)
    tables = [torch.from_numpy(x).to(dev) for x in (off, pw.P, pw.c)]
    p = lambda t: t.data_ptr()
    assert bc.bc_prefill_attn_bwd(shape, p(q), p(k), p(v), p(out), p(lse), p(do), *map(p, tables), int(pw.S.max()), total,
                                  p(dq), p(dk), p(dv), p(ws), ws.numel() * 4, None) == bc.BC_OK
    torch.cuda.synchronize()
    dq, dk, dv = (x.cpu().numpy() for x in (dq, dk, dv))
    assert np.isfinite(dq).all() and np.isfinite(dk).all() and np.isfinite(dv).all()
    for b in (0, 1, B - 1):
        _check_bwd(pw, qkv, dos, off, dq, dk, dv, b)


@pytest.mark.parametrize("B", [1, 31, 32, 62, 63, 249, 250, 700])
def test_tables_that_travel_in_kernel_arguments(dev, B):
    # 31 trajectories fit the small form (126 words), 249 one launch of the large one (1000); one array and three
    import torch
    from paper_2510_13797_amd import bc
    r = np.random.default_rng(B)
    host = np.empty(2 * B + 1, np.int64)
    host[:B + 1] = np.cumsum(r.integers(1, 1 << 33, B + 1))
    pc = host[B + 1:].view(np.int32)
    pc[:] = r.integers(-5, 1 << 30, 2 * B)
    off, P, c = host[:B + 1].copy(), pc[:B].copy(), pc[B:].copy()
    at = host.ctypes.data
    for arrays in ((at, at + 8 * (B + 1), at + 8 * (B + 1) + 4 * B), (off.ctypes.data, P.ctypes.data, c.ctypes.data)):
        out = torch.full((2 * B + 2,), -1, dtype=torch.int64, device=dev)
        assert bc.bc_trajectory_tables(*arrays, B, out.data_ptr(), None) == bc.BC_OK
        got = out.cpu().numpy()
        assert np.array_equal(got[:-1], host) and got[-1] == -1
    assert bc.bc_trajectory_tables(at, at, at, B, None, None) == bc.BC_ERR_ARG
    assert bc.bc_trajectory_tables(at, at, at, B, out.data_ptr() + 4, None) == bc.BC_ERR_ARG
    assert bc.bc_trajectory_tables(at, at, at, 0, out.data_ptr(), None) == bc.BC_ERR_SHAPE


def _small_training_step(dev, seed):
    import torch
    g = torch.Generator(device=dev).manual_seed(seed)
    off, P, c = np.array([0, 300, 700, 1900]), np.array([20, 0, 64], np.int32), np.array([4, 0, 16], np.int32)
    rnd = lambda h: torch.randn(1900, h, 128, generator=g, device=dev).to(torch.bfloat16)
    return (off, P, c, 6, 2, 128, 128 ** -0.5), [rnd(6), rnd(2), rnd(2)], rnd(6)


def test_inputs_of_another_stream_may_be_freed_behind_the_call(dev):
    # the calls only enqueue their work: memory of inputs that were made on another stream must not be given
    # out again there before that work has read it
    import torch
    from paper_2510_13797_amd import bc
    args, qkv, do = _small_training_step(dev, 7)
    want, lse = bc.prefill_attn(*qkv, *args)
    want_grads = bc.prefill_attn_bwd(*qkv, want, lse, do, *args)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    for _ in range(3):
        with torch.cuda.stream(side):
            copies, do2 = [x.clone() for x in qkv], do.clone()
        side.synchronize()
        big = torch.empty(1 << 28, dtype=torch.uint8, device=dev)
        for _ in range(4):
            big.fill_(1)                                  # keeps the calls' work waiting
        out, lse2 = bc.prefill_attn(*copies, *args)
        grads = bc.prefill_attn_bwd(*copies, out, lse2, do2, *args)
        sizes = [x.shape for x in copies] + [do2.shape]
        del copies, do2
        with torch.cuda.stream(side):
            junk = [torch.full(n, float("nan"), dtype=torch.bfloat16, device=dev) for n in sizes]
        torch.cuda.synchronize()
        assert torch.equal(out, want) and all(torch.equal(a, b) for a, b in zip(grads, want_grads))
        del junk


def test_training_calls_captured_in_a_graph(dev):
    # forward, gradients and both passes of the loss in one graph: replayed on other inputs, with eager work and
    # synchronizations between the replays, every replay equal to the eager calls
    import torch
    from paper_2510_13797_amd import bc
    args, qkv, do = _small_training_step(dev, 8)
    z = torch.randn(64, 3001, device=dev).to(torch.bfloat16)
    tl, idx = torch.randn(64, 9, device=dev), torch.randint(0, 3001, (64, 9), device=dev, dtype=torch.int32)

    def step():
        ws_out, _ = bc.prefill_attn(*qkv, *args, workspace=True)
        out, lse = bc.prefill_attn(*qkv, *args)
        loss, zlse, mean = bc.topk_kl_loss(z, tl, idx)
        return [ws_out, out, lse, loss, zlse, mean, bc.topk_kl_loss_bwd(z, tl, idx, zlse, 0.5),
                *bc.prefill_attn_bwd(*qkv, out, lse, do, *args)]

    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        step()
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            got = step()
    for seed in (11, 12, 13):
        _, qkv2, do2 = _small_training_step(dev, seed)
        for x, y in zip(qkv + [do], qkv2 + [do2]):
            x.copy_(y)
        z.normal_()
        torch.cuda.synchronize()
        want = [x.clone() for x in step()]
        with torch.cuda.stream(stream):
            graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want)), seed


@pytest.mark.parametrize("B", [1, 15, 16, 17, 40])
def test_host_tables_equal_device_tables(dev, B):
    # up to 16 trajectories travel in the kernels' arguments, more through device memory; all three forms, bit for bit
    import ctypes as C
    import torch
    from paper_2510_13797_amd import bc
    r = np.random.default_rng(B)
    S = r.integers(1, 150, B)
    off = np.concatenate([[0], np.cumsum(S)]).astype(np.int64)
    P, c = r.integers(0, 60, B).astype(np.int32), r.integers(0, 9, B).astype(np.int32)
    R, Hq, Hkv, d = int(off[-1]), 4, 2, 64
    q, k, v, do = (torch.randn(R, h, d, device=dev).to(torch.bfloat16) for h in (Hq, Hkv, Hkv, Hq))
    shape = bc.bc_shape(B, Hq, Hkv, d, bc.BC_BF16, 0.125)
    tab = [torch.from_numpy(x).to(dev) for x in (off, P, c)]
    ptr = lambda t: t.data_ptr()
    outs = [torch.full((R, h, d), float("nan"), device=dev) for h in (Hq, Hq, Hq, Hkv, Hkv)]
    lse = torch.full((R, Hq), float("nan"), device=dev)
    n1, n2 = bc.bc_prefill_workspace_bytes(shape, R), bc.bc_prefill_bwd_workspace_bytes(shape, R)
    ws1, ws2 = (torch.full((n,), 255, dtype=torch.uint8, device=dev) for n in (n1, n2))
    m = int(S.max())
    assert bc.bc_prefill_attn_ws(shape, ptr(q), ptr(k), ptr(v), *map(ptr, tab), m, R, ptr(outs[0]), None, ptr(ws1), n1, None) == 0
    assert bc.bc_prefill_attn(shape, ptr(q), ptr(k), ptr(v), *map(ptr, tab), m, ptr(outs[1]), ptr(lse), None) == 0
    assert bc.bc_prefill_attn_bwd(shape, ptr(q), ptr(k), ptr(v), ptr(outs[1]), ptr(lse), ptr(do), *map(ptr, tab), m, R,
                                  *map(ptr, outs[2:]), ptr(ws2), n2, None) == 0
    args = (off, P, c, Hq, Hkv, d, 0.125)
    got = [bc.prefill_attn(q, k, v, *args, workspace=True)[0], *bc.prefill_attn(q, k, v, *args)]
    got += bc.prefill_attn_bwd(q, k, v, got[1], got[2], do, *args)
    want = [outs[0], outs[1], lse, *outs[2:]]
    assert all(torch.equal(a, b) for a, b in zip(got, want))
    h = [x.ctypes.data for x in (off, P, c)]
    st = bc.bc_prefill_attn_host(shape, ptr(q), ptr(k), ptr(v), *h, m, R, ptr(outs[0]), None, None, None, 0, None)
    assert st == (bc.BC_OK if B <= 16 else bc.BC_ERR_ARG)
    assert bc.bc_prefill_attn_host(shape, ptr(q), ptr(k), ptr(v), *h, m, R, ptr(outs[0]), None, None, ptr(ws1), n1 - 1, None) \
        == bc.BC_ERR_WORKSPACE


@pytest.mark.parametrize("rows,at", [(3, 0), (257, 0), (257, 256), (9000, 8999), (9000, 4097), (16384, 16383), (17000, 16383),
                                     (17000, 16384), (17000, 16999), (70000, 0), (70000, 32767), (70000, 32768), (70000, 50000),
                                     (70000, 65535), (70000, 65536), (70000, 69999)])
def test_every_workgroup_of_the_conversion_pass_has_a_verdict(dev, rows, at):
    # V entries that do not fit half precision, in the first and last rows the pass reads, with few workgroups and
    # with all 256, of which each thread takes a unit in every 16384 rows here, four of them together: in each of the four, in the
    # next round and in the last row.  The two-part form's bits
    import torch
    from paper_2510_13797_amd import bc
    q, k, v = (torch.randn(rows, 2, 64, device=dev).to(torch.bfloat16) for _ in range(3))
    args = (np.array([0, rows]), np.array([min(rows, 32)], np.int32), np.array([4], np.int32), 2, 2, 64, 0.125)
    half = bc.prefill_attn(q, k, v, *args, workspace=True)[0]
    plain = bc.prefill_attn(q, k, v, *args)[0]
    assert not torch.equal(half, plain) and float((half - plain).abs().max()) < 2e-3
    v[at, 1, 63] = 70000.0
    assert torch.equal(bc.prefill_attn(q, k, v, *args, workspace=True)[0], bc.prefill_attn(q, k, v, *args)[0])
