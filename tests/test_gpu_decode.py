"""GPU parity: bc_append_kv / bc_decode_attn / bc_compress_evict against the CPU oracle,
through the C ABI, on the five-config shapes (decode side).  Tolerances: max-abs-error
1e-5 for fp32 inputs, 2e-3 for bf16 inputs (fp32 accumulation); tables, error bits and
resident slab rows bit-exact."""
import numpy as np
import pytest

from oracle import attention as OA
from oracle import residency as OR
from oracle.cache import BatchCache, ERR_CAPACITY, ERR_STATE
from paper_2510_13797_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-5, "bf16": 2e-3}


@pytest.fixture(scope="module")
def dev():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch.device("cuda:0")


def _bc():
    from paper_2510_13797_amd import bc
    bc.load()                       # fails loudly if libbc.so is missing
    return bc


def make(wl, dev, cap=None):
    bc = _bc()
    cap = wl.capacity() if cap is None else cap
    rt = bc.Runtime(wl.B, wl.Hq, wl.Hkv, wl.d, wl.dtype, wl.scale, wl.P, wl.c, cap, dev)
    pk, pv = zip(*[wl.prompt_kv(s) for s in range(wl.B)])
    rt.cache_init(list(pk), list(pv))
    oc = BatchCache(list(pk), list(pv), wl.c, cap)
    return rt, oc


def check_tables(rt, oc, t=None):
    nb, w, err = rt.tables()
    assert list(nb) == oc.nb, ("nb", t)
    assert list(w) == oc.w, ("w", t)
    assert err == oc.err, ("err", t, err, oc.err)
    return nb, w


def check_slabs(rt, oc, seqs=None, t=None):
    nb, w, _ = rt.tables()
    for s in (range(rt.B) if seqs is None else seqs):
        K, V = rt.resident(s, int(nb[s]), int(w[s]))
        Ko, Vo = oc.resident(s)
        assert K.shape == Ko.shape, (s, t)
        assert np.array_equal(K, Ko) and np.array_equal(V, Vo), ("slab", s, t)


def check_attention(o, q, oc, wl, seqs=None, t=None):
    worst = 0.0
    for s in (range(wl.B) if seqs is None else seqs):
        K, V = oc.resident(s)
        ref = OA.decode_attention(q[s], K, V, wl.scale)
        worst = max(worst, float(np.abs(o[s].astype(np.float64) - ref).max()))
    assert worst <= TOL[wl.dtype], (t, worst)
    return worst


def partials_written(rt, filler=0):
    """Whether a call left partial results of a cut sequence in the workspace, whose bytes were `filler` (behind the counters)."""
    counters = -(-rt.B * 128 // 256) * 256 + (-(-rt.B * rt.Hkv * 4 // 256) * 256 if rt.Hkv >= 32 else 0)
    return bool((rt.ws[counters:] != filler).any())


def rollout(wl, rt, oc, steps, attn_steps, slab_steps, table_every=1, tail_form=False,
            use_step_call=False, seq_sample=None, beacon_call=False, before_step=None):
    """Alg. 1 for `steps` decode steps; sequences whose generation is over stay resident."""
    attn_steps, slab_steps = set(attn_steps), set(slab_steps)
    worst = 0.0
    q_any = None
    for t in range(1, steps + 1):
        if before_step is not None:
            before_step(t)
        active = (wl.G >= t).astype(np.uint8)
        act = None if active.all() else active
        k, v = wl.step_kv(t)
        need_attn = t in attn_steps
        if need_attn:
            q = wl.step_q(t)
        elif use_step_call or beacon_call:
            # the step calls need a query; where the output is not compared any will do (drawing one
            # per step is most of the host time of a long rollout)
            q = q_any = wl.step_q(1) if q_any is None else q_any
        else:
            q = None
        bk, bv = wl.beacon_kv(t)
        if beacon_call:
            # token step without eviction, then the beacon's own step (bc_beacon_step): beacon row
            # at the tail, its attention, compaction - one launch each on the bf16 d=128 path
            o = rt.decode_step(k, v, q, None, None, active=act)
            oc.append(k, v, active=act)
            if need_attn:
                seqs = [s for s in (range(wl.B) if seq_sample is None else seq_sample) if active[s]]
                worst = max(worst, check_attention(o.cpu().numpy(), q, oc, wl, seqs, t))
            qb = wl.beacon_q(t) if need_attn else q
            ob = rt.beacon_step(bk, bv, qb, active=act)
            oc.append(bk, bv, active=act, beacon=True)
            due = [s for s in range(wl.B) if active[s] and oc.c[s] > 0 and oc.w[s] == oc.c[s] + 1]
            if need_attn and due:
                worst = max(worst, check_attention(ob.cpu().numpy(), qb, oc, wl, due, t))
            oc.compress_evict(active=act)
        elif use_step_call:
            o = rt.decode_step(k, v, q, bk, bv, active=act)
            oc.append(k, v, active=act)
            if need_attn:
                seqs = [s for s in (range(wl.B) if seq_sample is None else seq_sample) if active[s]]
                worst = max(worst, check_attention(o.cpu().numpy(), q, oc, wl, seqs, t))
            oc.compress_evict(bk, bv, active=act)
        else:
            rt.append_kv(k, v, active=act)
            oc.append(k, v, active=act)
            if need_attn:
                o = rt.decode_attn(q, active=act).cpu().numpy()
                seqs = [s for s in (range(wl.B) if seq_sample is None else seq_sample) if active[s]]
                worst = max(worst, check_attention(o, q, oc, wl, seqs, t))
            if tail_form:
                rt.append_kv(bk, bv, active=act, kind=1)
                oc.append(bk, bv, active=act, beacon=True)
                if need_attn:       # the beacon's own query sees prompt, beacons, window, itself
                    due = [s for s in range(wl.B) if active[s] and oc.c[s] > 0 and oc.w[s] == oc.c[s] + 1]
                    if due:
                        qb = wl.beacon_q(t)
                        dm = np.zeros(wl.B, np.uint8)
                        dm[due] = 1
                        ob = rt.decode_attn(qb, active=dm).cpu().numpy()
                        worst = max(worst, check_attention(ob, qb, oc, wl, due, t))
                rt.compress_evict(active=act)
                oc.compress_evict(active=act)
            else:
                rt.compress_evict(bk, bv, active=act)
                oc.compress_evict(bk, bv, active=act)
        if t % table_every == 0 or t in slab_steps or t == steps:
            check_tables(rt, oc, t)
        if t in slab_steps:
            check_slabs(rt, oc, seq_sample, t)
    return worst


# ---------------------------------------------------------------------------
def test_config1_tiny_every_step(dev):
    wl = W.tiny()
    rt, oc = make(wl, dev)
    steps = range(1, 257)
    worst = rollout(wl, rt, oc, 256, steps, steps)
    nb, w, _ = rt.tables()
    assert list(nb) == [16, 16] and list(w) == [0, 0]
    for s in range(wl.B):       # invariant: L = P + floor(t/c) + (t mod c)
        assert 32 + nb[s] + w[s] == OR.len_after_step(32, 16, 256)
    print("tiny worst", worst)


def test_config1_tail_form_with_beacon_query(dev):
    wl = W.tiny(seed=11)
    rt, oc = make(wl, dev)
    rollout(wl, rt, oc, 80, range(1, 81), range(1, 81), tail_form=True)


def test_config1_fused_step_call(dev):
    wl = W.tiny(seed=12)
    rt, oc = make(wl, dev)
    rollout(wl, rt, oc, 64, range(1, 65), (16, 17, 64), use_step_call=True)


@pytest.mark.parametrize("c,P,d", [(16, 256, 128), (1, 5, 128), (2, 0, 128), (3, 31, 128), (0, 40, 128),
                                   (16, 256, 64), (1, 5, 64), (3, 31, 64)])
def test_fused_step_bf16_every_step(dev, c, P, d):
    # bc_decode_step on the single-launch path (bf16, d = 128 or 64): tables, slabs, outputs each step
    wl = W.Workload("fused", 70 + c, 6, 12, 2, d, "bf16", np.full(6, P, np.int32),
                    np.array([150, 150, 90, 150, 33, 150], np.int32), np.full(6, c, np.int32))
    rt, oc = make(wl, dev)
    steps = range(1, 151)
    rollout(wl, rt, oc, 150, steps, steps, use_step_call=True)


@pytest.mark.parametrize("dtype,d,B", [("f32", 128, 6), ("f32", 64, 6), ("bf16", 128, 6), ("bf16", 64, 6),
                                       ("f32", 128, 2), ("bf16", 128, 2)])
def test_fused_step_on_the_plain_alu_kernel(dev, dtype, d, B):
    # the same single-launch step on the kernel that serves fp32 rows (and bf16 rows when the
    # plan asks for it): ragged ratios with c = 1 and no compression among them, sequences that
    # end early, the budget-free and the beacon-step forms; tables, slabs and outputs each step.
    # B = 2 with a long prompt spreads a sequence's rows over several workgroups, which arrive at
    # their pair's counter; the last folds the partials and takes the pair's ticket.
    P = np.array([1100, 1050], np.int32) if B == 2 else np.array([40, 0, 17, 64, 5, 33], np.int32)
    c = np.array([16, 3], np.int32) if B == 2 else np.array([16, 1, 0, 3, 2, 7], np.int32)
    G = np.array([70, 70], np.int32) if B == 2 else np.array([70, 70, 50, 70, 21, 70], np.int32)
    for beacon_call in (False, True):
        wl = W.Workload("fused_alu", 90 + d + B, B, 4, 2, d, dtype, P, G, c)
        rt, oc = make(wl, dev)
        if dtype == "bf16":
            rt.cache.plan = _bc().BC_PLAN_PLAIN_ALU
        st, text = _bc().bc_decode_plan_describe(rt.shape, rt.cache)
        assert st == 0 and "decode_valu_kernel" in text, text
        if B == 2:
            assert int(text.split("chunks=")[1].split()[0]) > 1, text
        steps = range(1, 71)
        rollout(wl, rt, oc, 70, steps, steps, use_step_call=not beacon_call, beacon_call=beacon_call)


@pytest.mark.parametrize("promise", ["as built", "none", "prompt too long", "prompt too short"])
@pytest.mark.parametrize("Hkv,d", [(2, 128), (8, 128), (2, 64)])
def test_uniform_layout_promise_is_only_a_hint(dev, promise, Hkv, d):
    # equal prompt lengths and capacities: the binding states the layout and the kernel requests prompt
    # rows before it has read the tables; a promise that names another prompt length must not change
    # any result (the rows are requested again); Hkv = 8 takes the one-workgroup-per-pair kernel
    B, P, G = 40, 100, 60
    wl = W.Workload("promise", 97, B, 2 * Hkv, Hkv, d, "bf16", np.full(B, P, np.int32),
                    np.full(B, G, np.int32), np.full(B, 8, np.int32))
    cap = np.full(B, 176, np.int32)
    rt, oc = make(wl, dev, cap)
    assert rt.cache.uniform_P == P and rt.cache.uniform_cap == 176
    if promise == "none":
        rt.cache.uniform_P = rt.cache.uniform_cap = 0
    elif promise == "prompt too long":
        rt.cache.uniform_P = 160           # rows 100..159 are not all resident yet: unwritten slab rows
    elif promise == "prompt too short":
        rt.cache.uniform_P = 64
    rollout(wl, rt, oc, G, (1, 2, 8, 9, 33, 60), (8, 60), use_step_call=True)


@pytest.mark.parametrize("B,Hkv,d,P", [(12, 2, 128, 410), (40, 4, 128, 270), (12, 2, 64, 270)])
def test_second_tiles_of_the_straight_line_kernel(dev, B, Hkv, d, P):
    # short caches run on the straight-line form of the kernel, where a wave has at most two tiles:
    # 24 pairs, d = 128: two twelve-wave workgroups per pair, second tiles from row 384; 160 pairs,
    # and d = 64: eight waves, second tiles from row 256.  The rollout crosses those rows, with the
    # appended row in a first tile, in a second tile and on a tile boundary.
    G, c = 70, 8
    wl = W.Workload("twotiles", 98, B, 2 * Hkv, Hkv, d, "bf16", np.full(B, P, np.int32),
                    np.where(np.arange(B) % 3 == 2, 40, G).astype(np.int32), np.full(B, c, np.int32))
    rt, oc = make(wl, dev, np.full(B, P + G // c + c + 1, np.int32))       # one capacity: uniform layout
    st, text = _bc().bc_decode_plan_describe(rt.shape, rt.cache)
    assert st == 0 and "true>" in text, text          # the straight-line kernel serves these shapes
    rollout(wl, rt, oc, G, range(1, G + 1), (8, 40, G), use_step_call=True)
    q = wl.step_q(G + 1)
    check_attention(rt.decode_attn(q).cpu().numpy(), q, oc, wl, None, "attn")
    # the same rows on the general tile loop
    rt.cache.plan = _bc().BC_PLAN_GENERAL_LOOP
    st, text = _bc().bc_decode_plan_describe(rt.shape, rt.cache)
    assert st == 0 and "true>" not in text, text
    check_attention(rt.decode_attn(q).cpu().numpy(), q, oc, wl, None, "attn, general loop")


@pytest.mark.parametrize("Hq,Hkv,dtype,d", [(1, 1, "bf16", 128), (4, 2, "bf16", 128), (3, 1, "bf16", 128),
                                             (10, 2, "bf16", 128), (7, 1, "bf16", 128), (16, 2, "bf16", 128),
                                             (8, 1, "f32", 64), (6, 2, "bf16", 64), (5, 1, "f32", 128),
                                             (1, 1, "bf16", 64), (7, 1, "bf16", 64), (16, 2, "bf16", 64)])
def test_group_sizes_one_to_eight(dev, Hq, Hkv, dtype, d):
    # every group size g = Hq / Hkv from 1 to 8, on the MFMA kernel and on the plain-ALU kernel
    wl = W.Workload("groups", 89, 5, Hq, Hkv, d, dtype, np.array([0, 3, 31, 64, 100], np.int32),
                    np.full(5, 70, np.int32), np.array([16, 4, 0, 1, 7], np.int32))
    rt, oc = make(wl, dev)
    rollout(wl, rt, oc, 70, (1, 2, 7, 8, 16, 17, 33, 70), (16, 70), use_step_call=True)


@pytest.mark.parametrize("name,dtype,d", [("bstep", "bf16", 128), ("bstep32", "f32", 64), ("bstep64", "bf16", 64)])
def test_beacon_step_rollout(dev, name, dtype, d):
    # the beacon's own step: single launch on the bf16 paths, three launches otherwise
    c = np.array([1, 2, 4, 8, 16, 32, 0, 3], np.int32)
    wl = W.Workload(name, 85, 8, 12, 2, d, dtype,
                    np.array([0, 1, 31, 32, 33, 64, 7, 100], np.int32),
                    np.array([120, 120, 120, 77, 120, 120, 120, 50], np.int32), c)
    cap = wl.capacity()
    cap[4] = 33 + 16           # sequence 4: room for one full window but not for its beacon
    rt, oc = make(wl, dev, cap)
    steps = range(1, 121)
    rollout(wl, rt, oc, 120, steps, (1, 2, 3, 16, 17, 50, 120), beacon_call=True)
    assert oc.err & ERR_CAPACITY


def test_beacon_step_leaves_other_sequences_alone(dev):
    wl = W.Workload("bstep2", 86, 4, 12, 2, 128, "bf16", np.full(4, 40, np.int32),
                    np.full(4, 64, np.int32), np.array([4, 4, 0, 8], np.int32))
    rt, oc = make(wl, dev)
    for t in range(1, 5):                       # after 4 tokens: sequences 0, 1 are due (c = 4)
        k, v = wl.step_kv(t)
        rt.decode_step(k, v, wl.step_q(t))
        oc.append(k, v)
    bk, bv = wl.beacon_kv(4)
    qb = wl.beacon_q(4)
    rt.out.fill_(-7.0)
    o = rt.beacon_step(bk, bv, qb, active=np.array([1, 0, 1, 1], np.uint8)).cpu().numpy()
    mask = np.array([1, 0, 1, 1], np.uint8)
    oc.append(bk, bv, active=mask, beacon=True)
    check_attention(o, qb, oc, wl, [0])
    oc.compress_evict(active=mask)
    assert np.all(o[1] == -7.0) and np.all(o[2] == -7.0) and np.all(o[3] == -7.0)
    nb, w = check_tables(rt, oc)
    assert list(nb) == [1, 0, 0, 0] and list(w) == [0, 4, 4, 4]
    check_slabs(rt, oc)


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 64), ("bf16", 64)])
def test_small_batch_rows_spread_over_workgroups(dev, dtype, d):
    # few (sequence, KV head) pairs and long sequences: the rows of a sequence are spread evenly
    # over several workgroups, the last of which folds their partials; a short sequence in the same
    # batch stays whole.  Fused steps (append + attention + eviction) against the oracle.
    B = 3
    Hq, Hkv = (12, 2) if d == 128 else (4, 1)
    wl = W.Workload("spread", 88, B, Hq, Hkv, d, dtype, np.array([1100, 2500, 300], np.int32),
                    np.full(B, 40, np.int32), np.array([0, 16, 4], np.int32))
    rt, oc = make(wl, dev)
    steps = range(1, 41)
    rollout(wl, rt, oc, 40, steps, (1, 16, 17, 40), use_step_call=True)
    q = wl.step_q(77)
    a = rt.decode_attn(q).cpu().numpy().copy()
    check_attention(a, q, oc, wl, None, 77)
    b = rt.decode_attn(q).cpu().numpy().copy()
    assert np.array_equal(a, b)                    # reproducible: fixed merge order, no atomics


def test_very_long_context_next_to_a_short_one(dev):
    # one sequence of 150,000 resident rows (64 chunks of 2,368 rows and their fold) beside
    # one of 40 rows that stays whole; a few fused steps, then attention, against the oracle
    wl = W.Workload("long", 89, 2, 12, 2, 128, "bf16", np.array([150000, 40], np.int32),
                    np.full(2, 6, np.int32), np.array([4, 2], np.int32))
    rt, oc = make(wl, dev)
    rollout(wl, rt, oc, 6, (1, 4, 5, 6), (6,), use_step_call=True)
    q = wl.step_q(9)
    a = rt.decode_attn(q).cpu().numpy().copy()
    check_attention(a, q, oc, wl, None, 9)


@pytest.mark.parametrize("B,Hq,Hkv,dtype,d", [(160, 12, 2, "bf16", 128), (300, 4, 1, "bf16", 128),
                                             (272, 2, 1, "f32", 64), (280, 8, 1, "bf16", 64)])
def test_longest_first_dispatch_large_ragged_batch(dev, B, Hq, Hkv, dtype, d):
    # more (sequence, KV head) pairs than compute units: bc_sort_by_length ranks the sequences by
    # resident length into the cache's dispatch order and workgroup i serves the i-th longest, in
    # bc_decode_attn and in the fused steps (B = 300: the ranking itself spans two workgroups).
    # The order is refreshed every fourth step only (a stale permutation is as good as a fresh
    # one).  Against the oracle with and without an inactive stripe, bit-equality with the plain
    # dispatch order (tuning variant 3), and a corrupt entry in the order.
    bc = _bc()
    rng = np.random.default_rng(23)
    P = rng.integers(1, 700, size=B).astype(np.int32)
    P[:4] = [1, 699, 350, 350]
    c = rng.choice([0, 2, 4, 16], size=B).astype(np.int32)
    wl = W.Workload("lpt", 87, B, Hq, Hkv, d, dtype, P, np.full(B, 40, np.int32), c)
    rt, oc = make(wl, dev)
    active = np.ones(B, np.uint8)
    active[5::7] = 0
    for t in range(1, 25):
        k, v = wl.step_kv(t)
        q = wl.step_q(t)
        bk, bv = wl.beacon_kv(t)
        act = active if t % 3 == 0 else None
        if t % 4 == 1:
            rt.sort_by_length(active=act)
        o = rt.decode_step(k, v, q, bk, bv, active=act).cpu().numpy()
        oc.append(k, v, active=act)
        seqs = [s for s in range(B) if act is None or act[s]]
        if t in (1, 2, 3, 16, 17, 24):
            check_attention(o, q, oc, wl, seqs, t)
        oc.compress_evict(bk, bv, active=act)
        check_tables(rt, oc, t)
    check_slabs(rt, oc, None, 24)
    q = wl.step_q(99)
    for act in (None, active):
        rt.out.fill_(-3.0)
        a = rt.decode_attn(q, active=act).cpu().numpy().copy()
        rt.cache.plan = bc.BC_PLAN_IGNORE_ORDER          # the same call in index order
        try:
            rt.out.fill_(-3.0)
            b = rt.decode_attn(q, active=act).cpu().numpy().copy()
        finally:
            rt.cache.plan = 0
        assert np.array_equal(a, b)
        seqs = [s for s in range(B) if act is None or act[s]]
        check_attention(a, q, oc, wl, seqs, 99)
        if act is not None:
            assert np.all(a[5::7] == -3.0)
    # the order really is the lengths sorted, longest first, inactive sequences last
    rt.sort_by_length(active=active)
    order = rt.order.cpu().numpy()
    assert sorted(order.tolist()) == list(range(B))
    L = np.array([wl.P[s] + oc.nb[s] + oc.w[s] for s in range(B)])
    key = np.where(active > 0, L + 1, 0)
    assert all(key[order[i]] >= key[order[i + 1]] for i in range(B - 1))
    # an entry that is no sequence index: state bit, its workgroups do nothing, the rest is served
    lost = int(order[3])
    rt.order[3] = B + 1000
    rt.out.fill_(-3.0)
    a = rt.decode_attn(q).cpu().numpy().copy()
    assert np.all(a[lost] == -3.0)
    check_attention(a, q, oc, wl, [s for s in range(B) if s != lost], 99)
    assert rt.tables()[2] & ERR_STATE


def test_fused_step_ragged_ratios_and_errors(dev):
    c = np.array([1, 2, 4, 8, 16, 32, 0, 3], np.int32)
    wl = W.Workload("fusedr", 80, 8, 12, 2, 128, "bf16",
                    np.array([0, 1, 31, 32, 33, 64, 7, 100], np.int32), np.full(8, 200, np.int32), c)
    cap = wl.capacity()
    cap[3] = 32 + 5            # sequence 3 runs out of slab: capacity bit, then untouched
    rt, oc = make(wl, dev, cap)
    steps = range(1, 201)
    rollout(wl, rt, oc, 200, steps, (1, 2, 3, 50, 200), use_step_call=True)
    assert oc.err == ERR_CAPACITY


@pytest.mark.parametrize("c", [16, 0])
def test_config2_batch64_full_rollout(dev, c):
    wl = W.batch64(c=c)
    rt, oc = make(wl, dev)
    rng = np.random.default_rng(5)
    sample = sorted(set([1, 2, 15, 16, 17, 31, 32, 33, 255, 256, 257, 1000, 2047, 2048, 4095, 4096])
                    | set(int(x) for x in rng.integers(1, 4097, size=48)))
    seqs = [0, 1, 31, 63] + [int(x) for x in rng.integers(0, 64, size=4)]
    worst = rollout(wl, rt, oc, 4096, sample, (16, 17, 1000, 4096), table_every=1, seq_sample=seqs,
                    use_step_call=(c > 0))
    nb, w, _ = rt.tables()
    if c > 0:
        assert int(nb[0]) == 256 and int(w[0]) == 0          # 256 + 256 + 0 = 512 rows resident
    else:
        assert int(nb[0]) == 0 and int(w[0]) == 4096
    check_slabs(rt, oc, None, 4096)
    # whole batch at the final state, fresh query
    q = wl.step_q(5000)
    o = rt.decode_attn(q).cpu().numpy()
    worst = max(worst, check_attention(o, q, oc, wl, None, 4096))
    print("batch64 c=%d worst %.3g" % (c, worst))


@pytest.mark.parametrize("mode", ["attention", "fused step in dispatch order"])
def test_config3_ragged_snapshot(dev, mode):
    wl = W.ragged256()
    T = wl.extra["T"]
    rt, oc = make(wl, dev)
    rollout(wl, rt, oc, T - 1, (), (), table_every=512)
    # snapshot at attention time of step T
    active = (wl.G >= T).astype(np.uint8)
    k, v = wl.step_kv(T)
    q = wl.step_q(T)
    if mode != "attention":
        # the way this state is timed: bc_decode_step (append + attention + eviction in one launch)
        # with the dispatch order of bc_sort_by_length attached; sequences that are over stay out
        bk, bv = wl.beacon_kv(T)
        rt.sort_by_length(active=active)
        st, text = _bc().bc_decode_plan_describe(rt.shape, rt.cache)
        assert st == 0 and "decode_lds_kernel" in text and "chunks=1" in text, text
        rt.out.fill_(-5.0)
        o = rt.decode_step(k, v, q, bk, bv, active=active).cpu().numpy()
        oc.append(k, v, active=active)
        live = [s for s in range(wl.B) if active[s]]
        worst = check_attention(o, q, oc, wl, live, T)
        assert all(np.all(o[s] == -5.0) for s in range(wl.B) if not active[s])
        oc.compress_evict(bk, bv, active=active)
        nb, w = check_tables(rt, oc, T)
        for s in live:
            assert (int(nb[s]), int(w[s])) == OR.tables_after_step(int(wl.c[s]), T)
        check_slabs(rt, oc, None, T)
        order = rt.order.cpu().numpy()
        assert sorted(order.tolist()) == list(range(wl.B))
        print("ragged fused T=%d worst %.3g" % (T, worst))
        return
    rt.append_kv(k, v, active=active)
    oc.append(k, v, active=active)
    nb, w = check_tables(rt, oc, T)
    for s in range(wl.B):       # closed form of the residency process
        t_s = min(T, int(wl.G[s]))
        if wl.G[s] >= T:
            assert (int(nb[s]), int(w[s])) == OR.tables_at_attention(int(wl.c[s]), t_s)
        else:
            assert (int(nb[s]), int(w[s])) == OR.tables_after_step(int(wl.c[s]), t_s)
    check_slabs(rt, oc, None, T)
    o = rt.decode_attn(q).cpu().numpy()          # all sequences, finished ones included
    worst = check_attention(o, q, oc, wl, None, T)
    print("ragged T=%d sumL=%d worst %.3g" % (T, sum(oc.L(s) for s in range(wl.B)), worst))


@pytest.mark.parametrize("mode", ["separate calls", "step with supplied beacon", "step and beacon step"])
def test_config4_long_peaked(dev, mode):
    # the whole 32768-token rollout, by the three separate calls, by the fused step that is handed
    # the beacon (the form the benchmark times) and by the fused step followed by the beacon
    # token's own step (bc_beacon_step)
    wl = W.long_reasoning()
    rt, oc = make(wl, dev)
    rng = np.random.default_rng(9)
    # steps whose window holds a x4 key: the 64th written row falls on a token (rows are counted
    # in write order: 512 prompt rows, then 32 tokens and one beacon per window)
    peaked = [t for t in range(1, 32769) if (512 + (t - 1) + (t - 1) // 32) % 64 == 63]
    assert len(peaked) > 400
    sample = sorted(set([1, 31, 32, 33, 63, 64, 65, 4096, 32767, 32768])
                    | set(int(x) for x in rng.integers(1, 32769, size=20))
                    | set(peaked[:2] + [peaked[len(peaked) // 2], peaked[-1], peaked[-1] + 1, peaked[-1] + 5]))
    sample = [t for t in sample if t <= 32768]
    seqs = [0, 7, 31]
    worst = rollout(wl, rt, oc, 32768, sample, (32, 33, 32768), table_every=1024, seq_sample=seqs,
                    use_step_call=(mode == "step with supplied beacon"),
                    beacon_call=(mode == "step and beacon step"))
    nb, w, _ = rt.tables()
    assert int(nb[0]) == 1024 and int(w[0]) == 0
    q = wl.step_q(40000)
    o = rt.decode_attn(q).cpu().numpy()
    worst = max(worst, check_attention(o, q, oc, wl, None, 32768))
    print("long worst %.3g" % worst)


# ---------------------------------------------------------------------------
def test_error_bits_and_inactive_rows_untouched(dev):
    import torch
    wl = W.Workload("edge", 90, 3, 4, 2, 64, "bf16", np.array([2, 0, 3], np.int32),
                    np.array([8, 8, 8], np.int32), np.array([2, 2, 0], np.int32))
    cap = np.array([2 + 1 + 2, 3, 5], np.int32)
    rt, oc = make(wl, dev, cap)
    # sequence 1 is empty: attention over it is a state error and leaves the output alone
    rt.out.fill_(123.0)
    q = wl.step_q(1)
    o = rt.decode_attn(q)
    nb, w, err = rt.tables()
    assert err == ERR_STATE
    assert torch.all(o[1] == 123.0)
    K, V = oc.resident(0)
    assert np.abs(o[0].cpu().numpy() - OA.decode_attention(q[0], K, V, wl.scale)).max() <= 2e-3
    rt.err.zero_()
    # inactive sequences: tables, slabs and outputs untouched
    k, v = wl.step_kv(1)
    rt.append_kv(k, v, active=[1, 0, 1]); oc.append(k, v, active=[1, 0, 1])
    rt.out.fill_(-7.0)
    o = rt.decode_attn(wl.step_q(2), active=[0, 0, 1])
    assert torch.all(o[0] == -7.0) and torch.all(o[1] == -7.0) and not torch.any(o[2] == -7.0)
    check_tables(rt, oc)
    # window full -> state bit; slab full -> capacity bit; sequence untouched both times
    k, v = wl.step_kv(2)
    rt.append_kv(k, v); oc.append(k, v)                 # seq0 w=2, seq1 w=1, seq2 w=2 (cap 5 reached)
    rt.append_kv(k, v, active=[1, 0, 0]); oc.append(k, v, active=[1, 0, 0])
    assert oc.err == ERR_STATE
    rt.append_kv(k, v, active=[0, 0, 1]); oc.append(k, v, active=[0, 0, 1])
    assert oc.err == ERR_STATE | ERR_CAPACITY
    check_tables(rt, oc)
    check_slabs(rt, oc)
    # partial-window compression is an opt-in extension
    bk, bv = wl.beacon_kv(2)
    rt.compress_evict(bk, bv); oc.compress_evict(bk, bv)             # seq0 only
    rt.compress_evict(bk, bv, require_full_window=False)
    oc.compress_evict(bk, bv, require_full=False)                    # seq1 (w=1)
    check_tables(rt, oc)
    check_slabs(rt, oc, [0, 2])


def test_host_side_argument_errors(dev):
    bc = _bc()
    wl = W.tiny()
    rt, _ = make(wl, dev)
    import ctypes as C
    sh = bc.bc_shape(2, 4, 3, 64, 0, 0.125)            # Hq % Hkv != 0
    assert bc.bc_decode_attn(sh, rt.cache, C.c_void_p(rt.out.data_ptr()), C.c_void_p(rt.out.data_ptr()),
                             None, C.c_void_p(rt.ws.data_ptr()), rt.ws_bytes, None) == -2
    assert bc.bc_decode_attn(rt.shape, rt.cache, None, C.c_void_p(rt.out.data_ptr()), None,
                             C.c_void_p(rt.ws.data_ptr()), rt.ws_bytes, None) == -1
    assert bc.bc_decode_attn(rt.shape, rt.cache, C.c_void_p(rt.out.data_ptr()),
                             C.c_void_p(rt.out.data_ptr()), None, C.c_void_p(rt.ws.data_ptr()), 8,
                             None) == -5
    assert bc.bc_compress_evict(rt.shape, rt.cache, None, None, None, 0, None) == -1
    assert "workspace" in bc.bc_status_str(-5)


def test_deterministic_and_split_invariant(dev):
    import torch
    bc = _bc()
    wl = W.batch64(c=0, G=1500, B=8)
    rt, oc = make(wl, dev)
    for t in range(1, 1201):
        k, v = wl.step_kv(t)
        rt.append_kv(k, v)
    q = wl.step_q(7)
    a = rt.decode_attn(q).clone()
    b = rt.decode_attn(q).clone()
    assert torch.equal(a, b)                               # fixed merge order
    rt.cache.rows_per_workgroup = 512                   # a forced chunk size, for this call only
    try:
        c = rt.decode_attn(q).clone()
    finally:
        rt.cache.rows_per_workgroup = 0
    assert float((a - c).abs().max()) < 1e-5               # independent of the split factor
    assert not torch.equal(a, torch.zeros_like(a))


# ---------------------------------------------------------------------------
# next rows: evaluation budget rule and mid-generation ratio change
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 64), ("bf16", 64)])
def test_budget_rule_interrupts_generation_on_device(dev, dtype, d):
    import torch
    B = 6
    c = np.array([1, 2, 4, 16, 0, 3], np.int32)
    wl = W.Workload("budget", 91, B, 12 if d == 128 else 4, 2 if d == 128 else 1, d, dtype,
                    np.array([3, 0, 17, 32, 5, 64], np.int32), np.full(B, 200, np.int32), c)
    rt, oc = make(wl, dev)
    budget = np.array([10, 12, 7, 20, 9, 15], np.int32)
    budget_rollout(wl, rt, oc, budget, 120, None, dev)


def budget_rollout(wl, rt, oc, budget, steps, attention_steps, dev, sort_every=0):
    """Steps under the evaluation cap: outputs, live flags, tables and the step at which every
    sequence ends against the oracle; attention_steps = None checks every step."""
    import torch
    B, c = wl.B, wl.c
    bud_d = torch.from_numpy(budget).to(dev)
    live_d = torch.ones(B, dtype=torch.uint8, device=dev)
    live = [1] * B
    last = [None] * B
    for t in range(1, steps + 1):
        k, v = wl.step_kv(t)
        q = wl.step_q(t)
        bk, bv = wl.beacon_kv(t)
        rt.out.fill_(77.0)
        if sort_every and t % sort_every == 1:
            rt.sort_by_length(active=live_d)
        o = rt.decode_step_budget(k, v, q, bk, bv, bud_d, live_d).cpu().numpy()
        was = list(live)
        oc.append(k, v, active=was)
        act = [s for s in range(B) if was[s]]
        if act and (attention_steps is None or t in attention_steps):
            check_attention(o, q, oc, wl, act, t)
        for s in range(B):
            if not was[s]:
                assert np.all(o[s] == 77.0), (s, t)          # finished sequences are skipped
        oc.apply_budget(budget, live)
        oc.compress_evict(bk, bv, active=was)
        assert live_d.cpu().tolist() == live, t
        check_tables(rt, oc, t)
        for s in range(B):
            if was[s] and not live[s]:
                last[s] = t
    check_slabs(rt, oc)
    for s in range(B):
        if last[s] is not None or OR.first_step_reaching(int(budget[s]), int(c[s])) <= steps:
            assert last[s] == OR.first_step_reaching(int(budget[s]), int(c[s])), (s, last[s])


def test_budget_rule_large_batch_longest_first(dev):
    # more pairs than compute units: the budget step follows a dispatch order that is refreshed
    # every fifth step from the live flags and lengths of that moment
    B = 300
    rng = np.random.default_rng(31)
    P = rng.integers(1, 400, size=B).astype(np.int32)
    c = rng.choice([0, 1, 3, 16], size=B).astype(np.int32)
    wl = W.Workload("budget_lpt", 93, B, 4, 1, 128, "bf16", P, np.full(B, 60, np.int32), c)
    rt, oc = make(wl, dev)
    budget = rng.integers(4, 30, size=B).astype(np.int32)
    budget_rollout(wl, rt, oc, budget, 36, (1, 2, 5, 17, 36), dev, sort_every=5)


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 64), ("bf16", 64)])
def test_admission_into_finished_slots(dev, dtype, d):
    # continuous batching: the budget rule ends generations at different steps; every 10 steps
    # the finished slots take new sequences (new prompt length and ratio) and carry on
    import torch
    B = 6
    c = np.array([1, 2, 4, 16, 0, 3], np.int32)
    Hq, Hkv = (12, 2) if d == 128 else (4, 1)
    wl = W.Workload("admit", 93, B, Hq, Hkv, d, dtype, np.array([3, 0, 17, 32, 5, 64], np.int32),
                    np.full(B, 400, np.int32), c)
    cap = np.full(B, 120, np.int32)
    rt, oc = make(wl, dev, cap)
    budget = np.array([10, 12, 7, 20, 9, 15], np.int32)
    bud_d = torch.from_numpy(budget).to(dev)
    live_d = torch.ones(B, dtype=torch.uint8, device=dev)
    live = [1] * B
    rng = np.random.default_rng(17)
    admitted = 0
    for t in range(1, 161):
        k, v = wl.step_kv(t)
        q = wl.step_q(t)
        bk, bv = wl.beacon_kv(t)
        o = rt.decode_step_budget(k, v, q, bk, bv, bud_d, live_d).cpu().numpy()
        was = list(live)
        oc.append(k, v, active=was)
        act = [s for s in range(B) if was[s]]
        if act:
            check_attention(o, q, oc, wl, act, t)
        oc.apply_budget(budget, live)
        oc.compress_evict(bk, bv, active=was)
        if t % 10 == 0:
            adm = np.array([0 if x else 1 for x in live], np.uint8)
            if t == 40:
                adm[:] = 0
                adm[[s for s in range(B) if not live[s]][:1]] = 1     # one slot with too long a prompt
            newP = [int(rng.integers(1, 90)) for _ in range(B)]
            if t == 40:
                newP = [121] * B
            pk = [W.round_to_dtype(rng.standard_normal((newP[s], Hkv, d)), dtype) for s in range(B)]
            pv = [W.round_to_dtype(rng.standard_normal((newP[s], Hkv, d)), dtype) for s in range(B)]
            new_c = rng.choice([0, 1, 2, 3, 5, 8], size=B).astype(np.int32)
            rt.cache_admit(adm, pk, pv, new_c, live_d)
            oc.admit(adm, pk, pv, new_c, live)
            admitted += int(adm.sum())
        assert live_d.cpu().tolist() == live, t
        check_tables(rt, oc, t)
        assert rt.c.cpu().tolist() == oc.c and rt.P.cpu().tolist() == oc.P, t
        if t % 10 == 0 or t == 160:
            check_slabs(rt, oc, None, t)
    assert admitted >= 12 and oc.err == ERR_CAPACITY


def test_ratio_change_mid_generation(dev):
    B = 4
    wl = W.Workload("ratio", 92, B, 12, 2, 128, "bf16", np.array([8, 0, 40, 3], np.int32),
                    np.full(B, 120, np.int32), np.array([4, 16, 0, 2], np.int32))
    cap = np.full(B, 40 + 120 + 40, np.int32)
    rt, oc = make(wl, dev, cap)
    changes = {9: [2, 16, 0, 2], 17: [2, 4, 0, 2], 30: [8, 4, 0, 0], 31: [1, 1, 1, 1], 70: [0, 5, 0, 16],
               90: [3, 5, 200, 200]}
    for t in range(1, 121):
        if t in changes:
            rt.set_ratio(changes[t])
            oc.set_ratio(changes[t])
            assert rt.c.cpu().tolist() == oc.c, t
        k, v = wl.step_kv(t)
        q = wl.step_q(t)
        bk, bv = wl.beacon_kv(t)
        o = rt.decode_step(k, v, q, bk, bv).cpu().numpy()
        oc.append(k, v)
        check_attention(o, q, oc, wl, None, t)
        oc.compress_evict(bk, bv)
        check_tables(rt, oc, t)
        if t in (9, 17, 30, 31, 32, 70, 90, 120):
            check_slabs(rt, oc)
    assert oc.err == ERR_STATE          # the change at step 31 did not fit some windows


@pytest.mark.parametrize("case", range(12))
def test_randomised_small_rollouts(dev, case):
    # seeded random shapes, prompt lengths, ratios and generation lengths; the call form (separate
    # calls, tail form, fused step, fused step + beacon step) rotates with the case number
    rng = np.random.default_rng([20251013, 77, case])
    dtype, d = [("bf16", 128), ("f32", 64), ("bf16", 64), ("f32", 128)][case % 4]
    Hq, Hkv = [(12, 2), (4, 4), (8, 1), (6, 2), (7, 1), (5, 5), (16, 2), (3, 1)][int(rng.integers(0, 8))]
    B = int(rng.integers(1, 10))
    P = rng.integers(0, 300, size=B).astype(np.int32)
    c = rng.choice([0, 1, 2, 3, 5, 8, 16], size=B).astype(np.int32)
    steps = 45
    G = rng.integers(1, steps + 1, size=B).astype(np.int32)
    G[int(rng.integers(0, B))] = steps
    for s in range(B):
        if P[s] == 0 and G[s] < 1:
            G[s] = 1
    wl = W.Workload("rand%d" % case, 200 + case, B, Hq, Hkv, d, dtype, P, G, c)
    rt, oc = make(wl, dev)
    form = case % 4
    attn = sorted(set(int(x) for x in rng.integers(1, steps + 1, size=8)) | {1, steps})
    rollout(wl, rt, oc, steps, attn, (steps // 2, steps), tail_form=(form == 1),
            use_step_call=(form == 2), beacon_call=(form == 3))


@pytest.mark.parametrize("case", range(24))
def test_randomised_rollouts_near_the_plan_boundaries(dev, case):
    # seeded random batches whose pair counts straddle the kernel choices (128 and 256 pairs) and
    # whose prompt lengths straddle the tile and capacity limits of the straight-line form (384 /
    # 768 rows) and of the twelve-wave and small-workgroup forms (1100 rows); call form, dispatch
    # order and uniform / ragged layout rotate with the seed
    rng = np.random.default_rng([424242, case])
    dtype, d = [("bf16", 128), ("bf16", 128), ("bf16", 64), ("f32", 64), ("f32", 128), ("bf16", 128)][case % 6]
    Hq, Hkv = [(12, 2), (4, 4), (8, 1), (6, 2), (7, 1), (16, 2), (3, 1), (32, 8), (24, 8), (2, 2)][int(rng.integers(0, 10))]
    kind = case % 4
    if kind == 0:
        B = max(1, int(rng.integers(120, 136)) // Hkv)
    elif kind == 1:
        B = max(1, int(rng.integers(250, 264)) // Hkv)
    elif kind == 2:
        B = int(rng.integers(1, 40))
    else:
        B = max(1, int(rng.integers(300, 400)) // Hkv)
    B = min(B, 200)
    uniform = bool(rng.integers(0, 2))
    pbase = int(rng.choice([0, 31, 33, 256, 352, 383, 384, 500, 700, 760, 1060, 1090, 1500]))
    if dtype == "f32":
        pbase = min(pbase, 400)
    P = np.full(B, pbase, np.int32) if uniform else np.maximum(0, pbase + rng.integers(-40, 40, size=B)).astype(np.int32)
    c = (np.full(B, int(rng.choice([0, 1, 2, 3, 7, 16, 32])), np.int32) if uniform
         else rng.choice([0, 1, 2, 5, 16, 32], size=B).astype(np.int32))
    steps = int(rng.integers(20, 50))
    G = np.full(B, steps, np.int32) if uniform else rng.integers(1, steps + 1, size=B).astype(np.int32)
    G[int(rng.integers(0, B))] = steps
    form = int(rng.integers(0, 4))
    wl = W.Workload("bound%d" % case, 5000 + case, B, Hq, Hkv, d, dtype, P, G, c)
    rt, oc = make(wl, dev)
    sort = B * Hkv > 256 and bool(rng.integers(0, 2))
    attn = sorted(set(int(x) for x in rng.integers(1, steps + 1, size=5)) | {1, steps})
    sample = None if B <= 24 else sorted(set(int(x) for x in rng.integers(0, B, size=16)))
    rollout(wl, rt, oc, steps, attn, (steps // 2, steps), table_every=7, tail_form=(form == 1),
            use_step_call=(form == 2), beacon_call=(form == 3), seq_sample=sample,
            before_step=(lambda t: rt.sort_by_length()) if sort else None)


def test_fused_steps_under_graph_replay(dev):
    # The benchmark replays a captured cycle of fused steps.  One runtime runs five 4-step cycles
    # eagerly, a twin runs the first cycle eagerly, captures the cycle as a HIP graph and replays
    # it four times with eager calls and synchronisations in between; every step's output, the
    # tables and the slabs must be bit-equal, and the last outputs match the oracle.
    import torch
    bc = _bc()
    B, cyc, ncyc = 8, 4, 5
    wl = W.Workload("graph", 95, B, 12, 2, 128, "bf16", np.array([3, 40, 0, 17, 64, 5, 33, 1], np.int32),
                    np.full(B, cyc * ncyc, np.int32), np.array([4, 2, 0, 1, 3, 4, 2, 4], np.int32))
    rtE, oc = make(wl, dev)
    rtG, _ = make(wl, dev)
    pool = []
    for j in range(1, cyc + 1):
        k, v = wl.step_kv(j)
        bk, bv = wl.beacon_kv(j)
        host = dict(k=k, v=v, q=wl.step_q(j), bk=bk, bv=bv)
        pool.append((host, {n: bc.to_device(a, "bf16", dev) for n, a in host.items()}))
    outsE = [torch.empty_like(rtE.out) for _ in range(cyc)]
    outsG = [torch.empty_like(rtG.out) for _ in range(cyc)]

    def cycle(rt, outs):
        for j in range(cyc):
            x = pool[j][1]
            rt.decode_step(x["k"], x["v"], x["q"], x["bk"], x["bv"], out=outs[j])

    st = torch.cuda.Stream()
    ref_out = []
    for _ in range(ncyc):                                   # eager twin + oracle
        cycle(rtE, outsE)
        torch.cuda.synchronize()
        ref_out.append([o.cpu().numpy().copy() for o in outsE])
        for j in range(cyc):
            h = pool[j][0]
            oc.append(h["k"], h["v"])
            last_ref = (h["q"], [OA.decode_attention(h["q"][s], *oc.resident(s), wl.scale) for s in range(B)])
            oc.compress_evict(h["bk"], h["bv"])
    with torch.cuda.stream(st):
        cycle(rtG, outsG)                                   # first cycle eagerly
        st.synchronize()
        assert all(np.array_equal(a.cpu().numpy(), b) for a, b in zip(outsG, ref_out[0]))
        saved = (rtG.nb.clone(), rtG.w.clone())
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st):
            cycle(rtG, outsG)
        rtG.nb.copy_(saved[0]); rtG.w.copy_(saved[1])       # capture does not run; restore anyway
        for r in range(1, ncyc):
            g.replay()
            st.synchronize()
            got = [o.cpu().numpy().copy() for o in outsG]
            for j in range(cyc):
                assert np.array_equal(got[j], ref_out[r][j]), (r, j)
            # the program's own eager work between replays: an attention call and a table read
            rtG.decode_attn(pool[0][1]["q"], out=torch.empty_like(rtG.out))
            nb, w, err = rtG.tables()
            assert err == 0
    nbE, wE, _ = rtE.tables()
    nbG, wG, _ = rtG.tables()
    assert list(nbE) == list(nbG) == oc.nb and list(wE) == list(wG) == oc.w
    check_slabs(rtG, oc)
    q, ref = last_ref
    worst = max(float(np.abs(ref_out[-1][-1][s] - ref[s]).max()) for s in range(B))
    assert worst <= TOL[wl.dtype], worst


@pytest.mark.parametrize("B,Hq,Hkv,d,dtype,P,chunks", [
    (2, 4, 2, 128, "bf16", (953, 940), 1),                  # one row of capacity short of being cut
    (2, 4, 2, 128, "bf16", (954, 940), 15),                 # chunks of two tiles
    (3, 6, 2, 128, "bf16", (507, 509, 1100), 16),           # sequences that come to be cut in the rollout
    (1, 33, 33, 64, "bf16", (1000,), 15),                   # more KV heads than counters beside the ticket
    (34, 2, 1, 128, "bf16", (1000, 30), 15),                # workgroups of four waves
    (33, 3, 1, 64, "bf16", (1030, 500), 15),
    (2, 8, 1, 128, "f32", (58, 59), 1),                     # capacities that never let a sequence be cut have no chunks
    (65, 2, 2, 64, "f32", (130, 90), 1),
    (2, 8, 1, 128, "f32", (126, 400), 7),
])
def test_sequences_cut_into_chunks(dev, B, Hq, Hkv, d, dtype, P, chunks):
    # partials folded by a pair's last workgroup, one ticket per pair, evictions among the steps (c = 3)
    G = 7
    P = np.resize(np.array(P, np.int32), B)
    wl = W.Workload("cut", 113, B, Hq, Hkv, d, dtype, P, np.full(B, G, np.int32), np.full(B, 3, np.int32))
    rt, oc = make(wl, dev)
    st, text = _bc().bc_decode_plan_describe(rt.shape, rt.cache)
    assert st == 0 and int(text.split("chunks=")[1].split()[0]) == chunks, text
    rollout(wl, rt, oc, G, range(1, G + 1), (3, G), use_step_call=True)


@pytest.mark.parametrize("B,Hq,Hkv,d,dtype,P,rows", [
    (100, 16, 2, 128, "f32", (59, 60, 61, 123, 20, 187), 64),      # one workgroup per compute unit, 600 of them
    (70, 12, 2, 128, "bf16", (252, 253, 500, 509, 30, 760), 256),
])
def test_cut_plans_of_more_workgroups_than_run_at_once(dev, B, Hq, Hkv, d, dtype, P, rows):
    # the later workgroups of a launch start when earlier ones are done; many of them have no rows, and the
    # appended rows cross the lines where a sequence gets one chunk more
    G = 9
    P = np.resize(np.array(P, np.int32), B)
    wl = W.Workload("rounds", 114, B, Hq, Hkv, d, dtype, P, np.full(B, G, np.int32),
                    np.resize(np.array([4, 0, 7, 2, 0], np.int32), B))
    rt, oc = make(wl, dev)
    rt.cache.rows_per_workgroup = rows
    st, text = _bc().bc_decode_plan_describe(rt.shape, rt.cache)
    assert st == 0 and int(text.split("chunks=")[1].split()[0]) >= 3, text
    rollout(wl, rt, oc, G, range(1, G + 1), (3, G), use_step_call=True)


@pytest.mark.parametrize("B,Hq,Hkv,d,dtype,P", [(3, 6, 2, 128, "bf16", (507, 40, 1100)), (1, 33, 33, 64, "bf16", (1000,)),
                                                (50, 2, 2, 64, "f32", (1300, 90)), (3, 8, 1, 128, "f32", (500, 400, 90))])
def test_attention_does_not_depend_on_what_the_workspace_holds(dev, B, Hq, Hkv, d, dtype, P):
    # a caller who only attends never has to clear the workspace, whatever other calls left in it
    P = np.resize(np.array(P, np.int32), B)
    wl = W.Workload("dirty", 115, B, Hq, Hkv, d, dtype, P, np.full(B, 8, np.int32), np.full(B, 3, np.int32))
    rt, oc = make(wl, dev)
    st, text = _bc().bc_decode_plan_describe(rt.shape, rt.cache)
    assert st == 0 and int(text.split("chunks=")[1].split()[0]) > 1, text
    for t, filler in enumerate((0xA5, 0x00, 0x01, 0xFF)):
        rt.ws.fill_(filler)
        rt.out.fill_(-3.0)
        q = wl.step_q(t)
        check_attention(rt.decode_attn(q).cpu().numpy(), q, oc, wl, None, t)
        assert partials_written(rt, filler)


@pytest.mark.parametrize("Hq,Hkv,d,dtype,batches", [
    (2, 1, 64, "f32", ((100, 930), (150, 1410), (300, 40))),       # cut, cut, whole
    (4, 2, 128, "bf16", ((3, 1100), (64, 200), (20, 1000))),       # cut, whole, cut
])
def test_steps_of_different_batches_share_a_workspace(dev, Hq, Hkv, d, dtype, batches):
    # one workspace, sized for the largest batch, serves caches of several sizes in turn: the partial
    # results of one do not lie over the counters of another.  Bit-equal to workspaces of their own.
    import torch
    runs = []
    for i, (B, P) in enumerate(batches):
        wl = W.Workload("share%d" % i, 116 + i, B, Hq, Hkv, d, dtype, np.full(B, P, np.int32), np.full(B, 8, np.int32),
                        np.full(B, 3, np.int32))
        runs.append((wl, make(wl, dev)[0], make(wl, dev)[0]))
    nbytes = max(_bc().bc_decode_workspace_bytes(rt.shape, rt.max_cap) for _, rt, _ in runs)
    ws = torch.zeros(nbytes, dtype=torch.uint8, device=dev)
    for _, _, shared in runs:
        shared.ws, shared.ws_bytes = ws, nbytes
    for t in range(1, 8):
        for wl, own, shared in runs:
            (k, v), q, (bk, bv) = wl.step_kv(t), wl.step_q(t), wl.beacon_kv(t)
            assert torch.equal(own.decode_step(k, v, q, bk, bv), shared.decode_step(k, v, q, bk, bv)), (t, wl.B)
            assert partials_written(own) == (wl.P[0] > 900), (t, wl.B)
    for _, own, shared in runs:
        (na, wa, ea), (nb, wb, eb) = own.tables(), shared.tables()
        assert list(na) == list(nb) and list(wa) == list(wb) and ea == eb == 0


@pytest.mark.parametrize("B,Hq,Hkv,d,P,chunks", [
    (2, 8, 1, 128, (62, 66), 1),
    (2, 2, 1, 64, (126, 250), 1),
    (2, 2, 1, 64, (126, 255), 3),
    (64, 16, 2, 128, (62, 260, 125), 2),             # groups of eight
    (65, 16, 2, 128, (62, 260, 125), 1),
    (128, 3, 1, 64, (126, 400, 255), 4),
])
def test_fp32_sequences_cut_at_their_passes(dev, B, Hq, Hkv, d, P, chunks):
    G = 7
    P = np.resize(np.array(P, np.int32), B)
    wl = W.Workload("passes", 119, B, Hq, Hkv, d, "f32", P, np.full(B, G, np.int32), np.full(B, 3, np.int32))
    rt, oc = make(wl, dev)
    st, text = _bc().bc_decode_plan_describe(rt.shape, rt.cache)
    assert st == 0 and int(text.split("chunks=")[1].split()[0]) == chunks, text
    rollout(wl, rt, oc, G, range(1, G + 1), (3, G), use_step_call=True)
    assert partials_written(rt) == (chunks > 1)
    q = wl.step_q(77)
    check_attention(rt.decode_attn(q).cpu().numpy(), q, oc, wl, None, 77)


@pytest.mark.parametrize("B,Hq,Hkv,d,line,alone", [
    (2, 8, 1, 128, 130, 194), (32, 1, 1, 64, 258, 386), (33, 6, 1, 128, 130, 258), (32, 4, 2, 64, 258, 386), (65, 2, 1, 128, 194, 258),
    (96, 1, 1, 64, 258, 514), (97, 7, 1, 128, 258, 514), (64, 4, 2, 64, 258, 1026), (129, 1, 1, 64, 1408, 1536), (170, 2, 1, 64, 1408, 1536)])
def test_fp32_sequences_come_to_their_cut_line(dev, B, Hq, Hkv, d, line, alone):
    # every seventh sequence reaches the line in the sixth of seven steps (c = 3), the others stay below it; attention alone has a
    # line of its own.  Partial results show whether a sequence was cut
    G = 7
    P = np.full(B, 9, np.int32)
    P[1:line // 7:3] = np.arange(len(P[1:line // 7:3])) * 5 + 1
    P[::7] = line - 4
    wl = W.Workload("line32", 126, B, Hq, Hkv, d, "f32", P, np.full(B, G, np.int32), np.full(B, 3, np.int32))
    rt, oc = make(wl, dev)
    sample = sorted({0, 1, B // 2, B - 1} | set(range(0, B, 7)[:4]) | set(range(0, B, 7)[-2:]))
    written = {}
    rollout(wl, rt, oc, G, range(1, G + 1), (), use_step_call=True, seq_sample=sample,
            before_step=lambda t: written.update({t: partials_written(rt)}))
    assert [written[t] for t in range(1, G + 1)] == [False] * 6 + [True]
    check_slabs(rt, oc, sample)
    for rows in (alone - 1, alone, alone + 70):
        wa = W.Workload("alone32", 127, B, Hq, Hkv, d, "f32", np.where(P == line - 4, rows, P).astype(np.int32), np.full(B, 0, np.int32),
                        np.full(B, 3, np.int32))
        ra, oa = make(wa, dev)
        q = wa.step_q(5)
        check_attention(ra.decode_attn(q).cpu().numpy(), q, oa, wa, sample, rows)
        assert partials_written(ra) == (rows >= alone), rows


@pytest.mark.parametrize("B,Hq,Hkv,d,P", [(5, 6, 2, 128, (126, 300, 40)), (40, 6, 2, 64, (254, 20, 700))])
def test_fp32_cut_sequences_and_the_beacons_own_step(dev, B, Hq, Hkv, d, P):
    G = 8
    wl = W.Workload("beacon32", 128, B, Hq, Hkv, d, "f32", np.resize(np.array(P, np.int32), B), np.full(B, G, np.int32), np.full(B, 3, np.int32))
    rt, oc = make(wl, dev)
    rollout(wl, rt, oc, G, range(1, G + 1), (3, G), beacon_call=True, seq_sample=range(min(B, 9)))
    assert partials_written(rt)


@pytest.mark.parametrize("B,Hq,Hkv,d,P,chunks", [
    (1, 4, 1, 64, (16900,), 34),                      # a chunk for every 512 rows: the fold takes three batches
    (2, 6, 2, 128, (9000, 8300), 18),
    (1, 3, 1, 128, (40000,), 64),                     # the most chunks there are
])
def test_long_sequences_get_a_chunk_for_every_512_rows(dev, B, Hq, Hkv, d, P, chunks):
    G = 5
    wl = W.Workload("chunks512", 120, B, Hq, Hkv, d, "bf16", np.array(P, np.int32), np.full(B, G, np.int32),
                    np.full(B, 2, np.int32))
    rt, oc = make(wl, dev)
    st, text = _bc().bc_decode_plan_describe(rt.shape, rt.cache)
    assert st == 0 and int(text.split("chunks=")[1].split()[0]) == chunks, text
    rollout(wl, rt, oc, G, range(1, G + 1), (G,), use_step_call=True)


@pytest.mark.parametrize("B,Hq,Hkv,d,P,chunks", [
    (8, 4, 2, 128, (762, 30), 1), (8, 4, 2, 128, (763, 318), 13), (24, 4, 2, 64, (763, 381), 10), (49, 2, 1, 128, (763, 30), 1),      # 16 to 48 pairs: from 769 rows on
    (32, 4, 2, 128, (1017, 318), 8), (32, 4, 2, 128, (1018, 318), 4), (65, 2, 1, 128, (1018, 510), 7)])      # eight waves from 1024 on, up to 64 pairs
def test_plans_of_steps_at_their_lines(dev, B, Hq, Hkv, d, P, chunks):
    # capacities and numbers of pairs on both sides of the plan's lines, short sequences that come to be cut in the rollout (320, 384 and 512 rows)
    G = 7
    P = np.resize(np.array(P, np.int32), B)
    wl = W.Workload("lines", 126, B, Hq, Hkv, d, "bf16", P, np.full(B, G, np.int32), np.full(B, 3, np.int32))
    rt, oc = make(wl, dev)
    st, text = _bc().bc_decode_plan_describe(rt.shape, rt.cache)
    assert st == 0 and int(text.split("chunks=")[1].split()[0]) == chunks, text
    rollout(wl, rt, oc, G, range(1, G + 1), (3, G), use_step_call=True)


@pytest.mark.parametrize("Hq,Hkv,d,dtype,chunk", [(8, 1, 128, "bf16", 512), (7, 1, 64, "bf16", 512), (10, 5, 128, "bf16", 128),
                                                  (9, 9, 64, "bf16", 192), (8, 1, 128, "f32", 64), (3, 1, 64, "f32", 128)])
def test_fold_of_every_number_of_chunks(dev, Hq, Hkv, d, dtype, chunk):
    # the fold takes chunks by fours and by eights or sixteens; beacon rows from LDS (up to eight KV heads of d = 128) and from the caller's tensors
    numbers = {1: (2, 3, 4, 5, 7, 8, 9, 12, 13, 16, 17, 18), 5: range(8, 15), 9: (5,)}[Hkv]
    P = np.array([n * chunk - 5 for n in numbers], np.int32)
    G = 6
    wl = W.Workload("fold", 122, len(P), Hq, Hkv, d, dtype, P, np.full(len(P), G, np.int32), np.full(len(P), 2, np.int32))
    rt, oc = make(wl, dev)
    st, text = _bc().bc_decode_plan_describe(rt.shape, rt.cache)
    assert st == 0 and int(text.split("chunks=")[1].split()[0]) > 4, text
    rollout(wl, rt, oc, G, range(1, G + 1), (G,), use_step_call=True)
    assert partials_written(rt)


@pytest.mark.parametrize("B,Hkv,d,line", [(1, 1, 64, 512), (1, 2, 64, 512), (2, 1, 64, 512), (1, 3, 64, 384), (2, 2, 64, 384), (1, 1, 128, 320), (1, 2, 128, 320)])
def test_rows_from_which_on_a_step_cuts_a_sequence(dev, B, Hkv, d, line):
    for rows, cut in ((line - 1, False), (line, True)):
        wl = W.Workload("line", 127, B, 2 * Hkv, Hkv, d, "bf16", np.full(B, rows - 1, np.int32), np.full(B, 1100 - rows, np.int32), np.full(B, 0, np.int32))
        rt, oc = make(wl, dev)
        rollout(wl, rt, oc, 1, (1,), (1,), use_step_call=True)
        assert partials_written(rt) == cut, rows


@pytest.mark.parametrize("B,Hq,Hkv,d,P", [(3, 6, 2, 128, (507, 509, 1100)), (3, 6, 2, 64, (827, 829, 1100)),
                                          (62, 4, 2, 128, (1019, 1021, 1100, 60))])
def test_sequences_come_to_their_cut_line(dev, B, Hq, Hkv, d, P):
    # cut from 512 rows on; by attention alone from 832 at d = 64, from 1024 where a sequence has at most four chunks
    G = 8
    P = np.resize(np.array(P, np.int32), B)
    wl = W.Workload("cutline", 121, B, Hq, Hkv, d, "bf16", P, np.full(B, G, np.int32), np.full(B, 5, np.int32))
    rt, oc = make(wl, dev)
    st, text = _bc().bc_decode_plan_describe(rt.shape, rt.cache)
    assert st == 0 and int(text.split("chunks=")[1].split()[0]) > 1, text
    sample = None if B <= 24 else range(0, B, 5)
    for t in range(1, G + 1):
        (k, v), q, (bk, bv) = wl.step_kv(t), wl.step_q(t), wl.beacon_kv(t)
        o = rt.decode_step(k, v, q, bk, bv).cpu().numpy()
        oc.append(k, v)
        check_attention(o, q, oc, wl, sample, t)
        oc.compress_evict(bk, bv)
        check_tables(rt, oc, t)
        check_attention(rt.decode_attn(q).cpu().numpy(), q, oc, wl, sample, t)
    check_slabs(rt, oc, sample)


@pytest.mark.parametrize("B,Hq,Hkv,d,P,width,bound", [
    (64, 4, 1, 64, 40, 4.0, 2.45e-7), (64, 4, 1, 64, 600, 2.0, 3.4e-7), (64, 6, 1, 128, 120, 1.0, 1.85e-7), (64, 6, 1, 128, 600, 2.0, 3.3e-7),
    (200, 6, 1, 128, 1500, 0.02, 2.5e-7)])
def test_fp32_sums_are_as_close_to_64_bits_as_short_ones(dev, B, Hq, Hkv, d, P, width, bound):
    # 2-norm of the difference over that of the result.  bound: 1.25 times what sums of four products, of eight rows, and over lanes
    # give for these inputs (1.96, 2.71, 1.49, 2.61, 2.00e-7); one running sum of a row's products and of a wave's rows gives 3.15, 4.40,
    # 2.55, 4.88, 3.57e-7
    import torch
    rt = _bc().Runtime(B, Hq, Hkv, d, "f32", d ** -0.5, np.full(B, P), np.zeros(B, np.int32), np.full(B, P + 2), dev)
    g = torch.Generator(device=dev).manual_seed(3)
    n = B * (P + 2) * Hkv * d
    rt.k_slab.copy_(torch.randn(n, generator=g, device=dev))
    rt.v_slab.copy_(torch.randn(n, generator=g, device=dev))
    q = width * torch.randn(B, Hq, d, generator=g, device=dev)
    o = rt.decode_attn(q).cpu().numpy().astype(np.float64)
    K, V = (x.view(B, Hkv, P + 2, d)[:, :, :P].cpu().numpy().astype(np.float64) for x in (rt.k_slab, rt.v_slab))
    q = q.cpu().numpy().astype(np.float64)
    e2 = r2 = 0.0
    for s in range(0, B, B // 32):
        ref = OA.decode_attention(q[s], K[s].transpose(1, 0, 2), V[s].transpose(1, 0, 2), d ** -0.5)
        e2 += float(((o[s] - ref) ** 2).sum())
        r2 += float((ref ** 2).sum())
    assert (e2 / r2) ** 0.5 < bound, (e2 / r2) ** 0.5


@pytest.mark.parametrize("g,d", [(7, 64), (8, 64), (7, 128), (8, 128)])
@pytest.mark.parametrize("B", [256, 257, 280, 281])
def test_fp32_groups_of_seven_and_eight_with_more_pairs_than_compute_units(dev, g, d, B):
    # one workgroup a compute unit from 257 to 280 pairs, two otherwise; lengths around the tiles, the last pairs longest.  1e-5: fp32 rows
    import torch
    P = np.array([1 + (7 * s) % 140 for s in range(B)], np.int32)
    P[-3:] = 300, 301, 433
    rt = _bc().Runtime(B, g, 1, d, "f32", d ** -0.5, P, np.zeros(B, np.int32), P, dev)
    gen = torch.Generator(device=dev).manual_seed(4)
    n = int(P.sum()) * d
    rt.k_slab.copy_(torch.randn(n, generator=gen, device=dev))
    rt.v_slab.copy_(torch.randn(n, generator=gen, device=dev))
    q = torch.randn(B, g, d, generator=gen, device=dev)
    o = rt.decode_attn(q).cpu().numpy()
    K, V = (x.view(-1, 1, d).cpu().numpy().astype(np.float64) for x in (rt.k_slab, rt.v_slab))
    at = np.concatenate([[0], np.cumsum(P)])
    for s in list(range(0, B, 17)) + [B - 4, B - 3, B - 2, B - 1]:
        ref = OA.decode_attention(q[s].cpu().numpy().astype(np.float64), K[at[s]:at[s + 1]], V[at[s]:at[s + 1]], d ** -0.5)
        assert np.abs(o[s] - ref).max() < 1e-5, s


@pytest.mark.parametrize("Hq,Hkv,d,rows", [(4, 1, 64, 0), (12, 2, 128, 0), (8, 1, 128, 0), (3, 3, 64, 0), (7, 1, 64, 128),
                                           (10, 2, 128, 64)])
def test_fp32_rows_at_the_edges_of_their_tiles(dev, Hq, Hkv, d, rows):
    # tiles of 16 rows (d = 128) or 32 (d = 64), four waves to a pass: sequences that end in front of, at and behind the edges
    # of blocks, tiles and passes, with one tile a wave, two, and more; the appended row first in a tile and last; whole
    # and in forced chunks
    P = np.array([0, 1, 14, 15, 16, 30, 31, 47, 62, 63, 64, 111, 126, 127, 128, 191, 254, 255, 383, 600], np.int32)
    B, G = len(P), 5
    wl = W.Workload("rows32", 123, B, Hq, Hkv, d, "f32", P, np.full(B, G, np.int32),
                    np.resize(np.array([3, 0, 1, 16], np.int32), B))
    rt, oc = make(wl, dev)
    rt.cache.rows_per_workgroup = rows
    rollout(wl, rt, oc, G, range(1, G + 1), (3, G), use_step_call=True)
    q = wl.step_q(77)
    check_attention(rt.decode_attn(q).cpu().numpy(), q, oc, wl, None, 77)


@pytest.mark.parametrize("Hkv,d,plan", [(8, 128, 0), (9, 128, 0), (8, 128, 16), (9, 128, 16), (16, 64, 0), (17, 64, 0)])
def test_beacon_rows_of_as_many_heads_as_fit_lds_and_one_more(dev, Hkv, d, plan):
    # the step's beacon rows of all KV heads wait in 4 KB of LDS; with more heads they are read when they are written.
    # Two workgroups per pair (d = 128), one, and d = 64; short and second-tile sequences, an inactive ratio among them
    P = np.array([3, 60, 290, 400], np.int32)
    wl = W.Workload("beaconrows", 124, 4, Hkv, Hkv, d, "bf16", P, np.full(4, 12, np.int32), np.array([3, 1, 0, 4], np.int32))
    rt, oc = make(wl, dev)
    rt.cache.plan = plan
    st, text = _bc().bc_decode_plan_describe(rt.shape, rt.cache)
    assert st == 0 and "chunks=1" in text, text
    rollout(wl, rt, oc, 12, range(1, 13), (4, 12), use_step_call=True)


@pytest.mark.parametrize("B,Hq,Hkv,d", [(65, 8, 8, 128), (161, 8, 8, 128), (129, 8, 8, 64), (65, 16, 8, 64), (65, 16, 8, 128)])
def test_fp32_groups_of_one_and_two_on_fma_instructions(dev, B, Hq, Hkv, d):
    # large batches of short sequences whose groups are so small that the FMA form is the faster one
    P = np.resize(np.array([0, 3, 31, 40, 17], np.int32), B)
    wl = W.Workload("fma", 125, B, Hq, Hkv, d, "f32", P, np.full(B, 12, np.int32), np.full(B, 3, np.int32))
    rt, oc = make(wl, dev)
    st, text = _bc().bc_decode_plan_describe(rt.shape, rt.cache)
    assert st == 0 and "false, true>" in text and "chunks=1" in text, text
    rollout(wl, rt, oc, 12, (1, 2, 3, 4, 12), (3, 12), use_step_call=True)
