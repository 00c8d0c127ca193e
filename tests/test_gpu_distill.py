"""GPU parity: bc_topk_kl_loss / bc_topk_kl_loss_bwd (Eq. 1, Sec. 3.2; top-k teacher of App. A)
against the fp64 oracle.  Inputs are exact in the logits' dtype; the kernels accumulate in fp32.
Loss and log-sum-exp: max-abs-error 2e-5.  Gradient: each probability carries the fp32 error of
its exponent (log-sum-exp good to ~1e-6, so ~2e-6 relative to the probability, which is <= 1), and
at a teacher id two probabilities cancel, so the absolute part of the bound is 2e-6 * grad_scale;
on top comes one rounding to the output dtype: 2^-8 relative for bf16, 1e-5 for fp32."""
import numpy as np
import pytest

from oracle import distill as OD
from paper_2510_13797_amd import workloads as W

pytestmark = pytest.mark.gpu
TOL = 2e-5


@pytest.fixture(scope="module")
def dev():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch.device("cuda:0")


def _to_dev(z, tl, idx, dtype, dev):
    import torch
    from paper_2510_13797_amd import bc
    return (bc.to_device(z, dtype, dev), torch.from_numpy(tl).to(dev), torch.from_numpy(idx).to(dev))


def _grad_close(got, ref, dtype, gs):
    rel = 2.0 ** -8 if dtype == "bf16" else 1e-5
    bad = np.abs(got - ref) > rel * np.abs(ref) + 2e-6 * gs
    assert not bad.any(), (int(bad.sum()), float(np.abs(got - ref).max()))


def _check(wl, ts, dev, gs=None):
    from paper_2510_13797_amd import bc
    z, tl, idx = wl.tokens(ts)
    zd, tld, idxd = _to_dev(z, tl, idx, wl.dtype, dev)
    loss, lse, mean = bc.topk_kl_loss(zd, tld, idxd)
    ref_loss, ref_lse = OD.topk_kl_loss(z, tl, idx)
    assert np.abs(loss.cpu().numpy() - ref_loss).max() <= TOL
    assert np.abs(lse.cpu().numpy() - ref_lse).max() <= TOL
    assert abs(float(mean.cpu()[0]) - OD.batch_loss(ref_loss)) <= TOL
    gs = 1.0 / len(ts) if gs is None else gs
    dz = bc.topk_kl_loss_bwd(zd, tld, idxd, lse, gs).float().cpu().numpy()
    _grad_close(dz, OD.topk_kl_loss_grad(z, tl, idx, gs), wl.dtype, gs)
    return loss, dz


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("V,k", [(1000, 100), (1001, 100), (4104, 1), (64, 64), (8, 3), (5000, 700)])
def test_small_vocabularies(dev, dtype, V, k):
    # 1000: whole 16-byte units; 1001: element-wise path; k = 1, k = V, k > 256 (several per thread)
    wl = W.DistillWorkload("small", 37, V, k, dtype)
    _check(wl, range(37), dev, gs=0.25)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T,V,k", [(5, 3, 2), (3, 31, 5), (9, 8200, 10), (7, 32771, 1000), (1024, 257, 20), (1025, 4099, 300)])
def test_rows_that_start_anywhere(dev, dtype, T, V, k):
    # rows shorter than the way to the first 16-byte boundary, one unit more than a batch of loads, several
    # batches and a rest; both workgroup sizes; logits that start inside a 16-byte unit themselves, where the
    # gradient's rows do not lie alike and its element-wise form runs
    import torch
    from paper_2510_13797_amd import bc
    wl = W.DistillWorkload("rows", T, V, k, dtype)
    z, tl, idx = wl.tokens(range(T))
    zd, tld, idxd = _to_dev(z, tl, idx, dtype, dev)
    room = torch.empty(T * V + 3, dtype=zd.dtype, device=dev)
    for shift in (0, 1, 3):
        zs = room[shift:shift + T * V].view(T, V)
        zs.copy_(zd)
        loss, lse, _ = bc.topk_kl_loss(zs, tld, idxd)
        ref_loss, ref_lse = OD.topk_kl_loss(z, tl, idx)
        assert np.abs(loss.cpu().numpy() - ref_loss).max() <= TOL
        assert np.abs(lse.cpu().numpy() - ref_lse).max() <= TOL
        dz = bc.topk_kl_loss_bwd(zs, tld, idxd, lse, 0.5).float().cpu().numpy()
        _grad_close(dz, OD.topk_kl_loss_grad(z, tl, idx, 0.5), dtype, 0.5)


@pytest.mark.parametrize("T,V", [(256, 15360), (256, 15359), (257, 15360), (3, 7679), (3, 7680)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_both_sides_of_the_workgroup_size(dev, dtype, T, V):
    # 1024 threads for up to 256 tokens whose rows have 30 KB or more, 256 otherwise
    _check(W.DistillWorkload("threads", T, V, 40, dtype), range(T), dev, gs=0.25)


def test_paper_vocabulary_all_rows(dev):
    wl = W.distill(T=24)
    _check(wl, range(24), dev)


def test_paper_vocabulary_fp32(dev):
    wl = W.distill(T=6, dtype="f32")
    _check(wl, range(6), dev)


def test_full_micro_batch_sampled_rows_and_invariants(dev):
    # T = 4096 tokens at the timed launch shape: logits drawn on the device (the same recipe with
    # torch's generator), 12 sampled rows copied back and checked one by one against the oracle,
    # and for all rows: loss > 0, mean == mean of the rows, gradient rows sum to ~0
    import torch
    from paper_2510_13797_amd import bc
    T, V, k = 4096, 151936, 100
    g = torch.Generator(device=dev).manual_seed(1234)
    z = (2.0 * torch.randn((T, V), generator=g, device=dev, dtype=torch.float32)).to(torch.bfloat16)
    tl = torch.empty((T, k), dtype=torch.float32, device=dev)
    idx = torch.empty((T, k), dtype=torch.int32, device=dev)
    for t0 in range(0, T, 512):
        teacher = z[t0:t0 + 512].float() + torch.randn((512, V), generator=g, device=dev)
        top = torch.topk(teacher, k, dim=1)
        tl[t0:t0 + 512] = top.values
        idx[t0:t0 + 512] = top.indices.to(torch.int32)
        del teacher
    loss, lse, mean = bc.topk_kl_loss(z, tl, idx)
    dz = bc.topk_kl_loss_bwd(z, tl, idx, lse, 1.0 / T)
    lossh = loss.cpu().numpy()
    assert np.all(lossh > 0) and np.all(np.isfinite(lossh))
    assert abs(float(mean.cpu()[0]) - float(lossh.astype(np.float64).mean())) <= 1e-6
    rows = np.random.default_rng(3).choice(T, 12, replace=False)
    rows = np.concatenate([rows, [0, T - 1]])
    zr = z[rows].float().cpu().numpy()
    tlr, idxr = tl[rows].cpu().numpy(), idx[rows].cpu().numpy()
    ref_loss, ref_lse = OD.topk_kl_loss(zr, tlr, idxr)
    assert np.abs(lossh[rows] - ref_loss).max() <= TOL
    assert np.abs(lse.cpu().numpy()[rows] - ref_lse).max() <= TOL
    _grad_close(dz[rows].float().cpu().numpy(), OD.topk_kl_loss_grad(zr, tlr, idxr, 1.0 / T), "bf16", 1.0 / T)
    # softmax and the teacher both sum to one: every gradient row sums to zero up to bf16 rounding
    rs = dz.float().sum(dim=1).abs().max().item()
    assert rs <= 2.0 ** -8 / T * 4, rs


def test_argument_errors_and_bad_ids(dev):
    import torch
    from paper_2510_13797_amd import bc
    bc.load()
    wl = W.DistillWorkload("err", 4, 256, 10, "bf16")
    z, tl, idx = wl.tokens(range(4))
    idx[2, 3] = 256                      # out of range: that token's loss is NaN, the others are fine
    zd, tld, idxd = _to_dev(z, tl, idx, "bf16", dev)
    loss, lse, _ = bc.topk_kl_loss(zd, tld, idxd)
    lh = loss.cpu().numpy()
    assert np.isnan(lh[2]) and np.all(np.isfinite(lh[[0, 1, 3]]))
    dz = bc.topk_kl_loss_bwd(zd, tld, idxd, lse, 1.0)
    assert torch.isfinite(dz.float()).all()
    p = lambda t: t.data_ptr()
    out = torch.zeros(4, device=dev)
    assert bc.bc_topk_kl_loss(4, 256, 300, p(zd), bc.BC_BF16, p(tld), p(idxd), p(out), None, None, None) == bc.BC_ERR_SHAPE
    assert bc.bc_topk_kl_loss(4, 256, 10, None, bc.BC_BF16, p(tld), p(idxd), p(out), None, None, None) == bc.BC_ERR_ARG
    assert bc.bc_topk_kl_loss(4, 256, 10, p(zd), 7, p(tld), p(idxd), p(out), None, None, None) == bc.BC_ERR_SHAPE
    assert bc.bc_topk_kl_loss_bwd(4, 256, 10, p(zd), bc.BC_BF16, p(tld), p(idxd), p(lse), 1.0, p(zd), None) == bc.BC_ERR_ARG
    assert bc.bc_topk_kl_loss(0, 256, 10, p(zd), bc.BC_BF16, p(tld), p(idxd), p(out), None, None, None) == bc.BC_OK
