"""Reductions over the packed layout at the sizes where their loops change: one position per thread and batches of eight
(256 threads a sample, 1,024 the batch of the monitor), four samples to a workgroup, pairs of one workgroup or several."""
import numpy as np
import pytest
import torch

from gpu_util import Guarded, dev
from paper_2605_05940_amd import binding

pytestmark = pytest.mark.gpu


def _rel_bound(n, threads):
    """Non-negative fp32 terms, ceil(n / threads) of them added one after another, then at most 20 additions of the tree."""
    return (n / threads + 22) * 2.0 ** -24


@pytest.mark.parametrize("n", [1, 255, 256, 257, 511, 512, 513, 1024, 1025, 2048, 2049, 2304, 2305, 2560, 2561, 3072, 3073, 4096,
                               4097, 4609, 20000])
def test_segments_around_the_batches(oracle, n):
    rng = np.random.default_rng(n)
    cu = np.array([0, n, n, n + 3, 2 * n + 3, 2 * n + 260], np.int32)
    T = int(cu[-1]) + 5
    x = rng.random(T).astype(np.float32)
    mask = (rng.random(T) < 0.7).astype(np.uint8)
    x[mask == 0] = np.nan                                  # not scored: read, but never added
    d = lambda a: torch.from_numpy(a).to(dev())
    S = len(cu) - 1
    s, m, c, t2s = (Guarded(k, t) for k, t in ((S, torch.float32), (S, torch.float32), (S, torch.int32), (T, torch.int32)))
    binding.npd_segment_reduce(d(x), d(mask), d(cu), seg_sum=s.t, seg_mean=m.t, seg_count=c.t, token_to_sample=t2s.t)
    lag = {k: Guarded(z, t) for k, z, t in (("seg_kl_mean", S, torch.float32), ("seg_count", S, torch.int32),
                                           ("batch_kl_mean", 1, torch.float32), ("batch_count", 1, torch.int32),
                                           ("lag_exceeded", 1, torch.int32))}
    binding.npd_policy_lag(d(x), d(mask), d(cu), 0.4, **{k: g.t for k, g in lag.items()})
    torch.cuda.synchronize()
    ref = oracle.segment_reduce(np.where(mask, x, 0.0), mask, cu)
    np.testing.assert_array_equal(c.check().cpu().numpy(), ref["count"])
    np.testing.assert_array_equal(t2s.check().cpu().numpy(), ref["token_to_sample"])
    for got, want in ((s, ref["sum"]), (m, ref["mean"]), (lag["seg_kl_mean"], ref["mean"])):
        np.testing.assert_allclose(got.check().cpu().numpy(), want, rtol=_rel_bound(n, 256), atol=0)
    np.testing.assert_array_equal(lag["seg_count"].check().cpu().numpy(), ref["count"])
    want = oracle.policy_lag(np.where(mask, x, 0.0), mask, cu, 0.4)
    assert int(lag["batch_count"].check().item()) == want["batch_count"]
    np.testing.assert_allclose(lag["batch_kl_mean"].check().item(), want["batch_mean"], rtol=_rel_bound(T, 1024))
    assert int(lag["lag_exceeded"].check().item()) == want["exceeded"]


@pytest.mark.parametrize("P", [1, 256, 257, 1024, 1025, 3000])
def test_kept_pairs_of_one_workgroup_or_several(oracle, P):
    rng = np.random.default_rng(P)
    S = 64
    ms, mt = (rng.uniform(0.5, 2.0, S).astype(np.float32) for _ in range(2))
    cnt = rng.integers(0, 3, S).astype(np.int32)
    pc, pu = (rng.integers(0, S, P).astype(np.int32) for _ in range(2))
    d = lambda a: torch.from_numpy(a).to(dev())
    zone, keep, count = Guarded(P, torch.uint8), Guarded(P, torch.uint8), Guarded(1, torch.int32)
    for _ in range(2):                                     # written, not accumulated
        binding.npd_delta_ifd_score(d(ms), d(mt), d(cnt), d(pc), d(pu), -0.3, 0.3, zone=zone.t, keep=keep.t,
                                    keep_count=count.t)
    torch.cuda.synchronize()
    ref = oracle.delta_ifd(ms, mt, cnt, pc, pu, -0.3, 0.3)
    clear = np.abs(np.abs(np.nan_to_num(ref["delta"], nan=9.0)) - 0.3) > 1e-5    # fp32 and fp64 agree off the thresholds
    np.testing.assert_array_equal(zone.check().cpu().numpy()[clear], ref["zone"][clear])
    assert int(count.check().item()) == int(keep.check().sum().item())
    kept = keep.check().clone()
    zone.poison()
    keep.poison()
    binding.npd_delta_ifd_score(d(ms), d(mt), d(cnt), d(pc), d(pu), -0.3, 0.3, zone=zone.t, keep=keep.t)   # no count
    assert torch.equal(keep.check(), kept)
    np.testing.assert_array_equal(zone.check().cpu().numpy()[clear], ref["zone"][clear])


@pytest.mark.parametrize("S", [(1 << 24) - 9, (1 << 24) - 8, (1 << 24) - 1])
def test_monitor_of_as_many_samples_as_a_grid_takes(S):
    """Almost all of them empty; the last three and one in the middle are not."""
    T = 64
    cu = torch.zeros(S + 1, dtype=torch.int32, device=dev())
    cu[S // 2:] += 10
    cu[S - 2:] += 20
    cu[S - 1:] += 15
    cu[S:] += 9
    x = torch.arange(T, device=dev(), dtype=torch.float32)
    mask = torch.ones(T, dtype=torch.uint8, device=dev())
    mean, count = Guarded(S, torch.float32), Guarded(S, torch.int32)
    batch, n, status = (torch.zeros(1, dtype=t, device=dev()) for t in (torch.float32, torch.int32, torch.int32))
    binding.npd_policy_lag(x, mask, cu, 0.1, seg_kl_mean=mean.t, seg_count=count.t, batch_kl_mean=batch, batch_count=n,
                           dev_status=status)
    torch.cuda.synchronize()
    want_n, want = torch.zeros(S, dtype=torch.int32, device=dev()), torch.zeros(S, device=dev())
    for i, a, b in ((S // 2 - 1, 0, 10), (S - 3, 10, 30), (S - 2, 30, 45), (S - 1, 45, 54)):
        want_n[i], want[i] = b - a, (a + b - 1) / 2
    assert torch.equal(count.check(), want_n) and torch.equal(mean.check(), want)      # (whole and half numbers: exact)
    assert int(n.item()) == 54 and float(batch.item()) == 26.5 and int(status.item()) == 0


def test_more_samples_than_a_grid_takes_are_refused():
    S = 1 << 24
    cu, mask = torch.zeros(S + 1, dtype=torch.int32, device=dev()), torch.ones(4, dtype=torch.uint8, device=dev())
    count = torch.zeros(S, dtype=torch.int32, device=dev())
    with pytest.raises(binding.NpdError) as e:
        binding.npd_segment_reduce(None, mask, cu, seg_count=count)
    assert e.value.status == 7
    binding.npd_segment_reduce(None, mask, cu[:4], seg_count=count[:3])
    torch.cuda.synchronize()
