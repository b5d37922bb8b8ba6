"""Forward-only calls whose rows are split over several workgroups, against the oracle and against the same call with a
workgroup per row."""
import ctypes

import numpy as np
import pytest
import torch

from gpu_util import compare_kd, dev, guarded_rows, run_gpu_kd
from paper_2605_05940_amd import binding, synth

pytestmark = pytest.mark.gpu


def _scratch(T, V, teacher, tau):
    d = binding.KdDesc(T, V, teacher, V, V, 0, binding.NPD_FLAG_FWD_ONLY, tau, 1.0, 0.0, 0, 0.0)
    return binding.load().npd_forward_scratch_bytes(ctypes.byref(d))


# slices of 1,024 groups of eight logits a tensor (up to 256 rows) or 2,048 (more, or no teacher): one more and one less than
# a whole number of them, rows at any offset, last slices that hold edge elements alone, the most slices a row may have (64)
DENSE = [
    (40968, 40968, 24), (49152, 49152, 24), (49160, 49160, 24), (50003, 50003, 24), (65537, 65600, 20), (98305, 98305, 20),
    (151936, 151936, 16), (262144, 262144, 8), (524288, 524288, 8), (40976, 40976, 300), (49159, 49159, 280),
    (65544, 65544, 270),
]
ALONE = [
    (65536, 65536, 24), (65544, 65544, 24), (81920, 81920, 24), (81931, 81931, 24), (98304, 98304, 100), (98305, 98408, 20),
    (114696, 114696, 40), (151936, 151936, 16), (262144, 262144, 8), (1048576, 1048576, 8), (240003, 240003, 290),
    (262151, 262151, 280),
]


@pytest.mark.parametrize("V,pitch,T,dense", [(*x, True) for x in DENSE] + [(*x, False) for x in ALONE])
def test_split_rows(oracle, V, pitch, T, dense):
    w = synth.scaled(synth.config(1), n_rows=1, row_len=T, vocab=V, length_lo=4, length_hi=16)
    lay = synth.make_layout(w)
    g = torch.Generator(device=dev()).manual_seed(V + T)
    s, t = (guarded_rows(T, V, pitch)[1] for _ in range(2))
    s.copy_(3.0 * torch.randn((T, V), generator=g, device=dev()))
    t.copy_(0.8 * s.float() + 1.5 * torch.randn((T, V), generator=g, device=dev()))
    m = lay.loss_mask.copy()
    m[1:8] = 1
    s[2] = torch.log_softmax(s[2].float(), 0) - 40.0            # negative logits alone
    s[3, V // 2:] = float("-inf")                               # masked vocabulary entries, in both and in one
    t[3, V // 2:] = float("-inf")
    t[4, ::3] = float("-inf")
    s[5, V - 1] = 700.0                                         # far above the other slices
    t[6, 0] = 900.0
    mask, lab = torch.from_numpy(m).to(dev()), torch.from_numpy(lay.labels).to(dev())
    lab[7] = V - 1
    lab[3:5] = 1                                                # (not a masked entry)
    labels = lab.cpu().numpy()
    assert _scratch(T, V, binding.NPD_TEACHER_NONE if not dense else 0, 1.0) > 0
    for tau in (1.0, 2.0) if dense else (1.0,):
        print(f"[split] V={V} pitch={pitch} T={T} dense={dense} tau={tau}", flush=True)
        got, one = (run_gpu_kd(s, mask, t=t if dense else None, labels=lab, tau=tau, want_grad=False, no_workspace=n)
                    for n in (False, True))
        if dense:
            ref = oracle.kd_dense(synth.bf16_bits(s.contiguous()), synth.bf16_bits(t.contiguous()), labels, m, tau=tau,
                                  want_grad=False)
        else:
            alone = oracle.nll(synth.bf16_bits(s.contiguous()), labels, m)
            ref = dict(nll_s=alone["nll"], lse_s=alone["lse"])
        compare_kd(got, ref, m)
        assert got["status"] == one["status"] == 0
        for key in ("kd", "nll_s", "nll_t", "lse_s"):
            if got[key] is not None:
                np.testing.assert_allclose(got[key], one[key], rtol=2e-5, atol=2e-5)


def test_split_rows_bad_label_and_replays():
    """A label outside the vocabulary marks its own row; a call that was captured gives the same on every replay."""
    T, V = 12, 65536
    g = torch.Generator(device=dev()).manual_seed(3)
    s, t = (torch.randn((T, V), generator=g, device=dev()).mul_(3).to(torch.bfloat16) for _ in range(2))
    mask, lab = torch.ones(T, dtype=torch.uint8, device=dev()), torch.arange(T, dtype=torch.int32, device=dev())
    kd, nll, tnll = (torch.empty(T, device=dev()) for _ in range(3))
    status = torch.zeros(1, dtype=torch.int32, device=dev())

    def call():
        binding.npd_kd_loss_fwd_bwd(s, mask, teacher_dense=t, labels=lab, kd_tok=kd, nll_tok=nll, teacher_nll_tok=tnll,
                                    dev_status=status)

    call()
    want = [x.clone() for x in (kd, nll, tnll)]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for _ in range(3):
        for x in (kd, nll, tnll):
            x.fill_(-1.0)
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip((kd, nll, tnll), want)) and status.item() == 0
    lab[5] = V
    call()
    assert status.item() == binding.NPD_DEV_BAD_LABEL and torch.isnan(nll[5]) and torch.isnan(tnll[5])
    assert torch.equal(kd, want[0]) and torch.equal(nll[:5], want[1][:5]) and torch.equal(nll[6:], want[1][6:])


@pytest.mark.parametrize("native", [True, False])
def test_forward_only_call_with_no_memory_left_for_its_scratch(native, monkeypatch):
    """Torch may allocate no more and its pools are used up: the call runs unsplit, as with no_workspace."""
    T, V = 24, 65536
    assert _scratch(T, V, 0, 1.0) > 0 and (not native or binding._host is not None)
    if not native:
        monkeypatch.setattr(binding, "_host", None)
    g = torch.Generator(device=dev()).manual_seed(9)
    s, t = (torch.randn((T, V), generator=g, device=dev()).mul_(3).to(torch.bfloat16) for _ in range(2))
    mask, kd, want = torch.ones(T, dtype=torch.uint8, device=dev()), torch.empty(T, device=dev()), torch.empty(T, device=dev())
    binding.npd_kd_loss_fwd_bwd(s, mask, teacher_dense=t, kd_tok=want, no_workspace=True)
    binding.npd_kd_loss_fwd_bwd(s, mask, teacher_dense=t, kd_tok=kd)
    torch.cuda.synchronize()
    assert not torch.equal(kd, want)                       # (summed in another order)
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    used = []
    try:
        torch.cuda.set_per_process_memory_fraction(torch.cuda.memory_reserved() / total)
        for n in (1 << 20, 1 << 16, 1 << 12, 512):         # what the allocator still holds
            try:
                while True:
                    used.append(torch.empty(n, dtype=torch.uint8, device=dev()))
            except torch.cuda.OutOfMemoryError:
                pass
        binding.npd_kd_loss_fwd_bwd(s, mask, teacher_dense=t, kd_tok=kd)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
        used.clear()
    torch.cuda.synchronize()
    assert torch.equal(kd, want)


@pytest.mark.parametrize("T,teacher_nll,split", [(1401, False, False), (1401, True, True), (600, False, True), (512, False, False)])
def test_which_sums_at_tau_one_are_split(T, teacher_nll, split):
    """The student's sum alone: many rows of a middling vocabulary stay whole (bit for bit as with no_workspace)."""
    V = 65536
    g = torch.Generator(device=dev()).manual_seed(T)
    s, t = (torch.randn((T, V), generator=g, device=dev()).mul_(3).to(torch.bfloat16) for _ in range(2))
    mask, lab = torch.ones(T, dtype=torch.uint8, device=dev()), torch.arange(T, dtype=torch.int32, device=dev())
    out = {}
    for n in (False, True):
        kd, nll, tnll = (torch.empty(T, device=dev()) for _ in range(3))
        binding.npd_kd_loss_fwd_bwd(s, mask, teacher_dense=t, labels=lab, tau=2.0, kd_tok=kd, nll_tok=nll,
                                    teacher_nll_tok=tnll if teacher_nll else None, no_workspace=n)
        out[n] = [kd, nll] + ([tnll] if teacher_nll else [])
    torch.cuda.synchronize()
    for a, b in zip(out[False], out[True]):
        torch.testing.assert_close(a, b, rtol=2e-5, atol=2e-5)
    assert all(torch.equal(a, b) for a, b in zip(out[False], out[True])) != split


def test_forward_entry_point_with_scratch_that_does_not_do():
    """NULL, too small, unaligned or overlapping another argument: the same call without, and nothing else is written."""
    T, V, L = 12, 65536, binding.load()
    g = torch.Generator(device=dev()).manual_seed(11)
    s, t = (torch.randn((T, V), generator=g, device=dev()).mul_(3).to(torch.bfloat16) for _ in range(2))
    mask = torch.ones(T, dtype=torch.uint8, device=dev())
    whole, split = torch.empty(T, device=dev()), torch.empty(T, device=dev())
    binding.npd_kd_loss_fwd_bwd(s, mask, teacher_dense=t, kd_tok=whole, no_workspace=True)
    binding.npd_kd_loss_fwd_bwd(s, mask, teacher_dense=t, kd_tok=split)
    d = binding.KdDesc(T, V, 0, V, V, 0, binding.NPD_FLAG_FWD_ONLY, 1.0, 1.0, 0.0, 0, 0.0)
    need = L.npd_forward_scratch_bytes(ctypes.byref(d))
    block = torch.full((need + 256,), 7, dtype=torch.uint8, device=dev())    # its first words are kd_tok in one call
    for name, kd, scratch, n, want in (("fits", None, 128, need, split), ("none", None, None, 0, whole),
                                       ("too small", None, 128, need - 1, whole), ("unaligned", None, 132, need, whole),
                                       ("overlaps kd_tok", block[64:64 + 4 * T].view(torch.float32), 0, need, whole),
                                       ("touches kd_tok", block[64:64 + 4 * T].view(torch.float32), 128, need, split)):
        block.fill_(7)
        kd = torch.empty(T, device=dev()) if kd is None else kd
        print(f"[split] scratch {name}", flush=True)
        st = L.npd_kd_loss_forward(ctypes.byref(d), s.data_ptr(), t.data_ptr(), None, None, None, mask.data_ptr(), kd.data_ptr(),
                                   None, None, None, None, None if scratch is None else block.data_ptr() + scratch, n,
                                   binding._stream())
        torch.cuda.synchronize()
        assert st == 0 and torch.equal(kd, want), name
        assert (block[:64] == 7).all() and (block[128 + need:] == 7).all(), name
        if want is whole:
            assert (block[128:] == 7).all(), name
    # one slice more than a row may have
    assert _scratch(8, 524288, 0, 1.0) > 0 and _scratch(8, 524296, 0, 1.0) == 0
    assert _scratch(8, 1048576, binding.NPD_TEACHER_NONE, 1.0) > 0 and _scratch(8, 1048584, binding.NPD_TEACHER_NONE, 1.0) == 0
