"""Rows shared by workgroups with slices of 10, 7 or 5 groups per thread: which of them a call runs follows from its rows and
from whether its workspace has room for the record of the shorter ones."""
import ctypes

import numpy as np
import pytest
import torch

from gpu_util import compare_kd, dev
from paper_2605_05940_amd import binding, synth

pytestmark = pytest.mark.gpu
DIVS = {"forward": 0, "reverse": 1}


def _edges(V):
    """First and last elements of slices of all three lengths, next to a boundary that a row's address moves, and the tail."""
    nvec, e = V // 8, {0, V // 2, 8 * (V // 8) - 1, V - 1}
    for cap in (2552, 1784, 1272):
        g = -(-nvec // cap)
        per = -(-(-(-nvec // g)) // 8) * 8
        e |= {8 * per - 1, 8 * per, 8 * (per - 3), 8 * (g - 1) * per}
    return sorted(x for x in e if 0 <= x < V)


@pytest.mark.parametrize("V,pitch,T", [
    (30624, 30624, 24), (36000, 36008, 24), (40816, 40816, 24), (50003, 50003, 24), (65536, 65536, 24), (101760, 101760, 14),
    (151936, 151936, 12), (262144, 262144, 8), (36000, 36000, 360), (40817, 40832, 300), (42816, 42816, 290),
])
@pytest.mark.parametrize("what", ["forward", "forward_tau2", "reverse", "topk"])
def test_slices_of_every_length(oracle, V, pitch, T, what):
    w = synth.scaled(synth.config(1), n_rows=1, row_len=T, vocab=V, length_lo=4, length_hi=9)
    lay = synth.make_layout(w)
    g = torch.Generator(device=dev()).manual_seed(V + T)
    s, t, grad = (torch.empty((T, pitch), dtype=torch.bfloat16, device=dev())[:, :V] for _ in range(3))
    s.copy_(3.0 * torch.randn((T, V), generator=g, device=dev()))
    t.copy_(0.8 * s.float() + 1.5 * torch.randn((T, V), generator=g, device=dev()))
    mask = torch.from_numpy(lay.loss_mask).to(dev())
    edges = _edges(V)
    lab = np.array([edges[i % len(edges)] for i in range(T)], np.int32)
    sb, tb = synth.bf16_bits(s.contiguous()), synth.bf16_bits(t.contiguous())
    tau, ce = (2.0, 0.25) if what == "forward_tau2" else (1.0, 0.0 if T > 100 else 0.25)
    kw, kind = dict(tau=tau, grad_scale=0.75, ce_grad_scale=ce), binding.NPD_TEACHER_DENSE_BF16
    if what == "topk":
        k, kind = 24, binding.NPD_TEACHER_TOPK
        idx = torch.topk(t.float(), k, dim=1)[1].to(torch.int32)
        for r in range(T):                              # support positions on the edges; the label is one of them or not
            have = [e for e in edges if r % 2 == 0 or e != lab[r]][:k]
            rest = [int(i) for i in idx[r].tolist() if int(i) not in have and int(i) != lab[r]][:k - len(have)]
            idx[r] = torch.tensor(have + rest, dtype=torch.int32)
        val = t.float().gather(1, idx.long()).contiguous()
        ref = oracle.kd_topk(sb, idx.cpu().numpy(), val.cpu().numpy(), lab, lay.loss_mask, **kw)
        teacher = dict(teacher_idx=idx, teacher_val=val)
    else:
        div = what.split("_")[0]
        if div == "forward":
            ref = oracle.kd_dense(sb, tb, lab, lay.loss_mask, **kw)
        else:
            ref = oracle.div_dense(sb, tb, div, 0.1, labels=lab, mask=lay.loss_mask, **kw)
            nl = oracle.kd_dense(sb, tb, lab, lay.loss_mask, want_grad=False)
            ref.update(nll_s=nl["nll_s"], nll_t=nl["nll_t"], lse_s=nl["lse_s"])
        teacher = dict(teacher_dense=t, divergence=DIVS[div])
    d = binding.KdDesc(T, V, kind, pitch, pitch, 24 if what == "topk" else 0, 0, tau, 0.75, ce, teacher.get("divergence", 0),
                       0.0)
    need = int(binding.load().npd_workspace_bytes(ctypes.byref(d)))
    assert need > 0
    bits = {}
    for name, size in (("least", need), ("twice", 2 * need), ("more", 5 * need), ("binding", None)):
        print(f"[slices] V={V} pitch={pitch} T={T} {what} workspace {name}", flush=True)
        grad.fill_(float("nan"))
        out = {n: torch.full((T,), -1.0, device=dev()) for n in ("kd", "nll_s", "lse_s")}
        status = torch.zeros(1, dtype=torch.int32, device=dev())
        ws = None if size is None else torch.full((size + 64,), 7, dtype=torch.uint8, device=dev())
        binding.npd_kd_loss_fwd_bwd(s, mask, labels=torch.from_numpy(lab).to(dev()), grad_out=grad, kd_tok=out["kd"],
                                    nll_tok=out["nll_s"], lse_tok=out["lse_s"], dev_status=status,
                                    workspace=None if ws is None else ws[:size], **kw, **teacher)
        torch.cuda.synchronize()
        assert int(status.item()) == 0 and (ws is None or (ws[size:] == 7).all())
        got = {n: x.cpu().numpy().astype(np.float64) for n, x in out.items()}
        got["grad"] = grad.float().cpu().numpy().astype(np.float64)
        compare_kd(got, ref, lay.loss_mask, lay.cu_seqlens, oracle, grad_scale=0.75 + ce * tau, tau=tau,
                   amp_from_ref=what == "reverse")
        bits[name] = [grad.contiguous().view(torch.int16)] + [x.view(torch.int32) for x in out.values()]
    # what runs does not depend on how much more than twice the least a call is given
    for name in ("more", "binding"):
        assert all(torch.equal(a, b) for a, b in zip(bits[name], bits["twice"])), name


@pytest.mark.parametrize("V,pitch,T,tau,ce", [
    # slices of seven groups, two of them in LDS: fewer than of six, and more than 1,400 of those ...
    (26624, 26624, 470, 1.0, 0.0), (28675, 28675, 470, 1.0, 0.25), (26632, 26640, 470, 2.0, 0.25),
    # ... or sums at tau = 1 of their own, any number: two slices, a last slice of one group, 32 slices of six groups
    (18344, 18344, 12, 3.0, 0.25), (28560, 28576, 12, 3.0, 0.0), (42819, 42819, 12, 3.0, 0.25), (391168, 391168, 4, 3.0, 0.25),
])
@pytest.mark.parametrize("div", ["skew", "skew_reverse"])
def test_skew_slices_with_groups_in_lds(oracle, V, pitch, T, tau, ce, div):
    w = synth.scaled(synth.config(1), n_rows=1, row_len=T, vocab=V, length_lo=4, length_hi=min(9, T))
    lay = synth.make_layout(w)
    mask_np = lay.loss_mask.copy()
    mask_np[:3] = 1
    g = torch.Generator(device=dev()).manual_seed(V + T)
    s, t, grad = (torch.empty((T, pitch), dtype=torch.bfloat16, device=dev())[:, :V] for _ in range(3))
    s.copy_(3.0 * torch.randn((T, V), generator=g, device=dev()))
    t.copy_(0.8 * s.float() + 1.5 * torch.randn((T, V), generator=g, device=dev()))
    # waves that sum once more in the careful form: logits far above the first group's, entries of probability 0
    s[1, V // 2] = 420.0
    t[1, V // 2 + 300] = 400.0
    s[2, V - 70:] = float("-inf")
    t[2, V - 70:] = float("-inf")
    lab = np.minimum(lay.labels, V - 71).astype(np.int32)
    ref = oracle.div_dense(synth.bf16_bits(s.contiguous()), synth.bf16_bits(t.contiguous()), div, 0.1, labels=lab, mask=mask_np,
                           tau=tau, grad_scale=0.75, ce_grad_scale=ce)
    grad.fill_(float("nan"))
    kd, nll = (torch.full((T,), -1.0, device=dev()) for _ in range(2))
    status = torch.zeros(1, dtype=torch.int32, device=dev())
    print(f"[skew slices] V={V} pitch={pitch} T={T} tau={tau} {div}", flush=True)
    binding.npd_kd_loss_fwd_bwd(s, torch.from_numpy(mask_np).to(dev()), teacher_dense=t, labels=torch.from_numpy(lab).to(dev()),
                                tau=tau, grad_scale=0.75, ce_grad_scale=ce, divergence=2 if div == "skew" else 3, skew_alpha=0.1,
                                grad_out=grad, kd_tok=kd, nll_tok=nll, dev_status=status)
    torch.cuda.synchronize()
    assert int(status.item()) == 0
    got = dict(kd=kd.cpu().numpy().astype(np.float64), grad=grad.float().cpu().numpy().astype(np.float64))
    compare_kd(got, ref, mask_np, None, oracle, grad_scale=0.75 + ce * tau, tau=tau, amp_from_ref=True)


@pytest.mark.parametrize("V,pitch,T", [
    # four slices of four pieces of 256 groups: full, one group more and less, the last piece begun by the shift alone
    (32768, 32768, 12), (32776, 32776, 12), (32760, 32768, 12), (32747, 32752, 12), (32768, 32776, 12),
    (61440, 61448, 12), (40928, 40936, 290),
])
@pytest.mark.parametrize("what", ["forward", "forward_tau2", "reverse", "skew", "skew_tau3", "topk"])
def test_pieces_dealt_to_the_slices(oracle, V, pitch, T, what):
    if T > 100 and what in ("skew_tau3", "topk"):
        pytest.skip("short rows cover it")
    w = synth.scaled(synth.config(1), n_rows=1, row_len=T, vocab=V, length_lo=4, length_hi=9)
    lay = synth.make_layout(w)
    mask_np = lay.loss_mask.copy()
    mask_np[:9] = 1
    g = torch.Generator(device=dev()).manual_seed(V + pitch)
    s, t, grad = (torch.empty((T, pitch), dtype=torch.bfloat16, device=dev())[:, :V] for _ in range(3))
    s.copy_(3.0 * torch.randn((T, V), generator=g, device=dev()))
    t.copy_(0.8 * s.float() + 1.5 * torch.randn((T, V), generator=g, device=dev()))
    # No logit near 0 in some rows, most of the probability at the ends of pieces' first threads: a thread whose first group lies
    # in front of the row must not take that group for its reference.  (200, not 1,500: a top-k loss is a sum of differences of
    # logits times log2(e) and normalisers, three roundings of half of 2^-15 at 289, 3.2e-5 in all; at 2,164 they are 2.5e-4,
    # beyond the bar for positions whose loss is small.)
    for x in (s, t):
        x[2:9] -= 200.0
        for j in range(1, V // 2048):
            x[2:9, 8 * (256 * j - 7):8 * 256 * j] += 12.0
    # labels and support positions around the beginnings of pieces, whatever the shift
    edges = sorted({min(max(0, 8 * (256 * j - r) + d), V - 1) for j in range(0, V // 2048 + 1, 3) for r in (0, 3, 7) for d in (-1, 0)} |
                   {V - 1})
    lab = np.array([edges[(5 * i) % len(edges)] for i in range(T)], np.int32)
    sb, tb = synth.bf16_bits(s.contiguous()), synth.bf16_bits(t.contiguous())
    tau = 3.0 if what == "skew_tau3" else 2.0 if what == "forward_tau2" else 1.0
    ce = 0.25 if T < 100 else 0.0
    kw = dict(tau=tau, grad_scale=0.75, ce_grad_scale=ce)
    div = what.split("_")[0]
    if what == "topk":
        k = 24
        idx = torch.topk(t.float(), k, dim=1)[1].to(torch.int32)
        for r in range(T):
            have = edges[r % 3::max(3, len(edges) // 12)][:12]
            rest = [int(i) for i in idx[r].tolist() if int(i) not in have][:k - len(have)]
            idx[r] = torch.tensor(have + rest, dtype=torch.int32)
        val = t.float().gather(1, idx.long()).contiguous()
        ref = oracle.kd_topk(sb, idx.cpu().numpy(), val.cpu().numpy(), lab, mask_np, **kw)
        teacher = dict(teacher_idx=idx, teacher_val=val)
    elif div == "forward":
        ref = oracle.kd_dense(sb, tb, lab, mask_np, **kw)
        teacher = dict(teacher_dense=t)
    else:
        ref = oracle.div_dense(sb, tb, div, 0.1, labels=lab, mask=mask_np, **kw)
        teacher = dict(teacher_dense=t, divergence=1 if div == "reverse" else 2, skew_alpha=0.1)
    print(f"[pieces] V={V} pitch={pitch} T={T} {what}", flush=True)
    out = {}
    for in_place in (False, True):
        grad.fill_(float("nan"))
        if in_place:
            grad.copy_(s)
        kd = torch.full((T,), -1.0, device=dev())
        status = torch.zeros(1, dtype=torch.int32, device=dev())
        binding.npd_kd_loss_fwd_bwd(grad if in_place else s, torch.from_numpy(mask_np).to(dev()),
                                    labels=torch.from_numpy(lab).to(dev()), grad_out=grad, kd_tok=kd, dev_status=status, **kw,
                                    **teacher)
        torch.cuda.synchronize()
        assert int(status.item()) == 0
        got = dict(kd=kd.cpu().numpy().astype(np.float64), grad=grad.float().cpu().numpy().astype(np.float64))
        compare_kd(got, ref, mask_np, None, oracle, grad_scale=0.75 + ce * tau, tau=tau, amp_from_ref=div in ("reverse", "skew"),
                   folded=True)
        out[in_place] = grad.contiguous().view(torch.int16).clone()
    assert torch.equal(out[False], out[True])


@pytest.mark.parametrize("V,pitch,T,what", [
    (30624, 30624, 8192, "forward"), (30631, 30632, 8191, "forward"), (50003, 50003, 5462, "forward"), (56007, 56007, 5462, "forward"),
    (56008, 56064, 5462, "forward"), (26000, 26000, 5470, "skew"), (45000, 45000, 5470, "topk"), (45003, 45003, 5470, "topk"),
])
def test_zeros_around_a_few_scored_rows(oracle, V, pitch, T, what):
    """Many rows that are not scored around a few that are: every group and edge of theirs is zeroed, and nothing else."""
    g = torch.Generator(device=dev()).manual_seed(V + T)
    s, t = (torch.zeros((T, pitch), dtype=torch.bfloat16, device=dev())[:, :V] for _ in range(2))
    grad = torch.full((T, pitch), float("nan"), dtype=torch.bfloat16, device=dev())[:, :V]
    rows = [0, 1, T // 2, T - 2]
    x = 3.0 * torch.randn((len(rows), V), generator=g, device=dev())
    s[rows] = x.to(torch.bfloat16)
    t[rows] = (0.8 * x + 1.5 * torch.randn(x.shape, generator=g, device=dev())).to(torch.bfloat16)
    mask = torch.zeros(T, dtype=torch.uint8, device=dev())
    mask[rows] = 1
    kw = {}
    ones = np.ones(len(rows), np.uint8)
    lab = np.zeros(len(rows), np.int32)
    sb, tb = synth.bf16_bits(s[rows].contiguous()), synth.bf16_bits(t[rows].contiguous())
    if what == "topk":
        idx = torch.arange(9, dtype=torch.int32, device=dev()).repeat(T, 1)
        val = torch.zeros((T, 9), device=dev())
        val[rows], i = torch.topk(t[rows].float(), 9, dim=1)
        idx[rows] = i.to(torch.int32)
        kw.update(teacher_idx=idx, teacher_val=val)
        ref = oracle.kd_topk(sb, idx[rows].cpu().numpy(), val[rows].cpu().numpy(), lab, ones, tau=1.0, grad_scale=0.75)
    else:
        kw.update(teacher_dense=t)
        if what == "skew":
            kw.update(divergence=2, skew_alpha=0.1)
            ref = oracle.div_dense(sb, tb, "skew", 0.1, labels=lab, mask=ones, tau=1.0, grad_scale=0.75)
        else:
            ref = oracle.kd_dense(sb, tb, lab, ones, tau=1.0, grad_scale=0.75)
    kd = torch.full((T,), -1.0, device=dev())
    print(f"[zeros] V={V} pitch={pitch} T={T} {what}", flush=True)
    binding.npd_kd_loss_fwd_bwd(s, mask, grad_scale=0.75, grad_out=grad, kd_tok=kd, **kw)
    torch.cuda.synchronize()
    off = mask == 0
    assert all((grad[i:i + 512][off[i:i + 512]].view(torch.int16) == 0).all() for i in range(0, T, 512)) and (kd[off] == 0).all()
    if pitch > V:                                          # the padding between rows is nobody's
        whole = grad.as_strided((T - 1, pitch - V), (pitch, 1), V)
        assert torch.isnan(whole.float()).all()
    got = dict(kd=kd[rows].cpu().numpy().astype(np.float64), grad=grad[rows].float().cpu().numpy().astype(np.float64))
    compare_kd(got, ref, ones, None, oracle, grad_scale=0.75, amp_from_ref=what == "skew")
