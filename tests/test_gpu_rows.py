"""GPU parity of rows that begin and end anywhere: unpadded vocabularies that are not a multiple of 8, tensors whose
first element is not on a 16-byte boundary, and tensors that do not share their offsets."""
import numpy as np
import pytest
import torch

from paper_2605_05940_amd import binding, synth

from gpu_util import Guarded, check_row_canaries, compare_kd, dev

pytestmark = pytest.mark.gpu
DIVS = {"forward": 0, "reverse": 1, "skew": 2, "skew_reverse": 3}
PAD = 64


def _rows(T, V, pitch, off):
    """A NaN-poisoned buffer and its bf16 view [T, V] with row pitch `pitch`, `off` elements past a 16-byte boundary."""
    full = torch.full((T * pitch + 2 * PAD + off,), float("nan"), dtype=torch.bfloat16, device=dev())
    return full, full[PAD + off:PAD + off + T * pitch].view(T, pitch)[:, :V]


def _batch(V, k=0):
    """Logits of a few packed samples and labels on the edges of the row."""
    edges = [0, 1, 6, 7, 8, V // 2, V - 9, V - 8, V - 2, V - 1]
    T = 2 * len(edges)
    w = synth.scaled(synth.config(1), n_rows=1, row_len=T, vocab=V, length_lo=4, length_hi=9, topk=max(k, 1))
    lay = synth.make_layout(w)
    s = torch.empty((T, V), dtype=torch.bfloat16, device=dev())
    t = torch.empty_like(s)
    synth.fill_logits(w, s, t)
    lab = np.array([max(0, min(V - 1, edges[i % len(edges)])) for i in range(T)], np.int32)
    return w, lay, s, t, lab


def _call(lay, s, t, lab, *, V, pitch, offs, pitch_t=None, div="forward", tau=1.0, gs=0.75, ce=0.0, grad=True,
          inplace=False, topk=None, no_workspace=False):
    """The call on copies of the logits at the offsets `offs` = (student, teacher, gradient); checks the guards."""
    T = s.shape[0]
    fs, vs = _rows(T, V, pitch, offs[0])
    vs.copy_(s)
    vt = None
    if topk is None:
        _, vt = _rows(T, V, pitch_t or pitch, offs[1])
        vt.copy_(t)
    fg, vg = (fs, vs) if inplace else _rows(T, V, pitch, offs[2])
    out = {n: Guarded(T, torch.float32) for n in ("kd", "nll_s", "lse_s") + (("nll_t",) if topk is None else ())}
    status = torch.zeros(1, dtype=torch.int32, device=dev())
    binding.npd_kd_loss_fwd_bwd(
        vs, torch.from_numpy(lay.loss_mask).to(dev()), teacher_dense=vt, teacher_idx=topk[0] if topk else None,
        teacher_val=topk[1] if topk else None, labels=torch.from_numpy(lab).to(dev()), tau=tau, grad_scale=gs,
        ce_grad_scale=ce, divergence=DIVS[div], skew_alpha=0.1, grad_out=vg if grad else None, kd_tok=out["kd"].t,
        nll_tok=out["nll_s"].t, teacher_nll_tok=out["nll_t"].t if topk is None else None, lse_tok=out["lse_s"].t,
        dev_status=status, no_workspace=no_workspace)
    torch.cuda.synchronize()
    assert int(status.item()) == 0
    got = {n: b.check().cpu().numpy().astype(np.float64) for n, b in out.items()}
    if grad:
        check_row_canaries(fg[offs[0 if inplace else 2]:], T, V, pitch)
        got["grad"] = vg.float().cpu().numpy().astype(np.float64)
    return got


def _reference(oracle, lay, s, t, lab, div, tau, gs, ce):
    sb, tb = synth.bf16_bits(s), synth.bf16_bits(t)
    if div == "forward":
        return oracle.kd_dense(sb, tb, lab, lay.loss_mask, tau=tau, grad_scale=gs, ce_grad_scale=ce)
    ref = oracle.div_dense(sb, tb, div, 0.1, labels=lab, mask=lay.loss_mask, tau=tau, grad_scale=gs, ce_grad_scale=ce)
    nl = oracle.kd_dense(sb, tb, lab, lay.loss_mask, want_grad=False)
    ref.update(nll_s=nl["nll_s"], nll_t=nl["nll_t"], lse_s=nl["lse_s"])
    return ref


@pytest.mark.parametrize("V,pitch,offs,pitch_t", [
    (30631, 30631, (0, 0, 0), None),      # two slices; rows at every offset in turn
    (50003, 50003, (3, 3, 3), None),      # the tensors themselves begin inside a group
    (151937, 151937, (0, 0, 0), None),    # eight slices, one element beyond a multiple of 8
    (30624, 30624, (0, 0, 0), None),      # 16-byte aligned rows: two slices; padded rows
    (100005, 100008, (0, 0, 0), None),
    (151936, 151944, (5, 5, 5), None),    # every row at the same odd offset
    (50003, 50003, (1, 2, 1), None),      # teacher elsewhere: no common groups
    (50003, 50003, (1, 1, 4), None),      # gradient elsewhere
    (50003, 50003, (0, 0, 0), 50008),     # teacher padded, student not
    (50003, 50003, (0, 0, 0), 50011),     # another pitch, the same offsets
    (8199, 8199, (0, 0, 0), None),        # rows of one workgroup
    (20481, 20483, (7, 7, 7), None),
    (5003, 5003, (2, 2, 2), None),        # short rows
    (1001, 1001, (0, 0, 0), None),
    (17, 17, (0, 0, 0), None),            # one or two groups, most elements are edges
    (9, 9, (5, 5, 5), None),              # rows without a whole group among them
    # rows of one workgroup, 16-byte aligned: the last row of a shape and the first of the next
    (1024, 1024, (0, 0, 0), None), (1032, 1032, (0, 0, 0), None), (2048, 2048, (0, 0, 0), None),
    (2056, 2056, (0, 0, 0), None), (4096, 4096, (0, 0, 0), None), (4104, 4104, (0, 0, 0), None),
    (8192, 8192, (0, 0, 0), None), (8200, 8200, (0, 0, 0), None), (12288, 12288, (0, 0, 0), None),
    (12296, 12296, (0, 0, 0), None), (16384, 16384, (0, 0, 0), None), (16392, 16392, (0, 0, 0), None),
    (20480, 20480, (0, 0, 0), None), (20488, 20488, (0, 0, 0), None), (32768, 32768, (0, 0, 0), None),
    (32776, 32776, (0, 0, 0), None),
])
@pytest.mark.parametrize("div,tau,ce", [("forward", 1.0, 0.25), ("forward", 2.0, 0.0), ("reverse", 1.0, 0.25),
                                        ("skew", 1.0, 0.25), ("skew_reverse", 2.0, 0.0),
                                        ("forward", 2.0, 0.25), ("reverse", 0.5, 0.25), ("skew", 2.0, 0.25),
                                        ("skew_reverse", 2.0, 0.25),   # the CE term with a softmax of its own: squares
                                        ("forward", 0.5, 0.25), ("reverse", 2.0, 0.25), ("skew", 3.0, 0.25),
                                        ("skew_reverse", 0.5, 0.25)])  # and exponentials of its own
def test_dense_rows_at_any_offset(oracle, V, pitch, offs, pitch_t, div, tau, ce):
    w, lay, s, t, lab = _batch(V)
    ref = _reference(oracle, lay, s, t, lab, div, tau, 0.75, ce)
    bars = dict(grad_scale=0.75 + ce * max(1.0, tau), tau=tau, amp_from_ref=div != "forward",
                folded=div != "forward" or (tau == 1.0 or ce == 0.0) and pitch % 8 == 0 and offs == (0, 0, 0) and V >= 8192)
    kw = dict(V=V, pitch=pitch, offs=offs, pitch_t=pitch_t, div=div, tau=tau, ce=ce)
    for mode in (dict(), dict(inplace=True), dict(no_workspace=True)):
        print(f"[rows] V={V} pitch={pitch} offs={offs} pitch_t={pitch_t} {div} tau={tau} {mode}", flush=True)
        compare_kd(_call(lay, s, t, lab, **kw, **mode), ref, lay.loss_mask, lay.cu_seqlens, oracle, **bars)
    fwd = _call(lay, s, t, lab, **kw | dict(ce=0.0), grad=False)
    compare_kd(fwd, {n: ref[n] for n in ("kd", "nll_s", "nll_t", "lse_s")}, lay.loss_mask, lay.cu_seqlens, oracle)


@pytest.mark.parametrize("V,pitch,offs", [
    (30631, 30631, (0, 0, 0)), (151936, 151936, (0, 0, 0)), (151937, 151937, (3, 3, 3)), (50003, 50003, (1, 1, 4)), (8199, 8199, (0, 0, 0)),
    (2003, 2003, (6, 6, 6)), (40, 43, (0, 0, 0)),
    (1024, 1024, (0, 0, 0)), (1032, 1032, (0, 0, 0)), (2056, 2056, (0, 0, 0)), (4096, 4096, (0, 0, 0)),
    (4104, 4104, (0, 0, 0)), (8200, 8200, (0, 0, 0)), (16392, 16392, (0, 0, 0)), (20488, 20488, (0, 0, 0)),
    (32768, 32768, (0, 0, 0)),
])
@pytest.mark.parametrize("tau,ce", [(1.0, 0.25), (2.0, 0.0), (2.0, 0.25)])
def test_topk_rows_at_any_offset(oracle, V, pitch, offs, tau, ce):
    k = 20
    w, lay, s, t, lab = _batch(V, k)
    idx, val = synth.make_topk_teacher(w, s)
    idx_np = idx.cpu().numpy().copy()
    for r in range(idx_np.shape[0]):  # support on both edges of the row; in even rows the label is in it
        want = [0, 1, 7, V - 1, V - 2, V - 8] + ([int(lab[r])] if r % 2 == 0 else [])
        want = list(dict.fromkeys(want))
        idx_np[r] = want + [int(v) for v in idx_np[r] if int(v) not in want][:k - len(want)]
    topk = (torch.from_numpy(idx_np).to(dev()), val)
    ref = oracle.kd_topk(synth.bf16_bits(s), idx_np, val.cpu().numpy(), lab, lay.loss_mask, tau=tau, grad_scale=0.75,
                         ce_grad_scale=ce)
    kw = dict(V=V, pitch=pitch, offs=offs, tau=tau, ce=ce, topk=topk)
    for mode in (dict(), dict(inplace=True), dict(no_workspace=True)):
        print(f"[rows] top-k V={V} pitch={pitch} offs={offs} tau={tau} {mode}", flush=True)
        compare_kd(_call(lay, s, None, lab, **kw, **mode), ref, lay.loss_mask, lay.cu_seqlens, oracle,
                   grad_scale=0.75 + ce * max(1.0, tau), tau=tau,
                   folded=(tau == 1.0 or ce == 0.0) and pitch % 8 == 0 and offs == (0, 0, 0) and V >= 8192)
    fwd = _call(lay, s, None, lab, **kw | dict(ce=0.0), grad=False)
    compare_kd(fwd, {n: ref[n] for n in ("kd", "nll_s", "lse_s")}, lay.loss_mask, lay.cu_seqlens, oracle)


def test_composite_at_a_temperature_without_its_workspace(oracle):
    """The CE term at tau != 1 takes the shared-row kernels with a workspace and the ones that need none without, be it
    absent, short, off its alignment or over an output: never an error, the same result to rounding."""
    V, tau, ce = 50264, 2.0, 0.25
    w, lay, s, t, lab = _batch(V)
    T = s.shape[0]
    ref = _reference(oracle, lay, s, t, lab, "forward", tau, 0.75, ce)
    need = 16 * 4 * T * 3 + 256
    buf = torch.empty(need + 512, dtype=torch.uint8, device=dev())
    off = -buf.data_ptr() % 256
    mask, labels = torch.from_numpy(lay.loss_mask).to(dev()), torch.from_numpy(lab).to(dev())
    grad = torch.empty_like(s)
    for ws in (buf[off:off + need], buf[off:off + 512], buf[off + 8:off + 8 + need],
               grad.view(torch.uint8).view(-1)[-grad.data_ptr() % 256:]):
        kd, nll = (torch.empty(T, device=dev()) for _ in range(2))
        binding.npd_kd_loss_fwd_bwd(s, mask, teacher_dense=t, labels=labels, tau=tau, grad_scale=0.75,
                                    ce_grad_scale=ce, grad_out=grad, kd_tok=kd, nll_tok=nll, workspace=ws)
        torch.cuda.synchronize()
        got = dict(kd=kd.cpu().numpy().astype(np.float64), nll_s=nll.cpu().numpy().astype(np.float64),
                   grad=grad.float().cpu().numpy().astype(np.float64))
        compare_kd(got, ref, lay.loss_mask, lay.cu_seqlens, oracle, grad_scale=0.75 + ce * tau, tau=tau, folded=False)


@pytest.mark.parametrize("V,k", [(600, 600), (1000, 513), (3001, 1300), (9000, 4096)])
def test_long_topk_records_on_short_rows(oracle, V, k):
    """Records of hundreds of entries, up to the whole vocabulary: many support positions per group of eight."""
    w, lay, s, _, lab = _batch(V, 1)
    T = s.shape[0]
    g = torch.Generator(device=dev()).manual_seed(V)
    idx = torch.rand((T, V), generator=g, device=dev()).argsort(dim=1)[:, :k].to(torch.int32).contiguous()
    val = torch.randn((T, k), generator=g, device=dev())
    for tau, ce in ((1.0, 0.25), (3.0, 0.0)):
        print(f"[rows] long record V={V} k={k} tau={tau}", flush=True)
        ref = oracle.kd_topk(synth.bf16_bits(s), idx.cpu().numpy(), val.cpu().numpy(), lab, lay.loss_mask, tau=tau,
                             grad_scale=0.75, ce_grad_scale=ce)
        got = _call(lay, s, None, lab, V=V, pitch=V, offs=(0, 0, 0), tau=tau, ce=ce, topk=(idx, val))
        compare_kd(got, ref, lay.loss_mask, lay.cu_seqlens, oracle, grad_scale=0.75 + ce, tau=tau)


@pytest.mark.parametrize("V", [1000, 6003, 16384])
@pytest.mark.parametrize("low", [False, True])
def test_extreme_logits_on_short_rows(oracle, V, low):
    """Logits whose largest is far from a thread's first ones, rows of negative logits alone, and logits of a thousand:
    sums whose references have to follow the data."""
    w, lay, s, t, lab = _batch(V)
    s, t = s.float(), t.float()
    s[::3] = s[::3] * 40.0
    t[1::3] = t[1::3] * 40.0
    if low:
        s -= 900.0
        t -= 1200.0
    s[:, V // 3] += 500.0
    s, t = s.to(torch.bfloat16), t.to(torch.bfloat16)
    for div, tau, ce in (("forward", 1.0, 0.25), ("forward", 2.0, 0.25), ("skew", 1.0, 0.0)):
        print(f"[rows] extreme V={V} low={low} {div} tau={tau}", flush=True)
        ref = _reference(oracle, lay, s, t, lab, div, tau, 0.75, ce)
        got = _call(lay, s, t, lab, V=V, pitch=V, offs=(0, 0, 0), div=div, tau=tau, ce=ce)
        # per-position scalars are differences of numbers in the thousands: 1e-4 relative of those
        compare_kd(got, ref, lay.loss_mask, lay.cu_seqlens, oracle, grad_scale=0.75 + ce * tau, tau=tau,
                   amp_from_ref=div != "forward")


@pytest.mark.parametrize("V,pitch,off", [
    (1024, 1024, 0), (1000, 1003, 5), (2048, 2048, 0), (2056, 2056, 0), (4096, 4096, 0), (4104, 4104, 0),
    (8192, 8192, 0), (8199, 8199, 0), (16384, 16384, 0), (16392, 16392, 0), (32768, 32768, 0),
    (32775, 32775, 3), (32777, 32777, 3), (50003, 50003, 0), (151937, 151937, 1), (300, 301, 2), (17, 17, 1), (9, 9, 5),
])
@pytest.mark.parametrize("k", [1, 10, 64, 65, 256, 300])
def test_teacher_topk_rows_at_any_offset(oracle, V, pitch, off, k):
    _check_teacher_topk(oracle, V, pitch, off, k, 12)


@pytest.mark.parametrize("V,pitch", [(1024, 1024), (1032, 1032), (2048, 2048), (2051, 2051), (2056, 2056), (4100, 4100),
                                     (8192, 8192), (12291, 12291), (16384, 16384)])
@pytest.mark.parametrize("k", [10, 100, 256])
def test_teacher_topk_of_many_rows(oracle, V, pitch, k):
    """The same with so many rows that a row gets fewer threads."""
    _check_teacher_topk(oracle, V, pitch, 0, k, 1100)


def _check_teacher_topk(oracle, V, pitch, off, k, T):
    """The record of rows of every shape and offset, plain rows and rows of ties: distinct logits, a handful of values
    (long runs of equal logits at the cut), one value, negative ones alone, zeros of both signs, the largest on the
    edges."""
    k = min(k, V)
    g = torch.Generator(device=dev()).manual_seed(V * 1000 + k)
    x = 3.0 * torch.randn((T, V), generator=g, device=dev())
    x[1] = torch.randint(0, 3, (V,), generator=g, device=dev()).float()
    x[2] = 1.5
    x[3] = -x[3].abs() - 0.01
    x[4] = torch.where(torch.rand(V, generator=g, device=dev()) < 0.5, 0.0, -0.0)
    x[5, 0] = x[5, V - 1] = x[5, V // 2] = 50.0
    x[6] = -0.0
    x[6, V // 3:] = 0.0
    x[7] = torch.arange(V, device=dev()).float() - V
    x[8] = -x[7]
    _, t = _rows(T, V, pitch, off)
    t.copy_(x)
    mask = torch.ones(T, dtype=torch.uint8, device=dev())
    mask[10] = 0
    idx, val = Guarded(T * k, torch.int32), Guarded(T * k, torch.float32)
    print(f"[rows] teacher top-k V={V} pitch={pitch} off={off} k={k}", flush=True)
    for log_probs in (True, False):
        binding.npd_teacher_topk(t, k, topk_idx=idx.t.view(T, k), topk_val=val.t.view(T, k), loss_mask=mask,
                                 log_probs=log_probs)
        torch.cuda.synchronize()
        ref = oracle.teacher_topk(synth.bf16_bits(t.contiguous()), k, mask.cpu().numpy(), log_probs)
        np.testing.assert_array_equal(idx.check().cpu().numpy().reshape(T, k), ref["idx"])
        # the log-softmax subtracts one fp32 number near the row's largest logit (up to V in rows 7 and 8): its rounding
        # is half a step, at most 2^-23 of it
        bar = 2e-5 + 2.0 ** -23 * t.float().abs().amax(1, keepdim=True).cpu().numpy()
        assert (np.abs(val.check().cpu().numpy().reshape(T, k) - ref["val"]) <= bar).all()


def _scalar_errors(oracle, s, t, pitch, tau=1.0, ce=0.0, topk=None):
    """Root mean square over the rows of the errors of lse and kd, with a gradient and forward only."""
    T, V = s.shape
    mask, lab = np.ones(T, np.uint8), np.arange(T, dtype=np.int32)
    lay = synth.Layout(T, np.array([0, T], np.int32), mask, lab, np.zeros(1, bool))
    sb = synth.bf16_bits(s)
    ref = (oracle.kd_dense(sb, synth.bf16_bits(t), lab, mask, tau=tau, want_grad=False) if topk is None else
           oracle.kd_topk(sb, topk[0].cpu().numpy(), topk[1].cpu().numpy(), lab, mask, tau=tau, want_grad=False))
    kw = dict(V=V, pitch=pitch, offs=(0, 0, 0), tau=tau, topk=topk)
    errs = {}
    for mode, got in (("grad", _call(lay, s, t, lab, ce=ce, **kw)), ("forward", _call(lay, s, t, lab, grad=False, **kw))):
        for n in ("lse_s", "kd"):
            errs[mode, n] = float(np.sqrt(np.mean((got[n] - ref[n]) ** 2)))
    print(f"[rows] errors V={V} pitch={pitch} tau={tau} ce={ce} {errs}", flush=True)
    return errs


@pytest.mark.parametrize("V,pitch", [(2048, 2048), (8192, 8192), (5003, 5003), (24576, 24576), (50003, 50003)])
def test_rows_of_log_probabilities(oracle, V, pitch):
    """Rows of negative logits alone: exponents are taken against a thread's largest logit there too.

    The terms that carry a thread's sum lie within 8 bits of its largest, so an argument's rounding is at most 2^-22 of
    the term and the exponential's and the sum's own are of that size: 4e-7 for a log-sum-exp near 0.  kd weighs the same
    errors with differences of logits of about 4.  (Arguments as long as the row's spread, 64 bits and more, carry 2^-18.)"""
    g = torch.Generator(device=dev()).manual_seed(V)
    x = 8.0 * torch.randn((64, V), generator=g, device=dev())
    y = 0.8 * x + 4.0 * torch.randn((64, V), generator=g, device=dev())
    s, t = (torch.log_softmax(v, dim=1).to(torch.bfloat16) for v in (x, y))
    val, idx = torch.topk(t.float(), 50, dim=1)
    for topk in (None, (idx.to(torch.int32).contiguous(), val.contiguous())):
        errs = _scalar_errors(oracle, s, t, pitch, topk=topk)
        assert max(errs["grad", "lse_s"], errs["forward", "lse_s"]) <= 4e-7
        assert max(errs["grad", "kd"], errs["forward", "kd"]) <= 1.5e-6


@pytest.mark.parametrize("V", [32768, 50304])
@pytest.mark.parametrize("tau", [0.5, 2.0])
def test_composite_at_a_temperature_keeps_its_precision(oracle, V, tau):
    """Rows that a CE term at tau != 1 brings to the shared-row kernels: the errors of the streaming ones, whose exponents
    are as short as they can be.  Terms within 8 bits of a thread's largest: 2^-22 of the term for the argument, as much
    again for the exponential and the sums, times differences of logits of 2 / tau in kd."""
    g = torch.Generator(device=dev()).manual_seed(V)
    x = torch.randn((48, V), generator=g, device=dev())
    y = 0.8 * x + 0.5 * torch.randn((48, V), generator=g, device=dev())
    for scale, log_probs in ((3.0, False), (8.0, True)):
        s, t = ((torch.log_softmax(scale * v, dim=1) if log_probs else scale * v).to(torch.bfloat16) for v in (x, y))
        errs = _scalar_errors(oracle, s, t, V, tau=tau, ce=0.25)
        assert errs["grad", "kd"] <= (1.5e-6 if log_probs else 1e-6)
        if log_probs:  # near 0: the rounding of the result itself is out of the way
            assert errs["grad", "lse_s"] <= 2e-7


@pytest.mark.parametrize("V,k,T", [
    (1000, 20, 1030), (1000, 600, 30),      # 64 threads to a row, four rows to a workgroup | 128 threads
    (1032, 64, 1030), (2048, 255, 1030), (2048, 256, 1030), (2051, 300, 30),
    (3000, 200, 1030), (4096, 128, 1030), (4096, 129, 1030), (4096, 1025, 30),
    (5000, 100, 1030), (8192, 200, 1030), (8192, 513, 1030), (8195, 40, 30),
    (8200, 64, 1030), (16384, 300, 1030), (16387, 20, 30),
    (16392, 300, 30), (20480, 64, 1030), (20488, 300, 30), (20488, 65, 1030), (20488, 65, 1300), (32768, 100, 640),
])
def test_topk_teacher_by_rows_and_record(oracle, V, k, T):
    """Every shape of the one-workgroup kernels for a top-k teacher: few rows and many, short records and long ones."""
    g = torch.Generator(device=dev()).manual_seed(V + k)
    s = (3.0 * torch.randn((T, V), generator=g, device=dev())).to(torch.bfloat16)
    idx = torch.empty((T, k), dtype=torch.int32, device=dev())
    for r in range(0, T, 128):
        idx[r:r + 128] = torch.rand((min(128, T - r), V), generator=g, device=dev()).topk(k, dim=1)[1]
    val = torch.randn((T, k), generator=g, device=dev())
    mask = np.ones(T, np.uint8)
    mask[::17] = 0
    lay = synth.Layout(T, np.array([0, T], np.int32), mask, None, np.zeros(1, bool))
    lab = idx[:, k // 2].cpu().numpy().copy()  # the label among the entries, elsewhere in every other row
    lab[::2] = np.random.default_rng(V).integers(0, V, lab[::2].size)
    for tau, ce in ((1.0, 0.25), (2.0, 0.0)):
        print(f"[rows] by rows and record V={V} k={k} T={T} tau={tau}", flush=True)
        ref = oracle.kd_topk(synth.bf16_bits(s), idx.cpu().numpy(), val.cpu().numpy(), lab, mask, tau=tau,
                             grad_scale=0.75, ce_grad_scale=ce)
        kw = dict(V=V, pitch=V, offs=(0, 0, 0), tau=tau, topk=(idx, val), no_workspace=True)
        compare_kd(_call(lay, s, None, lab, ce=ce, **kw), ref, mask, lay.cu_seqlens, oracle, grad_scale=0.75 + ce, tau=tau)
        compare_kd(_call(lay, s, None, lab, grad=False, **kw), {n: ref[n] for n in ("kd", "nll_s", "lse_s")}, mask,
                   lay.cu_seqlens, oracle)


# one row to a compute unit, half of one, two streams per compute unit, four; bounds from threads, groups and pairs of
# elements; lists that one wave sorts as they are (64, 128, 256, 512 words), cuts first, or leaves to the workgroup
@pytest.mark.parametrize("V,T,k", [
    (1000, 40, 256), (1100, 40, 128), (1100, 2000, 64), (520, 40, 256), (16391, 40, 256), (16400, 1024, 100),
    (16400, 1025, 100), (32775, 40, 200), (32776, 257, 64), (65536, 256, 256), (65543, 12, 20), (65544, 256, 200),
    (65544, 300, 200), (65544, 513, 48), (65544, 513, 49), (50304, 600, 256), (131080, 280, 500), (131080, 12, 513),
    (163840, 12, 190), (163848, 12, 192), (262144, 12, 256),
])
def test_teacher_topk_by_rows_and_length(oracle, V, T, k):
    _check_teacher_topk(oracle, V, V, 0, k, T)


# the register window of a streamed row: one window exactly, one and a part, two less a group, two, two and a part, three,
# with a whole and with a partial last group, at windows of 8 groups of 512 threads and of 12 and 20 of 1,024; and the
# numbers of rows, groups and k between which the kernel changes
@pytest.mark.parametrize("V,T,k", [
    (16400, 513, 10), (32776, 260, 10), (32768, 513, 10), (36864, 260, 20), (61440, 260, 20), (65536, 260, 7),
    (65544, 12, 10), (69632, 260, 64), (98304, 260, 33), (98312, 129, 52), (98312, 128, 51), (98312, 128, 53),
    (98304, 12, 190), (106496, 12, 190), (188416, 12, 140), (196608, 12, 140), (200008, 12, 140), (163840, 12, 140),
    (163848, 129, 55), (327680, 12, 200), (335872, 12, 10), (98304, 257, 256), (106496, 257, 256), (188416, 257, 256),
    (196616, 257, 256), (65600, 513, 201), (50304, 512, 250), (50304, 512, 251),
])
@pytest.mark.parametrize("off", [0, 3])
def test_teacher_topk_windows(oracle, V, T, k, off):
    _check_teacher_topk(oracle, V, V, off, k, T)


# lists longer than one wave takes: k around 512, every element a candidate, records of up to 1,024 entries; one window and more
@pytest.mark.parametrize("V,T,k", [
    (1040, 40, 512), (1040, 40, 513), (1030, 12, 1024), (2048, 40, 300), (2056, 12, 257), (4096, 40, 512), (4100, 12, 512),
    (4104, 12, 512), (8192, 12, 513), (8192, 12, 1024), (16400, 260, 700), (65600, 12, 500), (65600, 260, 1000),
    (98304, 12, 513), (98312, 12, 512), (98312, 40, 600), (131080, 260, 513), (200008, 12, 1024), (262144, 12, 700),
])
@pytest.mark.parametrize("off", [0, 3])
def test_teacher_topk_long_records(oracle, V, T, k, off):
    _check_teacher_topk(oracle, V, V, off, k, T)


@pytest.mark.parametrize("V,off,k,T", [(262144, 0, 10, 2747), (262144, 0, 10, 2746), (262131, 3, 40, 2760), (262144, 0, 41, 2760)])
def test_teacher_topk_of_rows_on_one_memory_channel(oracle, V, off, k, T):
    """Many rows with a pitch of 524,288 bytes: sixteen different ones over and over."""
    n, pitch = 16, 262144
    g = torch.Generator(device=dev()).manual_seed(V + k)
    x = 3.0 * torch.randn((n, V), generator=g, device=dev())
    x[1] = torch.randint(0, 3, (V,), generator=g, device=dev()).float()
    x[2] = -x[2].abs() - 0.01
    x[3] = torch.where(torch.rand(V, generator=g, device=dev()) < 0.5, 0.0, -0.0)
    x[4, 0] = x[4, V - 1] = x[4, V // 2] = 50.0
    _, t = _rows(T, V, pitch, off)
    for r in range(0, T, n):
        t[r:r + n].copy_(x[:min(n, T - r)])
    mask = torch.ones(T, dtype=torch.uint8, device=dev())
    idx, val = Guarded(T * k, torch.int32), Guarded(T * k, torch.float32)
    print(f"[rows] teacher top-k V={V} off={off} k={k} T={T}", flush=True)
    binding.npd_teacher_topk(t, k, topk_idx=idx.t.view(T, k), topk_val=val.t.view(T, k), loss_mask=mask, log_probs=False)
    torch.cuda.synchronize()
    ref = oracle.teacher_topk(synth.bf16_bits(x.to(torch.bfloat16)), k, np.ones(n, np.uint8), False)
    at = np.arange(T) % n
    np.testing.assert_array_equal(idx.check().cpu().numpy().reshape(T, k), ref["idx"][at])
    np.testing.assert_array_equal(val.check().cpu().numpy().reshape(T, k), ref["val"][at].astype(np.float32))


@pytest.mark.parametrize("T", [8, 300, 520])
def test_teacher_topk_keys_of_both_signs(oracle, T):
    """Candidates that span so many keys that one does not fit 32 bits beside its id: fewer positive logits than k."""
    V, k = 140000, 64
    g = torch.Generator(device=dev()).manual_seed(T)
    x = -1.0 - torch.rand((T, V), generator=g, device=dev())
    x[:, ::4000] = 300.0 + torch.randn((T, 35), generator=g, device=dev())
    t = x.to(torch.bfloat16)
    idx, val = torch.empty((T, k), dtype=torch.int32, device=dev()), torch.empty((T, k), device=dev())
    binding.npd_teacher_topk(t, k, topk_idx=idx, topk_val=val, log_probs=False)
    ref = oracle.teacher_topk(synth.bf16_bits(t), k, None, False)
    np.testing.assert_array_equal(idx.cpu().numpy(), ref["idx"])
    np.testing.assert_array_equal(val.cpu().numpy().astype(np.float64), ref["val"])


# threads of eight and ten groups unpack with the matrix cores, four values of a lane at a time, unless one of the wave's
# logits is not finite
@pytest.mark.parametrize("V", [12288, 16384, 20480, 24576, 50304, 50003])
@pytest.mark.parametrize("div,tau,ce", [("forward", 1.0, 0.0), ("forward", 1.0, 0.25), ("forward", 2.0, 0.25),
                                        ("forward", 3.0, 0.0), ("reverse", 1.0, 0.0), ("reverse", 2.0, 0.25)])
def test_masked_entries_among_finite_ones(oracle, V, div, tau, ce):
    w, lay, s, t, lab = _batch(V)
    s, t = s.clone(), t.clone()
    n = s.shape[0]
    for r in range(n):                                  # rows 0, 4, ...: none; one; every 67th; both tensors or one
        at = [] if r % 4 == 0 else [5 * r + 3] if r % 4 == 1 else list(range(r, V, 67))
        s[r, at] = float("-inf")
        if r % 4 != 2 or div == "reverse":              # (a teacher entry that the student masks: kd is infinite)
            t[r, at] = float("-inf")
        if r % 4 == 2 and div == "forward":
            s[r, at], t[r, at] = 1.0, float("-inf")
    y = lab.copy()
    y[:] = 1                                            # (not a masked entry)
    print(f"[rows] masked entries V={V} {div} tau={tau} ce={ce}", flush=True)
    ref = _reference(oracle, lay, s, t, y, div, tau, 0.75, ce)
    got = _call(lay, s, t, y, V=V, pitch=V, offs=(0, 0, 0), div=div, tau=tau, ce=ce)
    compare_kd(got, ref, lay.loss_mask, lay.cu_seqlens, oracle, grad_scale=0.75 + ce * tau, tau=tau,
               amp_from_ref=div != "forward")


# six groups per thread, the last one partly or fully there, and the first rows of eight; aligned and not
@pytest.mark.parametrize("V,off", [(8200, 0), (10241, 3), (12285, 5), (12288, 0), (12291, 1), (12296, 0)])
@pytest.mark.parametrize("tau", [1.0, 2.0, 3.0])
def test_forward_only_rows_of_six_groups(oracle, V, off, tau):
    w, lay, s, t, lab = _batch(V)
    s, t = s.clone(), t.clone()
    for r in range(1, s.shape[0], 2):                   # masked entries: one group of a thread is not finite
        s[r, r::613] = t[r, r::613] = float("-inf")
    y = lab.copy()
    y[1::2] = 0
    print(f"[rows] forward only V={V} off={off} tau={tau}", flush=True)
    ref = _reference(oracle, lay, s, t, y, "forward", tau, 1.0, 0.0)
    got = _call(lay, s, t, y, V=V, pitch=V, offs=(off, off, off), tau=tau, grad=False)
    compare_kd(got, {n: ref[n] for n in ("kd", "nll_s", "nll_t", "lse_s")}, lay.loss_mask, lay.cu_seqlens, oracle)
