"""Performance cases of the packed KD loss: what a distillation program has this library do, through its Python entry
points, from the smallest call to a full pack of 32,768 positions.

Every case is one of five operations on a packed batch that is already in device memory:

  kd           one training step's loss: npd_kd_loss_fwd_bwd with a dense teacher (any divergence, with or without the CE
               term of the composite loss) and the per-sample means of its KD loss and NLL
  kd_topk      the same against a stored top-k teacher record
  ifd          the Delta-IFD scoring pass: forward-only NLLs of student and teacher, per-sample means, score and zones
  lag          the policy-latency monitor: forward-only KL(learner || generator) and its mean against the bound
  teacher_topk the teacher-side record: npd_teacher_topk

`tokens` are the positions of the batch, `vocab` the vocabulary, `pitch` the elements between rows of the logits
(vocab: an unpadded tensor, as a model's head returns it).
"""
import random

import torch

import paper_2605_05940_amd as npd
from paper_2605_05940_amd import binding

DEVICE = "cuda:0"
CHUNK = 1 << 26                 # logits generated / checked at a time
DIVERGENCES = {"forward": 0, "reverse": 1, "skew": 2, "skew_reverse": 3}
MAX_ELEMENTS = 1_500_000_000    # tokens * vocab of a drawn case: below the largest listed one


def listed():
    return [
        # A full training step at a 1B student's vocabulary: one pack of 32,768 positions, dense teacher, forward KL.
        dict(name="kd_32k_tokens", op="kd", tokens=32768, vocab=151936, pitch=151936, tau=1.0, divergence="forward",
             lam=1.0, values="normal"),
        # The largest vocabulary, heavy-tailed logits, the composite loss (CE + KD) at tau = 1.
        dict(name="kd_wide_vocab", op="kd", tokens=8192, vocab=262144, pitch=262144, tau=1.0, divergence="forward",
             lam=0.9, values="student_t3"),
        # The composite loss at a temperature, the textbook form of distillation: soft targets at tau = 2, hard labels.
        dict(name="kd_composite_tau2", op="kd", tokens=4096, vocab=151936, pitch=151936, tau=2.0,
             divergence="forward", lam=0.9, values="normal"),
        # A vocabulary that nobody padded: rows begin at any even byte.
        dict(name="kd_odd_vocab", op="kd", tokens=8192, vocab=50003, pitch=50003, tau=1.0, divergence="forward",
             lam=0.9, values="normal"),
        # Skew KL, the alternative divergence with the most arithmetic, on one row of 8,192 positions.
        dict(name="kd_skew", op="kd", tokens=8192, vocab=151936, pitch=151936, tau=1.0, divergence="skew", lam=1.0,
             values="normal"),
        # Reverse KL at a 32,000-entry vocabulary.
        dict(name="kd_reverse_32k_vocab", op="kd", tokens=16384, vocab=32000, pitch=32000, tau=1.0,
             divergence="reverse", lam=1.0, values="normal"),
        # A micro-batch of one short sample: too few rows to fill the chip by rows.
        dict(name="kd_64_tokens", op="kd", tokens=64, vocab=151936, pitch=151936, tau=1.0, divergence="forward",
             lam=1.0, values="normal"),
        # The smallest call: a few hundred positions of a 1,024-entry vocabulary, where launches and latency count.
        dict(name="kd_tiny", op="kd", tokens=512, vocab=1024, pitch=1024, tau=1.0, divergence="forward", lam=1.0,
             values="normal"),
        # Training against the stored record: top 64 at tau = 2.
        dict(name="kd_topk64_tau2", op="kd_topk", tokens=8192, vocab=151936, pitch=151936, tau=2.0, k=64, lam=1.0,
             values="normal"),
        # Data selection: score every sample with and without its instruction.
        dict(name="ifd_16k_tokens", op="ifd", tokens=16384, vocab=151936, pitch=151936, values="normal"),
        # The monitor that runs beside training on a small probe batch.
        dict(name="lag_256_tokens", op="lag", tokens=256, vocab=151936, pitch=151936, tau=1.0, values="normal"),
        # Writing the teacher's record: the 64 largest of every position.
        dict(name="teacher_topk64", op="teacher_topk", tokens=8192, vocab=151936, pitch=151936, k=64,
             values="normal"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    op = rng.choice(["kd", "kd", "kd", "kd", "kd", "kd_topk", "kd_topk", "ifd", "lag", "teacher_topk", "teacher_topk"])
    vocab = _log_uniform(rng, 1000, 262144)
    how = rng.random()
    if how < 0.5:
        vocab = max(64, vocab // 64 * 64)     # padded by the model
    elif how < 0.7:
        vocab = max(8, vocab // 8 * 8)
    else:
        vocab |= 1                            # as the tokenizer left it
    pitch = vocab
    if vocab % 64 and rng.random() < 0.4:
        pitch = (vocab + 63) // 64 * 64       # the tensor is padded, the vocabulary is not
    tokens = min(_log_uniform(rng, 256 if op == "ifd" else 16, 32768), MAX_ELEMENTS // vocab)
    case = dict(op=op, tokens=tokens, vocab=vocab, pitch=pitch, values=rng.choice(["normal", "normal", "student_t3"]))
    if op == "kd":
        case.update(tau=rng.choice([1.0, 1.0, 2.0]), lam=rng.choice([1.0, 0.9]),
                    divergence=rng.choice(["forward", "forward", "forward", "reverse", "skew", "skew_reverse"]))
    elif op == "kd_topk":
        case.update(tau=rng.choice([1.0, 1.0, 2.0]), lam=rng.choice([1.0, 0.9]), k=_log_uniform(rng, 5, 256))
    elif op == "lag":
        case.update(tau=1.0)
    elif op == "teacher_topk":
        case.update(k=_log_uniform(rng, 5, 256))
    return case


# ------------------------------------------------------------------------------------------------------ the packed batch

def _layout(case):
    """(cu_seqlens, scored positions as a list of (begin, end), pairs) of the batch, from its sizes alone: samples are
    appended to rows of up to 8,192 positions until one does not fit; the rest of the row is padding.  The Delta-IFD
    batch holds every response twice, once behind an instruction and once alone."""
    T = case["tokens"]
    rng = random.Random(T)
    row = min(T, 8192)
    cu, scored, pairs = [0], [], []

    def add(n, lead):
        cu.append(cu[-1] + n)
        if n > lead:
            scored.append((cu[-1] - n + lead, cu[-1]))

    while cu[-1] < T:
        end = min(T, cu[-1] + row)
        while True:
            if case["op"] == "ifd":
                n = _log_uniform(rng, row // 32, row // 4)
                q = rng.randint(row // 128 + 1, row // 16)
                if cu[-1] + q + 2 * n > end:
                    break
                add(q + n, q)
                add(n, 0)
                pairs.append((len(cu) - 3, len(cu) - 2))
            else:
                n = _log_uniform(rng, max(2, min(64, row // 8)), max(4, min(4096, row // 2)))
                if cu[-1] + n > end:
                    break
                add(n, int(n * rng.uniform(0.1, 0.3)))
        if cu[-1] < end:
            n = end - cu[-1]
            add(n, n)                           # padding: a segment without a scored position
    return cu, scored, pairs


def _n_scored(case):
    return sum(e - b for b, e in _layout(case)[1])


def _draw_values(shape, case, g):
    z = torch.randn(shape, generator=g, device=DEVICE)
    if case["values"] == "student_t3":
        chi = torch.zeros(shape, device=DEVICE)
        for _ in range(3):
            chi += torch.randn(shape, generator=g, device=DEVICE).square_()
        z /= chi.div_(3.0).sqrt_()
        return z.mul_(4.0 / 3.0)
    return z


def _rows(case):
    step = max(1, CHUNK // case["vocab"])
    return [(r, min(case["tokens"], r + step)) for r in range(0, case["tokens"], step)]


def _inputs(case, seed):
    """The batch on the GPU.  Student logits 3 N(0, 1) (or Student-t(3) times 4), teacher 0.8 student + 1.5 noise."""
    T, V, P = case["tokens"], case["vocab"], case["pitch"]
    g = torch.Generator(device=DEVICE)
    g.manual_seed(1000003 * int(seed) + 17)
    cu, scored, pairs = _layout(case)
    mask = torch.zeros(T, dtype=torch.uint8)
    for b, e in scored:
        mask[b:e] = 1
    st = dict(case=case, mask=mask.to(DEVICE), cu=torch.tensor(cu, dtype=torch.int32, device=DEVICE),
              labels=torch.randint(0, V, (T,), generator=g, device=DEVICE, dtype=torch.int32))
    need_s, need_t = case["op"] != "teacher_topk", case["op"] != "kd_topk"
    s = torch.empty((T, P), dtype=torch.bfloat16, device=DEVICE)[:, :V] if need_s else None
    t = torch.empty((T, P), dtype=torch.bfloat16, device=DEVICE)[:, :V] if need_t else None
    boost = None
    if case["op"] == "ifd":
        # both copies of a response predict the same tokens, better behind the instruction than without
        rng = random.Random(int(seed))
        boost = torch.zeros((2, T))
        for pc, pu in pairs:
            n = cu[pu + 1] - cu[pu]
            st["labels"][cu[pu]:cu[pu + 1]] = st["labels"][cu[pc + 1] - n:cu[pc + 1]]
            for m in (0, 1):
                base = rng.uniform(4.0, 10.0)
                boost[m, cu[pu]:cu[pu + 1]] = base
                boost[m, cu[pc]:cu[pc + 1]] = base + rng.uniform(-1.0, 4.0 + 2 * m)
        boost = boost.to(DEVICE)
        st["pairs"] = [torch.tensor([p[i] for p in pairs], dtype=torch.int32, device=DEVICE) for i in (0, 1)]
    if case["op"] == "kd_topk":
        st["idx"] = torch.empty((T, case["k"]), dtype=torch.int32, device=DEVICE)
        st["val"] = torch.empty((T, case["k"]), device=DEVICE)
    for r0, r1 in _rows(case):
        xs = _draw_values((r1 - r0, V), case, g).mul_(3.0)
        xt = _draw_values((r1 - r0, V), case, g).mul_(1.5).add_(xs, alpha=0.8)
        if boost is not None:
            at = torch.arange(r1 - r0, device=DEVICE), st["labels"][r0:r1].long()
            xs[at] += boost[0, r0:r1]
            xt[at] += boost[1, r0:r1]
        if need_s:
            s[r0:r1] = xs
        if need_t:
            t[r0:r1] = xt
        if case["op"] == "kd_topk":
            val, idx = torch.topk(xt, case["k"], dim=1)
            st["idx"][r0:r1] = idx
            st["val"][r0:r1] = torch.log_softmax(val, dim=1)
    st["s"], st["t"] = s, t
    n = max(1, _n_scored(case))
    lam, tau = case.get("lam", 1.0), case.get("tau", 1.0)
    st["grad_scale"], st["ce_grad_scale"] = lam * tau * tau / n, (1.0 - lam) / n
    return st


def prepare(case, seed):
    st = _inputs(case, seed)
    T, S = case["tokens"], st["cu"].numel() - 1

    def floats(n):
        return torch.empty(n, dtype=torch.float32, device=DEVICE)

    def ints(n):
        return torch.empty(n, dtype=torch.int32, device=DEVICE)

    op = case["op"]
    if op in ("kd", "kd_topk"):
        grad = torch.empty((T, case["pitch"]), dtype=torch.bfloat16, device=DEVICE)[:, :case["vocab"]]
        st["out"] = dict(grad=grad, kd=floats(T), nll=floats(T), mean_kd=floats(S), mean_nll=floats(S), count=ints(S),
                         status=torch.zeros(1, dtype=torch.int32, device=DEVICE))
        if op == "kd":
            st["out"]["teacher_nll"] = floats(T)
    elif op == "ifd":
        n = st["pairs"][0].numel()
        st["out"] = dict(nll=floats(T), teacher_nll=floats(T), mean=floats(S), teacher_mean=floats(S), count=ints(S),
                         delta=floats(n), zone=torch.empty(n, dtype=torch.uint8, device=DEVICE),
                         keep=torch.empty(n, dtype=torch.uint8, device=DEVICE), keep_count=ints(1))
    elif op == "lag":
        st["out"] = dict(kl=floats(T), mean=floats(S), count=ints(S), batch_mean=floats(1), batch_count=ints(1),
                         exceeded=ints(1))
    else:
        st["out"] = dict(idx=ints((T, case["k"])), val=floats((T, case["k"])))
    return st


def run(st):
    case, o = st["case"], st["out"]
    op, mask = case["op"], st["mask"]
    if op == "kd":
        npd.npd_kd_loss_fwd_bwd(st["s"], mask, teacher_dense=st["t"], labels=st["labels"], tau=case["tau"],
                                grad_scale=st["grad_scale"], ce_grad_scale=st["ce_grad_scale"],
                                divergence=DIVERGENCES[case["divergence"]], skew_alpha=0.1, grad_out=o["grad"],
                                kd_tok=o["kd"], nll_tok=o["nll"], teacher_nll_tok=o["teacher_nll"],
                                dev_status=o["status"])
    elif op == "kd_topk":
        npd.npd_kd_loss_fwd_bwd(st["s"], mask, teacher_idx=st["idx"], teacher_val=st["val"], labels=st["labels"],
                                tau=case["tau"], grad_scale=st["grad_scale"], ce_grad_scale=st["ce_grad_scale"],
                                grad_out=o["grad"], kd_tok=o["kd"], nll_tok=o["nll"], dev_status=o["status"])
    elif op == "ifd":
        npd.npd_kd_loss_fwd_bwd(st["s"], mask, labels=st["labels"], nll_tok=o["nll"])
        npd.npd_kd_loss_fwd_bwd(st["t"], mask, labels=st["labels"], nll_tok=o["teacher_nll"])
        npd.npd_segment_reduce(o["nll"], mask, st["cu"], seg_mean=o["mean"], seg_count=o["count"])
        npd.npd_segment_reduce(o["teacher_nll"], mask, st["cu"], seg_mean=o["teacher_mean"])
        npd.npd_delta_ifd_score(o["mean"], o["teacher_mean"], o["count"], st["pairs"][0], st["pairs"][1], 0.0, 0.8,
                                delta=o["delta"], zone=o["zone"], keep=o["keep"], keep_count=o["keep_count"])
        return o
    elif op == "lag":
        # the generator's logits in the student slot, the learner's in the teacher slot
        npd.npd_kd_loss_fwd_bwd(st["s"], mask, teacher_dense=st["t"], kd_tok=o["kl"])
        binding.npd_policy_lag(o["kl"], mask, st["cu"], 0.10, seg_kl_mean=o["mean"], seg_count=o["count"],
                               batch_kl_mean=o["batch_mean"], batch_count=o["batch_count"],
                               lag_exceeded=o["exceeded"])
        return o
    else:
        npd.npd_teacher_topk(st["t"], case["k"], topk_idx=o["idx"], topk_val=o["val"], loss_mask=mask, log_probs=True)
        return o
    npd.npd_segment_reduce(o["kd"], mask, st["cu"], seg_mean=o["mean_kd"], seg_count=o["count"])
    npd.npd_segment_reduce(o["nll"], mask, st["cu"], seg_mean=o["mean_nll"])
    return o


# ------------------------------------------------------------------------------------------------------ what it costs

def work(case):
    """Logits of scored positions read once (positions that are not scored are not looked at), every gradient row
    written once, the record where there is one.  Operations: per logit of a softmax a multiply-add, an exponential
    and an addition, per logit of a gradient the same again for each softmax in it."""
    T, V = case["tokens"], case["vocab"]
    n = _n_scored(case)
    op = case["op"]
    if op == "kd":
        return {"bytes": n * 6 * V + (T - n) * 2 * V + T * 17, "flops": n * V * 16}
    if op == "kd_topk":
        return {"bytes": n * (4 * V + 8 * case["k"]) + (T - n) * 2 * V + T * 13, "flops": n * V * 8}
    if op == "ifd":
        return {"bytes": n * 4 * V + T * 17, "flops": n * V * 8}
    if op == "lag":
        return {"bytes": n * 4 * V + T * 5, "flops": n * V * 10}
    return {"bytes": n * 2 * V + T * (1 + 8 * case["k"]), "flops": n * V}


def tolerance(case):
    if case["op"] in ("kd", "kd_topk"):
        # the gradient is rounded to bf16 once: half a step is 2^-9 of a value at most, 1.6e-3 in the 2-norm
        return {"rel": 6e-3}
    return {"rel": 1e-5, "max": 1e-3, "differ": 0.0}


# ------------------------------------------------------------------------------------------------------ the same in 64 bits

def _segment_means(x, mask, cu):
    owner = torch.repeat_interleave(torch.arange(cu.numel() - 1, device=DEVICE), (cu[1:] - cu[:-1]).long())
    m = mask.double()
    total = torch.zeros(cu.numel() - 1, dtype=torch.float64, device=DEVICE).index_add_(0, owner, x * m)
    count = torch.zeros_like(total).index_add_(0, owner, m)
    return torch.where(count > 0, total / count.clamp(min=1), 0.0), count.to(torch.int32)


def _softmax64(x, tau):
    l = torch.log_softmax(x / tau, dim=1)
    return l, l.exp()


def _exact_rows(case, st, r0, r1, out):
    """Fills rows [r0, r1) of the per-position outputs (and the gradient) of `out`."""
    op, tau = case["op"], case.get("tau", 1.0)
    m = st["mask"][r0:r1].double()
    y = st["labels"][r0:r1].long().unsqueeze(1)
    s = st["s"][r0:r1].double()
    ls1 = torch.log_softmax(s, dim=1)
    t = None if st["t"] is None else st["t"][r0:r1].double()
    if "nll" in out:
        out["nll"][r0:r1] = -ls1.gather(1, y).squeeze(1) * m
    if "teacher_nll" in out:
        out["teacher_nll"][r0:r1] = -torch.log_softmax(t, dim=1).gather(1, y).squeeze(1) * m
    if op == "ifd":
        return
    ls, ps = _softmax64(s, tau)
    if op == "kd_topk":
        idx = st["idx"][r0:r1].long()
        lt, pt = _softmax64(st["val"][r0:r1].double(), tau)
        d = (pt * (lt - ls.gather(1, idx))).sum(1)
        g = ps.scatter_add(1, idx, -pt)
    else:
        lt, pt = _softmax64(t, tau)
        div, a = case.get("divergence", "forward"), 0.1
        if div == "forward":
            d = (pt * (lt - ls)).sum(1)
            g = ps - pt
        else:
            if div == "reverse":
                e = ps * (ls - lt)
                u = ls - lt + 1.0
            elif div == "skew":
                mix = (a * pt + (1.0 - a) * ps).clamp_(min=1e-300)  # both 0: no term
                e = pt * (lt - mix.log())
                u = (a - 1.0) * pt / mix
            else:
                mix = ((1.0 - a) * pt + a * ps).clamp_(min=1e-300)
                e = ps * (ls - mix.log())
                u = ls - mix.log() + 1.0 - a * ps / mix
            d = e.sum(1)
            g = ps * (u - (ps * u).sum(1, keepdim=True))
    out["kl" if op == "lag" else "kd"][r0:r1] = d * m
    if op == "lag":
        return
    g *= st["grad_scale"] / tau
    if st["ce_grad_scale"]:
        g += st["ce_grad_scale"] * ls1.exp()
        g.scatter_add_(1, y, torch.full_like(y, -st["ce_grad_scale"], dtype=torch.float64))
    out["grad"][r0:r1] = g * m.unsqueeze(1)


def exact(case, seed):
    st = _inputs(case, seed)
    T, V, op = case["tokens"], case["vocab"], case["op"]

    def floats(*shape):
        return torch.zeros(shape, dtype=torch.float64, device=DEVICE)

    if op == "teacher_topk":
        out = dict(idx=torch.empty((T, case["k"]), dtype=torch.int32, device=DEVICE), val=floats(T, case["k"]))
        for r0, r1 in _rows(case):
            # stable: equal logits in order of their ids
            val, idx = torch.sort(st["t"][r0:r1].float(), dim=1, descending=True, stable=True)
            m = st["mask"][r0:r1].unsqueeze(1).bool()
            first = torch.arange(case["k"], device=DEVICE).unsqueeze(0)
            out["idx"][r0:r1] = torch.where(m, idx[:, :case["k"]], first)
            out["val"][r0:r1] = torch.where(m, torch.log_softmax(val[:, :case["k"]].double(), dim=1), 0.0)
        return out
    if op in ("kd", "kd_topk"):
        out = dict(kd=floats(T), nll=floats(T), grad=floats(T, V), status=torch.zeros(1, dtype=torch.int32))
        if op == "kd":
            out["teacher_nll"] = floats(T)
    elif op == "ifd":
        out = dict(nll=floats(T), teacher_nll=floats(T))
    else:
        out = dict(kl=floats(T))
    for r0, r1 in _rows(case):
        _exact_rows(case, st, r0, r1, out)
    mask, cu = st["mask"], st["cu"]
    if op in ("kd", "kd_topk"):
        out["mean_kd"], out["count"] = _segment_means(out["kd"], mask, cu)
        out["mean_nll"] = _segment_means(out["nll"], mask, cu)[0]
    elif op == "ifd":
        out["mean"], out["count"] = _segment_means(out["nll"], mask, cu)
        out["teacher_mean"] = _segment_means(out["teacher_nll"], mask, cu)[0]
        c, u = (p.long() for p in st["pairs"])
        d = out["teacher_mean"][c] / out["teacher_mean"][u] - out["mean"][c] / out["mean"][u]
        keep = ((d >= 0.0) & (d <= 0.8)).to(torch.uint8)
        out.update(delta=d, zone=keep + 2 * (d > 0.8).to(torch.uint8), keep=keep,
                   keep_count=keep.sum(dtype=torch.int32).reshape(1))
    else:
        out["mean"], out["count"] = _segment_means(out["kl"], mask, cu)
        n = mask.sum(dtype=torch.int32)
        mean = out["kl"].sum() / n.clamp(min=1)
        out.update(batch_mean=mean.reshape(1), batch_count=n.reshape(1),
                   exceeded=(mean > 0.10).to(torch.int32).reshape(1))
    return out
