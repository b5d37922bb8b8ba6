"""The binding's native marshalling against its Python code: the same outputs, the same refusals."""
import pytest
import torch

from paper_2605_05940_amd import binding
from gpu_util import dev

CALLS = ("kd", "kd_bad_aligned", "kd_ce_tau2", "kd_inplace", "kd_workspace", "kd_no_workspace", "kd_kept_too_small", "kd_topk",
         "forward", "forward_split", "forward_alone", "segments", "segments_no_values", "lag", "ifd", "ifd_all", "topk")


def _call(name, T=24, V=65536):
    """Runs one call on fresh outputs; returns them."""
    g = torch.Generator(device=dev()).manual_seed(5)
    f = lambda *n: torch.full(n, -7.0, device=dev())
    i = lambda *n: torch.full(n, -7, dtype=torch.int32, device=dev())
    pitch = V + 3 if name == "kd_bad_aligned" else V
    V = 2048 if name == "forward" else V
    s, t = (torch.randn((T, pitch), generator=g, device=dev()).mul_(3).to(torch.bfloat16)[:, :V] for _ in range(2))
    mask = (torch.rand(T, generator=g, device=dev()) < 0.8).to(torch.uint8)
    lab = torch.randint(0, V, (T,), generator=g, device=dev(), dtype=torch.int32)
    cu = torch.tensor([0, 5, 9, T], dtype=torch.int32, device=dev())
    if name in ("kd_inplace", "kd_workspace", "kd_no_workspace", "kd_kept_too_small"):
        n = 2 * binding.npd_workspace_bytes(T, V)
        out = dict(grad_out=s if name == "kd_inplace" else torch.zeros_like(s), kd_tok=f(T))
        ws = torch.empty(n, dtype=torch.uint8, device=dev()) if name == "kd_workspace" else None
        if name == "kd_kept_too_small":                    # (enough for the call, less than it prefers: a block of its own)
            binding._workspaces[0] = torch.empty(n // 2, dtype=torch.uint8, device=dev())
        binding.npd_kd_loss_fwd_bwd(s, mask, teacher_dense=t, skew_alpha=0.5, workspace=ws,
                                    no_workspace=name == "kd_no_workspace", **out)
    elif name in ("kd", "kd_bad_aligned", "kd_ce_tau2"):
        out = dict(grad_out=torch.zeros((T, pitch), dtype=torch.bfloat16, device=dev())[:, :V], kd_tok=f(T), nll_tok=f(T),
                   teacher_nll_tok=f(T), lse_tok=f(T), dev_status=torch.zeros(1, dtype=torch.int32, device=dev()))
        ce = dict(tau=2.0, ce_grad_scale=0.25) if name == "kd_ce_tau2" else dict(divergence=1)
        binding.npd_kd_loss_fwd_bwd(s, mask, teacher_dense=t, labels=lab, grad_scale=0.5, **ce, **out)
    elif name == "kd_topk":
        val, idx = torch.topk(t.float(), 9, dim=1)
        out = dict(grad_out=torch.zeros_like(s), kd_tok=f(T))
        binding.npd_kd_loss_fwd_bwd(s, mask, teacher_idx=idx.to(torch.int32).contiguous(), teacher_val=val.contiguous(), **out)
    elif name in ("forward", "forward_split"):
        out = dict(kd_tok=f(T), nll_tok=f(T))
        binding.npd_kd_loss_fwd_bwd(s, mask, teacher_dense=t, labels=lab, **out)
    elif name == "forward_alone":
        out = dict(nll_tok=f(T), lse_tok=f(T))
        binding.npd_kd_loss_fwd_bwd(s, mask, labels=lab, **out)
    elif name == "segments_no_values":
        out = dict(seg_count=i(3), dev_status=torch.zeros(1, dtype=torch.int32, device=dev()))
        binding.npd_segment_reduce(None, mask, cu, **out)
    elif name == "segments":
        out = dict(seg_sum=f(3), seg_count=i(3), seg_mean=f(3), token_to_sample=i(T))
        binding.npd_segment_reduce(s[:, 0].float(), mask, cu, **out)
    elif name == "lag":
        out = dict(seg_kl_mean=f(3), seg_count=i(3), batch_kl_mean=f(1), batch_count=i(1), lag_exceeded=i(1))
        binding.npd_policy_lag(s[:, 0].float().abs(), mask, cu, 0.2, **out)
    elif name == "ifd":
        out = dict(delta=f(2), keep=torch.zeros(2, dtype=torch.uint8, device=dev()), keep_count=i(1))
        ones = torch.tensor([1.0, 2.0, 1.5], device=dev())
        binding.npd_delta_ifd_score(ones, ones * 1.5, cu[1:], cu[:2] * 0, cu[:2] * 0 + 1, 0.0, 0.8, **out)
    elif name == "ifd_all":
        out = dict(ifd_student=f(2), ifd_teacher=f(2), delta=f(2), zone=torch.zeros(2, dtype=torch.uint8, device=dev()))
        ones = torch.tensor([1.0, 2.0, 1.5], device=dev())
        binding.npd_delta_ifd_score(ones, ones * 1.5, cu[1:], cu[:2] * 0, cu[:2] * 0 + 1, -1.0, 0.8, flags=1, **out)
    else:
        out = dict(topk_idx=i(T, 7), topk_val=f(T, 7))
        binding.npd_teacher_topk(t, 7, loss_mask=mask, log_probs=False, **out)
    torch.cuda.synchronize()
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("name", CALLS)
def test_the_same_results_as_from_python(name, monkeypatch):
    binding.load()
    assert binding._host is not None
    seen = []
    functions = {k: getattr(binding._host, k) for k in ("kd", "segment_reduce", "delta_ifd", "teacher_topk", "policy_lag")}

    class Watched:
        pass

    def watch(f):
        def g(*a):
            seen.append(f(*a))
            return seen[-1]
        return staticmethod(g)

    for k, f in functions.items():
        setattr(Watched, k, watch(f))
    monkeypatch.setattr(binding, "_host", Watched)
    binding.workspace_for(1 << 20, dev())                  # (the kept buffer: made by Python code)
    got = _call(name)
    assert seen == [0]                                     # it was not left to the Python code
    monkeypatch.setattr(binding, "_host", None)
    want = _call(name)
    for k in want:
        assert torch.equal(got[k], want[k]), k


@pytest.mark.gpu
def test_the_same_refusals():
    T, V = 8, 1024
    s, t, g = (torch.zeros((T, V), dtype=torch.bfloat16, device=dev()) for _ in range(3))
    mask, kd = torch.ones(T, dtype=torch.uint8, device=dev()), torch.zeros(T, device=dev())
    binding.load()
    call = binding.npd_kd_loss_fwd_bwd
    for error, args, kw in (
            (ValueError, (s.float(), mask), dict(teacher_dense=t, grad_out=g)),
            (ValueError, (s, mask), dict(teacher_dense=t[:, :512], grad_out=g)),
            (ValueError, (s, mask), dict(teacher_dense=t, grad_out=g, kd_tok=kd[:4])),
            (ValueError, (s, mask), dict(teacher_dense=t, grad_out=g, kd_tok=kd.cpu())),
            (ValueError, (s.t(), mask), dict(teacher_dense=t, grad_out=g)),
            (binding.NpdError, (s, mask), dict(teacher_dense=t, grad_out=t)),
            (binding.NpdError, (s, mask), dict(teacher_dense=t, grad_out=g, tau=0.0)),
            (binding.NpdError, (s, mask), dict(teacher_dense=t, teacher_idx=mask.int().view(T, 1), teacher_val=kd.view(T, 1),
                                               grad_out=g)),
            (TypeError, (s, mask), dict(teacher_dense=t, grad_out=g, tau="1"))):
        with pytest.raises(error):
            call(*args, **kw)
    call(s, mask, teacher_dense=t, grad_out=g, kd_tok=kd, tau=torch.tensor(2.0))   # a number is a number
    with pytest.raises(ValueError):
        binding.npd_segment_reduce(kd[:4], mask, mask.int()[:2])
    with pytest.raises(ValueError):
        binding.npd_teacher_topk(t, 3, topk_idx=mask.int().view(T, 1), topk_val=kd.view(T, 1))


def test_leaves_tensors_on_the_cpu_to_python():
    binding.load()
    s, mask = torch.zeros((4, 64), dtype=torch.bfloat16), torch.ones(4, dtype=torch.uint8)
    none = [None] * 2
    assert binding._host.kd(s, mask, s, *none, None, 1.0, 1.0, 0.0, 0, 0.0, s, None, None, None, None, None, None, False) == -1
    assert binding._host.kd(s) == -1 and binding._host.segment_reduce(1, 2, 3, 4, 5, 6, 7, 8) == -1
    assert binding._host.teacher_topk(s, 2, s, s, None, True) == -1
