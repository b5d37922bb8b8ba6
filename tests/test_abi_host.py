"""Host-side checks that need no GPU: the C-ABI library loads, exports what include/npd.h declares,
rejects bad arguments before touching HIP, and the synthetic layouts are deterministic."""
import ctypes
import os
import re

import numpy as np
import pytest
import torch

from paper_2605_05940_amd import binding, synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
OK, E_NULL, E_SHAPE, E_VALUE, E_ALIAS, E_UNSUP, E_WS, E_HIP = range(8)


@pytest.fixture(scope="module")
def lib():
    return binding.load()


def test_exports_match_header(lib):
    text = open(os.path.join(ROOT, "include", "npd.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    declared = set(re.findall(r"\b(npd_[a-z_0-9]+)\s*\(", text))
    assert declared == set(binding.EXPORTS)
    for name in declared:
        assert getattr(lib, name) is not None
    assert lib.npd_version() >= 103
    for st in range(8):
        assert len(lib.npd_status_string(st)) > 0
    assert lib.npd_status_string(0) == b"ok"


def test_header_is_plain_c_and_its_layout_is_what_the_binding_assumes(tmp_path):
    """include/npd.h compiles as C99 and as C++ without warnings; struct size and limits as the binding has them."""
    import subprocess
    src = tmp_path / "use_npd.c"
    src.write_text('#include "npd.h"\n'
                   "typedef char desc_is_64_bytes[sizeof(npd_kd_desc) == 64 ? 1 : -1];\n"
                   "typedef char limits[(NPD_MAX_VOCAB == 67108864 && NPD_MAX_TOKENS == 2147483647LL) ? 1 : -1];\n"
                   "int use(void) { return (int)NPD_DIV_SKEW_REVERSE_KL + (int)NPD_ZONE_INVALID + npd_version(); }\n")
    inc = os.path.join(ROOT, "include")
    for cc, std in (("gcc", "-std=c99"), ("g++", "-std=c++11")):
        lang = ["-x", "c++"] if cc == "g++" else []
        subprocess.run([cc, std, "-pedantic", "-Wall", "-Wextra", "-Werror", "-fsyntax-only", "-I", inc, *lang,
                        str(src)], check=True)


def test_desc_layout_matches_header():
    # n_tokens i64, vocab i32, teacher_kind i32, student_stride i64, teacher_stride i64, topk i32, flags u32,
    # tau f32, grad_scale f32, ce_grad_scale f32, divergence i32, skew_alpha f32 (+ tail padding)
    assert ctypes.sizeof(binding.KdDesc) == 64 and binding.KdDesc.ce_grad_scale.offset == 48
    assert binding.KdDesc.divergence.offset == 52 and binding.KdDesc.skew_alpha.offset == 56
    assert binding.KdDesc.student_stride.offset == 16 and binding.KdDesc.tau.offset == 40


FAKE = 0x10000  # a non-null address that is never dereferenced: every call below fails validation first


def _desc(**kw):
    d = binding.KdDesc()
    d.n_tokens, d.vocab, d.teacher_kind = 16, 64, binding.NPD_TEACHER_DENSE_BF16
    d.student_stride = d.teacher_stride = 64
    d.topk, d.flags, d.tau, d.grad_scale, d.ce_grad_scale = 0, 0, 1.0, 1.0, 0.0
    for k, v in kw.items():
        setattr(d, k, v)
    return d


def _kd(lib, d, student=FAKE, teacher=FAKE + 0x100000, idx=None, val=None, labels=None, mask=FAKE + 0x200000,
        grad=FAKE + 0x300000, kd=None, nll=None, tnll=None, lse=None, ws=None, ws_bytes=0):
    return lib.npd_kd_loss_fwd_bwd(ctypes.byref(d), student, teacher, idx, val, labels, mask, grad, kd, nll, tnll, lse,
                                   None, ws, ws_bytes, None)


def test_kd_argument_validation(lib):
    assert lib.npd_kd_loss_fwd_bwd(None, *([None] * 13), 0, None) == E_NULL
    assert _kd(lib, _desc(n_tokens=0)) == E_SHAPE
    assert _kd(lib, _desc(vocab=0)) == E_SHAPE
    assert _kd(lib, _desc(student_stride=63)) == E_SHAPE
    assert _kd(lib, _desc(teacher_stride=10)) == E_SHAPE
    assert _kd(lib, _desc(tau=0.0)) == E_VALUE
    assert _kd(lib, _desc(tau=-1.0)) == E_VALUE
    assert _kd(lib, _desc(tau=float("nan"))) == E_VALUE
    assert _kd(lib, _desc(tau=float("inf"))) == E_VALUE
    assert _kd(lib, _desc(grad_scale=float("nan"))) == E_VALUE
    assert _kd(lib, _desc(teacher_kind=7)) == E_VALUE
    assert _kd(lib, _desc(flags=64)) == E_VALUE
    assert _kd(lib, _desc(flags=3)) == E_VALUE                      # forward-only and in-place together
    assert _kd(lib, _desc(), student=None) == E_NULL
    assert _kd(lib, _desc(), mask=None) == E_NULL
    assert _kd(lib, _desc(), teacher=None) == E_NULL
    assert _kd(lib, _desc(), grad=None) == E_NULL                   # gradient wanted but no buffer
    assert _kd(lib, _desc(flags=1)) == E_VALUE                      # forward-only with a gradient buffer
    assert _kd(lib, _desc(), nll=FAKE + 0x400000) == E_NULL         # NLL without labels
    assert _kd(lib, _desc(ce_grad_scale=0.1)) == E_NULL             # CE gradient without labels
    assert _kd(lib, _desc(ce_grad_scale=float("inf")), labels=FAKE + 0x800000) == E_VALUE
    assert _kd(lib, _desc(ce_grad_scale=0.1, flags=1), labels=FAKE + 0x800000, grad=None) == E_VALUE
    assert _kd(lib, _desc(), grad=FAKE) == E_ALIAS                  # in place without the flag
    assert _kd(lib, _desc(flags=2)) == E_ALIAS                      # flag without aliasing
    assert _kd(lib, _desc(), grad=FAKE + 2) == E_ALIAS              # partial overlap with the student
    assert _kd(lib, _desc(), grad=FAKE + 0x100000 + 64) == E_ALIAS  # overlap with the teacher
    assert _kd(lib, _desc(), grad=FAKE + 0x200000 - 8) == E_ALIAS   # overlap with the mask
    # top-k teacher
    tk = dict(teacher_kind=binding.NPD_TEACHER_TOPK, topk=8)
    assert _kd(lib, _desc(**tk), teacher=None, idx=None, val=FAKE + 0x500000) == E_NULL
    assert _kd(lib, _desc(teacher_kind=1, topk=0), teacher=None, idx=FAKE + 0x500000, val=FAKE + 0x600000) == E_SHAPE
    assert _kd(lib, _desc(teacher_kind=1, topk=65), teacher=None, idx=FAKE + 0x500000, val=FAKE + 0x600000) == E_SHAPE
    assert _kd(lib, _desc(**tk), idx=FAKE + 0x500000, val=FAKE + 0x600000) == E_VALUE   # dense tensor given too
    big = _desc(teacher_kind=1, topk=5000, vocab=8192, student_stride=8192)
    assert _kd(lib, big, teacher=None, idx=FAKE + 0x500000, val=FAKE + 0x600000) == E_UNSUP
    # divergences other than the forward KL
    assert _kd(lib, _desc(divergence=4)) == E_VALUE
    assert _kd(lib, _desc(divergence=-1)) == E_VALUE
    assert _kd(lib, _desc(divergence=binding.NPD_DIV_SKEW_KL, skew_alpha=1.0)) == E_VALUE
    assert _kd(lib, _desc(divergence=binding.NPD_DIV_SKEW_REVERSE_KL, skew_alpha=-0.1)) == E_VALUE
    assert _kd(lib, _desc(divergence=binding.NPD_DIV_SKEW_KL, skew_alpha=float("nan"))) == E_VALUE
    assert _kd(lib, _desc(divergence=binding.NPD_DIV_REVERSE_KL, **tk), teacher=None, idx=FAKE + 0x500000,
               val=FAKE + 0x600000) == E_UNSUP                      # needs the full teacher row
    assert _kd(lib, _desc(divergence=binding.NPD_DIV_REVERSE_KL, skew_alpha=7.0), grad=FAKE) == E_ALIAS  # alpha ignored
    # no teacher: forward-only scoring
    nt = dict(teacher_kind=binding.NPD_TEACHER_NONE)
    assert _kd(lib, _desc(**nt), teacher=None) == E_VALUE           # gradient without a teacher
    assert _kd(lib, _desc(flags=1, **nt), teacher=None, grad=None, kd=FAKE + 0x700000) == E_VALUE
    assert lib.npd_workspace_bytes(ctypes.byref(_desc())) == 0
    # pointers must be multiples of their element size
    assert _kd(lib, _desc(), student=FAKE + 1) == E_VALUE
    assert _kd(lib, _desc(), teacher=FAKE + 0x100001) == E_VALUE
    assert _kd(lib, _desc(), grad=FAKE + 0x300001) == E_VALUE
    assert _kd(lib, _desc(), labels=FAKE + 0x800002, nll=FAKE + 0x400000) == E_VALUE
    assert _kd(lib, _desc(), kd=FAKE + 0x400002) == E_VALUE
    # limits of one call: positions, vocabulary, and strides whose byte extents would not fit 64 bits
    assert _kd(lib, _desc(n_tokens=2**31)) == E_UNSUP
    huge = (1 << 26) + 8
    assert _kd(lib, _desc(vocab=huge, student_stride=huge, teacher_stride=huge)) == E_UNSUP
    assert _kd(lib, _desc(student_stride=2**61)) == E_SHAPE
    assert _kd(lib, _desc(teacher_stride=2**61)) == E_SHAPE


def test_every_output_is_checked_against_every_input_and_output(lib):
    """No output may overlap an input (other than the declared in-place gradient) or another output."""
    L, K = FAKE + 0x800000, FAKE + 0x400000                         # labels, kd_tok: 64 bytes each
    assert _kd(lib, _desc(), kd=FAKE + 64) == E_ALIAS               # kd_tok inside the student logits
    assert _kd(lib, _desc(), kd=FAKE + 0x100000) == E_ALIAS         # ... inside the teacher logits
    assert _kd(lib, _desc(), kd=FAKE + 0x200000 + 12) == E_ALIAS    # ... over the loss mask
    assert _kd(lib, _desc(), labels=L, nll=L + 32) == E_ALIAS       # nll_tok over the labels
    assert _kd(lib, _desc(), labels=L, kd=K, nll=K + 60) == E_ALIAS  # two outputs share four bytes
    assert _kd(lib, _desc(), labels=L, kd=K, tnll=K) == E_ALIAS
    assert _kd(lib, _desc(), lse=FAKE + 0x300000 + 8) == E_ALIAS    # lse_tok inside the gradient
    assert lib.npd_kd_loss_fwd_bwd(ctypes.byref(_desc()), FAKE, FAKE + 0x100000, None, None, None, FAKE + 0x200000,
                                   FAKE + 0x300000, K, None, None, None, K + 4, None, 0, None) == E_ALIAS  # dev_status
    tk = _desc(teacher_kind=binding.NPD_TEACHER_TOPK, topk=8)
    assert _kd(lib, tk, teacher=None, idx=FAKE + 0x600000, val=FAKE + 0x700000, kd=FAKE + 0x600000 + 16) == E_ALIAS
    assert _kd(lib, tk, teacher=None, idx=FAKE + 0x600000, val=FAKE + 0x700000, grad=FAKE + 0x700000 - 64) == E_ALIAS
    # the other entry points
    t, idx, val = FAKE, FAKE + 0x100000, FAKE + 0x200000
    assert lib.npd_teacher_topk(16, 64, 64, 8, 0, t, None, t + 128, val, None) == E_ALIAS
    assert lib.npd_teacher_topk(16, 64, 64, 8, 0, t, None, idx, idx + 256, None) == E_ALIAS
    assert lib.npd_teacher_topk(16, 64, 64, 8, 0, t, idx + 8, idx, val, None) == E_ALIAS   # record over the mask
    v, m, cu, o = FAKE, FAKE + 0x1000, FAKE + 0x2000, FAKE + 0x3000
    assert lib.npd_segment_reduce(8, 2, v, m, cu, v + 16, None, None, None, None, None) == E_ALIAS
    assert lib.npd_segment_reduce(8, 2, v, m, cu, o, o + 4, None, None, None, None) == E_ALIAS
    assert lib.npd_segment_reduce(8, 2, v, m, cu, None, None, None, m, None, None) == E_ALIAS
    ins = [FAKE, FAKE + 0x1000, FAKE + 0x2000, FAKE + 0x3000, FAKE + 0x4000]
    assert lib.npd_delta_ifd_score(2, 4, *ins, 0.0, 1.0, 0, ins[0], None, None, None, None, None, None) == E_ALIAS
    assert lib.npd_delta_ifd_score(2, 4, *ins, 0.0, 1.0, 0, o, o + 4, None, None, None, None, None) == E_ALIAS
    assert lib.npd_delta_ifd_score(2, 4, *ins, 0.0, 1.0, 0, None, None, None, o, o + 1, None, None) == E_ALIAS


def test_workspace_rules(lib):
    """Long rows with a dense teacher and a gradient exchange partial sums through a workspace: its size, what
    happens without it, and the limit of the entry point that brings its own."""
    far = 1 << 44                                                   # fake buffers of several GB each, far apart
    big = dict(n_tokens=64, vocab=151936, student_stride=151936, teacher_stride=151936)
    args = dict(student=far, teacher=2 * far, mask=3 * far, grad=4 * far)
    d = _desc(**big)
    need = lib.npd_workspace_bytes(ctypes.byref(d))
    assert need == 64 * 8 * 32 + 256                                # 8 slices of <= 2,552 groups, 32 bytes each, + tail
    assert lib.npd_workspace_bytes(ctypes.byref(_desc(tau=2.0, **big))) == 64 * 8 * 64 + 256
    assert lib.npd_workspace_bytes(ctypes.byref(_desc(flags=binding.NPD_FLAG_NO_WORKSPACE, **big))) == 0
    assert lib.npd_workspace_bytes(ctypes.byref(_desc(flags=binding.NPD_FLAG_FWD_ONLY, **big))) == 0
    assert lib.npd_workspace_bytes(ctypes.byref(_desc(vocab=20416, n_tokens=64, student_stride=20416,
                                                     teacher_stride=20416))) == 0   # one slice: nothing to exchange
    assert lib.npd_workspace_bytes(ctypes.byref(_desc(vocab=30616, n_tokens=64, student_stride=30616,
                                                     teacher_stride=30616))) == 0   # less than one and a half slices
    assert lib.npd_workspace_bytes(ctypes.byref(_desc(vocab=30624, n_tokens=64, student_stride=30624,
                                                     teacher_stride=30624))) == 64 * 2 * 32 + 256
    assert lib.npd_workspace_bytes(ctypes.byref(_desc(tau=-1.0, **big))) == 0       # invalid descriptor
    assert _kd(lib, d, **args) == E_WS                              # no workspace
    assert _kd(lib, d, ws=5 * far, ws_bytes=need - 1, **args) == E_WS
    assert _kd(lib, d, ws=5 * far + 128, ws_bytes=need, **args) == E_WS             # not 256-byte aligned
    assert _kd(lib, d, ws=4 * far + 256, ws_bytes=need, **args) == E_ALIAS          # inside the gradient
    # the entry point with built-in scratch refuses what its array cannot hold, before any HIP call
    limit = 16 << 20
    assert binding.NOALLOC_WORKSPACE_BYTES == limit
    too_many = limit // (8 * 32) + 1
    dn = _desc(**dict(big, n_tokens=too_many))
    assert lib.npd_workspace_bytes(ctypes.byref(dn)) > limit
    call = lambda desc, **kw: lib.npd_kd_loss_fwd_bwd_noalloc(
        ctypes.byref(desc), kw.get("student", far), 2 * far, None, None, None, 3 * far, 4 * far, None, None, None,
        None, None, None)
    assert call(dn) == E_WS
    assert call(_desc(tau=0.0, **big)) == E_VALUE                   # same argument checks as the main entry point
    assert call(d, student=None) == E_NULL


@pytest.mark.parametrize("name,desc", [
    # no teacher: rows of up to 2,048 groups live in one workgroup's registers, longer ones are faster streamed
    ("kd_solo_kernel", dict(teacher_kind=2, vocab=16384, flags=1)),
    ("kd_cached_kernel", dict(teacher_kind=2, vocab=16392, flags=1)),
    ("kd_cached_kernel", dict(teacher_kind=2, vocab=32768, flags=1, n_tokens=257)),
    ("kd_solo_kernel", dict(teacher_kind=2, vocab=32768, flags=1, n_tokens=256)),
    # forward and reverse KL with a sum at tau = 1: not where 512 threads would be filled badly, unless the CE term
    # leaves no other kernel for whole groups
    ("kd_solo_kernel", dict(vocab=20480, tau=2.0, n_tokens=2048)),
    ("kd_cached_kernel", dict(vocab=20488, tau=2.0, n_tokens=2048)),
    ("kd_solo_kernel", dict(vocab=20488, tau=2.0, n_tokens=2047)),
    ("kd_cached_kernel", dict(vocab=23544, tau=2.0, divergence=1, n_tokens=2048)),
    ("kd_solo_kernel", dict(vocab=23552, tau=2.0, n_tokens=2048)),
    ("kd_cached_kernel", dict(vocab=26616, tau=3.0)), ("kd_solo_kernel", dict(vocab=26624, tau=3.0, divergence=1)),
    ("kd_solo_kernel", dict(vocab=20488, tau=3.0, n_tokens=1023)),
    ("kd_solo_kernel", dict(vocab=20488, tau=2.0, ce_grad_scale=0.5, n_tokens=2048)),
    ("kd_solo_kernel", dict(vocab=20489, tau=3.0)),
    # top-k teacher: short records on long rows, and the forward pass over many rows of a short vocabulary
    ("kd_solo_kernel", dict(teacher_kind=1, topk=32, vocab=20480)),
    ("kd_cached_kernel", dict(teacher_kind=1, topk=32, vocab=20488)),
    ("kd_solo_kernel", dict(teacher_kind=1, topk=33, vocab=20488)),
    ("kd_solo_kernel", dict(teacher_kind=1, topk=32, vocab=20488, tau=2.0)),
    ("kd_cached_kernel", dict(teacher_kind=1, topk=20, vocab=26624)),
    ("kd_solo_kernel", dict(teacher_kind=1, topk=20, vocab=26624, n_tokens=256)),
    ("kd_solo_kernel", dict(teacher_kind=1, topk=20, vocab=26632)),
    ("kd_rows_kernel", dict(teacher_kind=1, topk=64, vocab=2048, n_tokens=11719, flags=1)),
    ("kd_solo_kernel", dict(teacher_kind=1, topk=64, vocab=2048, n_tokens=11718, flags=1)),
    ("kd_solo_kernel", dict(teacher_kind=1, topk=200, vocab=2048, n_tokens=65536, flags=1)),
])
def test_kernel_choice(lib, name, desc):
    d = _desc(**dict(dict(n_tokens=1024), **desc))
    d.student_stride = d.teacher_stride = d.vocab
    assert lib.npd_kd_kernel_name(ctypes.byref(d)).decode() == name


def test_segment_and_ifd_argument_validation(lib):
    assert lib.npd_segment_reduce(-1, 1, *([FAKE] * 8), None) == E_SHAPE
    assert lib.npd_segment_reduce(8, -1, *([FAKE] * 8), None) == E_SHAPE
    assert lib.npd_segment_reduce(8, 2, FAKE, None, FAKE, FAKE, FAKE, FAKE, None, None, None) == E_NULL
    assert lib.npd_segment_reduce(8, 2, FAKE, FAKE, None, FAKE, FAKE, FAKE, None, None, None) == E_NULL
    assert lib.npd_segment_reduce(8, 2, None, FAKE, FAKE, FAKE, FAKE, FAKE, None, None, None) == E_NULL
    assert lib.npd_segment_reduce(8, 2, FAKE + 2, FAKE, FAKE, FAKE, FAKE, FAKE, None, None, None) == E_VALUE
    assert lib.npd_segment_reduce(2**31, 2, *([FAKE] * 8), None) == E_UNSUP
    args = [FAKE] * 5
    outs = [None] * 6
    assert lib.npd_delta_ifd_score(-1, 4, *args, 0.0, 1.0, 0, *outs, None) == E_SHAPE
    assert lib.npd_delta_ifd_score(2, 4, *args, 1.0, 0.5, 0, *outs, None) == E_VALUE
    assert lib.npd_delta_ifd_score(2, 4, *args, float("nan"), 0.5, 0, *outs, None) == E_VALUE
    assert lib.npd_delta_ifd_score(2, 4, *args, 0.0, 1.0, 8, *outs, None) == E_VALUE
    assert lib.npd_delta_ifd_score(2, 4, None, FAKE, FAKE, FAKE, FAKE, 0.0, 1.0, 0, *outs, None) == E_NULL
    assert lib.npd_delta_ifd_score(2, 4, FAKE + 1, FAKE, FAKE, FAKE, FAKE, 0.0, 1.0, 0, *outs, None) == E_VALUE


def test_policy_lag_and_ppl_argument_validation(lib):
    kl, m, cu, o = FAKE, FAKE + 0x1000, FAKE + 0x2000, FAKE + 0x3000
    call = lambda T=8, S=2, kl=kl, m=m, cu=cu, eps=0.1, outs=(None,) * 6: lib.npd_policy_lag(
        T, S, kl, m, cu, ctypes.c_float(eps), *outs, None)
    assert call(T=-1) == E_SHAPE and call(S=-1) == E_SHAPE and call(T=2**31) == E_UNSUP
    assert call(eps=-0.1) == E_VALUE and call(eps=float("nan")) == E_VALUE and call(eps=float("inf")) == E_VALUE
    assert call(kl=None) == E_NULL and call(m=None) == E_NULL and call(cu=None) == E_NULL
    assert call(kl=FAKE + 2) == E_VALUE
    assert call(outs=(kl + 8, None, None, None, None, None)) == E_ALIAS        # seg_kl_mean over kl_tok
    assert call(outs=(None, None, o, o, None, None)) == E_ALIAS                # two scalar outputs on one word
    assert call(outs=(None, None, None, None, m + 4, None)) == E_ALIAS         # lag_exceeded over the mask
    ppl = lambda S=4, a=FAKE, c=FAKE + 0x1000, p=FAKE + 0x2000: lib.npd_segment_ppl(S, a, c, p, None)
    assert ppl(S=-1) == E_SHAPE and ppl(a=None) == E_NULL and ppl(p=None) == E_NULL and ppl(c=FAKE + 0x1002) == E_VALUE
    assert ppl(p=FAKE + 8) == E_ALIAS and ppl(p=FAKE + 0x1000) == E_ALIAS


def test_teacher_topk_argument_validation(lib):
    ok = (16, 64, 64, 8, 0, FAKE, None, FAKE + 0x100000, FAKE + 0x200000, None)
    def call(**kw):
        names = ("T", "V", "stride", "k", "flags", "t", "mask", "idx", "val", "stream")
        args = dict(zip(names, ok))
        args.update(kw)
        return lib.npd_teacher_topk(*[args[n] for n in names])
    assert call(T=0) == E_SHAPE and call(V=0) == E_SHAPE and call(stride=63) == E_SHAPE
    assert call(T=2**31) == E_UNSUP and call(V=(1 << 26) + 8, stride=(1 << 26) + 8) == E_UNSUP
    assert call(stride=2**61) == E_SHAPE
    assert call(t=FAKE + 1) == E_VALUE and call(idx=FAKE + 0x100002) == E_VALUE
    assert call(k=0) == E_SHAPE and call(k=65) == E_SHAPE
    assert call(flags=2) == E_VALUE
    assert call(t=None) == E_NULL and call(idx=None) == E_NULL and call(val=None) == E_NULL
    assert call(V=8192, stride=8192, k=5000) == E_UNSUP


def test_binding_refuses_host_tensors():
    import torch
    with pytest.raises(ValueError):
        binding.npd_kd_loss_fwd_bwd(torch.zeros(4, 8, dtype=torch.bfloat16), torch.ones(4, dtype=torch.uint8))


# --------------------------------------------------------------------------- synthetic layouts

@pytest.mark.parametrize("pitch,off,tau,ce,own", [
    (50048, 0, 1.0, 0.5, False), (50048, 0, 2.0, 0.0, False),   # aligned rows: the buffer the module keeps
    (50048, 0, 2.0, 0.5, True),                                 # a CE term at tau != 1
    (50003, 0, 1.0, 0.0, True), (50048, 3, 1.0, 0.0, True),     # rows that are not 16-byte aligned
])
def test_calls_that_may_overlap_get_scratch_of_their_own(lib, monkeypatch, pitch, off, tau, ce, own):
    """Two calls on two streams share no scratch where such calls once needed none."""
    seen = []

    class Library:
        npd_workspace_bytes = staticmethod(lib.npd_workspace_bytes)

        @staticmethod
        def npd_kd_loss_fwd_bwd(*args):
            seen.append(args[13])
            return 0

    monkeypatch.setattr(binding, "load", lambda: Library)
    monkeypatch.setattr(binding, "_stream", lambda: None)
    monkeypatch.setattr(binding, "_ptr", lambda t, dtype=None: None if t is None else t.data_ptr())
    monkeypatch.setattr(binding, "_array", lambda name, t, n, dtype: None if t is None else t.data_ptr())
    monkeypatch.setattr(binding, "_workspaces", {})
    kept, devices = [], []
    empty = torch.empty

    def record(*a, device, **kw):
        devices.append(device)
        kept.append(empty(*a, **kw))
        return kept[-1]

    monkeypatch.setattr(binding.torch, "empty", record)
    T, V = 4, 50000
    s, t, g = (empty(T * pitch + 64, dtype=torch.bfloat16) for _ in range(3))
    s, t, g = (x[-(x.data_ptr() // 2) % 8 + off:][:T * pitch].view(T, pitch)[:, :V] for x in (s, t, g))
    mask, labels = torch.ones(T, dtype=torch.uint8), torch.zeros(T, dtype=torch.int32)
    for _ in range(2):
        binding.npd_kd_loss_fwd_bwd(s, mask, teacher_dense=t, labels=labels, tau=tau, ce_grad_scale=ce, grad_out=g)
    assert (seen[0] != seen[1]) == own
    assert bool(binding._workspaces) != own
    if own:  # on the device and the stream that run the kernels, whatever device the logits are on
        assert devices == ["cuda", "cuda"]


def _in_a_copy(tmp_path, code, library=None, host=None):
    """Runs `code` with a copy of the package that has the given files as its libraries, and `library` as NPD_LIB_PATH."""
    import shutil
    import subprocess
    import sys
    pkg = tmp_path / "paper_2605_05940_amd"
    pkg.mkdir()
    for name in ("__init__.py", "binding.py", "build.py", "synth.py"):
        shutil.copy(os.path.join(ROOT, "paper_2605_05940_amd", name), pkg)
    (pkg / "libnpd.so").symlink_to(os.path.join(ROOT, "paper_2605_05940_amd", "libnpd.so"))
    if host:
        (pkg / "npd_host.so").write_bytes(host)
    env = {k: v for k, v in os.environ.items() if k != "NPD_LIB_PATH"}
    env.update(PYTHONPATH=str(tmp_path), **({"NPD_LIB_PATH": str(library)} if library else {}))
    r = subprocess.run([sys.executable, "-W", "always", "-c", code], cwd=tmp_path, env=env, capture_output=True, text=True,
                       timeout=300)
    assert r.returncode == 0, r.stderr
    return r.stdout + r.stderr


@pytest.mark.parametrize("host", [None, b"not a library"])
def test_loads_without_the_native_marshalling(tmp_path, host):
    """The Python code makes every call: a warning, no error."""
    out = _in_a_copy(tmp_path, "from paper_2605_05940_amd import binding as b\n"
                     "assert b.load().npd_version() >= 120 and b._host is None\n"
                     "assert b.npd_workspace_bytes(64, 151936) > 0", host=host)
    assert "RuntimeWarning" in out and "npd_host.so" in out


def test_loads_a_library_without_the_newer_entry_points(tmp_path):
    """NPD_LIB_PATH may name one that has no forward scratch and no preferred workspace: its calls are made as before."""
    import subprocess
    old = [n for n in binding.EXPORTS
           if n not in ("npd_forward_scratch_bytes", "npd_kd_loss_forward", "npd_workspace_bytes_preferred")]
    src = tmp_path / "old.c"
    src.write_text("long last_ws;\n" + "".join(f"long {n}() {{ return 0; }}\n" for n in old
                                                if n not in ("npd_kd_loss_fwd_bwd", "npd_workspace_bytes")) +
                   "long npd_workspace_bytes() { return 777; }\n"
                   "long npd_kd_loss_fwd_bwd(void *d, void *a, void *b, void *c, void *e, void *f, void *g, void *h, void *i,"
                   " void *j, void *k, void *l, void *m, void *n, unsigned long bytes) { last_ws = n ? (long)bytes : -1;"
                   " return 0; }\n")
    lib = tmp_path / "libold.so"
    subprocess.run(["gcc", "-shared", "-fPIC", "-w", "-o", str(lib), str(src)], check=True)
    _in_a_copy(tmp_path, """
import ctypes, torch
from paper_2605_05940_amd import binding as b
b._ptr = lambda t, dtype=None: None if t is None else t.data_ptr()
b._array = lambda name, t, n, dtype: None if t is None else t.data_ptr()
b._stream = lambda: None
L = b.load()
assert b._host is None and not hasattr(L, "npd_kd_loss_forward")
s, m = torch.zeros((4, 64), dtype=torch.bfloat16), torch.ones(4, dtype=torch.uint8)
last = ctypes.c_long.in_dll(L, "last_ws")
b.npd_kd_loss_fwd_bwd(s, m, teacher_dense=s, kd_tok=torch.zeros(4))
assert last.value == -1
b.npd_kd_loss_fwd_bwd(s, m, teacher_dense=s, grad_out=s)
assert last.value >= 777
""", library=lib)


def test_native_marshalling_of_a_library_without_kept_records(tmp_path):
    """NPD_LIB_PATH may name one whose calls all clear their record: native code makes them all the same."""
    import subprocess
    src = tmp_path / "old.c"
    src.write_text("".join(f"long {n}() {{ return 0; }}\n" for n in binding.EXPORTS if "kept" not in n))
    lib = tmp_path / "libold.so"
    subprocess.run(["gcc", "-shared", "-fPIC", "-w", "-o", str(lib), str(src)], check=True)
    with open(binding.HOST_PATH, "rb") as f:
        host = f.read()
    out = _in_a_copy(tmp_path, """
import torch
from paper_2605_05940_amd import binding as b
L = b.load()
assert b._host is not None and not hasattr(L, "npd_kd_loss_fwd_bwd_kept")
s = torch.zeros((4, 64), dtype=torch.bfloat16)
assert b._host.kd(s) == -1
good = (b._raw_stream, {}, (1,) * 9 + (0, 0))
b._host.bind(*good)
for bad in ((1,) * 9, (1,) * 8 + (0, 0, 0), (1,) * 9 + (1, 0), (1,) * 9 + (0, 1)):
    try:
        b._host.bind(b._raw_stream, {}, bad)
    except ValueError:
        continue
    raise AssertionError(bad)
""", library=lib, host=host)
    assert "RuntimeWarning" not in out


def test_workspace_that_a_call_prefers(lib):
    """As much as the record of the shorter slices takes where a call has them, else the least."""
    def ask(V, T, **kw):
        d = _desc(vocab=V, n_tokens=T, student_stride=V, teacher_stride=V, **kw)
        return lib.npd_workspace_bytes(ctypes.byref(d)), lib.npd_workspace_bytes_preferred(ctypes.byref(d))

    assert ask(151936, 64) == (64 * 8 * 32 + 256, 64 * 15 * 32 + 256)
    assert ask(151936, 64, tau=2.0) == (64 * 8 * 64 + 256, 64 * 15 * 64 + 256)
    assert ask(36000, 10000, divergence=1) == (10000 * 2 * 32 + 256, 10000 * 3 * 32 + 256)
    assert ask(40960, 64, teacher_kind=1, topk=8) == (64 * 3 * 32 + 256, 64 * 5 * 32 + 256)
    for V, T, kw in ((151936, 32768, {}), (36000, 10000, dict(tau=2.0)), (65536, 64, dict(divergence=2, skew_alpha=0.1)),
                     (151936, 64, dict(flags=4)), (151936, 64, dict(flags=1)), (4096, 64, {}), (151936, 64, dict(tau=-1.0))):
        least, preferred = ask(V, T, **kw)
        assert preferred == least, (V, T, kw)
    # where shorter slices are the faster ones: by how many slices fall to the fullest compute unit, times their length
    for V, T, kw, more in ((32000, 320, {}, True), (32000, 330, {}, True), (32000, 351, {}, False),
                           (32000, 330, dict(tau=2.0), False), (65536, 128, {}, True),
                           (65536, 194, {}, True), (65536, 189, {}, False), (65536, 189, dict(tau=2.0), False), (151936, 88, {}, True),
                           (151936, 89, {}, False), (262144, 53, {}, True), (262144, 54, {}, False), (36000, 351, {}, False), (36000, 420, {}, True),
                           (36000, 512, {}, False), (36000, 640, {}, True), (33600, 512, {}, True),
                           (36000, 470, dict(teacher_kind=1, topk=8), True), (36000, 560, dict(teacher_kind=1, topk=8), False),
                           (36000, 1024, dict(teacher_kind=1, topk=8), True)):
        least, preferred = ask(V, T, **kw)
        assert (preferred > least) == more, (V, T, kw)
    for V in range(30624, 262144, 1499):
        for T in (1, 63, 256, 700, 5000):
            least, preferred = ask(V, T)
            assert 0 < least <= preferred <= 2 * least


def test_kept_workspace_is_replaced_only_where_it_does_not_do(lib, monkeypatch):
    """A buffer of npd_workspace_bytes made before (for a graph's sake, say) stays; a call that prefers more has a block of its
    own, or the kept one where there is no memory."""
    seen, left = [], [True]

    class Library:
        npd_workspace_bytes = staticmethod(lib.npd_workspace_bytes)
        npd_workspace_bytes_preferred = staticmethod(lib.npd_workspace_bytes_preferred)
        npd_kd_loss_fwd_bwd = staticmethod(lambda *args: seen.append((args[13], args[14])) or 0)

    monkeypatch.setattr(binding, "load", lambda: Library)
    monkeypatch.setattr(binding, "_stream", lambda: None)
    monkeypatch.setattr(binding, "_ptr", lambda t, dtype=None: None if t is None else t.data_ptr())
    monkeypatch.setattr(binding, "_array", lambda name, t, n, dtype: None if t is None else t.data_ptr())
    monkeypatch.setattr(binding, "_workspaces", {})
    empty = torch.empty

    def allocate(n, dtype, device):
        if device == "cuda" and not left[0]:
            raise torch.cuda.OutOfMemoryError("no memory")
        return empty(n, dtype=dtype)

    monkeypatch.setattr(binding.torch, "empty", allocate)
    T, V = 10000, 36000
    s = empty(1, dtype=torch.bfloat16).expand(T, V)
    monkeypatch.setattr(binding, "_row_stride", lambda x: V)
    d = _desc(vocab=V, n_tokens=T, student_stride=V, teacher_stride=V)
    need = lib.npd_workspace_bytes(ctypes.byref(d))
    want = lib.npd_workspace_bytes_preferred(ctypes.byref(d))
    kept = binding.workspace_for(need, "cpu")
    assert need <= kept.numel() < want
    call = lambda **kw: binding.npd_kd_loss_fwd_bwd(s, torch.ones(T, dtype=torch.uint8), teacher_dense=s, grad_out=s, **kw)
    call()
    assert seen[-1][1] == want and binding._workspaces[0] is kept
    left[0] = False
    call()
    assert seen[-1] == (kept.data_ptr(), need) and binding._workspaces[0] is kept
    call(tau=2.0)                                           # the wider record: twice the least of before
    assert seen[-1][1] > need and binding._workspaces[0] is not kept
    binding._workspaces.clear()
    kept = binding.workspace_for(1, "cpu")                  # of the smallest size: enough for every call of few rows
    for T in range(1, 280, 31):
        s = empty(1, dtype=torch.bfloat16).expand(T, V)
        call = lambda **kw: binding.npd_kd_loss_fwd_bwd(s, torch.ones(T, dtype=torch.uint8), teacher_dense=s, grad_out=s, **kw)
        call(tau=2.0)
        assert seen[-1][0] == kept.data_ptr()


def test_forward_only_calls_run_without_memory_for_their_scratch(monkeypatch):
    """The scratch of a forward-only call is optional: where it cannot be allocated, the call is made without."""
    calls = []

    class Library:
        npd_forward_scratch_bytes = staticmethod(lambda desc: 4096)
        npd_kd_loss_forward = staticmethod(lambda *args: calls.append(("split", args[12], args[13])) or 0)
        npd_kd_loss_fwd_bwd = staticmethod(lambda *args: calls.append(("whole", args[13], args[14])) or 0)

    def none_left(n, device, **kw):
        raise torch.cuda.OutOfMemoryError("no memory")

    monkeypatch.setattr(binding, "load", lambda: Library)
    monkeypatch.setattr(binding, "_stream", lambda: None)
    monkeypatch.setattr(binding, "_ptr", lambda t, dtype=None: None if t is None else t.data_ptr())
    monkeypatch.setattr(binding, "_array", lambda name, t, n, dtype: None if t is None else t.data_ptr())
    s, mask, kd = torch.zeros((4, 64), dtype=torch.bfloat16), torch.ones(4, dtype=torch.uint8), torch.zeros(4)
    empty = torch.empty
    monkeypatch.setattr(binding.torch, "empty", none_left)
    binding.npd_kd_loss_fwd_bwd(s, mask, teacher_dense=s, kd_tok=kd)
    assert calls == [("whole", None, 0)]
    monkeypatch.setattr(binding.torch, "empty", lambda n, dtype, device: empty(n, dtype=dtype))
    binding.npd_kd_loss_fwd_bwd(s, mask, teacher_dense=s, kd_tok=kd)
    assert calls[1][0] == "split" and calls[1][1] and calls[1][2] == 4096


def test_layouts_are_deterministic_and_well_formed():
    for i in range(5):
        w = synth.config(i)
        a, b = synth.make_layout(w), synth.make_layout(w)
        for f in ("cu_seqlens", "loss_mask", "labels", "is_pad_segment", "pair_cond", "pair_uncond"):
            np.testing.assert_array_equal(getattr(a, f), getattr(b, f))
        cu = a.cu_seqlens
        assert cu[0] == 0 and cu[-1] == w.n_tokens and (np.diff(cu) >= 0).all()
        assert a.loss_mask.shape == (w.n_tokens,) and a.labels.min() >= 0 and a.labels.max() < w.vocab
        # no sample straddles a row boundary; pad segments are fully masked
        for s in range(a.n_segments):
            if cu[s + 1] > cu[s]:
                assert cu[s] // w.row_len == (cu[s + 1] - 1) // w.row_len
            if a.is_pad_segment[s]:
                assert a.loss_mask[cu[s]:cu[s + 1]].sum() == 0


def test_config0_and_paired_layout_details():
    lay = synth.make_layout(synth.config(0))
    assert lay.cu_seqlens.tolist() == [0, 37, 101, 191, 312, 512]
    # floor(25 %) of each sample is prompt
    assert [int(lay.loss_mask[a:b].sum()) for a, b in zip(lay.cu_seqlens[:-1], lay.cu_seqlens[1:])] == [28, 48, 68, 91, 0]
    w3 = synth.config(3)
    lay3 = synth.make_layout(w3)
    assert len(lay3.pair_cond) == len(lay3.pair_uncond) >= 4
    cu = lay3.cu_seqlens
    for pc, pu in zip(lay3.pair_cond, lay3.pair_uncond):
        n = cu[pu + 1] - cu[pu]
        q = cu[pc + 1] - cu[pc] - n
        assert w3.prefix_lo <= q <= w3.prefix_hi and w3.length_lo <= n <= w3.length_hi
        assert lay3.loss_mask[cu[pc]:cu[pc] + q].sum() == 0 and lay3.loss_mask[cu[pc] + q:cu[pc + 1]].all()
        assert lay3.loss_mask[cu[pu]:cu[pu + 1]].all()
        np.testing.assert_array_equal(lay3.labels[cu[pc] + q:cu[pc + 1]], lay3.labels[cu[pu]:cu[pu + 1]])


def test_cpu_logit_generation_is_reproducible():
    import torch
    w = synth.scaled(synth.config(1), n_rows=1, row_len=300, vocab=520)
    s1 = torch.empty((300, 520), dtype=torch.bfloat16)
    t1 = torch.empty_like(s1)
    s2, t2 = torch.empty_like(s1), torch.empty_like(s1)
    synth.fill_logits(w, s1, t1)
    synth.fill_logits(w, s2, t2)
    assert torch.equal(s1, s2) and torch.equal(t1, t2)
    assert 2.5 < s1.float().std().item() < 3.5
    w2 = synth.scaled(synth.config(2), n_rows=1, row_len=300, vocab=520, topk=16)
    idx, val = synth.make_topk_teacher(w2, s1)
    assert idx.shape == (300, 16) and all(len(set(r.tolist())) == 16 for r in idx)
    assert idx.min() >= 0 and idx.max() < 520
    assert torch.allclose(val.double().exp().sum(1), torch.ones(300, dtype=torch.float64), atol=1e-6)


def test_bench_refuses_more_than_one_gpu():
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                       timeout=300)
    assert r.returncode == 2 and "one GPU" in r.stderr and r.stdout.strip() == ""


def test_forward_scratch(lib):
    """Scratch of the forward-only entry point: which calls ask for it, and the argument checks it shares."""
    F = binding.NPD_FLAG_FWD_ONLY
    big = dict(vocab=151936, n_tokens=64, student_stride=151936, teacher_stride=151936, flags=F)
    ask = lambda **kw: lib.npd_forward_scratch_bytes(ctypes.byref(_desc(**{**big, **kw})))
    assert ask() == 64 * 19 * 6 * 4 and ask(tau=2.0) == 64 * 19 * 12 * 4          # slices of 1,024 groups of 8 logits
    assert ask(n_tokens=1000) == 1000 * 10 * 6 * 4                                # of 2,048
    assert ask(teacher_kind=binding.NPD_TEACHER_NONE) == 64 * 10 * 3 * 4
    assert ask(flags=0) == ask(flags=F | binding.NPD_FLAG_NO_WORKSPACE) == 0
    assert ask(teacher_stride=151937) == 0                                        # rows that drift apart: element by element
    assert ask(divergence=1) == ask(vocab=32768) == ask(tau=-1.0) == 0
    assert ask(teacher_kind=binding.NPD_TEACHER_TOPK, topk=8) == 0
    # the lines of the rule: rows per compute unit, and rows whose kernel with a workgroup per row is as fast
    none = binding.NPD_TEACHER_NONE
    for V, T, kind, tau, split in ((50304, 128, 0, 1.0, True), (50304, 129, 0, 1.0, False), (50304, 256, 0, 1.0, False),
                                   (131072, 129, 0, 1.0, True), (50304, 432, 0, 1.0, True), (50304, 433, 0, 1.0, False),
                                   (50304, 512, 0, 1.0, False), (50304, 513, 0, 1.0, True), (50304, 512, 0, 2.0, True),
                                   (100352, 512, 0, 1.0, True), (70000, 51, none, 1.0, True), (70000, 52, none, 1.0, False),
                                   (90000, 64, none, 1.0, True), (90000, 65, none, 1.0, False), (100352, 104, none, 1.0, True),
                                   (100352, 105, none, 1.0, False), (116000, 128, none, 1.0, True),
                                   (116000, 129, none, 1.0, False), (240000, 128, none, 1.0, True),
                                   (240000, 256, none, 1.0, False), (240000, 300, none, 1.0, True),
                                   (240000, 449, none, 1.0, False), (240000, 1025, none, 1.0, True),
                                   (262144, 256, none, 1.0, True)):
        d = dict(vocab=V, n_tokens=T, student_stride=V, teacher_stride=V, teacher_kind=kind, tau=tau)
        assert (ask(**d) > 0) == split, (V, T, kind, tau)

    def forward(d, kd=FAKE + 0x10000000, student=FAKE):
        return lib.npd_kd_loss_forward(ctypes.byref(d), student, FAKE + 0x4000000, None, None, None, FAKE + 0x8000000, kd,
                                       None, None, None, None, None, 0, None)

    assert forward(_desc(**{**big, "flags": 0})) == E_NULL                        # a gradient call has no gradient here
    assert forward(_desc(**{**big, "tau": 0.0})) == E_VALUE
    assert forward(_desc(**big), student=None) == E_NULL
    assert forward(_desc(**big), kd=FAKE + 2) == E_VALUE
    assert forward(_desc(**big), kd=FAKE + 16) == E_ALIAS
