"""Gradient calls whose scratch record is kept and not cleared: its words carry a number that each launch takes anew.  Whatever
an earlier call left in the record, the results are those of a call on a workspace of its own, bit by bit."""
import ctypes

import pytest
import torch

from gpu_util import dev
from paper_2605_05940_amd import binding

pytestmark = pytest.mark.gpu

CASES = {  # rows, vocabulary, what: records of 8 and 16 words per slice, of 2 .. 8 slices per row, a second exchange
    "few": (24, 40960, dict()), "few_tau2": (24, 40960, dict(tau=2.0, ce_grad_scale=0.25)), "reverse": (300, 50304, dict(divergence=1)),
    "odd": (40, 50003, dict(ce_grad_scale=0.25)), "skew": (40, 36000, dict(divergence=2, skew_alpha=0.1)),
    "skew_tau3": (40, 36000, dict(divergence=3, skew_alpha=0.1, tau=3.0)), "topk": (24, 65536, "topk"), "long": (500, 65536, dict()),
}


def _inputs(name):
    T, V, kw = CASES[name]
    g = torch.Generator(device=dev()).manual_seed(T + V)
    s = (3.0 * torch.randn((T, V), generator=g, device=dev())).to(torch.bfloat16)
    t = (0.8 * s.float() + 1.5 * torch.randn((T, V), generator=g, device=dev())).to(torch.bfloat16)
    mask = (torch.rand(T, generator=g, device=dev()) < 0.8).to(torch.uint8)
    lab = torch.randint(0, V, (T,), generator=g, device=dev(), dtype=torch.int32)
    if kw == "topk":
        val, idx = torch.topk(t.float(), 24, dim=1)
        kw = dict(teacher_idx=idx.to(torch.int32).contiguous(), teacher_val=val.contiguous())
    else:
        kw = dict(kw, teacher_dense=t)
    return s, mask, dict(kw, labels=lab)


def _out(s):
    return (torch.full_like(s, float("nan")), torch.full((s.shape[0],), -1.0, device=dev()),
            torch.full((s.shape[0],), -1.0, device=dev()), torch.zeros(1, dtype=torch.int32, device=dev()))


def _call(s, mask, kw, out, workspace=None):
    binding.npd_kd_loss_fwd_bwd(s, mask, grad_out=out[0], kd_tok=out[1], nll_tok=out[2], dev_status=out[3], workspace=workspace, **kw)


def _same(got, want):
    return all(torch.equal(a.view(torch.uint8), b.view(torch.uint8)) for a, b in zip(got, want))


@pytest.fixture(scope="module")
def reference():
    """Inputs, and the results on a workspace that the call clears."""
    all_of = {}
    for name in CASES:
        s, mask, kw = _inputs(name)
        want = _out(s)
        _call(s, mask, kw, want, torch.full((8 << 20,), 0xab, dtype=torch.uint8, device=dev()))
        all_of[name] = s, mask, kw, want
    torch.cuda.synchronize()
    return all_of


@pytest.fixture
def fresh():
    binding.load()
    assert binding._host is not None
    torch.cuda.synchronize()
    host = binding._host                                   # (a test may replace it)
    host.release()
    yield
    torch.cuda.synchronize()
    host.release()


def test_calls_of_all_kinds_on_one_record(reference, fresh):
    order = list(CASES) + list(CASES)[::-1] + ["few", "long", "few", "skew", "few_tau2", "topk"] * 3
    for name in order:
        s, mask, kw, want = reference[name]
        got = _out(s)
        print(f"[kept] {name}", flush=True)
        _call(s, mask, kw, got)
        torch.cuda.synchronize()
        assert _same(got, want), name
    base = torch.cuda.memory_allocated()
    binding.release_records()                              # the record goes back
    assert torch.cuda.memory_allocated() < base


def test_streams_share_no_record(reference, fresh):
    streams = [torch.cuda.Stream() for _ in range(11)]      # more than have a record at a time
    names = ["odd", "few_tau2", "reverse", "few", "topk", "skew"]
    torch.cuda.synchronize()
    got = []
    for i, st in enumerate(streams):
        with torch.cuda.stream(st):
            for name in names:
                s, mask, kw, _ = reference[name]
                got.append((name, _out(s)))
                _call(s, mask, kw, got[-1][1])
    torch.cuda.synchronize()
    for name, out in got:
        assert _same(out, reference[name][3]), name


def _under_fake_tensors(f):
    from torch._subclasses.fake_tensor import FakeTensorMode
    with FakeTensorMode(allow_non_fake_inputs=True):
        f()


def _under_grad(f):
    def g(x):
        f()
        return x.sum()
    torch.func.grad(g)(torch.ones(3, device=dev()))


def _under_vmap(f):
    def g(x):
        f()
        return x + 1.0
    torch.func.vmap(g)(torch.ones(3, device=dev()))


@pytest.mark.parametrize("under", [_under_fake_tensors, _under_grad, _under_vmap])
def test_scratch_is_memory_whatever_mode_is_on(reference, fresh, monkeypatch, under):
    """Tensors made under such a mode have none; a record made there would stand in the way of all later calls."""
    s, mask, kw, want = reference["few"]
    x = torch.randn((513, 100352), generator=torch.Generator(device=dev()).manual_seed(3), device=dev()).to(torch.bfloat16)
    ones, status = torch.ones(513, dtype=torch.uint8, device=dev()), []
    first, second = (torch.full((513,), -1.0, device=dev()) for _ in range(2))
    host = binding._host

    class Watched:
        @staticmethod
        def kd(*a):
            status.append(host.kd(*a))
            return status[-1]

    monkeypatch.setattr(binding, "_host", Watched)
    got = _out(s)
    under(lambda: _call(s, mask, kw, got))
    under(lambda: binding.npd_kd_loss_fwd_bwd(x, ones, lse_tok=first))     # (two launches, a block of its own)
    torch.cuda.synchronize()
    assert _same(got, want)
    got = _out(s)
    _call(s, mask, kw, got)
    binding.npd_kd_loss_fwd_bwd(x, ones, lse_tok=second)
    torch.cuda.synchronize()
    assert _same(got, want) and _same([first], [second]) and status == [0] * 4


class _Watched:
    """The native marshalling with entry points that note the scratch they are given (`seen`: entry point, address, bytes,
    stream) and launch nothing."""

    def __init__(self, lib, host):
        kd = ctypes.CFUNCTYPE(ctypes.c_int, *[ctypes.c_void_p] * 14, ctypes.c_size_t, ctypes.c_void_p)
        self.seen = []
        self.calls = tuple(kd(lambda *a, name=name: self.seen.append((name, a[13], a[14], a[15])) or 0)
                           for name in ("cleared", "kept"))
        real = (lib.npd_workspace_bytes, lib.npd_workspace_bytes_preferred, lib.npd_forward_scratch_bytes, lib.npd_kd_loss_fwd_bwd,
                lib.npd_kd_loss_forward, lib.npd_segment_reduce, lib.npd_delta_ifd_score, lib.npd_teacher_topk, lib.npd_policy_lag,
                lib.npd_kept_workspace_bytes, lib.npd_kd_loss_fwd_bwd_kept)
        self.host = host
        self.real = tuple(ctypes.cast(f, ctypes.c_void_p).value for f in real)

    def __enter__(self):
        to = list(self.real)
        to[3], to[10] = (ctypes.cast(f, ctypes.c_void_p).value for f in self.calls)
        self.host.bind(binding._raw_stream, binding._workspaces, tuple(to))
        return self

    def __exit__(self, *_):
        self.host.bind(binding._raw_stream, binding._workspaces, self.real)


def test_no_stream_uses_the_scratch_of_another(fresh):
    """Calls that once took the buffer kept per device too: with a record, with none to be had (more bytes than one may have),
    beside a graph that holds that buffer."""
    streams = [torch.cuda.Stream() for _ in range(11)]
    buffer = binding.workspace_for(64 << 20, dev())
    s = torch.empty((24, 40960), dtype=torch.bfloat16, device=dev())
    wide = torch.empty((140000, 32000), dtype=torch.bfloat16, device=dev())   # 2 x 140,000 slices of 16 words of 64 bits: 36 MB
    with _Watched(binding.load(), binding._host) as w:
        for x, kw in ((s, dict()), (s, dict(divergence=1)), (wide, dict(tau=2.0))):
            mask, out = torch.ones(x.shape[0], dtype=torch.uint8, device=dev()), torch.empty(x.shape[0], device=dev())
            del w.seen[:]
            for st in streams:
                with torch.cuda.stream(st):
                    binding.npd_kd_loss_fwd_bwd(x, mask, teacher_dense=x, grad_out=x, kd_tok=out, **kw)
            assert [st.cuda_stream for st in streams] == [call[3] for call in w.seen]
            ranges = sorted((at, at + n) for _, at, n, _ in w.seen) + [(1 << 63, 0)]
            assert all(a[1] <= b[0] for a, b in zip(ranges, ranges[1:])), [call[0] for call in w.seen]
            assert all(e <= buffer.data_ptr() or b >= buffer.data_ptr() + buffer.numel() for b, e in ranges[:-1])
        assert {call[0] for call in w.seen} == {"cleared"}


def test_streams_that_come_later_have_a_record_too(fresh):
    """Of the stream that has been idle longest; no more than eight are held."""
    s = torch.empty((24, 40960), dtype=torch.bfloat16, device=dev())
    mask, out = torch.ones(24, dtype=torch.uint8, device=dev()), torch.empty(24, device=dev())
    streams = [torch.cuda.Stream() for _ in range(20)]
    base = torch.cuda.memory_allocated()
    with _Watched(binding.load(), binding._host) as w:
        def call(st):
            with torch.cuda.stream(st):
                binding.npd_kd_loss_fwd_bwd(s, mask, teacher_dense=s, grad_out=s, kd_tok=out)
            return w.seen[-1][:2]

        at = {st: call(st) for st in streams[:8]}
        assert call(streams[0]) == at[streams[0]]           # (used: the second is the one that is idle longest)
        for st in streams[8:]:
            assert call(st)[0] == "kept"
            assert call(streams[0]) == at[streams[0]]
        assert {name for name, _ in at.values()} == {"kept"}
        held = torch.cuda.memory_allocated() - base
        assert held == 8 * ((1 << 18) + 512)                # (the least that a record has)
    binding.release_records()
    assert torch.cuda.memory_allocated() == base


def test_sizes_of_records(fresh):
    """Batches that get longer by little share one; the longest is of 2^22 words, and the 64 behind them do not count."""
    x = torch.empty((131073, 32000), dtype=torch.bfloat16, device=dev())
    mask, out = torch.ones(131073, dtype=torch.uint8, device=dev()), torch.empty(131073, device=dev())
    with _Watched(binding.load(), binding._host) as w:
        for T in list(range(1000, 1500, 50)) + [131072, 131073]:     # two slices of 16 words each
            binding.npd_kd_loss_fwd_bwd(x[:T], mask[:T], teacher_dense=x[:T], grad_out=x[:T], kd_tok=out[:T], tau=2.0)
        assert len({(at, n) for _, at, n, _ in w.seen[:10]}) <= 2
        assert [name for name, *_ in w.seen] == ["kept"] * 11 + ["cleared"]
        assert w.seen[10][2] == 2 * 4 * ((1 << 22) + 64)


def test_another_library_finds_no_record_of_the_last_one(fresh):
    """Each library counts its own calls: a record that stayed would hold words with the numbers of the next one's calls."""
    lib, host = binding.load(), binding._host
    s = torch.empty((24, 40960), dtype=torch.bfloat16, device=dev())
    t, mask, out = torch.empty_like(s), torch.ones(24, dtype=torch.uint8, device=dev()), torch.empty(24, device=dev())
    base = torch.cuda.memory_allocated()
    with _Watched(lib, host) as w:
        binding.npd_kd_loss_fwd_bwd(s, mask, teacher_dense=t, grad_out=s, kd_tok=out)
        assert w.seen[0][0] == "kept" and torch.cuda.memory_allocated() > base
    assert torch.cuda.memory_allocated() == base


def test_a_library_without_kept_records(reference, fresh):
    """The native marshalling makes its calls on workspaces that they clear."""
    w = _Watched(binding.load(), binding._host)
    binding.workspace_for(1 << 20, dev())
    binding._host.bind(binding._raw_stream, binding._workspaces, w.real[:9] + (0, 0))
    try:
        base = torch.cuda.memory_allocated()
        for name in CASES:
            s, mask, kw, want = reference[name]
            got = _out(s)
            _call(s, mask, kw, got)
            torch.cuda.synchronize()
            assert _same(got, want), name
        s, mask, kw, _ = reference["topk"]
        nll = torch.empty(s.shape[0], device=dev())
        binding.npd_kd_loss_fwd_bwd(s, mask, labels=kw["labels"], nll_tok=nll)
        del got, nll
        assert torch.cuda.memory_allocated() == base        # (no record)
    finally:
        binding._host.bind(binding._raw_stream, binding._workspaces, w.real)


def test_capture_takes_no_kept_record(reference, fresh):
    s, mask, kw, want = reference["few"]
    s2, mask2, kw2, want2 = reference["reverse"]
    got, other = _out(s), _out(s2)
    _call(s, mask, kw, got)                                # (the record and the kept workspace are there)
    binding.workspace_for(1 << 20, dev())
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        _call(s, mask, kw, got)
    for _ in range(4):
        for x in got[:3]:
            x.fill_(-3.0)
        graph.replay()
        _call(s2, mask2, kw2, other)                       # the program's own call between the replays
        torch.cuda.synchronize()
        assert _same(got, want) and _same(other, want2)


def test_a_call_that_gave_up_leaves_nothing_behind(reference, fresh):
    s, mask, kw, want = reference["reverse"]
    lib = binding.load()
    got = _out(s)
    lib.npd_debug_gang_spin_limit(1)                       # (waits that end at once: the rows are marked and the kernel exits)
    try:
        _call(s, mask, kw, got)
        torch.cuda.synchronize()
    finally:
        lib.npd_debug_gang_spin_limit(0)
    assert int(got[3].item()) in (0, 8)
    for name in ("reverse", "few", "reverse"):
        s, mask, kw, want = reference[name]
        got = _out(s)
        _call(s, mask, kw, got)
        torch.cuda.synchronize()
        assert _same(got, want), name


@pytest.mark.parametrize("route,what", [(r, w) for r in ("kept", "cleared") for w in ("forward", "skew", "topk")] +
                         [("forward", "forward")])         # (one launch: forward KL and no teacher)
def test_rows_that_gave_up_are_marked(fresh, route, what):
    """With a limit of one poll (the waits end at once and the kernel exits) every value is what it should be or NaN, and if there
    is NaN the flag says so; the next call with the default limit is exact.  Gradient calls on a kept record, on a workspace
    that the call clears, and forward-only calls in one launch."""
    T, V = 384, 151936
    g = torch.Generator(device=dev()).manual_seed(23)
    s = torch.randn((T, V), generator=g, device=dev()).mul_(3.0).to(torch.bfloat16)
    mask = (torch.rand(T, generator=g, device=dev()) < 0.8).to(torch.uint8)
    kw = dict(labels=torch.randint(0, V, (T,), generator=g, device=dev(), dtype=torch.int32))
    t = torch.randn((T, V), generator=g, device=dev()).add_(s).to(torch.bfloat16)
    if what == "topk":
        val, idx = torch.topk(t[:, :4096].float(), 24, dim=1)
        kw.update(teacher_idx=idx.to(torch.int32), teacher_val=val)
    else:
        kw.update(teacher_dense=t, **(dict(divergence=2, skew_alpha=0.1) if what == "skew" else {}))
    ws = torch.empty(1 << 20, dtype=torch.uint8, device=dev()) if route == "cleared" else None
    lib = binding.load()

    def run():
        out = [torch.full((T,), -1.0, device=dev()) for _ in range(3)]
        out.append(torch.full((T,), -1.0, device=dev()) if route == "forward" else torch.full_like(s, float("nan")))
        status = torch.zeros(1, dtype=torch.int32, device=dev())
        last = dict(teacher_nll_tok=out[3]) if route == "forward" else dict(grad_out=out[3])
        binding.npd_kd_loss_fwd_bwd(s, mask, kd_tok=out[0], nll_tok=out[1], lse_tok=out[2], dev_status=status, workspace=ws, **last,
                                    **kw)
        torch.cuda.synchronize()
        return out, int(status.item())

    with _Watched(lib, binding._host) as w:                 # the route that the call takes
        run()
        assert w.seen[-1][0] == ("cleared" if route == "cleared" else "kept")
    good, status = run()
    assert status == 0 and not any(torch.isnan(x).any() for x in good)
    lib.npd_debug_gang_spin_limit(1)
    try:
        hurried, status = run()
    finally:
        lib.npd_debug_gang_spin_limit(0)
    gave_up = [torch.isnan(x) for x in hurried]
    for x, y, nan in zip(hurried, good, gave_up):
        assert (nan | (x == y)).all()
        assert not nan[mask == 0].any()                     # rows that are not scored wait for nothing
    rows = sum(int(n.any(dim=1).sum() if n.dim() == 2 else n.sum()) for n in gave_up)
    print(f"[gave up] {route} {what}: status {status}, {rows} rows and scalars", flush=True)
    assert status == (8 if rows else 0)
    if route == "forward":                                  # one workgroup writes the scalars of a row
        assert all((n == gave_up[0]).all() for n in gave_up)
    for _ in range(2):
        again, status = run()
        assert status == 0 and _same(again, good)


def test_what_the_entry_point_refuses(reference):
    lib = binding.load()
    s, mask, kw, want = reference["few"]
    T, V = s.shape
    d = binding.KdDesc(T, V, binding.NPD_TEACHER_DENSE_BF16, V, V, 0, 0, 1.0, 1.0, 0.0, 0, 0.0)
    stream = torch.cuda.current_stream().cuda_stream
    need = lib.npd_kept_workspace_bytes(ctypes.byref(d), stream)
    assert need == 2 * lib.npd_workspace_bytes_preferred(ctypes.byref(d)) > 0
    short = binding.KdDesc(T, 1024, binding.NPD_TEACHER_DENSE_BF16, V, V, 0, 0, 1.0, 1.0, 0.0, 0, 0.0)
    none = binding.KdDesc(T, V, binding.NPD_TEACHER_DENSE_BF16, V, V, 0, 4, 1.0, 1.0, 0.0, 0, 0.0)
    assert lib.npd_kept_workspace_bytes(ctypes.byref(short), stream) == lib.npd_kept_workspace_bytes(ctypes.byref(none), stream) == 0
    got = _out(s)
    ws = torch.zeros(need + 512, dtype=torch.uint8, device=dev())

    def call(desc, at, size, grad):
        return lib.npd_kd_loss_fwd_bwd_kept(ctypes.byref(desc), s.data_ptr(), kw["teacher_dense"].data_ptr(), None, None,
                                            kw["labels"].data_ptr(), mask.data_ptr(), grad, got[1].data_ptr(), got[2].data_ptr(),
                                            None, None, got[3].data_ptr(), at, size, stream)

    assert call(d, ws.data_ptr(), need - 1, got[0].data_ptr()) == 6 and call(d, None, need, got[0].data_ptr()) == 6
    assert call(d, ws.data_ptr() + 4, need, got[0].data_ptr()) == 6 and call(none, ws.data_ptr(), need, got[0].data_ptr()) == 6
    assert call(d, got[0].data_ptr(), need, got[0].data_ptr()) == 4
    torch.cuda.synchronize()
    assert (ws == 0).all() and (got[1] == -1.0).all()       # nothing was enqueued
    assert call(d, ws.data_ptr(), need, got[0].data_ptr()) == 0
    torch.cuda.synchronize()
    assert _same(got, want) and (ws[need:] == 0).all()


@pytest.mark.parametrize("flags", [0, binding.NPD_FLAG_FWD_ONLY])
def test_the_entry_point_refuses_a_stream_under_capture(reference, flags):
    """A replay would repeat the number of the call.  Nothing is enqueued: what the capture holds besides replays as it should."""
    lib = binding.load()
    s, mask, kw, _ = reference["topk"]                     # (its rows; the teacher: the student)
    T, V = s.shape
    side = torch.cuda.Stream()
    d = binding.KdDesc(T, V, binding.NPD_TEACHER_DENSE_BF16, V, V, 0, flags, 1.0, 1.0, 0.0, 0, 0.0)
    need = lib.npd_kept_workspace_bytes(ctypes.byref(d), side.cuda_stream)
    assert need > 0
    ws = torch.zeros(need, dtype=torch.uint8, device=dev())
    got = _out(s)
    count = torch.zeros(1, device=dev())
    args = (ctypes.byref(d), s.data_ptr(), s.data_ptr(), None, None, kw["labels"].data_ptr(), mask.data_ptr(),
            None if flags else got[0].data_ptr(), got[1].data_ptr(), got[2].data_ptr(), None, None, got[3].data_ptr(),
            ws.data_ptr(), need, side.cuda_stream)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        count.add_(1.0)
        asked = lib.npd_kept_workspace_bytes(ctypes.byref(d), side.cuda_stream)
        status = lib.npd_kd_loss_fwd_bwd_kept(*args)
        count.add_(1.0)
    assert (asked, status) == (0, 5)
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
    assert count.item() == 6.0 and (ws == 0).all() and (got[1] == -1.0).all() and (got[2] == -1.0).all()
    with torch.cuda.stream(side):
        assert lib.npd_kd_loss_fwd_bwd_kept(*args) == 0    # the same call beside a capture
    torch.cuda.synchronize()
    assert (got[1] != -1.0).all()


@pytest.mark.parametrize("T,V,pitch,what", [
    (1, 50304, 50304, "tau1"), (24, 65536, 65536, "tau2"), (40, 50003, 50003, "tau1"), (60, 151936, 151936, "none"), (130, 131080, 131088, "tau2"),
    (512, 100352, 100352, "tau1"), (513, 100352, 100352, "tau1"), (3, 524288, 524288, "tau1"),
])
def test_forward_only_in_one_launch(T, V, pitch, what, fresh, monkeypatch):
    g = torch.Generator(device=dev()).manual_seed(T + V)
    s, t = ((3.0 * torch.randn((T, pitch), generator=g, device=dev())).to(torch.bfloat16)[:, :V] for _ in range(2))
    if T > 2:
        s[1, V // 3] = 300.0                               # waves that sum once more in the careful form
        t[2, 5:900] = float("-inf")
    mask = (torch.rand(T, generator=g, device=dev()) < 0.8).to(torch.uint8)
    mask[0] = 1
    lab = torch.randint(5000, V, (T,), generator=g, device=dev(), dtype=torch.int32)
    if T > 4:
        lab[4], mask[4] = V, 1                             # a label out of range
    results = []
    for native in (True, True, False):
        if not native:
            monkeypatch.setattr(binding, "_host", None)
        out = [torch.full((T,), -1.0, device=dev()) for _ in range(4)]
        status = torch.zeros(1, dtype=torch.int32, device=dev())
        kw = dict(labels=lab, nll_tok=out[0], lse_tok=out[1], dev_status=status)
        if what != "none":
            kw.update(teacher_dense=t, kd_tok=out[2], teacher_nll_tok=out[3], tau=2.0 if what == "tau2" else 1.0)
        print(f"[kept] forward only T={T} V={V} {what} native={native}", flush=True)
        binding.npd_kd_loss_fwd_bwd(s, mask, **kw)
        torch.cuda.synchronize()
        results.append(out + [status])
    assert _same(results[0], results[2]) and _same(results[1], results[2])
    assert int(results[0][4].item()) == (1 if T > 4 else 0)
