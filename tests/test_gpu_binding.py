"""The native form of the binding's plain calls against its own checks: the
same results, and the same errors."""
import pytest
import torch

from paper_2609_39859_amd import _binding

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


def _step_call(fn):
    B, L, BL, d, V = 2, 40, 16, 64, 300
    g = torch.Generator().manual_seed(1)
    h = torch.randn(B * L, d, generator=g).bfloat16().to(DEV)
    W = torch.randn(V, d, generator=g).bfloat16().to(DEV)
    kw = dict(hidden=h, W_head=W, tokens=torch.full((B * L,), -1, dtype=torch.int32, device=DEV),
              mask=torch.ones(B * L, dtype=torch.uint8, device=DEV),
              block_start=torch.zeros(B, dtype=torch.int32, device=DEV), block_len=BL, tau=0.9,
              B=B, L=L, rule=_binding.FORK_RULE_RANDOM, rows_mode=_binding.FORK_ROWS_ACTIVE,
              fallback_uniform=torch.rand(B, generator=g).to(DEV), temperature=0.5,
              seed=-3, counter=2 ** 32 + 5)
    for k in ("out_conf", "out_entropy", "out_logp", "out_lse"):
        kw[k] = torch.zeros(B * L, device=DEV)
    kw["out_argmax"] = torch.zeros(B * L, dtype=torch.int32, device=DEV)
    for k, n in (("out_fallback", B), ("out_ncommit", B), ("out_commit_pos", B * BL)):
        kw[k] = torch.zeros(n, dtype=torch.int32, device=DEV)
    return fn, kw


def _calls():
    yield "step", _step_call(_binding.fork_step_ex)
    yield "noalloc", _step_call(_binding.fork_step_noalloc)
    g = torch.Generator().manual_seed(2)
    h = torch.randn(9, 32, generator=g).to(DEV)
    W = torch.randn(50, 32, generator=g).to(DEV)
    i32 = dict(dtype=torch.int32, device=DEV)
    yield "logprob", (_binding.logprob, dict(
        hidden=h, W_head=W, tokens=torch.arange(5, **i32), out_logp=torch.zeros(5, device=DEV),
        rows=torch.tensor([8, 0, 3, 3, 1], **i32), out_q=torch.zeros(5, device=DEV)))
    yield "grpo", (_binding.grpo_objective, dict(
        rewards=torch.tensor([0., 1., 1., 1.], device=DEV), offsets=torch.tensor([0, 1, 3, 3, 4], **i32),
        lp_new=torch.rand(4, generator=g).to(DEV), lp_old=torch.rand(4, generator=g).to(DEV), G=2,
        eps=0.2, out_group_obj=torch.zeros(2, device=DEV),
        out_skipped=torch.zeros(2, dtype=torch.uint8, device=DEV), out_J=torch.zeros(1, device=DEV),
        out_ratio=torch.zeros(4, device=DEV)))
    yield "select", (_binding.select, dict(
        conf=torch.rand(24, generator=g).to(DEV), argmax=torch.arange(24, **i32),
        tokens=torch.zeros(24, **i32), mask=torch.ones(24, dtype=torch.uint8, device=DEV),
        block_start=torch.zeros(3, **i32), block_len=4, tau=0.5, B=3, L=8,
        out_fallback=torch.zeros(3, **i32), out_ncommit=torch.zeros(3, **i32)))
    yield "top", (_binding.top_entropy, dict(
        entropy=torch.rand(3, 70, generator=g).to(DEV), k=7,
        out_sel=torch.zeros(3, 70, dtype=torch.uint8, device=DEV)))


class _Spy:
    """_fastcall, keeping what its functions returned."""

    def __init__(self, fast):
        self.fast, self.returned = fast, []

    def __getattr__(self, name):
        def call(*args):
            self.returned.append(getattr(self.fast, name)(*args))
            return self.returned[-1]
        return call


def _both(monkeypatch, fn, kw, change, taken=False):
    """(outcome natively, outcome by the binding's own checks) of fn(**kw)
    with `change` applied to fresh copies of the arguments; taken: the native
    function made the call."""
    _binding.lib()
    assert _binding._fast is not None
    out = []
    for native in (True, False):
        args = {k: v.clone() if isinstance(v, torch.Tensor) else v for k, v in kw.items()}
        change(args)
        with monkeypatch.context() as m:
            spy = _Spy(_binding._fast) if native else None
            m.setattr(_binding, "_fast", spy)
            try:
                fn(**args)
                torch.cuda.synchronize()
                out.append({k: v.cpu() for k, v in args.items() if isinstance(v, torch.Tensor)})
            except (TypeError, ValueError, _binding.ForkError) as e:
                out.append((type(e), str(e)))
            assert not (native and taken) or spy.returned == [_binding.FORK_OK]
    return out


@pytest.mark.parametrize("name", ["step", "noalloc", "logprob", "grpo", "select", "top"])
def test_native_calls_match_the_bindings_own(monkeypatch, name):
    fn, kw = dict(_calls())[name]

    def own_stream(a):
        a["stream"] = torch.cuda.current_stream()
    for change in (lambda a: None, own_stream):
        a, b = _both(monkeypatch, fn, kw, change, taken=True)
        assert set(a) == set(b)
        for k in a:
            assert torch.equal(a[k].view(torch.uint8), b[k].view(torch.uint8)), k
    tensors = [k for k, v in kw.items() if isinstance(v, torch.Tensor)]
    for k in tensors:
        def wrong_device(a, k=k):
            a[k] = a[k].cpu()

        def wrong_dtype(a, k=k):
            a[k] = a[k].to(torch.float64)

        def wrong_size(a, k=k):
            a[k] = torch.cat([a[k], a[k][:1]])

        def strided(a, k=k):
            a[k] = torch.stack([a[k], a[k]], dim=-1)[..., 0]
        for change in (wrong_device, wrong_dtype, wrong_size, strided):
            a, b = _both(monkeypatch, fn, kw, change)
            if isinstance(b, tuple):
                assert a == b, (k, change.__name__)
            else:
                assert all(torch.equal(a[n], b[n]) for n in a), (k, change.__name__)


@pytest.mark.parametrize("name", ["step", "noalloc", "logprob"])
def test_native_calls_take_the_lm_head_events(monkeypatch, name):
    """The pair of events is recorded by the native call, around the LM head;
    a pair of another form is left to the binding."""
    fn, kw = dict(_calls())[name]
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    for e in ev:
        e.record()
    pair = tuple(e.cuda_event for e in ev)
    _binding.lib()
    for events, returned in ((pair, _binding.FORK_OK), (list(pair), None)):
        spy = _Spy(_binding._fast)
        monkeypatch.setattr(_binding, "_fast", spy)
        begin = torch.cuda.Event(enable_timing=True)
        begin.record()
        fn(**kw, events=events)
        monkeypatch.undo()
        assert spy.returned == [returned]
        torch.cuda.synchronize()
        assert begin.elapsed_time(ev[0]) >= 0
        assert ev[0].elapsed_time(ev[1]) > 0
