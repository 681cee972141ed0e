"""Captured runs of table steps: consecutive local steps in one launch (runs of
8, with a rest), one advance for the whole graph, and a table that ends inside
a run, against the same steps called one by one, bit for bit."""
import pytest
import torch

from paper_2607_21224_amd import cpdp
from paper_2607_21224_amd.state import CpdpState, Optimizer, StepTable

pytestmark = pytest.mark.gpu


def _opt(kind, s):
    if kind == "adamw":
        return Optimizer("adamw", 5e-4 / (s + 1), 0.9, 0.999, 1e-8, 0.05)
    return Optimizer("sgd", 0.1 / (s + 1), 0.9, weight_decay=5e-4 if kind == "sgd_wd" else 0.0)


def _bits(st):
    P = st.P
    xs = [st.params[:, :P], st.mom[:, :P], st.slow_mom, st.anchor]
    if st.mom2 is not None:
        xs.append(st.mom2[:, :P])
    return [x.contiguous().view(torch.uint8) for x in xs]


@pytest.mark.parametrize("kind,param,method,W,P,K,table_steps", [
    ("adamw", "f32", "cpdp", 3, 1, 12, 24), ("adamw", "bf16", "cpdp", 8, 1023, 11, 22),
    ("sgd", "f32", "localsgd", 2, 257, 3, 6), ("sgd_wd", "bf16", "cpdp", 5, 3, 9, 18),
    ("sgd", "f32", "ddp", 4, 260, 2, 4), ("adamw", "f32", "cpdp", 4, 515, 6, 9),
    ("sgd", "f32", "cpdp", 33, 255, 10, 4)])
def test_captured_runs_equal_single_steps(kind, param, method, W, P, K, table_steps):
    dt = torch.bfloat16 if param == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(7)
    theta = (torch.randn(P, generator=gen, device="cuda") * 0.02).to(dt)
    a, b = (CpdpState(W, P, K=K, param_dt=param, adamw=kind == "adamw") for _ in range(2))
    for st in (a, b):
        st.init_opt(theta, _opt(kind, 0))
    grads = [torch.zeros((W, a.ld), device="cuda") for _ in range(K)]
    for g in grads:
        g[:, :P] = torch.randn((W, P), generator=gen, device="cuda") * 1e-3
    table = StepTable([(_opt(kind, s), s + 1, 0.5, 0.75) for s in range(table_steps)])
    graph, kinds = b.capture_steps(grads, table, method=method)
    assert kinds == ["reconcile" if method == "ddp" or j == K - 1 else "local" for j in range(K)]
    for period in range(3):
        graph.replay()
        for j in range(K):
            s = period * K + j
            if s < table_steps:
                a.step_opt(j + 1, grads[j], _opt(kind, s), 0.5, 0.75, method=method)
        torch.cuda.synchronize()
        assert table.position() == min((period + 1) * K, table_steps)
        for x, y in zip(_bits(a), _bits(b)):
            assert torch.equal(x, y), (kind, param, method, period)


def test_capture_before_the_table_is_refilled():
    """A run captured while the table is shorter than the run, which then gets
    all its entries: what a replay steps is decided when it runs."""
    W, P, K = 4, 515, 4
    gen = torch.Generator(device="cuda").manual_seed(5)
    theta = torch.randn(P, generator=gen, device="cuda") * 0.02
    a, b = (CpdpState(W, P, K=K) for _ in range(2))
    for st in (a, b):
        st.init_opt(theta, _opt("sgd", 0))
    grads = [torch.zeros((W, a.ld), device="cuda") for _ in range(K)]
    for g in grads:
        g[:, :P] = torch.randn((W, P), generator=gen, device="cuda") * 1e-3
    table = StepTable([(_opt("sgd", s), s + 1, 0.5, 0.75) for s in range(K)])

    def fill(n):
        cpdp.cpdp_step_table_fill(table.handle, table.buf.numel(),
                                  [_opt("sgd", s).c_struct(s + 1) for s in range(n)],
                                  [0.5] * n, [0.75] * n)

    fill(1)
    graph, _ = b.capture_steps(grads, table)
    fill(K)
    graph.replay()
    for j in range(K):
        a.step_opt(j + 1, grads[j], _opt("sgd", j), 0.5, 0.75)
    torch.cuda.synchronize()
    assert table.position() == K
    for x, y in zip(_bits(a), _bits(b)):
        assert torch.equal(x, y)


@pytest.mark.parametrize("flags", [1, 2, 3])
@pytest.mark.parametrize("kind,param,method,W,P,K", [
    ("adamw", "f32", "cpdp", 4, 515, 3), ("sgd", "bf16", "ddp", 17, 260, 2),
    ("sgd_wd", "f32", "localsgd", 32, 1023, 4)])
def test_captured_variants_equal_single_steps(kind, param, method, W, P, K, flags):
    """The synchronisation variants inside a captured run.  One step writes its
    gradient rows, so every step has rows of its own on both sides."""
    dt = torch.bfloat16 if param == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(11)
    theta = (torch.randn(P, generator=gen, device="cuda") * 0.02).to(dt)
    a, b = (CpdpState(W, P, K=K, param_dt=param, adamw=kind == "adamw") for _ in range(2))
    for st in (a, b):
        st.init_opt(theta, _opt(kind, 0))
    grads = [torch.zeros((W, a.ld), device="cuda") for _ in range(K)]
    for g in grads:
        g[:, :P] = torch.randn((W, P), generator=gen, device="cuda") * 1e-3
    single = [g.clone() for g in grads]
    table = StepTable([(_opt(kind, s), s + 1, 0.5, 0.75) for s in range(2 * K)])
    graph, _ = b.capture_steps(grads, table, method=method, flags=flags)
    for period in range(2):
        graph.replay()
        for j in range(K):
            a.step_opt(j + 1, single[j], _opt(kind, period * K + j), 0.5, 0.75, method=method,
                       flags=flags)
        torch.cuda.synchronize()
        for x, y in zip(_bits(a) + single, _bits(b) + grads):
            assert torch.equal(x, y), (kind, param, method, flags, period)
