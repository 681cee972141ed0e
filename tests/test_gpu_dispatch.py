"""The same step through every kernel that can take it gives the same bits:
states whose size goes to the thread-per-coordinate kernel against the same
columns as small states that the split step takes, flat rows against step
tables and plans, for the types and replica counts at the lines between them."""
import pytest
import torch

from paper_2607_21224_amd.multi import CpdpMultiState
from paper_2607_21224_amd.state import CpdpState, Hyper, Optimizer, StepTable

pytestmark = pytest.mark.gpu

BF = {"f32": torch.float32, "bf16": torch.bfloat16}
BETA, ALPHA = 0.5, 0.75
OPTS = {"sgd": Optimizer("sgd", 0.1, 0.9), "sgd_wd": Optimizer("sgd", 0.1, 0.9, weight_decay=5e-4),
        "adamw": Optimizer("adamw", 5e-4, 0.9, 0.999, 1e-8, 0.05)}


def _state(W, P, param="f32", grad="f32", mom="f32", adamw=False, seed=3):
    st = CpdpState(W, P, K=1, param_dt=param, grad_dt=grad, mom_dt=mom, adamw=adamw)
    g = torch.Generator(device="cuda").manual_seed(seed)
    n = lambda s, *shape: torch.randn(shape, generator=g, device="cuda") * s  # noqa: E731
    st.anchor.copy_(n(0.02, P))
    st.slow_mom.copy_(n(1e-2, P))
    st.params[:, :P] = n(1e-3, W, P) + st.anchor
    st.mom[:, :P] = n(1e-2, W, P)
    if adamw:
        st.mom2[:, :P] = n(1e-3, W, P).square()
    grads = torch.zeros((W, st.ld), dtype=BF[grad], device="cuda")
    grads[:, :P] = n(1e-3, W, P)
    st.opt_step = 20
    return st, grads


def _rows(st, grads):
    d = {"params": st.params, "mom": st.mom, "grads": grads}
    if st.mom2 is not None:
        d["mom2"] = st.mom2
    return d


def _columns(st, grads, lo, n):
    """The coordinates lo .. lo + n - 1 as a state of their own."""
    c = CpdpState(st.W, n, K=1, param_dt=st.param_dt, grad_dt=st.grad_dt, mom_dt=st.mom_dt,
                  adamw=st.mom2 is not None)
    g = torch.zeros((st.W, c.ld), dtype=grads.dtype, device="cuda")
    for k, dst in _rows(c, g).items():
        dst[:, :n] = _rows(st, grads)[k][:, lo:lo + n]
    c.anchor.copy_(st.anchor[lo:lo + n])
    c.slow_mom.copy_(st.slow_mom[lo:lo + n])
    c.opt_step = st.opt_step
    return c, g


def _values(st, grads, lo=0, n=None):
    n = st.P - lo if n is None else n
    d = {k: v[:, lo:lo + n] for k, v in _rows(st, grads).items()}
    d["anchor"], d["slow_mom"] = st.anchor[lo:lo + n], st.slow_mom[lo:lo + n]
    return {k: v.contiguous().view(torch.uint8) for k, v in d.items()}


# types and replica counts with a band of their own, inside it: 1100 wavefronts
# (all-bf16 DDP needs 24 replicas, 8 replicas of AdamW are past its line at 1600)
@pytest.mark.parametrize("waves,W,method,opt,types,flags", [
    (1100, 12, "cpdp", "sgd", ("f32", "f32", "f32"), 0),
    (1100, 17, "localsgd", "sgd_wd", ("f32", "f32", "f32"), 0),
    (1100, 32, "ddp", "sgd", ("f32", "f32", "f32"), 1),
    (1100, 12, "cpdp", "sgd", ("f32", "f32", "f32"), 2),
    (1100, 16, "cpdp", "adamw", ("f32", "f32", "f32"), 0),
    (1600, 8, "cpdp", "adamw", ("f32", "f32", "f32"), 3),
    (1100, 32, "localsgd", "adamw", ("bf16", "f32", "f32"), 2),
    (1100, 16, "cpdp", "sgd", ("bf16", "f32", "f32"), 0),
    (1100, 8, "cpdp", "sgd", ("f32", "bf16", "f32"), 0),
    (1100, 4, "localsgd", "sgd", ("bf16", "bf16", "f32"), 0),
    (1100, 32, "cpdp", "sgd", ("f32", "bf16", "bf16"), 0),
    (1100, 24, "ddp", "sgd", ("bf16", "bf16", "bf16"), 0),
    (9000, 9, "cpdp", "sgd", ("bf16", "bf16", "bf16"), 0),
    (9000, 28, "ddp", "sgd", ("bf16", "f32", "bf16"), 0),
    (9000, 30, "cpdp", "sgd", ("f32", "bf16", "bf16"), 0),
    # past the cache with the gradient mean written back
    (11000, 3, "ddp", "sgd_wd", ("f32", "f32", "f32"), 1),
    (5500, 6, "ddp", "adamw", ("f32", "f32", "f32"), 3)])
def test_both_sides_of_the_line(waves, W, method, opt, types, flags):
    P = waves * 256 + 3  # a last wavefront of one lane
    st, grads = _state(W, P, *types, adamw=opt == "adamw")
    cuts = [(0, 1), (5, 3), (64, 257), (1000, 1023), (P - 3, 3), (P - 259, 259)]
    small = [_columns(st, grads, lo, n) for lo, n in cuts]
    for s, g in [(st, grads)] + small:
        if types[1:] == ("f32", "f32"):
            s.step_opt(1, g, OPTS[opt], BETA, ALPHA, method=method, flags=flags)
        else:
            _plain(s, g, method)
    torch.cuda.synchronize()
    for (lo, n), (s, g) in zip(cuts, small):
        want = _values(st, grads, lo, n)
        for k, x in _values(s, g).items():
            assert torch.equal(x, want[k]), (waves, W, method, opt, types, flags, lo, n, k)


def _plain(st, grads, method):
    o = OPTS["sgd"]
    st.step(1, grads, Hyper.fp32(o.lr, o.momentum, BETA, ALPHA), method=method)


@pytest.mark.parametrize("P", [4, 16 * 256, 1023 * 256, 64 * 256])
@pytest.mark.parametrize("W,types", [(4, ("f32", "f32", "f32")), (8, ("f32", "bf16", "f32")),
                                     (16, ("f32", "f32", "f32")), (4, ("bf16", "bf16", "bf16"))])
@pytest.mark.parametrize("method", ["cpdp", "localsgd", "ddp"])
def test_rows_of_whole_vectors(P, W, types, method):
    """Small rows of whole vectors go to the compile-time-W kernels, one
    coordinate more to the split step."""
    st, grads = _state(W, P + 1, *types)
    whole, g = _columns(st, grads, 0, P)
    for s, x in ((st, grads), (whole, g)):
        _plain(s, x, method)
    torch.cuda.synchronize()
    want = _values(st, grads, 0, P)
    for k, x in _values(whole, g).items():
        assert torch.equal(x, want[k]), (P, W, types, method, k)


@pytest.mark.parametrize("flags", [0, 3])
@pytest.mark.parametrize("W,P", [(17, 515), (30, 1023), (32, 260), (12, 1100 * 256 + 5),
                                 (4, 4096), (32, 3), (40, 259),
                                 (2, (1 << 23) + 5)])
@pytest.mark.parametrize("opt,param,method", [("sgd", "bf16", "cpdp"), ("adamw", "f32", "localsgd"),
                                              ("sgd_wd", "f32", "ddp"), ("adamw", "bf16", "cpdp")])
def test_tables_and_plans_equal_flat_steps(W, P, opt, param, method, flags):
    """Step tables and plans at two and four replicas a group, in the band and
    beyond what the split step takes."""
    o = OPTS[opt]
    adamw = opt == "adamw"
    st, grads = _state(W, P, param, adamw=adamw)
    tab, tg = _columns(st, grads, 0, P)
    sizes = [P] if P < 8 else [1, 3, P - 4 - P // 3, P // 3]
    multi = CpdpMultiState(W, sizes, param_dt=param, adamw=adamw)
    offs = [sum(sizes[:i]) for i in range(len(sizes))]
    for t, (lo, n) in enumerate(zip(offs, sizes)):
        for k, rows in _rows(st, grads).items():
            for i in range(W):
                getattr(multi, k)[i][t][:n] = rows[i, lo:lo + n]
        multi.anchor[t][:n] = st.anchor[lo:lo + n]
        multi.slow_mom[t][:n] = st.slow_mom[lo:lo + n]
    multi.opt_step = st.opt_step
    table = StepTable([(o, st.opt_step + 1, BETA, ALPHA)])
    st.step_opt(1, grads, o, BETA, ALPHA, method=method, flags=flags)
    tab.step_table(1, tg, table, method=method, flags=flags)
    multi.step(1, o, BETA, ALPHA, method=method, flags=flags)
    torch.cuda.synchronize()
    want = _values(st, grads)
    for k, x in _values(tab, tg).items():
        assert torch.equal(x, want[k]), ("table", W, P, opt, param, method, flags, k)
    for k, rows in _rows(st, grads).items():
        for i in range(W):
            assert torch.equal(multi.gather(k, i), rows[i, :P]), ("plan", W, P, k, i)
    assert torch.equal(multi.gather("anchor"), st.anchor) and \
        torch.equal(multi.gather("slow_mom"), st.slow_mom)


@pytest.mark.parametrize("W,n,blocks", [(1, 1, 3), (1, 8, 40), (1, 9, 40), (2, 9, 2048),
                                        (1, 9, 2049), (1, 256, 2049), (2, 129, 2049),
                                        (1, 257, 6144), (1, 257, 6145), (33, 10, 660),
                                        (1, 33, 2049), (2, 64, 6144), (1, 64, 6145),
                                        (1, 65, 2049)])
@pytest.mark.parametrize("kind", ["local", "sync"])
def test_plan_blocks_find_their_tensors(W, n, blocks, kind):
    """Both searches of a plan, on each side of the lines between them: `blocks`
    blocks over n tensors of 1 to 3 chunks, the last with the rest."""
    chunks = blocks // W if kind == "local" else blocks
    sizes = [(1 + i % 3) * 256 - i % 5 for i in range(n)]
    sizes[-1] = 3
    sizes[-1] += (chunks - sum((s + 255) // 256 for s in sizes)) * 256
    assert sizes[-1] > 0
    P = sum(sizes)
    st, grads = _state(W, P)
    multi = CpdpMultiState(W, sizes)
    for k, rows in _rows(st, grads).items():
        for i in range(W):
            for dst, src in zip(getattr(multi, k)[i], rows[i, :P].split(sizes)):
                dst[:len(src)] = src
    for k in ("anchor", "slow_mom"):
        for dst, src in zip(getattr(multi, k), getattr(st, k).split(sizes)):
            dst[:len(src)] = src
    multi.opt_step = st.opt_step
    st.K = multi.K = 2 if kind == "local" else 1
    assert st.step_opt(1, grads, OPTS["sgd"], BETA, ALPHA) == \
        multi.step(1, OPTS["sgd"], BETA, ALPHA) == ("local" if kind == "local" else "reconcile")
    torch.cuda.synchronize()
    for k, rows in _rows(st, grads).items():
        for i in range(W):
            assert torch.equal(multi.gather(k, i), rows[i, :P]), (W, n, blocks, kind, k, i)
    assert torch.equal(multi.gather("anchor"), st.anchor)
    assert torch.equal(multi.gather("slow_mom"), st.slow_mom)
