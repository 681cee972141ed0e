"""The synchronisation step where its replicas are split over the block: edges
of the 256-coordinate blocks and of the 4-coordinate lanes, the smallest and
largest replica counts of its range and those just outside, every strategy,
update, storage type and variant, against a float64 step; and bit for bit
against the thread-per-coordinate kernel on the same coordinates."""
import math

import pytest
import torch

from paper_2607_21224_amd.state import CpdpState, Hyper, Optimizer

pytestmark = pytest.mark.gpu

BF = {"f32": torch.float32, "bf16": torch.bfloat16}
EDGES = (1, 3, 4, 5, 255, 256, 257, 1023)
BETA, ALPHA = 0.5, 0.75


def _state(W, P, param="f32", grad="f32", mom="f32", adamw=False, seed=1):
    st = CpdpState(W, P, K=1, param_dt=param, grad_dt=grad, mom_dt=mom, adamw=adamw)
    g = torch.Generator(device="cuda").manual_seed(seed)
    n = lambda s, *shape: torch.randn(shape, generator=g, device="cuda") * s  # noqa: E731
    for buf in (st.params, st.mom, *((st.mom2,) if adamw else ())):
        buf.fill_(7.0)  # pads keep their value
    st.anchor.copy_(n(0.02, P))
    st.slow_mom.copy_(n(1e-2, P))
    st.params[:, :P] = n(1e-3, W, P) + st.anchor
    st.mom[:, :P] = n(1e-2, W, P)
    if adamw:
        st.mom2[:, :P] = n(1e-3, W, P).square()
    grads = torch.full((W, st.ld), 7.0, dtype=BF[grad], device="cuda")
    grads[:, :P] = n(1e-3, W, P)
    st.opt_step = 20
    return st, grads


def _reference(st, grads, method, opt, flags):
    """The step in float64, rounded where the library stores bf16."""
    P = st.P
    store = lambda x, like: x.to(like.dtype).double()  # noqa: E731
    th, m = st.params[:, :P].double(), st.mom[:, :P].double()
    a, u, g = st.anchor.double(), st.slow_mom.double(), grads[:, :P].double()
    out = {}
    if method != "localsgd":
        g = g.mean(0, keepdim=True).expand_as(g)
        if flags & 1:
            out["grads"] = g
    v = None
    if opt.kind == "adamw":
        t = st.opt_step + 1
        th = store(th * (1 - opt.lr * opt.weight_decay), st.params)
        m = opt.momentum * m + (1 - opt.momentum) * g
        v = opt.beta2 * st.mom2[:, :P].double() + (1 - opt.beta2) * g * g
        den = v.sqrt() / math.sqrt(1 - opt.beta2 ** t) + opt.eps
        th = store(th - opt.lr / (1 - opt.momentum ** t) * m / den, st.params)
    else:
        m = store(opt.momentum * m + (g + opt.weight_decay * th), st.mom)
        th = store(th - opt.lr * m, st.params)
    if flags & 2:
        m = m.mean(0, keepdim=True).expand_as(m)
        v = v.mean(0, keepdim=True).expand_as(m) if v is not None else None
    if method == "cpdp":
        u = BETA * u + (a - th.mean(0)) / opt.lr
        a = a - ALPHA * opt.lr * u
        th = store(a, st.params).expand_as(th)
    elif method == "localsgd":
        a = th.mean(0)
        th = store(a, st.params).expand_as(th)
    out.update(params=th, mom=m, slow_mom=u, anchor=a)
    if v is not None:
        out["mom2"] = v
    return out


def _views(st, grads):
    P = st.P
    d = {"params": st.params[:, :P], "mom": st.mom[:, :P], "slow_mom": st.slow_mom,
         "anchor": st.anchor, "grads": grads[:, :P]}
    if st.mom2 is not None:
        d["mom2"] = st.mom2[:, :P]
    return d


OPTS = {"sgd": Optimizer("sgd", 0.1, 0.9), "sgd_wd": Optimizer("sgd", 0.1, 0.9, weight_decay=5e-4),
        "adamw": Optimizer("adamw", 5e-4, 0.9, 0.999, 1e-8, 0.05)}


@pytest.mark.parametrize("method,opt,param,flags", [
    ("cpdp", "sgd_wd", "f32", 0), ("cpdp", "adamw", "f32", 3), ("cpdp", "adamw", "bf16", 0),
    ("cpdp", "sgd_wd", "bf16", 2), ("localsgd", "adamw", "f32", 2), ("localsgd", "sgd", "bf16", 0),
    ("ddp", "sgd_wd", "f32", 1), ("ddp", "adamw", "bf16", 3)])
@pytest.mark.parametrize("W", [1, 2, 3, 5, 16, 17, 30, 32, 33])
def test_step_against_float64(method, opt, param, flags, W):
    o = OPTS[opt]
    for P in EDGES:
        st, grads = _state(W, P, param, adamw=opt == "adamw")
        want = _reference(st, grads, method, o, flags)
        st.step_opt(1, grads, o, BETA, ALPHA, method=method, flags=flags)
        torch.cuda.synchronize()
        for k, x in _views(st, grads).items():
            if k not in want:
                continue
            # fp32: W <= 33 terms and a few roundings, 40 * 2^-24, against
            # u's (a - mean)/lr, whose terms are 1/lr larger than their
            # difference; bf16 parameters: a neighbour, 2^-8, for the few
            # values next to a rounding boundary, and through them the mean
            err = (x.double() - want[k]).norm() / want[k].norm()
            tol = 4e-3 if param == "bf16" else 4e-5
            assert err < tol, (method, opt, param, flags, W, P, k, float(err))
        for buf in (st.params, st.mom, grads):
            assert (buf[:, P:] == 7.0).all(), ("pad written", W, P)


@pytest.mark.parametrize("grad,mom", [("bf16", "f32"), ("bf16", "bf16"), ("f32", "bf16")])
@pytest.mark.parametrize("param", ["f32", "bf16"])
@pytest.mark.parametrize("W", [3, 8, 32])
def test_narrow_rows_against_float64(grad, mom, param, W):
    h = Hyper.fp32(0.1, 0.9, BETA, ALPHA)
    for method in ("cpdp", "localsgd", "ddp"):
        for P in EDGES:
            st, grads = _state(W, P, param, grad, mom)
            want = _reference(st, grads, method, OPTS["sgd"], 0)
            st.step(1, grads, h, method=method)
            torch.cuda.synchronize()
            for k, x in _views(st, grads).items():
                if k in want:
                    err = (x.double() - want[k]).norm() / want[k].norm()
                    assert err < 4e-3, (method, grad, mom, param, W, P, k, float(err))
            for buf in (st.params, st.mom, grads):
                assert (buf[:, P:] == 7.0).all(), ("pad written", W, P)


@pytest.mark.parametrize("W", [4, 8, 16])
@pytest.mark.parametrize("method,opt", [("cpdp", "sgd"), ("localsgd", "sgd_wd"), ("ddp", "sgd")])
def test_both_kernels_give_the_same_bits(W, method, opt):
    """A cached-size state takes the thread-per-coordinate kernel, the same
    columns as a small state the split one."""
    big, gbig = _state(W, 262_144 + 1023, seed=3)
    cuts = [(0, 1), (5, 3), (8, 4), (64, 257), (1000, 1023), (262_144, 1023)]
    small = []
    for lo, n in cuts:
        st, g = _state(W, n)
        for d, s in ((st.params, big.params), (st.mom, big.mom), (g, gbig)):
            d[:, :n] = s[:, lo:lo + n]
        st.anchor.copy_(big.anchor[lo:lo + n])
        st.slow_mom.copy_(big.slow_mom[lo:lo + n])
        small.append((st, g))
    for st, g in [(big, gbig)] + small:
        st.step_opt(1, g, OPTS[opt], BETA, ALPHA, method=method)
    torch.cuda.synchronize()
    for (lo, n), (st, g) in zip(cuts, small):
        for k, x in _views(st, g).items():
            y = _views(big, gbig)[k][..., lo:lo + n]
            assert torch.equal(x.contiguous().view(torch.int32),
                               y.contiguous().view(torch.int32)), (W, method, lo, n, k)
