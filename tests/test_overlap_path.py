"""The overlapped optimizer path of fpo_pseudograd (each matrix's update on a
side stream beside the GEMM launches that follow), which layers of enough work
take, against the pseudogradient followed by fpo_apply_update: bit-identical
eagerly (W3 and full MLP, SGD-momentum and AdamW), from two threads at once with
the library's side stream or the caller's, and from a captured graph."""
import threading

import pytest
import torch

from paper_2608_14563_amd import _lib as L_
from paper_2608_14563_amd import api

pytestmark = pytest.mark.gpu
BF = torch.bfloat16
# ragged; T d d_ff (x 4 with the full MLP) above the path's threshold
W3 = dict(T=4000, d=2056, d_ff=7560, L=2, full=False)
FULL = dict(T=1000, d=1032, d_ff=5000, L=2, full=True)


def make(dev, T, d, d_ff, L, full, adam, seed=0):
    assert T * d * d_ff * (4 if full else 1) >= (2e10 if full else 6e10)
    g = torch.Generator(device=dev).manual_seed(seed)
    rn = lambda *s, std=1.0, dt=BF: torch.empty(*s, device=dev).normal_(0, std, generator=g).to(dt)  # noqa: E731
    shapes = [(d, d_ff)] * L + ([(d_ff, d)] * (2 * L) if full else [])
    W = [rn(*s, std=0.02, dt=torch.float32) for s in shapes]
    s = dict(g=rn(T, d, std=0.02), a=[rn(T, d_ff) for _ in range(L)], W=W, s1=[torch.zeros_like(w) for w in W],
             s2=[torch.zeros_like(w) for w in W] if adam else None, lp=[torch.zeros_like(w, dtype=BF) for w in W],
             Wsq=torch.stack([(w.double() ** 2).sum() for w in W]), dW=[torch.empty_like(w) for w in W],
             ss=torch.zeros(len(W), dtype=torch.float64, device=dev), cs=torch.zeros(len(W), device=dev), kw={})
    s["kw"] = dict(dW3=s["dW"][:L], sumsq=s["ss"],
                   ws=api.workspace(api.fpo_pseudograd_workspace(T, d, d_ff, L, BF, full_mlp=full), dev))
    if full:
        s["kw"].update(W3_init=[rn(d, d_ff, std=0.02) for _ in range(L)], gate=[rn(T, d_ff) for _ in range(L)],
                       up=[rn(T, d_ff) for _ in range(L)], x_in=[rn(T, d) for _ in range(L)], dW1=s["dW"][L:2 * L],
                       dW2=s["dW"][2 * L:])
    return s


def opt(adam, step):
    return api.OptConfig(kind=L_.FPO_OPT_ADAMW if adam else L_.FPO_OPT_SGD, lr=1e-2, clip_frac=1e-3, step=step)


def fused(s, adam, step, overlap=None):
    api.fpo_pseudograd(s["g"], s["a"], opt=opt(adam, step), W_master=s["W"], W_lp=s["lp"], state1=s["s1"],
                       state2=s["s2"], W_sumsq=s["Wsq"], clip_scale=s["cs"], overlap=overlap, **s["kw"])


def separate(s, adam, step):
    api.fpo_pseudograd(s["g"], s["a"], **s["kw"])
    api.fpo_apply_update(opt(adam, step), s["dW"], s["ss"], s["W"], s["s1"], s["Wsq"], W_lp=s["lp"], state2=s["s2"],
                         clip_scale=s["cs"])


def same(a, b):
    torch.cuda.synchronize()
    for k in ("W", "s1", "s2", "lp", "dW"):
        for x, y in zip(a[k] or [], b[k] or []):
            assert torch.equal(x, y), k
    for k in ("Wsq", "ss", "cs"):
        assert torch.equal(a[k], b[k]), k


@pytest.mark.parametrize("adam", [False, True], ids=["sgd", "adamw"])
@pytest.mark.parametrize("case", [W3, FULL], ids=["w3", "full"])
def test_matches_separate_calls(dev, case, adam):
    a, b = make(dev, adam=adam, **case), make(dev, adam=adam, **case)
    for step in (1, 2):
        separate(a, adam, step)
        fused(b, adam, step)
        same(a, b)


@pytest.mark.parametrize("own", [False, True], ids=["library-side-stream", "caller-side-streams"])
def test_two_threads(dev, own):
    ref = [make(dev, adam=False, seed=k, **W3) for k in (0, 1)]
    got = [make(dev, adam=False, seed=k, **W3) for k in (0, 1)]
    for s in ref:
        for step in (1, 2, 3):
            fused(s, False, step)
    torch.cuda.synchronize()
    err = []

    def work(s):
        try:
            st = torch.cuda.Stream(device=dev)
            ov = api.Overlap(dev) if own else None
            with torch.cuda.stream(st):
                for step in (1, 2, 3):
                    fused(s, False, step, ov)
            st.synchronize()
        except Exception as e:  # pragma: no cover
            err.append(e)

    th = [threading.Thread(target=work, args=(s,)) for s in got]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert not err
    for a, b in zip(ref, got):
        same(a, b)


@pytest.mark.parametrize("case", [W3, FULL], ids=["w3", "full"])
def test_graph_replays(dev, case):
    a, b = make(dev, adam=False, **case), make(dev, adam=False, **case)
    ov = api.Overlap(dev)
    for s in (a, b):
        fused(s, False, 1, ov)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    st = torch.cuda.Stream(device=dev)
    with torch.cuda.graph(g, stream=st):
        fused(b, False, 2, ov)
    for _ in range(3):
        fused(a, False, 2, ov)
        g.replay()
        same(a, b)
