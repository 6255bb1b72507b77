"""The overlapped optimizer path of fpo_pseudograd (each matrix's update on a
side stream beside the GEMM launches that follow), against the pseudogradient
followed by fpo_apply_update: bit-identical eagerly over two steps (W3, with
fp32 and bf16-staged gradients, one and two update workgroups a CU, a post-FFN
norm; full MLP in whole and ragged tiles; SGD with and without momentum, AdamW),
from two threads at once with the library's side stream or the caller's, and
from a captured graph. Every case is checked to take that path, by the number of
update launches."""
import threading

import pytest
import torch

from paper_2608_14563_amd import _lib as L_
from paper_2608_14563_amd import api
from tests._util import kernel_stats

pytestmark = pytest.mark.gpu
BF = torch.bfloat16
# ragged; one update workgroup a CU
W3 = dict(T=1300, d=4104, d_ff=7560, L=3)
# two (SGD; AdamW's go one a CU): fp32 gradients below 1200 tokens, staged ones below 3072
FEW = dict(T=1030, d=4104, d_ff=7560, L=3)
STAGED = dict(T=2050, d=4104, d_ff=7560, L=4, staged=True)
NORM = dict(STAGED, pffn=True)
# W3 first in both; the second in whole tiles (errh's LDS epilogue); the third W3 last
FULL = dict(T=1000, d=1032, d_ff=11016, L=2, full=True)
FULL_WHOLE = dict(T=512, d=1024, d_ff=11264, L=2, full=True)
FULL_LAST = dict(T=4000, d=2040, d_ff=7896, L=1, full=True)
IDS = {id(v): k.lower() for k, v in dict(globals()).items() if isinstance(v, dict) and "d_ff" in v}


def ids(v):
    return IDS.get(id(v)) if isinstance(v, dict) else v


def make(dev, T, d, d_ff, L, full=False, staged=False, pffn=False, opt="sgd", seed=0):
    g = torch.Generator(device=dev).manual_seed(seed)
    rn = lambda *s, std=1.0, dt=BF: torch.empty(*s, device=dev).normal_(0, std, generator=g).to(dt)  # noqa: E731
    shapes = [(d, d_ff)] * L + ([(d_ff, d)] * (2 * L) if full else [])
    W = [rn(*s, std=0.02, dt=torch.float32) for s in shapes]
    s = dict(g=rn(T, d, std=0.02), a=[rn(T, d_ff) for _ in range(L)], W=W,
             s1=None if opt == "plain" else [torch.zeros_like(w) for w in W],
             s2=[torch.zeros_like(w) for w in W] if opt == "adamw" else None,
             lp=[torch.zeros_like(w, dtype=BF) for w in W], Wsq=torch.stack([(w.double() ** 2).sum() for w in W]),
             dW=[torch.empty_like(w) for w in W], ss=torch.zeros(len(W), dtype=torch.float64, device=dev),
             cs=torch.zeros(len(W), device=dev), kw={}, opt=opt, staged=staged)
    s["kw"] = dict(sumsq=s["ss"], ws=api.workspace(
        api.fpo_pseudograd_workspace(T, d, d_ff, L, BF, full_mlp=full, grad_bf16=staged, post_ffn=pffn), dev))
    if pffn:
        s["kw"]["post_ffn"] = api.PostFfn(rn(T, d, std=0.02, dt=torch.float32), [rn(T, d) for _ in range(L)],
                                          [rn(d) for _ in range(L)])
    if full:
        s["kw"].update(W3_init=[rn(d, d_ff, std=0.02) for _ in range(L)], gate=[rn(T, d_ff) for _ in range(L)],
                       up=[rn(T, d_ff) for _ in range(L)], x_in=[rn(T, d) for _ in range(L)], dW1=s["dW"][L:2 * L],
                       dW2=s["dW"][2 * L:])
    s["dW3"] = s["dW"][:L]
    return s


def opt(s, step):
    return api.OptConfig(kind=L_.FPO_OPT_ADAMW if s["opt"] == "adamw" else L_.FPO_OPT_SGD, lr=1e-2, clip_frac=1e-3,
                         step=step, momentum=0.0 if s["opt"] == "plain" else 0.9)


def fused(s, step, overlap=None):
    api.fpo_pseudograd(s["g"], s["a"], dW3=None if s["staged"] else s["dW3"], grad_bf16=s["staged"], opt=opt(s, step),
                       W_master=s["W"], W_lp=s["lp"], state1=s["s1"], state2=s["s2"], W_sumsq=s["Wsq"],
                       clip_scale=s["cs"], overlap=overlap, **s["kw"])


def separate(s, step, staged_norms=None):
    """staged_norms: the squared norms of the gradients rounded to bf16, which the
    update then takes in place of the fp32 ones."""
    api.fpo_pseudograd(s["g"], s["a"], dW3=s["dW3"], **s["kw"])
    dW, ss = s["dW"], s["ss"]
    if s["staged"]:
        dW, ss = [w.to(BF).float() for w in dW], staged_norms
        for w, n in zip(dW, ss):
            n2 = float((w.double() ** 2).sum())
            assert abs(float(n) - n2) <= 1e-6 * n2
    api.fpo_apply_update(opt(s, step), dW, ss, s["W"], s["s1"], s["Wsq"], W_lp=s["lp"], state2=s["s2"],
                         clip_scale=s["cs"])


def same(a, b, keys=("W", "s1", "s2", "lp", "dW", "Wsq", "ss", "cs")):
    torch.cuda.synchronize()
    for k in keys:
        for x, y in zip(a[k] if a[k] is not None else [], b[k] if b[k] is not None else []):
            assert torch.equal(x, y), k


def update_launches(call):
    """Launches of the update kernel that call makes: one a matrix on the
    overlapped path, one for up to 32 matrices otherwise."""
    return kernel_stats("update", call)[1]


@pytest.mark.parametrize("case,kind", [(W3, "sgd"), (W3, "adamw"), (FEW, "sgd"), (FEW, "plain"), (FEW, "adamw"),
                                       (STAGED, "sgd"), (STAGED, "plain"), (STAGED, "adamw"), (NORM, "sgd"),
                                       (FULL, "sgd"), (FULL, "adamw"), (FULL_WHOLE, "sgd"), (FULL_WHOLE, "adamw"),
                                       (FULL_LAST, "sgd"), (FULL_LAST, "adamw")], ids=ids)
def test_matches_separate_calls(dev, case, kind):
    a, b = make(dev, opt=kind, **case), make(dev, opt=kind, **case)
    for step in (1, 2):
        assert update_launches(lambda: fused(b, step)) == len(b["W"])
        separate(a, step, b["ss"])
        same(a, b, ("W", "s1", "s2", "lp", "Wsq", "cs") + (() if b["staged"] else ("dW", "ss")))


@pytest.mark.parametrize("case", [W3, STAGED], ids=ids)
@pytest.mark.parametrize("own", [False, True], ids=["library-side-stream", "caller-side-streams"])
def test_two_threads(dev, own, case):
    ref = [make(dev, seed=k, **case) for k in (0, 1)]
    got = [make(dev, seed=k, **case) for k in (0, 1)]
    for s in ref:
        for step in (1, 2, 3):
            fused(s, step)
    torch.cuda.synchronize()
    err = []

    def work(s):
        try:
            st = torch.cuda.Stream(device=dev)
            ov = api.Overlap(dev) if own else None
            with torch.cuda.stream(st):
                for step in (1, 2, 3):
                    fused(s, step, ov)
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
        same(a, b, ("W", "s1", "s2", "lp", "Wsq", "cs", "ss"))


@pytest.mark.parametrize("case,kind", [(W3, "sgd"), (STAGED, "sgd"), (STAGED, "adamw"), (NORM, "sgd"), (FULL, "sgd"),
                                       (FULL_LAST, "adamw")], ids=ids)
def test_graph_replays(dev, case, kind):
    a, b = make(dev, opt=kind, **case), make(dev, opt=kind, **case)
    ov = api.Overlap(dev)
    for s in (a, b):
        fused(s, 1, ov)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    st = torch.cuda.Stream(device=dev)
    with torch.cuda.graph(g, stream=st):
        fused(b, 2, ov)
    for _ in range(3):
        fused(a, 2, ov)
        g.replay()
        same(a, b, ("W", "s1", "s2", "lp", "Wsq", "cs", "ss"))
