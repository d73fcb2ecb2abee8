"""The native marshalling of the decode-step calls against the Python checks:
every accepted form of the arguments gives the same results both ways, what
one refuses the other refuses with the same message, and argument forms the
native path does not know fall through to the Python checks.  Each form states which of these it is."""
import numpy as np
import pytest
import torch

import synth
from gpu_util import dev, dev_bf16

pytestmark = pytest.mark.gpu


class _Decline:
    """Stands in for the native module: declines every call."""

    def __getattr__(self, name):
        return lambda *a: None


class _Record:
    """The native module; how = what it made of the last call: "native", "declined" or "raised"."""

    def __init__(self, fast):
        self.fast, self.how = fast, None

    def __getattr__(self, name):
        def call(*a):
            self.how = "raised"
            r = getattr(self.fast, name)(*a)
            self.how = "declined" if r is None else "native"
            return r
        return call


def _both(monkeypatch, call, how="native"):
    """Outcome of call() natively marshalled and through the Python checks; how: what the native
    module makes of it (declined: both outcomes come from the Python checks)."""
    from paper_2606_08411_amd import _lib
    _lib.library()
    got = []
    rec = _Record(_lib._fast)
    for fast in (rec, _Decline()):
        with monkeypatch.context() as m:
            m.setattr(_lib, "_fast", fast)
            try:
                r = call()
                r = list(r.values()) if isinstance(r, dict) else list(r)
                torch.cuda.synchronize()
                got.append([None if x is None else x.clone() for x in r])
            except Exception as e:   # noqa: BLE001 - compared below
                got.append((type(e), str(e)))
    assert rec.how == how
    return got


def _same(got):
    a, b = got
    assert type(a) is type(b), (a, b)
    if isinstance(a, tuple):
        assert a == b
        return
    for x, y in zip(a, b):
        assert (x is None) == (y is None)
        if x is not None:
            assert x.dtype == y.dtype and x.shape == y.shape and torch.equal(x, y)


def _attn_args(n_ref=0, L=3):
    s = synth.make_step("tiny", 3, with_weight=False, L=L, tree="random", depth_max=2, P=70,
                        refresh_frac=n_ref / 70)
    a = dict(q=dev_bf16(s.q), k_lane=dev_bf16(s.k_lane), v_lane=dev_bf16(s.v_lane),
             k_prefix=dev_bf16(s.k_pre), v_prefix=dev_bf16(s.v_pre), parent=s.parent, B=s.B)
    if n_ref:
        a.update(refresh_idx=dev(s.refresh_idx), q_ref=dev_bf16(s.q_ref), k_ref=dev_bf16(s.k_ref),
                 v_ref=dev_bf16(s.v_ref))
    return a


class _Subclass(torch.Tensor):
    pass


ATTN = {
    "plain": lambda a: a,
    "list": lambda a: dict(a, parent=[int(x) for x in a["parent"]]),
    "tuple": lambda a: dict(a, parent=tuple(int(x) for x in a["parent"])),
    "int64": lambda a: dict(a, parent=a["parent"].astype(np.int64)),
    "strided": lambda a: dict(a, parent=np.repeat(a["parent"], 2)[::2]),
    "numpy B": lambda a: dict(a, B=np.int64(a["B"])),
    "no lse": lambda a: dict(a, want_lse=False),
    "scale": lambda a: dict(a, scale=np.float64(0.2)),
    "outputs": lambda a: dict(a, o=torch.empty_like(a["q"])),
    "parameter": lambda a: dict(a, q=torch.nn.Parameter(a["q"], requires_grad=False)),
    "subclass": lambda a: dict(a, q=a["q"].as_subclass(_Subclass)),
    "bad tree": lambda a: dict(a, parent=[0, 0, 0]),
    "short parent": lambda a: dict(a, parent=a["parent"][:2]),
    "dtype": lambda a: dict(a, q=a["q"].float()),
    "shape": lambda a: dict(a, k_lane=a["k_lane"][:-1]),
    "layout": lambda a: dict(a, k_prefix=a["k_prefix"].transpose(0, 1).contiguous().transpose(0, 1)),
    "cpu": lambda a: dict(a, v_lane=a["v_lane"].cpu()),
    "missing": lambda a: dict(a, v_lane=None),
    "small workspace": lambda a: dict(a, workspace=torch.empty(16, dtype=torch.uint8, device="cuda")),
    "no workspace tensor": lambda a: dict(a, workspace=7),
    "empty host index": lambda a: a if "q_ref" in a else dict(
        a, refresh_idx=torch.empty(0, dtype=torch.int32)),
    "index dtype": lambda a: dict(a, refresh_idx=a["refresh_idx"].long()) if "q_ref" in a else a,
}
# What the native module makes of a form, where not "native".
ATTN_HOW = dict.fromkeys(
    ("int64", "strided", "numpy B", "subclass", "short parent", "dtype", "shape", "layout", "cpu",
     "missing", "no workspace tensor"), "declined")
ATTN_HOW.update({"bad tree": "raised", ("empty host index", 0): "declined", ("index dtype", 7): "declined"})


@pytest.mark.parametrize("form", ATTN)
@pytest.mark.parametrize("n_ref", [0, 7])
def test_attention_forms(form, n_ref, monkeypatch):
    import paper_2606_08411_amd as al
    a = ATTN[form](_attn_args(n_ref))
    how = ATTN_HOW.get((form, n_ref), ATTN_HOW.get(form, "native"))
    _same(_both(monkeypatch, lambda: al.lane_attn_forward(**a), how))


def test_attention_refresh_only(monkeypatch):
    import paper_2606_08411_amd as al
    a = _attn_args(7)
    a.update(q=None, k_lane=None, v_lane=None, parent=[])
    _same(_both(monkeypatch, lambda: al.lane_attn_forward(**a)))


@pytest.mark.parametrize("parent,how", [
    ([], "native"), ((), "native"), (np.zeros(0, np.int32), "native"), (np.zeros(0), "declined"),
    ({}, "declined"), ("", "declined"), (b"", "declined"), (np.zeros((0, 3), np.int32), "declined")], ids=repr)
def test_no_lanes_forms(parent, how, monkeypatch):
    """Without lanes the parent is still an empty list of ints or refused."""
    import paper_2606_08411_amd as al
    a = _attn_args(7)
    a.update(q=None, k_lane=None, v_lane=None, parent=parent)
    _same(_both(monkeypatch, lambda: al.lane_attn_forward(**a), how))


LM = {
    "plain": lambda a: a,
    "all rows": lambda a: dict(a, row_idx=None, suppress_eos=None),
    "no lse": lambda a: dict(a, want_lse=False),
    "outputs": lambda a: dict(a, conf=torch.zeros(40, device="cuda"),
                              argmax=torch.zeros(40, dtype=torch.int32, device="cuda")),
    "short outputs": lambda a: dict(a, conf=torch.zeros(5, device="cuda")),
    "no rows": lambda a: dict(a, row_idx=a["row_idx"][:0]),
    "row dtype": lambda a: dict(a, row_idx=a["row_idx"].long()),
    "eos": lambda a: dict(a, eos_id=10 ** 7),
    "numpy eos": lambda a: dict(a, eos_id=np.int32(3)),
    "hidden": lambda a: dict(a, hidden=a["hidden"][:, ::2]),
}
LM_HOW = dict.fromkeys(("short outputs", "no rows", "row dtype", "numpy eos", "hidden"), "declined")
LM_HOW["eos"] = "raised"


@pytest.mark.parametrize("packed", [False, True], ids=["plain", "packed"])
@pytest.mark.parametrize("form", LM)
def test_lmhead_forms(form, packed, monkeypatch):
    import paper_2606_08411_amd as al
    g = np.random.default_rng(4)
    bf = lambda *s: dev_bf16(synth.f32_to_bf16_bits(g.standard_normal(s, dtype=np.float32)))
    a = LM[form](dict(hidden=bf(50, 64), row_idx=dev(np.arange(0, 40, dtype=np.int32)),
                      suppress_eos=dev((np.arange(40) % 2).astype(np.uint8)), eos_id=3))
    W = bf(700, 64)
    if packed:
        Wp = al.lmhead_pack_weight(W)
        call = lambda: al.lmhead_confidence_packed(W_packed=Wp, V=700, **a)
    else:
        call = lambda: al.lmhead_confidence(W=W, **a)
    _same(_both(monkeypatch, call, LM_HOW.get(form, "native")))


SEL = {
    "plain": {}, "topk": dict(mode=1, k_lane=[1, 2]), "topk without k": dict(mode=1),
    "drafts": dict(tau_future=0.3, b_len=np.array([20, 32], np.int32)),
    "ids": dict(delim_ids=[5, 6], digit_ids=(7,), open_ids=(8,), close_ids=(9,)),
    "id array": dict(delim_ids=np.array([5, 6])), "many ids": dict(delim_ids=tuple(range(17))),
    "role list": dict(role=[0, 1]), "role value": dict(role=np.array([0, 9], np.uint8)),
    "nan": dict(tau=float("nan")), "t_lane": dict(t_lane=(3, 4)), "short": dict(t_lane=(3,)),
    "role bytes": dict(role=b"\0\1"), "role bytearray": dict(role=bytearray(b"\0\1")),
    "t_lane bytes": dict(t_lane=b"\0\1"), "int64 t_lane": dict(t_lane=np.array([3, 4])),
}
SEL_HOW = dict.fromkeys(("id array", "many ids", "role list", "short", "role bytes", "t_lane bytes",
                         "int64 t_lane"), "declined")
SEL_HOW.update(dict.fromkeys(("topk without k", "role value", "nan"), "raised"))


@pytest.mark.parametrize("form", SEL)
def test_select_forms(form, monkeypatch):
    import paper_2606_08411_amd as al
    s = synth.make_step("tiny", 6, with_weight=False)
    conf, arg = synth.random_confidences(2, s.N, s.V)
    kw = dict(dict(L=s.L, B=s.B, role=s.role, tau=0.6, fallback_k=1), **SEL[form])

    def call():
        tok, msk = dev(s.tokens), dev(s.is_masked)
        z = lambda n, dt: torch.zeros(n, dtype=dt, device="cuda")
        out = dict(unmask_flag=z(s.N, torch.uint8), unmasked_pos=z(s.N, torch.int32),
                   still_masked_pos=z(s.N, torch.int32), counts=z(2, torch.int32),
                   lane_stats=z((s.L, 6), torch.int32), delim_flag=z(s.L * s.B, torch.uint8))
        r = al.select_unmask(dev(conf), dev(arg), dev(s.row_pos), tok, msk, out=out, **kw)
        assert r is out
        return dict(r, tok=tok, msk=msk)

    _same(_both(monkeypatch, call, SEL_HOW.get(form, "native")))


def test_outputs_given_are_returned():
    import paper_2606_08411_amd as al
    a = _attn_args()
    o = torch.empty_like(a["q"])
    assert al.lane_attn_forward(**a, o=o)[0] is o


def test_capture_without_workspace_is_refused(monkeypatch):
    """While a graph is captured a call that needs a workspace must be given one."""
    import paper_2606_08411_amd as al
    W = torch.zeros((700, 64), dtype=torch.bfloat16, device="cuda")
    h = torch.zeros((8, 64), dtype=torch.bfloat16, device="cuda")
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: True)
    _same(_both(monkeypatch, lambda: al.lmhead_confidence(h, W), "raised"))
    with pytest.raises(al.AsyncLaneError, match="being captured"):
        al.lmhead_confidence(h, W)
