"""The marshalling extension against the ctypes path of the same functions: the same bits for calls it takes, and for every call that
one of the two refuses the same error from both."""
import pytest
import torch

import gpu_util as gu
from paper_2512_05754_amd import binding

pytestmark = pytest.mark.gpu


def stages(dtype, d=64, B=1, Hh=2, nb=16, k=3):
    gen = torch.Generator(device=gu.DEV).manual_seed(d)
    q, kk, v = (torch.randn((B, Hh, nb * 64, d), device=gu.DEV, generator=gen).to(dtype) for _ in range(3))
    e = lambda shape, t: torch.empty(shape, dtype=t, device=gu.DEV)
    return dict(q=q, k=kk, v=v, scores=e((B, Hh, nb, nb), torch.float32), ws=e((2 * B * Hh * nb * d * 4,), torch.uint8), idx=e((B, Hh, nb, k), torch.int32),
                cnt=e((B, Hh, nb), torch.int32), wo=e((B, Hh, nb), torch.int32), out=e(q.shape, torch.float32), lse=e(q.shape[:3], torch.float32),
                budgets=torch.randint(0, k + 1, (B, Hh, nb), device=gu.DEV, generator=gen, dtype=torch.int32))


def run(s, nv, **change):
    t = {**s, **change}
    binding.block_scores(t["q"], t["k"], seq_valid=nv, out=t["scores"], workspace=t["ws"])
    binding.select_topk(t["scores"], k=t.get("keep", 3), seq_valid=nv, budgets=t.get("use_budgets"), kmax=t.get("kmax"), idx=t["idx"], cnt=t["cnt"],
                        force_local=t.get("local", False))
    wo = t["wo"] if t.get("ordered") else None
    if wo is not None:
        binding.attn_work_order(t["cnt"], t["idx"].shape[3], idx=t["idx"], out=wo)
    binding.block_sparse_attn(t["q"], t["k"], t["v"], t["idx"], t["cnt"], seq_valid=nv, scale=t.get("scale", 0.0), out=t["out"], lse=t.get("use_lse"),
                              work_order=wo)
    return [t[n].clone() for n in ("scores", "idx", "cnt", "out", "lse")]


class Recorded:
    """The extension, and what each of its functions returned: a status, or None for what it leaves to the binding."""

    def __init__(self, calls):
        self.calls, self.returned = calls, {}

    def __getattr__(self, name):
        def call(*args):
            status = getattr(self.calls, name)(*args)
            self.returned[name] = status
            return status

        return call


def both(monkeypatch, f):
    """Result or error of f with the extension and without; what the extension returned."""
    got = []
    binding.lib()
    assert binding._calls is not None, "the build step builds the extension"
    extension = Recorded(binding._calls)
    for calls in (extension, None):
        with monkeypatch.context() as m:
            m.setattr(binding, "_calls", calls)
            try:
                got.append(f())
            except Exception as e:
                got.append((type(e), str(e)))
    return (*got, extension.returned)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("nv", [None, 1000])
def test_the_same_bits(usv, monkeypatch, dtype, nv):
    s = stages(dtype)
    for change in ({}, {"local": True}, {"use_budgets": s["budgets"], "keep": 0, "kmax": 3}, {"scale": 0.3, "use_lse": s["lse"]},
                   {"ordered": dtype == torch.bfloat16}, {"scale": 1}):
        s["lse"].zero_()
        a, b, returned = both(monkeypatch, lambda: run(s, nv, **change))
        assert isinstance(a, list) and isinstance(b, list), (a, b)
        # the extension did it all, but for a scale that is not a float
        taken = {"block_scores": 0, "select_topk": 0, "block_sparse_attn": None if "scale" in change and isinstance(change["scale"], int) else 0}
        if change.get("ordered"): taken["attn_work_order"] = 0
        assert returned == taken, change
        for x, y in zip(a, b):
            assert torch.equal(x.view(torch.int32), y.view(torch.int32)), change


@pytest.mark.parametrize("what", ["cpu q", "strided q", "k of another shape", "k of another type", "half", "three dimensions", "scores not fp32",
                                  "workspace too small", "idx int64", "idx of another shape", "cnt of another shape", "out of another shape", "out half",
                                  "seq_valid too large", "seq_valid a string", "k too large", "tokens not whole blocks", "work order of another shape",
                                  "lse not fp32", "not a tensor", "head dimension"])
def test_the_same_errors(usv, monkeypatch, what):
    s, nv, change = stages(torch.bfloat16), 1000, {}
    q = s["q"]
    if what == "cpu q": change["q"] = q.cpu()
    if what == "strided q": change["q"] = q.transpose(1, 2).contiguous().transpose(1, 2)
    if what == "k of another shape": change["k"] = s["k"][:, :, :512].contiguous()
    if what == "k of another type": change["k"] = s["k"].float()
    if what == "half": change.update(q=q.half(), k=s["k"].half())
    if what == "three dimensions": change.update(q=q[0], k=s["k"][0])
    if what == "scores not fp32": change["scores"] = s["scores"].to(torch.bfloat16)
    if what == "workspace too small": change["ws"] = s["ws"][:64]
    if what == "idx int64": change["idx"] = s["idx"].long()
    if what == "idx of another shape": change["idx"] = s["idx"].view(1, 1, 32, 3)
    if what == "cnt of another shape": change["cnt"] = s["cnt"].view(1, 1, 32)
    if what == "out of another shape": change["out"] = s["out"].view(1, 1, 2048, 64)
    if what == "out half": change["out"] = s["out"].half()
    if what == "seq_valid too large": nv = 1025
    if what == "seq_valid a string": nv = "all"
    if what == "k too large": change["keep"] = 17
    if what == "tokens not whole blocks": change.update(q=q[:, :, :1000].contiguous(), k=s["k"][:, :, :1000].contiguous())
    if what == "work order of another shape": change.update(ordered=True, wo=s["wo"].view(1, 1, 32))
    if what == "lse not fp32": change["use_lse"] = s["lse"].half()
    if what == "not a tensor": change["q"] = [1.0]
    if what == "head dimension": change.update(q=q[..., :32].contiguous(), k=s["k"][..., :32].contiguous())
    a, b, _ = both(monkeypatch, lambda: run(s, nv, **change))
    assert isinstance(a, tuple) and a == b, (a, b)
