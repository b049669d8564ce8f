"""The Python binding rejects caller buffers of the wrong dtype, layout or size
before any device work (the C entry points take plain pointers and cannot check
sizes).  CPU only: the checks run on tensor metadata."""
import os
import subprocess
import sys

import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

cm = pytest.importorskip("paper_2508_15371_amd.cmsd")


def _f(*shape):
    return torch.zeros(*shape, dtype=torch.float32)


def _i(*shape):
    return torch.zeros(*shape, dtype=torch.int32)


def test_confidence_stats_buffer():
    x = _f(4, 100)
    with pytest.raises(ValueError, match="device"):
        cm.cmsd_confidence(x, _f(4, 8))           # sizes fine: only the device check fails
    with pytest.raises(ValueError, match="stats"):
        cm._buf(_f(3, 8), "stats", torch.float32, 32, x.device)
    with pytest.raises(ValueError, match="stats"):
        cm._buf(_f(8, 4).t(), "stats", torch.float32, 32, x.device)   # not contiguous
    with pytest.raises(ValueError, match="stats"):
        cm._buf(_i(4, 8), "stats", torch.float32, 32, x.device)
    cm._buf(_f(4, 8), "stats", torch.float32, 32, x.device)


def test_draft_len_buffers():
    with pytest.raises(ValueError, match="stats"):
        cm.cmsd_draft_len(_f(10, 8), 3, k_min=1, k_max=4, alpha=1.0, draft_len=_i(3), target_offsets=_i(4))
    with pytest.raises(ValueError, match="draft_len"):
        cm.cmsd_draft_len(_f(12, 8), 3, k_min=1, k_max=4, alpha=1.0, draft_len=_i(2), target_offsets=_i(4))
    with pytest.raises(ValueError, match="target_offsets"):
        cm.cmsd_draft_len(_f(12, 8), 3, k_min=1, k_max=4, alpha=1.0, draft_len=_i(3), target_offsets=_i(3))


def _verify(**kw):
    B, K, V, R = 3, 4, 50, 15
    a = dict(draft_logits=_f(B * K, V), draft_stats=_f(B * K, 8), target_logits=_f(R, V),
             target_offsets=_i(B + 1), draft_len=_i(B), drafted=_i(B * K), uniforms=_f(R),
             target_stats=_f(R, 8), n_accepted=_i(B), next_token=_i(B),
             workspace=torch.zeros(10000, dtype=torch.float64))
    a.update(kw)
    return cm.cmsd_verify(a.pop("draft_logits"), a.pop("draft_stats"), a.pop("target_logits"),
                          a.pop("target_offsets"), a.pop("draft_len"), a.pop("drafted"), a.pop("uniforms"),
                          batch=B, k_max=K, **a)


@pytest.mark.parametrize("name,bad", [
    ("draft_logits", _f(11, 50)), ("draft_stats", _f(11, 8)), ("target_offsets", _i(3)),
    ("draft_len", _i(2)), ("drafted", _i(11)), ("uniforms", _f(14)), ("target_stats", _f(14, 8)),
    ("n_accepted", _i(2)), ("next_token", _i(2)), ("drafted", torch.zeros(12, dtype=torch.int64)),
    ("workspace", torch.zeros(10000, dtype=torch.float32)),
])
def test_verify_buffers(name, bad):
    with pytest.raises(ValueError, match=name):
        _verify(**{name: bad})


def test_verify_sizes_ok_reach_device_check():
    with pytest.raises(ValueError, match="device"):
        _verify()


def test_draft_sample_buffers():
    x = _f(5, 70)
    with pytest.raises(ValueError, match="device"):
        cm.cmsd_draft_sample(x, _f(5, 8), _f(5), drafted=_i(5), workspace=torch.zeros(100, dtype=torch.float64))


def test_native_marshalling_leaves_the_rest_to_python():
    # built with the library; host tensors, missing or misfitting arguments and numbers of
    # another type are not its case: it answers None and the Python path checks and raises
    n = cm._native
    assert n is not None
    x, lam = _f(4, 100), (0.2, 0.5, 0.3)
    for args in ((x, _f(4, 8), lam, 1.0, 0), (x, None, lam, 1.0, 0), (x, _f(4, 8), list(lam), 1.0, 0),
                 (x, _f(4, 8), lam, 1, 0), (x, _f(4, 8), lam), (), (x, _f(4, 8), lam, 1.0, 0, 0)):
        assert n.confidence(*args) is None
    assert n.draft_len(3, 1, 4, 1.0, _f(12, 8), _i(3), _i(4), 0) is None
    assert n.draft_len(1 << 40, 1, 4, 1.0, _f(12, 8), _i(3), _i(4), 0) is None
    with pytest.raises(TypeError):
        n.bind(0)
    with pytest.raises(ValueError):
        n.bind(*[0] * 7)


class _Recorder:
    """The native module, with the answers of each of its functions kept."""

    def __init__(self, native):
        self._n, self.answers = native, {}

    def __getattr__(self, name):
        f = getattr(self._n, name)

        def call(*args):
            s = f(*args)
            self.answers.setdefault(name, []).append(s)
            return s
        return call


@pytest.mark.gpu
def test_native_marshalling_same_calls():
    # the same call through the native and the Python marshalling: every well-formed call is
    # the native one's case, equal outputs, and the same refusals (status and message) for
    # misfitting device buffers
    dev = torch.device("cuda:0")
    B, K, V = 3, 4, 500
    g = torch.Generator().manual_seed(0)
    dd, td = torch.randn(B * K, V, generator=g).to(dev), torch.randn(B * (K + 1), V, generator=g).to(dev)
    dr = torch.randint(0, V, (B * K,), generator=g, dtype=torch.int32).to(dev)
    u = torch.rand(B * (K + 1), generator=g).to(dev)
    ws, fws = cm.verify_workspace(B, K, V, dev), cm.fused_workspace(B, K, V, dev)

    def outputs():
        z = lambda t: t.to(dev)
        st, k, off, ts = z(_f(B * K, 8)), z(_i(B)), z(_i(B + 1)), z(_f(B * (K + 1), 8))
        na, nt, var, y = z(_i(B)), z(_i(B)), z(_f(B * K)), z(_i(B * K))
        cm.cmsd_confidence(dd, st)
        cm.cmsd_draft_len(st, B, k_min=K, k_max=K, alpha=1.0, draft_len=k, target_offsets=off)
        cm.cmsd_verify(dd, st, td, off, k, dr, u, batch=B, k_max=K, target_stats=ts, n_accepted=na, next_token=nt,
                       workspace=ws)
        cm.cmsd_confidence_var(dd, st, var)
        cm.cmsd_draft_sample(dd, st, u[:B * K].contiguous(), y,
                             torch.empty(cm.cmsd_draft_sample_workspace_bytes(B * K, V) // 8, dtype=torch.float64,
                                         device=dev))
        got = [st, k, off, ts, na, nt, var, y]
        for f, w in ((cm.cmsd_logit_pass, ws), (cm.cmsd_logit_pass_fused, fws)):
            o = f(dd, td, dr, u, batch=B, k_max=K, draft_stats=z(_f(B * K, 8)), draft_len=z(_i(B)),
                  target_stats=z(_f(B * (K + 1), 8)), n_accepted=z(_i(B)), next_token=z(_i(B)), workspace=w)
            got += [o[n] for n in ("draft_stats", "draft_len", "target_stats", "n_accepted", "next_token")]
            assert o["workspace"] is w
        # GREEDY without uniforms, on a stream of the caller's
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        greedy = dict(batch=B, k_max=K, mode=cm.CMSD_MODE_GREEDY, stream=side)
        gst, gts, gna, gnt = z(_f(B * K, 8)), z(_f(B * (K + 1), 8)), z(_i(B)), z(_i(B))
        side.wait_stream(torch.cuda.current_stream())
        cm.cmsd_confidence(dd, gst, stream=side)
        cm.cmsd_verify(dd, gst, td, off, k, dr, None, target_stats=gts, n_accepted=gna, next_token=gnt, workspace=ws,
                       **greedy)
        got += [gst, gts, gna, gnt]
        for f, w in ((cm.cmsd_logit_pass, ws), (cm.cmsd_logit_pass_fused, fws)):
            o = dict(draft_stats=z(_f(B * K, 8)), draft_len=z(_i(B)), target_stats=z(_f(B * (K + 1), 8)),
                     n_accepted=z(_i(B)), next_token=z(_i(B)))
            side.wait_stream(torch.cuda.current_stream())
            f(dd, td, dr, None, workspace=w, **o, **greedy)
            got += list(o.values())
        torch.cuda.synchronize()
        if isinstance(cm._native, _Recorder):
            answers = dict(cm._native.answers)
            assert set(answers) == {"confidence", "confidence_var", "draft_len", "draft_sample", "verify", "logit_pass",
                                    "logit_pass_fused"}
            assert all(s == cm.CMSD_OK for f in answers for s in answers[f]), answers
        errs = []
        for call in (lambda: cm.cmsd_confidence(dd, z(_f(2, 8))), lambda: cm.cmsd_confidence(dd.t(), st),
                     lambda: cm.cmsd_confidence(dd, st, beta_margin=-1.0),
                     lambda: cm.cmsd_draft_len(st, B, k_min=5, k_max=K, alpha=1.0, draft_len=k, target_offsets=off),
                     lambda: cm.cmsd_logit_pass(dd, td, dr, u, batch=B, k_max=K, draft_stats=st, draft_len=k,
                                                target_stats=ts, n_accepted=na, next_token=nt, workspace=ws[:1])):
            with pytest.raises(Exception) as e:
                call()
            errs.append((type(e.value), str(e.value)))
        return got, errs

    keep = cm._native
    assert keep is not None
    try:
        cm._native = _Recorder(keep)
        native, errs = outputs()
        cm._native = None
        plain, plain_errs = outputs()
    finally:
        cm._native = keep
    for a, b in zip(native, plain):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))
    assert errs == plain_errs


def test_build_without_a_host_compiler(tmp_path, monkeypatch):
    # the native marshalling is optional: no compiler means a warning and no module, and
    # not one of an earlier build either
    from paper_2508_15371_amd import build as B
    lib = tmp_path / "_binding.so"
    lib.write_bytes(b"of an earlier build")
    monkeypatch.setattr(B, "BINDING_LIB", str(lib))
    monkeypatch.setenv("CXX", str(tmp_path / "no-such-compiler"))
    with pytest.warns(RuntimeWarning, match="not built"):
        assert B.build_binding_if_possible() is False
    assert not lib.exists()


def test_missing_native_marshalling_is_said():
    # a module that cannot be imported is not passed over silently, and calls still work
    code = """
import sys, warnings, torch
class Block:
    def find_spec(self, name, path=None, target=None):
        if name.endswith("._binding"):
            raise ImportError("of another torch")
sys.meta_path.insert(0, Block())
with warnings.catch_warnings(record=True) as w:
    warnings.simplefilter("always")
    from paper_2508_15371_amd import cmsd
assert cmsd._native is None
assert any("of another torch" in str(x.message) and x.category is RuntimeWarning for x in w), w
try:
    cmsd.cmsd_confidence(torch.zeros(4, 100), torch.zeros(4, 8))
except ValueError as e:
    assert "device" in str(e)
else:
    raise SystemExit("no error")
"""
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
