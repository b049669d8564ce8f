"""GPU parity of cmsd_confidence (Sec. III.B(1)) against the oracle, through the C ABI."""
import math

import numpy as np
import pytest
import torch

import workloads as W
from oracle import cmsd_oracle as O
from tests import harness as Hn

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2508_15371_amd import cmsd
    return cmsd


def _invariant_rows(V: int, g: np.random.Generator) -> list:
    rows = []
    rows.append(np.full(V, 0.5))                                  # uniform
    z = np.full(V, -math.inf); z[g.integers(0, V)] = 1.0; rows.append(z)     # one-hot, masked
    z = np.full(V, -800.0); z[V - 1] = 0.0; rows.append(z)        # one-hot by a huge gap
    for d in (0.0, 0.5, 3.0):                                     # two finite logits
        z = np.full(V, -math.inf); z[0] = 2.0 + d; z[V // 2] = 2.0; rows.append(z)
    z = g.integers(-2, 2, V).astype(np.float64); rows.append(z)  # heavy ties
    z = g.normal(0, 3, V); z[g.random(V) < 0.3] = -math.inf; z[int(np.argmax(z))] = 9.0; rows.append(z)
    z = g.normal(0, 1, V); z[[3 % V, (V - 2) % V]] = 7.0; rows.append(z)      # duplicate max
    rows.append(g.normal(0, 0.01, V))                            # nearly flat
    rows.append(g.normal(0, 20, V))                              # very sharp
    z = g.normal(0, 1, V); z[V - 1] = 30.0; rows.append(z)        # max in the tail
    return rows


def _store(rows, dtype):
    x = np.stack(rows).astype(np.float32)
    return x if dtype == "f32" else W.bf16_bits_from_f32(x)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("V", [2, 3, 7, 8, 9, 31, 255, 1023, 1024, 1025, 4099, 32000, 50257, 131072 + 17])
@pytest.mark.parametrize("pad", [0, 5])
def test_invariant_rows(cm, dtype, V, pad):
    g = np.random.default_rng(V * 7 + pad)
    stored = _store(_invariant_rows(V, g), dtype)
    n = stored.shape[0]
    buf = np.zeros((n, V + pad), dtype=stored.dtype)
    buf[:, :V] = stored
    dev = torch.device("cuda:0")
    tdev = Hn.to_device(buf, dtype, dev)[:, :V]
    lam = (0.2, 0.5, 0.3)
    st = cm.cmsd_confidence(tdev, lambdas=lam, beta_margin=0.7)
    torch.cuda.synchronize()
    gs = Hn.stats_np(st)
    t = Hn.Tally()
    lam32 = tuple(Hn.f32(x) for x in lam)
    for r in range(n):
        Hn.check_row_stats(t, gs, r, Hn.decode(stored[r], dtype), V, lam32, Hn.f32(0.7))
    t.assert_ok()


@pytest.mark.parametrize("block", [64, 128, 256])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("V", [9, 1025, 50257])
def test_each_row_block(cm, row_shape, block, dtype, V):
    # every workgroup size the library may pick for a launch (forced by cmsd_set_row_shape)
    row_shape(block)
    g = np.random.default_rng(V + block)
    stored = _store(_invariant_rows(V, g), dtype)
    tdev = Hn.to_device(stored, dtype, torch.device("cuda:0"))
    st = cm.cmsd_confidence(tdev, lambdas=(0.2, 0.5, 0.3), beta_margin=0.7)
    torch.cuda.synchronize()
    gs = Hn.stats_np(st)
    t = Hn.Tally()
    lam32 = tuple(Hn.f32(x) for x in (0.2, 0.5, 0.3))
    for r in range(stored.shape[0]):
        Hn.check_row_stats(t, gs, r, Hn.decode(stored[r], dtype), V, lam32, Hn.f32(0.7))
    t.assert_ok()


@pytest.mark.parametrize("depth", [2, 3])
@pytest.mark.parametrize("block", [64, 128, 256])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_rounds_across_the_ring(cm, row_shape, block, dtype, depth):
    # a row streams in rounds of 32 elements per thread with `depth` rounds of loads in
    # flight: rows of 1..9 full rounds (plus a partial round, a tail and an unaligned
    # head) take the ring's main loop zero or more times and leave depth..2*depth-1
    # rounds (or the whole row) to its guarded last part
    row_shape(block, depth)
    lam = (0.2, 0.5, 0.3)
    lam32 = tuple(Hn.f32(x) for x in lam)
    for nr in range(1, 10):
        V = 32 * block * nr + 37
        g = np.random.default_rng(nr * 1000 + block)
        rows = _invariant_rows(V, g)[:4] + [g.normal(0, 2, V)]
        stored = _store(rows, dtype)
        buf = np.zeros((stored.shape[0], V + 3), dtype=stored.dtype)
        buf[:, 3:] = stored                     # rows start 3 elements into their stride
        tdev = Hn.to_device(buf, dtype, torch.device("cuda:0"))[:, 3:]
        st = cm.cmsd_confidence(tdev, lambdas=lam, beta_margin=0.7)
        torch.cuda.synchronize()
        gs = Hn.stats_np(st)
        t = Hn.Tally()
        for r in range(stored.shape[0]):
            Hn.check_row_stats(t, gs, r, Hn.decode(stored[r], dtype), V, lam32, Hn.f32(0.7))
        t.assert_ok()


@pytest.mark.parametrize("depth", [2, 3])
@pytest.mark.parametrize("block", [64, 256])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_round_edges_between_nans(cm, row_shape, block, dtype, depth):
    # rows whose vectors end on, one before and one after the edge of a round, for every
    # count of rounds the ring can be left with, between NaNs: a head, a tail or a vector
    # taken one element past a row's ends would make its sums NaN.  (That the loads
    # themselves stop at the row is test_gpu_row_rounds.py's: their lanes past it are
    # replaced before the sums, whatever they loaded.)
    row_shape(block, depth)
    lam = (0.2, 0.5, 0.3)
    lam32 = tuple(Hn.f32(x) for x in lam)
    vec = 4 if dtype == "f32" else 8
    for nr in range(0, 2 * depth + 2):
        for edge in (-1, 0, 1):
            V = 32 * block * nr + vec * edge + (1 if nr % 2 else 0)     # odd: a tail element
            if V < 2:
                continue
            g = np.random.default_rng(nr * 10 + edge + block)
            rows = np.stack([g.normal(0, 2, V), g.normal(0, 0.1, V) - 50.0]).astype(np.float32)
            buf32 = np.full((2, V + 16), np.nan, dtype=np.float32)
            for head in (0, 5):                                        # aligned, and with a head
                buf32[:] = np.nan
                buf32[:, head:head + V] = rows
                buf = buf32 if dtype == "f32" else W.bf16_bits_from_f32(buf32)
                tdev = Hn.to_device(buf, dtype, torch.device("cuda:0"))[:, head:head + V]
                st = cm.cmsd_confidence(tdev, lambdas=lam, beta_margin=0.7)
                torch.cuda.synchronize()
                gs = Hn.stats_np(st)
                t = Hn.Tally()
                for r in range(2):
                    Hn.check_row_stats(t, gs, r, Hn.decode(np.ascontiguousarray(buf[r, head:head + V]), dtype), V,
                                       lam32, Hn.f32(0.7))
                t.assert_ok()


def _sample_rows(cfg, k):
    n = cfg.draft_rows
    if n <= k:
        return list(range(n))
    g = np.random.default_rng(cfg.cid)
    return sorted(set([0, n - 1] + g.choice(n, k, replace=False).tolist()))


@pytest.mark.parametrize("name,nsample", [("tiny", 99), ("c2", 99), ("c3", 512), ("c4", 40), ("c5", 48), ("v152k", 40)])
def test_config_rows(cm, name, nsample):
    cfg = W.CONFIGS[name]
    print(f"[confidence parity] {name}", flush=True)
    d = Hn.workload(name, 0)
    dev = torch.device("cuda:0")
    draft = d["draft_dev"]
    st = cm.cmsd_confidence(draft)
    torch.cuda.synchronize()
    gs = Hn.stats_np(st)
    t = Hn.Tally()
    lam = tuple(Hn.f32(1 / 3) for _ in range(3))
    for r in _sample_rows(cfg, nsample):
        Hn.check_row_stats(t, gs, r, Hn.decode(d["draft"][r], cfg.dtype), cfg.V, lam, 1.0)
    t.assert_ok()


def test_repeat_bitwise_identical(cm):
    d = Hn.workload("c3", 0)
    a = cm.cmsd_confidence(d["draft_dev"]).clone()
    b = cm.cmsd_confidence(d["draft_dev"]).clone()
    torch.cuda.synchronize()
    assert torch.equal(a.view(torch.int32), b.view(torch.int32))


def test_empty_and_errors(cm):
    dev = torch.device("cuda:0")
    x = torch.zeros((0, 100), device=dev)
    st = cm.cmsd_confidence(x)
    assert st.shape == (0, 8)
    with pytest.raises(cm.CmsdError):
        cm.cmsd_confidence(torch.zeros((4, 1), device=dev))            # V < 2
    with pytest.raises(cm.CmsdError):
        cm.cmsd_confidence(torch.zeros((4, 16), device=dev), lambdas=(0.5, 0.5, 0.5))


def _check_var(got, ref, what):
    assert abs(got - ref) <= 1e-4 * max(abs(ref), 1e-2), (what, got, ref)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("V", [2, 9, 1025, 4099, 50257, 131072 + 17])
@pytest.mark.parametrize("pad", [0, 5])
def test_logit_variance_rows(cm, dtype, V, pad):
    # cmsd_confidence_var: the same stats as cmsd_confidence, and the variance of the
    # finite logits against the oracle's two-pass definition (Sec. I proxy)
    g = np.random.default_rng(V * 3 + pad)
    rows = _invariant_rows(V, g)
    rows.append(1000.0 + g.normal(0, 1, V))                      # large common offset
    z = g.normal(0, 0.3, V); z[g.integers(0, V)] += 15.0; rows.append(z)   # near-one-hot
    stored = _store(rows, dtype)
    n = stored.shape[0]
    buf = np.zeros((n, V + pad), dtype=stored.dtype)
    buf[:, :V] = stored
    tdev = Hn.to_device(buf, dtype, torch.device("cuda:0"))[:, :V]
    st, var = cm.cmsd_confidence_var(tdev, lambdas=(0.2, 0.5, 0.3), beta_margin=0.7)
    st0 = cm.cmsd_confidence(tdev, lambdas=(0.2, 0.5, 0.3), beta_margin=0.7)
    torch.cuda.synchronize()
    assert torch.equal(st.view(torch.int32), st0.view(torch.int32))
    var = var.cpu().numpy()
    for r in range(n):
        _check_var(float(var[r]), O.logit_variance(Hn.decode(stored[r], dtype)), (r, V, dtype))


@pytest.mark.parametrize("block", [64, 128, 256])
def test_logit_variance_each_row_block(cm, row_shape, block):
    row_shape(block)
    g = np.random.default_rng(block)
    V = 20011
    stored = _store(_invariant_rows(V, g), "bf16")
    tdev = Hn.to_device(stored, "bf16", torch.device("cuda:0"))
    _, var = cm.cmsd_confidence_var(tdev)
    torch.cuda.synchronize()
    var = var.cpu().numpy()
    for r in range(stored.shape[0]):
        _check_var(float(var[r]), O.logit_variance(Hn.decode(stored[r], "bf16")), (r, block))


@pytest.mark.parametrize("name,nsample", [("c3", 64), ("c4", 24), ("c5", 24)])
def test_logit_variance_config_rows(cm, name, nsample):
    cfg = W.CONFIGS[name]
    d = Hn.workload(name, 0)
    _, var = cm.cmsd_confidence_var(d["draft_dev"])
    torch.cuda.synchronize()
    var = var.cpu().numpy()
    for r in _sample_rows(cfg, nsample):
        _check_var(float(var[r]), O.logit_variance(Hn.decode(d["draft"][r], cfg.dtype)), (name, r))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_many_short_rows(cm, dtype):
    # more rows than the chip holds workgroups at once (one-wave groups); odd V and a
    # padded stride make consecutive rows start at different alignments
    g = np.random.default_rng(77)
    n, V, pad = 20011, 37, 3
    z = g.normal(0, 2, (n, V))
    z[::7, ::5] = -math.inf                       # masked entries on some rows
    z[::11, 4] = z[::11].max(axis=1) + 1.0         # a clear max on others
    z[::13, 9] = z[::13, 4]                        # ties with it
    stored = _store(list(z), dtype)
    buf = np.zeros((n, V + pad), dtype=stored.dtype)
    buf[:, :V] = stored
    tdev = Hn.to_device(buf, dtype, torch.device("cuda:0"))[:, :V]
    st, var = cm.cmsd_confidence_var(tdev, lambdas=(0.2, 0.5, 0.3), beta_margin=0.7)
    st0 = cm.cmsd_confidence(tdev, lambdas=(0.2, 0.5, 0.3), beta_margin=0.7)
    torch.cuda.synchronize()
    assert torch.equal(st.view(torch.int32), st0.view(torch.int32))
    gs = Hn.stats_np(st)
    var = var.cpu().numpy()
    t = Hn.Tally()
    lam32 = tuple(Hn.f32(x) for x in (0.2, 0.5, 0.3))
    for r in range(0, n, 3):
        zr = Hn.decode(stored[r], dtype)
        Hn.check_row_stats(t, gs, r, zr, V, lam32, Hn.f32(0.7))
        _check_var(float(var[r]), O.logit_variance(zr), r)
    t.assert_ok()


def test_rows_past_one_launch_grid(cm):
    # more rows than one confidence launch's grid of 2^22 workgroups: the kernel's loop
    # over rows takes the rest, with and without the variance moment.  Rows on both
    # sides of the grid's end and a random sample, at alternating 16-byte alignments (5
    # bf16 logits per row), some masked.
    g = np.random.default_rng(4242)
    n, V = (1 << 22) + 37, 5
    z = g.normal(0, 2, (n, V)).astype(np.float32)
    z[::9, 2] = -np.inf
    stored = W.bf16_bits_from_f32(z)
    tdev = Hn.to_device(stored, "bf16", torch.device("cuda:0"))
    st = cm.cmsd_confidence(tdev, lambdas=(0.2, 0.5, 0.3), beta_margin=0.7)
    st_v, var = cm.cmsd_confidence_var(tdev, lambdas=(0.2, 0.5, 0.3), beta_margin=0.7)
    torch.cuda.synchronize()
    assert torch.equal(st.view(torch.int32), st_v.view(torch.int32))
    gs = Hn.stats_np(st)
    var = var.cpu().numpy()
    rows = set(range(0, 8)) | set(range((1 << 22) - 8, n)) | set(g.choice(n, 300, replace=False).tolist())
    t = Hn.Tally()
    lam32 = tuple(Hn.f32(x) for x in (0.2, 0.5, 0.3))
    for r in sorted(rows):
        zr = Hn.decode(stored[r], "bf16")
        Hn.check_row_stats(t, gs, r, zr, V, lam32, Hn.f32(0.7))
        _check_var(float(var[r]), O.logit_variance(zr), r)
    t.assert_ok()
