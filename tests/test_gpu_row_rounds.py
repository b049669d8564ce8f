"""The row kernels load whole rounds of vectors, the last one past the row's end and the
ring's refills past its last round: the buffer descriptor's range check must end each at
the row.  Shown by the loads alone (csrc/row_buffer.h, through the probe library) on a
patterned buffer that holds every round, so that no load leaves it whatever the check does."""
import ctypes as C
import re
import subprocess

import pytest

torch = pytest.importorskip("torch")
B = pytest.importorskip("paper_2508_15371_amd.build")


def _probe():
    f = C.CDLL(B.PROBE_LIB).cmsd_probe_row_rounds
    i64, vp = C.c_int64, C.c_void_p
    f.argtypes = [vp, i64, i64, C.c_int, C.c_int, C.c_int, vp, i64, vp]
    f.restype = C.c_int
    return f


def test_probe_checks_its_arguments():
    f, p = _probe(), C.c_void_p(4096)
    n = 3 * 4 * 64
    assert f(p, n, 1, 3, 96, 4, p, n, None) == 1           # workgroup size
    assert f(p, n, 1, 3, 64, 5, p, n, None) == 1           # vectors per thread
    assert f(p, n, 1, 0, 64, 4, p, n, None) == 1           # no round
    assert f(p, n - 1, 1, 3, 64, 4, p, n, None) == 1       # a buffer that ends before the rounds do
    assert f(p, n, 1, 3, 64, 4, p, n - 1, None) == 1
    assert f(p, n, n + 1, 3, 64, 4, p, n, None) == 1       # a row past them
    assert f(C.c_void_p(4104), n, 1, 3, 64, 4, p, n, None) == 1
    assert f(None, n, 1, 3, 64, 4, p, n, None) == 1


def test_positions_are_lane_offsets(tmp_path):
    # the range check covers a lane's own offset and the instruction's, not by contract a
    # scalar offset: no load of a round may carry one
    out = tmp_path / "probe.s"
    r = subprocess.run([B.hipcc(), f"--offload-arch={B.ARCH}", *[f for f in B.FLAGS if f != "-shared"],
                        "--cuda-device-only", "-S", "-o", str(out), B.PROBE_SRC], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    loads = re.findall(r"^\s*buffer_load_dwordx4 .*$", out.read_text(), re.M)
    assert len(loads) >= 6 * 4                              # every shape's first vectors at least
    for l in loads:
        assert re.search(r"s\[\d+:\d+\], 0 offen( offset:\d+)? nt", l), l


@pytest.mark.gpu
@pytest.mark.parametrize("bd", [64, 128, 256])
@pytest.mark.parametrize("u", [4, 8])
def test_rounds_end_at_the_row(bd, u):
    # a round whose records end in each of its vectors' spans (and none, so that every
    # vector of a round lies past them), two rounds past the row and a full one before it
    f = _probe()
    dev = torch.device("cuda:0")
    rounds, per = 4, u * bd
    x = torch.randint(1, 1 << 30, (rounds * per, 4), dtype=torch.int32, device=dev)
    out = torch.empty_like(x)
    edges = sorted({max(0, min(2 * per, r * per + s * bd + e)) for r in (0, 1) for s in range(u + 1) for e in (-1, 0, 1)})
    for nvec in edges:
        out.fill_(-1)
        st = torch.cuda.current_stream().cuda_stream
        assert f(x.data_ptr(), x.shape[0], nvec, rounds, bd, u, out.data_ptr(), out.shape[0], st) == 0
        torch.cuda.synchronize()
        assert torch.equal(out[:nvec], x[:nvec]), (bd, u, nvec)
        assert not out[nvec:].any(), (bd, u, nvec)
