"""The mean's backward when a wait of the transpose's scan runs out: the input
gradients, or the embedding update, of that call are unknown, and the call
says so.  The wait is made to run out from the host: the ticket counter
starts at 1, so no workgroup takes tile 0, and the spin limit is small (every
wait ends; the buffers hold the tile past the last one)."""
import ctypes
import subprocess

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU on this machine", allow_module_level=True)

import paper_2010_05337_amd as gmb  # noqa: E402

TICKET_WORDS = 32   # the scan's state: the ticket's line, two words, 2 words per tile
N_DST, N_SRC, CAP_SRC, D, FANOUT, LR = 4, 2048, 4096, 4, 3, 0.5


def launch_mean_backward():
    lib = gmb.lib()
    names = subprocess.check_output(["nm", "-D", "--defined-only", gmb.LIB_PATH], text=True)
    name, = [l.split()[-1] for l in names.splitlines() if "launch_mean_backward" in l]
    f = getattr(lib, name)
    f.restype = ctypes.c_int
    vp, i64, i32 = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int
    f.argtypes = [vp, vp, vp, i64, i32, vp, vp, i32, i32, vp, i64, i64, vp, vp, vp, vp, vp, vp, vp, vp, vp, i64,
                  ctypes.c_float, vp, vp, vp, vp, i32]
    return f


@pytest.mark.parametrize("table", [False, True], ids=["rows", "table"])
@pytest.mark.parametrize("runs_out", [False, True])
def test_a_scan_wait_that_runs_out_is_reported(table, runs_out):
    print(f"table {table}, runs out {runs_out}", flush=True)
    rng = np.random.default_rng(3)
    local = np.array([0, 5, 1500, 1, 1500, 2047, 2, 1024, 1023, 3, 5], np.int32)
    indptr = np.array([0, 3, 6, 9, 11], np.int32)
    dm = rng.standard_normal((N_DST, D)).astype(np.float32)
    dh = rng.standard_normal((CAP_SRC, D)).astype(np.float32)
    emb = rng.standard_normal((N_SRC, D)).astype(np.float32)
    want = np.zeros((N_SRC, D))
    want[:N_DST] = dh[:N_DST]
    for v in range(N_DST):
        for e in range(indptr[v], indptr[v + 1]):
            want[local[e]] += dm[v] / np.float64(indptr[v + 1] - indptr[v])
    want_emb = emb - LR * want
    dev = "cuda"

    def ints(a, n=None):
        t = torch.zeros(n or len(a), dtype=torch.int32, device=dev)
        t[:len(a)] = torch.from_numpy(np.asarray(a, np.int32)).to(dev)
        return t
    sizes, ip, lo = ints([N_DST, N_SRC, len(local), 0]), ints(indptr), ints(local)
    cnt = ints(np.bincount(local, minlength=N_SRC), CAP_SRC)
    off, pos, long_rows = ints([], CAP_SRC + 1), ints([], CAP_SRC), ints([], CAP_SRC)
    state = ints([1 if runs_out else 0], TICKET_WORDS + 2 + 2 * (CAP_SRC // 1024))
    csc, ids = ints([], 2 * len(local)), ints(np.arange(N_SRC))
    m, h, t = (torch.from_numpy(a).to(dev) for a in (dm, dh, emb))
    out, report = torch.ones((CAP_SRC, D), device=dev), torch.full((1,), 2.5, device=dev)
    p = lambda x: x.data_ptr()   # noqa: E731
    rc = launch_mean_backward()(
        p(sizes), p(ip), p(lo), len(local), FANOUT, p(m), p(out), 0, D, p(h), N_DST, CAP_SRC, p(cnt), p(off), p(pos),
        None, p(state), p(csc), p(long_rows), p(t) if table else None, p(ids), N_SRC, LR, None, None, p(report),
        torch.cuda.current_stream().cuda_stream, 200 if runs_out else 0)
    assert rc == 0
    torch.cuda.synchronize()
    if runs_out:
        assert torch.isnan(report).all()
        if table:
            assert np.array_equal(t.cpu().numpy(), emb)
        else:
            assert torch.isnan(h[:N_SRC]).all()
        return
    assert float(report) == 2.5
    got, ref = (t.cpu().numpy(), want_emb) if table else (h[:N_SRC].cpu().numpy(), want)
    # sums of at most four fp32 terms of size about 1, and the update's rounding
    assert np.abs(got - ref).max() <= 8 * 2.0 ** -23 * max(1.0, np.abs(ref).max())
