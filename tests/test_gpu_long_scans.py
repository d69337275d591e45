"""Scans of more than 1,024 tiles, which look back window by window (shorter ones
read all their predecessors at once): the relabel of a table hop and of owner
hops, and the transpose's scan."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU on this machine", allow_module_level=True)

from gpu_util import assert_blocks_equal, csr_on_device, gpu_blocks  # noqa: E402
import paper_2010_05337_amd as gmb  # noqa: E402


@pytest.fixture(scope="module")
def graph(dg):
    return dg.rmat(18, 250_000, 6_000_000, (0.45, 0.22, 0.22), 9)


@pytest.mark.parametrize("fanouts, num_seeds", [
    ([2, 64], 200_000),    # table hop: 4.8M edges in tiles of 4096, two values
    ([64], 100_000),       # owner hop: 1,563 routers, planned as 1,792
    ([2, 70], 70_000)])    # owner hop of two values: 1,207 routers, planned as 1,280
def test_relabel_of_many_tiles(orc, dg, graph, fanouts, num_seeds):
    print(f"fanouts {fanouts}, {num_seeds} seeds", flush=True)
    csr = csr_on_device(graph)
    seeds = dg.permutation(graph.num_nodes, 4)[:num_seeds]
    _, host = gpu_blocks(csr, seeds, fanouts, 3)
    ref = orc.sample_blocks(graph.indptr, graph.indices, seeds, fanouts, 3)
    if fanouts[-1] == 64 and len(fanouts) == 2:
        assert ref[1].nnz > 1024 * 4096
    assert_blocks_equal(host, ref)
    csr.check_status()
    assert bool((csr.state[256:256 + 4 * graph.num_nodes].view(torch.int32) == -1).all())


def test_transpose_of_many_sources(orc, dg):
    """1.5M sources, 1,502 tiles: the embedding update of a one-layer model
    against the oracle's fp64 step, within 1e-4 of the largest step (fp32 sums
    of a source's few terms) plus the update's rounding."""
    n, deg, rows, lr = 2_000_000, 8, 300_000, 3.0e4
    dims, fanouts = [4, 3], [deg]
    offsets = np.array([1, 77_777, 300_007, 555_555, 900_001, 1_234_567, 1_600_033, 1_999_993])
    indices = np.sort((np.arange(n)[:, None] + offsets) % n, axis=1).astype(np.int32).reshape(-1)

    class G:
        num_nodes, indptr = n, np.arange(0, n * deg + 1, deg, dtype=np.int64)
    G.indices = indices
    csr = csr_on_device(G)
    table_np = dg.features(n, dims[0], 5, "f32")
    table = torch.from_numpy(table_np).cuda()
    w = dg.sage_weights(dims, 6)
    wt = gmb.SageWeights(*([torch.from_numpy(a).cuda() for a in arrays] for arrays in (w.w_self, w.w_neigh, w.bias)))
    seeds = dg.permutation(n, 7)[:rows]
    labels = dg.labels(n, dims[-1], 9)[seeds]
    print("sampling", flush=True)
    blocks = gmb.sample_blocks(csr, torch.from_numpy(seeds).cuda(), fanouts, 8)
    ref = orc.sample_blocks(G.indptr, G.indices, seeds, fanouts, 8)
    assert ref[0].n_src > 1024 * 1024
    ws = gmb._aligned_bytes(gmb.forward_workspace_bytes(blocks, wt), table.device)[1]
    logits, x_dst = gmb.sage_forward_fused(blocks, table, wt, workspace=ws)
    print("backward", flush=True)
    gmb.sage_backward(blocks, x_dst, wt, logits, torch.from_numpy(labels).cuda(), ws, embedding=table, emb_lr=lr)
    got = table.cpu().numpy()
    csr.check_status()
    w64 = w.as_f64()
    _, _, dX, _, ref_table = orc.sage_train_step_embed(ref, table_np.astype(np.float64), *w64, labels, 0.1, lr)
    step = lr * np.abs(dX).max()
    assert step > 0.1   # the steps are far above the table's rounding
    assert np.abs(got - ref_table).max() <= 1e-4 * step + 2.0 ** -23 * (np.abs(table_np).max() + step)
    rest = np.ones(n, bool)
    rest[ref[0].src] = False
    assert np.array_equal(got[rest], table_np[rest])
