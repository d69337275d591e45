"""Backward over blocks that a caller describes: every edge of the row offsets
counts, whatever the block's size words say of the edge count and however the
rows compare with its fan-out (the forward's mean reads them all)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU on this machine", allow_module_level=True)

import paper_2010_05337_amd as gmb  # noqa: E402
from gpu_util import csr_on_device, max_rel, to_torch_feats, to_torch_weights  # noqa: E402


@pytest.fixture(scope="module")
def graph(dg):
    return dg.rmat(15, 30_000, 250_000, (0.57, 0.19, 0.19), 9)


def described(blocks, fanout, nnz_word):
    """The same blocks with another fan-out and edge-count word."""
    s = gmb.BlocksStruct.from_buffer_copy(blocks.struct)
    keep = []
    for l, (n_dst, n_src, nnz) in enumerate(blocks.sizes()):
        words = torch.tensor([n_dst, n_src, nnz if nnz_word else 0, 0], dtype=torch.int32, device="cuda")
        keep.append(words)
        s.blk[l].sizes = words.data_ptr()
        if fanout is not None:
            s.blk[l].fanout = fanout
    out = gmb.Blocks(s, blocks.workspace, blocks.csr)
    out.keep = keep
    return out


@pytest.mark.parametrize("rows, fanouts", [(300, [12, 9]), (17_000, [16, 2])], ids=["cursors", "places"])
@pytest.mark.parametrize("fanout, nnz_word", [(None, False), (3, True), (1, False), (0, True)])
def test_every_edge_counts(orc, dg, graph, rows, fanouts, fanout, nnz_word):
    """Weight gradients and the embedding update against the same backward over
    the sampler's own description (fp32 sums of up to a few hundred terms in
    another order: 1e-5; the step is large so that the table's own rounding is
    not what is compared).  The workspace starts as entries that would show:
    destination 1, weight 1e6."""
    print(f"{rows} rows, fan-outs {fanouts} described as {fanout}, edge count {nnz_word}", flush=True)
    dims = [12, 8, 5]
    table_np = dg.features(graph.num_nodes, dims[0], 5, "f32")
    csr = csr_on_device(graph)
    seeds = torch.from_numpy(dg.permutation(graph.num_nodes, 7)[:rows]).cuda()
    y = torch.from_numpy(dg.labels(graph.num_nodes, dims[-1], 9)[seeds.cpu().numpy()]).cuda()
    w = to_torch_weights(dg.sage_weights(dims, 6))
    sampled = gmb.sample_blocks(csr, seeds, fanouts, 8)
    results = []
    for blocks in (sampled, described(sampled, fanout, nnz_word)):
        table = to_torch_feats(table_np)
        ws = gmb._aligned_bytes(gmb.forward_workspace_bytes(blocks, w), table.device)[1]
        logits, x_dst = gmb.sage_forward_fused(blocks, table, w, workspace=ws)
        need = (gmb.backward_embedding_workspace_bytes(blocks, w) + 7) // 8 * 8
        bws = gmb._aligned_bytes(need, table.device)[1]
        entry = np.array([1, np.float32(1e6).view(np.int32)], np.int32)
        bws.view(torch.int32).view(-1, 2).copy_(torch.from_numpy(entry).cuda())
        grads, loss = gmb.sage_backward(blocks, x_dst, w, logits, y, ws, workspace=bws, embedding=table,
                                        emb_lr=10.0 * rows)
        arrays = list(grads.d_self) + list(grads.d_neigh) + list(grads.d_bias)
        results.append([float(loss), table.cpu().numpy() - table_np] + [a.cpu().numpy() for a in arrays])
    csr.check_status()
    assert results[0][0] == results[1][0]
    errs = [max_rel(got, want) for want, got in zip(results[0][1:], results[1][1:])]
    assert max(errs) <= 1e-5, errs
