"""The linear layers at the sizes where their kernels change: widths that no
vector load divides, the last group of eight k overlapping the one before,
ragged row and column tiles, every column width of the slab."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU on this machine", allow_module_level=True)

import paper_2010_05337_amd as gmb  # noqa: E402
from gpu_util import csr_on_device, to_torch_feats, to_torch_weights  # noqa: E402
from test_gpu_parity import TOL_BF16, TOL_F32, _forward_case  # noqa: E402


@pytest.fixture(scope="module")
def graph(dg):
    return dg.rmat(15, 30_000, 250_000, (0.57, 0.19, 0.19), 9)


@pytest.mark.parametrize("d_in, d_out, rows", [
    (8, 5, 1), (9, 7, 127), (75, 41, 300), (33, 130, 4000), (250, 255, 17001), (128, 256, 17000), (31, 64, 9000),
    (256, 172, 1000), (320, 47, 5000), (513, 10, 200)])
def test_linear_bf16_widths(orc, dg, graph, d_in, d_out, rows):
    """One layer of d_in -> d_out over `rows` destinations (the 2e-2 of every
    bf16 forward: the mean is rounded to bf16)."""
    print(f"bf16 {d_in} -> {d_out}, {rows} rows", flush=True)
    feats = dg.features(graph.num_nodes, d_in, 5, "bf16")
    w = dg.sage_weights([d_in, d_out], 6, "bf16")
    _forward_case(orc, dg, graph, feats, w, dg.permutation(graph.num_nodes, 7)[:rows], [5], 8, TOL_BF16)


@pytest.mark.parametrize("d_in, d_out, rows", [
    (3, 5, 100), (9, 7, 127), (10, 300, 333), (75, 41, 2600), (101, 64, 4000), (75, 256, 17001), (125, 255, 17000),
    (250, 130, 3000), (255, 33, 17)])
def test_linear_f32_widths(orc, dg, graph, d_in, d_out, rows):
    """One fp32 layer whose input width four does not divide: the part
    products with each half padded to groups of eight (3: the general
    kernel), every tiling; fp32-level accuracy as for the other widths."""
    print(f"f32 {d_in} -> {d_out}, {rows} rows", flush=True)
    feats = dg.features(graph.num_nodes, d_in, 5, "f32")
    w = dg.sage_weights([d_in, d_out], 6)
    errs = _forward_case(orc, dg, graph, feats, w, dg.permutation(graph.num_nodes, 7)[:rows], [5], 8, TOL_F32)
    assert max(errs) <= 5e-6, errs


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d_in", [9, 75, 101])
def test_linear_infinities_stay_in_their_element(dg, graph, dtype, d_in):
    """An infinite feature gives infinities of its weights' signs, no NaN, at
    every position (the elements that two groups of the reduction read, too).
    No edges: the mean is zero."""
    n, d_out = 40, 20

    class G:
        num_nodes, indptr, indices = 128, np.zeros(129, np.int64), np.zeros(0, np.int32)
    feats = to_torch_feats(dg.features(128, d_in, 3, dtype))
    seeds = torch.arange(n, dtype=torch.int32, device="cuda")
    for i in range(n):
        feats[i, i % d_in] = float("inf") if i % 3 else float("-inf")
    w = to_torch_weights(dg.sage_weights([d_in, d_out], 6, dtype))
    blocks = gmb.sample_blocks(csr_on_device(G), seeds, [5], 1)
    x = gmb.gather_features(blocks, feats)
    out = gmb.sage_forward(blocks, x, w).cpu()
    wm = w.w_self[0].float().cpu()
    for i in range(n):
        want = torch.sign(wm[i % d_in]) * (float("inf") if i % 3 else float("-inf"))
        assert torch.equal(out[i], want), i


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d", [1, 2, 3, 4, 5, 7, 8, 9, 15, 17, 33, 63, 75, 101, 130, 257, 300])
def test_rows_of_any_width(orc, dg, graph, dtype, d):
    """Gathered rows bit for bit, also from a table and into a buffer whose
    addresses are multiples of the element size only, with nothing written
    past the last row; the fused forward (means from the same table) equal to
    the three calls'."""
    feats = dg.features(graph.num_nodes, d, 5, dtype)
    ft = to_torch_feats(feats)
    odd = torch.empty(ft.numel() + 1, dtype=ft.dtype, device="cuda")[1:].view(ft.shape)
    odd.copy_(ft)
    ids = torch.from_numpy(dg.permutation(graph.num_nodes, 3)[:1001]).cuda()
    want = ft[ids.long()]
    out = torch.full((1002 * d + 1,), 7.0, dtype=ft.dtype, device="cuda")
    gmb.gather_features(ids, odd, out=out[1:1 + 1002 * d].view(1002, d))
    bits = torch.int16 if dtype == "bf16" else torch.int32
    assert torch.equal(out[1:1 + 1001 * d].view(bits), want.view(-1).view(bits))
    assert bool((out[1 + 1001 * d:] == 7).all()) and float(out[0]) == 7
    csr = csr_on_device(graph)
    w = to_torch_weights(dg.sage_weights([d, 12], 6, dtype))
    blocks = gmb.sample_blocks(csr, ids, [6], 5)
    logits = gmb.sage_forward(blocks, gmb.gather_features(blocks, odd), w)
    fused, x_dst = gmb.sage_forward_fused(blocks, odd, w)
    assert torch.equal(fused, logits)
    assert torch.equal(x_dst[:1001].view(bits), want.view(bits))
    csr.check_status()
