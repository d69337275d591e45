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
    (256, 172, 1000), (320, 47, 5000), (513, 10, 200),
    # four waves per workgroup; a slab that leaves no LDS for the bias; a wide
    # tile of fewer tiles than CUs; no wider than the columns
    (640, 256, 17000), (602, 47, 20000), (640, 13, 65), (512, 172, 4000), (16, 47, 30000), (24, 16, 30000)])
def test_linear_bf16_widths(orc, dg, graph, d_in, d_out, rows):
    """One layer of d_in -> d_out over `rows` destinations (the 2e-2 of every
    bf16 forward: the mean is rounded to bf16)."""
    print(f"bf16 {d_in} -> {d_out}, {rows} rows", flush=True)
    feats = dg.features(graph.num_nodes, d_in, 5, "bf16")
    w = dg.sage_weights([d_in, d_out], 6, "bf16")
    _forward_case(orc, dg, graph, feats, w, dg.permutation(graph.num_nodes, 7)[:rows], [5], 8, TOL_BF16)


@pytest.mark.parametrize("dims", [[33, 47, 9], [640, 255, 41], [16, 26, 21]])
def test_bf16_hidden_rows_of_any_width(orc, dg, graph, dims):
    """bf16 rows whose width four does not divide: misaligned stores of four
    columns, the last columns one by one, nothing past a row's end.  (Of 640 ->
    255 -> 6, the rounding of the means and hidden rows alone, taken in 64 bits,
    moves one row whose six logits are all near zero by 2.6e-2; of 41 columns by
    less than 1e-2.  Narrow hidden rows do the same.)"""
    print(f"bf16 hidden {dims}", flush=True)
    feats = dg.features(graph.num_nodes, dims[0], 5, "bf16")
    w = dg.sage_weights(dims, 6, "bf16")
    _forward_case(orc, dg, graph, feats, w, dg.permutation(graph.num_nodes, 7)[:700], [5, 4], 8, TOL_BF16)


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


@pytest.mark.parametrize("d_in, d_out, rows", [(13, 255, 17001), (18, 255, 20000), (18, 41, 900), (33, 172, 20000),
                                               (75, 255, 17001), (125, 100, 20000), (127, 255, 20000), (125, 41, 2000),
                                               (253, 47, 3000)])
def test_linear_f32_error_is_no_larger_than_fp32_sums(dg, graph, d_in, d_out, rows):
    """Widths that four does not divide, on rows with many zeros (ReLU outputs):
    the error of the part products against 64 bits (2-norm) is no larger than
    that of a plain fp32 sum, one fused multiply-add after another."""
    print(f"f32 {d_in} -> {d_out}, {rows} rows", flush=True)
    w = to_torch_weights(dg.sage_weights([d_in, d_out], 6))
    seeds = torch.from_numpy(dg.permutation(graph.num_nodes, 7)[:rows]).cuda()
    blocks = gmb.sample_blocks(csr_on_device(graph), seeds, [5], 8)
    x = gmb.gather_features(blocks, to_torch_feats(dg.features(graph.num_nodes, d_in, 5, "f32"))).clamp_min(0)
    ws = gmb._aligned_bytes(gmb.forward_workspace_bytes(blocks, w), x.device)[1]
    got = gmb.sage_forward(blocks, x, w, workspace=ws).double()
    mean = ws[:4 * rows * d_in].view(torch.float32).view(rows, d_in)   # the first array of the workspace
    a = torch.cat((x[:rows], mean), 1).double()
    b = torch.cat((w.w_self[0], w.w_neigh[0])).double()
    bias = w.bias[0].double()
    want = a @ b + bias
    plain = torch.zeros((rows, d_out), device="cuda")
    for k in range(2 * d_in):   # products and sums of fp32 values are exact enough in 64 bits, then rounded once
        plain = (plain.double() + a[:, k:k + 1] * b[k]).float()
    plain = (plain.double() + bias).float().double()
    err, bound = (got - want).norm() / want.norm(), (plain - want).norm() / want.norm()
    print(f"error {float(err):.3e}, of a plain fp32 sum {float(bound):.3e}", flush=True)
    assert float(err) <= float(bound)


@pytest.mark.parametrize("d_in, d_out", [(9, 47), (16, 33), (17, 100), (31, 255), (33, 64), (63, 172), (64, 47)])
def test_linear_f32_tilings_agree(dg, graph, d_in, d_out):
    """The same rows in batches on either side of the line between the split
    tiles and the 128-row tiles: the same bits (d_in 16 and 64 by rows that are
    not 16-byte aligned)."""
    print(f"f32 {d_in} -> {d_out}", flush=True)
    cols = (d_out + 31) // 32
    rows = 16 * (1500 // cols + 1) + 5
    csr = csr_on_device(graph)
    w = to_torch_weights(dg.sage_weights([d_in, d_out], 6))
    seeds = torch.from_numpy(dg.permutation(graph.num_nodes, 7)[:rows]).cuda()

    def forward(s):
        blocks = gmb.sample_blocks(csr, s, [5], 8)
        x = gmb.gather_features(blocks, feats)
        odd = torch.empty(x.numel() + 1, device="cuda")[1:].view(x.shape)
        odd.copy_(x)
        return gmb.sage_forward(blocks, odd, w)
    feats = to_torch_feats(dg.features(graph.num_nodes, d_in, 5, "f32"))
    whole = forward(seeds)
    part = rows // 7
    for at in range(0, rows, part):
        assert torch.equal(whole[at:at + part], forward(seeds[at:at + part].contiguous())), at
    csr.check_status()


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


@pytest.mark.parametrize("dims, rows", [([9, 5], 70), ([75, 41], 700), ([130, 47], 2000), ([1, 4], 33),
                                        ([37, 16, 9], 129), ([128, 64, 10], 64)])
def test_bf16_weight_gradient_widths(orc, dg, graph, dims, rows):
    """Layer 0's weight gradient read from bf16 inputs and means, at widths
    that four does not divide: the last layer's gradients (a one-layer model:
    all of them, no ReLU in between) against the oracle's fp64 step within the
    bf16 training tests' 2e-2; lower layers against the same backward run in
    fp32 on the same values, where only the order of the transpose's sums may
    differ (1e-4, the fp32 training tests' bound)."""
    import ctypes
    print(f"bf16 training widths {dims}, {rows} rows", flush=True)
    fanouts = [4] * (len(dims) - 1)
    feats = dg.features(graph.num_nodes, dims[0], 5, "bf16")
    w = dg.sage_weights(dims, 6, "bf16")
    seeds = dg.permutation(graph.num_nodes, 7)[:rows]
    labels = dg.labels(graph.num_nodes, dims[-1], 9)[seeds]
    y = torch.from_numpy(labels).cuda()
    csr = csr_on_device(graph)
    wt = to_torch_weights(w)
    blocks = gmb.sample_blocks(csr, torch.from_numpy(seeds).cuda(), fanouts, 8)
    x = gmb.gather_features(blocks, to_torch_feats(feats))
    ws = gmb._aligned_bytes(gmb.forward_workspace_bytes(blocks, wt), x.device)[1]
    logits = gmb.sage_forward(blocks, x, wt, workspace=ws)
    grads, loss = gmb.sage_backward(blocks, x, wt, logits, y, ws)
    ref = orc.sample_blocks(graph.indptr, graph.indices, seeds, fanouts, 8)
    X = orc.widen(orc.gather(feats, ref[0].src), w.dtype)
    _, _, (dws, dwn, dbs), _ = orc.sage_train_step(ref, X, *w.as_f64(), labels, 0.1)
    for got, want in ((grads.d_self, dws), (grads.d_neigh, dwn), (grads.d_bias, dbs)):
        err = np.abs(got[-1].cpu().numpy() - want[-1]).max() / np.abs(want[-1]).max()
        assert err <= 2e-2, err
    # the same values in fp32: x, the weights, and the forward workspace with
    # its means and hidden outputs widened
    w32 = wt.master()
    ws32 = gmb._aligned_bytes(gmb.forward_workspace_bytes(blocks, w32), x.device)[1]
    gmb.sage_forward(blocks, x.float(), w32, workspace=ws32)
    sizes = blocks.sizes()

    def copy(dst_off, src_off, rows_, cols):
        src = ws[src_off:src_off + 2 * rows_ * cols].view(torch.bfloat16)
        ws32[dst_off:dst_off + 4 * rows_ * cols].view(torch.float32).copy_(src.float())

    at16 = at32 = 0
    for l in range(len(dims) - 1):   # the means come first, one per layer, 256-byte aligned
        cap = int(blocks.struct.blk[l].cap_dst)
        copy(at32, at16, sizes[l][0], dims[l])
        at16 += (2 * cap * dims[l] + 255) // 256 * 256
        at32 += (4 * cap * dims[l] + 255) // 256 * 256
    for l in range(len(dims) - 2):
        off16 = gmb.lib().gmb_forward_hidden_offset(ctypes.byref(blocks.struct), ctypes.byref(wt.struct), l)
        off32 = gmb.lib().gmb_forward_hidden_offset(ctypes.byref(blocks.struct), ctypes.byref(w32.struct), l)
        copy(off32, off16, sizes[l][0], dims[l + 1])
    grads32, _ = gmb.sage_backward(blocks, x.float(), w32, logits, y, ws32)
    for got, want in ((grads.d_self, grads32.d_self), (grads.d_neigh, grads32.d_neigh), (grads.d_bias, grads32.d_bias)):
        for a, b in zip(got, want):
            assert float((a - b).abs().max()) <= 1e-4 * float(b.abs().max())
    csr.check_status()


@pytest.mark.parametrize("rows", [16384, 16385])
def test_embedding_update_at_the_place_threshold(orc, dg, graph, rows):
    """The transpose of a block of 2^18 edges of capacity takes cursors in its
    fill, of more the places from the count: every updated embedding row and
    the untouched ones against the oracle's fp64 step (a one-layer model, no
    ReLU), within 1e-4 of the largest gradient (fp32 sums of a source's few
    hundred terms) plus the update's rounding."""
    print(f"{rows} rows", flush=True)
    dims, fanouts, lr = [12, 5], [16], 0.5
    table_np = dg.features(graph.num_nodes, dims[0], 5, "f32")
    table = to_torch_feats(table_np)
    w = dg.sage_weights(dims, 6)
    seeds = dg.permutation(graph.num_nodes, 7)[:rows]
    labels = dg.labels(graph.num_nodes, dims[-1], 9)[seeds]
    csr = csr_on_device(graph)
    wt = to_torch_weights(w)
    blocks = gmb.sample_blocks(csr, torch.from_numpy(seeds).cuda(), fanouts, 8)
    ws = gmb._aligned_bytes(gmb.forward_workspace_bytes(blocks, wt), table.device)[1]
    logits, x_dst = gmb.sage_forward_fused(blocks, table, wt, workspace=ws)
    gmb.sage_backward(blocks, x_dst, wt, logits, torch.from_numpy(labels).cuda(), ws, embedding=table, emb_lr=lr)
    ref = orc.sample_blocks(graph.indptr, graph.indices, seeds, fanouts, 8)
    ws_, wn_, bs_ = w.as_f64()
    _, _, dX, _, ref_table = orc.sage_train_step_embed(ref, table_np.astype(np.float64), ws_, wn_, bs_, labels, 0.1, lr)
    got = table.cpu().numpy()
    bound = lr * 1e-4 * np.abs(dX).max() + 2.0 ** -23 * np.abs(table_np).max()
    assert np.abs(got - ref_table).max() <= bound
    rest = np.ones(graph.num_nodes, bool)
    rest[ref[0].src] = False
    assert np.array_equal(got[rest], table_np[rest])
    csr.check_status()
