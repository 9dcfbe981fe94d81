"""GPU parity of the kernels that the automatic choice picks by size, at the
sizes where they can go wrong: partial last tiles in rows and columns, tiles
that span images, single images, split ranges of every K group, and the
smallest shapes that reach each kernel. Every configuration runs through the
operator entry points against the oracle (tolerances as in test_gpu_ops: the
rounding of the storage type, 1e-5 for fp32 sums)."""
import numpy as np
import pytest

from paper_2509_26092_amd import binding as B
import test_gpu_ops as op

pytestmark = pytest.mark.gpu


def forced(cfg, fn, *args):
    try:
        B.rn18_debug_set(None, B.RN18_DBG_GATHER_CONFIG, cfg)
        fn(*args)
    finally:
        B.rn18_debug_set(None, B.RN18_DBG_GATHER_CONFIG, 0)


# (N, Cin, Cin_padded, H, W, Cout, k, s, p)
@pytest.mark.parametrize("case", [
    (2, 64, 64, 28, 28, 128, 3, 1, 1),      # 9-row tiles, the last of 2 rows, one tile over both images
    (5, 128, 128, 7, 7, 192, 3, 1, 1),      # one tile of five whole images, a column tile of 64
    (6, 64, 64, 7, 7, 136, 3, 1, 1),        # ... and a sixth image alone, a column tile of 8
    (3, 64, 64, 14, 14, 128, 3, 1, 1),      # tiles that start inside an image and cross two borders
    (1, 192, 192, 16, 16, 256, 3, 1, 1),    # one tile exactly, three channel blocks, two column tiles
    (2, 64, 64, 9, 48, 128, 3, 1, 1),       # five rows per tile at the widest patch
    (3, 64, 64, 5, 51, 72, 3, 1, 1),        # 204-pixel tiles over image borders, odd width
], ids=op.case_id)
@pytest.mark.parametrize("direction", [op.test_conv_fwd, op.test_conv_dgrad], ids=["fwd", "dgrad"])
def test_wide_halo(case, direction):
    """The wide halo kernel (16-bit, whole channel blocks, more than 64
    columns); the data gradient runs it where its own columns (the input
    channels) exceed 64."""
    forced(34, direction, "bf16", case)


@pytest.mark.parametrize("direction", [op.test_conv_fwd, op.test_conv_dgrad], ids=["fwd", "dgrad"])
def test_more_column_tiles_than_compute_units(direction):
    """One 16x16 image whose columns make one 128-column tile more than there
    are compute units (a block of the wide halo kernel keeps its columns, so
    that kernel cannot take it): launched by another kernel, not refused."""
    import torch
    wide = 128 * torch.cuda.get_device_properties(0).multi_processor_count + 8
    cin, cout = (64, wide) if direction is op.test_conv_fwd else (wide, 64)
    direction("bf16", (1, cin, cin, 16, 16, cout, 3, 1, 1))


@pytest.mark.parametrize("cfg", [4, 5, 6, 8, 10, 11, 12, 17, 18, 19, 20, 21, 22])
@pytest.mark.parametrize("case", [
    (1, 64, 64, 3, 3, 72, 3, 1, 1),         # 9 rows in any tile, 72 columns
    (2, 64, 64, 16, 15, 264, 1, 1, 0),      # one K stage (fewer than any ring holds), 264 columns
    (3, 32, 32, 13, 12, 128, 3, 1, 1),      # two taps per row in 16 bits: not a uniform row, the plain loop runs
    (7, 128, 128, 9, 9, 320, 3, 2, 1),      # stride 2, 18 stages, three column tiles
], ids=op.case_id)
@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_pipelined_tiles(prec, cfg, case):
    """Every pipelined tile: rows and columns past the end, rings longer than
    the K loop, odd and even numbers of stages for the K-split waves."""
    forced(cfg, op.test_conv_fwd, prec, case)
    forced(cfg, op.test_conv_dgrad, prec, case)


@pytest.mark.parametrize("case", [
    (74, 192, 192, 28, 27, 128, 3, 1, 1),   # six and three quarter column tiles, ranges that end inside an image row
    (84, 64, 64, 57, 55, 136, 3, 2, 1),     # odd sizes, stride 2, a channel tile of 8 rows
    (120, 256, 256, 14, 13, 256, 3, 1, 1),  # nine whole column tiles, more than one channel tile
    (64, 128, 128, 57, 56, 256, 1, 2, 0),   # half a column tile: below its columns, the 128x128 tile
], ids=op.case_id)
def test_pipelined_weight_gradient(case):
    """The 128x256 weight gradient at sizes that reach it automatically (and
    one next to them), against the oracle's sums: 1e-5, fp32 sums of exact
    products over up to 68,208 pixels in ranges of a few thousand."""
    op.test_conv_wgrad("bf16", case)


def test_average_pool_sizes():
    """Feature maps of one pixel and of odd sizes end in the average pool: the
    logits of an evaluation equal those of the same images one by one."""
    import torch
    from oracle import net
    from paper_2509_26092_amd import inputs
    for arch, classes, n, h in (("tiny", 10, 5, 17), ("cifar", 100, 3, 17), ("imagenet", 10, 2, 65)):
        L = net.Layout(arch, classes)
        st = torch.from_numpy(net.init_state(L, 3).astype(np.float32)).cuda()
        x = torch.from_numpy(inputs.images(4, n, h, h)).cuda()
        w = B.Worker(arch, classes, "fp32")
        out = torch.empty(n, classes, device="cuda")
        w.eval_logits(st, x, out)
        one = torch.empty(1, classes, device="cuda")
        for i in range(n):
            w.eval_logits(st, x[i:i + 1].clone(), one)
            # fp32 sums in another tile order, through at most 18 layers
            assert torch.allclose(one[0], out[i], rtol=1e-4, atol=1e-4 * float(out.abs().max())), (arch, i)
        w.close()


def step_kernels(arch, classes, prec, n, h, cls):
    """Layer and kernel name of every launch of one class in a training step."""
    import torch
    from oracle import net
    from paper_2509_26092_amd import inputs
    L = net.Layout(arch, classes)
    w = B.Worker(arch, classes, prec)
    st = torch.from_numpy(net.init_state(L, 3).astype(np.float32)).cuda()
    x = torch.from_numpy(inputs.images(4, n, h, h)).cuda()
    y = torch.from_numpy(inputs.labels(4, n, classes)).cuda()
    B.rn18_profile_enable(w.ctx, True)
    w.train_step(st, x, y, 0.1, torch.zeros(1, device="cuda"))
    recs = [(r["layer"], r["kernel"]) for r in B.rn18_profile_read(w.ctx) if r["cls"] == cls]
    w.close()
    return L, recs


@pytest.mark.parametrize("n", [127, 128, 129, 520])
def test_choice_of_64_column_tiles(n):
    """Full precision, 64 columns: the matrix units bound both tiles alike, so
    the 256x64 tile runs only where the fullest compute unit gets no more work
    than with 64x64 tiles, and nearly equal grids get the same kernel."""
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    L, recs = step_kernels("cifar", 10, "fp32", n, 32, "conv_fwd")
    names = [k for layer, k in recs if 1 <= layer <= 4]
    assert len(names) == 4 and len(set(names)) == 1, names
    M = n * 32 * 32
    share = {"64, 64": -(-(-(-M // 64)) // cus), "256, 64": 4 * -(-(-(-M // 256)) // cus)}
    tile = next(t for t in share if "<float, %s," % t in names[0])
    assert share[tile] == min(share.values()), (names[0], share)
    if cus == 256 and n in (127, 128):
        assert tile == "256, 64", names[0]


def test_deep_rings_run_one_round():
    """The deep-ring tiles (16-bit 64x64 and 128x128, four stages) are for
    grids that one round of resident blocks covers."""
    import torch
    from gpu_util import tensor_shapes
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    deep = {"<bf16, 64, 64, 2, 2, 1, 4>": (64, 64, 2), "<bf16, 128, 128, 2, 4, 1, 4>": (128, 128, 1)}
    for n, h in ((96, 224), (256, 192), (64, 128)):
        L, recs = step_kernels("imagenet", 10, "bf16", n, h, "conv_fwd")
        shapes = tensor_shapes(L, n, h)
        for layer, kernel in recs:
            for name, (bm, bn, per_cu) in deep.items():
                if kernel.endswith(name):
                    _, c, ho, wo = shapes[("y", L.convs[layer][0])]
                    tiles = -(-n * ho * wo // bm) * -(-c // bn)
                    assert tiles <= per_cu * cus, (n, h, layer, kernel, tiles)
