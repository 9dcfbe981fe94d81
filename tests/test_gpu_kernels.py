"""GPU parity of the kernels that the automatic choice picks by size, at the
sizes where they can go wrong: partial last tiles in rows and columns, tiles
that span images, single images, several tiles per block, and the smallest
shapes that reach each kernel. The operator entry points run against the oracle
(tolerances as in test_gpu_ops: the rounding of the storage type, 1e-5 for fp32
sums); they pass no split-K scratch, so split ranges and the epilogues of a
training step run in whole steps. Where a choice is the subject, the profiled
step names the kernels."""
import numpy as np
import pytest

from paper_2509_26092_amd import binding as B
import test_gpu_ops as op
import test_gpu_step as step
from gpu_util import PREC, torch_dtype

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
    (3, 64, 64, 14, 14, 128, 3, 1, 1),      # 18-row tiles that start inside an image and cross a border
    (6, 64, 64, 14, 14, 128, 3, 1, 1),      # ... one of them crosses two borders
    (7, 64, 64, 5, 15, 72, 3, 1, 1),        # 16-row tiles over up to four images, odd width
    (4, 64, 64, 13, 27, 136, 3, 1, 1),      # 243-pixel tiles over image borders, odd width
    (1, 192, 192, 16, 16, 256, 3, 1, 1),    # one tile exactly, three channel blocks, two column tiles
    (2, 64, 64, 9, 48, 128, 3, 1, 1),       # the smallest tile that it takes: four rows of 48 pixels
    (3, 64, 64, 5, 51, 72, 3, 1, 1),        # 255-pixel tiles of one image each, odd width
], ids=op.case_id)
@pytest.mark.parametrize("direction", [op.test_conv_fwd, op.test_conv_dgrad], ids=["fwd", "dgrad"])
@pytest.mark.parametrize("prec", ["bf16", "fp16"])
def test_wide_halo(prec, case, direction):
    """The wide halo kernel (16-bit, whole channel blocks, more than 64
    columns); the data gradient runs it where its own columns (the input
    channels) exceed 64."""
    forced(34, direction, prec, case)


@pytest.mark.parametrize("case", [
    (700, 14, 14, 128, 128),     # 545 tiles: two rounds and 33 blocks of a third, the last tile of 8 rows
    (1400, 7, 7, 128, 192),      # 280 tiles of five images, two columns of them: two rounds and 48 blocks
    (300, 14, 14, 256, 128),     # 234 tiles: one round, four channel blocks (the data gradient: two columns of tiles)
], ids=str)
@pytest.mark.parametrize("prec", ["bf16", "fp16"])
def test_wide_halo_several_tiles_per_block(prec, case):
    """Blocks that walk several tiles (the next patch in flight, the stores of
    the last tile counted into the waits), forward and data gradient: bit for
    bit what the 128x128 pipelined tile gives, which adds in the same order."""
    import torch
    N, H, W, cin, cout = case
    gen = torch.Generator(device="cuda").manual_seed(21)
    dt = torch_dtype(prec)
    x = torch.randn(N, H, W, cin, generator=gen, device="cuda").to(dt)
    dy = torch.randn(N, H, W, cout, generator=gen, device="cuda").to(dt)
    wt = (torch.randn(cout, 3, 3, cin, generator=gen, device="cuda") * 0.05).to(dt)
    wd = wt.permute(3, 1, 2, 0).contiguous()
    out = {}
    for cfg in (34, 4):
        y, dx = torch.full_like(dy, float("nan")), torch.full_like(x, float("nan"))
        forced(cfg, B.rn18op_conv2d_fwd, PREC[prec], x, wt, y, N, H, W, cin, cout, 3, 1, 1)
        forced(cfg, B.rn18op_conv2d_dgrad, PREC[prec], dy, wd, dx, N, H, W, cin, cout, 3, 1, 1)
        out[cfg] = (y, dx)
    torch.cuda.synchronize()
    assert torch.isfinite(out[4][0].float()).all() and torch.isfinite(out[4][1].float()).all()
    assert torch.equal(out[34][0], out[4][0]), "forward"
    assert torch.equal(out[34][1], out[4][1]), "data gradient"


@pytest.mark.parametrize("prec", ["bf16", "fp16"])
def test_wide_halo_statistics_over_several_tiles(prec):
    """Batch statistics that a block gathers over its tiles (551 of 32 rows at
    stage 2, the last one partial, and 180 of 49 rows at stage 3): mean and
    1/std of every 3x3 stride-1 layer against fp64 sums of the stored conv
    output. A lane adds up to 12 values and 16 lanes are added up, so a sum is
    off by at most about 16 roundings (2^-24 each) of values that are within a
    few standard deviations of the shift: 2e-5 of a standard deviation."""
    import torch
    from oracle import net
    from gpu_util import tensor_shapes
    N, H = 2203, 64
    L = net.Layout("imagenet", 10)
    st = torch.from_numpy(net.init_state(L, 3).astype(np.float32)).cuda()
    gen = torch.Generator(device="cuda").manual_seed(22)
    x = torch.randn(N, 3, H, H, generator=gen, device="cuda")
    y = torch.randint(0, 10, (N,), generator=gen, device="cuda", dtype=torch.int32)
    w = B.Worker("imagenet", 10, prec)
    B.rn18_profile_enable(w.ctx, True)
    forced(34, w.train_step, st, x, y, 0.1, torch.zeros(1, device="cuda"))
    names = {r["layer"]: r["kernel"] for r in B.rn18_profile_read(w.ctx) if r["cls"] == "conv_fwd"}
    shapes = tensor_shapes(L, N, H)
    seen = 0
    for li, (name, cin, cout, k, s, p) in enumerate(L.convs):
        if k != 3 or s != 1 or cout not in (128, 256):
            continue
        assert "conv_halow_kernel" in names[li], (name, names[li])
        n, c, h, wd = shapes[("y", name)]
        out = torch.empty(n, h, wd, c, dtype=torch_dtype(prec), device="cuda")
        mean, rstd = torch.empty(c, device="cuda"), torch.empty(c, device="cuda")
        for what, t in (("y", out), ("mean", mean), ("rstd", rstd)):
            B.rn18_debug_copy(w.ctx, N, H, H, what, li, t)
        v = out.reshape(-1, c).double()
        m, std = v.mean(0), torch.sqrt(v.var(0, unbiased=False) + 1e-5)
        assert ((mean.double() - m).abs() <= 2e-5 * std + 1e-7 * m.abs()).all(), name
        assert ((rstd.double() * std - 1).abs() <= 2e-5).all(), name
        seen += 1
    w.close()
    assert seen == 6


@pytest.mark.parametrize("direction", [op.test_conv_fwd, op.test_conv_dgrad], ids=["fwd", "dgrad"])
def test_more_column_tiles_than_compute_units(direction):
    """One 16x16 image whose columns make one 128-column tile more than there
    are compute units (a block of the wide halo kernel keeps its columns, so
    that kernel cannot take it): launched by another kernel, not refused."""
    import torch
    wide = 128 * torch.cuda.get_device_properties(0).multi_processor_count + 8
    cin, cout = (64, wide) if direction is op.test_conv_fwd else (wide, 64)
    direction("bf16", (1, cin, cin, 16, 16, cout, 3, 1, 1))


@pytest.mark.parametrize("prec,cfg", [(p, c) for p, cfgs in (
    ("bf16", (4, 5, 6, 8, 9, 10, 11, 12, 17, 18, 19, 20, 22)),
    ("fp32", (4, 5, 6, 8, 9, 10, 11, 20, 22)),    # built for fp32 (forcing another one there runs 4)
) for c in cfgs])
@pytest.mark.parametrize("case", [
    (1, 64, 64, 3, 3, 72, 3, 1, 1),         # 9 rows in any tile, 72 columns
    (2, 64, 64, 16, 15, 264, 1, 1, 0),      # one K stage (fewer than any ring holds), 264 columns
    (3, 32, 32, 13, 12, 128, 3, 1, 1),      # two taps per row in 16 bits: not a uniform row, the plain loop runs
    (7, 128, 128, 9, 9, 320, 3, 2, 1),      # stride 2, 18 stages, three column tiles
], ids=op.case_id)
def test_pipelined_tiles(prec, cfg, case):
    """Every pipelined tile: rows and columns past the end, rings longer than
    the K loop, odd and even numbers of stages for the K-split waves."""
    forced(cfg, op.test_conv_fwd, prec, case)
    forced(cfg, op.test_conv_dgrad, prec, case)


@pytest.mark.parametrize("cfg,split", [(6, 1), (6, 3), (11, 3), (20, 1), (20, 3), (10, 3), (12, 1), (17, 1)])
def test_pipelined_tiles_in_a_step(cfg, split):
    """Every convolution of a bf16 step that can run it forced to one tile,
    whole and with its K stages in ranges: the K-split wave pairs' partial tiles,
    and the epilogues that operators don't reach (statistics, masked residual,
    BN backward partials)."""
    try:
        B.rn18_debug_set(None, B.RN18_DBG_GATHER_SPLIT, split)
        forced(cfg, step._run_parity, "imagenet", 1000, "bf16", 3, 64, 190 + cfg)
    finally:
        B.rn18_debug_set(None, B.RN18_DBG_GATHER_SPLIT, 0)


@pytest.mark.parametrize("case", [
    (74, 192, 192, 28, 27, 128, 3, 1, 1),   # six and three quarter column tiles, ranges that end inside an image row
    (84, 64, 64, 57, 55, 136, 3, 2, 1),     # odd sizes, stride 2, a channel tile of 8 rows
    (120, 256, 256, 14, 13, 256, 3, 1, 1),  # nine whole column tiles, more than one channel tile
    (64, 128, 128, 57, 56, 256, 1, 2, 0),   # half a column tile: below its columns, the 128x128 tile
], ids=op.case_id)
@pytest.mark.parametrize("prec", ["bf16", "fp16"])
def test_pipelined_weight_gradient(prec, case):
    """The 128x256 weight gradient at sizes that reach it automatically (and
    one next to them), against the oracle's sums: 1e-5, fp32 sums of exact
    products over up to 68,208 pixels in ranges of a few thousand."""
    op.test_conv_wgrad(prec, case)


@pytest.mark.parametrize("arch,n,h", [("imagenet", 3, 32), ("imagenet", 2, 64), ("imagenet", 2, 65), ("cifar", 2, 8),
                                      ("cifar", 3, 17), ("tiny", 5, 17)])
def test_average_pool_sizes(arch, n, h):
    """Feature maps of 1x1, 2x2, 3x3, 1x1, 3x3 and 17x17 pixels end in the
    average pool (eight threads share a map's pixels): the logits of an
    evaluation against the oracle (fp32 sums through at most 18 layers)."""
    import torch
    from gpu_util import TOL, assert_close, make_state
    from oracle import net
    from paper_2509_26092_amd import inputs
    L, st = make_state(arch, 10, 180 + h)
    x = inputs.images(180 + h, n, h, h)
    w = B.Worker(arch, 10, "fp32")
    out = torch.empty(n, 10, device="cuda")
    w.eval_logits(torch.from_numpy(st.astype(np.float32)).cuda(), torch.from_numpy(x).cuda(), out)
    torch.cuda.synchronize()
    w.close()
    assert_close(out.cpu().numpy(), net.eval_logits(net.Config(arch, 10), L, st, x), TOL["fp32"], "logits")


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
