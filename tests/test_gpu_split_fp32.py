"""The fp32 kernels that multiply on the bf16 MFMA (operands split in three bf16
parts) against 64-bit sums: every tile of the convolution passes split and
unsplit, at ragged sizes, aligned and not; sums over many pixels, whose rounding
must not drift; infinities, NaNs and tiny values; the FC products; and the
rules that choose these kernels, host-side."""
import pytest
import torch

from paper_2112_15317_amd import sb
from tests.helpers import print_case, rel_l2

# The products are exact to half an fp32 rounding and a sum is rounded to fp32
# once per 32 terms.  The shapes here sum up to 113 such blocks in a row (397
# channels x 9 taps): sqrt(113 / 2) * 2^-24 = 4.5e-7 for a random walk of
# roundings against a random walk of terms.
REL = 5e-7

# (n, c, h, w, k): between them every tile of the forward and of the data
# gradient, with and without split partials, and the three tiles of the weight
# gradient with whole and with broken pixel quads.
SHAPES = [(27, 95, 9, 33, 26), (43, 29, 9, 40, 27), (27, 24, 9, 33, 90), (22, 375, 9, 7, 77),
          (41, 40, 9, 4, 678), (100, 261, 8, 4, 48), (45, 91, 9, 7, 162), (30, 171, 9, 6, 145),
          (303, 23, 8, 4, 180), (154, 131, 9, 6, 37), (286, 151, 4, 9, 17), (49, 41, 5, 40, 30),
          (76, 18, 8, 16, 129), (149, 20, 4, 16, 64), (65, 82, 8, 9, 106), (19, 18, 16, 33, 67),
          (17, 246, 9, 16, 67), (59, 139, 16, 8, 16), (36, 70, 30, 8, 20), (50, 19, 16, 8, 157),
          (4, 151, 9, 20, 369), (29, 36, 30, 8, 48), (51, 99, 5, 5, 317), (40, 65, 9, 8, 217),
          (72, 22, 30, 8, 32), (39, 397, 8, 5, 66), (40, 50, 14, 14, 60), (21, 223, 5, 5, 50),
          (80, 18, 9, 5, 290), (161, 92, 8, 5, 27), (110, 26, 9, 6, 102)]
PASSES = (sb.SB_PASS_FWD, sb.SB_PASS_BWD_DATA, sb.SB_PASS_BWD_WEIGHT)


# Of these, one or more for every tile of the three kernels.
SPECIAL = [(49, 41, 5, 40, 30), (19, 18, 16, 33, 67), (43, 29, 9, 40, 27), (22, 375, 9, 7, 77),
           (161, 92, 8, 5, 27), (76, 18, 8, 16, 129), (21, 223, 5, 5, 50), (29, 36, 30, 8, 48),
           (110, 26, 9, 6, 102), (80, 18, 9, 5, 290), (40, 50, 14, 14, 60), (30, 171, 9, 6, 145)]


def _plan(shape, p):
    n, c, h, w, k = shape
    return sb.sb_conv3x3_plan_string(sb.conv_desc(n, c, h, w, k, sb.SB_F32), p)


@pytest.mark.parametrize("shapes,splits", [(SHAPES, True), (SPECIAL, False)])
def test_shapes_reach_every_tile(shapes, splits):
    for p in PASSES[:2]:
        seen = {(s.split("STile<")[1].split(">")[0], splits and s.endswith("x1"))
                for s in (_plan(q, p) for q in shapes) if "conv3x3_split_f32" in s}
        assert len(seen) == (16 if splits else 8), seen     # 8 tiles, split or not
    seen = {s.split(" grid")[0] for s in (_plan(q, PASSES[2]) for q in shapes)}
    assert len([s for s in seen if "conv3x3_wgrad_split" in s]) == 6, seen


# f, d, w: the pass runs on the split kernel.  Times in us, fp32 MFMA and split.
@pytest.mark.parametrize("shape,passes", [
    ((16, 512, 4, 4, 512), "fdw"),       # forward and data gradient 85, 64
    ((8, 512, 4, 4, 512), "fdw"),
    ((4, 512, 4, 4, 512), "fd-"),        # weight gradient 7.0, 11.3: half a tile of images
    ((24, 64, 16, 16, 64), "--w"),       # 64-channel blocks of 3 rounds
    ((74, 24, 20, 20, 32), "-dw"),       # one chunk: forward 23, 31
    ((128, 32, 8, 8, 256), "fdw"),
    ((64, 24, 32, 32, 16), "--w"),       # 16 outputs; the data gradient has 16 inputs
    ((64, 16, 32, 32, 64), "--w"),       # a chunk is 32 channels; the gradient has 16 outputs
    ((128, 512, 2, 2, 512), "---"),
    ((128, 3, 32, 32, 64), "---"),
    ((12, 64, 8, 8, 16), "---"),         # weight gradients: 9.2, 11.9
    ((2, 40, 15, 16, 32), "---"),        # 9.1, 11.5
    ((8, 32, 24, 16, 40), "---"),
    ((5, 64, 28, 36, 16), "--w"),        # 20.7, 12.9: rows of 64 on the fp32 MFMA
    ((8, 32, 24, 17, 40), "-d-"),        # rows of broken quads: weight gradient 14.4, 16.2
    ((24, 64, 16, 15, 64), "--w"),
    ((100, 64, 4, 6, 64), "---"),        # narrow images: 15, 20
])
def test_rule(shape, passes):
    for p, want in zip(PASSES, passes):
        assert ("split" in _plan(shape, p)) == (want != "-"), _plan(shape, p)


def test_large_images_take_a_tile_within_range():
    # 8 images of this size pass 2^31 bytes, 2 do not.  The size's least padded
    # tiles would be 4 x 4 x 8 images.
    assert "WsTile<8, 8, 2>" in _plan((8, 64, 1364, 1364, 64), sb.SB_PASS_BWD_WEIGHT)


def _rand(*shape, seed=0, scale=1.0):
    g = torch.Generator().manual_seed(seed)
    return torch.randn(*shape, generator=g) * scale


def _dev(t, off=0):
    """On the GPU, starting `off` floats past a 16-byte boundary."""
    buf = torch.empty(t.numel() + off, device="cuda")
    buf[off:].copy_(t.reshape(-1))
    return buf[off:].view(t.shape)


def _ws(nbytes):
    return torch.full((max(int(nbytes), 256),), 0xFF, dtype=torch.uint8, device="cuda")


def _run(shape, x, w, b, dy, off=0, mask=None):
    n, c, h, wd, k = shape
    d = sb.conv_desc(n, c, h, wd, k, sb.SB_F32)
    ws = _ws(max(sb.sb_conv3x3_workspace_bytes(d, p) for p in PASSES))
    xd, wt, bd, dyd = _dev(x, off), _dev(w), _dev(b), _dev(dy, off)
    y, dx = _dev(torch.full_like(dy, 7.0), off), _dev(torch.full_like(x, 7.0), off)
    dw, db = torch.full((k, c, 3, 3), 7.0, device="cuda"), torch.full((k,), 7.0, device="cuda")
    sb.sb_conv3x3_fwd(d, xd, wt, bd, y, ws)
    sb.sb_conv3x3_bwd_data(d, dyd, wt, _dev(mask, off) if mask is not None else None, dx, ws)
    sb.sb_conv3x3_bwd_weight(d, xd, dyd, dw, db, ws)
    torch.cuda.synchronize()
    return [t.cpu() for t in (y, dx, dw, db)]


def _ref(x, w, b, dy, dt=torch.float64):
    x, w, b, dy = (t.to(dt) for t in (x, w, b, dy))
    return [torch.nn.functional.conv2d(x, w, b, padding=1),
            torch.nn.grad.conv2d_input(x.shape, w, dy, padding=1),
            torch.nn.grad.conv2d_weight(x, w.shape, dy, padding=1), dy.sum((0, 2, 3))]


def _inputs(shape, xs=1.0, ws=1.0):
    n, c, h, w, k = shape
    return (_rand(n, c, h, w, seed=1, scale=xs), _rand(k, c, 3, 3, seed=2, scale=ws / (3 * c ** 0.5)),
            _rand(k, seed=3, scale=0.1 * xs * ws), _rand(n, k, h, w, seed=4, scale=xs))


@pytest.mark.gpu
@pytest.mark.parametrize("off", [0, 1])
@pytest.mark.parametrize("shape", SHAPES)
def test_conv_against_64_bits(shape, off):
    print_case("split conv", shape=shape, off=off)
    x, w, b, dy = _inputs(shape)
    mask = _rand(*x.shape, seed=5)
    got, ref = _run(shape, x, w, b, dy, off, mask), _ref(x, w, b, dy)
    ref[1] = ref[1] * (mask > 0)
    for name, a, r in zip(("y", "dx", "dw", "db"), got, ref):
        assert rel_l2(a, r) < REL, (name, rel_l2(a, r))


@pytest.mark.gpu
def test_weight_gradient_does_not_drift():
    # 131072 pixels of positive x against zero-mean dy.  Local sums that are all
    # rounded in one direction leave 4.4e-7; without a drift the blocks of 32
    # pixels, the waves and the splits add about 20 roundings in a row:
    # sqrt(20 / 2) * 2^-24 = 1.9e-7.
    shape = (128, 32, 32, 32, 24)
    print_case("wgrad drift", shape=shape)
    x, w, b, dy = _inputs(shape)
    x = torch.relu(x)
    dw, ref = _run(shape, x, w, b, dy)[2], _ref(x, w, b, dy)[2]
    assert rel_l2(dw, ref) < 2.2e-7, rel_l2(dw, ref)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SPECIAL)
def test_conv_values_the_split_cannot_carry(shape):
    print_case("split conv special", shape=shape)
    # Products of 2^-110: below the range that three parts of each would reach on
    # their own.  Plain fp32 sums, 9 * 512 roundings in a row at most.
    x, w, b, dy = _inputs(shape, xs=2.0 ** -60, ws=2.0 ** -50)
    got, ref = _run(shape, x, w, torch.zeros_like(b), dy), _ref(x, w, torch.zeros_like(b), dy)
    for a, r in zip(got[:2], ref[:2]):
        assert rel_l2(a, r) < (4608 / 2) ** 0.5 * 2.0 ** -24, rel_l2(a, r)
    # One infinity of each sign and one NaN (that of dy inside the image, where no
    # tap meets the padding); a value that would round to infinity in bf16, apart
    # from them, as its products may pass the fp32 range.
    for case in ("inf", "large"):
        x, w, b, dy = _inputs(shape)
        if case == "inf":
            x[1, 3, 1, 2], x[2, 5, 3, 0], dy[4, 6, 2, 1] = float("inf"), float("nan"), float("-inf")
        else:
            x[3, 4, 0, 3] = 3.4e38
        got, ref = _run(shape, x, w, b, dy), [r.float() for r in _ref(x, w, b, dy)]
        for name, a, r in zip(("y", "dx", "dw", "db"), got, ref):
            assert case == "large" or not torch.isfinite(r).all(), name
            assert torch.equal(torch.isnan(a), torch.isnan(r)), (case, name)
            inf = torch.isinf(r)
            assert torch.equal(torch.isinf(a), inf) and torch.equal(a[inf], r[inf]), (case, name)
            for ok in (torch.isfinite(r) & (r.abs() < 1e30), torch.isfinite(r)):
                assert rel_l2(a[ok] * 2.0 ** -20, r[ok] * 2.0 ** -20) < 1e-5, (case, name)


POOL_SHAPES = [(24, 64, 16, 16, 64), (33, 256, 4, 4, 300), (18, 68, 30, 8, 136), (28, 69, 4, 40, 78),
               (1, 346, 2, 4, 1), (288, 52, 4, 4, 1), (66, 177, 6, 12, 1), (69, 65, 16, 12, 1),
               (91, 28, 2, 6, 494), (42, 135, 2, 6, 235), (23, 73, 4, 20, 227), (255, 28, 4, 4, 277),
               (139, 80, 8, 4, 208)]


@pytest.mark.gpu
@pytest.mark.parametrize("shape", POOL_SHAPES)
def test_pooled_forward_is_the_forward_pooled(shape):
    print_case("split conv pool", shape=shape)
    n, c, h, wd, k = shape
    x, w, b, _ = _inputs(shape)
    d = sb.conv_desc(n, c, h, wd, k, sb.SB_F32)
    need = max(sb.sb_conv3x3_workspace_bytes(d, p) for p in (sb.SB_PASS_FWD, sb.SB_PASS_FWD_POOL))
    xd, wt, bd, ws = _dev(x), _dev(w), _dev(b), _ws(need)
    z = torch.empty(n, k, h, wd, device="cuda")
    sb.sb_conv3x3_fwd(d, xd, wt, bd, z, ws)
    out = []
    for fused in (False, True):
        y = torch.full((n, k, h // 2, wd // 2), 7.0, device="cuda")
        idx = torch.full(y.shape, 99, dtype=torch.uint8, device="cuda")
        if fused:
            sb.sb_conv3x3_fwd_pool(d, xd, wt, bd, y, idx, ws)
        else:
            sb.sb_relu_maxpool_fwd(n, k, h, wd, sb.SB_F32, sb.SB_NCHW, z, y, idx)
        out.append((y, idx))
    torch.cuda.synchronize()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


@pytest.mark.gpu
@pytest.mark.parametrize("m,ki,ns", [(1, 33, 1), (63, 65, 127), (64, 64, 64), (65, 31, 130),
                                     (128, 256, 128), (129, 1000, 66), (512, 512, 1024),
                                     (1000, 130, 40), (32, 4100, 257), (1024, 128, 2048),
                                     (1023, 129, 2047), (128, 4096, 512), (479, 741, 1859),
                                     (65, 607, 314), (96, 300, 1500), (250, 2729, 599)])
def test_fc_against_64_bits(m, ki, ns):
    print_case("split fc", m=m, ki=ki, ns=ns)
    x, w, b = _rand(m, ki, seed=1), _rand(ki, ns, seed=2, scale=ki ** -0.5), _rand(ns, seed=3)
    dy, mask = _rand(m, ns, seed=4), _rand(m, ns, seed=5)
    g = dy.double() * (mask > 0)
    ref = [x.double() @ w.double() + b.double(), g @ w.double().T, x.double().T @ g, g.sum(0)]

    def run(x, dy):
        d = sb.fc_desc(m, ki, ns, sb.SB_F32)
        ws = _ws(max(sb.sb_fc_workspace_bytes(d, p) for p in (sb.SB_FC_FWD, sb.SB_FC_BWD)))
        xd, wt, dyd = _dev(x), _dev(w), _dev(dy)
        y, dx = torch.full((m, ns), 7.0, device="cuda"), torch.full((m, ki), 7.0, device="cuda")
        dw, db = torch.full((ki, ns), 7.0, device="cuda"), torch.full((ns,), 7.0, device="cuda")
        sb.sb_fc_shard_fwd(d, xd, wt, _dev(b), y, ws)
        sb.sb_fc_shard_bwd(d, xd, wt, dyd, _dev(mask), dx, dw, db, False, ws)
        torch.cuda.synchronize()
        return [t.cpu() for t in (y, dx, dw, db)]

    for name, a, r in zip(("y", "dx", "dw", "db"), run(x, dy), ref):
        assert rel_l2(a, r) < REL, (name, rel_l2(a, r))
    # An infinity in x reaches its row of y and of dw alone.
    x[m // 2, ki // 2] = float("inf")
    y, _, dw, _ = run(x, dy)
    assert torch.isinf(y).any(1).nonzero().flatten().tolist() == [m // 2]
    bad = ~torch.isfinite(dw).all(1)
    assert bad.nonzero().flatten().tolist() == [ki // 2] and not torch.isfinite(dw[ki // 2]).any()


@pytest.mark.gpu
@pytest.mark.parametrize("m,ki,ns,forward", [(1024, 128, 2048, True), (1024, 64, 2048, True),
                                             (128, 4096, 512, False), (224, 5536, 192, False)])
def test_short_reductions_fill_the_chip(m, ki, ns, forward):
    # Many outputs of 64 to 224 terms beside the 512 x 4096 x 1024 forward (41
    # us) of the same process: 0.20 to 0.29 of it (8 to 12 us), the fp32 MFMA's 9
    # to 15 us likewise.  Output loops that wait for their bias piece by piece
    # and one block a CU take 0.36 to 0.45 (15 to 19 us).
    print_case("fc short reduction", m=m, ki=ki, ns=ns, forward=forward)

    def call(m, ki, ns, forward):
        d = sb.fc_desc(m, ki, ns, sb.SB_F32)
        ws = _ws(max(sb.sb_fc_workspace_bytes(d, p) for p in (sb.SB_FC_FWD, sb.SB_FC_BWD)))
        x, w, b, dy = (_dev(_rand(*s)) for s in ((m, ki), (ki, ns), (ns,), (m, ns)))
        y, dw, db = (torch.empty_like(t) for t in (dy, w, b))
        if forward:
            return lambda: sb.sb_fc_shard_fwd(d, x, w, b, y, ws)
        return lambda: sb.sb_fc_shard_bwd(d, x, w, dy, None, None, dw, db, False, ws)

    def us(f):
        f()
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            for _ in range(20):
                f()
        best = []
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            g.replay()
            b.record()
            torch.cuda.synchronize()
            best.append(a.elapsed_time(b) * 50)
        return min(best)

    t, whole = us(call(m, ki, ns, forward)), us(call(512, 4096, 1024, True))
    print("us", t, whole)
    assert t < 0.325 * whole, (t, whole)


@pytest.mark.gpu
@pytest.mark.parametrize("m,ki,ns", [(1024, 1024, 1024), (1024, 128, 64), (1000, 300, 200)])
def test_bf16_fc_weight_gradient_does_not_drift(m, ki, ns):
    # Positive terms, exact products: a split's sum is rounded at its own size
    # once per 128 rows, eight times here, and the splits' sums twice: as random
    # roundings of a sum that grows evenly sqrt(10 / 3) * 2^-25 = 5.4e-8.  The
    # bf16 MFMA drops low bits always downwards within the 128 rows: 4 steps of
    # half a unit at an eighth of the sum's size, 2^-24 / 4 = 1.5e-8.
    print_case("bf16 fc dw", m=m, ki=ki, ns=ns)
    x, dy = (_rand(*s, seed=i).abs().bfloat16() for i, s in enumerate(((m, ki), (m, ns))))
    w = _rand(ki, ns, seed=3).bfloat16()
    d = sb.fc_desc(m, ki, ns, sb.SB_BF16)
    dw = torch.full((ki, ns), 7.0, device="cuda")
    sb.sb_fc_shard_bwd(d, x.cuda(), w.cuda(), dy.cuda(), None, None, dw, None, False,
                       _ws(sb.sb_fc_workspace_bytes(d, sb.SB_FC_BWD)))
    err = rel_l2(dw.cpu(), x.double().T @ dy.double())
    print("error", err)
    assert err < 7e-8


# Scales of x, w and dy: small operands that meet large ones, so that their
# products are ordinary numbers (sums of 1e4 products of 2^108 stay below 2^117);
# 2^-140 against 1, whose products are subnormal.
SMALL = [(-118, 24, 24), (24, -118, 24), (24, 24, -118), (-140, 100, 8), (8, -140, 100),
         (100, 8, -140), (-140, 0, 0), (0, -140, 0), (0, 0, -140)]


def _scaled(t, e, rows=None):
    """t * 2^e in fp32 (exact but for subnormal results), all of it or its rows of dim 1."""
    if rows is None:
        return (t.double() * 2.0 ** e).float()
    t = t.clone()
    t[:, rows] = (t[:, rows].double() * 2.0 ** e).float()
    return t


def _small_ok(name, a, r, e, terms):
    """Products of 2^e (times the inputs' own sizes), fp32 sums of `terms`
    roundings; below 2^-100 every product may be off by half of the last
    subnormal bit, 2^-150, of a size of 2^(e - 6) with filters of 400 channels."""
    err = (a.double() - r).norm() / r.norm()
    bound = (terms / 2) ** 0.5 * 2.0 ** -24 + (2.0 ** (-144 - e) if e < -100 else 0.0)
    assert torch.isfinite(a).all() and err < bound, (name, float(err), bound)


@pytest.mark.gpu
@pytest.mark.parametrize("exps", SMALL, ids=str)
@pytest.mark.parametrize("shape", SPECIAL)
def test_conv_small_operands_keep_their_bits(shape, exps):
    print_case("split conv small operands", shape=shape, exps=exps)
    ex, ew, ed = exps
    x, w, b, dy = _inputs(shape)
    x, w, dy, b = _scaled(x, ex), _scaled(w, ew), _scaled(dy, ed), torch.zeros_like(b)
    got, ref = _run(shape, x, w, b, dy), _ref(x, w, b, dy)
    # The filters' own size is about 1 / (3 sqrt(c)).
    for name, a, r, e in zip(("y", "dx", "dw"), got, ref, (ex + ew, ed + ew, ex + ed)):
        _small_ok(name, a, r, e, max(9 * shape[1], 9 * shape[4], shape[0] * shape[2] * shape[3]))


@pytest.mark.gpu
@pytest.mark.parametrize("m,ki,ns", [(65, 130, 130), (512, 512, 1024)])
@pytest.mark.parametrize("exps", SMALL, ids=str)
def test_fc_small_operands_keep_their_bits(m, ki, ns, exps):
    print_case("split fc small operands", m=m, ki=ki, ns=ns, exps=exps)
    ex, ew, ed = exps
    x, w, dy = (_scaled(_rand(*s, seed=i), e) for i, (s, e) in
                enumerate((((m, ki), ex), ((ki, ns), ew), ((m, ns), ed))))
    d = sb.fc_desc(m, ki, ns, sb.SB_F32)
    ws = _ws(max(sb.sb_fc_workspace_bytes(d, p) for p in (sb.SB_FC_FWD, sb.SB_FC_BWD)))
    y, dx, dw = (torch.full_like(t, 7.0, device="cuda") for t in (dy, x, w))
    sb.sb_fc_shard_fwd(d, _dev(x), _dev(w), None, y, ws)
    sb.sb_fc_shard_bwd(d, _dev(x), _dev(w), _dev(dy), None, dx, dw, None, False, ws)
    torch.cuda.synchronize()
    x, w, dy = x.double(), w.double(), dy.double()
    for name, a, r, e in (("y", y, x @ w, ex + ew), ("dx", dx, dy @ w.T, ed + ew),
                          ("dw", dw, x.T @ dy, ex + ed)):
        _small_ok(name, a.cpu(), r, e, 1024)


@pytest.mark.gpu
def test_a_few_small_operands_among_ordinary_ones():
    # One channel of 2^-120 against filters (and dy) of 2^120: as large in every
    # sum as the others.
    shape = (40, 50, 14, 14, 60)
    print_case("split conv few small operands", shape=shape)
    x, w, b, dy = _inputs(shape)
    x1, w1 = _scaled(x, -120, [5]), _scaled(w, 120, [5])
    y = _run(shape, x1, w1, torch.zeros_like(b), dy)[0]
    assert rel_l2(y, _ref(x1, w1, torch.zeros_like(b), dy)[0]) < 4e-6
    x1, w1 = _scaled(x, 120, [5]), _scaled(w, -120, [5])
    y = _run(shape, x1, w1, torch.zeros_like(b), dy)[0]
    assert rel_l2(y, _ref(x1, w1, torch.zeros_like(b), dy)[0]) < 4e-6
    m, ki, ns = 129, 300, 200
    a, f = _scaled(_rand(m, ki), -120, [7]), _scaled(_rand(ki, ns, seed=1).T.contiguous(), 120, [7]).T
    d = sb.fc_desc(m, ki, ns, sb.SB_F32)
    out = torch.full((m, ns), 7.0, device="cuda")
    sb.sb_fc_shard_fwd(d, _dev(a), _dev(f.contiguous()), None, out,
                       _ws(sb.sb_fc_workspace_bytes(d, sb.SB_FC_FWD)))
    assert rel_l2(out.cpu(), a.double() @ f.double()) < 4e-6


@pytest.mark.gpu
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("everywhere", [True, False])
def test_special_values_cost_a_bounded_time(value, everywhere):
    # A block that meets such values redoes its tile on the fp32 MFMA: 3 to 7
    # times an ordinary call on these sizes.  Output by output on the vector
    # ALU it was 45 to 130 times.
    print_case("split special cost", value=value, everywhere=everywhere)

    def best(f):
        ms = []
        for _ in range(4):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            f()
            b.record()
            torch.cuda.synchronize()
            ms.append(a.elapsed_time(b))
        return min(ms)

    def fill(t):
        (t if everywhere else t.view(-1)[:1]).fill_(value)

    n, c, h, w, k = 128, 64, 32, 32, 64
    d = sb.conv_desc(n, c, h, w, k, sb.SB_F32)
    ws = _ws(max(sb.sb_conv3x3_workspace_bytes(d, p) for p in PASSES))
    x, wt, b, dy = (_dev(t) for t in _inputs((n, c, h, w, k)))
    y, dx, dw, db = (torch.empty_like(t) for t in (dy, x, wt, b))
    m, ki, ns = 512, 4096, 1024
    fd = sb.fc_desc(m, ki, ns, sb.SB_F32)
    fws = _ws(max(sb.sb_fc_workspace_bytes(fd, p) for p in (sb.SB_FC_FWD, sb.SB_FC_BWD)))
    fx, fw, fdy = (_dev(_rand(*s, seed=9)) for s in ((m, ki), (ki, ns), (m, ns)))
    fy, fdx, fdw = (torch.empty_like(t) for t in (fdy, fx, fw))
    calls = [lambda: sb.sb_conv3x3_fwd(d, x, wt, b, y, ws),
             lambda: sb.sb_conv3x3_bwd_data(d, dy, wt, None, dx, ws),
             lambda: sb.sb_conv3x3_bwd_weight(d, x, dy, dw, db, ws),
             lambda: sb.sb_fc_shard_fwd(fd, fx, fw, None, fy, fws),
             lambda: sb.sb_fc_shard_bwd(fd, fx, fw, fdy, None, fdx, fdw, None, False, fws)]
    plain = [best(f) for f in calls]
    for t in (x, dy, fx, fdy):
        fill(t)
    ratios = [best(f) / p for f, p in zip(calls, plain)]
    print("ratios", ["%.1f" % r for r in ratios])
    assert max(ratios) < 14, ratios
