"""sb_conv3x3_bwd_weight_many: several layers' weight gradients in one call
(consecutive layers on the same kernel share a launch) give exactly the
per-layer sb_conv3x3_bwd_weight results, on runs of layers of every kernel that
batches (the split ones with whole and with broken or unaligned pixel quads,
the fp32-MFMA ones with full-width rows, whole images and neither), layers that
take other kernels, and channel-blocked bf16 layers in the same list."""
import pytest
import torch

from paper_2112_15317_amd import sb, synth
from tests.helpers import print_case

# (n, c, h, w, k, dtype, layout, floats past alignment): pairs of equal kernels
# between layers that take other ones (3 input channels, 2x2 images,
# channel-blocked).
LAYERS = [(8, 3, 32, 32, 64, "f32", "nchw", 0),
          # split: 8x16 tiles
          (8, 64, 32, 32, 64, "f32", "nchw", 0), (8, 128, 16, 16, 128, "f32", "nchw", 0),
          (16, 64, 14, 14, 64, "f32", "nchw", 0), (8, 64, 32, 32, 64, "f32", "nchw", 1),
          # 8x8 tiles
          (8, 256, 8, 8, 256, "f32", "nchw", 0), (8, 256, 8, 8, 128, "f32", "nchw", 0),
          (8, 256, 8, 8, 256, "f32", "nchw", 0),
          (64, 64, 7, 7, 64, "f32", "nchw", 0), (64, 64, 7, 7, 80, "f32", "nchw", 0),
          # 4x4 tiles
          (8, 512, 4, 4, 512, "f32", "nchw", 0), (16, 256, 4, 4, 512, "f32", "nchw", 0),
          (64, 64, 4, 9, 64, "f32", "nchw", 0), (9, 512, 4, 4, 256, "f32", "nchw", 1),
          (128, 16, 2, 2, 16, "f32", "nchw", 0),
          # fp32 MFMA: 2x32 tiles, full-width rows and not
          (1, 16, 32, 32, 32, "f32", "nchw", 0), (2, 16, 30, 32, 24, "f32", "nchw", 0),
          (1, 16, 20, 36, 32, "f32", "nchw", 0), (1, 16, 21, 37, 24, "f32", "nchw", 0),
          # 4x16
          (2, 24, 16, 16, 40, "f32", "nchw", 0), (3, 24, 14, 16, 24, "f32", "nchw", 1),
          (2, 24, 16, 20, 40, "f32", "nchw", 0), (3, 24, 12, 20, 40, "f32", "nchw", 0),
          # 8x8: whole images, full-width rows, neither
          (4, 40, 8, 8, 24, "f32", "nchw", 0), (3, 24, 8, 8, 40, "f32", "nchw", 0),
          (3, 24, 10, 8, 40, "f32", "nchw", 0), (2, 24, 12, 8, 40, "f32", "nchw", 0),
          (3, 24, 8, 12, 40, "f32", "nchw", 0), (5, 40, 8, 12, 24, "f32", "nchw", 0),
          (2, 16, 16, 16, 32, "bf16", "c8", 0), (3, 24, 12, 20, 40, "f32", "nchw", 0)]


def _desc(n, c, h, w, k, dt, lay, off):
    return sb.conv_desc(n, c, h, w, k, sb.SB_BF16 if dt == "bf16" else sb.SB_F32,
                        layout=sb.SB_NCHW8C if lay == "c8" else sb.SB_NCHW)


def _form(layer):
    """The kernel instantiation a layer takes, from its plan and the forms that
    the plan string leaves out."""
    n, c, h, w, k, dt, lay, off = layer
    s = sb.sb_conv3x3_plan_string(_desc(*layer), sb.SB_PASS_BWD_WEIGHT).split(" grid=")[0]
    if "wgrad_split" in s:
        return s.rsplit(", ", 1)[0], w % 4 == 0 and off == 0
    if "conv3x3_wgrad_f32<sb::WgTile<" in s and ", 0>, float" in s:
        tile = int(s.split("WgTile<")[1].split(",")[1])
        return s, w == tile, tile == 8 and h == 8 and w == 8
    return None


def test_layers_batch_every_form():
    runs = [a for a, b in zip(map(_form, LAYERS), map(_form, LAYERS[1:])) if a and a == b]
    assert len([f for f in set(runs) if "split" in f[0]]) == 6, set(runs)
    assert len([f for f in set(runs) if "split" not in f[0]]) == 7, set(runs)


def _tensors(i, n, c, h, w, k, dtype, layout, off):
    x = torch.from_numpy(synth.normal((n, c, h, w), i, synth.TID.MISC)).cuda()
    dy = torch.from_numpy(synth.normal((n, k, h, w), i, synth.TID.DY_TOP)).cuda()
    if dtype == "bf16":
        x, dy = x.bfloat16(), dy.bfloat16()
    if layout == "c8":
        x = x.reshape(n, c // 8, 8, h, w).permute(0, 1, 3, 4, 2).contiguous()
        dy = dy.reshape(n, k // 8, 8, h, w).permute(0, 1, 3, 4, 2).contiguous()
    if off:
        x, dy = (torch.cat([t.new_zeros(off), t.reshape(-1)])[off:].view(t.shape) for t in (x, dy))
    return x, dy


@pytest.mark.gpu
@pytest.mark.parametrize("with_db", [True, False])
def test_bwd_weight_many_equals_single_calls(with_db):
    print_case("bwd_weight_many", layers=len(LAYERS), with_db=with_db)
    descs, xs, dys, ref_w, ref_b = [], [], [], [], []
    for i, layer in enumerate(LAYERS):
        n, c, h, w, k = layer[:5]
        d = _desc(*layer)
        x, dy = _tensors(i, *layer)
        dw = torch.full((k, c, 3, 3), float("nan"), device="cuda")
        db = torch.full((k,), float("nan"), device="cuda") if with_db else None
        need = sb.sb_conv3x3_workspace_bytes(d, sb.SB_PASS_BWD_WEIGHT)
        ws = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")
        sb.sb_conv3x3_bwd_weight(d, x, dy, dw, db, ws)
        descs.append(d); xs.append(x); dys.append(dy); ref_w.append(dw); ref_b.append(db)
    torch.cuda.synchronize()
    dws = [torch.full_like(t, float("nan")) for t in ref_w]
    dbs = [torch.full_like(t, float("nan")) if t is not None else None for t in ref_b]
    wl = sb.WgradList(descs, xs, dys, dws, dbs)
    need = wl.workspace_bytes()
    # A dirty workspace: its contents must not matter.
    ws = torch.full((need,), 0x7f, dtype=torch.uint8, device="cuda")
    for rep in range(2):
        sb.sb_conv3x3_bwd_weight_many(wl, ws)
        torch.cuda.synchronize()
        for i, (a, b) in enumerate(zip(dws, ref_w)):
            assert torch.equal(a, b), "layer %d dW differs (call %d)" % (i, rep)
        for i, (a, b) in enumerate(zip(dbs, ref_b)):
            assert (a is None) == (b is None)
            if a is not None:
                assert torch.equal(a, b), "layer %d db differs (call %d)" % (i, rep)
