"""Texel loads of the gathers: the two texels of a footprint's row are read by
one access (a texel at a time in buckets of one sample and for 16-byte texels).
Every storage format and channel count, at bucket sizes where the rows start at
every alignment, with footprints in the texture's first and last texels; the
last texel is the last of its allocation.

The forward is within 1e-5 of the oracle on the same codes (the formats'
decoding is exact); the view gradient within check_grad_vec's bounds.
"""
import pytest
import torch

import oracle
from helpers import (away_from_edges, bucket_edge_mask, check_fwd, check_grad_vec, host, round_s,
                     round_w)

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
FMT = {"bf16": oracle.FMT_BF16, "fp8": oracle.FMT_FP8_E4M3}


@pytest.mark.parametrize("mode", ["nearest", "bilinear"])
@pytest.mark.parametrize("n", [1, 2, 3, 5])
@pytest.mark.parametrize("C", [1, 2, 3, 4])
@pytest.mark.parametrize("fmt", ["f32", "bf16", "fp8"])
def test_rows_of_two_texels(fmt, C, n, mode):
    from paper_2301_01719_amd import radtex as rt
    W, H, N = 3, 2, 600
    g = torch.Generator().manual_seed(100 * n + 10 * C + len(fmt))
    values = torch.rand((H, W, n, n, C), generator=g)
    tex = rt.Texture(values.to(DEV), W, H, n, C)
    otex = oracle.Tex(values.numpy(), W, H, n, C)
    if fmt != "f32":
        codes, scales = rt.quantize(tex, fmt)
        tex = rt.Texture(codes, W, H, n, C, fmt, scales)
        ocodes, oscales = oracle.quantize(values.numpy(), W * H, n * n * C, FMT[fmt])
        otex = oracle.Tex(ocodes, W, H, n, C, FMT[fmt], oscales)
    uv = torch.rand((N, 2), generator=g)
    vt = torch.randn((N, 3), generator=g)
    vt[:, 2] = vt[:, 2].abs() * 0.3  # low directions reach the buckets' border texels
    tbn = torch.eye(3).expand(N, 3, 3).contiguous()
    uv[0] = torch.tensor([0.5 / W, 0.5 / H])
    uv[1] = torch.tensor([1 - 0.5 / W, 1 - 0.5 / H])
    vt[0], vt[1] = torch.tensor([-1.0, -1.0, 0.0]), torch.tensor([1.0, 1.0, 0.0])
    go = torch.randn((N, C), generator=g)
    d = [x.to(DEV) for x in (uv, tbn, vt)]
    out = rt.lookup_fwd(tex, *d, mode=mode)
    _, gv, _ = rt.lookup_bwd(tex, *d, go.to(DEV), mode=mode)
    torch.cuda.synchronize()
    h = [x.numpy() for x in (uv, tbn, vt)]
    m = oracle.MODE_NEAREST if mode == "nearest" else oracle.MODE_BILINEAR
    inside = bucket_edge_mask(*h, W, H, n) if mode == "nearest" else None
    check_fwd(host(out), oracle.lookup_fwd(otex, *h, mode=m), inside)
    keep = away_from_edges(*h, W, H, n, mode)
    ref = oracle.lookup_bwd(otex, *h, go.numpy(), mode=m)
    rnd, _ = oracle.lookup_bwd_round(otex, *h, go.numpy(), round_s(n), round_w(W, H, h[0]), mode=m)
    check_grad_vec(host(gv)[keep], ref["grad_view"][keep], ref["scale_view"][keep],
                   go.numpy()[keep], rnd[keep])


# Lights read the rows of a plain texture as the lookups do, those of BF16 RGB with
# one bucket by word-aligned accesses: rows that start on a word and between two,
# the first and the last texels of the allocation among them.
@pytest.mark.parametrize("mode", ["nearest", "bilinear"])
@pytest.mark.parametrize("n", [1, 2, 3, 5])
@pytest.mark.parametrize("C", [1, 2, 3, 4])
@pytest.mark.parametrize("fmt", ["f32", "bf16", "fp8"])
def test_rows_of_two_texels_under_lights(fmt, C, n, mode):
    from paper_2301_01719_amd import radtex as rt
    from test_shadow import _frags, _light_vecs
    W, H, N, S = 3, 1, 600, 5
    g = torch.Generator().manual_seed(1000 * n + 10 * C + len(fmt))
    values = torch.rand((H, W, n, n, C), generator=g)
    tex = rt.Texture(values.to(DEV), W, H, n, C)
    otex = oracle.Tex(values.numpy(), W, H, n, C)
    if fmt != "f32":
        codes, scales = rt.quantize(tex, fmt)
        tex = rt.Texture(codes, W, H, n, C, fmt, scales)
        ocodes, oscales = oracle.quantize(values.numpy(), W * H, n * n * C, FMT[fmt])
        otex = oracle.Tex(ocodes, W, H, n, C, FMT[fmt], oscales)
    uv, tbn, _ = _frags(n * 10 + C, N)
    uv[0] = torch.tensor([0.5 / W, 0.5 / H])
    uv[1] = torch.tensor([1 - 0.5 / W, 1 - 0.5 / H])
    tbn[:2] = torch.eye(3)
    vec = _light_vecs("directional", S, seed=n + C)
    vec[0], vec[1] = torch.tensor([-1.0, -1.0, 0.0]), torch.tensor([1.0, 1.0, 0.0])
    out = rt.lookup_light(tex, uv.to(DEV), tbn.to(DEV), rt.make_light(vec.numpy(), "directional"),
                          mode=mode)
    torch.cuda.synchronize()
    m = oracle.MODE_NEAREST if mode == "nearest" else oracle.MODE_BILINEAR
    ref = oracle.lookup_light(otex, uv.numpy(), tbn.numpy(), vec.numpy(),
                              oracle.LIGHT_DIRECTIONAL, mode=m)
    keep = None
    if mode == "nearest":
        keep = bucket_edge_mask(uv.numpy(), tbn.numpy(), torch.ones(N, 3).numpy(), W, H, n)
    check_fwd(host(out), ref, keep)
