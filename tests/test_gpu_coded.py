"""Stage entry points with the boundary codec fused in: bit-identical to decode -> stage -> encode
(which test_gpu_codec.py / test_gpu_stage.py tie to the oracle), and checked against the oracle chain."""
import numpy as np
import pytest
import torch

import swarm_synth as synth
from oracle import codec as ocodec, stage as osg

pytestmark = pytest.mark.gpu


def _run(wl, scale_bits=32):
    """Fused entry points against decode -> stage -> encode on the GPU, bit for bit, with fp32 (32) or 16-bit block
    scales on all four boundary tensors.  Returns the parameters and the oracle's / the GPU's codes and scales."""
    import paper_2301_11913_amd as sw
    s16 = scale_bits == 16
    enc = sw.swarm_codec_encode_s16 if s16 else sw.swarm_codec_encode
    dec = sw.swarm_codec_decode_s16 if s16 else sw.swarm_codec_decode
    params = synth.make_params(wl)
    x, G = synth.make_x_in(wl), synth.make_grad_out(wl)
    bf = wl.dtype == "bf16"
    dt = torch.bfloat16 if bf else torch.float32
    dev = lambda a: (torch.from_numpy(np.ascontiguousarray(a)).to(dt)).cuda()
    cx, sx = ocodec.encode(x.reshape(-1), scale_bits=scale_bits)
    cg, sg = ocodec.encode(G.reshape(-1), scale_bits=scale_bits)
    if s16:
        sx, sg = sx.view(np.int16), sg.view(np.int16)              # bf16 bit patterns in a 16-bit torch tensor
    cfg = sw.StageConfig(wl.d_model, wl.n_heads, wl.d_ffn, wl.n_layers, wl.n_repeat, wl.batch, wl.seq, wl.dtype,
                         block_kind=wl.block)
    dp = [{k: dev(p[k]) for k in sw.PARAM_FIELDS} for p in params]
    n = x.size
    i8 = lambda: torch.full((n,), 55, dtype=torch.int8, device="cuda")
    f32 = lambda: torch.full((n // 64,), -3, dtype=torch.int16 if s16 else torch.float32, device="cuda")
    cxd, sxd, cgd, sgd = (torch.from_numpy(a).cuda() for a in (cx, sx, cg, sg))

    # --- unfused reference path on the GPU
    xd = torch.empty(x.shape, dtype=dt, device="cuda"); gd = torch.empty_like(xd)
    dec(cxd, sxd, xd); dec(cgd, sgd, gd)
    ws = torch.empty(sw.swarm_stage_workspace_bytes(cfg, True), dtype=torch.uint8, device="cuda")
    y = torch.empty_like(xd); gin = torch.empty_like(xd)
    gp = [{k: torch.zeros(p[k].shape, dtype=torch.float32, device="cuda") for k in sw.PARAM_FIELDS} for p in params]
    sw.swarm_stage_forward(cfg, dp, xd, y, ws)
    sw.swarm_stage_backward(cfg, dp, xd, gd, gin, gp, ws)
    cy, sy, cgi, sgi = i8(), f32(), i8(), f32()
    enc(y, cy, sy); enc(gin, cgi, sgi)

    # --- fused path
    ws2 = torch.empty(max(sw.swarm_stage_coded_workspace_bytes(cfg, True), sw.swarm_stage_coded_workspace_bytes(cfg, False)),
                      dtype=torch.uint8, device="cuda")
    xdec = torch.full(x.shape, 9.0, dtype=dt, device="cuda")
    cy2, sy2, cgi2, sgi2 = i8(), f32(), i8(), f32()
    gp2 = [{k: torch.zeros(p[k].shape, dtype=torch.float32, device="cuda") for k in sw.PARAM_FIELDS} for p in params]
    sw.swarm_stage_forward_coded(cfg, dp, cxd, sxd, xdec, cy2, sy2, ws2)
    sw.swarm_stage_backward_coded(cfg, dp, xdec, cgd, sgd, cgi2, sgi2, gp2, ws2)
    torch.cuda.synchronize()
    assert torch.equal(xdec, xd)
    assert torch.equal(cy2, cy) and torch.equal(sy2, sy)
    assert torch.equal(cgi2, cgi) and torch.equal(sgi2, sgi)
    for a, b in zip(gp, gp2):
        for k in a:
            assert torch.equal(a[k], b[k]), k
    u16 = lambda a: a.view(np.uint16) if s16 else a
    return params, cx, u16(sx), cg, u16(sg), cy2.cpu().numpy(), u16(sy2.cpu().numpy()), cgi2.cpu().numpy(), \
        u16(sgi2.cpu().numpy())


@pytest.mark.parametrize("shape", [
    # dtype, d, H, f, S, B, L, R   (fused kernels: bf16 and d % 256 == 0; the others take the unfused route)
    ("bf16", 256, 2, 512, 160, 2, 1, 2),
    ("bf16", 512, 4, 1024, 75, 3, 2, 1),
    ("bf16", 1024, 8, 4096, 512, 2, 1, 1),
    ("bf16", 128, 2, 192, 37, 3, 1, 1),
    ("f32", 256, 4, 1024, 64, 2, 1, 1),
    # widths whose chunks do not fill the last pass of the decoding / encoding LayerNorm kernels' lanes
    ("bf16", 768, 6, 1536, 40, 2, 1, 1),
    ("bf16", 1536, 12, 1024, 50, 2, 1, 1),
    ("bf16", 6144, 48, 1024, 24, 2, 1, 1),
])
@pytest.mark.parametrize("scale_bits", [32, 16])
def test_coded_equals_unfused(shape, scale_bits):
    dtype, d, H, f, S, B, L, R = shape
    wl = synth.Workload(name="coded", dtype=dtype, d_model=d, n_heads=H, d_ffn=f, seq=S, batch=B, n_layers=L,
                        n_repeat=R, grad_sigma=1.0 if dtype == "f32" else 1e-2, seed=911 + d + S)
    _run(wl, scale_bits)


@pytest.mark.parametrize("scale_bits", [32, 16])
@pytest.mark.parametrize("shape", [(1024, 8, 256, 528, 8), (1024, 8, 192, 768, 8), (2304, 18, 256, 1024, 8),
                                   (1024, 8, 256, 525, 8), (1024, 8, 2112, 700, 8), (1024, 8, 1024, 1025, 8)])
def test_coded_equals_unfused_on_every_route(shape, scale_bits):
    """Token counts at which the last product runs on 264 tiles of 128 x 128, on 192 of 256 x 128, and on 288 of 256 x 256
    of which the last columns are a product of their own; ragged ones on 128 x 128, 256 x 128 and 256 x 256 tiles."""
    d, H, f, S, B = shape
    wl = synth.Workload(name="coded", dtype="bf16", d_model=d, n_heads=H, d_ffn=f, seq=S, batch=B, n_layers=1, n_repeat=1,
                        grad_sigma=1e-2, seed=77 + d + S)
    _run(wl, scale_bits)

@pytest.mark.parametrize("scale_bits", [32, 16])
@pytest.mark.parametrize("shape", [(256, 2, 512, 96, 2, 1, 2), (512, 4, 1024, 75, 3, 2, 1), (1024, 8, 4096, 320, 1, 1, 1)])
def test_coded_against_oracle_chain(scale_bits, shape):
    """decode (oracle) -> oracle stage -> compare decoded GPU outputs within the bf16 tolerance plus half a
    quantisation step of the output codec; the GPU's codes and scales are also the oracle codec's on the GPU's
    own decoded values (re-encoding what was decoded gives the same codes)."""
    d, H, f, S, B, L, R = shape      # heads of 128 and of 64, shared and distinct blocks, a ragged token count
    wl = synth.Workload(name="coded", dtype="bf16", d_model=d, n_heads=H, d_ffn=f, seq=S, batch=B,
                        n_layers=L, n_repeat=R, grad_sigma=1e-2, seed=3 + d)
    params, cx, sx, cg, sg, cy, sy, cgi, sgi = _run(wl, scale_bits)
    shape = (wl.batch, wl.seq, wl.d_model)
    x = ocodec.bf16_bits_to_f32(ocodec.decode(cx, sx, out="bf16")).reshape(shape)
    G = ocodec.bf16_bits_to_f32(ocodec.decode(cg, sg, out="bf16")).reshape(shape)
    ry = osg.stage_forward(params, x, wl.n_heads, wl.n_repeat)
    rgin = osg.stage_backward(params, x, G, osg.zero_grads(params), wl.n_heads, wl.n_repeat)
    for codes, scales, ref in ((cy, sy, ry), (cgi, sgi, rgin)):
        got = ocodec.decode(codes, scales).reshape(shape).astype(np.float64)
        sc = ocodec.bf16_bits_to_f32(scales) if scale_bits == 16 else scales
        step = np.repeat(sc.astype(np.float64), 64).reshape(shape)
        assert np.all(np.abs(got - ref) <= 2e-2 * np.max(np.abs(ref)) + 0.5 * step + 1e-12)
        rc, _ = ocodec.encode(ocodec.decode(codes, scales), scale_bits=scale_bits)
        assert np.array_equal(rc, codes)
