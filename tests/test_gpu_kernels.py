"""Kernel-level GPU checks (single GEMM / attention launches) against plain fp64 numpy definitions.
These go through the kernel hooks of the library, not the stage ABI; the stage-level parity tests are
in test_gpu_stage.py."""
import ctypes as C
import math

import numpy as np
import pytest
import torch
from scipy.special import erf

import swarm_synth as synth

pytestmark = pytest.mark.gpu


def _lib():
    import paper_2301_11913_amd as sw
    lib = sw.load_hooks_library()
    lib.swarm_kernel_gemm.restype = C.c_int
    lib.swarm_kernel_gemm.argtypes = [C.c_int] * 4 + [C.c_void_p, C.c_int, C.c_int, C.c_void_p, C.c_int, C.c_int,
                                                      C.c_void_p, C.c_int, C.c_int, C.c_void_p, C.c_void_p, C.c_int,
                                                      C.c_void_p, C.c_int, C.c_void_p]
    return lib


def _bf(a):
    return torch.from_numpy(a).to(torch.bfloat16)


def _gelu(u):
    return 0.5 * u * (1 + erf(u / math.sqrt(2)))


def _gelu_grad(u):
    return 0.5 * (1 + erf(u / math.sqrt(2))) + u * np.exp(-0.5 * u * u) / math.sqrt(2 * math.pi)


def gemm_case(M, N, K, a_t, b_t, epi, seed=0):
    lib = _lib()
    A = _bf(synth.normal(seed, "A", (K, M) if a_t else (M, K)))
    B = _bf(synth.normal(seed, "B", (K, N) if b_t else (N, K)))
    bias = _bf(synth.normal(seed, "bias", (N,)))
    aux = _bf(synth.normal(seed, "aux", (M, N)))
    A64 = A.double().numpy(); B64 = B.double().numpy()
    ref = (A64.T if a_t else A64) @ (B64 if b_t else B64.T)
    Ad, Bd, bd, xd = A.cuda(), B.cuda(), bias.cuda(), aux.cuda()
    C2 = None
    if epi == 5:
        Cd = _bf(synth.normal(seed, "C0", (M, N))).float().cuda()
        ref = ref + Cd.double().cpu().numpy()
    else:
        Cd = torch.full((M, N), 9.0, dtype=torch.bfloat16, device="cuda")
        if epi == 1:
            ref = ref + bias.double().numpy()
        elif epi == 2:
            ref = ref + bias.double().numpy() + aux.double().numpy()
        elif epi == 3:
            C2 = torch.full((M, N), 9.0, dtype=torch.bfloat16, device="cuda")
            u = ref + bias.double().numpy()
            ref = _gelu(u)
        elif epi == 4:
            ref = ref * _gelu_grad(aux.double().numpy())
    st = lib.swarm_kernel_gemm(1, M, N, K, Ad.data_ptr(), A.shape[1], int(a_t), Bd.data_ptr(), B.shape[1], int(b_t),
                               Cd.data_ptr(), N, epi, bd.data_ptr(), xd.data_ptr(), N,
                               C2.data_ptr() if C2 is not None else None, N, None)
    assert st == 0
    torch.cuda.synchronize()
    got = Cd.double().cpu().numpy()
    err = np.max(np.abs(got - ref)) / np.max(np.abs(ref))
    assert err < (1e-5 if epi == 5 else 6e-3), err
    if C2 is not None:
        e2 = np.max(np.abs(C2.double().cpu().numpy() - u)) / np.max(np.abs(u))
        assert e2 < 6e-3, e2


LAYOUTS = [(False, False), (False, True), (True, True)]


@pytest.mark.parametrize("a_t,b_t", LAYOUTS)
@pytest.mark.parametrize("shape", [(256, 256, 64), (128, 128, 128), (512, 768, 256), (300, 192, 320),
                                   (37, 64, 64), (1000, 1088, 200), (4096, 4096, 512), (2048, 4096 + 64, 256 + 64),
                                   # whole tiles but K no multiple of 64, few and many of them, and a ragged M there
                                   (256, 384, 96), (4096, 2560, 96), (4104, 2560, 96),
                                   (40, 24, 20)])         # K no multiple of 8: the scalar kernel
def test_gemm_layouts(a_t, b_t, shape):
    M, N, K = shape
    if a_t and M % 8:
        M = (M + 7) // 8 * 8          # a transposed operand's row length is a feature dimension
    gemm_case(M, N, K, a_t, b_t, 5 if a_t else 0, seed=M + N + K)


@pytest.mark.parametrize("epi", [0, 1, 2, 3, 4, 5])
@pytest.mark.parametrize("shape", [(384, 256, 128), (4096, 4096, 128), (77, 192, 64)])
def test_gemm_epilogues(epi, shape):
    M, N, K = shape
    gemm_case(M, N, K, False, epi == 4, epi, seed=epi)


# ------------------------------------------------------------------ split-K
def _splitk_call(lib, M, N, K, Ad, lda, Bd, ldb, b_t, Cd, epi, bd, xd, scales, ws):
    lib.swarm_kernel_gemm_ws.restype = C.c_int
    lib.swarm_kernel_gemm_ws.argtypes = [C.c_int] * 3 + [C.c_void_p, C.c_int, C.c_int, C.c_void_p, C.c_int, C.c_int,
                                                        C.c_void_p, C.c_int, C.c_int, C.c_void_p, C.c_void_p, C.c_int,
                                                        C.c_void_p, C.c_void_p, C.c_size_t, C.c_void_p]
    st = lib.swarm_kernel_gemm_ws(M, N, K, Ad.data_ptr(), lda, 0, Bd.data_ptr(), ldb, int(b_t), Cd.data_ptr(), N, epi,
                                  bd.data_ptr(), xd.data_ptr(), N, scales.data_ptr() if scales is not None else None,
                                  ws.data_ptr() if ws is not None else None, ws.numel() if ws is not None else 0, None)
    assert st == 0
    torch.cuda.synchronize()


# (M, N, K, parts the kernel takes): one tile cut in four, 16 tiles cut in two (K / 4 would be below 4096),
# 128 tiles cut in two, and a product that is not cut (K too short) although scratch is offered
@pytest.mark.parametrize("shape", [(256, 256, 16384), (512, 2048, 8192), (2048, 4096, 8192), (256, 512, 4096)])
@pytest.mark.parametrize("b_t", [False, True])
@pytest.mark.parametrize("epi", [0, 1, 2])
def test_gemm_splitk(shape, b_t, epi):
    M, N, K = shape
    lib = _lib()
    lib.swarm_kernel_gemm_splitk_floats.restype = C.c_size_t
    nfl = lib.swarm_kernel_gemm_splitk_floats(M, N)
    assert nfl == (4 if (M // 256) * (N // 256) <= 64 else 2) * M * N
    seed = M + N + K + epi
    A = _bf(synth.normal(seed, "A", (M, K)))
    B = _bf(synth.normal(seed, "B", (K, N) if b_t else (N, K)))
    bias = _bf(synth.normal(seed, "bias", (N,)))
    aux = _bf(synth.normal(seed, "aux", (M, N)))
    ref = A.double().numpy() @ (B.double().numpy() if b_t else B.double().numpy().T)
    if epi >= 1:
        ref = ref + bias.double().numpy()
    if epi == 2:
        ref = ref + aux.double().numpy()
    Ad, Bd, bd, xd = A.cuda(), B.cuda(), bias.cuda(), aux.cuda()
    ws = torch.full((nfl,), float("nan"), dtype=torch.float32, device="cuda")
    C1 = torch.full((M, N), 9.0, dtype=torch.bfloat16, device="cuda")
    _splitk_call(lib, M, N, K, Ad, K, Bd, B.shape[1], b_t, C1, epi, bd, xd, None, ws)
    got = C1.double().cpu().numpy()
    err = np.max(np.abs(got - ref)) / np.max(np.abs(ref))
    assert err < 6e-3, err
    cut = K // 2 >= 4096
    assert bool(torch.isnan(ws).all()) == (not cut)            # the scratch is used exactly when K is long enough
    # the one-kernel product of the same operands: equal up to the summation order of the fp32 partial sums, i.e.
    # at most one bf16 unit (2^-7 of the element) apart after rounding
    C0 = torch.full((M, N), 9.0, dtype=torch.bfloat16, device="cuda")
    _splitk_call(lib, M, N, K, Ad, K, Bd, B.shape[1], b_t, C0, epi, bd, xd, None, None)
    d = np.max(np.abs(C0.double().cpu().numpy() - got)) / np.max(np.abs(ref))
    assert d <= 2.0 ** -7 and (cut or d == 0.0), d


@pytest.mark.parametrize("epi,b_t", [(0, False), (0, True), (1, False), (2, False), (3, False), (4, True)])
def test_gemm_ragged_last_round(epi, b_t):
    """384 tiles of 256 x 256 (one and a half rounds of the 256 compute units): the columns of the whole round and
    the remaining columns run as two products; every output column must come out as from one.  Epilogues with the
    layouts the stage uses them with."""
    gemm_case(2048, 12288, 256, False, b_t, epi, seed=40 + epi)


@pytest.mark.parametrize("epi,b_t", [(0, False), (0, True), (1, False), (2, False), (3, False), (4, True)])
@pytest.mark.parametrize("shape", [(2048, 4096, 64), (2048, 4096, 448), (1536, 4096, 256), (1792, 4224, 128)])
def test_gemm_256x128_tiles(shape, epi, b_t):
    """192 .. 256 tiles of 256 x 128 (a 2048-row microbatch times a 4096-wide weight): one round of those instead
    of two rounds of 128 x 128.  One, two, four and seven 64-deep slices; a column count that is no multiple of 256."""
    M, N, K = shape
    gemm_case(M, N, K, False, b_t, epi, seed=60 + epi)


@pytest.mark.parametrize("epi,b_t", [(0, False), (0, True), (1, False), (2, False), (3, False), (4, True)])
@pytest.mark.parametrize("shape", [(7936, 768, 192), (2176, 2048, 64), (4224, 1920, 128)])
def test_gemm_two_tiles_per_unit(shape, epi, b_t):
    """257 .. 512 tiles of 128 x 128 in the forward and data-gradient layouts: one, two and three slices."""
    M, N, K = shape
    gemm_case(M, N, K, False, b_t, epi, seed=100 + epi)


@pytest.mark.parametrize("epi,b_t", [(0, False), (0, True), (1, False), (2, False), (3, False), (4, True)])
def test_gemm_streaming_outputs(epi, b_t):
    """Outputs of 64 MB and more are written, and their residual / pre-activation rows read, with non-temporal
    accesses (another copy of the epilogue code): 8192 x 4096 in bf16 is 64 MB."""
    gemm_case(8192, 4096, 128, False, b_t, epi, seed=70 + epi)


@pytest.mark.parametrize("epi", [0, 1, 2, 3, 6])
@pytest.mark.parametrize("shape", [(4096, 4096, 192), (8192, 4096, 128), (2560, 4096, 64)])
def test_gemm_four_wavefront_kernel_same_bits(epi, shape):
    """Forward products on 256 x 256 tiles run on four wavefronts of 128 x 128 (accumulators in place, epilogue on
    the accumulator layout); the instrumented library can send them to the eight-wavefront kernel instead.  Both
    accumulate in the same order and round once, so every output (C, the kept pre-activations, int8 codes and
    scales) has to agree bit for bit; 160, 256 and 512 tiles, cached and streaming stores, one to three slices."""
    M, N, K = shape
    lib = _lib()
    lib.swarm_kernel_gemm_ws.restype = C.c_int
    lib.swarm_kernel_gemm_ws.argtypes = [C.c_int] * 3 + [C.c_void_p, C.c_int, C.c_int, C.c_void_p, C.c_int, C.c_int,
                                                        C.c_void_p, C.c_int, C.c_int, C.c_void_p, C.c_void_p, C.c_int,
                                                        C.c_void_p, C.c_void_p, C.c_size_t, C.c_void_p]
    A = _bf(synth.normal(90 + epi, "A", (M, K))).cuda(); B = _bf(synth.normal(90 + epi, "B", (N, K))).cuda()
    bias = _bf(synth.normal(90 + epi, "bias", (N,))).cuda(); aux = _bf(synth.normal(90 + epi, "aux", (M, N))).cuda()
    outs = []
    for four in (1, 0):
        lib.swarm_kernel_gemm_four_waves(four)
        try:
            if epi == 6:
                Cd = torch.zeros((M, N), dtype=torch.int8, device="cuda")
                sc = torch.zeros(M * N // 64, dtype=torch.float32, device="cuda")
                st = lib.swarm_kernel_gemm_ws(M, N, K, A.data_ptr(), K, 0, B.data_ptr(), K, 0, Cd.data_ptr(), N, 6,
                                              bias.data_ptr(), aux.data_ptr(), N, sc.data_ptr(), None, 0, None)
                assert st == 0
                outs.append((Cd, sc.view(torch.int32)))
            else:
                res = []
                for keep_u in ((True, False) if epi == 3 else (False,)):
                    Cd = torch.full((M, N), 9.0, dtype=torch.bfloat16, device="cuda")
                    C2 = torch.full((M, N), 9.0, dtype=torch.bfloat16, device="cuda") if keep_u else None
                    st = lib.swarm_kernel_gemm(1, M, N, K, A.data_ptr(), K, 0, B.data_ptr(), K, 0, Cd.data_ptr(), N, epi,
                                               bias.data_ptr(), aux.data_ptr(), N,
                                               C2.data_ptr() if keep_u else None, N, None)
                    assert st == 0
                    res += [Cd.view(torch.int16)] + ([C2.view(torch.int16)] if keep_u else [])
                outs.append(tuple(res))
        finally:
            lib.swarm_kernel_gemm_four_waves(1)
    torch.cuda.synchronize()
    for a, b in zip(*outs):
        assert torch.equal(a, b)
    if epi == 3:      # with and without the kept pre-activations: the same GeLU values
        assert torch.equal(outs[0][0], outs[0][2])


def test_gemm_splitk_encode_equals_encode_of_stored():
    """EPI 6 (bias + residual, int8-encoded) through the split path: codes and scales are those of the stand-alone
    codec applied to what the bias + residual epilogue stores (same scratch, same summation order)."""
    import paper_2301_11913_amd as sw
    M, N, K = 512, 1024, 8192
    lib = _lib()
    A = _bf(synth.normal(3, "A", (M, K))); B = _bf(synth.normal(3, "B", (N, K)))
    bias = _bf(synth.normal(3, "bias", (N,))); aux = _bf(synth.normal(3, "aux", (M, N)))
    Ad, Bd, bd, xd = A.cuda(), B.cuda(), bias.cuda(), aux.cuda()
    lib.swarm_kernel_gemm_splitk_floats.restype = C.c_size_t
    ws = torch.empty(lib.swarm_kernel_gemm_splitk_floats(M, N), dtype=torch.float32, device="cuda")
    Cb = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    _splitk_call(lib, M, N, K, Ad, K, Bd, K, False, Cb, 2, bd, xd, None, ws)
    codes = torch.empty((M, N), dtype=torch.int8, device="cuda")
    scales = torch.empty(M * N // 64, dtype=torch.float32, device="cuda")
    _splitk_call(lib, M, N, K, Ad, K, Bd, K, False, codes, 6, bd, xd, scales, ws)
    c2 = torch.empty(M * N, dtype=torch.int8, device="cuda"); s2 = torch.empty_like(scales)
    sw.swarm_codec_encode(Cb.reshape(-1), c2, s2)
    torch.cuda.synchronize()
    assert torch.equal(codes.reshape(-1), c2) and torch.equal(scales.view(torch.int32), s2.view(torch.int32))


# The int8-encoding epilogue takes the route of bias + residual, whatever the number of tiles: codes and scales are those of
# the stand-alone codec on what that epilogue stores, bit for bit.  256 x 256 tiles, whole and with the last columns as a
# product of their own (cut along K, and not), 192 and 256 tiles of 256 x 128, 264 to 2080 of 128 x 128 with cached stores and
# (8320 x 4096) streaming ones, few tiles, ragged rows.
@pytest.mark.parametrize("shape", [(4096, 4096, 192), (8192, 2304, 320), (8192, 3072, 8192), (6144, 1024, 192),
                                   (2048, 4096, 448), (4224, 1024, 320), (7936, 768, 192), (8192, 1024, 128),
                                   (3840, 4096, 256), (1920, 8192, 192), (8064, 4160, 128), (8320, 4096, 128),
                                   (640, 768, 256), (4001, 1024, 192), (2500, 4096, 96)])
def test_gemm_encode_takes_the_route_of_the_store(shape):
    import paper_2301_11913_amd as sw
    M, N, K = shape
    lib = _lib()
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)
    A, B, bias, aux = rnd(M, K), rnd(N, K), rnd(N), rnd(M, N)
    lib.swarm_kernel_gemm_splitk_floats.restype = C.c_size_t
    ws = torch.empty(max(1, lib.swarm_kernel_gemm_splitk_floats(M, N), 2 * M * 1024), dtype=torch.float32, device="cuda")
    stored = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    _splitk_call(lib, M, N, K, A, K, B, K, False, stored, 2, bias, aux, None, ws)
    codes = torch.full((M * N,), 55, dtype=torch.int8, device="cuda")
    scales = torch.full((M * N // 64,), -3.0, device="cuda")
    _splitk_call(lib, M, N, K, A, K, B, K, False, codes, 6, bias, aux, scales, ws)
    want_codes, want_scales = torch.empty_like(codes), torch.empty_like(scales)
    sw.swarm_codec_encode(stored.reshape(-1), want_codes, want_scales)
    torch.cuda.synchronize()
    assert torch.equal(scales.view(torch.int32), want_scales.view(torch.int32))
    assert torch.equal(codes, want_codes)


# ------------------------------------------------------------------ attention
def _attn_lib():
    lib = _lib()
    lib.swarm_kernel_attention_fwd.restype = C.c_int
    lib.swarm_kernel_attention_fwd.argtypes = [C.c_int, C.c_void_p, C.c_void_p, C.c_void_p] + [C.c_int] * 4 + [C.c_void_p]
    lib.swarm_kernel_attention_bwd.restype = C.c_int
    lib.swarm_kernel_attention_bwd.argtypes = [C.c_int] + [C.c_void_p] * 6 + [C.c_int] * 4 + [C.c_void_p]
    return lib


def _attn_ref(qkv, dout, B, S, H, dh):
    """fp64 definition: per (b,h) causal softmax(q k^T / sqrt(dh)) v and its gradient."""
    d = H * dh
    x = qkv.reshape(B, S, 3, H, dh).transpose(2, 0, 3, 1, 4)       # [3,B,H,S,dh]
    q, k, v = x[0], x[1], x[2]
    s = q @ k.transpose(0, 1, 3, 2) / math.sqrt(dh)
    mask = np.tril(np.ones((S, S), dtype=bool))
    s = np.where(mask, s, -np.inf)
    mx = s.max(-1, keepdims=True)
    e = np.exp(s - mx)
    den = e.sum(-1, keepdims=True)
    p = e / den
    o = p @ v
    lse = (mx + np.log(den))[..., 0]
    do = dout.reshape(B, S, H, dh).transpose(0, 2, 1, 3)
    dv = p.transpose(0, 1, 3, 2) @ do
    dp = do @ v.transpose(0, 1, 3, 2)
    ds = p * (dp - (p * dp).sum(-1, keepdims=True))
    dq = ds @ k / math.sqrt(dh)
    dk = ds.transpose(0, 1, 3, 2) @ q / math.sqrt(dh)
    back = lambda t: t.transpose(0, 2, 1, 3).reshape(B, S, d)
    return back(o), lse, np.concatenate([back(dq), back(dk), back(dv)], axis=-1)


@pytest.mark.parametrize("shape", [(2, 128, 2, 64), (1, 512, 3, 128), (3, 37, 2, 128), (2, 200, 1, 64),
                                   (1, 1, 2, 64), (1, 1000, 2, 128), (2, 2048, 2, 128),
                                   (1, 4100, 1, 128), (1, 2500, 2, 64), (5, 129, 3, 128), (1, 191, 1, 64),
                                   (2, 70, 3, 32)])       # a head size only the direct kernels take
def test_attention_bf16(shape):
    _attention_case(shape, 1.5)


# either side of 256 tiles of 128 rows (single tiles on two groups of wavefronts, then pairs of tiles), odd tile counts, and
# lengths where the second group has no tile or only a masked one
@pytest.mark.parametrize("shape", [(2, 129, 64, 64), (3, 300, 29, 64), (2, 65, 128, 128), (17, 200, 8, 128),
                                   (2, 64, 3, 64), (1, 65, 2, 128)])
def test_attention_bf16_launch_layouts(shape):
    _attention_case(shape, 1.5)


# up to 256 tiles: one group of wavefronts while a row has fewer than four (d_head 64) or six (128) tiles of 64 keys, then two
@pytest.mark.parametrize("shape", [(3, 192, 4, 64), (3, 193, 4, 64), (2, 256, 4, 64), (1, 257, 3, 64), (2, 320, 3, 128),
                                   (2, 321, 3, 128), (1, 384, 3, 128), (40, 64, 6, 64), (40, 33, 6, 128),
                                   # pairs of tiles, one pair per unit: either side of 8 (16) tiles of 64 keys, odd counts
                                   (10, 448, 7, 64), (9, 450, 8, 64), (5, 600, 11, 64), (2, 1000, 17, 128), (2, 960, 17, 128)])
def test_attention_bf16_wavefront_groups(shape):
    _attention_case(shape, 1.5)

@pytest.mark.parametrize("shape", [(1, 300, 2, 128), (2, 200, 2, 64), (1, 1100, 1, 128)])
def test_attention_bf16_peaked_scores(shape):
    """Scores with a standard deviation of several tens: nearly one-hot softmax rows, the running reference of the
    exponentials is raised again and again along a row, earlier keys underflow to exact zeros."""
    _attention_case(shape, 6.0)


def _attention_case(shape, std):
    B, S, H, dh = shape
    lib = _attn_lib()
    d = H * dh
    qkv = _bf(synth.normal(S + dh, "qkv", (B, S, 3 * d), std=std))
    dout = _bf(synth.normal(S + dh, "dout", (B, S, d)))
    ro, rlse, rdqkv = _attn_ref(qkv.double().numpy(), dout.double().numpy(), B, S, H, dh)
    qd, dod = qkv.cuda(), dout.cuda()
    o = torch.full((B, S, d), 9.0, dtype=torch.bfloat16, device="cuda")
    lse = torch.full((B, H, S), 9.0, dtype=torch.float32, device="cuda")
    assert lib.swarm_kernel_attention_fwd(1, qd.data_ptr(), o.data_ptr(), lse.data_ptr(), B, S, H, dh, None) == 0
    torch.cuda.synchronize()
    eo = np.max(np.abs(o.double().cpu().numpy() - ro)) / np.max(np.abs(ro))
    el = np.max(np.abs(lse.double().cpu().numpy() - rlse))
    assert eo < 1e-2, eo
    assert el < 2e-2, el
    delta = torch.empty((B, H, S), dtype=torch.float32, device="cuda")
    dqkv = torch.full((B, S, 3 * d), 9.0, dtype=torch.bfloat16, device="cuda")
    assert lib.swarm_kernel_attention_bwd(1, qd.data_ptr(), o.data_ptr(), dod.data_ptr(), lse.data_ptr(),
                                          delta.data_ptr(), dqkv.data_ptr(), B, S, H, dh, None) == 0
    torch.cuda.synchronize()
    got = dqkv.double().cpu().numpy()
    for name, sl in (("dq", slice(0, d)), ("dk", slice(d, 2 * d)), ("dv", slice(2 * d, 3 * d))):
        den = max(np.max(np.abs(rdqkv[..., sl])), 1e-3 * np.max(np.abs(rdqkv)))   # S = 1 has dq = dk = 0 exactly
        e = np.max(np.abs(got[..., sl] - rdqkv[..., sl])) / den
        assert e < 1.5e-2, (name, e)


# fp32 attention: tiles of 32 over four wavefronts - one row, a tile short of or past a full one, fewer blocks than
# wavefronts, many blocks, peaked scores, and a head size only the direct kernels take.
@pytest.mark.parametrize("shape,std", [((2, 128, 3, 64), 1.5), ((1, 1, 2, 64), 1.5), ((3, 31, 2, 128), 1.5),
                                       ((2, 33, 1, 64), 1.5), ((1, 161, 2, 128), 1.5), ((1, 1000, 2, 64), 1.5),
                                       ((2, 300, 2, 128), 6.0), ((1, 1100, 1, 64), 6.0), ((2, 70, 3, 32), 1.5)])
def test_attention_f32(shape, std):
    B, S, H, dh = shape
    lib, d = _attn_lib(), H * dh
    qkv = torch.from_numpy(synth.normal(S + dh, "qkv", (B, S, 3 * d), std=std)).float()
    dout = torch.from_numpy(synth.normal(S + dh, "dout", (B, S, d))).float()
    ro, rlse, rdqkv = _attn_ref(qkv.double().numpy(), dout.double().numpy(), B, S, H, dh)
    qd, dod = qkv.cuda(), dout.cuda()
    o, lse, dqkv = torch.full_like(dod, 9.0), torch.full((B, H, S), 9.0, device="cuda"), torch.full_like(qd, 9.0)
    delta = torch.empty_like(lse)
    assert lib.swarm_kernel_attention_fwd(0, qd.data_ptr(), o.data_ptr(), lse.data_ptr(), B, S, H, dh, None) == 0
    assert lib.swarm_kernel_attention_bwd(0, qd.data_ptr(), o.data_ptr(), dod.data_ptr(), lse.data_ptr(), delta.data_ptr(),
                                          dqkv.data_ptr(), B, S, H, dh, None) == 0
    torch.cuda.synchronize()
    # a score is a sum of dh products of size std^2: off by up to about 2^-24 sqrt(dh) std^2 sqrt(dh) / sqrt(dh), and a
    # probability is off by the same relatively
    tol = 2.0 ** -24 * (16 + 4 * math.sqrt(dh) * std * std)
    assert np.max(np.abs(o.double().cpu().numpy() - ro)) <= tol * np.max(np.abs(ro))
    assert np.max(np.abs(lse.double().cpu().numpy() - rlse)) <= tol * max(1, np.max(np.abs(rlse)))
    got = dqkv.double().cpu().numpy()
    # dp - delta: two sums of dh products of size std that may cancel (S = 1: exactly), times a row of size std
    floor = 2.0 ** -24 * 4 * math.sqrt(dh) * std * std
    for i in range(3):
        part = slice(i * d, (i + 1) * d)
        assert np.max(np.abs(got[..., part] - rdqkv[..., part])) <= 4 * tol * np.max(np.abs(rdqkv[..., part])) + floor


# fp32 calls either side of the line between the direct kernels and the matrix cores: B H S^2 = 512 d_head, S = d_head
@pytest.mark.parametrize("shape", [(1, 64, 8, 64), (1, 64, 9, 64), (2, 65, 1, 64), (8, 32, 4, 64), (8, 33, 4, 64), (1, 1, 3, 128),
                                   (1, 128, 4, 128), (1, 128, 5, 128), (1, 129, 2, 128), (64, 32, 1, 128)])
def test_attention_f32_few_short_rows(shape):
    test_attention_f32(shape, 1.5)


# The row sums of dO O that the backward leaves for dK / dV: one product of 1 and dh - 1 of less than half a unit of it.  Halves
# added to halves lose at most half a unit (2^-24) per addition on the way of the 1: bf16 seven in its eight columns and
# log2(dh / 8) behind, fp32 log2(dh).  One running sum of the dh / 2 products of a lane loses dh / 2 - 1 of them whole (fp32: 2^-26
# each, in fours).
@pytest.mark.parametrize("bf16,dh", [(1, 64), (1, 128), (0, 64), (0, 128)])
@pytest.mark.parametrize("at", [0, 1])
def test_attention_row_sums(bf16, dh, at):
    B, S, H = 1, 300, 2
    lib, dt = _attn_lib(), torch.bfloat16 if bf16 else torch.float32
    o, dout = (torch.full((B, S, H, dh), 2.0 ** -e, dtype=dt) for e in ((12, 13) if bf16 else (13, 13)))
    col = at * (8 if bf16 else 4)
    o[..., col] = 1
    dout[..., col] = 1
    qkv = torch.zeros((B, S, 3 * H * dh), dtype=dt, device="cuda")
    od, dod, dqkv = o.cuda(), dout.cuda(), torch.empty_like(qkv)
    lse = torch.arange(1, S + 1, dtype=torch.float32).log().expand(B, H, S).contiguous().cuda()
    delta = torch.full((B, H, S), 9.0, device="cuda")
    assert lib.swarm_kernel_attention_bwd(bf16, qkv.data_ptr(), od.data_ptr(), dod.data_ptr(), lse.data_ptr(), delta.data_ptr(),
                                          dqkv.data_ptr(), B, S, H, dh, None) == 0
    torch.cuda.synchronize()
    want = (o.double() * dout.double()).sum(-1).transpose(1, 2)
    additions = 7 + int(math.log2(dh // 8)) if bf16 else int(math.log2(dh))
    assert ((delta.double().cpu() - want).abs() <= additions * 2.0 ** -24).all()


def _attention_f32_run(qkv, dout, B, S, H, dh):
    lib = _attn_lib()
    qd, dod = qkv.cuda(), dout.cuda()
    o, lse, dqkv = torch.full_like(dod, 9.0), torch.full((B, H, S), 9.0, device="cuda"), torch.full_like(qd, 9.0)
    delta = torch.empty_like(lse)
    assert lib.swarm_kernel_attention_fwd(0, qd.data_ptr(), o.data_ptr(), lse.data_ptr(), B, S, H, dh, None) == 0
    assert lib.swarm_kernel_attention_bwd(0, qd.data_ptr(), o.data_ptr(), dod.data_ptr(), lse.data_ptr(), delta.data_ptr(),
                                          dqkv.data_ptr(), B, S, H, dh, None) == 0
    torch.cuda.synchronize()
    return o.cpu(), lse.cpu(), dqkv.cpu()


# A value that is not finite reaches only what depends on it: everything else is what it is without it, to the rounding of
# another order of at most S additions in the rows of the same block, bit for bit elsewhere.  Row `bad` of one of q, k, v
# (parts 0..2) or of dout (3), inside a block of 32 rows, first and last of one, in a last block that is short.
@pytest.mark.parametrize("value", [math.inf, -math.inf, math.nan])
@pytest.mark.parametrize("part", [0, 1, 2, 3])
@pytest.mark.parametrize("S,bad,dh", [(150, 45, 64), (150, 64, 64), (150, 149, 128), (200, 95, 128), (300, 17, 128)])
def test_attention_f32_keeps_masked_positions_apart(S, bad, dh, part, value):
    B, H, h = 2, 4, 1
    d = H * dh
    g = torch.Generator().manual_seed(S + dh)
    qkv, dout = torch.randn((B, S, 3 * d), generator=g), torch.randn((B, S, d), generator=g)
    clean = _attention_f32_run(qkv, dout, B, S, H, dh)
    if part < 3:
        qkv[0, bad, part * d + h * dh + 5] = value
    else:
        dout[0, bad, h * dh + 5] = value
    got = _attention_f32_run(qkv, dout, B, S, H, dh)
    views = lambda x: (x[0].view(B, S, H, dh), x[1], x[2].view(B, S, 3, H, dh))
    (o, lse, grads), (co, clse, cgrads) = views(got), views(clean)
    bound = S * 2.0 ** -24
    same = lambda a, b: bool((a == b).all())
    close = lambda a, b: bool(((a - b).abs() <= bound * b.abs().max()).all())
    other = [x for x in range(H) if x != h]
    assert same(o[1], co[1]) and same(lse[1], clse[1]) and same(grads[1], cgrads[1])             # the other sequence
    assert same(o[0][:, other], co[0][:, other]) and same(grads[0][:, :, other], cgrads[0][:, :, other])   # the other heads
    first = bad // 32 * 32                                                                       # earlier queries
    assert same(o[0, :first, h], co[0, :first, h]) and same(lse[0, h, :bad], clse[0, h, :bad])
    assert same(grads[0, :first, 0, h], cgrads[0, :first, 0, h])
    if bad > first:
        assert close(o[0, first:bad, h], co[0, first:bad, h]) and close(grads[0, first:bad, 0, h], cgrads[0, first:bad, 0, h])
    if part in (0, 3) and bad + 1 < S:      # a query (or its gradient) touches its own row and earlier keys only
        assert close(o[0, bad + 1:, h], co[0, bad + 1:, h]) and same(lse[0, h, bad + 1:], clse[0, h, bad + 1:])
        assert close(grads[0, bad + 1:, :, h], cgrads[0, bad + 1:, :, h])
    assert not torch.isfinite(torch.cat([got[0][0, bad], got[2][0, bad]])).all()                 # and its own row shows it


def test_attention_f32_scores_of_minus_infinity():
    """Keys whose scores overflow to -inf have no weight, also where they are all the keys that one wavefront takes; a row in
    which every score does gives NaN."""
    B, S, H, dh = 2, 260, 4, 64
    d = H * dh
    g = torch.Generator().manual_seed(5)
    qkv, dout = torch.randn((B, S, 3 * d), generator=g), torch.randn((B, S, d), generator=g)
    qkv[0, 200:, 7] = 3e38                     # queries 200 .. of head 0
    keys = torch.arange(S)
    hidden = (keys // 32 % 4 == 2) & (keys < 200)
    qkv[0, hidden, d + 7] = -4.0               # q k = -1.2e39 there, and 0 for this column elsewhere
    qkv[0, ~hidden, d + 7] = 0.0
    o, lse, dqkv = _attention_f32_run(qkv, dout, B, S, H, dh)
    x = qkv.double().view(B, S, 3, H, dh).permute(2, 0, 3, 1, 4)
    x[0][0, 0, 200:, 7] = 0.0                  # the same scores without the overflow: masked where it happens
    s = x[0] @ x[1].transpose(-1, -2) / math.sqrt(dh)
    mask = torch.tril(torch.ones(S, S, dtype=torch.bool)).expand(B, H, S, S).clone()
    mask[0, 0, 200:, hidden] = False
    s = s.masked_fill(~mask, -math.inf)
    want = (torch.softmax(s, -1) @ x[2]).permute(0, 2, 1, 3).reshape(B, S, d)
    assert torch.isfinite(o).all() and torch.isfinite(lse).all()
    assert (o.double() - want).abs().max() <= 1e-5 * want.abs().max()
    assert (lse.double() - torch.logsumexp(s, -1)).abs().max() <= 1e-5 * 6
    qkv[1, :, d + 7], qkv[1, 100, 7] = -4.0, 3e38     # every score of this row
    o, lse, dqkv = _attention_f32_run(qkv, dout, B, S, H, dh)
    assert torch.isnan(o[1, 100, :dh]).all() and torch.isfinite(o[1, :100]).all() and torch.isfinite(o[1, 101:]).all()


# fp32 GEMM on the matrix cores: every workgroup shape of its dispatch (32 x 32 blocks with K over 8 or 4 wavefronts,
# 64 x 64, 128 x 128), ragged rows and columns, a K that leaves a partial slice and (transposed operands) a partial
# 8-deep step, fewer 8-deep steps than wavefronts, every epilogue.
@pytest.mark.parametrize("M,N,K,a_t,b_t,epi", [
    (512, 256, 256, False, False, 2), (512, 1024, 256, False, False, 3), (33, 64, 64, False, False, 1),
    (1, 68, 8, False, False, 0), (1030, 1028, 72, False, False, 2), (2049, 2052, 64, False, False, 3),
    (512, 256, 768, False, True, 0), (77, 1024, 256, False, True, 4), (1665, 768, 104, False, True, 4),
    (2085, 2048, 64, False, True, 0), (256, 1024, 511, True, True, 5), (768, 256, 37, True, True, 5),
    (1024, 1024, 203, True, True, 5), (2048, 2304, 130, True, True, 5), (100, 36, 5, True, True, 5),
    (64, 30, 64, False, False, 1), (64, 64, 60, False, False, 0),
    # either side of the tile counts that the dispatch changes at
    (3390, 188, 72, False, False, 2), (1021, 640, 72, False, False, 3), (3390, 188, 8, False, False, 0),
    (15290, 60, 40, False, True, 0), (953, 1024, 104, False, True, 4), (960, 1024, 8, False, True, 0),
    (19070, 380, 64, False, False, 1), (3581, 2048, 64, False, False, 3), (3581, 2044, 40, False, True, 4),
    (1344, 1212, 65, True, True, 5), (1280, 1276, 37, True, True, 5), (4096, 4092, 33, True, True, 5)])
def test_gemm_f32(M, N, K, a_t, b_t, epi):
    lib = _lib()
    g = torch.Generator().manual_seed(M + N + K)
    rnd = lambda *s: torch.randn(s, generator=g)
    A, B, bias, aux, C0 = rnd(*((K, M) if a_t else (M, K))), rnd(*((K, N) if b_t else (N, K))), rnd(N), rnd(M, N), rnd(M, N)
    A64, B64 = (A.T if a_t else A).double(), (B if b_t else B.T).double()
    ref, size = A64 @ B64, A64.abs() @ B64.abs()
    Ad, Bd, bd, xd, Cd = (t.cuda() for t in (A, B, bias, aux, C0))
    C2 = torch.full((M, N), 9.0, device="cuda")
    s = lib.swarm_kernel_gemm(0, M, N, K, Ad.data_ptr(), A.shape[1], a_t, Bd.data_ptr(), B.shape[1], b_t, Cd.data_ptr(),
                              N, epi, bd.data_ptr(), xd.data_ptr(), N, C2.data_ptr() if epi == 3 else None, N, None)
    torch.cuda.synchronize()
    assert s == 0
    # K products and K additions, each off by half an ulp of at most the sum of magnitudes; two more for the epilogue
    bound = (2 * K + 2) * 2.0 ** -24
    if epi in (1, 2, 3):
        ref, size = ref + bias.double(), size + bias.double().abs()
    if epi == 2:
        ref, size = ref + aux.double(), size + aux.double().abs()
    if epi == 5:
        ref, size = ref + C0.double(), size + C0.double().abs()
    if epi == 3:
        assert ((C2.cpu().double() - ref).abs() <= bound * size).all()
        ref = torch.from_numpy(_gelu(ref.numpy()))
        size = 1.13 * size + 8 / bound * 2.0 ** -24 * ref.abs().clamp(min=1)     # slope of GeLU; a few ulp of erf
    if epi == 4:
        d = torch.from_numpy(_gelu_grad(aux.double().numpy()))
        size = size * d.abs() + 8 / bound * 2.0 ** -24 * ref.abs()
        ref = ref * d
    assert ((Cd.cpu().double() - ref).abs() <= bound * size).all()


# Kernel with K over the wavefronts (few tiles or ragged): both tile sizes, both stage counts, one row / one past a tile
# in every ragged dimension, K of one wavefront's 32, half a slice, fewer slices than stages and an odd number of them.
# The operands lie in front of NaNs: nothing behind them may reach a result.
@pytest.mark.parametrize("M,N,K,a_t,b_t,epi", [
    (1, 64, 32, False, False, 0), (65, 72, 96, False, False, 1), (512, 1024, 1024, False, False, 2),
    (333, 192, 288, False, False, 3), (1665, 2304, 768, False, False, 1), (1700, 3080, 160, False, False, 0),
    (63, 8, 64, False, True, 0), (129, 200, 352, False, True, 4), (1665, 768, 2304, False, True, 0),
    (1921, 1992, 96, False, True, 4), (1100, 1992, 224, False, True, 0),
    (8, 8, 1, True, True, 5), (72, 136, 63, True, True, 5), (768, 768, 1665, True, True, 5),
    (1536, 2304, 257, True, True, 5), (1024, 1160, 130, True, True, 5)])
def test_gemm_ragged_and_small(M, N, K, a_t, b_t, epi):
    lib = _lib()
    seed = 3 * M + N + K
    operand = lambda name, *shape: _bf(synth.normal(seed, name, shape))
    A, B = operand("A", *((K, M) if a_t else (M, K))), operand("B", *((K, N) if b_t else (N, K)))
    bias, aux = operand("bias", N), operand("aux", M, N)
    ref = (A.T if a_t else A).double().numpy() @ (B if b_t else B.T).double().numpy()
    fenced = lambda t: torch.cat([t.reshape(-1), torch.full((1 << 16,), float("nan"), dtype=t.dtype)]).cuda()
    Ad, Bd, bd, xd = (fenced(t) for t in (A, B, bias, aux))
    out = torch.float32 if epi == 5 else torch.bfloat16
    Cd = torch.full((M + 1, N), 3.0, dtype=out, device="cuda")
    C2 = torch.full((M + 1, N), 3.0, dtype=out, device="cuda")
    st = lib.swarm_kernel_gemm(1, M, N, K, Ad.data_ptr(), A.shape[1], a_t, Bd.data_ptr(), B.shape[1], b_t, Cd.data_ptr(), N,
                               epi, bd.data_ptr(), xd.data_ptr(), N, C2.data_ptr() if epi == 3 else None, N, None)
    torch.cuda.synchronize()
    assert st == 0
    assert (Cd[M] == 3).all() and (C2[M] == 3).all()
    if epi in (1, 2, 3):
        ref = ref + bias.double().numpy()
    if epi == 2:
        ref = ref + aux.double().numpy()
    if epi == 3:
        assert np.max(np.abs(C2[:M].double().cpu().numpy() - ref)) <= 6e-3 * np.max(np.abs(ref))
        ref = _gelu(ref)
    if epi == 4:
        ref = ref * _gelu_grad(aux.double().numpy())
    if epi == 5:
        ref = ref + 3.0
    # half a bf16 ulp of the largest result (2^-9 = 2e-3) with room for the epilogue's input roundings; fp32: the sums
    assert np.max(np.abs(Cd[:M].double().cpu().numpy() - ref)) <= (1e-5 if epi == 5 else 6e-3) * np.max(np.abs(ref))


# Either side of one round of 64 x 64 tiles (512), and what replaces those between 256 and 512: 128 x 64 tiles, or 64 x 64
# where 128 rows would be half empty.  One slice and part of one, fewer than stages, an odd number, in every layout.
@pytest.mark.parametrize("M,N,K,a_t,b_t,epi", [
    (2048, 1024, 192, False, False, 2), (2048, 1088, 192, False, False, 2), (1999, 1032, 96, False, False, 1),
    (1665, 768, 32, False, False, 1), (1700, 904, 288, False, False, 3), (1665, 768, 416, False, True, 0),
    (1921, 776, 96, False, True, 4), (1544, 768, 333, True, True, 5), (1664, 712, 1, True, True, 5),
    (64, 19264, 96, False, False, 0), (57, 20000, 160, False, True, 0)])
def test_gemm_rounds_of_small_tiles(M, N, K, a_t, b_t, epi):
    test_gemm_ragged_and_small(M, N, K, a_t, b_t, epi)


# Tiles of 16 and 32 rows for the fewest: one row, one more than a tile, either side of a round of each (256 workgroups) and of the
# K that the 16 rows start at, a K that leaves wavefronts without a part, fewer slices than stages and an odd number of them.
@pytest.mark.parametrize("M,N,K,a_t,b_t,epi", [
    (1, 64, 1024, False, False, 0), (17, 72, 1056, False, False, 1), (256, 1024, 1120, False, False, 2),
    (257, 1024, 1024, False, False, 3), (250, 1024, 992, False, False, 1), (33, 200, 4096, False, True, 4),
    (4096, 64, 1312, False, True, 0), (64, 4096, 2080, False, True, 0), (33, 64, 32, False, False, 0),
    (512, 1024, 96, False, False, 2), (513, 1024, 96, False, False, 3), (8192, 64, 352, False, False, 1),
    (31, 16384, 64, False, True, 4), (500, 1000, 256, False, True, 0), (8190, 56, 992, False, True, 4)])
def test_gemm_few_rows(M, N, K, a_t, b_t, epi):
    test_gemm_ragged_and_small(M, N, K, a_t, b_t, epi)


# Whole 128 x 128 tiles, two workgroups per unit: either side of 128, 256, 512 and 768 of them, one slice, an odd number and
# the longest K of its rules, every layout and epilogue (rotary, GeGLU and the encoding one through the stage tests).
@pytest.mark.parametrize("M,N,K,a_t,b_t,epi", [
    (1408, 1536, 64, False, False, 0), (1408, 1536, 512, False, False, 1), (1024, 2048, 192, False, False, 3),
    (640, 6656, 192, False, False, 2), (2176, 2176, 128, False, False, 1), (1664, 5120, 192, False, False, 3),
    (8064, 4224, 64, False, False, 0), (1408, 1536, 320, False, True, 0), (2176, 2176, 64, False, True, 4),
    (2944, 3456, 192, False, True, 0), (4480, 2944, 128, False, True, 4), (2944, 2944, 2048, False, True, 4),
    (1152, 2304, 64, True, True, 5), (1152, 4608, 448, True, True, 5), (3200, 3200, 192, True, True, 5),
    (3200, 3200, 2048, True, True, 5), (3200, 4480, 64, True, True, 5)])
def test_gemm_two_workgroups_per_unit(M, N, K, a_t, b_t, epi):
    test_gemm_ragged_and_small(M, N, K, a_t, b_t, epi)


# Ragged products either side of the line between the register-staged kernel and the one with K over the wavefronts: rows that
# fill most of a round of 256-row tiles and rows that do not, K at and past the limits, outputs large enough for streaming
# stores.
@pytest.mark.parametrize("M,N,K,a_t,b_t,epi", [
    (2500, 2048, 512, False, False, 3), (1500, 3072, 1024, False, False, 1), (1500, 3072, 1056, False, False, 1),
    (6001, 1536, 512, False, False, 2), (4001, 4096, 96, False, False, 3), (5000, 3072, 160, False, False, 2),
    (2600, 4096, 96, False, False, 1), (3900, 4096, 4128, False, False, 0), (5000, 1024, 256, False, True, 4),
    (4001, 4096, 96, False, True, 0), (1536, 4608, 65, True, True, 5), (1536, 4608, 641, True, True, 5),
    (3072, 3072, 321, True, True, 5), (4096, 4096, 130, True, True, 5), (4104, 4000, 1, True, True, 5),
    (3072, 4096, 700, True, True, 5), (4104, 4104, 65, True, True, 5), (16392, 1544, 200, True, True, 5), (8200, 4096, 64, False, False, 2), (8200, 4096, 96, False, False, 3),
    (8200, 4104, 64, False, True, 4), (8200, 4104, 96, False, True, 0), (8200, 3904, 64, True, True, 5),
    # K no multiple of 32: the register-staged kernel only, on both of its tiles
    (4096, 2560, 72, False, True, 0), (4104, 2560, 40, False, False, 1), (300, 256, 136, False, True, 4),
    (130, 264, 24, False, False, 3), (64, 19200, 65, True, True, 5)])
def test_gemm_ragged_routes(M, N, K, a_t, b_t, epi):
    test_gemm_ragged_and_small(M, N, K, a_t, b_t, epi)


# Ragged products on the kernels of whole tiles, whose last tile ends with the operand: either side of each of their rules (256 and
# 512 tiles of 128 x 128, 320 for a long K, full and not so full rounds), one row or eight columns past a tile, the fewest rows.
@pytest.mark.parametrize("M,N,K,a_t,b_t,epi", [
    (257, 11016, 192, False, False, 1), (2085, 2056, 64, False, False, 2), (2500, 2312, 2112, False, False, 2),
    (2500, 2312, 2048, False, False, 0), (300, 22024, 768, False, False, 3), (2309, 4104, 768, False, False, 0),
    (2309, 4104, 704, False, False, 2), (4100, 2568, 64, False, False, 3), (4097, 5128, 832, False, False, 1),
    (5001, 8200, 768, False, False, 2), (2085, 2056, 64, False, True, 4), (2500, 2312, 1600, False, True, 0),
    (2500, 2312, 1536, False, True, 4), (2309, 4104, 2048, False, True, 0), (3333, 4104, 64, False, True, 4),
    (4100, 2568, 128, False, True, 0), (5001, 8200, 128, False, True, 4), (2176, 2184, 64, False, False, 1),
    # an output that is added to: on tiles that do not overlap
    (2085, 2056, 64, False, False, 5), (2309, 4104, 768, False, False, 5), (2500, 2312, 2112, False, False, 5),
    (2085, 2056, 64, False, True, 5), (2309, 4104, 2048, False, True, 5)])
def test_gemm_overlapping_tiles(M, N, K, a_t, b_t, epi):
    test_gemm_ragged_and_small(M, N, K, a_t, b_t, epi)


# In place (the second operand of the epilogue is the output): every row is added to once, whatever the tiles.
@pytest.mark.parametrize("M,N,K,b_t,epi", [(2309, 4104, 768, False, 2), (2500, 2312, 2112, False, 2), (2085, 2056, 64, True, 4)])
def test_gemm_ragged_in_place(M, N, K, b_t, epi):
    lib = _lib()
    A, B, aux = (_bf(synth.normal(7, n, s)).cuda() for n, s in (("A", (M, K)), ("B", (K, N) if b_t else (N, K)), ("x", (M, N))))
    bias, got = _bf(synth.normal(7, "b", (N,))).cuda(), aux.clone()
    apart = torch.empty_like(aux)
    for x, c in ((aux, apart), (got, got)):
        assert lib.swarm_kernel_gemm(1, M, N, K, A.data_ptr(), K, 0, B.data_ptr(), B.shape[1], b_t, c.data_ptr(), N, epi,
                                     bias.data_ptr(), x.data_ptr(), N, None, N, None) == 0
    torch.cuda.synchronize()
    a, b = apart.double(), got.double()
    # two kernels, two orders of the same sums: one bf16 unit of the largest result
    assert (a - b).abs().max() <= 2.0 ** -7 * a.abs().max()


# Row sums of the left operand beside a weight gradient (the bias gradient), where the product's kernel takes them along:
# one tile, fewer and more columns of tiles than fragment rows, ragged rows and token counts, both dtypes.
@pytest.mark.parametrize("bf16,M,N,K", [(1, 64, 64, 33), (1, 200, 128, 333), (1, 768, 192, 1665), (1, 768, 3072, 130),
                                        (1, 1536, 2304, 257), (1, 1536, 768, 333), (1, 2048, 1024, 4096), (0, 64, 64, 33), (0, 256, 1024, 511),
                                        (0, 1000, 260, 77), (0, 1024, 1024, 203), (0, 2048, 2304, 130)])
def test_weight_gradient_row_sums(bf16, M, N, K):
    lib = _lib()
    lib.swarm_kernel_gemm_rowsum.argtypes = [C.c_int] * 4 + [C.c_void_p] * 5
    g = torch.Generator().manual_seed(M + N + K)
    dt = torch.bfloat16 if bf16 else torch.float32
    A, B = (torch.randn((K, n), generator=g).to(dt) for n in (M, N))
    db0, dW0 = torch.randn(M, generator=g), torch.randn((M, N), generator=g)
    Ad, Bd, db, dW = A.cuda(), B.cuda(), db0.cuda(), dW0.cuda()
    assert lib.swarm_kernel_gemm_rowsum(bf16, M, N, K, Ad.data_ptr(), Bd.data_ptr(), dW.data_ptr(), db.data_ptr(), None) == 0
    torch.cuda.synchronize()
    A, B = A.double(), B.double()
    # K additions (and products), each off by half an ulp of at most the sum of magnitudes
    assert ((db.cpu() - (db0 + A.sum(0))).abs() <= (K + 1) * 2.0 ** -24 * (A.abs().sum(0) + db0.abs())).all()
    assert ((dW.cpu() - (dW0 + A.T @ B)).abs() <= (2 * K + 1) * 2.0 ** -24 * (A.abs().T @ B.abs() + dW0.abs())).all()


# How often the bias gradient is rounded: positive values are added up, so every rounding is one of a growing running sum.  In units of
# the result, root mean square: fp32, values of 1..2, sums of four, doubles over the rest and one rounding at the end, 0.29 (with a
# quarter of K rounded by each wavefront and added up in fp32 0.5).  bf16 on 256 x 256 tiles, values that differ by up to 2^16: the sum of
# 2048 rows in two runs of 32 multiplies, each ending at half of it and so with half the roundings: 1.55 (in one run of 64 3.05).
@pytest.mark.parametrize("bf16,K,shapes,units", [
    (0, 512, [(256, 1024), (1024, 256), (256, 256), (768, 256)], 0.4), (0, 1000, [(1024, 1024), (1024, 2048)], 0.4),
    (1, 2048, [(1024, 4096), (4096, 1024), (1024, 1024), (3072, 1024)], 2.2)])
def test_bias_gradient_rounding(bf16, K, shapes, units):
    lib = _lib()
    g = torch.Generator().manual_seed(K)
    dt = torch.bfloat16 if bf16 else torch.float32
    A, B = ([((1 + torch.rand((K, s[i]), generator=g)) * 2.0 ** -torch.randint(0, 16 if bf16 else 1, (K, s[i]), generator=g)).to(dt)
             for s in shapes] for i in (0, 1))
    dev = [[a.cuda(), b.cuda(), torch.zeros(s, device="cuda"), torch.zeros(s[0], device="cuda")] for a, b, s in zip(A, B, shapes)]
    mn = (C.c_int * (2 * len(shapes)))(*[x for s in shapes for x in s])
    ptrs = (C.c_void_p * (4 * len(shapes)))(*[t.data_ptr() for p in dev for t in p])
    lib.swarm_kernel_wgrads.argtypes = [C.c_int, C.c_int, C.c_void_p, C.c_int, C.c_void_p, C.c_void_p]
    assert lib.swarm_kernel_wgrads(bf16, len(shapes), mn, K, ptrs, None) == 0
    torch.cuda.synchronize()
    for a, d in zip(A, dev):
        want = a.double().sum(0)
        off = (d[3].double().cpu() - want) / 2.0 ** (torch.floor(torch.log2(want)) - 23)
        assert off.square().mean().sqrt() <= units


# Several weight gradients over the same rows in one launch, bias gradients with them: every tile shape (64 x 64 with four and two
# stages, 128 x 64, 128 x 128, 256 x 256; fp32 32, 64 and 128), each with one k value, a whole slice and parts of one, ragged M
# and N, products smaller than a tile beside larger ones, and shares of the launch that are no multiple of 8 tiles.
@pytest.mark.parametrize("bf16,K,shapes", [
    (1, 1, [(64, 64), (192, 64)]), (1, 333, [(264, 520), (8, 264), (200, 72)]), (1, 130, [(136, 1032), (520, 2056), (264, 1032)]),
    (1, 65, [(640, 640), (640, 640), (320, 704)]), (1, 513, [(1000, 1096), (512, 512), (768, 264), (24, 2048)]),
    (1, 513, [(768, 1536), (1536, 768), (768, 768), (2304, 768)]), (1, 1, [(1032, 4104), (4104, 1032), (264, 1032), (520, 1032)]),
    (1, 63, [(1032, 4104), (4104, 1032), (264, 1032), (3096, 1032)]), (1, 64, [(1024, 4096), (4096, 1024), (1024, 1024), (3072, 1024)]),
    (1, 2113, [(1032, 4104), (4104, 1032), (1032, 1032), (3096, 1032)]), (1, 129, [(3080, 4104), (8, 264)]),
    (0, 1, [(64, 64), (33, 36)]), (0, 77, [(256, 1024), (1024, 256), (256, 256), (768, 256)]),
    (0, 130, [(1000, 1028), (777, 516), (64, 64)]), (0, 203, [(1024, 4096), (2052, 1024), (300, 68)]),
    (0, 33, [(4096, 4092), (132, 260)])])
def test_weight_gradients_in_one_launch(bf16, K, shapes):
    lib = _lib()
    g = torch.Generator(device="cuda").manual_seed(K + sum(map(sum, shapes)))
    dt = torch.bfloat16 if bf16 else torch.float32
    rn = lambda *s: torch.randn(s, generator=g, device="cuda")
    t = [(rn(K, M).to(dt), rn(K, N).to(dt), rn(M, N), rn(M)) for M, N in shapes]
    want = [(A.double().T @ B.double() + W.double(), A.double().sum(0) + b.double(),
             A.double().abs().T @ B.double().abs() + W.double().abs(), A.double().abs().sum(0) + b.double().abs())
            for A, B, W, b in t]
    for q in t[1::3]:                 # a bias gradient may be left out
        q[3].fill_(7.0)
    ptrs = [v.data_ptr() if j < 3 or i % 3 != 1 else None for i, q in enumerate(t) for j, v in enumerate(q)]
    flat = [v for s in shapes for v in s]
    call = lambda p: lib.swarm_kernel_wgrads(bf16, len(shapes), (C.c_int * len(flat))(*flat), K, (C.c_void_p * len(p))(*p), None)
    assert call(ptrs) == 0
    torch.cuda.synchronize()
    # K additions (and products), each off by half an ulp of at most the sum of magnitudes
    for i, ((A, B, W, b), (w64, b64, wsize, bsize)) in enumerate(zip(t, want)):
        assert ((W.double() - w64).abs() <= (2 * K + 1) * 2.0 ** -24 * wsize).all()
        if i % 3 == 1:
            assert (b == 7.0).all()
        else:
            assert ((b.double() - b64).abs() <= (K + 1) * 2.0 ** -24 * bsize).all()
    # two products that add to the same memory are not for one launch
    ptrs[6] = ptrs[2]
    assert call(ptrs) == -2


# The same over very many rows (the applications of shared layers are one K).  The blocked column sum that these replace adds
# at most 32 + 4 + ceil(K / 16384) + 24 values in a row, and every addition is off by half an ulp of at most the running sum of
# magnitudes: with rows of one sign the errors are independent and few standard deviations (half the square root of the chain,
# in ulps) cover 2048 rows.  A running sum over all K misses this by 2 to 6 times.
@pytest.mark.parametrize("bf16,M,N,K", [(1, 256, 128, 131105), (1, 2048, 1024, 131072), (1, 2048, 4096, 131105), (0, 256, 128, 131105),
                                        (0, 2048, 1024, 40000), (1, 64, 64, 1000003)])
def test_row_sums_over_many_rows(bf16, M, N, K):
    lib = _lib()
    lib.swarm_kernel_gemm_rowsum.argtypes = [C.c_int] * 4 + [C.c_void_p] * 5
    g = torch.Generator(device="cuda").manual_seed(M + K)
    dt = torch.bfloat16 if bf16 else torch.float32
    A = (torch.randn((K, M), generator=g, device="cuda") + 1.0).to(dt)
    B = torch.randn((K, N), generator=g, device="cuda").to(dt)
    db, dW = torch.zeros(M, device="cuda"), torch.zeros((M, N), device="cuda")
    assert lib.swarm_kernel_gemm_rowsum(bf16, M, N, K, A.data_ptr(), B.data_ptr(), dW.data_ptr(), db.data_ptr(), None) == 0
    torch.cuda.synchronize()
    rows = range(0, K, 1 << 16)
    want = sum(A[r:r + (1 << 16)].double().sum(0) for r in rows)
    size = sum(A[r:r + (1 << 16)].double().abs().sum(0) for r in rows)
    chain = 32 + 4 + -(-K // 16384) + 24
    assert ((db.double() - want).abs() <= 0.5 * math.sqrt(chain) * 2.0 ** -24 * size).all()
