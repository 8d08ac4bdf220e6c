"""Parity of the HIP path against the fp64 CPU oracle, through the C ABI.

Error measure (both tolerances come from the benchmark definition): the
max-norm relative error  max|gpu - ref| / max|ref|  per output tensor;
<= 1e-4 for fp32 paths, <= 2e-2 for bf16-input paths.  The oracle consumes the
same bf16-rounded inputs converted exactly to fp64, so only the GPU's
accumulation, intermediate and output rounding is judged.  Integer inputs must
match bit for bit."""
import sys

import numpy as np
import pytest
import torch

import oracle as orc
import rtp_workloads as wl
from paper_2311_01635_amd import binding as B
from paper_2311_01635_amd.layers import RtpLinear, RtpMlp, RtpMoe

pytestmark = pytest.mark.gpu

TOL_F32 = 1e-4
TOL_BF16 = 2e-2
DEV = "cuda:0"


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def relerr(gpu, ref):
    gpu = np.asarray(gpu, dtype=np.float64)
    assert gpu.shape == np.shape(ref)
    if gpu.size == 0:
        return 0.0
    den = np.abs(ref).max()
    return float(np.abs(gpu - ref).max() / (den if den > 0 else 1.0))


def dev(x, dtype):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV, dtype)


def host(t):
    return t.detach().float().cpu().numpy().astype(np.float64)


def f64(x):
    return np.ascontiguousarray(x, dtype=np.float64)


_TD = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
_BD = {"f32": B.RTP_F32, "bf16": B.RTP_BF16, "f16": B.RTP_F16}
TOL_F16 = 5e-3   # fp16 keeps 11 significant bits: stored intermediates round 8 times finer than bf16

# ------------------------------------------------------------ single GEMMs --

def _gemm_case(layout, M, N, K, variant, accumulate, out_f32, seed, dtype="bf16"):
    rng = np.random.default_rng(seed)
    shapes = {B.LAYOUT_NT: ((M, K), (N, K)), B.LAYOUT_NN: ((M, K), (K, N)), B.LAYOUT_TN: ((K, M), (K, N))}[layout]
    A = wl._store(rng.standard_normal(shapes[0], dtype=np.float32), dtype)
    Bm = wl._store(rng.standard_normal(shapes[1], dtype=np.float32), dtype)
    C0 = rng.standard_normal((M, N), dtype=np.float32)
    ref = np.zeros((M, N))
    {B.LAYOUT_NT: orc.gemm_nt, B.LAYOUT_NN: orc.gemm_nn, B.LAYOUT_TN: orc.gemm_tn}[layout](f64(A), f64(Bm), ref)
    if accumulate:
        ref = ref + f64(C0)
    dA, dB = dev(A, _TD[dtype]), dev(Bm, _TD[dtype])
    dC = dev(C0, torch.float32 if out_f32 else _TD[dtype])
    torch.cuda.synchronize()
    B.rtp_gemm(layout, _BD[dtype], B.RTP_F32 if out_f32 else _BD[dtype], accumulate, dA, shapes[0][1], dB,
               shapes[1][1], dC, N, M, N, K, variant)
    torch.cuda.synchronize()
    return relerr(host(dC), ref)


GEMM_SHAPES = [
    (256, 256, 64),      # exactly one large tile, one K step
    (128, 128, 128),
    (304, 520, 200),     # ragged in M, N and K (K tail of 8)
    (520, 264, 1376),    # K = 21.5 K-steps, as in the shard-width contractions
    (8, 8, 8),           # smallest the 16-byte loads allow
    (1000, 1376, 320),
]
# row counts that are not multiples of 8 are legal wherever the operand is contiguous along K
GEMM_ODD = {B.LAYOUT_NT: [(301, 77, 72), (301, 77, 96)], B.LAYOUT_NN: [(301, 72, 72), (301, 72, 96)],
            B.LAYOUT_TN: [(72, 72, 301), (72, 520, 320)]}


# variants 1-2: register-staged tiles; 4: the ping-pong kernel with the tile height picked by shape;
# 5, 6, 7, 8: tile height 256, 192, 128, and the 64 x 128 tile
@pytest.mark.parametrize("variant", [1, 2, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("layout", [B.LAYOUT_NT, B.LAYOUT_NN, B.LAYOUT_TN])
def test_gemm_bf16_layouts_and_tails(layout, variant):
    for i, (M, N, K) in enumerate(GEMM_SHAPES + GEMM_ODD[layout]):
        for accumulate, out_f32 in ((False, True), (True, True), (False, False)):
            say(f"gemm layout={layout} variant={variant} M={M} N={N} K={K} acc={accumulate} f32out={out_f32}")
            err = _gemm_case(layout, M, N, K, variant, accumulate, out_f32, seed=100 * layout + i)
            assert err <= (TOL_F32 if out_f32 else TOL_BF16), (layout, variant, M, N, K, accumulate, out_f32, err)


@pytest.mark.parametrize("variant", [4, 5, 6, 7, 8])
@pytest.mark.parametrize("layout", [B.LAYOUT_NT, B.LAYOUT_NN, B.LAYOUT_TN])
def test_gemm_fp16_layouts_and_tails(layout, variant):
    """fp16 inputs run on the tiled kernel (K a multiple of 32); same shapes, same oracle."""
    for i, (M, N, K) in enumerate(GEMM_SHAPES + GEMM_ODD[layout]):
        if K % 32:
            continue
        for accumulate, out_f32 in ((False, True), (True, True), (False, False)):
            say(f"fp16 gemm layout={layout} variant={variant} M={M} N={N} K={K} acc={accumulate} f32out={out_f32}")
            err = _gemm_case(layout, M, N, K, variant, accumulate, out_f32, seed=300 * layout + i, dtype="f16")
            assert err <= (TOL_F32 if out_f32 else TOL_F16), (layout, variant, M, N, K, accumulate, out_f32, err)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("layout", [B.LAYOUT_NT, B.LAYOUT_NN, B.LAYOUT_TN])
def test_gemm_split_k_accumulate(layout, dtype):
    """Few output tiles, long contraction, fp32 `C += A B`: the launcher cuts the K loop into chunks whose
    partial sums meet through atomic adds (the weight-gradient GEMM of a narrow shard).  Random inputs to the
    fp32 bar; integer inputs bit-exactly, whatever order the chunks arrive in."""
    for i, (M, N, K) in enumerate([(384, 768, 8192), (128, 264, 4096), (768, 384, 2048 + 96)]):
        for variant in (4, 7):
            say(f"split-K gemm layout={layout} dtype={dtype} M={M} N={N} K={K} variant={variant}")
            err = _gemm_case(layout, M, N, K, variant, True, True, seed=500 + 10 * layout + i, dtype=dtype)
            assert err <= TOL_F32, (layout, M, N, K, variant, err)
    M, N, K = 384, 520, 8192
    rng = np.random.default_rng(77)
    shapes = {B.LAYOUT_NT: ((M, K), (N, K)), B.LAYOUT_NN: ((M, K), (K, N)), B.LAYOUT_TN: ((K, M), (K, N))}[layout]
    A = rng.integers(-2, 3, size=shapes[0]).astype(np.float32)
    Bm = rng.integers(-2, 3, size=shapes[1]).astype(np.float32)
    C0 = rng.integers(-8, 9, size=(M, N)).astype(np.float32)
    Ad, Bd = torch.from_numpy(A).double(), torch.from_numpy(Bm).double()
    prod = {B.LAYOUT_NT: lambda: Ad @ Bd.T, B.LAYOUT_NN: lambda: Ad @ Bd, B.LAYOUT_TN: lambda: Ad.T @ Bd}[layout]()
    ref = (prod + torch.from_numpy(C0).double()).float()
    dA, dB, dC = dev(A, _TD[dtype]), dev(Bm, _TD[dtype]), dev(C0, torch.float32)
    B.rtp_gemm(layout, _BD[dtype], B.RTP_F32, True, dA, shapes[0][1], dB, shapes[1][1], dC, N, M, N, K, 4)
    torch.cuda.synchronize()
    assert torch.equal(dC.cpu(), ref)


@pytest.mark.parametrize("variant", [4, 5, 6, 7, 8])
def test_gemm_accumulates_onto_a_sum_beyond_32_bit_byte_offsets(variant):
    """fp32 `C += A B` where C's rows lie 128 MiB apart, 5 GiB from first to last: the tiled kernel reads the sum it
    adds onto through 32-bit byte offsets where they reach, and through 64-bit addresses where, as here, they do not."""
    M, N, K, ldc = 40, 64, 64, 1 << 25
    rng = np.random.default_rng(91)
    A = wl._store(rng.standard_normal((M, K), dtype=np.float32), "bf16")
    Bm = wl._store(rng.standard_normal((N, K), dtype=np.float32), "bf16")
    C0 = rng.standard_normal((M, N), dtype=np.float32)
    ref = np.zeros((M, N))
    orc.gemm_nt(f64(A), f64(Bm), ref)
    ref += f64(C0)
    big = torch.zeros((M - 1) * ldc + N, device=DEV, dtype=torch.float32)
    view = torch.as_strided(big, (M, N), (ldc, 1))
    view.copy_(torch.from_numpy(C0))
    say(f"gemm NT M={M} N={N} K={K} ldc={ldc} variant={variant} accumulate")
    B.rtp_gemm(B.LAYOUT_NT, B.RTP_BF16, B.RTP_F32, True, dev(A, torch.bfloat16), K, dev(Bm, torch.bfloat16), K, big, ldc,
               M, N, K, variant)
    torch.cuda.synchronize()
    assert relerr(host(view), ref) <= TOL_F32
    assert float(big[N:ldc].abs().max()) == 0.0          # nothing written between the rows
    del big, view
    torch.cuda.empty_cache()


def test_gemm_fp16_needs_the_tiled_kernel():
    a = torch.zeros(64, 72, device=DEV, dtype=torch.float16)
    c = torch.zeros(64, 64, device=DEV, dtype=torch.float32)
    with pytest.raises(B.RtpError) as e:
        B.rtp_gemm(B.LAYOUT_NT, B.RTP_F16, B.RTP_F32, False, a, 72, a, 72, c, 64, 64, 64, 72)    # K = 72: not a multiple of 32
    assert e.value.status == B.RTP_ERR_SHAPE
    with pytest.raises(B.RtpError) as e:
        B.rtp_gemm(B.LAYOUT_NT, B.RTP_F16, B.RTP_F32, False, a, 72, a, 72, c, 64, 64, 64, 64, 1)  # register-staged variant
    assert e.value.status == B.RTP_ERR_SHAPE


def test_gemm_rejects_misaligned_shapes():
    a = torch.zeros(64, 64, device=DEV, dtype=torch.bfloat16)
    c = torch.zeros(64, 64, device=DEV, dtype=torch.float32)
    with pytest.raises(B.RtpError) as e:
        B.rtp_gemm(B.LAYOUT_NT, B.RTP_BF16, B.RTP_F32, False, a, 64, a, 64, c, 64, 64, 64, 60)   # K not a multiple of 8
    assert e.value.status == B.RTP_ERR_SHAPE
    with pytest.raises(B.RtpError) as e:
        B.rtp_gemm(B.LAYOUT_NN, B.RTP_BF16, B.RTP_F32, False, a, 64, a, 64, c, 64, 64, 60, 64)   # N-contiguous operand
    assert e.value.status == B.RTP_ERR_SHAPE
    B.rtp_gemm(B.LAYOUT_NT, B.RTP_BF16, B.RTP_F32, False, a, 64, a, 64, c, 64, 0, 64, 64)        # empty M: no-op
    torch.cuda.synchronize()


# ------------------------------------------------------ rotated linear layer --

def _linear_case(w: wl.Workload, rank, mode, split, seed=0, grad0=True, integer=False):
    td, bd = _TD[w.dtype], _BD[w.dtype]
    inp = wl.make_integer_inputs(w, seed) if integer else wl.make_inputs(w, seed, grad0=grad0)
    X, W, dY = inp["X"], inp["W"], inp["dY"]
    G0 = inp.get("G0_W")
    fn = orc.rtp_linear_out if split == B.RTP_SPLIT_OUT else orc.rtp_linear_in
    ref = fn(f64(X), f64(W), f64(dY), w.n, rank, None if G0 is None else f64(G0))
    layer = RtpLinear(dev(W, td), w.T, w.n, rank, split, mode, bd, G0=None if G0 is None else dev(G0, torch.float32))
    dX_, dY_ = dev(X, td), dev(dY, td)
    Y_ = torch.full((w.T, w.O), float("nan"), device=DEV, dtype=td)
    dXo = torch.full((w.T, w.I), float("nan"), device=DEV, dtype=td)
    torch.cuda.synchronize()
    layer.forward(dX_, Y_)
    layer.sync()
    res_after_fwd = layer.ring.resident()
    layer.backward(dX_, dY_, dXo)
    layer.sync()
    res_after_bwd = layer.ring.resident()
    Wb, G = layer.gathered()
    trace = layer.ring.trace()
    out = dict(Y=host(Y_), dX=host(dXo), G=host(G), W_same=bool(torch.equal(Wb, dev(W, td))),
               res_after_fwd=res_after_fwd, res_after_bwd=res_after_bwd, trace=trace)
    layer.close()
    return out, ref


def _check_linear(out, ref, tol, exact=False):
    assert out["W_same"], "the weight store must be bit-identical after the round trip"
    assert out["res_after_fwd"] == ref["resident_after_fwd"]
    assert out["res_after_bwd"] == ref["resident_after_bwd"]
    assert [(s, k) for (kind, p, s, k, b) in out["trace"] if kind == "fwd"] == ref["fwd_log"]
    assert [(s, k) for (kind, p, s, k, b) in out["trace"] if kind == "bwd"] == ref["bwd_log"]
    for key in ("Y", "dX", "G"):
        assert np.isfinite(out[key]).all(), f"{key} holds values that were never written"
        if exact:
            assert np.array_equal(out[key], ref[key]), key
        else:
            assert relerr(out[key], ref[key]) <= tol, (key, relerr(out[key], ref[key]))


def test_cfg1_fp32_linear_all_ranks():
    w = wl.CONFIGS["cfg1_linear_f32"]
    for rank in range(w.n):
        say(f"cfg1 fp32 linear rank={rank}")
        out, ref = _linear_case(w, rank, B.RTP_DOUBLE_BUFFER, B.RTP_SPLIT_OUT)
        _check_linear(out, ref, TOL_F32)


@pytest.mark.parametrize("mode", [B.RTP_DOUBLE_BUFFER, B.RTP_INPLACE_STAGED, B.RTP_INPLACE_BLOCKING])
@pytest.mark.parametrize("split", [B.RTP_SPLIT_OUT, B.RTP_SPLIT_IN])
def test_fp32_linear_modes_and_splits(mode, split):
    w = wl.Workload("f32_small", "linear", T=70, I=96 if split == B.RTP_SPLIT_IN else 50, O=36 if split == B.RTP_SPLIT_IN else 96,
                    n=3, dtype="f32", mode="x", w_dist=("uniform", 0.1))
    for rank in (0, 2):
        say(f"fp32 linear split={split} mode={mode} rank={rank}")
        out, ref = _linear_case(w, rank, mode, split)
        _check_linear(out, ref, TOL_F32)


@pytest.mark.parametrize("mode", [B.RTP_DOUBLE_BUFFER, B.RTP_INPLACE_STAGED, B.RTP_INPLACE_BLOCKING])
@pytest.mark.parametrize("split", [B.RTP_SPLIT_OUT, B.RTP_SPLIT_IN])
def test_bf16_linear_ragged_multi_tile(mode, split):
    """Several tiles in every dimension plus ragged tails: T = 300 tokens,
    shard width 264 (= 8 * 33), 5 shards."""
    if split == B.RTP_SPLIT_OUT:
        w = wl.Workload("bf16_out", "linear", T=300, I=520, O=5 * 264, n=5, dtype="bf16", mode="x")
    else:
        w = wl.Workload("bf16_in", "linear", T=300, I=5 * 264, O=520, n=5, dtype="bf16", mode="x")
    for rank in (0, 3):
        say(f"bf16 linear split={split} mode={mode} rank={rank}")
        out, ref = _linear_case(w, rank, mode, split)
        _check_linear(out, ref, TOL_BF16)


@pytest.mark.parametrize("split", [B.RTP_SPLIT_OUT, B.RTP_SPLIT_IN])
def test_bf16_linear_integer_inputs_bit_exact(split):
    """Entries in {-2..2}: every product and partial sum is an integer below
    2^24, so the fp32 accumulators are exact whatever the tiling; outputs are
    compared after the same single rounding to bf16."""
    if split == B.RTP_SPLIT_OUT:
        w = wl.Workload("int_out", "linear", T=520, I=1376, O=4 * 344, n=4, dtype="bf16", mode="x")
    else:
        w = wl.Workload("int_in", "linear", T=520, I=4 * 344, O=1376, n=4, dtype="bf16", mode="x")
    say(f"integer-exact bf16 linear split={split}")
    out, ref = _linear_case(w, 1, B.RTP_INPLACE_STAGED, split, integer=True)
    for key in ("Y", "dX"):
        ref[key] = wl.round_to_bf16(ref[key].astype(np.float32)).astype(np.float64)
    _check_linear(out, ref, 0.0, exact=True)


@pytest.mark.parametrize("mode", [B.RTP_DOUBLE_BUFFER, B.RTP_INPLACE_STAGED, B.RTP_INPLACE_BLOCKING])
@pytest.mark.parametrize("split", [B.RTP_SPLIT_OUT, B.RTP_SPLIT_IN])
def test_fp16_linear_multi_tile(mode, split):
    """fp16 inputs (contraction lengths multiples of 32): several tiles and ragged tails in the free dimensions."""
    if split == B.RTP_SPLIT_OUT:
        w = wl.Workload("f16_out", "linear", T=320, I=544, O=5 * 288, n=5, dtype="f16", mode="x", w_dist=("normal", 0.05))
    else:
        w = wl.Workload("f16_in", "linear", T=320, I=5 * 288, O=544, n=5, dtype="f16", mode="x", w_dist=("normal", 0.05))
    for rank in (0, 3):
        say(f"fp16 linear split={split} mode={mode} rank={rank}")
        out, ref = _linear_case(w, rank, mode, split)
        _check_linear(out, ref, TOL_F16)


@pytest.mark.parametrize("mode", [B.RTP_DOUBLE_BUFFER, B.RTP_INPLACE_STAGED, B.RTP_INPLACE_BLOCKING])
@pytest.mark.parametrize("split", [B.RTP_SPLIT_OUT, B.RTP_SPLIT_IN])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_padded_partition(dtype, split, mode):
    """n does not divide the partitioned dimension: shards are padded to equal width and the last one
    is partly filled.  The result must still be the plain unsharded linear layer (forward, both
    gradients, arriving gradient content added), so the reference is the plain definition."""
    part, n = (50, 3) if dtype == "f32" else (520, 3)
    other = 36 if dtype == "f32" else 264
    O, I = (part, other) if split == B.RTP_SPLIT_OUT else (other, part)
    w = wl.Workload("padded", "linear", T=70 if dtype == "f32" else 300, I=I, O=O, n=n, dtype=dtype, mode="x",
                    w_dist=("uniform", 0.1))
    inp = wl.make_inputs(w, seed=9, grad0=True)
    X, W, dY, G0 = (f64(inp[k]) for k in ("X", "W", "dY", "G0_W"))
    dX_ref, dW_ref = orc.plain_linear_bwd(X, W, dY)
    ref = dict(Y=orc.plain_linear_fwd(X, W), dX=dX_ref, dW=dW_ref + G0)
    for rank in (0, n - 1):
        say(f"padded partition dtype={dtype} split={split} mode={mode} rank={rank}")
        layer = RtpLinear(dev(inp["W"], _TD[dtype]), w.T, n, rank, split, mode, _BD[dtype], G0=dev(inp["G0_W"], torch.float32))
        Xd, dYd = dev(inp["X"], _TD[dtype]), dev(inp["dY"], _TD[dtype])
        Y = torch.full((w.T, O), float("nan"), device=DEV, dtype=_TD[dtype])
        dX = torch.full((w.T, I), float("nan"), device=DEV, dtype=_TD[dtype])
        torch.cuda.synchronize()
        layer.forward(Xd, Y)
        layer.backward(Xd, dYd, dX)
        layer.sync()
        Wb, G = layer.gathered()
        assert torch.equal(Wb, dev(inp["W"], _TD[dtype]))
        tol = TOL_F32 if dtype == "f32" else TOL_BF16
        for key, got in (("Y", Y), ("dX", dX), ("dW", G)):
            assert torch.isfinite(got.float()).all(), key
            assert relerr(host(got), ref[key]) <= tol, (key, relerr(host(got), ref[key]))
        layer.close()


@pytest.mark.parametrize("mode", [B.RTP_DOUBLE_BUFFER, B.RTP_INPLACE_STAGED, B.RTP_INPLACE_BLOCKING])
@pytest.mark.parametrize("dtype,act", [("f32", B.RTP_ACT_NONE), ("bf16", B.RTP_ACT_NONE), ("f16", B.RTP_ACT_NONE),
                                       ("bf16", B.RTP_ACT_GELU_ERF), ("f32", B.RTP_ACT_GELU_ERF)])
def test_linear_with_bias(dtype, act, mode):
    """Y = act(X W^T + b) with the bias riding in the flat parameter: forward, input gradient, weight
    gradient and bias gradient (column sums of dY onto what arrives with the shard) against the oracle's
    rotated layer with bias; weights and bias come back unchanged.  The fp32 and bf16 cases have a padded last
    shard, with and without the activation."""
    if dtype == "f32":
        T, I, O, n = 70, 36, 50, 3           # padded: shards of 17, 17, 16 rows (with or without the activation)
    elif dtype == "bf16":
        T, I, O, n = 300, 264, 520, 3        # padded: 176, 176, 168 (with or without the activation)
    else:
        T, I, O, n = 320, 288, 4 * 160, 4
    w = wl.Workload("bias", "linear", T=T, I=I, O=O, n=n, dtype=dtype, mode="x", w_dist=("uniform", 0.1))
    inp = wl.make_inputs(w, seed=21, grad0=True)
    rng = np.random.default_rng(22)
    b = wl._store(rng.standard_normal(O).astype(np.float32) * 0.5, dtype)
    gb0 = rng.standard_normal(O).astype(np.float32)
    X, W, dY, G0 = (f64(inp[k]) for k in ("X", "W", "dY", "G0_W"))
    td, bd = _TD[dtype], _BD[dtype]
    tol = {"f32": TOL_F32, "bf16": TOL_BF16, "f16": TOL_F16}[dtype]
    Z = orc.plain_linear_fwd(X, W, f64(b))
    dX_ref, dW_ref = orc.plain_linear_bwd(X, W, dY)
    ref = dict(Y=Z if act == B.RTP_ACT_NONE else orc.act(Z, orc.GELU_ERF), dX=dX_ref, dW=dW_ref + G0,
               gb=f64(gb0) + orc.plain_bias_grad(dY))
    for rank in (0, n - 1):
        say(f"linear with bias dtype={dtype} act={act} mode={mode} rank={rank}")
        if O % n == 0:   # the rotated oracle (equal shards) must agree with the plain definitions used above
            rot = orc.rtp_linear_out_bias(X, W, f64(b), dY, n, rank, G0, f64(gb0))
            assert relerr(rot["gb"], ref["gb"]) < 1e-12 and relerr(rot["G"], ref["dW"]) < 1e-12
        preact = torch.empty(T, O, device=DEV, dtype=td) if act != B.RTP_ACT_NONE else None
        layer = RtpLinear(dev(inp["W"], td), T, n, rank, B.RTP_SPLIT_OUT, mode, bd, act=act, preact=preact,
                          G0=dev(inp["G0_W"], torch.float32), bias=dev(b, td), gb0=dev(gb0, torch.float32))
        Xd, dYd = dev(inp["X"], td), dev(inp["dY"], td)
        Y = torch.full((T, O), float("nan"), device=DEV, dtype=td)
        dX = torch.full((T, I), float("nan"), device=DEV, dtype=td)
        torch.cuda.synchronize()
        layer.forward(Xd, Y)
        layer.backward(Xd, dYd, dX)      # dY is the gradient at the pre-activation, as the layer's backward takes it
        layer.sync()
        Wb, G = layer.gathered()
        bb, gb = layer.gathered_bias()
        assert torch.equal(Wb, dev(inp["W"], td)) and torch.equal(bb, dev(b, td))
        if preact is not None:
            assert relerr(host(preact), Z) <= tol
        for key, got in (("Y", Y), ("dX", dX), ("dW", G), ("gb", gb)):
            assert torch.isfinite(got.float()).all(), key
            assert relerr(host(got), ref[key]) <= tol, (key, relerr(host(got), ref[key]))
        layer.close()


@pytest.mark.parametrize("mode", [B.RTP_DOUBLE_BUFFER, B.RTP_INPLACE_STAGED, B.RTP_INPLACE_BLOCKING])
@pytest.mark.parametrize("dtype,T,I,O,n", [("f32", 70, 48, 50, 3), ("bf16", 300, 512, 104, 8), ("bf16", 96, 64, 40, 1),
                                           ("f16", 320, 256, 96, 4), ("bf16", 64, 128, 8, 4)])
def test_input_partitioned_linear_with_bias(dtype, T, I, O, n, mode):
    """Y = X W^T + b with b spread over the shards in pieces (widths that N does not divide, a piece
    per shard narrower than 16 bytes' worth, more shards than pieces, a single shard): forward, both
    gradients and the pieces' gradients (onto what arrives) against the oracle's rotated layer."""
    w = wl.Workload("bias_in", "linear_in", T=T, I=I, O=O, n=n, dtype=dtype, mode="x", w_dist=("uniform", 0.1))
    inp = wl.make_inputs(w, seed=31, grad0=True)
    rng = np.random.default_rng(32)
    b = wl._store(rng.standard_normal(O).astype(np.float32) * 0.5, dtype)
    gb0 = rng.standard_normal(O).astype(np.float32)
    td, bd = _TD[dtype], _BD[dtype]
    tol = {"f32": TOL_F32, "bf16": TOL_BF16, "f16": TOL_F16}[dtype]
    for rank in sorted({0, n - 1}):
        say(f"input-partitioned linear with bias dtype={dtype} T={T} I={I} O={O} n={n} mode={mode} rank={rank}")
        ref = orc.rtp_linear_in(f64(inp["X"]), f64(inp["W"]), f64(inp["dY"]), n, rank, G0=f64(inp["G0_W"]), b=f64(b),
                                gb0=f64(gb0))
        layer = RtpLinear(dev(inp["W"], td), T, n, rank, B.RTP_SPLIT_IN, mode, bd, G0=dev(inp["G0_W"], torch.float32),
                          bias=dev(b, td), gb0=dev(gb0, torch.float32))
        Xd, dYd = dev(inp["X"], td), dev(inp["dY"], td)
        Y = torch.full((T, O), float("nan"), device=DEV, dtype=td)
        dX = torch.full((T, I), float("nan"), device=DEV, dtype=td)
        torch.cuda.synchronize()
        layer.forward(Xd, Y)
        layer.backward(Xd, dYd, dX)
        layer.sync()
        Wb, G = layer.gathered()
        bb, gb = layer.gathered_bias()
        assert torch.equal(Wb, dev(inp["W"], td)) and torch.equal(bb, dev(b, td))
        for key, got in (("Y", Y), ("dX", dX), ("G", G), ("gb", gb)):
            assert torch.isfinite(got.float()).all(), key
            assert relerr(host(got), ref[key]) <= tol, (key, relerr(host(got), ref[key]))
        layer.close()


@pytest.mark.parametrize("n", [1, 8])
@pytest.mark.parametrize("mode", [B.RTP_DOUBLE_BUFFER, B.RTP_INPLACE_STAGED, B.RTP_INPLACE_BLOCKING])
def test_gradients_accumulate_over_passes(mode, n):
    """Two forward + backward passes without reading the store in between: every gradient shard, the
    one the worker ends a pass on included, holds arriving content + twice the pass's contribution
    (integer inputs: bit-exact), and the weights are unchanged."""
    T, I, O = 512, 1024, 2048
    g = torch.Generator(device="cpu").manual_seed(4)
    ri = lambda lo, hi, shape: torch.randint(lo, hi, shape, generator=g).float()
    W, X, dY, G0 = ri(-2, 3, (O, I)), ri(-2, 3, (T, I)), ri(-2, 3, (T, O)), ri(-4, 5, (O, I))
    layer = RtpLinear(W.to(DEV, torch.bfloat16), T, n, n // 2, B.RTP_SPLIT_OUT, mode, B.RTP_BF16, G0=G0.to(DEV))
    Xd, dYd = X.to(DEV, torch.bfloat16), dY.to(DEV, torch.bfloat16)
    Y = torch.empty(T, O, device=DEV, dtype=torch.bfloat16)
    dX = torch.empty(T, I, device=DEV, dtype=torch.bfloat16)
    for _ in range(2):
        layer.forward(Xd, Y)
        layer.backward(Xd, dYd, dX)
    layer.sync()
    Wb, G = layer.gathered()
    assert torch.equal(Wb.cpu().float(), W)
    assert torch.equal(G.cpu(), G0 + 2 * (dY.double().T @ X.double()).float())
    assert torch.equal(Y.cpu(), (X.double() @ W.double().T).to(torch.bfloat16))
    layer.close()


@pytest.mark.parametrize("how", ["zero_grads", "flush_then_clear"])
@pytest.mark.parametrize("mode", [B.RTP_DOUBLE_BUFFER, B.RTP_INPLACE_STAGED, B.RTP_INPLACE_BLOCKING])
def test_cleared_gradients_start_from_zero(mode, how):
    """An optimizer step between passes: after the store is cleared (by the library's call, or by the
    caller after a flush) the next pass's gradients hold that pass alone: the copy of its own
    shard the worker kept from the previous pass does not come back (integer inputs: bit-exact)."""
    T, I, O, n = 256, 512, 1024, 4
    g = torch.Generator(device="cpu").manual_seed(5)
    ri = lambda lo, hi, shape: torch.randint(lo, hi, shape, generator=g).float()
    W, X, dY, G0 = ri(-2, 3, (O, I)), ri(-2, 3, (T, I)), ri(-2, 3, (T, O)), ri(-4, 5, (O, I))
    layer = RtpLinear(W.to(DEV, torch.bfloat16), T, n, 1, B.RTP_SPLIT_OUT, mode, B.RTP_BF16, G0=G0.to(DEV))
    Xd, dYd = X.to(DEV, torch.bfloat16), dY.to(DEV, torch.bfloat16)
    Y = torch.empty(T, O, device=DEV, dtype=torch.bfloat16)
    dX = torch.empty(T, I, device=DEV, dtype=torch.bfloat16)
    layer.forward(Xd, Y)
    layer.backward(Xd, dYd, dX)
    if how == "zero_grads":
        layer.zero_grads()
    else:
        layer.ring.flush()
        layer.sync()
        layer.home_g.zero_()
        torch.cuda.synchronize()
    layer.forward(Xd, Y)
    layer.backward(Xd, (2 * dY).to(DEV, torch.bfloat16), dX)
    layer.sync()
    _, G = layer.gathered()
    assert torch.equal(G.cpu(), 2 * (dY.double().T @ X.double()).float())
    layer.close()


@pytest.mark.parametrize("mode", [B.RTP_DOUBLE_BUFFER, B.RTP_INPLACE_STAGED, B.RTP_INPLACE_BLOCKING])
def test_weights_written_after_a_flush_are_the_ones_the_next_pass_uses(mode):
    """An optimizer step on the weights: a backward pass leaves the worker's own shard in its buffer and the
    next forward pass starts on it without loading it; after rtp_ring_flush the caller may write to the weight
    store, and the next pass must compute with what it wrote, own shard included (integer inputs: bit-exact)."""
    T, I, O, n, rank = 256, 512, 1024, 4, 2
    g = torch.Generator(device="cpu").manual_seed(6)
    ri = lambda lo, hi, shape: torch.randint(lo, hi, shape, generator=g).float()
    W, X, dY = ri(-2, 3, (O, I)), ri(-2, 3, (T, I)), ri(-2, 3, (T, O))
    layer = RtpLinear(W.to(DEV, torch.bfloat16), T, n, rank, B.RTP_SPLIT_OUT, mode, B.RTP_BF16)
    Xd, dYd = X.to(DEV, torch.bfloat16), dY.to(DEV, torch.bfloat16)
    Y = torch.empty(T, O, device=DEV, dtype=torch.bfloat16)
    dX = torch.empty(T, I, device=DEV, dtype=torch.bfloat16)
    for _ in range(2):                                   # the second pass starts on the shard the first one ended on
        layer.forward(Xd, Y)
        layer.backward(Xd, dYd, dX)
    layer.sync()
    assert torch.equal(Y.cpu(), (X.double() @ W.double().T).to(torch.bfloat16))
    layer.ring.flush()
    layer.sync()
    W2 = W - ri(-1, 2, (O, I))                           # "W -= lr * G", every shard touched
    layer.store_w.pack("W", W2.to(DEV, torch.bfloat16), 0, B.RTP_SPLIT_OUT, layer.o)
    torch.cuda.synchronize()
    layer.forward(Xd, Y)
    layer.backward(Xd, dYd, dX)
    layer.sync()
    assert torch.equal(Y.cpu(), (X.double() @ W2.double().T).to(torch.bfloat16))
    assert torch.equal(dX.cpu(), (dY.double() @ W2.double()).to(torch.bfloat16))
    Wb, _ = layer.gathered()
    assert torch.equal(Wb.cpu().float(), W2)
    layer.close()


@pytest.mark.parametrize("mode", [B.RTP_DOUBLE_BUFFER, B.RTP_INPLACE_STAGED])
@pytest.mark.parametrize("schedule", ["default", "grouped"])
def test_own_gradient_shard_reaches_its_slot(schedule, mode):
    """A backward pass ends on the worker's own shard, which travels no further.  The unit's default schedule has the
    last step's kernels store `arrived + own` straight into the own slot: the store is current without a flush and
    the ring holds nothing back.  The grouped schedule leaves the shard in the buffer: the ring says so, and the next
    backward pass (or a flush) writes it back.  Either way two passes give the oracle's `2 x own + arrived`."""
    T, I, O, O2, n, rank = 192, 128, 4 * 128, 96, 4, 1
    w = wl.Workload("own_g", "swiglu", T=T, I=I, O=O, O2=O2, n=n, dtype="bf16", mode="x", w_dist=("normal", 0.08))
    inp = wl.make_inputs(w, seed=83, grad0=True)
    names = ("Wg", "Wu", "Wd")
    ref = orc.rtp_swiglu(f64(inp["X"]), *[f64(inp[k]) for k in names], f64(inp["dY"]), n, rank,
                         *[f64(inp["G0_" + k]) for k in names])
    mlp = RtpMlp([dev(inp[k], torch.bfloat16) for k in names], T, n, rank, B.RTP_ACT_SWIGLU, mode, B.RTP_BF16,
                 G0=[dev(inp["G0_" + k], torch.float32) for k in names], grouped=schedule == "grouped")
    ring = B.lib.rtp_mlp_ring(mlp.handle)
    X, dY = dev(inp["X"], torch.bfloat16), dev(inp["dY"], torch.bfloat16)
    Y = torch.empty(T, O2, device=DEV, dtype=torch.bfloat16)
    dX = torch.empty(T, I, device=DEV, dtype=torch.bfloat16)
    for p in (1, 2):
        say(f"own gradient shard schedule={schedule} mode={mode} pass {p}")
        mlp.forward(X, Y)
        mlp.backward(X, dY, dX)
        mlp.sync()
        held = B.lib.rtp_ring_resident_grad(ring)
        assert held == (-1 if schedule == "default" else rank)
        if held < 0:                                          # no flush: read the store as it is
            rows = slice(rank * (O // n), (rank + 1) * (O // n))
            for key, k, g in zip(("dWg", "dWu", "dWd"), names, [mlp.store_g.unpack(nm) for nm in names]):
                want = p * ref[key] - (p - 1) * f64(inp["G0_" + k])
                got, want = (host(g)[rows], want[rows]) if k != "Wd" else (host(g)[:, rows], want[:, rows])
                assert relerr(got, want) <= TOL_BF16, (key, p)
    _, Gs = mlp.gathered()
    assert B.lib.rtp_ring_resident_grad(ring) == -1
    for key, k, g in zip(("dWg", "dWu", "dWd"), names, Gs):
        assert relerr(host(g), 2.0 * ref[key] - f64(inp["G0_" + k])) <= TOL_BF16, key
    mlp.close()


def test_degenerate_partitions():
    # n = 1 is the plain linear; one token; n equal to the number of 8-wide column groups
    for (T, I, O, n) in ((40, 64, 72, 1), (1, 64, 64, 2), (33, 16, 64, 8)):
        w = wl.Workload("deg", "linear", T=T, I=I, O=O, n=n, dtype="bf16", mode="x")
        say(f"degenerate T={T} I={I} O={O} n={n}")
        out, ref = _linear_case(w, n - 1, B.RTP_DOUBLE_BUFFER, B.RTP_SPLIT_OUT)
        _check_linear(out, ref, TOL_BF16)
    w = wl.Workload("deg32", "linear", T=5, I=8, O=12, n=12, dtype="f32", mode="x", w_dist=("uniform", 0.5))
    out, ref = _linear_case(w, 5, B.RTP_DOUBLE_BUFFER, B.RTP_SPLIT_OUT)   # one output column per step
    _check_linear(out, ref, TOL_F32)


def test_empty_batch_is_a_no_op():
    w = wl.Workload("empty", "linear", T=0, I=64, O=64, n=2, dtype="bf16", mode="x")
    inp = wl.make_inputs(w, 0, grad0=True)
    layer = RtpLinear(dev(inp["W"], torch.bfloat16), 0, 2, 0, G0=dev(inp["G0_W"], torch.float32))
    X = torch.empty(0, 64, device=DEV, dtype=torch.bfloat16)
    Y = torch.empty(0, 64, device=DEV, dtype=torch.bfloat16)
    layer.forward(X, Y)
    layer.backward(X, Y, X)
    layer.sync()
    Wb, G = layer.gathered()
    assert torch.equal(Wb, dev(inp["W"], torch.bfloat16))
    assert torch.equal(G, dev(inp["G0_W"], torch.float32)), "no tokens: the travelling gradients pass through unchanged"
    layer.close()


# -------------------------------------------------------------------- MLP unit --

def _schedule(name):
    """Keyword arguments of RtpMlp for a schedule name.  default: forward grouped (independent GEMMs of a step as
    one launch), backward one launch per GEMM with the weight gradients on the auxiliary stream; pipelined: two
    decoupled kernel chains on the compute and the auxiliary stream; grouped: grouped launches in both passes,
    weight gradients on the auxiliary stream; grouped_one_stream: the same on one compute stream; stepwise*: one
    launch per linear and step."""
    return dict(stepwise=name.startswith("stepwise"), grouped=name.startswith("grouped"),
                pipelined=name == "pipelined", fused=name.startswith("fused"), aux_stream=not name.endswith("one_stream"))


SCHEDULES = ["default", "pipelined", "grouped", "grouped_one_stream", "stepwise", "stepwise_one_stream", "fused", "fused_one_stream"]


def _mlp_case(w: wl.Workload, rank, mode, seed=0, grad0=True, **schedule):
    td, bd = _TD[w.dtype], _BD[w.dtype]
    inp = wl.make_inputs(w, seed, grad0=grad0)
    X, dY = inp["X"], inp["dY"]
    if w.kind == "swiglu":
        names, act = ("Wg", "Wu", "Wd"), B.RTP_ACT_SWIGLU
        g0 = [f64(inp["G0_" + k]) for k in names] if grad0 else [None] * 3
        ref = orc.rtp_swiglu(f64(X), *[f64(inp[k]) for k in names], f64(dY), w.n, rank, *g0)
        gkeys = ("dWg", "dWu", "dWd")
    else:
        names, act = ("W1", "W2"), w.extra.get("act", B.RTP_ACT_GELU_ERF)
        g0 = [f64(inp["G0_" + k]) for k in names] if grad0 else [None] * 2
        kind = orc.GELU_TANH if act == B.RTP_ACT_GELU_TANH else orc.GELU_ERF
        ref = orc.rtp_mlp(f64(X), f64(inp["W1"]), f64(inp["W2"]), f64(dY), w.n, rank, kind, *g0)
        gkeys = ("dW1", "dW2")
    mlp = RtpMlp([dev(inp[k], td) for k in names], w.T, w.n, rank, act, mode, bd,
                 G0=[dev(inp["G0_" + k], torch.float32) for k in names] if grad0 else None, **schedule)
    Xd, dYd = dev(X, td), dev(dY, td)
    Y = torch.full((w.T, w.O2), float("nan"), device=DEV, dtype=td)
    dX = torch.full((w.T, w.I), float("nan"), device=DEV, dtype=td)
    torch.cuda.synchronize()
    mlp.forward(Xd, Y)
    mlp.backward(Xd, dYd, dX)
    mlp.sync()
    Ws, Gs = mlp.gathered()
    same = all(torch.equal(a, dev(inp[k], td)) for a, k in zip(Ws, names))
    out = dict(Y=host(Y), dX=host(dX), W_same=same, H=host(mlp.hidden))
    for key, g in zip(gkeys, Gs):
        out[key] = host(g)
    mlp.close()
    return out, ref, gkeys


@pytest.mark.parametrize("mode", [B.RTP_DOUBLE_BUFFER, B.RTP_INPLACE_STAGED, B.RTP_INPLACE_BLOCKING])
@pytest.mark.parametrize("kind,dtype", [("mlp_gelu", "f32"), ("swiglu", "f32"), ("mlp_gelu", "bf16"), ("swiglu", "bf16")])
def test_mlp_unit_small(kind, dtype, mode):
    w = wl.Workload("mlp_small", kind, T=200, I=136, O=4 * 136, O2=120, n=4, dtype=dtype, mode="x",
                    w_dist=("normal", 0.08))
    for rank in (0, 2):
        say(f"mlp kind={kind} dtype={dtype} mode={mode} rank={rank}")
        out, ref, gkeys = _mlp_case(w, rank, mode)
        assert out["W_same"]
        tol = TOL_F32 if dtype == "f32" else TOL_BF16
        for key in ("H", "Y", "dX") + tuple(gkeys):
            assert np.isfinite(out[key]).all(), key
            assert relerr(out[key], ref[key]) <= tol, (key, relerr(out[key], ref[key]))


@pytest.mark.parametrize("schedule", SCHEDULES)
@pytest.mark.parametrize("mode", [B.RTP_DOUBLE_BUFFER, B.RTP_INPLACE_STAGED])
@pytest.mark.parametrize("kind,n", [("mlp_gelu", 4), ("swiglu", 4), ("swiglu", 3), ("swiglu", 2), ("swiglu", 1)])
def test_mlp_unit_grouped_launches(kind, n, mode, schedule):
    """Shapes the tiled kernel takes (every contraction length a multiple of 32), so the unit can run
    its pipelined and grouped schedules; ragged tiles in every dimension.  Every schedule (see _schedule)
    must give the oracle's results."""
    w = wl.Workload("mlp_grouped", kind, T=288, I=160, O=n * 128, O2=96, n=n, dtype="bf16", mode="x",
                    w_dist=("normal", 0.08))
    for rank in sorted({0, n - 1}):
        say(f"grouped mlp kind={kind} n={n} mode={mode} schedule={schedule} rank={rank}")
        out, ref, gkeys = _mlp_case(w, rank, mode, **_schedule(schedule))
        assert out["W_same"]
        for key in ("H", "Y", "dX") + tuple(gkeys):
            assert np.isfinite(out[key]).all(), key
            assert relerr(out[key], ref[key]) <= TOL_BF16, (key, relerr(out[key], ref[key]))


@pytest.mark.parametrize("schedule", ["default", "pipelined", "grouped_one_stream", "stepwise", "fused"])
@pytest.mark.parametrize("kind", ["mlp_gelu", "swiglu"])
def test_mlp_unit_fp16(kind, schedule):
    w = wl.Workload("mlp_f16", kind, T=288, I=160, O=4 * 128, O2=96, n=4, dtype="f16", mode="x", w_dist=("normal", 0.08))
    say(f"fp16 mlp kind={kind} schedule={schedule}")
    out, ref, gkeys = _mlp_case(w, 2, B.RTP_INPLACE_STAGED, **_schedule(schedule))
    assert out["W_same"]
    for key in ("H", "Y", "dX") + tuple(gkeys):
        assert np.isfinite(out[key]).all(), key
        assert relerr(out[key], ref[key]) <= TOL_F16, (key, relerr(out[key], ref[key]))


def test_mlp_grouped_and_stepwise_agree_bitwise_on_integers():
    """Integer-valued inputs: every partial sum is exact, so the grouped and the step-by-step
    schedule must give identical bits whatever the order of their launches."""
    w = wl.Workload("mlp_int", "swiglu", T=320, I=192, O=512, O2=128, n=4, dtype="bf16", mode="x")
    inp = wl.make_inputs(w, seed=5)
    rng = np.random.default_rng(5)
    ints = lambda shape: rng.integers(-2, 3, size=shape).astype(np.float32)
    Ws = [ints(inp[k].shape) for k in ("Wg", "Wu", "Wd")]
    X, dY = ints(inp["X"].shape), ints(inp["dY"].shape)
    res = []
    for sched in ("grouped_one_stream", "default", "pipelined", "grouped", "stepwise", "fused"):
        mlp = RtpMlp([dev(a, torch.bfloat16) for a in Ws], w.T, w.n, 1, B.RTP_ACT_SWIGLU, B.RTP_INPLACE_STAGED, B.RTP_BF16,
                     **_schedule(sched))
        Y = torch.empty(w.T, w.O2, device=DEV, dtype=torch.bfloat16)
        dX = torch.empty(w.T, w.I, device=DEV, dtype=torch.bfloat16)
        Xd, dYd = dev(X, torch.bfloat16), dev(dY, torch.bfloat16)
        torch.cuda.synchronize()
        mlp.forward(Xd, Y)
        mlp.backward(Xd, dYd, dX)
        mlp.sync()
        _, Gs = mlp.gathered()
        res.append([Y.clone(), mlp.hidden.clone(), Gs[2].clone()])
        mlp.close()
    # Y and the hidden activations go through silu (not exact), but both schedules run the same
    # kernels on the same operands; the down-projection gradient sums exact products of dY and H
    for other in res[1:]:
        for a, b in zip(res[0], other):
            assert torch.equal(a, b)


@pytest.mark.parametrize("schedule", ["default", "pipelined", "grouped", "grouped_one_stream", "stepwise", "fused"])
def test_mlp_gradients_accumulate_over_passes(schedule):
    """Two passes of the unit without reading the store in between add the pass's weight gradients twice
    onto what arrived (all shards, the one the worker ends on included): G = G0 + 2 dW, with dW the oracle's."""
    w = wl.Workload("mlp_twice", "swiglu", T=288, I=160, O=4 * 128, O2=96, n=4, dtype="bf16", mode="x", w_dist=("normal", 0.08))
    inp = wl.make_inputs(w, seed=12, grad0=True)
    names = ("Wg", "Wu", "Wd")
    res = []
    for passes in (1, 2):
        mlp = RtpMlp([dev(inp[k], torch.bfloat16) for k in names], w.T, w.n, 1, B.RTP_ACT_SWIGLU, B.RTP_INPLACE_STAGED,
                     B.RTP_BF16, G0=[dev(inp["G0_" + k], torch.float32) for k in names], **_schedule(schedule))
        X, dY = dev(inp["X"], torch.bfloat16), dev(inp["dY"], torch.bfloat16)
        Y = torch.empty(w.T, w.O2, device=DEV, dtype=torch.bfloat16)
        dX = torch.empty(w.T, w.I, device=DEV, dtype=torch.bfloat16)
        for _ in range(passes):
            mlp.forward(X, Y)
            mlp.backward(X, dY, dX)
        mlp.sync()
        _, Gs = mlp.gathered()
        res.append([host(g) for g in Gs])
        mlp.close()
    # the oracle's one-pass result from the same arriving gradients: ref = G0 + dW, so two passes give 2 ref - G0
    ref = orc.rtp_swiglu(f64(inp["X"]), *[f64(inp[k]) for k in names], f64(inp["dY"]), w.n, 1,
                         *[f64(inp["G0_" + k]) for k in names])
    for k, key, g1, g2 in zip(names, ("dWg", "dWu", "dWd"), *res):
        g0 = f64(inp["G0_" + k])
        assert relerr(g1, ref[key]) <= TOL_BF16, (k, relerr(g1, ref[key]))
        assert relerr(g2, 2.0 * ref[key] - g0) <= TOL_BF16, (k, relerr(g2, 2.0 * ref[key] - g0))
        assert relerr(g2 - g0, 2.0 * (g1 - g0)) <= 1e-5, (k, relerr(g2 - g0, 2.0 * (g1 - g0)))


def test_mlp_gelu_tanh_variant():
    w = wl.Workload("mlp_tanh", "mlp_gelu", T=64, I=64, O=128, O2=64, n=2, dtype="bf16", mode="x",
                    w_dist=("normal", 0.1), extra={"act": B.RTP_ACT_GELU_TANH})
    out, ref, gkeys = _mlp_case(w, 1, B.RTP_DOUBLE_BUFFER)
    for key in ("H", "Y", "dX") + tuple(gkeys):
        assert relerr(out[key], ref[key]) <= TOL_BF16, (key, relerr(out[key], ref[key]))


@pytest.mark.parametrize("mode", [B.RTP_DOUBLE_BUFFER, B.RTP_INPLACE_STAGED, B.RTP_INPLACE_BLOCKING])
@pytest.mark.parametrize("dtype,act", [("bf16", B.RTP_ACT_GELU_ERF), ("f32", B.RTP_ACT_GELU_ERF), ("f16", B.RTP_ACT_GELU_TANH)])
def test_mlp_unit_with_biases(dtype, act, mode):
    """The unit's flat parameter with both biases: [W1_k | b1_k | W2_k | piece k of b2]."""
    T, I, O, O2, n = (288, 160, 512, 96, 4) if dtype != "f32" else (100, 40, 48, 20, 4)
    w = wl.Workload("mlp_bias", "mlp_gelu", T=T, I=I, O=O, O2=O2, n=n, dtype=dtype, mode="x", w_dist=("normal", 0.08))
    inp = wl.make_inputs(w, seed=41, grad0=True)
    rng = np.random.default_rng(42)
    b1 = wl._store(rng.standard_normal(O).astype(np.float32) * 0.3, dtype)
    b2 = wl._store(rng.standard_normal(O2).astype(np.float32) * 0.3, dtype)
    gb1, gb2 = rng.standard_normal(O).astype(np.float32), rng.standard_normal(O2).astype(np.float32)
    td, bd = _TD[dtype], _BD[dtype]
    tol = {"f32": TOL_F32, "bf16": TOL_BF16, "f16": TOL_F16}[dtype]
    kind = orc.GELU_TANH if act == B.RTP_ACT_GELU_TANH else orc.GELU_ERF
    for rank in (0, 2):
        say(f"mlp with biases dtype={dtype} act={act} mode={mode} rank={rank}")
        ref = orc.rtp_mlp(f64(inp["X"]), f64(inp["W1"]), f64(inp["W2"]), f64(inp["dY"]), n, rank, kind,
                          f64(inp["G0_W1"]), f64(inp["G0_W2"]), b1=f64(b1), b2=f64(b2), gb1_0=f64(gb1), gb2_0=f64(gb2))
        mlp = RtpMlp([dev(inp[k], td) for k in ("W1", "W2")], T, n, rank, act, mode, bd,
                     G0=[dev(inp["G0_" + k], torch.float32) for k in ("W1", "W2")],
                     biases=[dev(b1, td), dev(b2, td)], gb0=[dev(gb1, torch.float32), dev(gb2, torch.float32)])
        Xd, dYd = dev(inp["X"], td), dev(inp["dY"], td)
        Y = torch.full((T, O2), float("nan"), device=DEV, dtype=td)
        dX = torch.full((T, I), float("nan"), device=DEV, dtype=td)
        torch.cuda.synchronize()
        mlp.forward(Xd, Y)
        mlp.backward(Xd, dYd, dX)
        mlp.sync()
        Ws, Gs = mlp.gathered()
        (bb1, bb2), (g1, g2) = mlp.gathered_biases()
        assert all(torch.equal(a, dev(inp[k], td)) for a, k in zip(Ws, ("W1", "W2")))
        assert torch.equal(bb1, dev(b1, td)) and torch.equal(bb2, dev(b2, td))
        got = dict(Y=Y, dX=dX, H=mlp.hidden, dW1=Gs[0], dW2=Gs[1], db1=g1, db2=g2)
        for key, val in got.items():
            assert torch.isfinite(val.float()).all(), key
            assert relerr(host(val), ref[key]) <= tol, (key, relerr(host(val), ref[key]))
        mlp.close()


@pytest.mark.parametrize("schedule", ["default", "pipelined", "grouped", "grouped_one_stream", "stepwise", "fused"])
@pytest.mark.parametrize("gated", [False, True])
def test_mlp_unit_with_biases_in_every_schedule(gated, schedule):
    """Biases of the unit's linears (for the gated unit: gate, up and down) in every launch schedule, shapes the
    tiled kernel takes; arriving bias gradients are added onto."""
    T, I, O, O2, n = 288, 160, 512, 96, 4
    w = wl.Workload("mlp_bias_sched", "swiglu" if gated else "mlp_gelu", T=T, I=I, O=O, O2=O2, n=n, dtype="bf16", mode="x",
                    w_dist=("normal", 0.08))
    inp = wl.make_inputs(w, seed=51, grad0=True)
    rng = np.random.default_rng(52)
    names = ("Wg", "Wu", "Wd") if gated else ("W1", "W2")
    sizes = [O] * (len(names) - 1) + [O2]
    bs = [wl._store(rng.standard_normal(sz).astype(np.float32) * 0.3, "bf16") for sz in sizes]
    gbs = [rng.standard_normal(sz).astype(np.float32) for sz in sizes]
    for mode in (B.RTP_INPLACE_STAGED, B.RTP_DOUBLE_BUFFER) + ((B.RTP_INPLACE_BLOCKING,) if schedule == "fused" else ()):
        rank = 2
        say(f"biased mlp gated={gated} schedule={schedule} mode={mode}")
        if gated:
            ref = orc.rtp_swiglu(f64(inp["X"]), *[f64(inp[k]) for k in names], f64(inp["dY"]), n, rank,
                                 *[f64(inp["G0_" + k]) for k in names], *[f64(b) for b in bs], *[f64(g) for g in gbs])
            gkeys, bkeys = ("dWg", "dWu", "dWd"), ("dbg", "dbu", "dbd")
        else:
            ref = orc.rtp_mlp(f64(inp["X"]), f64(inp["W1"]), f64(inp["W2"]), f64(inp["dY"]), n, rank, orc.GELU_ERF,
                              f64(inp["G0_W1"]), f64(inp["G0_W2"]), b1=f64(bs[0]), b2=f64(bs[1]), gb1_0=f64(gbs[0]), gb2_0=f64(gbs[1]))
            gkeys, bkeys = ("dW1", "dW2"), ("db1", "db2")
        mlp = RtpMlp([dev(inp[k], torch.bfloat16) for k in names], T, n, rank, B.RTP_ACT_SWIGLU if gated else B.RTP_ACT_GELU_ERF,
                     mode, B.RTP_BF16, G0=[dev(inp["G0_" + k], torch.float32) for k in names],
                     biases=[dev(b, torch.bfloat16) for b in bs], gb0=[dev(g, torch.float32) for g in gbs], **_schedule(schedule))
        Xd, dYd = dev(inp["X"], torch.bfloat16), dev(inp["dY"], torch.bfloat16)
        Y = torch.full((T, O2), float("nan"), device=DEV, dtype=torch.bfloat16)
        dX = torch.full((T, I), float("nan"), device=DEV, dtype=torch.bfloat16)
        torch.cuda.synchronize()
        mlp.forward(Xd, Y)
        mlp.backward(Xd, dYd, dX)
        mlp.sync()
        Ws, Gs = mlp.gathered()
        bb, gg = mlp.gathered_biases()
        assert all(torch.equal(a, dev(inp[k], torch.bfloat16)) for a, k in zip(Ws, names))
        assert all(torch.equal(a, dev(b, torch.bfloat16)) for a, b in zip(bb, bs))
        got = dict(Y=Y, dX=dX, H=mlp.hidden)
        got.update(zip(gkeys, Gs))
        got.update(zip(bkeys, gg))
        for key, val in got.items():
            assert torch.isfinite(val.float()).all(), key
            assert relerr(host(val), ref[key]) <= TOL_BF16, (key, relerr(host(val), ref[key]))
        mlp.close()


@pytest.mark.parametrize("schedule", ["default", "pipelined", "stepwise", "fused"])
@pytest.mark.parametrize("kind,dtype,O,n", [("mlp_gelu", "bf16", 232, 6), ("swiglu", "bf16", 232, 6), ("swiglu", "f16", 736, 6),
                                            ("mlp_gelu", "f32", 50, 4), ("swiglu", "f32", 50, 4)])
def test_mlp_unit_with_a_padded_partition(kind, dtype, O, n, schedule):
    """A hidden width the partition factor does not divide: the unit runs on n shards of the padded width
    (rtp_mlp_hidden_width); the padding units have zero weights, so act(0) = 0 and they change nothing.  The
    reference is the unsharded definition (the rotated oracle needs an even partition)."""
    if dtype == "f32" and schedule != "stepwise":
        pytest.skip("the fp32 unit has one schedule")
    T, I, O2 = (96, 64, 64) if dtype != "f32" else (40, 24, 20)
    w = wl.Workload("mlp_padded", kind, T=T, I=I, O=O, O2=O2, n=n, dtype=dtype, mode="x", w_dist=("normal", 0.1))
    inp = wl.make_inputs(w, seed=61, grad0=True)
    td, bd = _TD[dtype], _BD[dtype]
    tol = {"f32": TOL_F32, "bf16": TOL_BF16, "f16": TOL_F16}[dtype]
    gated = kind == "swiglu"
    names = ("Wg", "Wu", "Wd") if gated else ("W1", "W2")
    if gated:
        ref = orc.plain_swiglu(f64(inp["X"]), *[f64(inp[k]) for k in names], f64(inp["dY"]))
        gkeys = ("dWg", "dWu", "dWd")
    else:
        ref = orc.plain_mlp(f64(inp["X"]), f64(inp["W1"]), f64(inp["W2"]), f64(inp["dY"]))
        gkeys = ("dW1", "dW2")
    for mode in (B.RTP_INPLACE_STAGED, B.RTP_DOUBLE_BUFFER, B.RTP_INPLACE_BLOCKING):
        say(f"padded mlp kind={kind} dtype={dtype} O={O} n={n} schedule={schedule} mode={mode}")
        mlp = RtpMlp([dev(inp[k], td) for k in names], T, n, n - 1, B.RTP_ACT_SWIGLU if gated else B.RTP_ACT_GELU_ERF, mode, bd,
                     G0=[dev(inp["G0_" + k], torch.float32) for k in names], **_schedule(schedule))
        assert mlp.hidden_width > O and mlp.hidden_width % n == 0
        Xd, dYd = dev(inp["X"], td), dev(inp["dY"], td)
        Y = torch.full((T, O2), float("nan"), device=DEV, dtype=td)
        dX = torch.full((T, I), float("nan"), device=DEV, dtype=td)
        torch.cuda.synchronize()
        mlp.forward(Xd, Y)
        mlp.backward(Xd, dYd, dX)
        mlp.sync()
        Ws, Gs = mlp.gathered()
        assert all(torch.equal(a, dev(inp[k], td)) for a, k in zip(Ws, names)), "weights unchanged, padding dropped"
        H = mlp.hidden
        assert torch.count_nonzero(H[:, O:]) == 0, "padding units: act(0) = 0"
        got = dict(Y=Y, dX=dX, H=H[:, :O])
        for key, g, k in zip(gkeys, Gs, names):
            got[key] = g.double().cpu() - torch.from_numpy(f64(inp["G0_" + k]))     # arriving + own, minus arriving
        for key, val in got.items():
            assert torch.isfinite(val.float()).all(), key
            assert relerr(host(val), ref[key]) <= tol, (key, relerr(host(val), ref[key]))
        mlp.close()


def test_units_cleared_gradients_start_from_zero():
    """zero_grads between two passes of the MLP unit and of the expert-partitioned layer: the second
    pass's gradients are those of one pass from zero (the shard the worker kept is dropped)."""
    w = wl.Workload("mlp_zero", "swiglu", T=288, I=160, O=512, O2=96, n=4, dtype="bf16", mode="x", w_dist=("normal", 0.08))
    inp = wl.make_inputs(w, seed=8, grad0=True)
    names = ("Wg", "Wu", "Wd")
    ref = orc.rtp_swiglu(f64(inp["X"]), *[f64(inp[k]) for k in names], f64(inp["dY"]), 4, 1)
    mlp = RtpMlp([dev(inp[k], torch.bfloat16) for k in names], w.T, 4, 1, B.RTP_ACT_SWIGLU, B.RTP_INPLACE_STAGED, B.RTP_BF16,
                 G0=[dev(inp["G0_" + k], torch.float32) for k in names])
    Xd, dYd = dev(inp["X"], torch.bfloat16), dev(inp["dY"], torch.bfloat16)
    Y = torch.empty(w.T, w.O2, device=DEV, dtype=torch.bfloat16)
    dX = torch.empty(w.T, w.I, device=DEV, dtype=torch.bfloat16)
    say("mlp: pass, zero_grads, pass")
    mlp.forward(Xd, Y)
    mlp.backward(Xd, dYd, dX)
    mlp.zero_grads()
    mlp.forward(Xd, Y)
    mlp.backward(Xd, dYd, dX)
    mlp.sync()
    _, Gs = mlp.gathered()
    for key, g in zip(("dWg", "dWu", "dWd"), Gs):
        assert relerr(host(g), ref[key]) <= TOL_BF16, key
    mlp.close()

    n, T = 4, 300
    mi = wl.make_moe_inputs(T, 64, 96, 64, n, seed=12)
    ex64 = [tuple(f64(m) for m in ex) for ex in mi["experts"]]
    mref = orc.rtp_moe(f64(mi["X"]), mi["route"], ex64, f64(mi["dY"]), n, 2)
    moe = RtpMoe([tuple(dev(m, torch.bfloat16) for m in ex) for ex in mi["experts"]], T, 2, B.RTP_ACT_GELU_ERF,
                 G0=[tuple(dev(g, torch.float32) for g in ex) for ex in mi["G0"]])
    Xd, dYd, rd = dev(mi["X"], torch.bfloat16), dev(mi["dY"], torch.bfloat16), dev(mi["route"], torch.int32)
    Y = torch.empty(T, 64, device=DEV, dtype=torch.bfloat16)
    dX = torch.empty(T, 64, device=DEV, dtype=torch.bfloat16)
    say("moe: pass, zero_grads, pass")
    moe.forward(Xd, rd, Y)
    moe.backward(dYd, dX)
    moe.zero_grads()
    moe.forward(Xd, rd, Y)
    moe.backward(dYd, dX)
    moe.sync()
    _, Gs = moe.gathered()
    for e in range(n):
        for j in range(2):
            assert relerr(host(Gs[e][j]), mref["G"][e][j]) <= TOL_BF16, (e, j)
    moe.close()


# ------------------------------------------------------------ HIP graphs --

def test_a_capturing_stream_is_refused_before_anything_is_enqueued():
    """Passes cannot be recorded into a HIP graph: with the compute stream capturing, every call that would open
    a pass or enqueue on the ring's streams returns RTP_ERR_UNSUPPORTED and enqueues nothing (the capture stays
    empty of the library's work and ends normally); afterwards the layer works as before."""
    T, I, O, n = 64, 64, 128, 4
    g = torch.Generator(device="cpu").manual_seed(9)
    ri = lambda lo, hi, shape: torch.randint(lo, hi, shape, generator=g).float()
    W, X = ri(-2, 3, (O, I)), ri(-2, 3, (T, I))
    layer = RtpLinear(W.to(DEV, torch.bfloat16), T, n, 1, B.RTP_SPLIT_OUT, B.RTP_DOUBLE_BUFFER, B.RTP_BF16)
    Xd = X.to(DEV, torch.bfloat16)
    Y = torch.zeros(T, O, device=DEV, dtype=torch.bfloat16)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    seen = []
    say("begin an (empty) capture on the compute stream")
    with torch.cuda.graph(graph, stream=layer.compute_stream, capture_error_mode="relaxed"):
        for call in (lambda: layer.ring.begin(B.RTP_PASS_FWD), layer.ring.seek_bwd_start, layer.ring.zero_grads):
            with pytest.raises(B.RtpError) as e:
                call()
            seen.append(e.value.status)
    say("capture ended")
    torch.cuda.synchronize()
    assert seen == [B.RTP_ERR_UNSUPPORTED] * 3
    layer.forward(Xd, Y)
    layer.sync()
    assert torch.equal(Y.float().cpu(), (X.double() @ W.double().T).float())
    layer.close()


@pytest.mark.skip(reason="capturing a linear layer's pass (double-buffer mode, three streams) crashed the host inside the "
                         "runtime's end-of-capture call; the cause is not established, so stream capture of a pass is "
                         "documented as unsupported and this case stays off the GPU")
@pytest.mark.parametrize("mode", [B.RTP_DOUBLE_BUFFER, B.RTP_INPLACE_STAGED])
def test_captured_pass_replays_like_eager(mode):
    """A forward + backward pass captured into a HIP graph (after one eager pass, so that the
    capture holds the write-back of the gradient shard the previous pass ended on) and replayed
    three times, with eager passes and synchronisations in between: every replay gives the eager
    outputs, and the gradients count every pass, eager or replayed (integer inputs: bit-exact)."""
    T, I, O, n = 256, 512, 1024, 4
    g = torch.Generator(device="cpu").manual_seed(6)
    ri = lambda lo, hi, shape: torch.randint(lo, hi, shape, generator=g).float()
    W, X, dY, G0 = ri(-2, 3, (O, I)), ri(-2, 3, (T, I)), ri(-2, 3, (T, O)), ri(-4, 5, (O, I))
    layer = RtpLinear(W.to(DEV, torch.bfloat16), T, n, 1, B.RTP_SPLIT_OUT, mode, B.RTP_BF16, G0=G0.to(DEV))
    Xd, dYd = X.to(DEV, torch.bfloat16), dY.to(DEV, torch.bfloat16)
    Y = torch.empty(T, O, device=DEV, dtype=torch.bfloat16)
    dX = torch.empty(T, I, device=DEV, dtype=torch.bfloat16)
    Y_ref = (X.double() @ W.double().T).to(torch.bfloat16)
    dX_ref = (dY.double() @ W.double()).to(torch.bfloat16)
    dW = (dY.double().T @ X.double()).float()
    passes = 0

    def eager():
        nonlocal passes
        layer.forward(Xd, Y)
        layer.backward(Xd, dYd, dX)
        layer.sync()
        passes += 1

    eager()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    say(f"capturing a pass, mode {mode}")
    with torch.cuda.graph(graph, stream=layer.compute_stream, capture_error_mode="relaxed"):
        layer.forward(Xd, Y)
        layer.backward(Xd, dYd, dX)
    torch.cuda.synchronize()             # capture enqueues nothing: the pass has not run
    for i in range(3):
        Y.fill_(float("nan"))
        dX.fill_(float("nan"))
        torch.cuda.synchronize()
        say(f"replay {i}")
        graph.replay()
        torch.cuda.synchronize()
        passes += 1
        assert torch.equal(Y.cpu(), Y_ref) and torch.equal(dX.cpu(), dX_ref), f"replay {i}"
        eager()
        assert torch.equal(Y.cpu(), Y_ref) and torch.equal(dX.cpu(), dX_ref)
    _, G = layer.gathered()
    assert torch.equal(G.cpu(), G0 + passes * dW), "every pass, eager or replayed, adds its weight gradient once"
    del graph
    layer.close()


# ------------------------------------------------------- expert partition --

def _moe_case(T, I, O, O2, n, rank, mode, gated, dtype="bf16", seed=0, skew=1.0, route=None, aux_stream=True, passes=1):
    td, bd = _TD[dtype], _BD[dtype]
    inp = wl.make_moe_inputs(T, I, O, O2, n, dtype=dtype, gated=gated, seed=seed, skew=skew)
    if route is not None:
        inp["route"] = np.asarray(route, dtype=np.int32)
    act = B.RTP_ACT_SWIGLU if gated else B.RTP_ACT_GELU_ERF
    ex64 = [tuple(f64(w) for w in ex) for ex in inp["experts"]]
    g64 = [tuple(f64(g) for g in ex) for ex in inp["G0"]]
    ref = orc.rtp_moe(f64(inp["X"]), inp["route"], ex64, f64(inp["dY"]), n, rank, G0=g64)
    moe = RtpMoe([tuple(dev(w, td) for w in ex) for ex in inp["experts"]], T, rank, act, mode, bd,
                 G0=[tuple(dev(g, torch.float32) for g in ex) for ex in inp["G0"]], aux_stream=aux_stream)
    Xd, dYd, rd = dev(inp["X"], td), dev(inp["dY"], td), dev(inp["route"], torch.int32)
    Y = torch.full((T, O2), float("nan"), device=DEV, dtype=td)
    dX = torch.full((T, I), float("nan"), device=DEV, dtype=td)
    torch.cuda.synchronize()
    for _ in range(passes):
        moe.forward(Xd, rd, Y)
        moe.backward(dYd, dX)
    moe.sync()
    counts, begin = moe.routing()
    perm = moe.perm.cpu().tolist()
    Ws, Gs = moe.gathered()
    same = all(torch.equal(a, dev(b, td)) for exa, exb in zip(Ws, inp["experts"]) for a, b in zip(exa, exb))
    out = dict(Y=host(Y), dX=host(dX), G=[[host(g) for g in ex] for ex in Gs], W_same=same, counts=counts, begin=begin,
               perm=perm, Tp=moe.Tp)
    moe.close()
    return out, ref, inp


def _check_moe(out, ref, inp, n, tol, passes=1):
    # integer work, bit-exact: group sizes, group starts, the token of every grouped row, padding rows
    c, b, perm = orc.moe_dispatch(inp["route"], n, 32)
    assert out["counts"] == c == ref["counts"] and out["begin"] == b
    assert out["perm"][:b[n]] == perm and all(p == -1 for p in out["perm"][b[n]:]) and len(out["perm"]) == out["Tp"]
    assert out["W_same"], "the expert weights come back unchanged"
    for key in ("Y", "dX"):
        assert np.isfinite(out[key]).all(), key
        assert relerr(out[key], ref[key]) <= tol, (key, relerr(out[key], ref[key]))
    for e in range(n):
        for j, g in enumerate(out["G"][e]):
            g0 = f64(inp["G0"][e][j])
            want = g0 + passes * (ref["G"][e][j] - g0)
            assert relerr(g, want) <= tol, (e, j, relerr(g, want))
            if c[e] == 0:
                assert np.array_equal(g, g0), "an expert without tokens passes through untouched"


@pytest.mark.parametrize("mode", [B.RTP_DOUBLE_BUFFER, B.RTP_INPLACE_STAGED, B.RTP_INPLACE_BLOCKING])
@pytest.mark.parametrize("gated", [False, True])
def test_moe_small(gated, mode):
    """Ragged group sizes, an output width that sends one GEMM to the register-staged kernel."""
    n = 4
    for rank in (0, 3):
        say(f"moe small gated={gated} mode={mode} rank={rank}")
        out, ref, inp = _moe_case(300, 64, 96, 72, n, rank, mode, gated, seed=rank)
        _check_moe(out, ref, inp, n, TOL_BF16)


@pytest.mark.parametrize("aux", [True, False])
@pytest.mark.parametrize("gated,skew", [(False, 0.0), (True, 1.0), (True, 2.5)])
def test_moe_several_tiles(gated, skew, aux):
    """Groups from a handful of rows to several row tiles; uniform to heavily skewed load."""
    n = 8
    say(f"moe tiles gated={gated} skew={skew} aux={aux}")
    out, ref, inp = _moe_case(1500, 256, 384, 256, n, 5, B.RTP_INPLACE_STAGED, gated, seed=3, skew=skew, aux_stream=aux)
    _check_moe(out, ref, inp, n, TOL_BF16)


def test_moe_degenerate_routings():
    n, T = 4, 200
    for name, route in (("one expert takes all", np.full(T, 2)), ("two experts idle", np.arange(T) % 2 * 3),
                        ("one token each", None)):
        say(f"moe degenerate: {name}")
        if route is None:
            T_, route = n, np.arange(n)[::-1].copy()
        else:
            T_ = T
        out, ref, inp = _moe_case(T_, 64, 64, 64, n, 1, B.RTP_DOUBLE_BUFFER, False, route=route)
        _check_moe(out, ref, inp, n, TOL_BF16)
    say("moe degenerate: a single expert, one worker")
    out, ref, inp = _moe_case(100, 64, 64, 64, 1, 0, B.RTP_INPLACE_STAGED, True)
    _check_moe(out, ref, inp, 1, TOL_BF16)
    say("moe degenerate: no tokens")
    out, ref, inp = _moe_case(0, 64, 64, 64, 4, 0, B.RTP_INPLACE_STAGED, False)
    _check_moe(out, ref, inp, 4, TOL_BF16)


def test_moe_fp16():
    say("moe fp16")
    out, ref, inp = _moe_case(500, 128, 256, 96, 4, 2, B.RTP_INPLACE_STAGED, True, dtype="f16", seed=2)
    _check_moe(out, ref, inp, 4, TOL_F16)


def test_moe_gradients_accumulate_over_passes():
    say("moe two passes")
    out, ref, inp = _moe_case(400, 64, 128, 64, 4, 1, B.RTP_INPLACE_STAGED, False, passes=2)
    _check_moe(out, ref, inp, 4, TOL_BF16, passes=2)


@pytest.mark.parametrize("mode", [B.RTP_DOUBLE_BUFFER, B.RTP_INPLACE_STAGED, B.RTP_INPLACE_BLOCKING])
def test_moe_own_experts_gradients_reach_their_slot(mode):
    """The backward pass ends on the worker's own expert, which travels no further: its weight-gradient kernels store
    `arrived + own` straight into the own slot (staged modes, an expert with tokens), so the store is current
    without a flush; the blocking mode leaves the shard in the buffer, and the ring says so."""
    n, T, rank = 4, 300, 2
    mi = wl.make_moe_inputs(T, 64, 96, 64, n, seed=87)
    ex64 = [tuple(f64(m) for m in ex) for ex in mi["experts"]]
    g64 = [tuple(f64(g) for g in ex) for ex in mi["G0"]]
    ref = orc.rtp_moe(f64(mi["X"]), mi["route"], ex64, f64(mi["dY"]), n, rank, G0=g64)
    assert ref["counts"][rank] > 0
    moe = RtpMoe([tuple(dev(m, torch.bfloat16) for m in ex) for ex in mi["experts"]], T, rank, B.RTP_ACT_GELU_ERF, mode,
                 G0=[tuple(dev(g, torch.float32) for g in ex) for ex in mi["G0"]])
    ring = B.lib.rtp_moe_ring(moe.handle)
    X, dY, route = dev(mi["X"], torch.bfloat16), dev(mi["dY"], torch.bfloat16), dev(mi["route"], torch.int32)
    Y = torch.empty(T, 64, device=DEV, dtype=torch.bfloat16)
    dX = torch.empty(T, 64, device=DEV, dtype=torch.bfloat16)
    for p in (1, 2):
        say(f"moe own expert mode={mode} pass {p}")
        moe.forward(X, route, Y)
        moe.backward(dY, dX)
        moe.sync()
        held = B.lib.rtp_ring_resident_grad(ring)
        assert held == (rank if mode == B.RTP_INPLACE_BLOCKING else -1)
        if held < 0:                                          # no flush: the store as it is
            for j, (rows, cols) in enumerate(moe.shapes):
                got = torch.empty(rows, cols, dtype=torch.float32, device=DEV)
                B.rtp_unpack_shards(got, moe.home_g.data_ptr() + rank * moe.g_bytes, moe.g_bytes, moe._offsets[j] * 4, 1,
                                    B.RTP_SPLIT_OUT, rows, cols, rows, B.RTP_F32)
                torch.cuda.synchronize()
                want = g64[rank][j] + p * (ref["G"][rank][j] - g64[rank][j])
                assert relerr(host(got), want) <= TOL_BF16, (j, p)
    _, Gs = moe.gathered()
    assert B.lib.rtp_ring_resident_grad(ring) == -1
    for e in range(n):
        for j in range(2):
            assert relerr(host(Gs[e][j]), g64[e][j] + 2 * (ref["G"][e][j] - g64[e][j])) <= TOL_BF16, (e, j)
    moe.close()


def test_moe_rejects_an_expert_id_out_of_range_and_goes_on():
    n, T = 4, 64
    inp = wl.make_moe_inputs(T, 64, 64, 64, n, seed=9)
    moe = RtpMoe([tuple(dev(w, torch.bfloat16) for w in ex) for ex in inp["experts"]], T, 0, B.RTP_ACT_GELU_ERF)
    Xd, Y = dev(inp["X"], torch.bfloat16), torch.empty(T, 64, device=DEV, dtype=torch.bfloat16)
    bad = inp["route"].copy()
    bad[5], bad[17] = n, -1
    with pytest.raises(B.RtpError):
        moe.forward(Xd, dev(bad, torch.int32), Y)
    with pytest.raises(B.RtpError):
        moe.backward(Xd, Y)                      # no forward has completed
    moe.forward(Xd, dev(inp["route"], torch.int32), Y)
    moe.sync()
    ex64 = [tuple(f64(w) for w in ex) for ex in inp["experts"]]
    ref = orc.plain_moe(f64(inp["X"]), inp["route"], ex64, f64(inp["dY"]))
    assert relerr(host(Y), ref["Y"]) <= TOL_BF16
    moe.close()
