"""Passes whose transfers ride in the GEMM launches (narrow shards) against the same passes on three streams: same
outputs, same gradients, same store, bit for bit (no sum here is split along K).  A test delay on any stream, here one
microsecond, keeps a pass on the streams."""
import ctypes as C

import pytest
import torch

import gemm_internal as G
from paper_2311_01635_amd import binding as B
from paper_2311_01635_amd.layers import RtpLinear, RtpMlp

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TD = {B.RTP_BF16: torch.bfloat16, B.RTP_F16: torch.float16, B.RTP_F32: torch.float32}
DB, IS = B.RTP_DOUBLE_BUFFER, B.RTP_INPLACE_STAGED


def normal(seed, *shape, dtype=torch.float32):
    return torch.randn(*shape, generator=torch.Generator(device=DEV).manual_seed(seed), device=DEV).to(dtype)


def off_by_one(t):
    """The same matrix two bytes past a 16-byte boundary, where no GEMM takes an operand."""
    flat = torch.empty(t.numel() + 8, device=DEV, dtype=t.dtype)[1:1 + t.numel()]
    return flat.copy_(t.flatten()).view(t.shape)


def passes(layer, ring, X, dY, linear, streams, plan=("fb", "fb", "f", "zfb"), shift=False):
    """Several passes in a row, so that what a pass leaves in the buffers is picked up by the next; every output of each.
    shift: the outputs start two bytes past a 16-byte boundary."""
    scratch = torch.zeros(2, dtype=torch.int64, device=DEV)
    B.check(B.lib.rtp_ring_set_test_delay_compute(ring, B._ptr(scratch), 1 if streams else 0), "delay")
    out = []
    for t in layer.buf_w + layer.buf_g:
        if t is not None:
            t.fill_(255)                       # nothing is legally read before it is written
    for p in plan:
        if "z" in p:
            layer.zero_grads()
        Y, dX = (off_by_one(t) if shift else torch.empty_like(t) for t in (dY, X))
        layer.forward(X, Y)
        out.append(Y)
        assert B.lib.rtp_ring_rides(ring) == (not streams), "forward"
        if "b" in p:
            layer.backward(X, dY, dX)
            out.append(dX)
            assert B.lib.rtp_ring_rides(ring) == (not streams), "backward"
    layer.sync()
    held = B.lib.rtp_ring_resident_grad(ring)
    W, G = layer.gathered()
    if linear:
        W, G = (W,), (G,)
    out += list(W) + list(G) + [layer.home_w.clone(), layer.home_g.clone()]
    assert (scratch[0].item() > 0) == streams
    return out, held


def same(make, X, dY, linear, shift=False):
    runs = []
    for streams in (False, True):
        layer = make()
        ring = layer.ring.handle if linear else B.lib.rtp_mlp_ring(layer.handle)
        runs.append(passes(layer, ring, X, dY, linear, streams, shift=shift))
        layer.close()
    (a, held_a), (b, held_b) = runs
    assert held_a == held_b
    assert all(torch.isfinite(t.float()).all() for t in a[:-2])
    for i, (x, y) in enumerate(zip(a, b)):
        assert torch.equal(x, y), i


@pytest.mark.parametrize("aux", [True, False])
@pytest.mark.parametrize("mode", [DB, IS])
@pytest.mark.parametrize("n,rank", [(2, 0), (2, 1), (3, 1), (8, 7)])
@pytest.mark.parametrize("split", [B.RTP_SPLIT_OUT, B.RTP_SPLIT_IN])
@pytest.mark.parametrize("dtype,bias", [(B.RTP_BF16, False), (B.RTP_BF16, True), (B.RTP_F16, True), (B.RTP_F32, False), (B.RTP_F32, True)])
def test_linear_layer(dtype, bias, split, n, rank, mode, aux):
    if not aux and n != 3:
        pytest.skip("one partition without an auxiliary stream is enough")
    td, u = TD[dtype], 32 if dtype == B.RTP_F16 else 8
    T = {B.RTP_F16: 96, B.RTP_BF16: 75, B.RTP_F32: 33}[dtype]
    part, other = n * u * 3, 136 if dtype != B.RTP_F16 else 160
    O, I = (part, other) if split == B.RTP_SPLIT_OUT else (other, part)
    X, dY, W = normal(1, T, I, dtype=td), normal(2, T, O, dtype=td), normal(3, O, I) * 0.1
    g0, b = normal(4, O, I), normal(5, O) if bias else None
    make = lambda: RtpLinear(W, T, n, rank, split, mode, dtype, G0=g0, bias=b, aux_stream=aux)
    same(make, X, dY, True)


@pytest.mark.parametrize("mode", [DB, IS])
@pytest.mark.parametrize("n,rank", [(2, 1), (3, 0), (8, 3)])
@pytest.mark.parametrize("act,bias,dtype,T", [(B.RTP_ACT_GELU_ERF, False, B.RTP_BF16, 77), (B.RTP_ACT_GELU_TANH, True, B.RTP_F16, 96),
                                              (B.RTP_ACT_SWIGLU, True, B.RTP_BF16, 77), (B.RTP_ACT_SWIGLU, False, B.RTP_F32, 77),
                                              (B.RTP_ACT_SWIGLU, True, B.RTP_BF16, 1990)])  # (the bias sums' main loop: 1024 rows a trip)
def test_mlp_unit(act, bias, dtype, T, n, rank, mode):
    td, u = TD[dtype], 32 if dtype == B.RTP_F16 else 8
    I, O, O2 = 128, n * u * 3, 160
    shapes = [(O, I)] * (2 if act == B.RTP_ACT_SWIGLU else 1) + [(O2, O)]
    X, dY = normal(1, T, I, dtype=td), normal(2, T, O2, dtype=td)
    ws, g0 = [normal(3 + i, *s) * 0.1 for i, s in enumerate(shapes)], [normal(13 + i, *s) for i, s in enumerate(shapes)]
    bs = [normal(23 + i, s[0]) for i, s in enumerate(shapes)] if bias else None
    make = lambda: RtpMlp(ws, T, n, rank, act, mode, dtype, G0=g0, biases=bs)
    same(make, X, dY, False)


BACKWARD = {B.RTP_ACT_GELU_ERF: G.EPI_GELU_ERF_BWD, B.RTP_ACT_SWIGLU: G.EPI_SWIGLU_BWD}
SQUARE, D128, D64, D64S = G.SMALL_128X128, G.DUO_128X128, G.DUO_64X128, G.DUO_64X64


# The kernel with a compute unit to itself, and the wider tiles of the one that shares it, in the launches that hold both
# layouts and have bias sums in front of their tiles: tiles of {dPre, dW2} and of {dX, dW1}
@pytest.mark.parametrize("mode", [DB, IS])
@pytest.mark.parametrize("act,dtype,T,I,o,first,second", [(B.RTP_ACT_SWIGLU, B.RTP_F16, 416, 960, 320, (D64S, D64S), (64, 64)),
                                                          (B.RTP_ACT_SWIGLU, B.RTP_BF16, 500, 1024, 272, (D64S, D64S), (64, 64)),
                                                          (B.RTP_ACT_SWIGLU, B.RTP_BF16, 1300, 960, 392, (64, 64), (SQUARE, 64)),
                                                          (B.RTP_ACT_GELU_ERF, B.RTP_BF16, 1990, 448, 432, (D128, D64S), (D128, D64S)),
                                                          (B.RTP_ACT_GELU_ERF, B.RTP_BF16, 1300, 768, 456, (D64, D64S), (D64, D64S)),
                                                          (B.RTP_ACT_SWIGLU, B.RTP_F16, 832, 1024, 224, (D64S, D64S), (D64, D64S))])
def test_biased_units_on_every_kernel(act, dtype, T, I, o, first, second, mode):
    g = 2 * o if act == B.RTP_ACT_SWIGLU else o
    assert tuple(G.riding_tiles([(B.LAYOUT_NN, T, o, I, BACKWARD[act]), (B.LAYOUT_TN, I, o, T, G.EPI_ACC_LAST)])) == first
    assert tuple(G.riding_tiles([(B.LAYOUT_NN, T, I, g, G.EPI_ACC_LAST), (B.LAYOUT_TN, g, I, T, G.EPI_ACC_LAST)])) == second
    td, n = TD[dtype], 2
    shapes = [(n * o, I)] * (g // o) + [(I, n * o)]
    ws, g0 = [normal(3 + i, *s) * 0.1 for i, s in enumerate(shapes)], [normal(13 + i, *s) for i, s in enumerate(shapes)]
    bs = [normal(23 + i, s[0]) for i, s in enumerate(shapes)]
    make = lambda: RtpMlp(ws, T, n, 1, act, mode, dtype, G0=g0, biases=bs)
    same(make, normal(1, T, I, dtype=td), normal(2, T, I, dtype=td), False)


@pytest.mark.parametrize("mode", [DB, IS])
def test_fp32_layer_on_the_large_tile(mode):
    """Past 4096 small tiles an fp32 step's GEMMs are launches of their own, behind the transfers'."""
    T, I, O, n = 2100, 256, 2100, 2
    make = lambda: RtpLinear(normal(1, O, I) * 0.1, T, n, 1, B.RTP_SPLIT_OUT, mode, B.RTP_F32, G0=normal(2, O, I))
    same(make, normal(3, T, I), normal(4, T, O), True)


@pytest.mark.parametrize("mode", [DB, IS])
@pytest.mark.parametrize("kind", ["linear", "mlp"])
def test_timing_aids_keep_the_schedule(kind, mode):
    """Compute alone (no rotation) rides like the pass it stands for, moves nothing within the pass and gives what the streams
    give without rotation; transfers alone leave the store as it is; timed forward launches are those of the pass."""
    T, n, rank, I, O = 96, 4, 1, 128, 384
    X, dY = normal(1, T, I, dtype=torch.bfloat16), normal(2, T, O if kind == "linear" else I, dtype=torch.bfloat16)
    W, W2, g0, g2 = normal(3, O, I) * 0.1, normal(4, I, O) * 0.1, normal(5, O, I), normal(6, I, O)
    runs = []
    for streams in (False, True):
        if kind == "linear":
            layer = RtpLinear(W, T, n, rank, B.RTP_SPLIT_OUT, mode, G0=g0)
            ring = layer.ring.handle
        else:
            layer = RtpMlp([W, W2], T, n, rank, B.RTP_ACT_GELU_ERF, mode, G0=[g0, g2])
            ring = B.lib.rtp_mlp_ring(layer.handle)
        scratch = torch.zeros(2, dtype=torch.int64, device=DEV)
        B.check(B.lib.rtp_ring_set_test_delay_compute(ring, B._ptr(scratch), 1 if streams else 0), "delay")
        count = lambda: B.lib.rtp_ring_trace(ring, None, 0, 1)
        Y, dX = torch.empty_like(dY), torch.empty_like(X)
        torch.cuda.synchronize()
        B.rtp_prof_begin()
        layer.forward(X, Y)
        layer.sync()
        launches = B.rtp_prof_end()["nt"][0]
        assert launches == (n if kind == "linear" else n + 1)
        home = layer.home_w.clone(), layer.home_g.clone()
        layer.set_ablation(rotate=True, compute=False)
        for _ in range(2):
            layer.forward(X, Y)
            assert B.lib.rtp_ring_rides(ring) == (not streams)
            layer.backward(X, dY, dX)
            assert B.lib.rtp_ring_rides(ring) == (not streams)
        layer.sync()
        assert torch.equal(home[0], layer.home_w) and torch.equal(home[1], layer.home_g)
        layer.set_ablation(rotate=False, compute=True)
        count()
        layer.forward(X, Y)
        assert B.lib.rtp_ring_rides(ring) == (not streams)
        forward = count()
        layer.backward(X, dY, dX)
        assert B.lib.rtp_ring_rides(ring) == (not streams)
        layer.sync()
        records = forward, count()
        held = [t.clone() for t in layer.buf_g[:1]]
        runs.append(([Y, dX, layer.home_w.clone(), layer.home_g.clone()] + held, records))
        layer.close()
    assert runs[0][1] == runs[1][1] and runs[0][1][0] == n + 1, "n computes and the own shard's load"
    for i, (x, y) in enumerate(zip(runs[0][0], runs[1][0])):
        assert torch.equal(x, y), i


@pytest.mark.parametrize("mode", [DB, IS])
@pytest.mark.parametrize("dtype", [B.RTP_BF16, B.RTP_F16])
@pytest.mark.parametrize("kind", ["out", "in", "mlp"])
def test_outputs_off_a_16_byte_boundary(kind, dtype, mode):
    """No four-wide epilogue: a backward step's two layouts are two launches, the transfers in the first, the bias sums in the
    second."""
    td, T, n, rank = TD[dtype], 96, 4, 2
    I, O = (128, 96 * n) if kind != "in" else (96 * n, 128)
    X, W, b = normal(1, T, I, dtype=td), normal(3, O, I) * 0.1, normal(4, O)
    if kind != "mlp":
        make = lambda: RtpLinear(W, T, n, rank, B.RTP_SPLIT_OUT if kind == "out" else B.RTP_SPLIT_IN, mode, dtype, G0=normal(5, O, I), bias=b)
        same(make, X, normal(2, T, O, dtype=td), True, shift=True)
        return
    make = lambda: RtpMlp([W, normal(6, I, O) * 0.1], T, n, rank, B.RTP_ACT_GELU_TANH, mode, dtype, biases=[b, normal(7, I)])
    same(make, X, normal(2, T, I, dtype=td), False, shift=True)


@pytest.mark.parametrize("mode", [DB, IS])
@pytest.mark.parametrize("kind", ["linear", "mlp"])
def test_gradients_whose_sum_is_split_along_k_travel_by_copy(kind, mode):
    """A split sum is added onto the buffer and sent from there by the next launches: integers, so that any order of the
    sum gives the same bits."""
    T, n, rank = 4096, 4, 1
    X, dY = [torch.randint(-2, 3, (T, 256), generator=torch.Generator().manual_seed(s)).to(DEV, torch.bfloat16) for s in (1, 2)]
    W = torch.randint(-1, 2, (256, 256), generator=torch.Generator().manual_seed(3)).float()
    if kind == "linear":
        make = lambda: RtpLinear(W, T, n, rank, B.RTP_SPLIT_OUT, mode, G0=torch.ones(256, 256, device=DEV))
        same(make, X, dY, True)
        return
    W1, W2 = W.repeat(2, 1), torch.zeros(256, 512)
    W2[torch.arange(256), torch.arange(256) * 2] = 1.0
    outs = []
    for streams in (False, True):                # the activation's values are no integers: the sums agree to fp32 rounding
        layer = RtpMlp([W1, W2], T, n, rank, B.RTP_ACT_GELU_ERF, mode)
        outs.append(passes(layer, B.lib.rtp_mlp_ring(layer.handle), X, dY, False, streams, ("fb", "fb"))[0][:-2])
        layer.close()
    for x, y in zip(*outs):                      # 4 x sqrt(4096) roundings of 2^-24 of the sum's size
        assert (x.double() - y.double()).norm() <= 2e-5 * y.double().norm()


@pytest.mark.parametrize("mode", [DB, IS])
def test_two_layers_on_one_ring_and_a_bare_ring(mode):
    """Two layers share the ring's rotations: the transfers ride in the launch of the first; a ring without layers moves
    them on its stage stream."""
    T, I, O, n, rank = 64, 64, 96, 4, 2
    for streams in (False, True):
        wb, gb = 2 * (O // n) * I * 2, 2 * (O // n) * I * 4
        home_w, home_g = normal(1, n, wb // 2, dtype=torch.bfloat16).view(torch.uint8), torch.zeros(n, gb, dtype=torch.uint8, device=DEV)
        bufs = [torch.full((s,), 255, dtype=torch.uint8, device=DEV) for s in (wb, wb, gb, gb)]
        cs, ss, aux = (torch.cuda.Stream() for _ in range(3))
        ring = B.Ring(n, rank, mode, wb, gb, home_w, home_g, bufs[:2], bufs[2:], cs, ss, aux_stream=aux)
        acc = [torch.empty(T, I, device=DEV) for _ in range(2)]
        lins = [B.Linear(ring, T, I, O, B.RTP_SPLIT_OUT, B.RTP_BF16, B.RTP_ACT_NONE, i * wb // 2, i * gb // 2, None, acc[i]) for i in range(2)]
        X, dY = normal(2, T, I, dtype=torch.bfloat16), normal(3, T, O, dtype=torch.bfloat16)
        Y, dX = [torch.empty(T, O, device=DEV, dtype=torch.bfloat16) for _ in range(2)], [torch.empty_like(X) for _ in range(2)]
        scratch = torch.zeros(2, dtype=torch.int64, device=DEV)
        B.check(B.lib.rtp_ring_set_test_delay_compute(ring.handle, B._ptr(scratch), 1 if streams else 0), "delay")
        torch.cuda.synchronize()
        ring.begin(B.RTP_PASS_FWD)
        assert ring.rides() == (not streams)
        for t in range(n):
            if t < n - 1:
                ring.rotate_step(B.RTP_CW, t)
            for i in range(2):
                lins[i].fwd(t, X, Y[i])
        ring.end()
        ring.begin(B.RTP_PASS_BWD)
        assert ring.rides() == (not streams)
        for t in range(n):
            if t < n - 1:
                ring.rotate_step(B.RTP_CCW, t)
            if t < n - 2:
                for i in (1, 0):
                    lins[i].bwd(t, X, dY, dX[i])
        for i in range(2):                       # at the end of a pass one layer may run a step ahead of the other
            for t in (n - 2, n - 1):
                lins[i].bwd(t, X, dY, dX[i])
        ring.end()
        ring.flush()
        ring.sync()
        got = [t.clone() for t in Y + dX + [home_w, home_g]]
        if streams:
            for x, y in zip(got, want):
                assert torch.equal(x, y)
        want = got
        for l in lins:
            l.close()
        ring.close()
    W = normal(1, n, 256).view(torch.uint8)
    bufs = [torch.full((1024,), 255, dtype=torch.uint8, device=DEV) for _ in range(2)]
    ring = B.Ring(n, rank, DB, 1024, 0, W, None, bufs, (None, None), cs, ss, aux_stream=aux)
    keep = W.clone()
    torch.cuda.synchronize()
    ring.begin(B.RTP_PASS_FWD)
    assert not ring.rides()                      # its transfers run beside what the caller enqueues on the compute stream
    for t in range(n - 1):
        ring.rotate_step(B.RTP_CW, t)
    ring.end()
    ring.sync()
    assert torch.equal(W, keep) and torch.equal(bufs[(n - 1) & 1], W[(rank + 1) % n]) and torch.equal(bufs[n & 1], W[(rank + 2) % n])
    ring.close()


@pytest.mark.parametrize("mode", [DB, IS])
def test_sync_covers_a_rotation_without_its_linear_call(mode):
    """rtp_ring_sync between rtp_rotate_step and the step's linear call: the next shard is in the worker's buffer."""
    T, I, O, n, rank = 32, 64, 96, 3, 1
    layer = RtpLinear(normal(1, O, I), T, n, rank, mode=mode, G0=normal(2, O, I))
    X, dY = normal(3, T, I, dtype=torch.bfloat16), normal(4, T, O, dtype=torch.bfloat16)
    Y, dX = torch.empty_like(dY), torch.empty_like(X)
    torch.cuda.synchronize()
    for pass_, turn, shard in ((B.RTP_PASS_FWD, B.RTP_CW, B.rtp_fwd_shard), (B.RTP_PASS_BWD, B.RTP_CCW, B.rtp_bwd_shard)):
        layer.ring.begin(pass_)
        assert layer.ring.rides()
        for t in range(n):
            if t < n - 1:
                layer.ring.rotate_step(turn, t)
                layer.ring.sync()
                dst = [r[4] for r in layer.ring.trace() if r[0] == "w_in"][-1]
                assert torch.equal(layer.buf_w[dst], layer.home_w[shard(rank, t + 1, n)]), (pass_, t)
            layer.lin.fwd(t, X, Y) if pass_ == B.RTP_PASS_FWD else layer.lin.bwd(t, X, dY, dX)
        layer.ring.end()
    layer.sync()
    layer.close()


@pytest.mark.parametrize("n,offsets", [(2, (0, 0)), (4, (0, 0)), (4, (0, 512, 0)), (3, (1536, 0, 512, 1024)),
                                       (4, (256, 1536, 2816, 4096))])   # (gaps: more segments than one launch takes)
def test_layers_of_one_ring_and_the_gradient_bytes_between_and_under_them(n, offsets):
    """fp32 layers on one ring whose parts of a slot overlap (a tied weight) or leave gaps: every byte is sent, and overwritten
    by the next shard's, once.  Integers, so that every order of a sum gives the same bits."""
    T, I, o, rank = 32, 32, 8, 1
    part = o * I * 4                                    # bytes of a layer's part; offsets of half a part overlap
    slot = max(offsets) + part + 256                    # a tail that no layer owns
    draw = lambda seed, *s: torch.randint(-2, 3, s, generator=torch.Generator().manual_seed(seed)).to(DEV, torch.float32)
    X, dY = draw(1, T, I), [draw(2 + i, T, o * n) for i in range(len(offsets))]
    got = []
    for streams in (False, True):
        home_w, home_g = draw(9, n, slot // 4).view(torch.uint8), draw(10, n, slot // 4).view(torch.uint8)
        bufs = [torch.full((slot,), 255, dtype=torch.uint8, device=DEV) for _ in range(4)]
        cs, ss, aux = (torch.cuda.Stream() for _ in range(3))
        ring = B.Ring(n, rank, DB, slot, slot, home_w, home_g, bufs[:2], bufs[2:], cs, ss, aux_stream=aux)
        lins = [B.Linear(ring, T, I, o * n, B.RTP_SPLIT_OUT, B.RTP_F32, B.RTP_ACT_NONE, at, at) for at in offsets]
        scratch = torch.zeros(2, dtype=torch.int64, device=DEV)
        B.check(B.lib.rtp_ring_set_test_delay_compute(ring.handle, B._ptr(scratch), 1 if streams else 0), "delay")
        Y, dX = torch.empty(T, o * n, device=DEV), [torch.empty_like(X) for _ in offsets]
        torch.cuda.synchronize()
        for _ in range(2):
            ring.begin(B.RTP_PASS_FWD)
            for t in range(n):
                if t < n - 1:
                    ring.rotate_step(B.RTP_CW, t)
                for l in lins:
                    l.fwd(t, X, Y)
            ring.end()
            ring.begin(B.RTP_PASS_BWD)
            assert ring.rides() == (not streams)
            for t in range(n):
                if t < n - 1:
                    ring.rotate_step(B.RTP_CCW, t)
                for l, d, dx in zip(lins, dY, dX):
                    l.bwd(t, X, d, dx)
            ring.end()
        ring.flush()
        ring.sync()
        got.append([home_g.view(torch.float32).clone()] + [d.clone() for d in dX])
        ring.close()
    want = draw(10, n, slot // 4).double()
    for at, d in zip(offsets, dY):
        for k in range(n):
            g = d[:, k * o:(k + 1) * o].double().T @ X.double()
            want[k, at // 4:(at + part) // 4] += 2 * g.flatten()
    assert torch.equal(got[0][0].double(), want)
    for x, y in zip(*got):
        assert torch.equal(x, y)


@pytest.mark.parametrize("timed", [False, True])
@pytest.mark.parametrize("mode", [DB, IS])
@pytest.mark.parametrize("split,T,n,bias", [(B.RTP_SPLIT_OUT, 75, 3, True), (B.RTP_SPLIT_IN, 75, 4, True),
                                            (B.RTP_SPLIT_OUT, 4096, 4, False)])   # (the last: sums split along K, sent by copy)
def test_a_refused_call_can_be_made_again(split, T, n, bias, mode, timed):
    """A call that is refused for an operand's alignment leaves the step's transfers to the call that follows it."""
    g = torch.Generator().manual_seed(1)
    draw = lambda *s: torch.randint(-2, 3, s, generator=g).to(DEV, torch.bfloat16)   # any order of a sum gives the same bits
    I = O = 256 if T > 75 else 48 * n
    X, dY, W, g0 = draw(T, I), draw(T, O), draw(O, I).float(), draw(O, I).float()
    b = draw(O).float() if bias else None
    bad_X, bad_dY = off_by_one(X), off_by_one(dY)
    runs = []
    for disturb in (False, True):
        layer = RtpLinear(W, T, n, 1, split, mode, G0=g0, bias=b)
        for t in layer.buf_w + layer.buf_g:
            if t is not None:
                t.fill_(255)
        Y, dX = torch.empty_like(dY), torch.empty_like(X)
        torch.cuda.synchronize()
        if timed:
            B.rtp_prof_begin()

        def call(f, *bad_then_good):
            for args in bad_then_good[:-1] if disturb else ():
                with pytest.raises(B.RtpError) as e:
                    f(*args)
                assert e.value.status == B.RTP_ERR_HIP
            f(*bad_then_good[-1])

        for i in range(2):
            layer.ring.begin(B.RTP_PASS_FWD)
            for t in range(n):
                if t < n - 1:
                    layer.ring.rotate_step(B.RTP_CW, t)
                call(layer.lin.fwd, (t, bad_X, Y), (t, X, Y))
            layer.ring.end()
            layer.ring.begin(B.RTP_PASS_BWD)
            assert layer.ring.rides()
            for t in range(n):
                if t < n - 1:
                    layer.ring.rotate_step(B.RTP_CCW, t)
                call(layer.lin.bwd, (t, bad_X, dY, dX), (t, X, bad_dY, dX), (t, X, dY, dX))
            layer.ring.end()
        layer.ring.flush()
        layer.sync()
        if timed:
            B.rtp_prof_end()
        runs.append([Y, dX, layer.home_w.clone(), layer.home_g.clone()])
        layer.close()
    for i, (x, y) in enumerate(zip(*runs)):
        assert torch.equal(x, y), i


class Seg(C.Structure):
    _fields_ = [("out", C.c_void_p), ("buf", C.c_void_p), ("src", C.c_void_p), ("bytes", C.c_size_t)]


class Riders(C.Structure):
    _fields_ = [("count", C.c_int), ("sums", C.c_int), ("seg", Seg * 8), ("sum", C.c_uint64 * 12)]


def test_segments_of_every_kind_and_size():
    """out <- buf <- in, with either end missing, from one unit to past a workgroup's 64 KB; nothing beyond them is touched."""
    launch = getattr(B.lib, "_ZN3rtp13launch_ridersERKNS_6RidersEP12ihipStream_t")
    launch.restype, launch.argtypes = C.c_int, [C.POINTER(Riders), C.c_void_p]
    for units in (1, 255, 1023, 1024, 1025, 4095, 4096, 4097, 70001):
        for count in (1, 3, 8):
            r, state = Riders(), []
            r.count = count
            for i in range(count):
                out, buf, src = (torch.randint(0, 2 ** 31, (units * 4 + 8,), dtype=torch.int32, device=DEV) for _ in range(3))
                kind = i % 3
                r.seg[i] = Seg(out.data_ptr() + 16 if kind != 1 else None, buf.data_ptr() + 16, src.data_ptr() + 16 if kind != 2 else None, units * 16)
                state.append((kind, out, buf, src, out.clone(), buf.clone(), src.clone()))
            torch.cuda.synchronize()
            assert launch(C.byref(r), torch.cuda.current_stream().cuda_stream) == 0
            torch.cuda.synchronize()
            for kind, out, buf, src, o0, b0, s0 in state:
                if kind != 1:
                    o0[4:-4] = b0[4:-4]
                if kind != 2:
                    b0[4:-4] = s0[4:-4]
                assert torch.equal(out, o0) and torch.equal(buf, b0) and torch.equal(src, s0), (units, count, kind)
    r.seg[0].bytes = 8                            # not whole units: refused
    assert launch(C.byref(r), torch.cuda.current_stream().cuda_stream) != 0
