"""GPU attention forward vs the CPU oracle fed the GPU's own codes.

Tolerance (attention output, bf16 vs bf16): rel-L2 <= 2e-3 and max-abs <= 1e-2.
The oracle mirrors the kernel's KV tile width and fp32 rounding points; the
remaining differences are v_exp_f32's faithful (not always correctly rounded)
exponential, which can move an element of P~ across an E2M1 decision
threshold, and fp32 vs fp64 accumulation.
"""
import ctypes

import numpy as np
import pytest

import oracle
from parity import (MAX_ABS_TOL, REL_L2_TOL, bf16_ties, flat, full_size_sample, log, max_abs,
                    oracle_rows, rel_l2, sample_rows, workload_bits)
from paper_2607_24377_amd import inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
MODES = ["ocp_vanilla", "uos", "uos_pnq"]


@pytest.fixture(scope="module")
def mx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2607_24377_amd import mxattn

    mxattn.lib()
    return mxattn


def _gpu_codes(mx, qt, kt, vt, mode):
    qc, qs = mx.quantize(qt, mx.AXIS_HEAD_DIM, mode)
    kc, ks = mx.quantize(kt, mx.AXIS_HEAD_DIM, mode)
    vc, vs = mx.quantize(vt, mx.AXIS_TOKENS, mode)
    return {n: flat(t.cpu().numpy()) for n, t in
            dict(qc=qc, qs=qs, kc=kc, ks=ks, vc=vc, vs=vs).items()}


def _check_rows(mx, q, k, v, mode, heads_rows, N, label):
    """Run the forward on the GPU and compare the given (head, rows) with the oracle."""
    qt, kt, vt = (mx.bf16_from_bits(x) for x in (q, k, v))
    out = mx.forward(qt, kt, vt, mode)
    torch.cuda.synchronize()
    codes = _gpu_codes(mx, qt, kt, vt, mode)
    got_all = flat(mx.bits_from_bf16(out))
    bc = mx.kv_tile()
    worst = (0.0, 0.0)
    gots, refs = [], []
    for head, rows in heads_rows:
        ref, _ = oracle_rows(codes, head, N, rows, mode, bc)
        got = oracle.bf16_to_f64(got_all[head][rows])
        gots.append(got)
        refs.append(ref)
        worst = (max(worst[0], rel_l2(got, ref)), max(worst[1], max_abs(got, ref)))
    g = np.concatenate(gots)
    r = np.concatenate(refs)
    rl, ma = rel_l2(g, r), max_abs(g, r)
    log(f"[attn] {label} mode={mode}: rel-L2 {rl:.3e} max-abs {ma:.3e} (worst head {worst[0]:.3e})")
    assert np.all(np.isfinite(g))
    assert rl <= REL_L2_TOL, (label, mode, rl)
    assert ma <= MAX_ABS_TOL, (label, mode, ma)
    return out


@pytest.mark.parametrize("mode", MODES)
def test_tiny_all_rows(mx, mode):
    w = inputs.workload(0)
    q, k, v = workload_bits(0)
    hr = [(h, np.arange(w.N)) for h in range(w.B * w.H)]
    _check_rows(mx, q, k, v, mode, hr, w.N, w.name)


@pytest.mark.parametrize("mode", MODES)
def test_outlier_channels_sampled(mx, mode):
    w = inputs.workload(1)
    q, k, v = workload_bits(1)
    heads = [0, 7, 19, 39]
    hr = [(h, sample_rows(w.N, 48, 100 + h)) for h in heads]
    _check_rows(mx, q, k, v, mode, hr, w.N, w.name)


@pytest.mark.parametrize("mode", MODES + ["uos_pnq_rot"])
@pytest.mark.parametrize("cfg", [1, 2, 3, 4])
def test_full_size_stratified_rows(mx, cfg, mode):
    """Full-size workloads in the launch the benchmark times, every mode, with
    the oracle on >= 2048 stratified rows spread over every head (first and
    ragged last query tile, the joint workload's text rows, random rows).
    Each head, and the sample as a whole, must meet the tolerance; an element
    whose oracle value sits at a bf16 rounding midpoint may take either
    neighbouring bf16 value (bf16_ties).  The log
    gives the worst deviation and the oracle's audit of the exponential:
    P~ elements within 4 ulps of an E2M1 decision threshold and blocks whose
    maximum is within 4 ulps of a scale boundary, the only places where the
    GPU's faithful exp2 can choose another code than the correctly rounded
    one."""
    w = inputs.workload(cfg)
    smp = full_size_sample(cfg, mode)
    g, r, hd = smp["got"], smp["ref"], smp["head_of"]
    assert np.all(np.isfinite(g))
    # elements at a bf16 rounding midpoint (two valid roundings) are checked
    # to be one of them; every other element is held to max-abs
    ties = bf16_ties(g, r, smp["ref64"])
    err = np.where(ties, 0.0, np.abs(g - r))
    rl, ma = rel_l2(g, r), float(err.max())
    per_head = [rel_l2(g[hd == h], r[hd == h]) for h in range(w.B * w.H)]
    worst_row = int(np.argmax(err.max(axis=1)))
    near_el, near_blk = smp["diag"][:, 6].sum(), smp["diag"][:, 7].sum()
    log(f"[full] {w.name} mode={mode}: rows {g.shape[0]} over {w.B * w.H} heads, rel-L2 {rl:.3e}, "
        f"max-abs {ma:.3e} (head {hd[worst_row]}), worst head rel-L2 {max(per_head):.3e}; "
        f"{int((g != r).sum())} elements differ from the oracle's bf16, {int(ties.sum())} of them "
        f"rounding ties of fp32 vs fp64 (largest {np.abs(g - r)[ties].max() if ties.any() else 0:.3e}); "
        f"audit: {near_el:.0f} P~ near a threshold, {near_blk:.0f} blocks near a scale boundary")
    for i, j in np.argwhere(ties)[:8]:
        x = smp["ref64"][i, j]
        log(f"[full]   tie: head {hd[i]} ch {j}: gpu {g[i, j]:.7g} oracle bf16 {r[i, j]:.7g} oracle fp64 "
            f"{x:.12g}, {abs(x - (g[i, j] + r[i, j]) / 2) / abs(x):.2e} from the midpoint")
    assert rl <= REL_L2_TOL, (w.name, mode, rl)
    assert ma <= MAX_ABS_TOL, (w.name, mode, ma)
    assert max(per_head) <= REL_L2_TOL, (w.name, mode, int(np.argmax(per_head)), max(per_head))
    torch.cuda.empty_cache()


@pytest.mark.parametrize("N", [1, 2, 31, 32, 33, 64, 127, 128, 129, 200, 255, 257, 640, 1001])
def test_ragged_lengths(mx, N):
    w = inputs.custom(2, 3, N, kind="video", index=50 + N % 7)
    q, k, v = inputs.generate(w)
    hr = [(h, np.arange(N)) for h in range(6)]
    for mode in MODES:
        _check_rows(mx, q, k, v, mode, hr, N, f"ragged N={N}")


def test_v_all_ones(mx):
    """V = 1 gives V^ = 1 exactly; PNQ returns exactly 1.0 and the direct modes
    return the induced row sums (Eq. pnq_direct_full_rowsum)."""
    w = inputs.custom(1, 2, 700, kind="iid", index=61)
    q, k, _ = inputs.generate(w)
    v = np.full_like(q, 0x3F80)  # bf16 1.0
    qt, kt, vt = (mx.bf16_from_bits(x) for x in (q, k, v))
    for mode in MODES:
        out = mx.bits_from_bf16(mx.forward(qt, kt, vt, mode))
        if mode == "uos_pnq":
            assert np.all(out == 0x3F80)
        else:
            codes = _gpu_codes(mx, qt, kt, vt, mode)
            for hd in range(2):
                rows = np.arange(0, 700, 7)
                ref, _, dg = oracle_rows(codes, hd, 700, rows, mode, mx.kv_tile(), diag=True)
                got = oracle.bf16_to_f64(flat(out)[hd][rows])
                np.testing.assert_allclose(got[:, 0], oracle.bf16_to_f64(oracle.round_bf16(dg[:, 1])),
                                           rtol=8e-3)
                assert np.mean(dg[:, 1]) < 1.0


def test_identical_keys(mx):
    """Identical keys make every P~ equal to 1 (up to ulps above 1), so P^ = 1
    and O is the mean of the V^ rows in every mode."""
    w = inputs.custom(1, 1, 300, kind="iid", index=62)
    q, k, v = inputs.generate(w)
    k[:] = k[:, :, :1, :]
    qt, kt, vt = (mx.bf16_from_bits(x) for x in (q, k, v))
    for mode in MODES:
        out = oracle.bf16_to_f64(mx.bits_from_bf16(mx.forward(qt, kt, vt, mode)))[0, 0]
        vc, vs = mx.quantize(vt, mx.AXIS_TOKENS, mode)
        vh = oracle.dequant_keys(vc.cpu().numpy()[0, 0], vs.cpu().numpy()[0, 0], 300)
        want = oracle.bf16_to_f64(oracle.round_bf16(vh.mean(0)))
        assert max_abs(out, np.broadcast_to(want, out.shape)) <= 1e-2
        assert rel_l2(out, np.broadcast_to(want, out.shape)) <= 4e-3


def test_attend_matches_forward_and_is_deterministic(mx):
    w = inputs.custom(2, 2, 1000, kind="video", index=63)
    q, k, v = inputs.generate(w)
    qt, kt, vt = (mx.bf16_from_bits(x) for x in (q, k, v))
    for mode in MODES:
        a = mx.forward(qt, kt, vt, mode)
        torch.cuda.synchronize()
        mx.release_workspace()  # the next call takes fresh workspace from the library's pool
        b = mx.forward(qt, kt, vt, mode)
        qc, qs = mx.quantize(qt, mx.AXIS_HEAD_DIM, mode)
        kc, ks = mx.quantize(kt, mx.AXIS_HEAD_DIM, mode)
        vc, vs = mx.quantize(vt, mx.AXIS_TOKENS, mode)
        c = mx.attend(qc, qs, kc, ks, vc, vs, 1000, mode)
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
        assert torch.equal(a.view(torch.int16), c.view(torch.int16))


@pytest.mark.parametrize("Nq,Nkv", [(1, 1), (129, 127), (127, 129), (300, 513), (33, 1025)])
def test_forward_operands_equal_the_public_ones(mx, Nq, Nkv):
    """The forward quantizes K and V (and the rotated mode's Q) in one launch,
    tile by tile and with the scales in operand order; its output must equal
    the kernel run on the standalone quantizers' codes, bit for bit, with
    ragged and whole last tiles, several heads and all modes."""
    q = inputs.generate(inputs.custom(2, 3, Nq, kind="video", index=73))[0]
    _, k, v = inputs.generate(inputs.custom(2, 3, Nkv, kind="video", index=74))
    k[:, :, 0, :32] = 0  # an all-zero block of K and of V
    v[:, :, : min(32, Nkv), 5] = 0
    qt, kt, vt = (mx.bf16_from_bits(x) for x in (q, k, v))
    for mode in MODES + ["uos_pnq_rot"]:
        a = mx.cross_forward(qt, kt, vt, mode)
        qc, qs = mx.quantize(qt, mx.AXIS_HEAD_DIM, mode)
        kc, ks = mx.quantize(kt, mx.AXIS_HEAD_DIM, mode)
        vc, vs = mx.quantize(vt, mx.AXIS_TOKENS, mode)
        b = mx.cross_attend(qc, qs, kc, ks, vc, vs, Nq, Nkv, mode)
        torch.cuda.synchronize()
        log(f"[attn] forward operands Nq={Nq} Nkv={Nkv} mode={mode}")
        assert torch.equal(a.view(torch.int16), b.view(torch.int16)), (Nq, Nkv, mode)


@pytest.mark.parametrize("Nq,Nkv", [(1, 1), (7, 33), (16, 16), (50, 64), (3, 65), (31, 96), (5, 97), (2, 127)])
def test_many_short_heads(mx, Nq, Nkv):
    """300 heads shorter than a tile: the rotated mode's Q is prepared in tiles that
    run on over the heads, K and V in one tile per head; as above, the output
    equals the one on the standalone quantizers' codes bit for bit."""
    g = torch.Generator(device="cuda").manual_seed(100 * Nq + Nkv)
    q, k, v = (torch.randn((2, 150, n, 128), generator=g, device="cuda").bfloat16() for n in (Nq, Nkv, Nkv))
    for mode in MODES + ["uos_pnq_rot"]:
        a = mx.cross_forward(q, k, v, mode)
        qc, qs = mx.quantize(q, mx.AXIS_HEAD_DIM, mode)
        kc, ks = mx.quantize(k, mx.AXIS_HEAD_DIM, mode)
        vc, vs = mx.quantize(v, mx.AXIS_TOKENS, mode)
        b = mx.cross_attend(qc, qs, kc, ks, vc, vs, Nq, Nkv, mode)
        assert torch.equal(a.view(torch.int16), b.view(torch.int16)), (Nq, Nkv, mode)


def test_workspace_of_short_heads(mx):
    """65536 heads of one key: K^ and V^ of one block and 1 KiB of scales per head
    (206 MB in all), not a whole tile of V^ codes (8 KiB instead of 2)."""
    x = torch.ones((1, 65536, 1, 128), dtype=torch.bfloat16, device="cuda")
    out = torch.empty_like(x)
    torch.cuda.synchronize()
    mx.release_workspace()
    free = torch.cuda.mem_get_info()[0]
    mx.forward(x, x, x, "uos", out=out)
    torch.cuda.synchronize()
    taken = free - torch.cuda.mem_get_info()[0]
    mx.release_workspace()
    assert torch.all(out == 1)
    assert taken <= 65536 * (64 + 128 * 16 + 1024) + (32 << 20), taken  # and the pool's granularity


def test_workspace_across_streams_and_threads(mx):
    """Calls on the null stream share one kept block of workspace, those on
    other streams and of a second thread at the same time do not: every output
    equals the one computed alone, with sizes that grow the block, after it was
    given back, and beyond its limit."""
    import threading

    shapes = [(1, 2, 300), (2, 3, 1000), (1, 1, 40), (1, 8, 4000), (1, 40, 16000)]  # the last takes 87 MB
    data = []
    for i, (B, H, N) in enumerate(shapes):
        g = torch.Generator(device="cuda").manual_seed(i)
        t = [torch.randn((B, H, N, 128), generator=g, device="cuda").bfloat16() for _ in range(3)]
        data.append(t + [mx.forward(*t, "uos_pnq")])
    torch.cuda.synchronize()
    mx.release_workspace()
    bad = []

    def work(stream, order):
        for i in order:
            q, k, v, want = data[i]
            with torch.cuda.stream(stream):
                out = mx.forward(q, k, v, "uos_pnq")
                same = torch.equal(out.view(torch.int16), want.view(torch.int16))
            if not same:
                bad.append((stream, i))

    null, side = torch.cuda.default_stream(), torch.cuda.Stream()
    orders = ([0, 3, 1, 2, 4, 0, 1], [2, 1, 0, 3, 1, 4, 2], [1, 0, 2, 3, 0, 2, 1])
    threads = [threading.Thread(target=work, args=a) for a in zip((null, null, side), orders)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    mx.release_workspace()
    work(null, [0, 2])
    torch.cuda.synchronize()
    assert not bad, bad


def test_kept_block_is_reused_without_waiting(mx):
    """Calls enqueued one after another on the null stream, with no synchronization
    until the end, overwrite the kept block while earlier ones still run: sizes that
    grow it on the way, quantized operands and the sweep's partial sums beside the
    forward's, and calls of two threads and of another stream at the same time."""
    import threading

    shapes = [(1, 2, 300), (2, 3, 1000), (1, 1, 40), (1, 8, 4000), (1, 4, 2000), (1, 20, 3000)]
    data = []
    for i, (B, H, N) in enumerate(shapes):
        g = torch.Generator(device="cuda").manual_seed(50 + i)
        t = [torch.randn((B, H, N, 128), generator=g, device="cuda").bfloat16() for _ in range(3)]
        ops = [x for n, ax in zip(t, (mx.AXIS_HEAD_DIM, mx.AXIS_HEAD_DIM, mx.AXIS_TOKENS)) for x in mx.quantize(n, ax, "uos_pnq")]
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):  # pool memory of the call's own
            want = mx.forward(*t, "uos_pnq")
            sse = mx.qmax_sse(t[0], mx.AXIS_TOKENS, [6.0, 7.25])
        side.synchronize()
        data.append((t, ops, want, sse))
    mx.release_workspace()
    results = []

    def work(stream, order, outs):
        with torch.cuda.stream(stream):
            for n, i in enumerate(order):
                t, ops, want, sse = data[i]
                if n % 3 == 0:
                    mx.forward(*t, "uos_pnq", out=outs[n])
                elif n % 3 == 1:
                    mx.attend(*ops, t[0].shape[2], "uos_pnq", out=outs[n])
                else:
                    mx.qmax_sse(t[0], mx.AXIS_TOKENS, [6.0, 7.25], out=outs[n])

    rng = np.random.default_rng(8)
    threads = []
    null, side = torch.cuda.default_stream(), torch.cuda.Stream()
    for stream in (null, null, side):
        order = [2, 0, 0, 2, 4, 1] + [int(i) for i in rng.integers(0, len(shapes), 54)]
        outs = [torch.empty_like(data[i][3] if n % 3 == 2 else data[i][2]) for n, i in enumerate(order)]
        results.append((order, outs))
        threads.append(threading.Thread(target=work, args=(stream, order, outs)))
    torch.cuda.synchronize()
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for order, outs in results:
        for n, (i, out) in enumerate(zip(order, outs)):
            if n % 3 == 2:
                torch.testing.assert_close(out, data[i][3], rtol=1e-12, atol=0.0)
            else:
                assert torch.equal(out.view(torch.int16), data[i][2].view(torch.int16)), (n, shapes[i])


def test_release_does_not_wait_for_the_null_stream(mx):
    """A release while calls are under way returns at once; the block that they
    use is given back by a release after they have completed."""
    g = torch.Generator(device="cuda").manual_seed(5)
    q, k, v = (torch.randn((1, 8, 4000, 128), generator=g, device="cuda").bfloat16() for _ in range(3))
    null = torch.cuda.default_stream()
    with torch.cuda.stream(null):
        want = mx.forward(q, k, v, "uos_pnq")
        out = torch.empty_like(want)
        torch.cuda.synchronize()
        for _ in range(200):  # about 10 ms of GPU work, enqueued in 2
            mx.forward(q, k, v, "uos_pnq", out=out)
        done = null.record_event()
        mx.release_workspace()
        assert not done.query()
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), want.view(torch.int16))
        free = torch.cuda.mem_get_info()[0]
        mx.release_workspace()
        assert torch.cuda.mem_get_info()[0] > free
        again = mx.forward(q, k, v, "uos_pnq")
    assert torch.equal(again.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("flags", [1, 0])  # hipStreamNonBlocking, hipStreamDefault
def test_release_beside_a_capture(mx, flags):
    """A release while another stream is captured leaves the capture alone, also
    where that stream synchronizes with the null stream (flags 0)."""
    hip = ctypes.CDLL("libamdhip64.so")
    x = torch.zeros((1, 1, 64, 128), dtype=torch.bfloat16, device="cuda")
    with torch.cuda.stream(torch.cuda.default_stream()):
        mx.forward(x, x, x, "uos_pnq")
    torch.cuda.synchronize()
    stream, graph, status = ctypes.c_void_p(), ctypes.c_void_p(), ctypes.c_int(-1)
    assert hip.hipStreamCreateWithFlags(ctypes.byref(stream), flags) == 0
    try:
        assert hip.hipStreamBeginCapture(stream, 0) == 0
        mx.release_workspace()
        assert hip.hipStreamIsCapturing(stream, ctypes.byref(status)) == 0 and status.value == 1
        assert hip.hipStreamEndCapture(stream, ctypes.byref(graph)) == 0
        assert hip.hipGraphDestroy(graph) == 0
    finally:
        hip.hipStreamDestroy(stream)
    mx.release_workspace()
    with torch.cuda.stream(torch.cuda.default_stream()):
        out = mx.forward(x, x, x, "uos_pnq")
    assert torch.count_nonzero(out) == 0


def _edge_q_rows(q):
    """Overwrite the first query rows of every head with values that exercise
    the quantizer's scale rule: an all-zero block (sigma = 1), bf16
    subnormals, negative zeros, and block maxima exactly on and just past the
    UOS boundary 7.25 * 2^k and the OCP boundary 2^k."""
    q = q.copy()
    f32 = lambda x: (np.float32(x).view(np.uint32) >> 16).astype(np.uint16)
    for bh in range(q.shape[0] * q.shape[1]):
        rows = q.reshape(-1, q.shape[2], q.shape[3])[bh]
        rows[0, :32] = 0
        rows[0, 32:64] = 0x8000  # -0
        rows[1, :] = np.arange(1, 129, dtype=np.uint16)  # bf16 subnormals (exponent field 0)
        rows[2, :] = f32(0.5)
        rows[2, 0] = f32(7.25)        # UOS boundary: M = 7.25 * 2^0
        rows[2, 32] = f32(7.28125)    # next bf16 above it
        rows[2, 64] = f32(4.0)        # OCP boundary 2^2
        rows[2, 96] = f32(-7.96875)   # largest bf16 below 8, negative
    return q


@pytest.mark.parametrize("Nkv", [300, 1000])
def test_in_kernel_q_quantization_is_bit_exact(mx, Nkv):
    """The forward quantizes Q inside the attention kernel (unrotated modes);
    its output must equal the same kernel run on Q^ from the standalone
    quantizer, bit for bit, on the resident (Nkv <= 512) and streaming paths."""
    Nq = 300
    wq = inputs.custom(2, 2, Nq, kind="video", index=71)
    wk = inputs.custom(2, 2, Nkv, kind="video", index=72)
    q = _edge_q_rows(inputs.generate(wq)[0])
    _, k, v = inputs.generate(wk)
    qt, kt, vt = (mx.bf16_from_bits(x) for x in (q, k, v))
    for mode in MODES:
        a = mx.cross_forward(qt, kt, vt, mode)
        qc, qs = mx.quantize(qt, mx.AXIS_HEAD_DIM, mode)
        kc, ks = mx.quantize(kt, mx.AXIS_HEAD_DIM, mode)
        vc, vs = mx.quantize(vt, mx.AXIS_TOKENS, mode)
        b = mx.cross_attend(qc, qs, kc, ks, vc, vs, Nq, Nkv, mode)
        torch.cuda.synchronize()
        log(f"[attn] in-kernel Q quantization Nkv={Nkv} mode={mode}")
        assert torch.equal(a.view(torch.int16), b.view(torch.int16)), (Nkv, mode)


def test_error_paths_leave_stream_usable(mx):
    w = inputs.custom(1, 1, 64, kind="iid", index=64)
    q, k, v = inputs.generate(w)
    qt, kt, vt = (mx.bf16_from_bits(x) for x in (q, k, v))
    L = mx.lib()
    s = torch.cuda.current_stream().cuda_stream
    assert L.mxattn_forward(qt.data_ptr(), kt.data_ptr(), vt.data_ptr(), None, 1, 1, 64, 128, 2, s) == 1
    assert L.mxattn_forward(qt.data_ptr(), kt.data_ptr(), vt.data_ptr(), qt.data_ptr() + 2, 1, 1,
                            64, 128, 2, s) == 3
    assert L.mxattn_quantize(qt.data_ptr(), qt.data_ptr(), qt.data_ptr(), 4, 2, 1, 1, 64, 128, s) == 5
    with pytest.raises(mx.MxattnError):
        mx.forward(qt, kt, vt, 5)
    out = mx.forward(qt, kt, vt, "uos_pnq")
    torch.cuda.synchronize()
    assert torch.isfinite(out.float()).all()
