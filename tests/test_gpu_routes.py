"""GPU parity of the kernels and dispatch branches that tests/test_gpu_parity.py reaches only in part:
each at the sizes where it can go wrong, against the CPU oracle (bars as stated there) or bit-exact."""
import os

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("needs a GPU", allow_module_level=True)

import oracle  # noqa: E402
import rounding_model as RM  # noqa: E402
from paper_1611_09482_amd import binding  # noqa: E402

TOL = {W.F32: 1e-4, W.BF16: 2e-2}


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def row_rel_err(g, o):
    return (np.abs(g - o).max(axis=-1) / np.maximum(np.abs(o).max(axis=-1), 1e-6)).max()


def model(cfg, w, max_batch, **env):
    os.environ.update(env)
    try:
        return binding.from_model(cfg, w, max_batch=max_batch)
    finally:
        for k in env:
            os.environ.pop(k, None)


@pytest.mark.parametrize("n_layers", [6, 7, 8, 9, 10, 11, 13, 14, 15, 16, 17, 31])
def test_split_layer_counts_closed_form(n_layers):
    """The split kernels at every remainder of the six-layer loop (7-layer tails for a remainder of
    1) and past 32 streams' worth of skip registers: bit-exact logits of the rounding-point closed
    form, over a step count that rotates the register rings through every phase."""
    cfg, w = RM.make_model(n_layers)
    T = 9
    want, _ = RM.closed_form(T)
    fw = model(cfg, w, 5)
    assert fw.lib.fwg_waits(fw.handle) == 1
    lg = fw.teacher_forced(dev(W.sequences(6, 5, T))).cpu().numpy()
    assert np.array_equal(lg, np.broadcast_to(want.astype(np.float32), lg.shape))


@pytest.mark.parametrize("width,n_layers,B", [(2, 6, 3), (2, 7, 40), (2, 8, 1), (3, 6, 20), (3, 7, 2),
                                              (3, 8, 9), (2, 9, 1), (2, 10, 37), (2, 13, 130), (2, 20, 5), (3, 9, 17), (3, 12, 1),
                                              (3, 13, 5), (3, 14, 33), (3, 16, 3), (3, 17, 130)])
def test_split_widths_and_ragged_groups(width, n_layers, B):
    """Both widths, odd and even layer counts, ragged group rows (1, 2, 3, 9 groups): teacher forcing
    and online prediction resumed across launches against the oracle on sampled streams; every queue
    wraps.  Generation equals the class drawn from the same prefix's logits in one piece or two."""
    dil = tuple((1, 3, 2, 7, 1, 5)[i % 6] for i in range(n_layers))
    cfg = W.ModelConfig(W.GATED, W.BF16, 64, dil, 512, 512, filter_width=width)
    w = W.make_weights(cfg, 40 + n_layers, bias_scale=0.1)
    fw = model(cfg, w, B)
    assert fw.lib.fwg_waits(fw.handle) == 1
    T = 70
    x = W.sequences(41, B, T)
    sel = sorted({0, B // 2, B - 1})
    want = oracle.Oracle(w).teacher_forced(x[sel])
    lg = fw.teacher_forced(dev(x)).cpu().numpy()
    assert row_rel_err(lg[sel], want) <= TOL[W.BF16]
    # online prediction over x[:, 1:] after a first observed sample: the same logits, bit by bit
    cfg0 = np.full((B, 1), cfg.seed_input, np.int32)
    y = np.concatenate([cfg0, x[:, :-1]], axis=1)
    ref = fw.teacher_forced(dev(y)).cpu().numpy()
    a = fw.step_forced(dev(x[:, :33])).cpu().numpy()
    b = fw.step_forced(dev(x[:, 33:])).cpu().numpy()
    assert np.array_equal(np.concatenate([a, b], axis=1), ref)
    u = W.uniforms(42, B, 40)
    fw.reset()
    g = fw.generate(dev(u)).cpu().numpy()
    fw.reset()
    g1 = fw.generate(dev(u[:, :7])).cpu().numpy()
    g2 = fw.generate(dev(u[:, 7:])).cpu().numpy()
    assert np.array_equal(np.concatenate([g1, g2], axis=1), g)


@pytest.mark.parametrize("n_layers,B", [(12, 11), (14, 20)])
def test_split_graph_replays(n_layers, B):
    """A generation recorded into a graph (queues reset, then generate) gives the eager samples on
    every replay, with eager launches on the same handle between the replays."""
    cfg = W.ModelConfig(W.GATED, W.BF16, 64, tuple(2 ** (i % 5) for i in range(n_layers)), 512, 512)
    w = W.make_weights(cfg, 50, bias_scale=0.1)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        fw = binding.from_model(cfg, w, max_batch=B)
        u = dev(W.uniforms(51, B, 30))
        out = torch.empty((B, 30), dtype=torch.int32, device="cuda")
        want = fw.generate(u).cpu().numpy()
        x = dev(W.sequences(52, B, 20))
        lg = fw.teacher_forced(x).cpu().numpy()
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            fw.reset()
            fw.generate(u, out=out, check=False)
        for _ in range(3):
            out.zero_()
            g.replay()
            s.synchronize()
            assert np.array_equal(out.cpu().numpy(), want)
            assert np.array_equal(fw.teacher_forced(x).cpu().numpy(), lg)
        fw.device_status()


# width, layers, streams of shapes not "mfma_split" by name (400 streams: groups whose blocks sit on several XCDs)
SPLIT_OTHER = [(2, 7, 37), (2, 20, 100), (3, 14, 20), (2, 9, 400)]


def split_other(width, n_layers, B, **env):
    cfg = W.ModelConfig(W.GATED, W.BF16, 64, tuple((1, 3, 2, 7, 1, 5)[i % 6] for i in range(n_layers)), 512, 512,
                        filter_width=width)
    w = W.make_weights(cfg, 45, bias_scale=0.1)
    return cfg, w, model(cfg, w, B, **env)


@pytest.mark.parametrize("width,n_layers,B", SPLIT_OTHER)
@pytest.mark.parametrize("polls", ["-1", "1", "24", "30", "36"])
def test_split_groups_that_give_up(width, n_layers, B, polls):
    """Groups that give up (all of them; about 30 polls are what the blocks of an idle device need, so that then
    some do and some do not) run on the single-block kernel: teacher forcing, online prediction and
    generation over several launches whose groups may change sides, against the oracle and (all of them)
    the single-block kernel's bits."""
    cfg, w, fw = split_other(width, n_layers, B, FWG_SPLIT_POLLS=polls)
    one = model(cfg, w, B, FWG_REGIME="mfma")
    assert fw.lib.fwg_waits(fw.handle) == 1 and one.lib.fwg_waits(one.handle) == 0
    x = W.sequences(46, B, 50)
    want = one.teacher_forced(dev(x))
    sel = [0, B // 2, B - 1]
    assert row_rel_err(want.cpu().numpy()[sel], oracle.Oracle(w).teacher_forced(x[sel])) <= TOL[W.BF16]
    for _ in range(3):
        got = fw.teacher_forced(dev(x))
        assert row_rel_err(got.cpu().numpy(), want.cpu().numpy()) <= TOL[W.BF16]
        assert polls != "-1" or torch.equal(got, want)
    steps, ref = [], one.step_forced(dev(x))
    for a, b in ((0, 1), (1, 2), (2, 17), (17, 50)):
        steps.append(fw.step_forced(dev(x[:, a:b])))
    assert row_rel_err(torch.cat(steps, 1).cpu().numpy(), ref.cpu().numpy()) <= TOL[W.BF16]
    u = dev(W.uniforms(47, B, 30))
    g = fw.generate(u)
    fw.device_status()
    assert int(g.min()) >= 0 and int(g.max()) <= 255
    assert polls != "-1" or torch.equal(g, one.generate(u))


@pytest.mark.parametrize("width,n_layers,B", [(2, 7, 400), (3, 14, 384)])
def test_split_launches_that_share_the_device(width, n_layers, B):
    """Two handles whose launches would each fill the device, on two streams at once, with default
    arguments: valid logits and samples on both, whichever groups find room."""
    cfg, w, ref = split_other(width, n_layers, B)
    x, u = dev(W.sequences(48, B, 120)), dev(W.uniforms(49, B, 120))
    want = ref.teacher_forced(x).cpu().numpy()
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    fws = []
    for s in streams:
        with torch.cuda.stream(s):
            fws.append(binding.from_model(cfg, w, max_batch=B))
    got = []
    for _ in range(4):
        for s, fw in zip(streams, fws):
            with torch.cuda.stream(s):
                got.append((fw.teacher_forced(x), fw.generate(u)))
    torch.cuda.synchronize()
    for fw in fws:
        fw.device_status()
    for lg, g in got:
        assert row_rel_err(lg.cpu().numpy(), want) <= TOL[W.BF16]
        assert int(g.min()) >= 0 and int(g.max()) <= 255


@pytest.mark.parametrize("width,n_layers,B", SPLIT_OTHER)
def test_split_other_layer_counts_return_after_the_enqueue(width, n_layers, B):
    """With default arguments the calls of these shapes do not synchronise: they can be recorded into a graph,
    whose replays give the eager results, with eager calls in between."""
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        cfg, w, fw = split_other(width, n_layers, B)
        x, u = dev(W.sequences(43, B, 20)), dev(W.uniforms(44, B, 20))
        lg, g = torch.empty((B, 20, 256), device="cuda"), torch.empty((B, 20), dtype=torch.int32, device="cuda")
        fw.step_forced(x, out=lg)
        fw.generate(u, out=g)
        want = lg.clone(), g.clone()
        s.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            fw.reset()
            fw.step_forced(x, out=lg)
            fw.generate(u, out=g)
        for _ in range(3):
            lg.zero_()
            g.zero_()
            graph.replay()
            s.synchronize()
            assert torch.equal(lg, want[0]) and torch.equal(g, want[1])
            fw.teacher_forced(x)


@pytest.mark.parametrize("n_layers,B,T,rows", [(2, 1, 40, None), (9, 3, 700, None), (12, 5, 257, None), (10, 17, 300, 64),
                                               (30, 2, 1100, None), (7, 33, 31, 96)])
def test_parallel_stack(n_layers, B, T, rows):
    """The whole-stack kernel: parts of 256 steps, ragged parts and waves, dilations shorter and longer
    than a part, small chunks (queues refreshed between launches).  Teacher forcing against the
    per-layer kernels on every stream and the oracle on one; priming in two pieces leaves the queues
    the step kernels leave (their logits on the following steps)."""
    cfg = W.ModelConfig(W.GATED, W.BF16, 64, tuple((1, 2, 4, 8, 16, 32, 64, 128, 256, 512)[i % 10] for i in range(n_layers)),
                        512, 512)
    w = W.make_weights(cfg, 60, bias_scale=0.1)
    env = {} if rows is None else {"FWG_PAR_ROWS": str(rows * (-(-B // 16) * 16))}
    fw = model(cfg, w, B, FWG_PAR_STACK="1", **env)
    ref = model(cfg, w, B, FWG_PAR_STACK="0", **env)
    x = W.sequences(61, B, T)
    got = fw.teacher_forced_parallel(dev(x)).cpu().numpy()
    assert row_rel_err(got[-1:], oracle.Oracle(w).teacher_forced(x[-1:])) <= TOL[W.BF16]
    assert row_rel_err(got, ref.teacher_forced_parallel(dev(x)).cpu().numpy()) <= TOL[W.BF16]
    h = T // 3 + 1
    a = fw.prime(dev(x[:, :h]), logits=True).cpu().numpy()
    fw.prime(dev(x[:, h:]))
    ra = ref.step_forced(dev(x[:, :h])).cpu().numpy()
    ref.step_forced(dev(x[:, h:]))
    y = dev(W.sequences(62, B, 12))
    assert row_rel_err(a, ra) <= TOL[W.BF16]
    assert row_rel_err(fw.step_forced(y).cpu().numpy(), ref.step_forced(y).cpu().numpy()) <= TOL[W.BF16]


@pytest.mark.parametrize("width", [2, 3])
@pytest.mark.parametrize("B,T", [(1, 1), (1, 63), (5, 13), (3, 43), (1, 129)])
def test_parallel_head_row_tails(B, T, width):
    """The fused head at row counts around its 64-row blocks (1, 63, 65, 129 rows), both widths'
    row producers, against the step kernels on every row."""
    for dtype, R, S in ((W.BF16, 64, 512), (W.F32, 32, 256)):
        cfg = W.ModelConfig(W.GATED, dtype, R, (1, 2, 4, 1, 2, 4, 8, 1, 3), S, S, filter_width=width)
        w = W.make_weights(cfg, 70, bias_scale=0.1)
        fw = model(cfg, w, B, FWG_PAR_HEAD="1")
        x = dev(W.sequences(71, B, T))
        got = fw.teacher_forced_parallel(x).cpu().numpy()
        assert row_rel_err(got, fw.teacher_forced(x).cpu().numpy()) <= TOL[dtype]


def test_parallel_head_large_blocks():
    """Past 16,384 rows a chunk's head runs in 128-row blocks: ragged last block, sampled streams."""
    for dtype, R, S in ((W.BF16, 64, 512), (W.F32, 32, 256)):
        cfg = W.ModelConfig(W.GATED, dtype, R, (1, 2, 4, 8), S, S)
        w = W.make_weights(cfg, 72, bias_scale=0.1)
        B, T = 129, 131
        fw = model(cfg, w, B)
        x = W.sequences(73, B, T)
        got = fw.teacher_forced_parallel(dev(x)).cpu().numpy()
        sel = [0, 64, 128]
        assert row_rel_err(got[sel], oracle.Oracle(w).teacher_forced(x[sel])) <= TOL[dtype]


@pytest.mark.parametrize("dtype,R,S", [(W.BF16, 64, 512), (W.F32, 32, 256)])
def test_parallel_head_element_aligned_arrays(dtype, R, S):
    """Weights and logits at addresses that are only a multiple of their element's size (views into flat
    buffers): the same logits, bit by bit, as with arrays of their own."""
    cfg = W.ModelConfig(W.GATED, dtype, R, (1, 2), S, S)
    w = W.make_weights(cfg, 79, bias_scale=0.1)
    x = dev(W.sequences(79, 3, 30))
    want = model(cfg, w, 3, FWG_PAR_HEAD="1").teacher_forced_parallel(x)

    def off(t):  # a copy one element past an aligned address
        flat = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
        flat[1:] = t.reshape(-1)
        return flat[1:].view(t.shape)

    dw = binding.upload_weights(w, dtype)
    for name in ("embed", "head", "out"):
        setattr(dw, name, off(getattr(dw, name)))
    for name in ("conv", "res", "skip"):
        setattr(dw, name, [off(t) for t in getattr(dw, name)])
    os.environ["FWG_PAR_HEAD"] = "1"
    try:
        fw = binding.FastWavenet(cfg.kind, dtype, R, cfg.dilations, 3, dw, skip_channels=S, head_channels=S)
    finally:
        os.environ.pop("FWG_PAR_HEAD")
    out = off(torch.zeros((3, 30, 256), device="cuda"))
    assert torch.equal(fw.teacher_forced_parallel(x, out=out), want)


def test_parallel_head_beyond_4gb_of_rows():
    """A chunk whose z rows take more than 4 GB (65,664 streams x 512 layers: one step per chunk is the
    least): streams with the same input have the same logits, bit by bit, on both sides of 4 GB."""
    B = 65664
    cfg = W.ModelConfig(W.GATED, W.F32, 32, (1,) * 512, 256, 256)
    fw = model(cfg, W.make_weights(cfg, 76, bias_scale=0.1), B, FWG_PAR_HEAD="1")
    x = (torch.arange(B, dtype=torch.int32, device="cuda") % 251).view(B, 1).contiguous()
    lg = fw.teacher_forced_parallel(x)[:, 0]
    assert torch.isfinite(lg).all() and not torch.equal(lg[0], lg[1])
    assert torch.equal(lg[251:], lg[:-251])


def test_parallel_stack_queue_beyond_64gb():
    """A queue more than 64 GB into the queue region (33 layers of 2 GB each before it): priming through
    the whole-stack kernel leaves its states where the step kernels read them."""
    if torch.cuda.mem_get_info()[0] < 160e9:
        pytest.skip("needs 160 GB of free device memory")
    cfg = W.ModelConfig(W.GATED, W.BF16, 64, (2 ** 20 - 1,) * 33 + (64,), 512, 512)
    w = W.make_weights(cfg, 77, bias_scale=0.1)
    w.conv[33][:, :, 0] *= 4  # the last layer's recurrent tap counts
    fw = model(cfg, w, 1, FWG_PAR_STACK="1")
    x = dev(W.sequences(78, 1, 212))
    want = fw.step_forced(x).cpu().numpy()[:, 200:]
    fw.reset()
    fw.prime(x[:, :200].contiguous())
    got = fw.step_forced(x[:, 200:].contiguous()).cpu().numpy()
    del fw
    torch.cuda.empty_cache()
    assert row_rel_err(got, want) <= TOL[W.BF16]


@pytest.mark.parametrize("B,T", [(5, 1000), (4, 2047)])
def test_parallel_f32_tiles(B, T):
    """float32 products of 512 channels over 5,000 rows (small tiles: 3 rounds of a quarter against 1 of
    4) and 8,188 rows (256 large tiles, one per compute unit), ragged: the oracle on one stream."""
    cfg = W.ModelConfig(W.RELU_RESIDUAL, W.F32, 512, (1, 2))
    w = W.make_weights(cfg, 74, bias_scale=0.1)
    fw = model(cfg, w, B)
    x = W.sequences(75, B, T)
    got = fw.teacher_forced_parallel(dev(x)).cpu().numpy()
    assert row_rel_err(got[-1:], oracle.Oracle(w).teacher_forced(x[-1:])) <= TOL[W.F32]


@pytest.mark.parametrize("stack", ["0", "1"])
def test_parallel_gate_small_arguments(stack):
    """The gate of the time-parallel kernels where |a| is small: conv weights of ~1e-6, so that z is ~1e-6
    and below (skip weights of ~1e6 bring it back), where 1 - 2 / (exp(2a) + 1) keeps only a few bits.
    The whole-stack and the per-layer kernel against the oracle at the bf16 bar."""
    cfg = W.ModelConfig(W.GATED, W.BF16, 64, (1, 2, 4), 512, 512)
    w = W.make_weights(cfg, 64)
    for l in range(cfg.n_layers):
        w.conv[l] *= 2.0 ** -20
        w.skip[l] *= 2.0 ** 20
    fw = model(cfg, w, 5, FWG_PAR_STACK=stack)
    x = W.sequences(65, 5, 40)
    got = fw.teacher_forced_parallel(dev(x)).cpu().numpy()
    assert row_rel_err(got, oracle.Oracle(w).teacher_forced(x)) <= TOL[W.BF16]


@pytest.mark.parametrize("B,T", [(1, 1), (3, 43), (5, 300), (17, 257)])
def test_parallel_kernels_give_the_same_bits(B, T):
    """The whole-stack kernel and the fused head take their sums in the order of the per-layer and GEMM
    kernels (from zero, the bias last) and the same gate: teacher forcing and priming agree with them
    bit by bit, logits and (through the step kernels' next logits) queues."""
    for dtype, R, S, env in ((W.BF16, 64, 512, ("FWG_PAR_STACK", "FWG_PAR_HEAD")), (W.F32, 32, 256, ("FWG_PAR_HEAD",))):
        cfg = W.ModelConfig(W.GATED, dtype, R, (1, 2, 4, 8, 64, 300, 3), S, S)
        w = W.make_weights(cfg, 66, bias_scale=0.1)
        x, y = W.sequences(67, B, T), dev(W.sequences(68, B, 9))
        outs = []
        for on in ("0", "1"):
            fw = model(cfg, w, B, **{k: on for k in env})
            outs.append([fw.teacher_forced_parallel(dev(x)), fw.prime(dev(x), logits=True), fw.step_forced(y)])
        for a, b in zip(*outs):
            assert torch.equal(a, b)


# shapes of the general kernel: 512 and 256 threads, several columns per thread (N > 512, N no multiple of
# the thread count), K-groups with fewer than 8 and more than 8 k-blocks, wide pops, more streams than
# compute units
GENERAL = {
    "gated_f32_r64": (W.ModelConfig(W.GATED, W.F32, 64, (1, 2, 4, 1), 256, 128), 3),
    "gated_bf16_r64": (W.ModelConfig(W.GATED, W.BF16, 64, (1, 3, 2), 128, 320), 2),
    "gated_f32_r128": (W.ModelConfig(W.GATED, W.F32, 128, (2, 1), 640, 512), 5),
    "relu_f32_c320": (W.ModelConfig(W.RELU, W.F32, 320, (1, 2)), 2),
    "relures_bf16_c576": (W.ModelConfig(W.RELU_RESIDUAL, W.BF16, 576, (1, 2, 3)), 2),
    "relu_f32_c256_l1": (W.ModelConfig(W.RELU, W.F32, 256, (3,)), 1),
    "relures_f32_c128_w5": (W.ModelConfig(W.RELU_RESIDUAL, W.F32, 128, (1, 2, 1), filter_width=5), 2),
    "gated_f32_r64_b300": (W.ModelConfig(W.GATED, W.F32, 64, (1, 2), 64, 64), 300),
    # past 512 streams: four blocks per compute unit, and two streams per block from 100 KB of weights per layer
    # on (an odd batch leaves the last block one stream)
    "gated_f32_r32_b600": (W.ModelConfig(W.GATED, W.F32, 32, (1, 2, 5), 64, 64), 600),
    "gated_f32_r32_w3_b513": (W.ModelConfig(W.GATED, W.F32, 32, (1, 2), 64, 64, filter_width=3), 513),
    "gated_bf16_r64_b600": (W.ModelConfig(W.GATED, W.BF16, 64, (1, 2), 64, 64), 600),
    "relu_bf16_c64_w3_b700": (W.ModelConfig(W.RELU, W.BF16, 64, (1, 3), filter_width=3), 700),
    "relures_f32_c128_b513": (W.ModelConfig(W.RELU_RESIDUAL, W.F32, 128, (1, 2, 3)), 513),
    "relu_f32_c128_l1_b514": (W.ModelConfig(W.RELU, W.F32, 128, (2,)), 514),
    "relures_bf16_c320_w3_b515": (W.ModelConfig(W.RELU_RESIDUAL, W.BF16, 320, (1, 2), filter_width=3), 515),
    "relu_f32_c1024_b513": (W.ModelConfig(W.RELU, W.F32, 1024, (1,)), 513),
}


@pytest.mark.parametrize("name", list(GENERAL))
def test_general_kernel_shapes(name):
    """Teacher forcing through the step kernel against the oracle (sampled streams), and the state
    carried across calls: online prediction in two pieces equals one, bit by bit.  Generation on a
    handle for more streams than 512 equals that of one for 300 (256 threads and one stream per block: the
    same sums, bit by bit)."""
    cfg, B = GENERAL[name]
    w = W.make_weights(cfg, 80, bias_scale=0.1)
    fw = model(cfg, w, B)
    assert fw.regime == "valu"
    T = 30
    x = W.sequences(81, B, T)
    sel = sorted({0, B // 2, B - 1})
    got = fw.teacher_forced(dev(x)).cpu().numpy()
    assert row_rel_err(got[sel], oracle.Oracle(w).teacher_forced(x[sel])) <= TOL[cfg.dtype]
    one = fw.step_forced(dev(x)).cpu().numpy()
    fw.reset()
    a = fw.step_forced(dev(x[:, :11])).cpu().numpy()
    b = fw.step_forced(dev(x[:, 11:])).cpu().numpy()
    assert np.array_equal(np.concatenate([a, b], axis=1), one)
    if B > 512:
        u = W.uniforms(82, B, 20)
        fw.reset()
        g = fw.generate(dev(u)).cpu().numpy()
        alone = model(cfg, w, 300, FWG_REGIME="valu")
        for i in sel:
            alone.reset()
            assert np.array_equal(alone.generate(dev(u[i:i + 1])).cpu().numpy()[0], g[i])


@pytest.mark.parametrize("B", [1, 6])
@pytest.mark.parametrize("t0", [0, 1, 2, 5, 40])
def test_wide_state_across_launches(t0, B):
    """The wide kernel's state pass at launch: nothing written yet, fewer steps than the shortest and
    the longest dilation, every queue wrapped.  The second launch's logits against the oracle's."""
    cfg = W.ModelConfig(W.RELU_RESIDUAL, W.F32, 512, (1, 2, 4, 8, 16, 3))
    w = W.make_weights(cfg, 90, bias_scale=0.1)
    fw = model(cfg, w, B)
    assert fw.regime == "wide_f32_c512"
    x = W.sequences(91, B, t0 + 9)
    if t0:
        fw.step_forced(dev(x[:, :t0]))
    got = fw.step_forced(dev(x[:, t0:])).cpu().numpy()
    st = oracle.Oracle(w).state(B)
    want = st.step_forced(x)
    assert row_rel_err(got, want[:, t0:]) <= TOL[W.F32]


@pytest.mark.parametrize("name", ["pair", "pair_w3", "wide"])
def test_exchange_tags_across_launches(name):
    """The gated chain pair and wide kernels' exchange words are cleared only before a handle's first
    launch and when the 32-bit tags would wrap: on poisoned memory, a small batch's launch before a
    larger one, launches that cross the wrap, and graph replays between eager launches give the logits
    and samples of a fresh handle."""
    cfg = {"pair": W.ModelConfig(W.GATED, W.F32, 32, (1, 2, 4, 8), 256, 256),
           "pair_w3": W.ModelConfig(W.GATED, W.F32, 32, (1, 3, 9), 256, 256, filter_width=3),
           "wide": W.ModelConfig(W.RELU_RESIDUAL, W.F32, 512, (1, 2, 4))}[name]
    w = W.make_weights(cfg, 95, bias_scale=0.1)
    B = 11
    x, u = dev(W.sequences(96, B, 30)), dev(W.uniforms(97, B, 90))
    ref = model(cfg, w, B)
    assert ref.lib.fwg_waits(ref.handle) == 1
    lg = ref.teacher_forced(x).cpu().numpy()
    want = ref.generate(u).cpu().numpy()
    words = (ref.ws_bytes + 7) // 8
    poison = ((torch.arange(words, dtype=torch.int64, device="cuda") % 64 + 1) << 32) | 5
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        clean = binding.from_model(cfg, w, max_batch=B, workspace=poison.view(torch.uint8))
        clean.generate(u[:3, :10].contiguous())
        clean.reset()
        assert np.array_equal(clean.teacher_forced(x).cpu().numpy(), lg)
        out = torch.empty((B, 90), dtype=torch.int32, device="cuda")
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            clean.reset()
            clean.generate(u, out=out, check=False)
        for _ in range(3):
            out.zero_()
            g.replay()
            s.synchronize()
            assert np.array_equal(out.cpu().numpy(), want)
            assert np.array_equal(clean.teacher_forced(x).cpu().numpy(), lg)
        clean.device_status()
    wrap = model(cfg, w, B, FWG_SPLIT_TAG_BASE=str(0xFFFFFFFF - 60))
    got = [wrap.generate(u[:, i:i + 30].contiguous()).cpu().numpy() for i in (0, 30, 60)]
    assert np.array_equal(np.concatenate(got, axis=1), want)


@pytest.mark.parametrize("kind,dtype,C,S", [(W.GATED, W.BF16, 64, 512), (W.GATED, W.F32, 32, 256), (W.RELU, W.F32, 64, 0)])
def test_parallel_chunks_of_a_small_batch(kind, dtype, C, S):
    """A call with fewer streams than the handle's largest batch cuts its steps into longer chunks:
    teacher forcing and priming of 1 and 3 streams on handles for 20 whose buffers hold 40 steps of
    all of them, against the oracle and the step kernels' state."""
    cfg = W.ModelConfig(kind, dtype, C, (1, 2, 4, 8, 16, 32, 64), S, S)
    w = W.make_weights(cfg, 99, bias_scale=0.1)
    brows = 32 if dtype == W.BF16 else 20
    fw = model(cfg, w, 20, FWG_PAR_ROWS=str(40 * brows))
    orc = oracle.Oracle(w)
    for B in (1, 3):
        x = W.sequences(98, B, 1000)
        assert row_rel_err(fw.teacher_forced_parallel(dev(x)).cpu().numpy(), orc.teacher_forced(x)) <= TOL[dtype]
        fw.reset()
        fw.prime(dev(x[:, :777]))
        got = fw.step_forced(dev(x[:, 777:800])).cpu().numpy()
        assert row_rel_err(got, orc.state(B).step_forced(x[:, :800])[:, 777:]) <= TOL[dtype]
