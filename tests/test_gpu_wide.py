"""The projections of large batches (17 to 64 sequences, mfma_wide.hip)
against the fp64 oracle, through the C ABI (MI355X), to the bars of the other
projection paths: sequence tiles of 16 filled and ragged, one stripe per block
up to several passes of stripes, k-tiles fewer than the block's waves, padded
stripes and k-tiles, parts, and steps below and above the 16-sequence
limit on one handle; the attention kernels as these steps run them (q|k|v in
two parts), over bf16 and 8-bit caches; and what the test and measurement
hooks read after such steps."""
import numpy as np
import pytest

from gpu_harness import full_check, log, run_gpu
from oracle import ref
from paper_2607_11211_amd import inputs
from paper_2607_11211_amd.configs import LayerConfig

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_11211_amd.layer  # noqa: F401  (fails loudly if the library is missing)


def _cfg(name, index, batch, hidden, heads, kv, d, inter, max_seq=40):
    return LayerConfig(name=name, index=index, batch=batch, hidden=hidden, n_heads=heads, n_kv_heads=kv, head_dim=d,
                       intermediate=inter, rope_base=10000.0, max_seq=max_seq,
                       pos=tuple((7 * i + 3) % max_seq for i in range(batch)))


# sizes past the line of the dispatch (25 MB of weights read again by the kernels of 16 sequences)
SHAPES = [
    # one sequence past the limit; hidden 776 pads stripes and k-tiles
    _cfg("w_b17", 100, 17, 776, 8, 8, 96, 6408, 130),
    # two full sequence tiles; QKV in 12 stripes per block (two passes of 6), gate/up in two of 5;
    # hidden 192: six k-tiles for eight waves
    _cfg("w_b32_rows", 101, 32, 192, 64, 64, 128, 20000),
    # the same with four sequence tiles and two k-tiles
    _cfg("w_b64_rows", 102, 64, 64, 64, 64, 128, 20000),
    # three tiles, the last of one sequence; groups of four
    _cfg("w_b33", 103, 33, 512, 8, 2, 64, 5224, 70),
    # O and down projections in 4 parts (4096 and 4192 inputs), 49 and 20 sequences
    _cfg("w_parts_b49", 104, 49, 256, 32, 8, 128, 4192),
    _cfg("w_parts_b20", 105, 20, 264, 32, 8, 128, 17408),
    # wide inputs against few units
    _cfg("w_din_b48", 106, 48, 4096, 4, 4, 64, 384),
    # the widest MLP: 1024 k-tiles in the down projection
    _cfg("w_longk_b18", 107, 18, 168, 1, 1, 128, 32768),
]


@pytest.mark.parametrize("cfg", SHAPES, ids=lambda c: c.name)
def test_wide_matches_oracle(cfg):
    log(f"start {cfg.name}")
    inp = inputs.make_layer_inputs(cfg)
    r = ref.decode_layer_cfg(cfg, inp.x, inp.pos, inp.k_cache, inp.v_cache, inp.weights)
    gpu = run_gpu(cfg, inp)
    full_check(cfg, inp, gpu, r)


def _long(name, index, hidden, heads, kv, d, inter, pos):
    cfg = LayerConfig(name=name, index=index, batch=len(pos), hidden=hidden, n_heads=heads, n_kv_heads=kv, head_dim=d,
                      intermediate=inter, rope_base=10000.0, max_seq=max(pos) + 2, pos=tuple(pos))
    # past the line of the dispatch: 25 MB read again by the kernels of 16 sequences
    weights = 2 * hidden * ((2 * heads + 2 * kv) * d + 3 * inter)
    assert weights * ((cfg.batch - 1) // 16) >= 25 << 20, name
    return cfg


def _spread(n, lo, hi):
    return tuple(lo + (i * 37) % (hi - lo + 1) for i in range(n))


# the attention kernels as these steps run them: q|k|v in two parts, o into the operand of 16-sequence tiles
ATTENTION = [
    # matrix cores: groups of two and four, several splits and one
    _long("w_g2_d128", 150, 512, 8, 4, 128, 8704, _spread(19, 0, 400)),
    _long("w_g2_d96", 151, 512, 4, 2, 96, 8704, _spread(17, 60, 300)),
    _long("w_g2_d64_128", 152, 512, 4, 2, 64, 8704, _spread(18, 70, 128)),
    _long("w_g4_one", 153, 512, 64, 16, 128, 8000, _spread(17, 1, 1000)),
    # vector kernel: groups of two at d = 64
    _long("w_g2_d64_vec", 154, 512, 4, 2, 64, 8704, _spread(17, 100, 500)),
    _long("w_g2_d64_vec_xch", 174, 512, 32, 16, 64, 8000, (1000,) + _spread(16, 0, 200)),
    # one head: tiles exchanged through LDS (8 or more per split), in two splits and in one
    _long("w_xch_d128", 155, 512, 16, 16, 128, 8000, _spread(17, 1060, 1100)),
    _long("w_xch_d96_one", 156, 512, 16, 16, 96, 8704, _spread(17, 600, 1000)),
    _long("w_xch_d64", 157, 512, 16, 16, 64, 8704, _spread(17, 1100, 1200)),
    # more than 32 splits: the block-wide combine
    _long("w_combine", 158, 512, 2, 1, 128, 8704, (6000,) + _spread(16, 0, 60)),
    _long("w_combine_d96", 159, 512, 1, 1, 96, 8704, (3000,) + _spread(32, 0, 60)),
]


@pytest.mark.parametrize("cfg", ATTENTION, ids=lambda c: c.name)
def test_attention_of_large_batches(cfg):
    log(f"start {cfg.name}")
    inp = inputs.make_layer_inputs(cfg)
    r = ref.decode_layer_cfg(cfg, inp.x, inp.pos, inp.k_cache, inp.v_cache, inp.weights)
    full_check(cfg, inp, run_gpu(cfg, inp), r)


# the same over 8-bit caches, on both sides of the matrix cores' lines (2^18 rows; 17 * 2^15 for
# groups of two at d = 64)
KV8 = [
    _long("w8_g1_d128", 160, 512, 4, 4, 128, 8704, _spread(20, 0, 300)),
    _long("w8_g1_d96", 161, 512, 4, 4, 96, 8704, _spread(33, 0, 200)),
    _long("w8_g1_d64", 162, 512, 4, 4, 64, 8704, _spread(17, 5, 300)),
    _long("w8_g2_d128", 163, 512, 4, 2, 128, 8704, _spread(17, 5, 300)),
    _long("w8_g2_d96", 164, 512, 4, 2, 96, 8704, _spread(18, 0, 200)),
    _long("w8_g2_d64", 165, 512, 4, 2, 64, 8704, _spread(18, 0, 200)),
    _long("w8_g4_d64", 166, 512, 8, 2, 64, 8704, _spread(18, 0, 300)),
    _long("w8_g4_d96", 167, 512, 4, 1, 96, 8704, _spread(17, 0, 300)),
    _long("w8_g4_d128", 168, 512, 8, 2, 128, 8704, _spread(33, 0, 300)),
    _long("w8_g1_d128_long", 169, 512, 16, 16, 128, 8000, _spread(17, 965, 1005)),
    _long("w8_g1_d96_long", 170, 512, 16, 16, 96, 8704, _spread(17, 1025, 1060)),
    _long("w8_g2_d128_long", 171, 256, 32, 16, 128, 14000, _spread(17, 965, 1100)),
    _long("w8_g2_d96_long", 172, 256, 32, 16, 96, 15000, _spread(17, 965, 1005)),
    _long("w8_g2_d64_long", 173, 256, 64, 32, 64, 7000, _spread(33, 530, 560)),
]


@pytest.mark.parametrize("fmt", inputs.KV8_FORMATS)
@pytest.mark.parametrize("cfg", KV8, ids=lambda c: c.name)
def test_kv8_attention_of_large_batches(cfg, fmt):
    from test_gpu_kv8 import run_case
    log(f"start {cfg.name} {fmt}")
    run_case(cfg, inputs.make_layer_inputs(cfg), fmt)


@pytest.mark.parametrize("cfg", [c for c in ATTENTION if c.name in ("w_g2_d128", "w_g2_d64_vec", "w_xch_d96_one")],
                         ids=lambda c: c.name)
def test_study_switch_of_large_batches(cfg):
    """The accuracy study's bf16 weights (vector kernel) with q|k|v in two parts."""
    from gpu_harness import check_y
    from paper_2607_11211_amd import layer as L
    log(f"start {cfg.name} p_bf16")
    inp = inputs.make_layer_inputs(cfg)
    r = ref.decode_layer_cfg(cfg, inp.x, inp.pos, inp.k_cache, inp.v_cache, inp.weights)
    lay = L.Layer(cfg)
    lay.set_attention_p_bf16(True)
    got = run_gpu(cfg, inp, layer=lay, keep=True)
    check_y(got, r)
    got["_weights"].free()
    lay.destroy()


def test_batches_around_the_limit_on_one_handle():
    """Steps of 40, 16, 17 and 3 sequences on one handle: each reads operands
    that another layout and another batch left in the buffers."""
    from paper_2607_11211_amd import layer as L
    big = _cfg("w_mix", 108, 40, 512, 32, 8, 128, 7200, 60)
    inp = inputs.make_layer_inputs(big)
    lay = L.Layer(big, max_batch=64)
    W = lay.pack({k: L.to_device(v) for k, v in inp.weights.items()})
    Wf = ref.widen_weights(inp.weights)
    for nb in (40, 16, 17, 3):
        cfg = _cfg(f"w_mix{nb}", 108, nb, 512, 32, 8, 128, 7200, 60)
        step = inputs.LayerInputs(cfg=cfg, x=inputs.make_x(cfg, seed=300 + nb), pos=inp.pos[:nb].copy(),
                                  weights=inp.weights, k_cache=inp.k_cache[:nb].copy(),
                                  v_cache=inp.v_cache[:nb].copy())
        r = ref.decode_layer_cfg(cfg, step.x, step.pos, step.k_cache, step.v_cache, Wf)
        log(f"start w_mix of {nb}")
        full_check(cfg, step, run_gpu(cfg, step, layer=lay, weights=W), r)
    W.free()
    lay.destroy()


def test_wide_replays_equal_eager():
    """Graph replays with eager steps in between give the first eager step's
    bits (operands and parts share buffers between the kernels of a step)."""
    import torch
    from paper_2607_11211_amd import layer as L
    cfg = next(c for c in SHAPES if c.name == "w_parts_b49")
    inp = inputs.make_layer_inputs(cfg)
    lay = L.Layer(cfg)
    W = lay.pack({k: L.to_device(v) for k, v in inp.weights.items()})
    x = L.to_device(inp.x)
    kc, vc = L.to_device(inp.k_cache), L.to_device(inp.v_cache)
    y = torch.empty_like(x)
    stream = torch.cuda.current_stream()
    lay.step(W, x, inp.pos, kc, vc, y, stream)
    torch.cuda.synchronize()
    want = L.from_device(y)
    g = torch.cuda.CUDAGraph()
    s = torch.cuda.Stream()
    s.wait_stream(stream)
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            lay.step(W, x, inp.pos, kc, vc, y, s)
    stream.wait_stream(s)
    torch.cuda.synchronize()
    for rep in range(4):
        y.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(L.from_device(y), want), f"replay {rep} differs from the eager step"
        lay.step(W, x, inp.pos, kc, vc, y, stream)
        torch.cuda.synchronize()
        assert np.array_equal(L.from_device(y), want)
    del g
    W.free()
    lay.destroy()


def test_qkv_hook_after_other_batches_and_replays():
    """FASTTPS_DBG_QKV gives each row as the last step that held it left it:
    steps of 40 and 20 sequences (two parts), of 3 and 1 (whole sums), and a
    replayed step of 3 after an eager one of 40, read at 40 sequences."""
    import torch
    from paper_2607_11211_amd import layer as L
    cfg = _cfg("w_hook", 109, 40, 512, 32, 8, 128, 7200, 60)
    inp = inputs.make_layer_inputs(cfg)
    lay = L.Layer(cfg)
    W = lay.pack({k: L.to_device(v) for k, v in inp.weights.items()})
    kc, vc = L.to_device(inp.k_cache), L.to_device(inp.v_cache)
    xs = {n: L.to_device(inputs.make_x(cfg, seed=400 + n)) for n in (40, 20, 3, 1)}
    y = torch.empty_like(xs[40])

    def step(n, stream=None):
        lay.step(W, xs[n][:n], inp.pos[:n], kc, vc, y[:n], stream)

    def read(n):
        t = torch.empty(n, cfg.qkv_rows, dtype=torch.float32, device="cuda")
        lay.debug_read(L.DBG_QKV, n, t)
        torch.cuda.synchronize()
        return t.cpu().numpy()

    want = {}
    for n in (40, 20, 3, 1):  # each step's own rows
        step(n)
        want[n] = read(n)
    rows = want[40].copy()
    step(40)
    for n in (20, 3, 1, 20):
        step(n)
        rows[:n] = want[n]
        assert np.array_equal(read(40), rows), f"after a step of {n}"

    g = torch.cuda.CUDAGraph()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            step(3, s)
    torch.cuda.current_stream().wait_stream(s)
    rows[:] = want[40]
    rows[:3] = want[3]
    for rep in range(3):
        step(40)
        g.replay()
        assert np.array_equal(read(40), rows), f"replay {rep}"
    del g
    W.free()
    lay.destroy()


def test_profile_covers_every_launch():
    """The per-kernel times of a step cover its small kernels too: on a layer
    where the QKV operand and the sums of the parts are a fifth of the step
    (83 us on MI355X, 68 of them without those, 86 with them: each launch
    timed alone takes a little longer), the times add up to the replayed step."""
    import torch
    from paper_2607_11211_amd import layer as L
    cfg = _cfg("w_prof", 110, 64, 8192, 1, 1, 64, 384)
    inp = inputs.make_layer_inputs(cfg)
    lay = L.Layer(cfg)
    W = lay.pack({k: L.to_device(v) for k, v in inp.weights.items()})
    x = L.to_device(inp.x)
    kc, vc = L.to_device(inp.k_cache), L.to_device(inp.v_cache)
    y = torch.empty_like(x)
    for _ in range(3):
        lay.step(W, x, inp.pos, kc, vc, y)
    torch.cuda.synchronize()
    lay.profile_begin(12)
    for _ in range(12):
        lay.step(W, x, inp.pos, kc, vc, y)
    per_kernel = np.median(lay.profile_end(12), axis=0) * 1e3
    g = torch.cuda.CUDAGraph()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            for _ in range(10):
                lay.step(W, x, inp.pos, kc, vc, y, s)
    torch.cuda.current_stream().wait_stream(s)
    steps = []
    for _ in range(4):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        g.replay()
        b.record()
        torch.cuda.synchronize()
        steps.append(a.elapsed_time(b) * 1e3 / 10)
    log(f"per kernel us {per_kernel.round(2)}, step {min(steps):.2f}")
    assert 0.92 * min(steps) <= per_kernel.sum() <= 1.5 * min(steps)
    del g
    W.free()
    lay.destroy()
