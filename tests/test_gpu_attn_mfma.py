"""The attention on the matrix cores (attn_mfma.hip) through the C ABI
(MI355X): groups of two and four query heads over bf16 caches and 8-bit caches
of every group size, at the edges of its 32-position wave tiles, 128-position
block tiles and splits, against the fp64 oracle to the bars of the vector
kernel; what non-finite cache entries give; and the accuracy study's variant,
which keeps the vector kernel."""
import numpy as np
import pytest

from gpu_harness import check_y, full_check, log, run_gpu
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


def _cfg(name, index, heads, kv, d, pos, max_seq=None):
    return LayerConfig(name=name, index=index, batch=len(pos), hidden=128, n_heads=heads, n_kv_heads=kv, head_dim=d,
                       intermediate=256, rope_base=10000.0, max_seq=max_seq or max(pos) + 3, pos=tuple(pos))


def _inputs(cfg):
    """The layer's inputs with W_q sixteen times as large (exact in bf16), so
    that the scores of these narrow layers spread over several units."""
    inp = inputs.make_layer_inputs(cfg)
    inp.weights["w_q"] = (inp.weights["w_q"] + np.uint16(4 << 7)).astype(np.uint16)
    return inp


EDGES = (0, 1, 15, 16, 17, 31, 32, 33, 63, 64, 96, 127, 128, 129, 255, 257)
BF16 = [
    _cfg("am_g4_d64", 110, 8, 2, 64, EDGES),
    _cfg("am_g4_d96", 111, 8, 2, 96, EDGES),
    _cfg("am_g4_d128", 112, 4, 1, 128, EDGES),
    _cfg("am_g2_d64", 113, 4, 2, 64, EDGES),
    _cfg("am_g2_d96", 114, 2, 1, 96, EDGES),
    _cfg("am_g2_d128", 115, 8, 4, 128, EDGES),
    # one sequence in many splits, and a batch whose short sequences leave splits empty
    _cfg("am_g4_one", 116, 4, 1, 64, (9000,)),
    _cfg("am_g2_ragged", 117, 16, 8, 128, (5, 4000, 130, 2049)),
    # groups of two at d = 64 on both sides of their lines: one sequence of up to 256 positions
    # (vector) and more, batches of up to 64 (vector), 128, and of 2^16 rows (vector) and one more
    _cfg("am_g2_d64_one256", 134, 4, 2, 64, (256,)),
    _cfg("am_g2_d64_one257", 135, 4, 2, 64, (257,)),
    _cfg("am_g2_d64_64", 136, 4, 2, 64, (64, 0, 17)),
    _cfg("am_g2_d64_65", 137, 4, 2, 64, tuple(e for e in EDGES if e <= 128) + (65,)),
    _cfg("am_g2_d64_2p16", 138, 64, 32, 64, (1900, 148)),
    _cfg("am_g2_d64_2p16_1", 139, 64, 32, 64, (1900, 149)),
    # one split of 8 tiles or more on the vector kernel: its tiles exchanged through LDS
    _cfg("am_g2_d64_xch", 142, 32, 16, 64, (1000,) + tuple(9 * i for i in range(15))),
]


@pytest.mark.parametrize("cfg", BF16, ids=lambda c: c.name)
def test_bf16_matches_oracle(cfg):
    log(f"start {cfg.name}")
    inp = _inputs(cfg)
    r = ref.decode_layer_cfg(cfg, inp.x, inp.pos, inp.k_cache, inp.v_cache, inp.weights)
    full_check(cfg, inp, run_gpu(cfg, inp), r)


# one split per (sequence, KV head): the attention writes the finished o, for
# the vector and the matrix-core attention, the operand layouts of up to 16 and
# of more sequences, and the vector projections
DIRECT = [
    _cfg("ad_g1_b16", 128, 16, 16, 64, tuple(range(0, 1024, 64))),
    _cfg("ad_g4_b16", 129, 64, 16, 128, tuple(3 + 60 * i for i in range(16))),
    _cfg("ad_g1_b64", 130, 8, 8, 96, tuple(1 + 31 * i for i in range(64)), 2049),
]


@pytest.mark.parametrize("cfg", DIRECT, ids=lambda c: c.name)
@pytest.mark.parametrize("path", ["matrix", "vector"])
def test_one_split_matches_oracle(cfg, path):
    from paper_2607_11211_amd import layer as L
    log(f"start {cfg.name} {path}")
    inp = _inputs(cfg)
    r = ref.decode_layer_cfg(cfg, inp.x, inp.pos, inp.k_cache, inp.v_cache, inp.weights)
    full_check(cfg, inp, run_gpu(cfg, inp, gemm_path=L.GEMM_MATRIX if path == "matrix" else L.GEMM_VECTOR), r)


KV8 = [
    _cfg("a8_g4_d64", 120, 8, 2, 64, EDGES),
    _cfg("a8_g4_d96", 121, 4, 1, 96, EDGES),
    _cfg("a8_g4_d128", 122, 8, 2, 128, EDGES),
    # smaller groups take this kernel from 2^18 cached rows up (at d = 64 from 17 * 2^15)
    _cfg("a8_g1_d96", 123, 32, 32, 96, (4099, 4110)),
    _cfg("a8_g1_d128", 124, 32, 32, 128, (8193, 33)),
    _cfg("a8_g2_d64", 125, 64, 32, 64, (127, 8200, 1)),
    _cfg("a8_g2_d96", 126, 32, 16, 96, (8192, 8193)),
    _cfg("a8_g2_d128", 127, 64, 32, 128, (4096, 4097)),
    # groups of two at d = 64: one row short of their line (vector) and on it
    _cfg("a8_g2_d64_below", 140, 64, 32, 64, (127, 17279, 1)),
    _cfg("a8_g2_d64_line", 141, 64, 32, 64, (127, 17280, 1)),
]


@pytest.mark.parametrize("fmt", inputs.KV8_FORMATS)
@pytest.mark.parametrize("cfg", KV8, ids=lambda c: c.name)
def test_kv8_matches_oracle(cfg, fmt):
    from test_gpu_kv8 import run_case
    log(f"start {cfg.name} {fmt}")
    run_case(cfg, _inputs(cfg), fmt)


def _softmax_o(q, k, v, scale):
    s = k @ q * scale
    p = np.exp(s - s.max())
    return p @ v / p.sum()


def test_nonfinite_entries():
    """An infinite V element reaches its output element alone, also when it is
    in the last cached row, which masked positions repeat; an infinite K element gives its
    position weight 0 where its score is -inf and a NaN head where it is
    +inf."""
    cfg = _cfg("am_inf", 118, 8, 2, 64, (40, 40, 40))
    inp = _inputs(cfg)
    inf = 0x7F80
    inp.v_cache[0, 1, 39, 10] = inf      # the last cached row
    inp.v_cache[1, 0, 3, 63] = inf | 0x8000
    inp.k_cache[2, 0, 7, 5] = inf
    with np.errstate(all="ignore"):
        g = run_gpu(cfg, inp)
    o = g["o"].reshape(3, 8, 64)
    q = g["qk_rope"].reshape(3, 10, 64)[:, :8]
    for b in range(3):
        for h in range(8):
            kv = h // 4
            k = ref.bf16_bits_to_f64(g["k_cache"][b, kv, :41])
            v = ref.bf16_bits_to_f64(g["v_cache"][b, kv, :41])
            if b == 2 and kv == 0:
                if q[b, h, 5] > 0:
                    assert np.all(np.isnan(o[b, h])), (b, h)
                    continue
                keep = np.arange(41) != 7
                want = _softmax_o(q[b, h], k[keep], v[keep], 0.125)
                bad = np.zeros(64, bool)
            else:
                bad = ~np.isfinite(v).all(axis=0)
                want = _softmax_o(q[b, h], k, np.where(np.isfinite(v), v, 0.0), 0.125)
            assert np.max(np.abs(o[b, h] - want)[~bad]) <= 1e-5 * np.max(np.abs(want)), (b, h)
            if bad.any():
                # (inf, or NaN where the merge of the splits multiplies it by 0)
                assert not np.any(np.isfinite(o[b, h][bad])), (b, h, o[b, h][bad])


def test_vector_kernel_still_serves_groups():
    """The accuracy study's bf16 weights keep the vector kernel for every group
    size: the layer's y stays within the bar."""
    import torch
    from paper_2607_11211_amd import layer as L
    cfg = _cfg("am_vec", 119, 8, 2, 128, (300, 128))
    inp = _inputs(cfg)
    r = ref.decode_layer_cfg(cfg, inp.x, inp.pos, inp.k_cache, inp.v_cache, inp.weights)
    lay = L.Layer(cfg)
    lay.set_attention_p_bf16(True)
    got = run_gpu(cfg, inp, layer=lay, keep=True)
    check_y(got, r)
    torch.cuda.synchronize()
    got["_weights"].free()
    lay.destroy()


@pytest.mark.parametrize("fmt", inputs.KV8_FORMATS)
@pytest.mark.parametrize("index,heads,kv", [(131, 4, 4), (132, 4, 2), (133, 8, 2)], ids=["g1", "g2", "g4"])
def test_study_switch_leaves_kv8_alone(index, heads, kv, fmt):
    """The accuracy study's switch is about bf16 caches: a step over an 8-bit
    cache runs with it on as without it, for every group size."""
    from paper_2607_11211_amd import layer as L
    from test_gpu_kv8 import run_case
    cfg = _cfg("a8_switch", index, heads, kv, 64, (130, 0, 33))
    inp = _inputs(cfg)
    lay = L.Layer(cfg)
    W = lay.pack({k: L.to_device(v) for k, v in inp.weights.items()})
    off, _ = run_case(cfg, inp, fmt, layer=lay, weights=W)
    lay.set_attention_p_bf16(True)
    on, _ = run_case(cfg, inp, fmt, layer=lay, weights=W)
    assert np.array_equal(on["y"], off["y"])
    W.free()
    lay.destroy()
