"""Parity of whole stages at shapes where tiles, splits and head widths end:
every product and attention kernel variant that the launchers choose by size,
against the fp64 oracle.  Bars are those of tests/test_gpu_parity.py (rel-L2
<= 1e-5 for fp32 stages, 2e-2 for bf16 ones); the small rows of a head of 8 or
32 sum fewer terms than the shapes those bars were set for."""
import pytest

import oracle
from paper_2405_14009_amd import RC_READ_GRAD, Stage
from synth import MB, gen_params, get_config
from tests.conftest import compare_grads, rel_l2
from tests.gpu_harness import log, run_gpu, takes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")


def check(cfg, t):
    log(f"[shape] L={cfg.layers} h={cfg.hidden} a={cfg.heads} f={cfg.ffn} s={cfg.seq} b={cfg.micro_batch} "
        f"n={cfg.n_mb} {cfg.dtype} causal={cfg.causal}")
    g = run_gpu(cfg)
    o = oracle.run_oplist(cfg)
    assert g.log == [tuple(r) for r in o.stage.log]
    for mb in o.y:
        assert rel_l2(g.y[mb], o.y[mb]) < t, ("y", mb, rel_l2(g.y[mb], o.y[mb]))
        assert rel_l2(g.dx[mb], o.dx[mb]) < t, ("dx", mb, rel_l2(g.dx[mb], o.dx[mb]))
    log(f"[shape] worst gradient rel-L2 {compare_grads(cfg, g.grads, o.grads, t):.2e}")


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("d,seq", [(8, 136), (32, 200), (40, 328), (64, 136), (64, 520), (80, 328), (96, 136),
                                   (104, 328), (120, 200), (64, 128)])
def test_attention_head_widths(d, seq, causal):
    """Head dimensions below 128, with as many columns as a kernel is compiled
    for and fewer; ragged last query and key blocks; d = 64 at s = 128 takes
    the materialised kernels.  These grids are small: the kernels that split a
    block's keys (or queries) over four waves, with one to four of them idle at
    the shortest sequences."""
    cfg = get_config("small_bf16").with_(layers=1, hidden=4 * d, heads=4, ffn=16 * d, seq=seq, n_mb=2,
                                         rerouted=(1,), causal=causal)
    takes(cfg, attention="materialised" if seq == 128 else "split")
    check(cfg, 2e-2)


@pytest.mark.parametrize("d", [64, 80])
def test_attention_head_widths_per_block(d):
    """The per-query-block causal kernels of narrow heads (160 pairs of query
    blocks fill 256 compute units poorly)."""
    cfg = get_config("block_bf16").with_(hidden=10 * d, ffn=20 * d, seq=1000, n_mb=1, rerouted=())
    takes(cfg, attention="block")
    check(cfg, 2e-2)


@pytest.mark.parametrize("d", [32, 64, 80, 120, 128])
@pytest.mark.parametrize("seq,micro_batch", [(1000, 4), (328, 8)])
def test_attention_head_widths_paired(d, seq, micro_batch):
    """Grids whose pairs of query blocks fill 256 compute units once: eight ragged
    query blocks, and three, whose middle one pairs with itself."""
    cfg = get_config("small_bf16").with_(layers=1, hidden=16 * d, heads=16, ffn=8 * d, seq=seq, micro_batch=micro_batch,
                                         n_mb=1, rerouted=())
    takes(cfg, attention="paired")
    check(cfg, 2e-2)


@pytest.mark.parametrize("d", [32, 64, 80, 120, 128])
def test_attention_head_widths_blocks_noncausal(d):
    """Bidirectional heads on a grid of more 32-row workgroups than compute units hold."""
    cfg = get_config("small_bf16").with_(layers=1, hidden=4 * d, heads=4, ffn=8 * d, seq=1128, micro_batch=4, n_mb=1,
                                         rerouted=(), causal=False)
    takes(cfg, attention="block")
    check(cfg, 2e-2)


# Token counts and widths one chunk of 8 to either side of 64, 128 and 256, a
# single k-tile and long reductions.
SHAPES = [dict(hidden=64, heads=1, ffn=64, seq=64, micro_batch=1, n_mb=1),
          dict(hidden=56, heads=1, ffn=72, seq=8, micro_batch=1, n_mb=2),
          dict(hidden=136, heads=1, ffn=264, seq=72, micro_batch=1, n_mb=3),
          dict(hidden=256, heads=2, ffn=2048, seq=248, micro_batch=1, n_mb=2),
          dict(hidden=264, heads=3, ffn=1032, seq=1000, micro_batch=3, n_mb=3),
          dict(hidden=512, heads=4, ffn=4096, seq=56, micro_batch=1, n_mb=5)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_product_shapes(dtype, shape):
    cfg = get_config("small_bf16").with_(layers=1, dtype=dtype, rerouted=(), schedule="1f1b_deferred_w", **shape)
    check(cfg, 1e-5 if dtype == "f32" else 2e-2)


def test_192_row_tiles():
    """FC1 forward and FC2 input gradient of [1800, 5032] over 768 fill 256
    compute units best in 192x256 tiles, ragged in both directions and in a
    tile count that is no multiple of the XCDs."""
    cfg = get_config("small_bf16").with_(layers=1, hidden=768, heads=6, ffn=5032, seq=600, micro_batch=3, n_mb=1,
                                         rerouted=())
    takes(cfg, f_fc1=("192x256", 1), d_fc2=("192x256", 1))
    check(cfg, 2e-2)


# One weight pass over several micro-batches whose token counts are no multiple
# of a k-tile: every tile of the weight-gradient layout, unsplit and with splits
# that end inside a segment; the persistent kernel over few and many k-tiles.
SEGMENTED = [
    (3, dict(hidden=64, heads=1, ffn=128, seq=72, micro_batch=1), dict(w_qkv=("32", 1), w_o=("32", 1), w_fc1=("32", 1))),
    (3, dict(hidden=264, heads=3, ffn=1032, seq=1000, micro_batch=3), dict(w_qkv=("64", 7), w_o=("64", 10))),
    (3, dict(hidden=768, heads=6, ffn=3080, seq=328, micro_batch=2), dict(w_qkv=("64", 1), w_fc1=("128", 3))),
    (3, dict(hidden=1152, heads=9, ffn=5128, seq=328, micro_batch=2), dict(w_qkv=("128", 1), w_fc1=("128", 1))),
    (3, dict(hidden=1280, heads=10, ffn=5128, seq=1000, micro_batch=1), dict(w_fc1=("256x128", 1))),
    (3, dict(hidden=1280, heads=10, ffn=5128, seq=1000, micro_batch=3),
     dict(w_qkv=("256", 3), w_o=("256x128", 5), w_fc1=("256", 2), w_fc2=("256", 2))),
    (2, dict(hidden=1152, heads=9, ffn=8008, seq=600, micro_batch=3), dict(w_fc1=("256", 1), w_fc2=("256", 1))),
    (3, dict(hidden=1152, heads=9, ffn=24400, seq=136, micro_batch=1), dict(w_fc1=("persist", 1), w_fc2=("persist", 1))),
    (3, dict(hidden=1152, heads=9, ffn=24400, seq=1000, micro_batch=3), dict(w_fc1=("persist", 1), w_fc2=("persist", 1))),
]


@pytest.mark.parametrize("n,shape,want", SEGMENTED)
def test_segmented_weight_products(n, shape, want):
    """The batched pass against one call per micro-batch (fp32 sums in another
    order: rel <= 1e-6) and against the oracle."""
    from synth.schedules import Op
    cfg = get_config("small_bf16").with_(layers=1, n_mb=n, rerouted=(), **shape)
    assert cfg.tokens % 64
    takes(cfg, n, **want)
    log(f"[segments] n={n} {shape} {want}")
    mbs = [MB(j, 0) for j in range(n)]
    ops = [Op(k, m) for k in ("F", "B") for m in mbs]
    got = {}
    for name, ws in (("one", [Op("W", m) for m in mbs]), ("batch", [Op("W*", mbs)])):
        stage = Stage.from_config(cfg)
        params = gen_params(cfg)
        stage.load_params(params)
        run_gpu(cfg, ops + ws, stage=stage, read_state=False, keep_outputs=False)
        got[name] = stage.read_all(RC_READ_GRAD)
        stage.close()
    for p in range(12):
        assert rel_l2(got["batch"][0][p], got["one"][0][p]) < 1e-6, p
    o = oracle.run_oplist(cfg, ops + [Op("W", m) for m in mbs], params=params)
    log(f"[segments] worst gradient rel-L2 {compare_grads(cfg, got['batch'], o.grads, 2e-2):.2e}")


def test_split_products_are_reproducible():
    """Partials of split reductions are added in a fixed order: the same
    iteration twice gives the same bits."""
    import numpy as np
    cfg = get_config("small_bf16").with_(layers=1, hidden=512, heads=4, ffn=4096, seq=328, n_mb=4, rerouted=())
    a, b = run_gpu(cfg), run_gpu(cfg)
    for mb in a.y:
        assert np.array_equal(a.y[mb], b.y[mb]) and np.array_equal(a.dx[mb], b.dx[mb])
    for p in range(12):
        assert np.array_equal(a.grads[0][p], b.grads[0][p]), p


def test_f32_rows_beyond_buffer_offsets():
    """An fp32 stage whose FFN rows are so wide (8 600 000) that the last of a
    tile's 64 token rows starts 2^31 bytes past its first.  The FFN's weights are
    zero but for 64 columns spread over it, where gelu(0) = 0 leaves the same
    stage as one of 64 FFN columns, which the oracle runs."""
    from synth.schedules import Op
    import numpy as np
    f = 8600000
    cfg = get_config("small_f32").with_(layers=1, hidden=64, heads=1, ffn=64, seq=64, micro_batch=1, n_mb=1, rerouted=())
    log(f"[shape] f32 h=64 s=64 f={f}")
    at = np.linspace(0, f - 1, 64).astype(np.int64)
    params = gen_params(cfg)
    wide = list(params[0])
    wide[8], wide[9], wide[10] = (np.zeros(n, np.float32) for n in ((64, f), (f,), (f, 64)))
    wide[8][:, at], wide[9][at], wide[10][at] = params[0][8], params[0][9], params[0][10]
    stage = Stage.from_config(cfg.with_(ffn=f))
    stage.load_params([wide])
    del wide
    mb = MB(0, 0)
    g = run_gpu(cfg, [Op("F", mb), Op("B", mb), Op("W", mb)], stage=stage, read_state=False)
    o = oracle.run_oplist(cfg, [Op("F", mb), Op("B", mb), Op("W", mb)], params=params)
    grads = [stage.read(RC_READ_GRAD, 0, p) for p in range(12)]
    stage.close()
    assert not np.any(np.delete(grads[9], at))
    grads[8], grads[9], grads[10] = grads[8][:, at], grads[9][at], grads[10][at]
    key = tuple(mb)
    log(f"[shape] f={f}: y {rel_l2(g.y[key], o.y[key]):.2e} dx {rel_l2(g.dx[key], o.dx[key]):.2e}")
    assert rel_l2(g.y[key], o.y[key]) < 1e-5 and rel_l2(g.dx[key], o.dx[key]) < 1e-5
    log(f"[shape] f={f}: worst gradient rel-L2 {compare_grads(cfg, [grads], o.grads, 1e-5):.2e}")
