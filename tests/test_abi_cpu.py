"""CPU checks of the C-ABI library: it loads, exports every symbol the header
declares, validates configurations, and its host bookkeeping (the
micro-batch state machine, stash slots and op log of a dry-run handle)
matches the oracle's on every workload's op list.  No compute call runs here.
"""
import ctypes
import os
import re

import numpy as np
import pytest

import oracle
from synth import CONFIGS, TEST_CONFIGS, MB, gen_params, get_config, op_list

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def lib_or_skip():
    import paper_2405_14009_amd._lib as L
    if not os.path.exists(L.LIB_PATH):
        pytest.skip("library not built (run __graft_entry__.build())")
    return L, L.load()


def header_functions():
    txt = open(os.path.join(ROOT, "include", "recycle_stage.h")).read()
    return set(re.findall(r"^(?:rc_status|const char\*)\s+(rc_\w+)\s*\(", txt, re.M))


def test_library_exports_every_declared_symbol():
    L, lib = lib_or_skip()
    declared = header_functions()
    assert declared == set(L.EXPORTED)
    for name in declared:
        assert hasattr(lib, name), name


def _cfg(**kw):
    import paper_2405_14009_amd._lib as L
    base = dict(num_layers=1, hidden=256, heads=4, ffn=1024, seq_len=128, micro_batch=1, causal=1,
                dtype=L.RC_FP32, ln_eps=1e-5, max_stashed_mb=4, max_inflight_mb=4)
    base.update(kw)
    return L.RcStageConfig(**base)


def _req(cfg):
    L, lib = lib_or_skip()
    a, b, c = ctypes.c_size_t(), ctypes.c_size_t(), ctypes.c_size_t()
    st = lib.rc_stage_memory_requirements(ctypes.byref(cfg), ctypes.byref(a), ctypes.byref(b),
                                          ctypes.byref(c))
    return st, a.value, b.value, c.value


def test_memory_requirements_and_validation():
    L, lib = lib_or_skip()
    st, state, stash, work = _req(_cfg())
    assert st == 0 and state > 0 and stash > 0 and work > 0
    # the stash is max_stashed weight-pass slots + max_inflight forward-only slots
    _, _, stash2, _ = _req(_cfg(max_stashed_mb=8, max_inflight_mb=4))
    _, _, stash3, _ = _req(_cfg(max_stashed_mb=8, max_inflight_mb=8))
    wslot = (stash2 - stash) // 4
    fslot = (stash3 - stash2) // 4
    h, f, T, a, s = 256, 1024, 128, 4, 128
    assert wslot >= 4 * (12 * T * h + 2 * T * f) and wslot < 4 * (12 * T * h + 2 * T * f) + 64 * 1024
    assert fslot >= 4 * (3 * T * h + T * f + a * s * s)
    assert _req(_cfg(hidden=250, heads=5))[0] == L.RC_ERR_UNSUPPORTED      # head_dim 50
    assert _req(_cfg(hidden=256, heads=3))[0] == L.RC_ERR_UNSUPPORTED
    assert _req(_cfg(seq_len=100))[0] == L.RC_ERR_UNSUPPORTED
    assert _req(_cfg(dtype=7))[0] == L.RC_ERR_INVALID_ARG
    assert _req(_cfg(max_inflight_mb=5))[0] == L.RC_ERR_INVALID_ARG
    assert _req(_cfg(num_layers=0))[0] == L.RC_ERR_INVALID_ARG
    assert lib.rc_stage_memory_requirements(None, None, None, None) == L.RC_ERR_INVALID_ARG
    assert b"null" in lib.rc_last_error()


def test_bf16_configs_beyond_the_descriptor_range_are_refused():
    """bf16 matrices are read through buffer descriptors of 2^31 - 1 bytes
    (a load beyond returns zeros), so a configuration with a larger operand
    is refused up front instead of computing on zeros."""
    L, lib = lib_or_skip()
    big = dict(dtype=L.RC_BF16, hidden=4096, heads=32, ffn=16384, seq_len=2048, max_stashed_mb=1,
               max_inflight_mb=1)
    # the 6.7B-shaped stage is accepted: 2 * 2048 * 16384 bytes per activation matrix
    assert _req(_cfg(**big, micro_batch=1))[0] == L.RC_OK
    # T * max(3h, f) * 2 bytes = 2^31 exactly (one past the range) is refused ...
    st = _req(_cfg(**big, micro_batch=32))[0]
    assert st == L.RC_ERR_UNSUPPORTED and b"activation" in lib.rc_last_error()
    # ... one token-block less fits (T = 63 * 1024: 2 * 64512 * 16384 < 2^31 - 1)
    assert _req(_cfg(**dict(big, seq_len=1024), micro_batch=63))[0] == L.RC_OK
    # the largest weight, hidden x ffn x 2 bytes = 2^31
    st = _req(_cfg(dtype=L.RC_BF16, hidden=16384, heads=128, ffn=65536, seq_len=8,
                   max_stashed_mb=1, max_inflight_mb=1))[0]
    assert st == L.RC_ERR_UNSUPPORTED and b"weight" in lib.rc_last_error()
    # one head's materialised probabilities (head_dim 64: no fused attention), 2 s^2 bytes
    st = _req(_cfg(dtype=L.RC_BF16, hidden=256, heads=4, ffn=256, seq_len=32768, max_stashed_mb=1,
                   max_inflight_mb=1))[0]
    assert st == L.RC_ERR_UNSUPPORTED and b"probabilities" in lib.rc_last_error()
    assert _req(_cfg(dtype=L.RC_BF16, hidden=256, heads=4, ffn=256, seq_len=32760, max_stashed_mb=1,
                     max_inflight_mb=1))[0] == L.RC_OK
    # fp32 stages do not use the descriptors
    assert _req(_cfg(**dict(big, dtype=L.RC_FP32), micro_batch=32))[0] == L.RC_OK


def test_static_work_entry_point_checks_its_limit_and_arenas():
    """rc_stage_create_static refuses a configuration whose work memory
    exceeds RC_STATIC_WORK_BYTES before touching any device, and needs the
    caller's two arenas (no dry run)."""
    L, lib = lib_or_skip()
    out = ctypes.c_void_p()
    adam = L.RcAdamConfig(1e-4, 0.9, 0.95, 1e-8, 0.1)
    big = _cfg(dtype=L.RC_BF16, num_layers=4, hidden=4096, heads=32, ffn=16384, seq_len=2048,
               max_stashed_mb=32, max_inflight_mb=1)
    assert _req(big)[3] > L.RC_STATIC_WORK_BYTES
    st = lib.rc_stage_create_static(ctypes.byref(big), ctypes.byref(adam), 0, 0, None, None, None,
                                    ctypes.byref(out))
    assert st == L.RC_ERR_UNSUPPORTED and b"work memory" in lib.rc_last_error()
    ok = _cfg(dtype=L.RC_BF16, num_layers=4, hidden=4096, heads=32, ffn=16384, seq_len=2048,
              max_stashed_mb=16, max_inflight_mb=16)
    assert _req(ok)[3] <= L.RC_STATIC_WORK_BYTES   # the 6.7B-shaped stage fits
    st = lib.rc_stage_create_static(ctypes.byref(ok), ctypes.byref(adam), 0, 0, None, None, None,
                                    ctypes.byref(out))
    assert st == L.RC_ERR_INVALID_ARG and not out.value


def test_attention_kernel_query_on_dry_run_handles():
    lib_or_skip()
    from paper_2405_14009_amd import Stage
    kw = dict(num_layers=1, ffn=256, micro_batch=1, dry_run=True)
    assert Stage(hidden=256, heads=4, seq_len=128, dtype="f32", **kw).attention_kernels() == "materialised"
    assert Stage(hidden=256, heads=4, seq_len=128, dtype="bf16", **kw).attention_kernels() == "materialised"
    # a small grid (at most one workgroup of 32 queries per compute unit, two for narrow heads)
    for causal in (True, False):
        assert Stage(hidden=256, heads=2, seq_len=128, dtype="bf16", causal=causal, **kw).attention_kernels() == "split"
        for heads, d, seq, kind in ((4, 128, 2048, "split"), (8, 64, 2048, "split"), (8, 64, 2056, "block")):
            assert Stage(hidden=heads * d, heads=heads, seq_len=seq, dtype="bf16", causal=causal,
                         **kw).attention_kernels() == kind, (heads, d, seq, causal)
    # 256 pairs of query blocks: one per compute unit; 96 heads of 8 pairs: three rounds
    kw["ffn"] = 64
    for heads, seq, causal, kind in ((32, 2048, True, "paired"), (32, 2048, False, "block"), (40, 2048, True, "block"),
                                     (96, 2048, True, "block"), (30, 2048, True, "paired")):
        assert Stage(hidden=128 * heads, heads=heads, seq_len=seq, dtype="bf16", causal=causal,
                     **kw).attention_kernels() == kind, (heads, seq, causal)


def test_bf16_state_holds_weight_copies():
    L, _ = lib_or_skip()
    _, s32, _, _ = _req(_cfg(dtype=L.RC_FP32))
    _, s16, _, _ = _req(_cfg(dtype=L.RC_BF16))
    n_mat = 4 * 256 * 256 + 2 * 256 * 1024
    assert s16 - s32 >= 2 * n_mat


def _drive(stage, ops):
    for op in ops:
        if op.kind == "F":
            stage.forward(op.mb)
        elif op.kind == "B":
            stage.backward_input(op.mb)
        elif op.kind == "W":
            stage.backward_weight(op.mb)
        else:
            stage.optimizer_step()


@pytest.mark.parametrize("name", list(CONFIGS) + list(TEST_CONFIGS))
def test_dry_run_op_log_matches_oracle(name):
    lib_or_skip()
    from paper_2405_14009_amd import Stage
    cfg = get_config(name)
    ops = op_list(cfg) * 2   # two iterations
    st = Stage.from_config(cfg, dry_run=True, stage_index=3, pipeline_id=0)
    _drive(st, ops)
    ref = oracle_bookkeeping(cfg, ops)
    assert st.op_log() == [(r[0], r[1], r[2], r[3], r[4], r[5]) for r in ref]


def oracle_bookkeeping(cfg, ops):
    """The oracle's state machine on the same op list, with the compute
    replaced by no-ops (tiny placeholder tensors)."""
    o = oracle.OracleStage(cfg.with_(layers=0), [], pipeline_id=0)
    for op in ops:
        if op.kind == "F":
            o.forward(op.mb, np.zeros((1, 1, 1)))
        elif op.kind == "B":
            o.backward_input(op.mb, np.zeros((1, 1, 1)))
        elif op.kind == "W":
            o.backward_weight(op.mb)
        else:
            o.optimizer_step()
    return [tuple(r) for r in o.log]


def test_dry_run_error_table_matches_oracle():
    lib_or_skip()
    import paper_2405_14009_amd as P
    cfg = get_config("tiny").with_(n_mb=3, max_stashed_mb=2, max_inflight_mb=1)
    st = P.Stage.from_config(cfg, dry_run=True)
    o = oracle.OracleStage(cfg.with_(layers=0), [])
    z = np.zeros((1, 1, 1))
    m0, m1, m2 = MB(0), MB(1), MB(2)
    seq = [("B", m0), ("W", m0), ("F", m0), ("F", m0), ("W", m0), ("F", m1), ("B", m0),
           ("B", m0), ("F", m1), ("F", m2), ("STEP", None), ("W", m0), ("W", m0), ("F", m0),
           ("B", m1), ("W", m1), ("STEP", None), ("F", m0)]
    codes = {P.BadStateError: "BAD_STATE", P.OutOfStashError: "OUT_OF_STASH"}
    for kind, mb in seq:
        got = want = "OK"
        try:
            {"F": lambda: st.forward(mb), "B": lambda: st.backward_input(mb),
             "W": lambda: st.backward_weight(mb), "STEP": st.optimizer_step}[kind]()
        except (P.BadStateError, P.OutOfStashError) as e:
            got = codes[type(e)]
        try:
            {"F": lambda: o.forward(mb, z), "B": lambda: o.backward_input(mb, z),
             "W": lambda: o.backward_weight(mb), "STEP": o.optimizer_step}[kind]()
        except oracle.StageError as e:
            want = e.code
        assert got == want, (kind, mb)
        assert st.stash_usage() == (o._n_stashed(), o._n_inflight())
    assert st.op_log() == [tuple(r) for r in o.log]


def group_w(ops):
    """Consecutive W ops of an op list merged into one batched weight pass."""
    out = []
    for op in ops:
        if op.kind == "W" and out and out[-1][0] == "W*" and len(out[-1][1]) < 32:
            out[-1][1].append(op.mb)
        elif op.kind == "W":
            out.append(("W*", [op.mb]))
        else:
            out.append((op.kind, op.mb))
    return out


@pytest.mark.parametrize("name", list(CONFIGS) + list(TEST_CONFIGS))
def test_dry_run_batched_weight_pass_logs_like_single_calls(name):
    lib_or_skip()
    from paper_2405_14009_amd import Stage
    cfg = get_config(name)
    ops = op_list(cfg) * 2
    st = Stage.from_config(cfg, dry_run=True, stage_index=3, pipeline_id=0)
    for kind, arg in group_w(ops):
        if kind == "W*":
            st.backward_weight_many(arg)
        elif kind == "F":
            st.forward(arg)
        elif kind == "B":
            st.backward_input(arg)
        else:
            st.optimizer_step()
    ref = oracle_bookkeeping(cfg, ops)
    assert st.op_log() == [(r[0], r[1], r[2], r[3], r[4], r[5]) for r in ref]


def test_dry_run_batched_weight_pass_errors_are_all_or_nothing():
    lib_or_skip()
    import paper_2405_14009_amd as P
    cfg = get_config("tiny").with_(n_mb=4, max_stashed_mb=4, max_inflight_mb=4)
    st = P.Stage.from_config(cfg, dry_run=True)
    for j in range(3):
        st.forward(MB(j))
    st.backward_input(MB(0))
    st.backward_input(MB(1))
    log0 = st.op_log()
    # MB 2 has not run B: nothing happens to MB 0 and 1 either
    with pytest.raises(P.BadStateError):
        st.backward_weight_many([MB(0), MB(1), MB(2)])
    with pytest.raises(P.BadStateError):
        st.backward_weight_many([MB(0), MB(0)])
    with pytest.raises(P.InvalidArgError):
        st.backward_weight_many([])
    assert st.op_log() == log0
    assert st.stash_usage() == (3, 1)
    st.backward_weight_many([MB(1), MB(0)])
    assert [(r[1], r[2]) for r in st.op_log()[len(log0):]] == [(2, 1), (2, 0)]
    assert st.stash_usage() == (1, 1)
    with pytest.raises(P.BadStateError):
        st.backward_weight_many([MB(0)])


def test_dry_run_skip_and_rollback_rules_match_oracle():
    """Post-step validation calls: the same accept / refuse decisions and op
    log as the oracle over a sequence that exercises every rule."""
    lib_or_skip()
    import paper_2405_14009_amd as P
    cfg = get_config("tiny").with_(n_mb=2, max_stashed_mb=2, max_inflight_mb=2)
    st = P.Stage.from_config(cfg, dry_run=True)
    o = oracle.OracleStage(cfg.with_(layers=0), [])
    z = np.zeros((1, 1, 1))
    m0, m1 = MB(0), MB(1)
    seq = [("ROLLBACK", None), ("F", m0), ("SKIP", None), ("B", m0), ("W", m0), ("SKIP", None),
           ("ROLLBACK", None), ("F", m0), ("B", m0), ("W", m0), ("STEP", None), ("ROLLBACK", None),
           ("ROLLBACK", None), ("STEP", None), ("ROLLBACK", None), ("STEP", None), ("F", m1),
           ("ROLLBACK", None), ("B", m1), ("W", m1), ("STEP", None), ("SKIP", None),
           ("ROLLBACK", None)]
    for kind, mb in seq:
        got = want = "OK"
        try:
            {"F": lambda: st.forward(mb), "B": lambda: st.backward_input(mb),
             "W": lambda: st.backward_weight(mb), "STEP": st.optimizer_step,
             "SKIP": st.optimizer_skip, "ROLLBACK": st.optimizer_rollback}[kind]()
        except P.BadStateError:
            got = "BAD_STATE"
        try:
            {"F": lambda: o.forward(mb, z), "B": lambda: o.backward_input(mb, z),
             "W": lambda: o.backward_weight(mb), "STEP": o.optimizer_step,
             "SKIP": o.optimizer_skip, "ROLLBACK": o.optimizer_rollback}[kind]()
        except oracle.StageError as e:
            want = e.code
        assert got == want, (kind, mb)
    assert st.op_log() == [tuple(r) for r in o.log]


def _fused(cfg):
    return cfg.dtype == "bf16" and cfg.hidden // cfg.heads == 128


@pytest.mark.parametrize("name", list(CONFIGS) + list(TEST_CONFIGS))
def test_stash_accounting_matches_oracle(name):
    """a_f / s_w equal the oracle's analytic counts; live and peak after every
    op of two iterations of the workload's op list equal the oracle's."""
    lib_or_skip()
    from paper_2405_14009_amd import Stage
    cfg = get_config(name)
    st = Stage.from_config(cfg, dry_run=True)
    o = oracle.OracleStage(cfg.with_(layers=0), [])
    o.a_f, o.s_w = oracle.stash_bytes(cfg, _fused(cfg))
    acct = st.stash_account()
    assert (acct["a_f"], acct["s_w"]) == (o.a_f, o.s_w)
    z = np.zeros((1, 1, 1))
    for op in op_list(cfg) * 2:
        if op.kind == "F":
            st.forward(op.mb); o.forward(op.mb, z)
        elif op.kind == "B":
            st.backward_input(op.mb); o.backward_input(op.mb, z)
        elif op.kind == "W":
            st.backward_weight(op.mb); o.backward_weight(op.mb)
        else:
            st.optimizer_step(); o.optimizer_step()
        a = st.stash_account()
        assert (a["live"], a["peak"]) == (o.live, o.peak), op
    assert st.stash_account()["live"] == 0


def test_stash_byte_formulas_pinned_by_the_oracles_arrays():
    """The element terms of a_f and s_w equal the sizes of the arrays the
    oracle's own decoupled backward keeps (its forward cache and its
    weight-pass stash), which are chosen by what the passes read, not by the
    formula: cache = 8 T h + 2 T f + attention probabilities (+ the LN rstd);
    weight stash = 12 T h + 2 T f."""
    from oracle import stage as ost
    cfg = get_config("tiny").with_(layers=2, micro_batch=2, seq=16, hidden=64, heads=2, ffn=128,
                                   dtype="f32")
    params = [[p.astype(np.float64) for p in layer] for layer in gen_params(cfg)]
    from synth import gen_dy, gen_x
    x = gen_x(cfg, 0).astype(np.float64)
    shp = ost.LayerShape(cfg.heads, cfg.causal, cfg.ln_eps)
    y, caches = ost.stage_forward(x, params, shp)
    dx, stashes = ost.stage_backward_input(gen_dy(cfg, 0).astype(np.float64), caches, params)
    T, h, f = cfg.micro_batch * cfg.seq, cfg.hidden, cfg.ffn
    probs = cfg.micro_batch * cfg.heads * cfg.seq * cfg.seq
    for c, w in zip(caches, stashes):
        kept = sum(v.size for k, v in c.items() if k not in ("p", "r1", "r2"))
        assert kept == 8 * T * h + 2 * T * f
        assert c["p"].size == probs and c["r1"].size + c["r2"].size == 2 * T
        assert sum(v.size for v in w.values()) == 12 * T * h + 2 * T * f
    a_f, s_w = oracle.stash_bytes(cfg, False)
    assert a_f == cfg.layers * (4 * (8 * T * h + 2 * T * f) + 16 * T + 4 * probs)
    assert s_w == cfg.layers * (4 * (12 * T * h + 2 * T * f) + 16 * T)


def test_stash_limit_refusal_matches_oracle():
    lib_or_skip()
    import paper_2405_14009_amd as P
    cfg = get_config("gpt1.3b")
    st = P.Stage.from_config(cfg, dry_run=True)
    o = oracle.OracleStage(cfg.with_(layers=0), [])
    o.a_f, o.s_w = oracle.stash_bytes(cfg, _fused(cfg))
    with pytest.raises(P.InvalidArgError):
        st.set_stash_limit(o.a_f - 1)
    limit = 3 * o.a_f + o.s_w
    st.set_stash_limit(limit)
    o.set_stash_limit(limit)
    z = np.zeros((1, 1, 1))
    for op in op_list(cfg):
        if op.kind == "STEP":
            break
        got = want = "OK"
        fn = {"F": (lambda: st.forward(op.mb), lambda: o.forward(op.mb, z)),
              "B": (lambda: st.backward_input(op.mb), lambda: o.backward_input(op.mb, z)),
              "W": (lambda: st.backward_weight(op.mb), lambda: o.backward_weight(op.mb))}[op.kind]
        try:
            fn[0]()
        except (P.OutOfStashError, P.BadStateError) as e:
            got = type(e).__name__
        try:
            fn[1]()
        except oracle.StageError as e:
            want = {"OUT_OF_STASH": "OutOfStashError", "BAD_STATE": "BadStateError"}[e.code]
        assert got == want, op
    assert st.op_log() == [tuple(r) for r in o.log]


@pytest.mark.parametrize("name,slots", [("gpt6.7b", 6), ("gpt6.7b", 1), ("gpt1.3b", 1),
                                        ("gpt13b", 2), ("gpt6.7b", 0)])
def test_executor_keeps_the_stash_within_the_limit(name, slots):
    """Selective decoupling: with a stash limit the executor couples or runs
    weight passes early so the stash never exceeds it; every micro-batch still
    runs F, B, W exactly once, in dependency order."""
    lib_or_skip()
    from paper_2405_14009_amd import RC_OP_B, RC_OP_F, RC_OP_W, Stage
    from paper_2405_14009_amd.executor import execute
    cfg = get_config(name)
    st = Stage.from_config(cfg, dry_run=True)
    a = st.stash_account()
    # room for the schedule's warm-up forwards plus `slots` deferred weight stashes
    limit = (cfg.warmup + 1) * a["a_f"] + slots * a["s_w"] if slots else 0
    rep = execute(st, op_list(cfg) * 2, stash_limit=limit)
    if limit:
        assert rep.peak <= limit
    else:
        assert not rep.coupled and not rep.flushed
    log = st.op_log()
    for it in (0, 1):
        seen = {}
        for r in log:
            if r[5] != it or r[1] not in (RC_OP_F, RC_OP_B, RC_OP_W):
                continue
            seen.setdefault((r[2], r[3]), []).append(r[1])
        assert all(v == [RC_OP_F, RC_OP_B, RC_OP_W] for v in seen.values()), seen
        assert len(seen) == cfg.n_mb
    if slots == 1:
        assert rep.coupled or rep.flushed


def test_executor_reports_an_infeasible_limit():
    """A limit below the schedule's warm-up activations cannot be met by any
    choice of coupling: the forward is refused (no state change)."""
    lib_or_skip()
    import paper_2405_14009_amd as P
    from paper_2405_14009_amd.executor import execute
    cfg = get_config("gpt6.7b")
    st = P.Stage.from_config(cfg, dry_run=True)
    a = st.stash_account()
    with pytest.raises(P.OutOfStashError):
        execute(st, op_list(cfg), stash_limit=2 * a["a_f"] + a["s_w"])
    assert st.stash_account()["live"] <= 2 * a["a_f"] + a["s_w"]


def test_product_fails_loudly_without_gpu():
    lib_or_skip()
    import torch
    if torch.cuda.is_available():
        pytest.skip("a GPU is present")
    import paper_2405_14009_amd as P
    with pytest.raises(RuntimeError, match="no HIP device"):
        P.Stage.from_config(get_config("tiny"))
