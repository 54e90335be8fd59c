"""Host-only checks of the C ABI (no GPU needed): the library loads, exports
every symbol include/psw.h declares, and the stage scheduler's dry run
(psw_net_plan) follows the stale-weight schedule and rejects bad input."""
import ctypes
import os
import re

import numpy as np
import pytest
import torch

from paper_1912_12675_amd import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "psw.h")


@pytest.fixture(scope="module")
def psw():
    from paper_1912_12675_amd import psw as P
    if not os.path.exists(P.LIB_PATH):
        pytest.fail("libpsw.so is not built (python -m paper_1912_12675_amd.build)")
    P.lib()
    return P


def declared_symbols():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(psw_[a-z0-9_]+)\s*\(", text)))


def test_calls_without_the_native_module(psw, monkeypatch):
    """With libpsw.so alone every per-layer call is left to ctypes, after one warning."""
    import sys

    monkeypatch.setattr(psw, "_fast", None)
    monkeypatch.setitem(sys.modules, "paper_1912_12675_amd._fastcall", None)  # the import fails
    monkeypatch.delattr(sys.modules["paper_1912_12675_amd"], "_fastcall", raising=False)
    t = torch.zeros(4)
    with pytest.warns(RuntimeWarning, match="ctypes"), pytest.raises(ValueError, match="device tensors"):
        psw.psw_relu_mask(t, t)
    with pytest.raises(ValueError, match="device tensors"):
        psw.psw_sgd_momentum_step(t, t, t, t, 0.1)


def test_header_symbols_exported(psw):
    syms = declared_symbols()
    assert len(syms) >= 25
    L = ctypes.CDLL(psw.LIB_PATH)
    missing = [s for s in syms if not hasattr(L, s)]
    assert not missing, missing
    # the binding covers the whole surface, with the header's names
    assert sorted(psw.SIGNATURES) == syms


def test_version_and_error_string(psw):
    assert b"gfx950" in psw.lib().psw_version()
    rc = psw.lib().psw_conv_fwd(0, 1, 1, 1, 1, 1, 1, 1, 0, None, None, None, 0, None, 0, None)
    assert rc == -2
    assert b"positive" in psw.lib().psw_last_error()
    rc = psw.lib().psw_conv_fwd(1, 1, 4, 4, 1, 3, 3, 1, 1, None, None, None, 0, None, 0, None)
    assert rc == -1
    rc = psw.lib().psw_conv_fwd(1, 1, 4, 4, 1, 3, 3, 1, 1, 8, 8, None, 0, 8, 7, None)
    assert rc == -3  # unknown precision
    rc = psw.lib().psw_pool_fwd(0, 1, 1, 8, 8, 3, 2, 8, 8, 8, None)
    assert rc == -3  # overlapping windows are not supported
    rc = psw.lib().psw_sgd_momentum_step(10, 1000, 1004, 8, 8, 0.1, 0.9, 0.0, 0, None)
    assert rc == -2  # partial overlap of w_in / w_out


def _plan(psw, wl, t, staleness, ring=None):
    ring = wl.ring_depth() if ring is None else ring
    return psw.net_plan_only(wl.ops, wl.batch, wl.in_shape, wl.stage_end, ring, t, staleness)


def test_plan_versions_follow_schedule(psw):
    wl = synth.resnet20_workload(batch=4)
    S = wl.n_stages
    stage_of = np.zeros(len(wl.ops), dtype=int)
    prev = 0
    for s, e in enumerate(wl.stage_end):
        stage_of[prev:e] = s
        prev = e
    for t in range(0, 9):
        d = [3, 2, 1, 0]
        plan = _plan(psw, wl, t, d)
        fwd = [p for p in plan if p[1] in (1, 2, 4)]           # conv / bn / fc forward
        bwd = [p for p in plan if p[1] in (8, 9, 11, 15)]      # bwd-data / bn bwd (folded) / fc bwd
        sgd = [p for p in plan if p[1] == 12]
        for op, what, stage, ver in fwd:
            assert stage == stage_of[op]
            assert ver == max(0, t - d[stage])                  # forward reads version t - d_s
        assert all(ver == t for _, _, _, ver in bwd)            # backward reads the current version
        assert [(s, v) for _, _, s, v in sgd] == [(s, t) for s in reversed(range(S))]
    # order: every forward before the loss, every backward after it; stage s
    # is updated right after the backward pass is done with it (its last
    # backward operation), before any backward operation of stage s-1
    plan = _plan(psw, wl, 5, [3, 2, 1, 0])
    kinds = [p[1] for p in plan]
    li = kinds.index(5)
    assert all(k in (1, 2, 3, 4) for k in kinds[:li])
    assert all(k not in (1, 2, 3, 4) for k in kinds[li + 1:])
    back = plan[li + 1:]
    for s in range(S):
        u = next(j for j, p in enumerate(back) if p[1] == 12 and p[2] == s)
        assert all(p[2] != s for p in back[u + 1:] if p[1] != 12)
        assert all(p[2] == s or p[1] == 12 for p in back[u - 1:u]) and all(p[2] != s - 1 for p in back[:u])
    assert kinds[-1] == 12
    # 19 conv forwards, 19 wgrads, 18 dgrads (none for the stem) in ResNet-20
    assert kinds.count(1) == 19 and kinds.count(7) == 19 and kinds.count(8) == 18


def test_plan_weight_stashing(psw):
    """With weight stashing on, the backward records read the forward's
    version r_s; forward records and updates are unchanged."""
    wl = synth.resnet20_workload(batch=4)
    d = [3, 2, 1, 0]
    for t in (0, 2, 7):
        base = _plan(psw, wl, t, d)
        st = psw.net_plan_only(wl.ops, 4, wl.in_shape, wl.stage_end, wl.ring_depth(20), t, d, stash=True)
        assert len(st) == len(base)
        for (o1, w1, s1, v1), (o2, w2, s2, v2) in zip(base, st):
            assert (o1, w1, s1) == (o2, w2, s2)
            if w1 in (8, 9, 11, 15):
                assert v1 == t and v2 == max(0, t - d[s1])
            else:
                assert v1 == v2
    with pytest.raises(psw.PswError) as e:
        psw._check(psw.lib().psw_net_set_weight_stashing(None, 1))
    assert e.value.code == -1


def test_plan_dropout_records(psw):
    """Dropout ops appear in the plan as a forward record after their input's
    producer and a backward record in reverse order, reading no weights."""
    wl = synth.vgg16_workload(batch=2, dropout=0.3)
    plan = psw.net_plan_only(wl.ops, 2, wl.in_shape, wl.stage_end, [4, 3, 2, 1], 5, [3, 2, 1, 0])
    drop_ops = [i for i, o in enumerate(wl.ops) if int(o[0]) == synth.DROPOUT]
    fwd = [(op, v) for op, what, _, v in plan if what == 13]
    bwd = [(op, v) for op, what, _, v in plan if what == 14]
    assert [op for op, _ in fwd] == drop_ops and all(v == -1 for _, v in fwd)
    assert [op for op, _ in bwd] == drop_ops[::-1] and all(v == -1 for _, v in bwd)
    # a bad threshold is rejected when the net is created
    ops = np.array(wl.ops).copy()
    ops[drop_ops[0], 5] = 1 << 24
    with pytest.raises(psw.PswError):
        psw.net_plan_only(ops, 2, wl.in_shape, wl.stage_end, [4, 3, 2, 1], 5, [3, 2, 1, 0])


def test_plan_rejects_bad_staleness(psw):
    wl = synth.resnet20_workload(batch=4)
    with pytest.raises(psw.PswError) as e:
        _plan(psw, wl, 3, [4, 2, 1, 0])        # ring depth of stage 0 is 4
    assert e.value.code == -4
    with pytest.raises(psw.PswError) as e:
        _plan(psw, wl, 3, [0, 0, 0, -1])
    assert e.value.code == -4
    with pytest.raises(psw.PswError) as e:
        _plan(psw, wl, -1, [0, 0, 0, 0])
    assert e.value.code == -5
    # a deeper ring accepts more staleness
    assert _plan(psw, wl, 3, [6, 4, 2, 0], ring=[7, 5, 3, 1])


def test_net_create_rejects_bad_descriptions(psw):
    ops, le, ins = synth.resnet_cifar(20)
    L = psw.lib()

    def create(o, se, rd, batch=2, shape=ins):
        layers = psw._layers(o)
        se = np.ascontiguousarray(se, dtype=np.int32)
        rd = np.ascontiguousarray(rd, dtype=np.int32)
        h = ctypes.c_void_p()
        rc = L.psw_net_create(layers, len(layers), batch, *shape, se.ctypes.data, len(se), rd.ctypes.data, 0,
                              ctypes.byref(h))
        if rc == 0:
            L.psw_net_destroy(h.value)
        return rc

    assert create(ops, [len(ops)], [1]) == 0
    assert create(ops, [10, 5, len(ops)], [1, 1, 1]) == -2          # stage ends not increasing
    assert create(ops, [len(ops) - 1], [1]) == -2                   # last stage must end at n_ops
    assert create(ops, [len(ops)], [0]) == -2                       # ring depth >= 1
    bad = ops.copy()
    bad[0][3] = 4                                                   # conv cin != input channels
    assert create(bad, [len(ops)], [1]) == -2
    bad = ops.copy()
    bad[-1][3] = 65                                                 # fc input features
    assert create(bad, [len(ops)], [1]) == -2
    lops, _, _ = synth.lenet5()
    assert create(lops, [len(lops)], [1], shape=(1, 28, 28)) == 0
    assert create(lops, [len(lops)], [1], shape=(1, 32, 32)) == -2  # fc1 would see 16*6*6 features, not 400
    assert create(lops, [len(lops)], [1], shape=(1, 3, 3)) == -2    # 5x5 kernel larger than the input


def test_net_sizes_match_oracle(psw, oracle):
    for wl in (synth.resnet20_workload(batch=2), synth.lenet5_workload(batch=2), synth.vgg16_workload(batch=2)):
        counts = oracle.param_counts(wl.ops, wl.in_shape, wl.batch, wl.stage_end)
        layers = psw._layers(wl.ops)
        se = np.ascontiguousarray(wl.stage_end, dtype=np.int32)
        rd = np.ascontiguousarray(wl.ring_depth(), dtype=np.int32)
        h = ctypes.c_void_p()
        L = psw.lib()
        assert L.psw_net_create(layers, len(layers), wl.batch, *wl.in_shape, se.ctypes.data, len(se), rd.ctypes.data,
                                0, ctypes.byref(h)) == 0
        sp = np.zeros(len(se), dtype=np.int64)
        rf, npar, nbn, ab = (ctypes.c_int64() for _ in range(4))
        assert L.psw_net_sizes(h.value, sp.ctypes.data, ctypes.byref(rf), ctypes.byref(npar), ctypes.byref(nbn),
                               ctypes.byref(ab)) == 0
        assert list(sp) == list(counts)
        assert rf.value == int(sum(c * d for c, d in zip(counts, rd)))
        layout, _ = synth.param_layout(wl)
        for op in range(len(wl.ops)):
            st, off, cnt = ctypes.c_int(), ctypes.c_int64(), ctypes.c_int64()
            assert L.psw_net_param_offset(h.value, op, ctypes.byref(st), ctypes.byref(off), ctypes.byref(cnt)) == 0
            mine = [(s, o, int(np.prod(shape))) for (i, _, shape, s, o) in layout if i == op]
            if mine:
                assert (st.value, off.value) == mine[0][:2]
                assert cnt.value == sum(m[2] for m in mine)
            else:
                assert cnt.value == 0
        L.psw_net_destroy(h.value)


def test_stage_step_requires_binding(psw):
    wl = synth.resnet20_workload(batch=2)
    L = psw.lib()
    layers = psw._layers(wl.ops)
    se = np.ascontiguousarray(wl.stage_end, dtype=np.int32)
    rd = np.ascontiguousarray(wl.ring_depth(), dtype=np.int32)
    h = ctypes.c_void_p()
    assert L.psw_net_create(layers, len(layers), 2, *wl.in_shape, se.ctypes.data, 4, rd.ctypes.data, 0,
                            ctypes.byref(h)) == 0
    st = np.zeros(4, dtype=np.int32)
    lr = np.full(4, 0.01, dtype=np.float32)
    rc = L.psw_stage_step(h.value, 0, st.ctypes.data, lr.ctypes.data, 0.9, 0.0, 0, 8, 8, 8, None, None)
    assert rc == -8
    p = ctypes.c_void_p()
    assert L.psw_net_slot(h.value, 0, 0, ctypes.byref(p)) == -8
    L.psw_net_destroy(h.value)


def test_profile_replay_argument_checks(psw):
    """The replay setting refuses a NULL net and a count outside [1, 1000]
    (host only, nothing launched)."""
    wl = synth.resnet20_workload(batch=2)
    L = psw.lib()
    layers = psw._layers(wl.ops)
    se = np.ascontiguousarray(wl.stage_end, dtype=np.int32)
    rd = np.ascontiguousarray(wl.ring_depth(), dtype=np.int32)
    h = ctypes.c_void_p()
    assert L.psw_net_create(layers, len(layers), 2, *wl.in_shape, se.ctypes.data, 4, rd.ctypes.data, 0,
                            ctypes.byref(h)) == 0
    assert L.psw_net_profile_replay(None, 2) == -1
    assert L.psw_net_profile_replay(h.value, 0) == -2
    assert L.psw_net_profile_replay(h.value, 1001) == -2
    assert L.psw_net_profile_replay(h.value, 20) == 0
    assert L.psw_net_profile_replay(h.value, 1) == 0
    L.psw_net_destroy(h.value)



def conv_residual_workload(batch=4):
    """A residual block whose BN adds the block conv's own input
    (x -> conv -> BN(+x) -> ReLU), between two ordinary conv + BN layers,
    then pool and classifier: 16 channels at 32x32, one stage."""
    b = synth._Builder()
    t = b.add(synth.CONV, 0, 3, 16, 3, 1, 1)
    x = b.add(synth.BN, t, 16, 16, flags=synth.F_RELU)
    b.end_layer()
    t = b.add(synth.CONV, x, 16, 16, 3, 1, 1)
    t = b.add(synth.BN, t, 16, 16, flags=synth.F_RELU, in1=x)
    b.end_layer()
    t = b.add(synth.CONV, t, 16, 16, 3, 1, 1)
    t = b.add(synth.BN, t, 16, 16, flags=synth.F_RELU)
    b.end_layer()
    t = b.add(synth.GAVG, t, 16, 16)
    b.add(synth.FC, t, 16, 10, flags=synth.F_BIAS)
    b.end_layer()
    return synth.Workload("conv_residual", b.desc(), (3, 32, 32), 10, batch, b.layer_end, [len(b.ops)],
                          lambda t: [0], 4, [0.01], seed=1918)


def test_plan_reports_folded_bn_backward(psw):
    """ResNet-20 folds 13 of its 19 BN backward passes (7 without residual,
    6 with an identity residual) into the backward-data kernels around
    them; the plan records them as folded."""
    wl = synth.resnet20_workload(batch=8)
    plan = _plan(psw, wl, 3, [3, 2, 1, 0])
    folded = [p[0] for p in plan if p[1] == 15]
    plain = [p[0] for p in plan if p[1] == 9]
    assert len(folded) == 13 and len(plain) == 6
    assert sum(1 for i in folded if wl.ops[i][2] >= 0) == 6


def test_plan_no_fold_when_residual_is_the_conv_input(psw):
    """x -> conv -> BN(+x): folding this BN would make the backward-data
    kernel write the residual's gradient (the conv's own input gradient)
    in some workgroups while others still read it, so it is not folded.
    """
    wl = conv_residual_workload()
    plan = _plan(psw, wl, 0, [0])
    bn_bwd = {p[0]: p[1] for p in plan if p[1] in (9, 15)}
    # every other fold condition holds for op 3 (identity residual written
    # first, stride-1 direct conv before it in the same stage, a conv after
    # it whose backward-data kernel forms its sums): only the aliasing
    # keeps it from being folded
    assert bn_bwd[3] == 9


def _unstored(psw, wl):
    L = psw.lib()
    layers = psw._layers(wl.ops)
    se = np.ascontiguousarray(wl.stage_end, dtype=np.int32)
    rd = np.ascontiguousarray(wl.ring_depth(), dtype=np.int32)
    h = ctypes.c_void_p()
    psw._check(L.psw_net_create(layers, len(layers), wl.batch, *wl.in_shape, se.ctypes.data, len(se), rd.ctypes.data,
                                psw._prec(wl.bf16), ctypes.byref(h)))
    try:
        out = []
        for k in range(1, len(layers) + 1):
            st = ctypes.c_int()
            psw._check(L.psw_net_tensor_stored(h.value, k, ctypes.byref(st)))
            if not st.value:
                out.append(k)
        for bad in (0, len(layers) + 1):
            assert L.psw_net_tensor_stored(h.value, bad, ctypes.byref(st)) != 0
        return out
    finally:
        L.psw_net_destroy(h.value)


def test_bn_applied_on_load_only_where_nothing_else_reads_it(psw):
    """The BN + ReLU before a residual block's second conv (one per block:
    its output has that conv as its only reader, no residual, statistics
    from the conv before it) is applied by the conv while loading, so its
    output is not stored; block outputs (BN with the residual, read by the
    next block's conv and by the shortcut) and the stem's BN are stored.
    VGG-16's convs outside the weight-gradient kernels' shapes, AlexNet
    (no BN) and LeNet store everything."""
    r20 = synth.resnet20_workload()
    got = _unstored(psw, r20)
    assert got == [4 * b + 4 for b in range(9)]
    for k in got:
        bn = r20.ops[k - 1]
        assert bn[0] == synth.BN and bn[2] < 0 and bn[8] & synth.F_RELU
        assert [i for i, o in enumerate(r20.ops) if o[1] == k or o[2] == k] == [k]
    assert _unstored(psw, synth.resnet20_workload(batch=8, bf16=True)) == got
    assert _unstored(psw, synth.resnet110_workload()) == [4 * b + 4 for b in range(54)]
    for wl in (synth.vgg16_workload(), synth.alexnet_workload(), synth.lenet5_workload()):
        assert _unstored(psw, wl) == []


@pytest.mark.parametrize("change", ["consumer_bias", "no_relu", "consumer_5x5"])
def test_bn_on_load_needs_a_plain_3x3_consumer_and_relu(psw, change):
    """The first block's BN + ReLU (tensor 4) stays stored when its consumer
    conv has a bias, when the BN has no ReLU, or when the consumer is not a
    3x3 / pad 1 conv (5x5 / pad 2, same output shape); the other eight
    blocks' BNs are still applied on load."""
    import dataclasses

    r20 = synth.resnet20_workload()
    ops = r20.ops.copy()
    assert ops[3][0] == synth.BN and ops[4][0] == synth.CONV and ops[4][1] == 4
    if change == "consumer_bias":
        ops[4][8] |= synth.F_BIAS
    elif change == "no_relu":
        ops[3][8] &= ~synth.F_RELU
    else:
        ops[4][5], ops[4][7] = 5, 2
    got = _unstored(psw, dataclasses.replace(r20, ops=ops))
    assert got == [4 * b + 4 for b in range(1, 9)]
