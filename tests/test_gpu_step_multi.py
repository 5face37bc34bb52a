"""GPU tests of zo2_step_multi: a whole round of directions in one pass over the model.  Its results and the state it
leaves must equal those of zo2_step + zo2_step_extra (which the other tests hold against the oracle) bit for bit, on
every path of the step: resident and streamed, sweep copies and perturbation in the weight loader, per-group scratch,
stochastic rounding of the stored update, 8-bit wire format, write-back interval; plus one direct comparison with the
oracle's q-direction estimator."""
import copy

import numpy as np
import pytest

import synth_inputs as si
from oracle import opt_model, zo_step

pytestmark = pytest.mark.gpu


def _b():
    from paper_2503_12668_amd import binding
    return binding


def _case(n_layers=5, tied=True, batch=3, seq=23, d_ffn=136):
    cfg = si.tiny_config(n_layers=n_layers, d_model=64, n_heads=4, d_ffn=d_ffn, vocab=211, max_pos=80, tied=tied)
    P = si.make_weights(cfg, seed=11, std=0.08, ln_jitter=True)
    tok = si.make_tokens(cfg["vocab"], batch, seq, seed=12)
    lab = si.next_token_labels(tok)
    lab[1, 4] = -100
    return cfg, P, tok, lab


def _sequential_round(ctx, tok, lab, seeds, eps, lr):
    out = [ctx.step(tok, lab, seeds[0], eps, lr)]
    out += [ctx.step_extra(tok, lab, s, eps, lr) for s in seeds[1:]]
    return [tuple(float(v) for v in r) for r in out]


def _multi_round(ctx, tok, lab, seeds, eps, lr):
    return [tuple(float(v) for v in r) for r in ctx.step_multi(tok, lab, seeds, eps, lr)]


def _run(b, cfg, P, tok, lab, multi, wire, compute, streamed, sr=False, fusion=0, sweeps=0, interval=1):
    ctx = b.Zo2Context(cfg, P, wire=wire, compute=compute, arena_bytes=96 << 20)
    ctx.set_wire_rounding(sr)
    ctx.set_loader_fusion(fusion)
    rnd = _multi_round if multi else _sequential_round
    out = [rnd(ctx, tok, lab, [7, 8, 9], 1e-3, 1e-4)]                    # first round: resident, nothing pending
    if streamed:
        esz = b.lib().zo2_dtype_size(ctx.wire_id)
        # 3 or 4 slots for 5 blocks (the slack pays for the residual streams of the further directions)
        ctx.set_resident_budget(ctx.plan()["bytes_used"] - 2 * ctx.offs[16] * esz + 40_000)
        ctx.debug_set_slot_poison(True)
        ctx.set_writeback_interval(interval)
    if sweeps:
        ctx.set_scratch_plan(sweeps)
    out.append(rnd(ctx, tok, lab, [20, 21], 1e-3, 1e-4))
    out.append(rnd(ctx, tok, lab, [30, 31, 32, 33], 1e-3, 5e-5))
    out.append([tuple(float(v) for v in ctx.step(tok, lab, 40, 1e-3, 1e-4))])   # an ordinary step applies the round of four
    out.append(rnd(ctx, tok, lab, [50, 51], 1e-3, 1e-4))
    ev = float(ctx.eval(tok, lab))
    out.append(rnd(ctx, tok, lab, [60, 61, 62], 1e-3, 1e-4))
    pend = ctx.pending_list()
    pl = ctx.plan()
    assert pl["resident"] == (not streamed), pl
    ctx.flush(); ctx.sync_to_host()
    res = (out, ev, [(int(s), float(c)) for s, c in pend], ctx.parameters())
    ctx.close()
    return res


def _same(a, b):
    assert a[0] == b[0]
    assert a[1] == b[1]
    assert a[2] == b[2] and len(a[2]) == 3
    for n in a[3]:
        assert np.array_equal(a[3][n], b[3][n]), n
    assert all(np.isfinite(v) for rnd in a[0] for r in rnd for v in r)


@pytest.mark.parametrize("wire,compute,sr", [("f32", "f32", False), ("bf16", "bf16", False), ("bf16", "bf16", True), ("fp8_e4m3", "bf16", True)])
@pytest.mark.parametrize("streamed", [False, True])
def test_one_pass_rounds_equal_sequential_rounds_bitwise(wire, compute, sr, streamed):
    b = _b()
    cfg, P, tok, lab = _case()
    one = _run(b, cfg, P, tok, lab, True, wire, compute, streamed, sr=sr, fusion=-1)
    seq = _run(b, cfg, P, tok, lab, False, wire, compute, streamed, sr=sr, fusion=-1)
    _same(one, seq)


@pytest.mark.parametrize("streamed,interval", [(False, 1), (True, 1), (True, 3)])
def test_one_pass_rounds_with_the_perturbation_in_the_weight_loader(streamed, interval):
    b = _b()
    cfg, P, tok, lab = _case(d_ffn=128)
    one = _run(b, cfg, P, tok, lab, True, "bf16", "bf16", streamed, fusion=1, interval=interval)
    seq = _run(b, cfg, P, tok, lab, False, "bf16", "bf16", streamed, fusion=1, interval=interval)
    _same(one, seq)


@pytest.mark.parametrize("sweeps,interval", [(2, 1), (4, 1), (1, 4)])
def test_one_pass_rounds_streamed_with_per_group_scratch_and_write_back_interval(sweeps, interval):
    b = _b()
    cfg, P, tok, lab = _case()
    one = _run(b, cfg, P, tok, lab, True, "bf16", "bf16", True, fusion=-1, sweeps=sweeps, interval=interval)
    seq = _run(b, cfg, P, tok, lab, False, "bf16", "bf16", True, fusion=-1, sweeps=sweeps, interval=interval)
    res = _run(b, cfg, P, tok, lab, True, "bf16", "bf16", False, fusion=-1)
    _same(one, seq)
    _same(one, res)


def test_one_pass_round_uploads_each_block_once():
    b = _b()
    cfg, P, tok, lab = _case(n_layers=7)
    ctx = b.Zo2Context(cfg, P, arena_bytes=96 << 20)
    ctx.step(tok, lab, 5, 1e-3, 1e-4)
    bucket = ctx.offs[16] * 4
    ctx.set_resident_budget(ctx.plan()["bytes_used"] - 3 * bucket)
    r = ctx.step_multi(tok, lab, [1, 2, 3, 4], 1e-3, 1e-4)
    st = ctx.step_stats()
    assert not ctx.plan()["resident"] and len(r) == 4
    assert st["bytes_up"] == 7 * bucket and st["bytes_down"] == 7 * bucket      # the pending update of step 5 went back
    r = ctx.step_multi(tok, lab, [11, 12], 1e-3, 1e-4)
    st = ctx.step_stats()
    assert st["bytes_up"] == 7 * bucket and st["bytes_down"] == 7 * bucket
    assert [s for s, _ in ctx.pending_list()] == [11, 12]
    ctx.close()


@pytest.mark.parametrize("tied", [True, False])
def test_fp32_one_pass_rounds_match_oracle(tied):
    b = _b()
    cfg, P, tok, lab = _case(n_layers=3, tied=tied)
    oz = zo_step.Zo2Blockwise(opt_model.OptShape(**cfg), copy.deepcopy(P))
    ctx = b.Zo2Context(cfg, P, arena_bytes=256 << 20)
    q = 3
    for j in range(3):
        seeds = [500 + 10 * j + i for i in range(q)]
        ro = [oz.step(tok, lab, seeds[0], 1e-3, 1e-4)] + [oz.step_extra(tok, lab, s, 1e-3, 1e-4) for s in seeds[1:]]
        rg = ctx.step_multi(tok, lab, seeds, 1e-3, 1e-4)
        for a, g in zip(ro, rg):
            assert abs(float(g[0]) - float(a[0])) <= 1e-5 * abs(float(a[0]))
            assert abs(float(g[1]) - float(a[1])) <= 1e-5 * abs(float(a[1]))
            assert abs(float(g[2]) - float(a[2])) <= 1e-5 * abs(float(a[0])) / 1e-3
    oz.flush(); ctx.flush(); ctx.sync_to_host()
    Pg = ctx.parameters()
    for n in oz.P:
        assert np.abs(Pg[n] - oz.P[n]).max() <= 1e-6, n
    ctx.close()


def test_step_multi_rejects_bad_arguments_and_one_direction_is_a_step():
    b = _b()
    cfg, P, tok, lab = _case(n_layers=2)
    ctx = b.Zo2Context(cfg, P, arena_bytes=64 << 20)
    ref = b.Zo2Context(cfg, P, arena_bytes=64 << 20)
    with pytest.raises(b.Zo2Error):
        ctx.step_multi(tok, lab, [], 1e-3, 1e-4)
    with pytest.raises(b.Zo2Error):
        ctx.step_multi(tok, lab, list(range(17)), 1e-3, 1e-4)
    with pytest.raises(b.Zo2Error):
        ctx.step_multi(tok, lab, [1, 2], 0.0, 1e-4)
    for j in range(3):
        a = ctx.step_multi(tok, lab, [70 + j], 1e-3, 1e-4)[0]
        r = ref.step(tok, lab, 70 + j, 1e-3, 1e-4)
        assert tuple(map(float, a)) == tuple(map(float, r))
    ctx.close(); ref.close()


@pytest.mark.parametrize("batch,seq,dirs,wire,sr", [(1, 70, 2, "bf16", False), (3, 97, 3, "fp8_e4m3", False), (4, 128, 4, "bf16", False),
                                                    (2, 190, 5, "bf16", False), (1, 300, 4, "f32", False), (2, 150, 3, "bf16", True)])
def test_directions_that_share_their_launches(batch, seq, dirs, wire, sr):
    """Directions of a round go through a resident block together where the budget has room for their scratch sets (here on sizes whose
    projections take 64- and 128-wide tiles, large tiles and pieces of k; five directions go as four and one), one after the
    other where it has none: the same bits, also of single directions one by one."""
    b = _b()
    cfg = si.tiny_config(n_layers=2, d_model=1024, n_heads=16, d_ffn=4096, vocab=515, max_pos=320, tied=True)
    P = si.make_weights(cfg, seed=21, std=0.03, ln_jitter=True)
    tok = si.make_tokens(cfg["vocab"], batch, seq, seed=22)
    lab = si.next_token_labels(tok)
    found = []
    for how in ("room", "no room", "one by one"):
        ctx = b.Zo2Context(cfg, P, wire=wire, compute="bf16", arena_bytes=1 << 30)
        ctx.set_wire_rounding(sr)
        ctx.set_loader_fusion(-1)
        rnd = _sequential_round if how == "one by one" else _multi_round
        out = [rnd(ctx, tok, lab, [7 + j for j in range(dirs)], 1e-3, 1e-4)]
        if how == "no room":
            ctx.set_resident_budget(ctx.plan()["bytes_used"])
        out += [rnd(ctx, tok, lab, [20 * k + j for j in range(dirs)], 1e-3, 1e-4) for k in (1, 2)]
        assert ctx.plan()["resident"]
        assert ctx.pass_facts()[0] == (min(dirs, 4) if how == "room" else 1)
        ctx.flush(); ctx.sync_to_host()
        found.append((out, ctx.parameters()))
        ctx.close()
    for out, params in found[1:]:
        assert out == found[0][0]
        for n in params:
            assert np.array_equal(params[n], found[0][1][n]), n


@pytest.mark.parametrize("batch,seq,d_ffn,dirs", [(1, 257, 320, 4), (2, 150, 2112, 4), (1, 290, 576, 3)])
def test_directions_on_tiles_of_256_rows(batch, seq, d_ffn, dirs):
    """At d_model 2048, six or eight problems of 257 - 300 rows: output projection and FC2 take tiles of 256 rows where one direction takes
    lower ones.  One row and 44 rows in the second tile, 5 to 33 slabs (a ring of three, an odd last slab): the bits of single directions."""
    b = _b()
    cfg = si.tiny_config(n_layers=1, d_model=2048, n_heads=32, d_ffn=d_ffn, vocab=260, max_pos=320, tied=True)
    P = si.make_weights(cfg, seed=31, std=0.03, ln_jitter=True)
    tok = si.make_tokens(cfg["vocab"], batch, seq, seed=32)
    lab = si.next_token_labels(tok)
    found = []
    for rnd in (_multi_round, _sequential_round):
        ctx = b.Zo2Context(cfg, P, wire="bf16", compute="bf16", arena_bytes=2 << 30)
        ctx.set_loader_fusion(-1)
        out = [rnd(ctx, tok, lab, [20 * k + j for j in range(dirs)], 1e-3, 1e-4) for k in (0, 1)]
        if rnd is _multi_round:
            assert ctx.pass_facts()[0] == dirs
        ctx.flush(); ctx.sync_to_host()
        found.append((out, ctx.parameters()))
        ctx.close()
    assert found[0][0] == found[1][0]
    for n in found[0][1]:
        assert np.array_equal(found[0][1][n], found[1][1][n]), n


@pytest.mark.parametrize("wire,sr,tied,dirs", [("bf16", False, True, 4), ("bf16", False, False, 5), ("fp8_e4m3", True, True, 3), ("f32", False, False, 2), ("bf16", True, True, 7)])
def test_head_of_several_directions(wire, sr, tied, dirs):
    """The head takes a round's directions together too, and the tables all deferred updates in one sweep behind a gather that makes them
    for the rows it reads: the bits of a budget that leaves no room for it, of one that leaves room for two directions, and of single directions.
    Vocabulary with a last tile of 4 columns and a last chunk of the sweep that is not full; more directions than go together; a last
    round of another size."""
    b = _b()
    cfg = si.tiny_config(n_layers=1, d_model=128, n_heads=4, d_ffn=256, vocab=516, max_pos=160, tied=tied)
    P = si.make_weights(cfg, seed=41, std=0.05, ln_jitter=True)
    tok = si.make_tokens(cfg["vocab"], 2, 150, seed=42)
    lab = si.next_token_labels(tok)
    lab[1, 7] = -100
    found = []
    for how in ("room", "room for two", "no room", "one by one"):
        scales = np.full(4 + 16 + (0 if tied else 1), 64.0, np.float32) if wire.startswith("fp8") else None
        ctx = b.Zo2Context(cfg, P, wire=wire, compute="bf16", arena_bytes=256 << 20, scales=scales)
        ctx.set_wire_rounding(sr)
        rnd = _sequential_round if how == "one by one" else _multi_round
        out = [rnd(ctx, tok, lab, [7 + j for j in range(dirs)], 1e-3, 1e-3)]
        used = ctx.plan()["bytes_used"]
        if how == "no room":
            ctx.set_resident_budget(used)
        elif how == "room for two":      # four copies of the vocabulary matrix, activations and the partials of two directions, and half a direction more
            ctx.set_resident_budget(used + 5 * (516 * 128 * 2 + 300 * 128 * 2 + 300 * (2 * 12 + 2) * 4) + 8192)
        out += [rnd(ctx, tok, lab, [20 * k + j for j in range(n)], 1e-3, 1e-3) for k, n in ((1, dirs), (2, 2))]
        out.append(tuple(float(v) for v in ctx.step(tok, lab, 90, 1e-3, 1e-3)))
        assert ctx.plan()["resident"]
        ctx.flush(); ctx.sync_to_host()
        found.append((out, ctx.parameters()))
        ctx.close()
    for out, params in found[1:]:
        assert out == found[0][0]
        for n in params:
            assert np.array_equal(params[n], found[0][1][n]), n


@pytest.mark.parametrize("batch,seq,vocab,dirs", [(10, 205, 8196, 4), (9, 257, 8196, 2), (13, 250, 4100, 3), (17, 250, 4100, 2)])
def test_head_of_several_directions_adds_a_span_as_one_direction_does(batch, seq, vocab, dirs):
    """More than 2048 rows, where a launch of 256-row tiles has eight wavefronts, which add a span of 64 columns in halves: by the count of tiles alone the
    head of several directions would take other tiles than that of one (two problems), in one sense or the other.  (Two labels, of
    losses near 0, the words that stand there: the mean over all rows, or a loss of 9, would hide the last digit.)"""
    b = _b()
    cfg = si.tiny_config(n_layers=1, d_model=128, n_heads=4, d_ffn=256, vocab=vocab, max_pos=270)
    P = si.make_weights(cfg, seed=41, std=0.2, ln_jitter=True)
    for n in ("blocks.0.o.w", "blocks.0.fc2.w"):
        P[n] = P[n] * np.float32(0.02)
    tok = si.make_tokens(vocab, batch, seq, seed=42)
    lab = np.full_like(tok, -100)
    lab[0, 3], lab[batch - 1, seq - 1] = tok[0, 3], tok[batch - 1, seq - 1]
    found = []
    for rnd in (_multi_round, _sequential_round):
        ctx = b.Zo2Context(cfg, P, wire="bf16", compute="bf16", arena_bytes=1 << 30)
        out = [rnd(ctx, tok, lab, [20 * k + j for j in range(dirs)], 1e-3, 1e-4) for k in range(12)]
        ctx.flush(); ctx.sync_to_host()
        found.append((out, ctx.parameters()))
        ctx.close()
    assert max(float(r[0]) for r in found[1][0][0]) < 2.0
    assert found[0][0] == found[1][0]
    for n in found[0][1]:
        assert np.array_equal(found[0][1][n], found[1][1][n]), n


@pytest.mark.parametrize("wire,first", [("f32", "small step"), ("f32", "nothing"), ("bf16", "nothing"), ("bf16", "evaluation")])
def test_rounds_are_refused_where_the_sweep_has_a_stream_of_its_own(wire, first):
    """With a stream for the sweep a block runs one direction.  The plan that gives it one may be that of the very call: the first of a context, or one
    behind a step of few tokens, which in float32 has no sweep.  Refused, and the context goes on as if it had not been asked."""
    b = _b()
    cfg = si.tiny_config(n_layers=2, d_model=64, n_heads=2, d_ffn=128, vocab=260, max_pos=80)
    P = si.make_weights(cfg, seed=11, std=0.08, ln_jitter=True)
    small, large = si.make_tokens(260, 1, 30, seed=1), si.make_tokens(260, 4, 50, seed=4)
    got = []
    for overlap in (True, False):
        ctx = b.Zo2Context(cfg, P, wire=wire, compute=wire, arena_bytes=64 << 20, overlap_k1=overlap)
        ctx.set_loader_fusion(0 if wire == "f32" else -1)
        out = []
        if first == "small step":
            out += [ctx.step(small, si.next_token_labels(small), 3, 1e-3, 1e-3)]
            assert ctx.plan()["loader_fusion"] and ctx.plan()["scratch_sets"] == 1
        elif first == "evaluation":
            out += [(ctx.eval(small, si.next_token_labels(small)),)]
        lab = si.next_token_labels(large)
        if overlap:
            with pytest.raises(b.Zo2Error, match="ESTATE"):
                ctx.step_multi(large, lab, [7, 8, 9], 1e-3, 1e-3)
        out += [ctx.step(large, lab, 5 + j, 1e-3, 1e-3) for j in range(2)]
        assert ctx.plan()["scratch_sets"] == 1 + overlap
        used = ctx.plan()["bytes_used"]
        ctx.flush(); ctx.sync_to_host()
        got.append(([float(x) for a in out for x in a], ctx.parameters(), used))
        if overlap:      # no residual streams are held for the directions that were refused
            other = b.Zo2Context(cfg, P, wire=wire, compute=wire, arena_bytes=64 << 20, overlap_k1=True)
            other.set_loader_fusion(-1)
            other.step(large, lab, 5, 1e-3, 1e-3)
            assert other.plan()["bytes_used"] == used
            other.close()
        ctx.close()
    assert got[0][0] == got[1][0]
    for n in P:
        assert np.array_equal(got[0][1][n], got[1][1][n]), n
