"""GPU tests of the per-group organisation of the W+ / W- scratch: the plan a tight HBM budget forces for wide
blocks (the OPT-175B shape under 18 GB), in which a block's perturbed copies exist one tensor group at a time
({ln1, q, k, v}, {o}, {ln2, fc1}, {fc2}) and the fused update + perturb sweep runs once per group, between the
projections.  It is a memory-layout choice only: results must equal the whole-block plan's bit for bit, and the
oracle's to the usual bars."""
import copy

import numpy as np
import pytest
import torch

import synth_inputs as si
from oracle import codec, opt_model, zo_step

pytestmark = pytest.mark.gpu

DEFAULT_SWEEPS = 1          # the planner's preferred organisation when the budget leaves the choice


def _b():
    from paper_2503_12668_amd import binding
    return binding


def _tiny(n_layers=6):
    cfg = si.tiny_config(n_layers=n_layers, d_model=64, n_heads=4, d_ffn=136, vocab=211, max_pos=40)
    P = si.make_weights(cfg, seed=11, std=0.08, ln_jitter=True)
    tok = si.make_tokens(cfg["vocab"], 3, 23, seed=12)
    lab = si.next_token_labels(tok)
    lab[1, 4] = -100
    return cfg, P, tok, lab


@pytest.mark.parametrize("tied", [True, False])
def test_per_group_scratch_fp32_steps_match_oracle(tied):
    """Forced per-group scratch, float32: losses within 1e-5 at every step (pending update from the second on),
    parameters within 1e-6 after the flush."""
    b = _b()
    cfg, P, tok, lab = _tiny(3)
    cfg["tied"] = tied
    P = si.make_weights(cfg, seed=11, std=0.08, ln_jitter=True)
    oz = zo_step.Zo2Blockwise(opt_model.OptShape(**cfg), copy.deepcopy(P))
    ctx = b.Zo2Context(cfg, P, arena_bytes=64 << 20)
    ctx.set_scratch_plan(4)
    lrs = [1e-4, 2e-4, 5e-5, 1e-4]
    for j in range(4):
        a, g = oz.step(tok, lab, 42 + j, 1e-3, lrs[j]), ctx.step(tok, lab, 42 + j, 1e-3, lrs[j])
        assert abs(float(g[0]) - float(a[0])) <= 1e-5 * abs(float(a[0])), j
        assert abs(float(g[1]) - float(a[1])) <= 1e-5 * abs(float(a[1])), j
    pl = ctx.plan()
    assert pl["sweeps_per_block"] == 4 and pl["resident"], pl
    assert abs(float(ctx.eval(tok, lab)) - float(oz.eval_loss(tok, lab))) <= 1e-5 * 6.0      # applies the pending update on the way
    a, g = oz.step(tok, lab, 50, 1e-3, 1e-4), ctx.step(tok, lab, 50, 1e-3, 1e-4)
    assert abs(float(g[0]) - float(a[0])) <= 1e-5 * abs(float(a[0]))
    oz.flush(); ctx.flush(); ctx.sync_to_host()
    Pg = ctx.parameters()
    for n in oz.P:
        assert np.abs(Pg[n] - oz.P[n]).max() <= 1e-6, n
    ctx.close()


@pytest.mark.parametrize("wire,compute,scale,sr", [("f32", "f32", 1.0, False), ("bf16", "bf16", 1.0, False),
                                                  ("fp8_e4m3", "bf16", 64.0, False), ("bf16", "bf16", 1.0, True)])
def test_per_group_scratch_streamed_equals_whole_block_resident_bitwise(wire, compute, scale, sr):
    """Five contexts on the same model: whole-block scratch resident (the reference); per-half and per-group scratch,
    each resident and streamed through 3 slots.  Steps with a pending update, a round of several directions,
    an evaluation in between and the final flush all give identical losses, g and stored parameters."""
    b = _b()
    cfg, P, tok, lab = _tiny(6)
    nt = 4 + 16 * cfg["n_layers"]
    scales = np.full(nt, scale, np.float32) if scale != 1.0 else None
    wsz = {"f32": 4, "bf16": 2, "fp8_e4m3": 1}[wire]
    runs = {}
    want_sweeps = {"whole_resident": 1, "half_resident": 2, "group_resident": 4, "half_streamed": 2, "group_streamed": 4}
    for name in want_sweeps:
        ctx = b.Zo2Context(cfg, P, wire=wire, compute=compute, arena_bytes=64 << 20, scales=scales)
        ctx.set_wire_rounding(sr)
        ctx.set_scratch_plan(want_sweeps[name])
        ctx.set_loader_fusion(-1)       # this test is about the sweep kernel's scratch
        r = [ctx.step(tok, lab, 5, 1e-3, 1e-3)]
        if name.endswith("streamed"):
            ctx.set_resident_budget(ctx.plan()["bytes_used"] - 3 * ctx.offs[16] * wsz)        # 3 slots for 6 blocks
        r.append(ctx.step(tok, lab, 6, 1e-3, 1e-3))
        r.append(ctx.step_extra(tok, lab, 7, 1e-3, 5e-4))                                   # a second direction of the round
        r.append(ctx.step(tok, lab, 8, 1e-3, 1e-3))
        ev = ctx.eval(tok, lab)
        r.append(ctx.step(tok, lab, 9, 1e-3, 1e-3))
        pl = ctx.plan()
        assert pl["sweeps_per_block"] == want_sweeps[name], (name, pl)
        assert pl["resident"] == (not name.endswith("streamed")) and (pl["resident"] or pl["n_slots"] == 3), (name, pl)
        if name != "whole_resident":
            assert pl["scratch_elems"] < ctx.offs[16]
        ctx.flush(); ctx.sync_to_host()
        runs[name] = ([tuple(map(float, x)) for x in r] + [float(ev)], ctx.parameters())
        ctx.close()
    for name in ("half_resident", "group_resident", "half_streamed", "group_streamed"):
        assert runs[name][0] == runs["whole_resident"][0], name
        for n in runs[name][1]:
            assert np.array_equal(runs[name][1][n], runs["whole_resident"][1][n]), (name, n)
    assert all(np.isfinite(x) for x in runs["whole_resident"][0][-1:])


@pytest.mark.parametrize("d,heads,vocab", [(512, 8, 4096), (768, 12, 6148), (4352, 34, 13060), (5248, 41, 15748)])
def test_float32_projections_in_pieces_give_the_same_bits_under_every_organisation(d, heads, vocab):
    """Widths at which the output projection is cut along k (its pieces then end in the LayerNorm's pass where no sweep comes
    between): losses and parameters of eight steps under 1, 2 and 4 sweeps per block, bit for bit; without pieces they differ."""
    b = _b()
    cfg = si.tiny_config(n_layers=1, d_model=d, n_heads=heads, d_ffn=72, vocab=vocab, max_pos=40)
    P = si.make_weights(cfg, seed=11, std=0.15, ln_jitter=True)      # few rows and large logits: a late digit shows in the losses
    tok = si.make_tokens(cfg["vocab"], 1, 5, seed=12)
    lab = si.next_token_labels(tok)
    runs = {}
    for name, sweeps in (("1", 1), ("2", 2), ("4", 4), ("uncut", 1)):
        ctx = b.Zo2Context(cfg, P, arena_bytes=(256 << 20) + 40 * vocab * d)
        ctx.set_scratch_plan(sweeps)
        if name == "uncut":
            ctx.set_split_k(-1)
        r = [tuple(map(float, ctx.step(tok, lab, 5 + j, 1e-3, 1e-6))) for j in range(8)]
        assert ctx.plan()["sweeps_per_block"] == sweeps
        ctx.flush(); ctx.sync_to_host()
        runs[name] = (r, {n: a for n, a in ctx.parameters().items() if n.startswith("blocks.")})
        ctx.close()
    for name in ("2", "4"):
        assert runs[name][0] == runs["1"][0], name
        for n in runs["1"][1]:
            assert np.array_equal(runs[name][1][n], runs["1"][1][n]), (name, n)
    assert runs["uncut"][0] != runs["1"][0] or any(not np.array_equal(runs["uncut"][1][n], runs["1"][1][n]) for n in runs["1"][1])


# the last three: no pieces at all, a scratch without room for a second copy of the biases, and more rows than are worth it.  step, evaluation:
# sums left to a LayerNorm's pass (the loader path's output projections, 1 x 13, are among them under every organisation)
@pytest.mark.parametrize("wire,compute,d,vocab,batch,seq,layers,step,evaluation", [
    ("bf16", "bf16", 1024, 13060, 5, 37, 3, 3, 3), ("f16", "f16", 1024, 13060, 1, 150, 2, 2, 2), ("bf16", "bf16", 1024, 13060, 1, 13, 3, 6, 3), ("f32", "f32", 768, 9476, 1, 40, 3, 6, 6),
    ("f32", "f32", 768, 212, 1, 40, 3, 0, 0), ("bf16", "bf16", 1024, 212, 5, 37, 3, 0, 3), ("bf16", "bf16", 1024, 13060, 3, 200, 2, 0, 2)])
def test_pieces_that_wait_for_the_next_layernorm_give_the_same_bits(wire, compute, d, vocab, batch, seq, layers, step, evaluation):
    """The second FFN projection's pieces are added up by the next block's first LayerNorm, or the final one (odd and even numbers of
    blocks), on every kernel that leaves pieces; with a sweep per tensor group they never wait.  Steps and an evaluation, bit for bit."""
    b = _b()
    cfg = si.tiny_config(n_layers=layers, d_model=d, n_heads=d // 64, d_ffn=4 * d, vocab=vocab, max_pos=256)
    P = si.make_weights(cfg, seed=11, std=0.05, ln_jitter=True)
    tok = si.make_tokens(vocab, batch, seq, seed=12)
    lab = si.next_token_labels(tok)
    runs = []
    for sweeps in (1, 4):
        ctx = b.Zo2Context(cfg, P, wire=wire, compute=compute, arena_bytes=1 << 30)
        ctx.set_scratch_plan(sweeps)
        r = [tuple(map(float, ctx.step(tok, lab, 5 + j, 1e-3, 1e-5))) for j in range(3)]
        assert ctx.pass_facts()[1] == (step if sweeps == 1 else layers if ctx.plan()["loader_fusion"] else 0)
        r += [float(ctx.eval(tok, lab))]
        assert ctx.pass_facts()[1] == (evaluation if sweeps == 1 else 0)
        assert ctx.plan()["sweeps_per_block"] == sweeps
        ctx.flush(); ctx.sync_to_host()
        runs.append((r, ctx.parameters()))
        ctx.close()
    assert runs[0][0] == runs[1][0]
    for n in runs[0][1]:
        assert np.array_equal(runs[0][1][n], runs[1][1][n]), n


def test_budget_too_small_for_whole_block_scratch_falls_back_to_per_group():
    """The planner's own choice: a budget that cannot hold 3 slots next to a whole-block scratch set, but can next to
    a per-group set, gives the per-group plan (and the same bits); one notch lower is ZO2_EBUDGET."""
    b = _b()
    cfg = si.tiny_config(n_layers=5, d_model=64, n_heads=4, d_ffn=512, vocab=97, max_pos=40)     # small vocabulary: the head matrix does not set the scratch size
    P = si.make_weights(cfg, seed=11, std=0.08, ln_jitter=True)
    tok = si.make_tokens(cfg["vocab"], 3, 23, seed=12)
    lab = si.next_token_labels(tok)
    ref = b.Zo2Context(cfg, P, arena_bytes=64 << 20)
    ctx = b.Zo2Context(cfg, P, arena_bytes=64 << 20)
    r0, r1 = [ref.step(tok, lab, 5, 1e-3, 1e-3)], [ctx.step(tok, lab, 5, 1e-3, 1e-3)]
    pl = ctx.plan()
    assert pl["resident"] and pl["sweeps_per_block"] == DEFAULT_SWEEPS
    bucket = ctx.offs[16] * 4
    whole3 = pl["bytes_used"] - 2 * bucket                    # exactly 3 slots next to the whole-block scratch
    ctx.set_resident_budget(whole3 - 4096)                    # a little less: 3 slots only fit with the smaller scratch
    for j in range(3):
        r0.append(ref.step(tok, lab, 6 + j, 1e-3, 1e-3))
        r1.append(ctx.step(tok, lab, 6 + j, 1e-3, 1e-3))
    pl = ctx.plan()
    assert pl["sweeps_per_block"] > DEFAULT_SWEEPS and not pl["resident"] and pl["n_slots"] >= 3, pl
    assert [tuple(map(float, x)) for x in r0] == [tuple(map(float, x)) for x in r1]
    ref.flush(); ctx.flush(); ref.sync_to_host(); ctx.sync_to_host()
    Pr, Pc = ref.parameters(), ctx.parameters()
    for n in Pr:
        assert np.array_equal(Pr[n], Pc[n]), n
    ctx.set_resident_budget(3 * bucket)                      # not even the per-group plan fits
    with pytest.raises(b.Zo2Error) as e:
        ctx.step(tok, lab, 99, 1e-3, 1e-3)
    assert e.value.status == 3
    assert b.lib().zo2_set_scratch_plan(ctx.handle, 3) == 1          # ZO2_EINVAL: 0, 1, 2 or 4
    ref.close(); ctx.close()


@pytest.mark.timeout(900)
def test_per_group_scratch_at_13b_width_two_blocks_matches_oracle_losses():
    """OPT-13B width (d 5120, 40 heads, FFN 20480: 315 M parameters per block, the largest tensor group 105 M), two
    decoder blocks, batch 2 x 128, bf16, with the per-group scratch: one whole step in steady state (an update is
    pending, so every sweep updates and perturbs) against the oracle's Alg. 2; bf16-mode bar: losses within 2e-2
    relative.  The vocabulary is cut to 4096 entries (the head matrix is not what this plan is about) to keep the
    oracle's share, 2 G roundings and Gaussians, within minutes."""
    b = _b()
    cfg = si.opt_config("opt-13b", n_layers=2)
    cfg["vocab"] = 4096
    P = si.make_weights(cfg, seed=1)
    tok = si.make_tokens(cfg["vocab"], 2, 128, seed=2, dist="zipf")
    lab = si.next_token_labels(tok)
    ctx = b.Zo2Context(cfg, P, wire="bf16", compute="bf16", arena_bytes=8 << 30)
    ctx.set_scratch_plan(4)
    ctx.set_loader_fusion(-1)           # 256 tokens per stream would otherwise perturb in the projections' loader: no sweeps to organise
    ctx.set_pending(True, 41, 2.5e-3)
    g = ctx.step(tok, lab, 42, 1e-3, 1e-7)
    pl = ctx.plan()
    print("gpu", g, pl, flush=True)
    assert pl["sweeps_per_block"] == 4 and pl["scratch_elems"] < ctx.offs[16], pl
    ctx.close()
    Po = {n: codec.round_to(a, "bf16") for n, a in P.items()}
    del P
    print("oracle: parameters rounded to bf16", flush=True)
    oz = zo_step.Zo2Blockwise(opt_model.OptShape(**cfg), Po, store="bf16", compute="bf16")
    oz.pending = (np.float32(2.5e-3), 41, np.float32(1.0))       # eta g = 2.5e-3 with the direction of seed 41
    a = oz.step(tok, lab, 42, 1e-3, 1e-7)
    print("oracle", a, flush=True)
    assert abs(float(g[0]) - float(a[0])) <= 2e-2 * abs(float(a[0]))
    assert abs(float(g[1]) - float(a[1])) <= 2e-2 * abs(float(a[1]))


@pytest.mark.timeout(900)
def test_fp8_wire_at_30b_width_one_block_matches_oracle():
    """OPT-30B width (d 7168, 56 heads of 128, FFN 28672: 617 M parameters per block) with the parameters held in
    fp8-E4M3 at scale 64 (Sec. 5.5) and bf16 compute, one block, batch 1 x 256, the planner's own scratch choice:
    one step in steady state (an update of visible size is pending) against the oracle's Alg. 2.  Losses to the
    bf16 bar; the block's stored fp8 codes after the update against the oracle's, on windows of every tensor.  The
    vocabulary is cut to 4096 entries to keep the oracle's share within minutes."""
    b = _b()
    from oracle import philox
    from oracle.zo_step import _fma32, _store
    cfg = si.opt_config("opt-30b", n_layers=1)
    cfg["vocab"] = 4096
    P = si.make_weights(cfg, seed=1)
    tok = si.make_tokens(cfg["vocab"], 1, 256, seed=2, dist="zipf")
    lab = si.next_token_labels(tok)
    shape = opt_model.OptShape(**cfg)
    names = [n for n, _, _ in opt_model.tensor_table(shape)]
    scale, c_prev = 64.0, 4e-3
    ctx = b.Zo2Context(cfg, P, wire="fp8_e4m3", compute="bf16", arena_bytes=8 << 30, scales=np.full(len(names), scale, np.float32))
    ctx.set_pending(True, 41, c_prev)
    g = ctx.step(tok, lab, 42, 1e-3, 1e-7)
    print("gpu", g, ctx.plan(), flush=True)
    ctx.sync_to_host()
    Pg = ctx.parameters()
    ctx.close()
    Po = {n: _store(P[n], "fp8_e4m3", scale) for n in names}
    del P
    print("oracle: parameters packed", flush=True)
    # the update alone, on windows of every block tensor: same codes wherever dz cannot move the decision
    ids = {n: tid for n, tid, _ in opt_model.tensor_table(shape)}
    tot = same = 0
    for n in names:
        if not n.startswith("blocks."):
            continue
        flat, got = Po[n].reshape(-1), Pg[n].reshape(-1)
        for e0 in sorted({0, max(0, (flat.size - 4096) // 8 * 8)}):
            w = min(4096, flat.size - e0)
            want = _store(_fma32(np.float32(-c_prev), philox.gaussian(41, ids[n], e0, w), flat[e0:e0 + w]), "fp8_e4m3", scale)
            d = np.abs(got[e0:e0 + w] - want)
            tot += w; same += int(np.sum(d == 0))
            assert np.all(d <= np.abs(want) * 2.0 ** -3 + 2.0 ** -9 / scale), (n, e0)
    print("stored fp8 codes identical to the oracle's:", same / tot, flush=True)
    assert same / tot > 0.98
    oz = zo_step.Zo2Blockwise(shape, Po, store="fp8_e4m3", compute="bf16", scales={n: scale for n in names})
    oz.pending = (np.float32(c_prev), 41, np.float32(1.0))
    a = oz.step(tok, lab, 42, 1e-3, 1e-7)
    print("oracle", a, flush=True)
    assert abs(float(g[0]) - float(a[0])) <= 2e-2 * abs(float(a[0]))
    assert abs(float(g[1]) - float(a[1])) <= 2e-2 * abs(float(a[1]))


@pytest.mark.parametrize("wire,compute,d,ffn,seq", [("f32", "f32", 256, 512, 144), ("f32", "f32", 256, 512, 137), ("bf16", "bf16", 192, 768, 144), ("f16", "f16", 320, 640, 129)])
def test_heads_logits_in_chunks_give_the_bits_of_one_piece(wire, compute, d, ffn, seq):
    """Where the head writes logits (float32; 16-bit widths that its fused kernel does not take), the budget says how many rows at a time.
    512 rows and a few left over, on which alone another kernel would run, against all at once: steps, a round, an evaluation, bit for bit."""
    b = _b()
    vocab, batch = 12068, 4
    cfg = si.tiny_config(n_layers=2, d_model=d, n_heads=d // 64, d_ffn=ffn, vocab=vocab, max_pos=160)
    P = si.make_weights(cfg, seed=11, std=0.2, ln_jitter=True)
    tok = si.make_tokens(vocab, batch, seq, seed=12)
    lab = si.next_token_labels(tok)
    lab[:3] = -100                             # losses of the rows left over alone: a mean over all rows would round their late digits away
    lab[3, :-4] = -100
    runs, launches = [], []
    for rows in (512, 640):                    # a chunk: an eighth of the budget, in 128 rows of both streams
        ctx = b.Zo2Context(cfg, P, wire=wire, compute=compute, arena_bytes=1 << 30)
        ctx.set_resident_budget(64 * vocab * rows + 1000)
        ctx.set_profiling(["ce"])
        r = [tuple(map(float, ctx.step(tok, lab, 5 + j, 1e-3, 1e-5))) for j in range(2)]
        launches.append(ctx.kernel_times()["ce"][1])
        r += [tuple(map(float, x)) for x in ctx.step_multi(tok, lab, [8, 9], 1e-3, 1e-5)] + [float(ctx.eval(tok, lab))]
        assert ctx.plan()["resident"]
        ctx.flush(); ctx.sync_to_host()
        runs.append((r, ctx.parameters()))
        ctx.close()
    assert launches[0] == launches[1] + 2      # a cross-entropy pass per stream and chunk
    assert runs[0][0] == runs[1][0]
    for n in runs[0][1]:
        assert np.array_equal(runs[0][1][n], runs[1][1][n]), n
