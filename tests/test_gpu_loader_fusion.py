"""GPU tests of whole steps in which the block projections perturb in their weight loader (steps of few tokens):
against the oracle's Alg. 2, against the sweep-kernel path, streamed against resident, and with the other features
of the step (several directions per update, evaluation in between, stochastic rounding of the stored update)."""
import copy

import numpy as np
import pytest
import torch

import synth_inputs as si
from oracle import codec, opt_model, zo_step

pytestmark = pytest.mark.gpu


def _b():
    from paper_2503_12668_amd import binding
    return binding


def _tiny(n_layers=4, tied=True):
    cfg = si.tiny_config(n_layers=n_layers, d_model=64, n_heads=4, d_ffn=128, vocab=211, max_pos=40, tied=tied)
    P = si.make_weights(cfg, seed=11, std=0.08, ln_jitter=True)
    tok = si.make_tokens(cfg["vocab"], 3, 23, seed=12)
    lab = si.next_token_labels(tok)
    lab[1, 4] = -100
    return cfg, P, tok, lab


@pytest.mark.parametrize("dt", ["bf16", "f16"])
@pytest.mark.parametrize("tied", [True, False])
def test_fused_loader_steps_track_oracle_and_the_sweep_path(dt, tied):
    b = _b()
    cfg, P, tok, lab = _tiny(tied=tied)
    Po = {n: codec.round_to(a, dt) for n, a in P.items()}
    oz = zo_step.Zo2Blockwise(opt_model.OptShape(**cfg), copy.deepcopy(Po), store=dt, compute=dt)
    fused = b.Zo2Context(cfg, P, wire=dt, compute=dt, arena_bytes=64 << 20)
    fused.set_loader_fusion(1)          # 69 tokens: above the default's 64
    plain = b.Zo2Context(cfg, P, wire=dt, compute=dt, arena_bytes=64 << 20)
    plain.set_loader_fusion(-1)
    for j in range(4):
        a = oz.step(tok, lab, 42 + j, 1e-3, 1e-2)
        f = fused.step(tok, lab, 42 + j, 1e-3, 1e-2)
        p = plain.step(tok, lab, 42 + j, 1e-3, 1e-2)
        for k in (0, 1):
            assert abs(float(f[k]) - float(a[k])) <= 2e-2 * abs(float(a[k])), (j, k)
            # same W+- bit for bit and the same products, added in another order, then rounded to 16 bits per layer
            assert abs(float(f[k]) - float(p[k])) <= (2e-3 if j == 0 else 2e-2) * abs(float(p[k])), (j, k)
    assert fused.plan()["loader_fusion"] and not plain.plan()["loader_fusion"]
    ev_f, ev_p = fused.eval(tok, lab), plain.eval(tok, lab)
    assert abs(float(ev_f) - float(ev_p)) <= 2e-2 * abs(float(ev_p))
    fused.close(); plain.close()


def test_first_step_of_both_paths_is_the_same_update_free_forward():
    """Without a pending update both paths start from identical parameters: the losses differ only by the summation
    order inside the projections (float32) and its effect on 16-bit roundings downstream."""
    b = _b()
    cfg, P, tok, lab = _tiny(n_layers=2)
    res = []
    for mode in (1, -1):
        ctx = b.Zo2Context(cfg, P, wire="bf16", compute="bf16", arena_bytes=64 << 20)
        ctx.set_loader_fusion(mode)
        res.append(ctx.step(tok, lab, 7, 1e-3, 0.0))
        ctx.close()
    assert abs(float(res[0][0]) - float(res[1][0])) <= 1e-3 * abs(float(res[1][0]))
    assert abs(float(res[0][1]) - float(res[1][1])) <= 1e-3 * abs(float(res[1][1]))


@pytest.mark.parametrize("sr", [False, True])
def test_fused_loader_streamed_equals_resident_bitwise(sr):
    b = _b()
    cfg, P, tok, lab = _tiny(n_layers=6)
    runs = {}
    for name in ("resident", "streamed"):
        ctx = b.Zo2Context(cfg, P, wire="bf16", compute="bf16", arena_bytes=64 << 20)
        ctx.set_loader_fusion(1)
        ctx.set_wire_rounding(sr)
        r = [ctx.step(tok, lab, 5, 1e-3, 1e-3)]
        if name == "streamed":
            ctx.set_resident_budget(ctx.plan()["bytes_used"] - 3 * ctx.offs[16] * 2)        # 3 slots for 6 blocks
            ctx.debug_set_slot_poison(True)
        r.append(ctx.step(tok, lab, 6, 1e-3, 1e-3))
        r.append(ctx.step_extra(tok, lab, 7, 1e-3, 5e-4))
        r.append(ctx.step(tok, lab, 8, 1e-3, 1e-3))
        ev = ctx.eval(tok, lab)
        r.append(ctx.step(tok, lab, 9, 1e-3, 1e-3))
        pl = ctx.plan()
        assert pl["loader_fusion"] and pl["resident"] == (name == "resident"), pl
        ctx.flush(); ctx.sync_to_host()
        runs[name] = ([tuple(map(float, x)) for x in r] + [float(ev)], ctx.parameters())
        ctx.close()
    assert runs["streamed"][0] == runs["resident"][0]
    for n in runs["resident"][1]:
        assert np.array_equal(runs["streamed"][1][n], runs["resident"][1][n]), n
    assert all(np.all(np.isfinite(x)) for x in runs["resident"][0])


def test_zero_lr_leaves_parameters_in_the_fused_path():
    b = _b()
    cfg, P, tok, lab = _tiny(n_layers=2)
    ctx = b.Zo2Context(cfg, P, wire="bf16", compute="bf16", arena_bytes=64 << 20)
    ctx.set_loader_fusion(1)
    r1 = ctx.step(tok, lab, 5, 1e-3, 0.0)
    r2 = ctx.step(tok, lab, 5, -1e-3, 0.0)
    assert ctx.plan()["loader_fusion"]
    ctx.flush(); ctx.sync_to_host()
    Pg = ctx.parameters()
    for n in P:
        assert np.array_equal(Pg[n], codec.round_to(P[n], "bf16")), n
    assert float(r1[0]) == float(r2[1]) and float(r1[1]) == float(r2[0]) and float(r1[2]) == float(r2[2])
    ctx.close()


@pytest.mark.timeout(600)
def test_fused_loader_one_block_at_opt1p3b_width_matches_oracle():
    """OPT-1.3B width (d 2048, 32 heads, FFN 8192), one block, batch 1 x 128: two steps (the second with a pending
    update) against the oracle's Alg. 2; bf16 bar.  Vocabulary cut to 4096 entries."""
    b = _b()
    cfg = si.opt_config("opt-1.3b", n_layers=1)
    cfg["vocab"] = 4096
    P = si.make_weights(cfg, seed=1)
    tok = si.make_tokens(cfg["vocab"], 1, 128, seed=2, dist="zipf")
    lab = si.next_token_labels(tok)
    Po = {n: codec.round_to(a, "bf16") for n, a in P.items()}
    oz = zo_step.Zo2Blockwise(opt_model.OptShape(**cfg), Po, store="bf16", compute="bf16")
    ctx = b.Zo2Context(cfg, P, wire="bf16", compute="bf16", arena_bytes=2 << 30)
    ctx.set_loader_fusion(1)
    for j in range(2):
        a = oz.step(tok, lab, 42 + j, 1e-3, 1e-4)
        g = ctx.step(tok, lab, 42 + j, 1e-3, 1e-4)
        print(j, a, g, flush=True)
        assert abs(float(g[0]) - float(a[0])) <= 2e-2 * abs(float(a[0]))
        assert abs(float(g[1]) - float(a[1])) <= 2e-2 * abs(float(a[1]))
    assert ctx.plan()["loader_fusion"]
    ctx.close()


def test_default_takes_the_loader_path_up_to_64_tokens_per_stream():
    b = _b()
    cfg, P, tok, lab = _tiny(n_layers=2)
    ctx = b.Zo2Context(cfg, P, wire="bf16", compute="bf16", arena_bytes=64 << 20)
    for batch, seq, want in ((2, 32, True), (4, 16, True), (3, 23, False), (5, 13, False)):
        t = si.make_tokens(cfg["vocab"], batch, seq, seed=3)
        ctx.step(t, si.next_token_labels(t), 9, 1e-3, 0.0)
        assert ctx.plan()["loader_fusion"] == want, (batch, seq)
    ctx.close()


@pytest.mark.parametrize("dt,d,f", [("bf16", 64, 128), ("f16", 192, 320), ("bf16", 1088, 1152), ("bf16", 4160, 64)])
@pytest.mark.parametrize("stochastic", [False, True])
def test_one_sweep_for_matrices_and_vectors_and_the_sum_with_the_layernorm(dt, d, f, stochastic):
    """Widths that leave threads idle in the pass that sums the output projection's slices and normalises, and that give them two pieces, tensors
    that end inside a chunk of the sweep: with a pending update the first losses are those of the ordinary path up to the order
    of the sums, and the stored parameters (lr 0 keeps them equal: a round's two updates of coefficient 0) the same bits."""
    b = _b()
    cfg = si.tiny_config(n_layers=2, d_model=d, n_heads=d // 16 if d % 64 else d // 64, d_ffn=f, vocab=211, max_pos=40)
    P = si.make_weights(cfg, seed=11, std=0.05, ln_jitter=True)
    tok = si.make_tokens(cfg["vocab"], 1, 9, seed=12)
    lab = si.next_token_labels(tok)
    got = {}
    for mode in (1, -1):
        ctx = b.Zo2Context(cfg, P, wire=dt, compute=dt, arena_bytes=512 << 20)
        ctx.set_loader_fusion(mode)
        ctx.set_wire_rounding(stochastic)
        ctx.set_pending(True, 7, 3e-4)                     # an update of a size that moves the stored values
        r = ctx.step(tok, lab, 42, 1e-3, 0.0)
        assert ctx.plan()["loader_fusion"] == (mode == 1)
        ctx.sync_to_host()
        got[mode] = (r, ctx.parameters())
        ctx.close()
    for k in (0, 1):
        assert abs(float(got[1][0][k]) - float(got[-1][0][k])) <= 2e-3 * abs(float(got[-1][0][k]))
    for n in P:
        assert np.array_equal(got[1][1][n], got[-1][1][n]), n
    assert any(not np.array_equal(got[1][1][n], codec.round_to(P[n], dt)) for n in P)


@pytest.mark.parametrize("d,f,vocab,line", [(256, 2048, 260, 64), (704, 2816, 260, 64), (1024, 512, 260, 64), (768, 768, 260, 16), (832, 832, 260, 32), (1536, 512, 260, 16),
                                              (1600, 384, 260, 37), (2048, 320, 260, 60), (2816, 192, 260, 64), (2816, 192, 34820, 126)])
def test_default_line_of_the_loader_path_by_width(d, f, vocab, line):
    """16 tokens up to d_model 1536, then 11 more per 128, 16 more for no multiple of 128; beyond 64 only where the vocabulary's logits
    have room for the slices; 64 where a matrix has at most 2^19 elements, d x d or d x ffn.  Under stochastic rounding 64."""
    b = _b()
    cfg = si.tiny_config(n_layers=1, d_model=d, n_heads=d // 64, d_ffn=f, vocab=vocab, max_pos=130)
    P = si.make_weights(cfg, seed=1)
    ctx = b.Zo2Context(cfg, P, wire="bf16", compute="bf16", arena_bytes=1 << 30)
    for stochastic, at in ((False, line), (True, 64)):
        ctx.set_wire_rounding(stochastic)
        for seq in (at, at + 1):
            t = si.make_tokens(vocab, 1, seq, seed=3)
            ctx.step(t, si.next_token_labels(t), 9, 1e-3, 0.0)
            assert ctx.plan()["loader_fusion"] == (seq == at), (stochastic, seq)
    ctx.close()


@pytest.mark.parametrize("d,f,line", [(64, 256, 32), (128, 512, 32), (128, 576, 64), (192, 768, 64), (512, 2048, 64), (576, 2048, 96)])
def test_default_line_of_the_float32_loader_path_by_width(d, f, line):
    """32 tokens where d_model d_ffn is at most 2^16, 64 where it is at most 2^20, 96 beyond; a forced loader path goes to 96 everywhere."""
    b = _b()
    cfg = si.tiny_config(n_layers=1, d_model=d, n_heads=d // 64, d_ffn=f, vocab=max(3 * d, f), max_pos=130)
    ctx = b.Zo2Context(cfg, si.make_weights(cfg, seed=1), arena_bytes=256 << 20)
    for mode, at in ((0, line), (1, 96)):
        ctx.set_loader_fusion(mode)
        for seq in (at, at + 1):
            t = si.make_tokens(cfg["vocab"], 1, seq, seed=3)
            ctx.step(t, si.next_token_labels(t), 9, 1e-3, 0.0)
            assert ctx.plan()["loader_fusion"] == (seq == at), (mode, seq)
    ctx.close()


@pytest.mark.parametrize("d,f,vocab,batch,seq,tied", [(64, 128, 212, 1, 2, True), (192, 320, 1092, 1, 31, False), (192, 64, 1091, 3, 11, True), (256, 1088, 2052, 1, 64, True),
                                                        (128, 192, 516, 5, 13, False), (448, 576, 1352, 2, 48, True)])
def test_float32_loader_updates_as_the_sweep_does(d, f, vocab, batch, seq, tied):
    """float32: the projections' loader applies the pending update too.  2 - 96 rows (edges of its three heights), features that end inside a
    workgroup's 128, one slab and several, a vocabulary that the head's loader takes or leaves: the stored parameters are the sweep's bit for bit, the
    losses those of the ordinary path and of the oracle to the float32 bar, and a second direction at the same parameters agrees as well."""
    b = _b()
    cfg = si.tiny_config(n_layers=2, d_model=d, n_heads=d // 64, d_ffn=f, vocab=vocab, max_pos=80, tied=tied)
    P = si.make_weights(cfg, seed=11, std=0.05, ln_jitter=True)
    tok = si.make_tokens(vocab, batch, seq, seed=12)
    lab = si.next_token_labels(tok)
    oz = zo_step.Zo2Blockwise(opt_model.OptShape(**cfg), copy.deepcopy(P))
    want = [oz.step(tok, lab, 42, 1e-3, 1e-4), oz.step(tok, lab, 43, 1e-3, 1e-4), oz.step_extra(tok, lab, 44, 1e-3, 1e-4)]
    got = {}
    for mode in (1, -1):
        ctx = b.Zo2Context(cfg, P, arena_bytes=512 << 20)
        ctx.set_loader_fusion(mode)
        r = [ctx.step(tok, lab, 42, 1e-3, 1e-4), ctx.step(tok, lab, 43, 1e-3, 1e-4), ctx.step_extra(tok, lab, 44, 1e-3, 1e-4)]
        assert ctx.plan()["loader_fusion"] == (mode == 1)
        for a, w in zip(r, want):
            for k in (0, 1):
                assert abs(float(a[k]) - float(w[k])) <= 1e-5 * abs(float(w[k])), (mode, a, w)
        ctx.close()
        # one update of the same coefficient on either path
        ctx = b.Zo2Context(cfg, P, arena_bytes=512 << 20)
        ctx.set_loader_fusion(mode)
        ctx.set_pending(True, 7, 3e-3)
        ctx.step(tok, lab, 42, 1e-3, 0.0)
        ctx.sync_to_host()
        got[mode] = ctx.parameters()
        ctx.close()
    for n in P:
        assert np.array_equal(got[1][n], got[-1][n]), n
        assert not np.array_equal(got[1][n], P[n]), n


def test_float32_loader_computes_sums_of_tiny_operands_with_float32_products():
    """Activations of 2^-100 behind the second LayerNorm: FC1's sums are below what three bfloat16 parts hold, FC2's weights of 2^100 bring them
    back to the residual stream's size.  (eps as small, so that the perturbation leaves them there.)"""
    b = _b()
    cfg = si.tiny_config(n_layers=2, d_model=128, n_heads=2, d_ffn=192, vocab=516, max_pos=40)
    P = si.make_weights(cfg, seed=11, std=0.05, ln_jitter=False)
    for l in range(2):
        P[f"blocks.{l}.ln2.w"] = np.full_like(P[f"blocks.{l}.ln2.w"], 2.0 ** -100)
        P[f"blocks.{l}.fc1.b"] = np.zeros_like(P[f"blocks.{l}.fc1.b"])
        P[f"blocks.{l}.fc2.w"] = P[f"blocks.{l}.fc2.w"] * np.float32(2.0 ** 100)
    tok = si.make_tokens(cfg["vocab"], 1, 35, seed=12)
    lab = si.next_token_labels(tok)
    want = zo_step.Zo2Blockwise(opt_model.OptShape(**cfg), copy.deepcopy(P)).step(tok, lab, 42, 1e-33, 0.0)
    plain = {n: (a * 0 if ".fc2.w" in n else a) for n, a in P.items()}
    without = zo_step.Zo2Blockwise(opt_model.OptShape(**cfg), plain).step(tok, lab, 42, 1e-33, 0.0)
    assert abs(float(want[0]) - float(without[0])) > 1e-3 * abs(float(want[0]))       # FC2 matters to the loss
    ctx = b.Zo2Context(cfg, P, arena_bytes=128 << 20)
    ctx.set_loader_fusion(1)
    got = ctx.step(tok, lab, 42, 1e-33, 0.0)
    assert ctx.plan()["loader_fusion"]
    for k in (0, 1):
        assert abs(float(got[k]) - float(want[k])) <= 1e-5 * abs(float(want[k])), (got, want)
    ctx.close()


@pytest.mark.parametrize("dt,rows,vocab,tied", [("bf16", 2, 212, True), ("f16", 32, 1092, False), ("bf16", 33, 1028, False), ("f16", 64, 260, True), ("bf16", 65, 2052, True),
                                                ("bf16", 96, 516, False), ("f16", 96, 132, True), ("bf16", 97, 516, True)])
def test_head_in_the_loader_by_rows_and_ragged_vocabularies(dt, rows, vocab, tied):
    """16-bit head whose logits stay in the kernel: 2 - 97 rows (edges of its three heights and the kernel beyond them), vocabularies that end inside
    a workgroup's 128 columns and inside a half's 64.  The losses are the ordinary path's but for the order of the float32 sums."""
    b = _b()
    cfg = si.tiny_config(n_layers=1, d_model=128, n_heads=2, d_ffn=192, vocab=vocab, max_pos=100, tied=tied)
    P = si.make_weights(cfg, seed=11, std=0.05, ln_jitter=True)
    tok = si.make_tokens(vocab, 1, rows, seed=12)
    lab = si.next_token_labels(tok)
    lab[0, rows // 3] = -100
    lab[0, rows // 2] = vocab - 1
    got = {}
    for mode in (1, -1):
        ctx = b.Zo2Context(cfg, P, wire=dt, compute=dt, arena_bytes=256 << 20)
        ctx.set_loader_fusion(mode)
        got[mode] = ctx.step(tok, lab, 42, 1e-3, 0.0)
        assert ctx.plan()["loader_fusion"] == (mode == 1)
        ctx.close()
    for k in (0, 1):
        assert abs(float(got[1][k]) - float(got[-1][k])) <= 2e-3 * abs(float(got[-1][k]))


@pytest.mark.parametrize("d,f,vocab,rows,tied", [(64, 128, 212, 2, True), (192, 320, 1092, 17, False), (256, 1088, 2052, 32, True), (448, 576, 1091, 32, False), (192, 320, 260, 33, True)])
def test_bf16_loader_updates_as_the_sweep_does(d, f, vocab, rows, tied):
    """bfloat16: the projections' loader applies the pending update too up to 32 tokens, the sweep from 33 on.  The stored parameters are the sweep's
    bit for bit (features that end inside a workgroup's 128, one slab and several, heads that the loader takes or leaves), resident and
    streamed, over a pending update and a round of two directions; the losses are the ordinary path's but for the order of the float32 sums."""
    b = _b()
    cfg = si.tiny_config(n_layers=5, d_model=d, n_heads=d // 64, d_ffn=f, vocab=vocab, max_pos=80, tied=tied)
    P = si.make_weights(cfg, seed=11, std=0.05, ln_jitter=True)
    tok = si.make_tokens(vocab, 1, rows, seed=12)
    lab = si.next_token_labels(tok)
    got = {}
    for mode, streamed in ((1, 0), (-1, 0), (1, 1)):
        ctx = b.Zo2Context(cfg, P, wire="bf16", compute="bf16", arena_bytes=512 << 20)
        ctx.set_loader_fusion(mode)
        r = [ctx.step(tok, lab, 41, 1e-3, 0.0)]
        if streamed:
            ctx.set_resident_budget(ctx.plan()["bytes_used"] - 2 * ctx.offs[16] * 2)        # 3 slots for 5 blocks
            ctx.debug_set_slot_poison(True)
        ctx.set_pending(True, 7, 3e-3)
        r += [ctx.step(tok, lab, 42, 1e-3, 0.0), ctx.step(tok, lab, 43, 1e-3, 0.0), ctx.step_extra(tok, lab, 44, 1e-3, 0.0)]
        assert ctx.plan()["loader_fusion"] == (mode == 1) and ctx.plan()["resident"] == (not streamed)
        ctx.sync_to_host()
        got[mode, streamed] = ([float(x) for a in r for x in a[:2]], ctx.parameters())
        ctx.close()
    for x, y in zip(got[1, 0][0], got[-1, 0][0]):
        assert abs(x - y) <= 2e-3 * abs(y)
    assert got[1, 0][0] == got[1, 1][0]
    for n in P:
        assert np.array_equal(got[1, 0][1][n], got[-1, 0][1][n]) and np.array_equal(got[1, 0][1][n], got[1, 1][1][n]), n
    assert any(not np.array_equal(got[1, 0][1][n], codec.round_to(P[n], "bf16")) for n in P)


@pytest.mark.parametrize("dt,d,f,rows", [("f32", 64, 128, 2), ("bf16", 192, 320, 32), ("f32", 448, 1856, 33), ("bf16", 2112, 64, 9)])
def test_vectors_of_resident_blocks_in_one_launch(dt, d, f, rows):
    """Resident blocks have their vectors swept by one launch ahead of the first block, streamed ones block by block: the same losses and parameters
    bit for bit, with no update pending, with one, with the several of a round, and in a further direction at the same parameters; vectors
    that are a fraction of a workgroup's 2048 elements, and more."""
    b = _b()
    cfg = si.tiny_config(n_layers=6, d_model=d, n_heads=d // 64, d_ffn=f, vocab=2052, max_pos=80)
    P = si.make_weights(cfg, seed=11, std=0.05, ln_jitter=True)
    tok = si.make_tokens(2052, 1, rows, seed=12)
    lab = si.next_token_labels(tok)
    got = []
    for streamed in (False, True):
        ctx = b.Zo2Context(cfg, P, wire=dt, compute=dt, arena_bytes=2 << 30)
        ctx.set_loader_fusion(1)
        r = [ctx.step(tok, lab, 41, 1e-3, 1e-4)]
        if streamed:
            ctx.set_resident_budget(ctx.plan()["bytes_used"] - 3 * ctx.offs[16] * (4 if dt == "f32" else 2))        # 3 slots for 6 blocks
            ctx.debug_set_slot_poison(True)
        r += [ctx.step(tok, lab, 42, 1e-3, 1e-4), ctx.step_extra(tok, lab, 43, 1e-3, 1e-4), ctx.step_extra(tok, lab, 44, 1e-3, 1e-4), ctx.step(tok, lab, 45, 1e-3, 1e-4)]
        assert ctx.plan()["loader_fusion"] and ctx.plan()["resident"] == (not streamed)
        ctx.flush(); ctx.sync_to_host()
        got.append(([float(x) for a in r for x in a], ctx.parameters()))
        ctx.close()
    assert got[0][0] == got[1][0] and all(np.isfinite(got[0][0]))
    for n in P:
        assert np.array_equal(got[0][1][n], got[1][1][n]), n


@pytest.mark.parametrize("dt,d,f,rows", [("bf16", 2048, 8192, 16), ("bf16", 2048, 6144, 30), ("bf16", 1536, 6144, 9), ("f16", 2048, 8192, 16), ("f32", 512, 2048, 40)])
def test_a_flush_does_not_show_in_the_losses_behind_it(dt, d, f, rows):
    """An update that the loader applies and one that a flush has applied before leave the same parameters, and the step behind them adds
    its products in the same order: the losses are the same bits."""
    b = _b()
    cfg = si.tiny_config(n_layers=2, d_model=d, n_heads=d // 64, d_ffn=f, vocab=8196, max_pos=40)
    P = si.make_weights(cfg, seed=11, std=0.02, ln_jitter=True)
    tok = si.make_tokens(8196, 1, rows, seed=12)
    lab = si.next_token_labels(tok)
    got = []
    for flush in (False, True):
        ctx = b.Zo2Context(cfg, P, wire=dt, compute=dt, arena_bytes=2 << 30)
        ctx.set_loader_fusion(1)
        r = [ctx.step(tok, lab, 41, 1e-3, 1e-4)]
        if flush:
            ctx.flush()
        r.append(ctx.step(tok, lab, 42, 1e-3, 1e-4))
        assert ctx.plan()["loader_fusion"]
        got.append([float(x) for a in r for x in a])
        ctx.close()
    assert got[0] == got[1] and all(np.isfinite(got[0]))


@pytest.mark.parametrize("dt,d,f,rows", [("bf16", 2048, 8192, 16), ("bf16", 2048, 8192, 30), ("bf16", 2560, 10240, 16), ("bf16", 1536, 6144, 20), ("f16", 2048, 8192, 16),
                                         ("f16", 1536, 6144, 9), ("bf16", 192, 320, 9), ("f32", 512, 2048, 40)])
def test_who_adds_a_projection_s_pieces_does_not_show(dt, d, f, rows):
    """The second FFN projection's pieces are added by the next LayerNorm or, in a round that goes through the blocks together and under smaller
    scratch sets, by a pass of their own.  Kernel and pieces are the shape's: the same losses and parameters bit for bit."""
    b = _b()
    vocab = max(3 * d, f) + 4 if dt == "f32" else 260
    cfg = si.tiny_config(n_layers=2, d_model=d, n_heads=d // 64, d_ffn=f, vocab=vocab, max_pos=40)
    P = si.make_weights(cfg, seed=11, std=0.03, ln_jitter=True)
    tok = si.make_tokens(vocab, 1, rows, seed=12)
    lab = si.next_token_labels(tok)
    got = {}
    for how in ("1", "2", "4", "multi"):
        ctx = b.Zo2Context(cfg, P, wire=dt, compute=dt, arena_bytes=2 << 30)
        ctx.set_loader_fusion(1)
        ctx.set_scratch_plan(0 if how == "multi" else int(how))
        r = []
        for seeds in ([41, 42], [51, 52, 53]):
            r += ctx.step_multi(tok, lab, seeds, 1e-3, 1e-4) if how == "multi" else [ctx.step(tok, lab, seeds[0], 1e-3, 1e-4)] + [ctx.step_extra(tok, lab, s, 1e-3, 1e-4) for s in seeds[1:]]
            waiting = ctx.pass_facts()[1]
        assert ctx.plan()["loader_fusion"] and waiting % 2 == 0
        ctx.flush(); ctx.sync_to_host()
        got[how] = ([float(x) for a in r for x in a], ctx.parameters(), waiting)
        ctx.close()
    assert got["1"][2] > got["2"][2]               # FC2's pieces waited here, and not there
    for how in ("2", "4", "multi"):
        assert got[how][0] == got["1"][0], how
        for n in P:
            assert np.array_equal(got[how][1][n], got["1"][1][n]), (how, n)
    assert all(np.isfinite(got["1"][0]))


@pytest.mark.parametrize("dt,rows", [("bf16", 16), ("f32", 40)])
def test_blocks_that_go_back_to_the_host_are_swept(dt, rows):
    """A streamed block's offload waits for its parameters: where the pass writes it back the sweep has updated it before its projections run, where
    the write-back interval lets it stay the loader does it (the projections' time says which: one draw a weight, 0.80 - 0.86 of that of two, and no less than that where the
    loader updates in both).  The losses and parameters of resident blocks, bit for bit."""
    b = _b()
    d, f, layers = 1536, 6144, 4
    cfg = si.tiny_config(n_layers=layers, d_model=d, n_heads=24, d_ffn=f, vocab=f + 4, max_pos=40)
    P = si.make_weights(cfg, seed=11, std=0.02, ln_jitter=True)
    tok = si.make_tokens(f, 1, rows, seed=12)
    lab = si.next_token_labels(tok)
    got, ms = {}, {}
    for interval in (0, 1, 16):                     # 0: resident
        ctx = b.Zo2Context(cfg, P, wire=dt, compute=dt, arena_bytes=4 << 30)
        ctx.set_loader_fusion(1)
        r = [ctx.step(tok, lab, 41, 1e-3, 1e-4)]
        if interval:
            ctx.set_resident_budget(ctx.plan()["bytes_used"] - ctx.offs[16] * (4 if dt == "f32" else 2))        # 3 slots for 4 blocks
            ctx.debug_set_slot_poison(True)
            ctx.set_writeback_interval(interval)
        r += [ctx.step(tok, lab, 42, 1e-3, 1e-4), ctx.step_extra(tok, lab, 43, 1e-3, 1e-4), ctx.step(tok, lab, 44, 1e-3, 1e-4)]
        ctx.set_profiling(["gemm"])
        times = []
        for k in range(8):
            r.append(ctx.step(tok, lab, 45 + k, 1e-3, 1e-4))
            times.append(ctx.kernel_times()["gemm"][0])
            assert (ctx.step_stats()["bytes_down"] > 0) == (interval == 1)
        ms[interval] = min(times)
        assert ctx.plan()["loader_fusion"] and ctx.plan()["resident"] == (not interval)
        ctx.set_profiling([])
        ctx.flush(); ctx.sync_to_host()
        got[interval] = ([float(x) for a in r for x in a], ctx.parameters())
        ctx.close()
    for interval in (1, 16):
        assert got[interval][0] == got[0][0]
        for n in P:
            assert np.array_equal(got[interval][1][n], got[0][1][n]), (interval, n)
    # (the least of eight passes: beside copies under way a single one takes up to a sixth longer)
    assert ms[1] < 0.93 * ms[16], ms


# bfloat16: skinny_few_kernel and, in FC2 of d 2048, all of d 4096 but FC1 and the head, skinny_rows_kernel, as in float32; 1 to 64 slabs a wavefront
@pytest.mark.parametrize("dt,d,f,vocab,rows", [("bf16", 2048, 8192, 4100, 16), ("bf16", 2048, 8192, 260, 31), ("bf16", 4096, 4096, 1028, 20), ("bf16", 768, 3072, 8196, 9),
                                               ("f32", 2048, 8192, 8196, 40), ("f32", 1024, 4096, 4100, 96)])
def test_updates_of_wide_blocks_reach_memory_as_the_sweep_s_do(dt, d, f, vocab, rows):
    """The loader stores theta' and forms theta' +- eps z in the registers behind it: over several updates of blocks whose wavefronts walk many slabs, every
    stored parameter is the sweep's, bit for bit."""
    b = _b()
    cfg = si.tiny_config(n_layers=2, d_model=d, n_heads=d // 64, d_ffn=f, vocab=vocab, max_pos=100, tied=False)
    P = si.make_weights(cfg, seed=11, std=0.05, ln_jitter=True)
    tok = si.make_tokens(vocab, 1, rows, seed=12)
    lab = si.next_token_labels(tok)
    got = {}
    for mode in (1, -1):
        ctx = b.Zo2Context(cfg, P, wire=dt, compute=dt, arena_bytes=4 << 30)
        ctx.set_loader_fusion(mode)
        for k in range(6):
            ctx.set_pending(True, 100 + k, 1e-3 * (k + 1))
            ctx.step(tok, lab, 42 + k, 1e-3, 0.0)
        assert ctx.plan()["loader_fusion"] == (mode == 1)
        ctx.sync_to_host()
        got[mode] = ctx.parameters()
        ctx.close()
    for n in P:
        assert np.array_equal(got[1][n], got[-1][n]), n
        assert not np.array_equal(got[1][n], P[n]), n


def test_float32_products_of_tiny_weights_see_the_pending_update():
    """FC1's weights of 2^-100, updated by as much on the way: its sums are computed once more with float32 products, from theta' as the loader has
    stored it.  FC2's weights of 2^100 bring them back to the residual stream's size; an update of that coefficient is nothing to the other tensors."""
    b = _b()
    cfg = si.tiny_config(n_layers=2, d_model=128, n_heads=2, d_ffn=192, vocab=516, max_pos=40)
    P = si.make_weights(cfg, seed=11, std=0.05, ln_jitter=False)
    for l in range(2):
        P[f"blocks.{l}.fc1.w"] = P[f"blocks.{l}.fc1.w"] * np.float32(2.0 ** -100)
        P[f"blocks.{l}.fc1.b"] = np.zeros_like(P[f"blocks.{l}.fc1.b"])
        P[f"blocks.{l}.fc2.w"] = P[f"blocks.{l}.fc2.w"] * np.float32(2.0 ** 100)
    tok = si.make_tokens(cfg["vocab"], 1, 35, seed=12)
    lab = si.next_token_labels(tok)
    c = np.float32(2.0 ** -105)
    want = []
    for pending in ((c, 7, 1.0), None):
        oz = zo_step.Zo2Blockwise(opt_model.OptShape(**cfg), copy.deepcopy(P))
        oz.pending = pending
        want.append(oz.step(tok, lab, 42, 1e-33, 0.0))
    assert abs(float(want[0][0]) - float(want[1][0])) > 1e-3 * abs(float(want[0][0]))       # the update matters to the loss
    for update, w in zip((True, False), want):
        ctx = b.Zo2Context(cfg, P, arena_bytes=128 << 20)
        ctx.set_loader_fusion(1)
        if update:
            ctx.set_pending(True, 7, float(c))
        got = ctx.step(tok, lab, 42, 1e-33, 0.0)
        assert ctx.plan()["loader_fusion"]
        for k in (0, 1):
            assert abs(float(got[k]) - float(w[k])) <= 1e-5 * abs(float(w[k])), (got, w)
        ctx.close()


@pytest.mark.parametrize("dt,rows,interval,sweeps", [("bf16", 16, 1, 0), ("bf16", 16, 4, 0), ("bf16", 32, 3, 4), ("f32", 40, 1, 0), ("f32", 40, 4, 2)])
def test_streamed_rounds_of_few_tokens_equal_resident_steps(dt, rows, interval, sweeps):
    """Streamed blocks, written back on every update or on every third or fourth, rounds in one pass and in several, whatever the scratch: the losses
    and parameters of resident blocks bit for bit, with the update in the loader where it may be there."""
    b = _b()
    cfg = si.tiny_config(n_layers=5, d_model=192, n_heads=3, d_ffn=320, vocab=580, max_pos=80)
    P = si.make_weights(cfg, seed=11, std=0.05, ln_jitter=True)
    tok = si.make_tokens(580, 1, rows, seed=12)
    lab = si.next_token_labels(tok)
    got = {}
    for streamed in (0, 1, 2):                     # 2: rounds in one pass
        ctx = b.Zo2Context(cfg, P, wire=dt, compute=dt, arena_bytes=128 << 20)
        ctx.set_loader_fusion(1)
        if streamed and sweeps:
            ctx.set_scratch_plan(sweeps)
        r = [ctx.step(tok, lab, 41, 1e-3, 1e-4)]
        if streamed:
            ctx.set_resident_budget(ctx.plan()["bytes_used"] - 2 * ctx.offs[16] * (4 if dt == "f32" else 2) + 2 * (2 * rows * 192 * 4) + 4096)      # and two more residual streams
            ctx.debug_set_slot_poison(True)
            ctx.set_writeback_interval(interval)
        for k in range(4):
            seeds = [50 + 4 * k + j for j in range(1 + k % 3)]
            r += ctx.step_multi(tok, lab, seeds, 1e-3, 1e-4) if streamed == 2 else [ctx.step(tok, lab, seeds[0], 1e-3, 1e-4)] + [ctx.step_extra(tok, lab, s, 1e-3, 1e-4) for s in seeds[1:]]
        r.append(ctx.step(tok, lab, 90, 1e-3, 1e-4))
        assert ctx.plan()["loader_fusion"] and ctx.plan()["resident"] == (not streamed)
        ctx.flush(); ctx.sync_to_host()
        got[streamed] = ([float(x) for a in r for x in a], ctx.parameters())
        ctx.close()
    for streamed in (1, 2):
        assert got[streamed][0] == got[0][0]
        for n in P:
            assert np.array_equal(got[streamed][1][n], got[0][1][n]), (streamed, n)
    assert all(np.isfinite(got[0][0]))
