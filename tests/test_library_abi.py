"""The C-ABI library loads and exports every symbol the header declares (no GPU needed)."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "zo2.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(zo2_[a-z0-9_]+)\s*\(", text)))


def test_header_declares_the_step_api():
    names = _declared()
    for must in ("zo2_init", "zo2_step", "zo2_set_resident_budget", "zo2_flush", "zo2_sync_to_host", "zo2_destroy"):
        assert must in names


def test_library_exports_every_declared_symbol():
    from paper_2503_12668_amd import binding
    L = binding.lib()
    for name in _declared():
        assert hasattr(L, name), name
    assert sorted(binding.EXPORTED) == _declared()


def test_layout_helpers_and_argument_errors():
    from paper_2503_12668_amd import binding
    import synth_inputs as si
    L = binding.lib()
    assert [L.zo2_dtype_size(i) for i in range(6)] == [4, 2, 2, 1, 1, 0]
    cfg = si.opt_config("opt-125m")
    offs = binding.block_tensor_offsets(binding.make_config(cfg))
    d, f = 768, 3072
    sizes = [d, d, d * d, d, d * d, d, d * d, d, d * d, d, d, d, f * d, f, d * f, d]
    assert offs[0] == 0 and all(o % 256 == 0 for o in offs)
    for k in range(16):
        assert offs[k + 1] - offs[k] >= sizes[k] and offs[k + 1] - offs[k] < sizes[k] + 256
    bad = dict(cfg, d_model=770)
    with pytest.raises(binding.Zo2Error):
        binding.block_tensor_offsets(binding.make_config(bad))
    # NULL context
    assert L.zo2_flush(None) == 1 and L.zo2_step(None, None, None, 1, 1, 0, 1e-3, 0.0, None, None, None) == 1


def test_split_gemm_refuses_operands_that_its_kernels_cannot_load():
    """Refused on the host before anything is launched: the addresses are nobody's."""
    from paper_2503_12668_amd import binding
    L = binding.lib()

    def call(X=1 << 16, W=1 << 16, ldx=1024, ldw=1024, Y=1 << 16, ldy=64, K=1024, splits=2):
        return L.zo2_op_gemm_split_k(binding.BF16, 64, 64, K, X, ldx, W, ldw, None, None, Y, binding.F32, ldy, 1.0, 0, splits, 1 << 16, 1 << 30, None)

    for bad in (dict(X=(1 << 16) + 8), dict(W=(1 << 16) + 2), dict(ldx=1028), dict(ldw=1020), dict(ldw=504), dict(ldx=8), dict(K=1032, splits=4), dict(X=None)):
        assert call(**bad) == 1, (bad, L.zo2_op_last_error())


def test_attention_of_columns_of_a_packed_tensor_gets_a_result_with_the_same_rows(monkeypatch):
    """The kernels write the result at q's distance between rows: the memory handed to them reaches as far.  (Nothing is launched.)"""
    import torch
    from paper_2503_12668_amd import binding
    calls = []

    class Recorder:
        def zo2_op_attention(self, *args):
            calls.append(args)
            return 0

    monkeypatch.setattr(binding, "lib", lambda: Recorder())
    monkeypatch.setattr(binding, "_stream_ptr", lambda stream=None: None)
    rows, d = 6, 128
    packed = torch.zeros(rows, 3 * d)
    q, k, v = packed.split(d, dim=1)
    for args in ((q, k, v), (packed[:, :d].contiguous(),) * 3, tuple(t.view(rows, 2, 64) for t in (packed[:, :d].contiguous(),) * 3)):
        out = binding.op_attention(*args, 2, 3, 2, 64)
        ld = calls[-1][9]
        assert ld == args[0].stride(0) and calls[-1][4].value == out.data_ptr()
        assert out.untyped_storage().nbytes() >= 4 * ((rows - 1) * ld + d) and out.shape == args[0].shape
    dense = q.contiguous()
    for args in ((q, dense, dense), (dense, k, dense), (dense, dense, v), (dense.t().contiguous().t(),) * 3):
        with pytest.raises(ValueError):
            binding.op_attention(*args, 2, 3, 2, 64)
    assert len(calls) == 3
