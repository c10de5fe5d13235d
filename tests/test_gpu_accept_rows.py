"""GPU parity of the vocabulary scan on rows that start at any element: a
vocabulary that is no multiple of a 16-byte vector leaves entries before and
after the aligned vectors of each row.  Ids exact; probabilities 1e-4 relative,
as in the other accept tests."""

import numpy as np
import pytest
import torch

import oracle
from gpu_util import check_accept, dev_tensor, int_tensor
from synth import bf16_bits_from_f32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("V", [1, 2, 7, 9, 15, 17, 31, 2049, 2055, 8191, 20007])
def test_unaligned_rows(dtype, V):
    """16 rows, so every alignment of a row start; per row the maximum (or a tie
    of two, or a masked vocabulary with -inf entries) at the row's first, last
    and middle entries; library's and forced chunk counts."""
    from paper_2606_02544_amd import binding
    rng = np.random.default_rng(V)
    b, B = 2, 8
    x = (rng.standard_normal((b, B, V)) * 2).clip(-12, 12).astype(np.float32)
    places = [0, V - 1, V // 2, min(1, V - 1), max(V - 2, 0), V // 3, min(8, V - 1), V * 2 // 3]
    for k in range(B):
        x[0, k, places[k]] = 13.0
        x[1, k, [places[k], places[(k + 3) % B]]] = 13.0           # ties
    if V > 4:
        x[1, 5, 1::2] = -np.inf
        x[1, 5, 0] = 13.0
        x[1, 6, : V - 1] = -np.inf                                 # one entry left, the last
        x[1, 6, V - 1] = 1.0
    step = np.array([[1, 2, 3, 4, 5, 6, 7, 8], [8, 7, 6, 5, 4, 3, 2, 1]], np.int32)
    gamma = np.array([8, 8], np.int32)
    stored = bf16_bits_from_f32(x) if dtype == "bf16" else x
    wide = x if dtype == "f32" else (stored.astype(np.uint32) << 16).view(np.float32)
    drafts = np.zeros((b, 8), np.int32)
    for s in range(b):
        for k in range(B):
            drafts[s, step[s, k] - 1] = int(np.argmax(wide[s, k]))
    drafts[1, 4] = V - 1
    ref = oracle.verify_accept(stored, drafts, step, gamma, dtype)
    for cpr in (0, 1, 2, 5):
        got = binding.verify_accept(dev_tensor(stored, dtype), int_tensor(drafts), int_tensor(step),
                                    int_tensor(gamma), chunks_per_row=cpr)
        torch.cuda.synchronize()
        check_accept(tuple(t.cpu().double().numpy() if t.dtype == torch.float32 else t.cpu().numpy()
                           for t in got), ref)


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("V", [2, 9, 2055, 20007, 20008])
def test_nan_and_inf_at_row_ends(dtype, V, bad):
    """A NaN or +inf as a row's first or last entry, on rows of every alignment:
    the probabilities are NaN wherever the entry falls; NaN is never the target
    and +inf is."""
    from paper_2606_02544_amd import binding
    rng = np.random.default_rng(V)
    b, B = 2, 8
    x = (rng.standard_normal((b, B, V)) * 2).clip(-12, 12).astype(np.float32)
    x[0, :, 0] = bad
    x[1, :, V - 1] = bad
    stored = bf16_bits_from_f32(x) if dtype == "bf16" else x
    if np.isnan(bad) and dtype == "bf16":
        stored[np.isnan(x)] = 0x7fc0
    wide = np.where(np.isnan(x), -np.inf, x if dtype == "f32" else (stored.astype(np.uint32) << 16).view(np.float32))
    step = np.tile(np.arange(1, B + 1, dtype=np.int32), (b, 1))
    target = wide.argmax(-1).astype(np.int32)
    for cpr in (0, 2):
        t, c, p, a = binding.verify_accept(dev_tensor(stored, dtype), int_tensor(target), int_tensor(step),
                                           int_tensor(np.full(b, B)), chunks_per_row=cpr)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(t.cpu().numpy(), target)
        assert torch.all(a == B)
        assert torch.all(torch.isnan(c)) and torch.all(torch.isnan(p)), (cpr, c, p)
