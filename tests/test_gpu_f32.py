"""GPU parity of the fp32 attention kernel at the edges of its tiling: 16-key
sub-tiles dealt to four waves, work-groups of one or two 16-row blocks, the new
slots as one more sub-tile per wave.  Same tolerance as the other fp32 tests
(1e-5 absolute: outputs are averages of N(0, 1) values, so a sum over n keys is
off by a few ulps of 1, about sqrt(n) * 6e-8 < 2e-6 at n = 1100)."""

import numpy as np
import pytest

import oracle
from gpu_util import DeviceInputs, run_attention, check_attention
from synth import VerifyConfig, generate

pytestmark = pytest.mark.gpu

CASES = [
    # head_dim, Hq, Hkv, B, L, prefix, page, kv_chunk, theta (small: 16-row work-groups)
    (128, 1, 1, 1, 0, (1, 1), 0, 0, 0.0),          # one row, one key: three waves idle
    (128, 2, 1, 4, 4, (15, 17), 0, 0, 0.0),        # 16 rows; around one sub-tile
    (128, 4, 2, 8, 1, (63, 65), 16, 0, 0.0),       # 18 rows: two blocks, around a chunk
    (128, 4, 1, 8, 1, (0, 40), 3, 0, 0.0),         # 36 rows: a second, partial row block
    (64, 16, 1, 1, 1, (47, 130), 0, 64, 0.0),      # 32 rows exactly, several splits
    (64, 8, 8, 32, 32, (0, 200), 64, 128, 0.0),    # 64 new slots: a sub-tile on every wave
    (128, 16, 2, 24, 24, (300, 1100), 16, 0, 0.0),  # 384 rows, long ranges per wave
    (128, 2, 2, 8, 8, (0, 100), 0, 64, 1e6),       # rotary: 16 rows, has_new with no prefix items
    (64, 12, 2, 17, 16, (5, 333), 8, 64, 1e4),     # rotary: slots shared by two row blocks
    (128, 3, 1, 32, 32, (0, 90), 0, 0, 1e6),       # rotary: 64 rotated keys, 192 rows
]
# The same with enough sequences for 32-row work-groups.
LARGE = [
    (128, 16, 8, 9, 1, (0, 900), 0, 0, 0.0),       # 20 rows: the second block partial
    (64, 16, 8, 8, 8, (700, 900), 16, 0, 0.0),     # 32 rows exactly, paged
    (128, 24, 8, 8, 7, (0, 450), 5, 0, 1e6),       # 45 rows: a second, partial group; rotary
    (64, 32, 8, 11, 11, (0, 450), 0, 64, 1e4),     # 88 rows, 64-key splits, rotary
]


@pytest.mark.parametrize("case", CASES + LARGE, ids=lambda c: "-".join(map(str, c)))
def test_f32_tiles(case):
    d, hq, hkv, B, L, prefix, page, kv_chunk, theta = case
    cfg = VerifyConfig(0, "f32", "f32", batch=16 if case in LARGE else 4, num_q_heads=hq, num_kv_heads=hkv, head_dim=d,
                       prefix=prefix, block_size=B, max_ref=L, vocab=100, page_size=page,
                       qkv_std=1.0, step_mode="mixed" if L else "full")
    inp = generate(cfg, seed=500 + d + B, poison=True)
    out, lse = run_attention(DeviceInputs(inp), kv_chunk, rope_theta=theta)
    ref_out, ref_lse = oracle.verify_attention(inp, rope_theta=theta)
    check_attention(out, lse, ref_out, ref_lse, "f32")


@pytest.mark.parametrize("prefix,B,L", [(37, 5, 3), (16, 9, 8), (1, 1, 0)])
def test_f32_infinite_last_value(prefix, B, L):
    """An infinity among the values of the prefix's or the block's last key
    reaches the rows that see the key as an infinity, also where the key's 16-key
    sub-tile has no other keys to fill it; the other dims are untouched."""
    cfg = VerifyConfig(0, "f32", "f32", batch=2, num_q_heads=4, num_kv_heads=2, head_dim=64,
                       prefix=(prefix, prefix), block_size=B, max_ref=L, vocab=100, qkv_std=0.5)
    inp = generate(cfg, seed=540 + prefix)
    clean = run_attention(DeviceInputs(inp), 64)[0]
    inp.v_cache[:, prefix - 1, :, 3] = np.inf
    inp.v_cache[:, prefix - 1, :, 40] = -np.inf
    # The last slot is a verification row, or a block slot where nothing is drafted.
    inp.v_new[:, -1, :, 7] = np.inf
    out = run_attention(DeviceInputs(inp), 64)[0]
    assert np.all(out[..., 3] == np.inf) and np.all(out[..., 40] == -np.inf)
    assert np.all(out[:, -1, :, 7] == np.inf)
    rest = np.delete(np.arange(64), (3, 7, 40))
    np.testing.assert_array_equal(out[..., rest], clean[..., rest])


@pytest.mark.parametrize("prefix,scale", [(90, 1e18), (90, 1e4), (700, 3e9), (5, 1e18)])
def test_f32_huge_scores(prefix, scale):
    """Scores past 2^24 and up to near the largest float: the largest one takes
    all the weight, and its row's output is that key's value."""
    cfg = VerifyConfig(0, "f32", "f32", batch=2, num_q_heads=8, num_kv_heads=2, head_dim=64,
                       prefix=(prefix, prefix), block_size=8, max_ref=5, vocab=100, qkv_std=1.0)
    inp = generate(cfg, seed=560 + prefix)
    for x in (inp.q, inp.k_new, inp.k_cache):
        x *= np.float32(scale)
    ref_out, ref_lse = oracle.verify_attention(inp)
    assert np.abs(ref_lse).max() > 1e7
    for chunk in (0, 64):
        out, lse = run_attention(DeviceInputs(inp), chunk)
        check_attention(out, lse, ref_out, ref_lse, "f32")


def test_f32_huge_values():
    """Values near the largest float, at a key whose score passes those before
    it: their weighted sum, three times 1e38 at most, does not overflow."""
    d, prefix = 64, 300
    cfg = VerifyConfig(0, "f32", "f32", batch=1, num_q_heads=4, num_kv_heads=2, head_dim=d,
                       prefix=(prefix, prefix), block_size=8, max_ref=8, vocab=100, qkv_std=1.0)
    inp = generate(cfg, seed=580)
    u = inp.q[0, 0, 0].copy()
    inp.q[:] = u
    for key in (70, 180, 299):                 # second to fifth sub-tiles of their waves
        inp.k_cache[0, key] = u * (4.5 * np.sqrt(d) / np.dot(u, u))
        inp.v_cache[0, key, :, 9] = 1e38
    ref_out, ref_lse = oracle.verify_attention(inp)
    assert 3e37 < ref_out[..., 9].min()
    rest = np.delete(np.arange(d), 9)
    for chunk in (0, 64, 320):
        out, lse = run_attention(DeviceInputs(inp), chunk)
        np.testing.assert_allclose(out[..., 9], ref_out[..., 9], rtol=1e-5)
        check_attention(out[..., rest], lse, ref_out[..., rest], ref_lse, "f32")
