"""The LDS-staged kernel where its splits and passes end, against the oracle (MI355X).

A sequence takes part with as many splits as its own count needs: the splits past its end leave without a
partial, one split stores its output without a merge, and the merge (direct, in batches, two-level) is the one
for that number.  Batches here mix sequences of one position up to all splits, with counts one short of, at and
one past the ends of passes (32), of a pass of every wavefront (128 and 256) and of splits, on both workgroup
sizes (grids within and beyond one dispatch round), through the range table, the index list, the fused step
(retained-set outputs bit for bit) and ring storage, twice in a row (the tickets are back at zero).
The tolerances are those of the parity tests (fp32 output, row-RMS-floored relative error)."""
import numpy as np
import pytest

import oracle
from _tol import LSE_TOL, REL_TOL, lse_err, rel_err_fp32
from paper_2606_01483_amd import murmur as M
from paper_2606_01483_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def ragged(counts, layers=1, hq=14, hkv=2, seed=77):
    """Dense sequences that retain counts[b] positions at step 0: 3 prompt tokens, speech, and outputs."""
    seg0 = []
    for n in counts:
        prompt = min(3, n - 1)
        out = (n - prompt + 1) // 2
        seg0.append([prompt, n - prompt - out, 0, out - 1])
    return W.build("ragged", seed, layers, np.array(seg0, dtype=np.int32), np.array([W.OFF, 0, 0, W.OFF, 0]), 1,
                   planted=False, hq=hq, hkv=hkv)


def check(wl, db, run, what):
    idx, cnt = oracle.retained(wl.seg(0), wl.policy)
    ref, ref_lse = oracle.attend(wl.q(0), wl.k, wl.v, idx, cnt, scale=wl.scale)
    for again in range(2):
        print(f"[case] {what}, call {again}", flush=True)
        db.out.fill_(float("nan"))
        db.lse.fill_(float("nan"))
        run()
        torch.cuda.synchronize()
        assert M.murmur_device_error() == 0
        assert rel_err_fp32(db.out.cpu().numpy(), ref) <= REL_TOL, (what, again)
        assert lse_err(db.lse.cpu().numpy(), ref_lse) <= LSE_TOL, (what, again)
    return idx, cnt


EDGES = [1, 31, 32, 33, 127, 128, 129, 255, 256, 257, 287, 288, 289, 511, 512, 513, 575, 576, 577, 1151, 1153]


@pytest.mark.parametrize("split_len,layers", [(288, 1), (288, 4), (0, 1), (0, 8), (320, 2), (1024, 1)])
def test_ragged_split_ends(split_len, layers):
    from paper_2606_01483_amd.decode import DecodeBatch
    counts = EDGES if split_len != 288 else EDGES + [288 * 8, 288 * 8 + 1, 288 * 16, 288 * 16 + 1, 288 * 18 - 5]
    wl = ragged(counts, layers)
    for use_ranges in (True, False):
        db = DecodeBatch(wl, out_dtype=M.MURMUR_DTYPE_F32, steps=[0], split_len=split_len, use_ranges=use_ranges)
        check(wl, db, lambda: db.step(0), f"split_len {split_len}, {layers} layers, ranges {use_ranges}")
    for t in db.sets[0]:
        t.fill_(-7)
    idx, cnt = check(wl, db, lambda: db.step_fused(0), f"split_len {split_len}, {layers} layers, fused")
    assert np.array_equal(db.count.cpu().numpy(), cnt)
    assert np.array_equal(db.idx.cpu().numpy(), idx[:, :db.max_keep])


@pytest.mark.parametrize("split_len", [1184, 2**30, 2**31 - 32])
def test_one_long_split(split_len):
    """Split lengths from just above the longest sequence to the largest that is accepted: every group whole."""
    from paper_2606_01483_amd.decode import DecodeBatch
    wl = ragged(EDGES, 1)
    db = DecodeBatch(wl, out_dtype=M.MURMUR_DTYPE_F32, steps=[0], split_len=split_len)
    assert db.ws_bytes == 256
    for t in db.sets[0]:
        t.fill_(-7)
    idx, cnt = check(wl, db, lambda: db.step_fused(0), f"split_len {split_len}")
    assert np.array_equal(db.count.cpu().numpy(), cnt)
    assert np.array_equal(db.idx.cpu().numpy(), idx[:, :db.max_keep])


@pytest.mark.parametrize("split_len,layers", [(288, 1), (288, 4), (0, 1), (0, 8)])
@pytest.mark.parametrize("max_keep", [1154, 2305, 9001])
def test_index_list_longer_than_the_sequences(split_len, layers, max_keep):
    """Lists of more entries than any sequence retains: the entries past each count are -1, whether its last split
    or a split past its end covers them."""
    from paper_2606_01483_amd.decode import DecodeBatch
    wl = ragged(EDGES, layers)
    db = DecodeBatch(wl, out_dtype=M.MURMUR_DTYPE_F32, steps=[0], split_len=split_len, max_keep=max_keep)
    for t in db.sets[0]:
        t.fill_(-7)
    check(wl, db, lambda: db.step_fused(0), f"lists of {max_keep}, split_len {split_len}, {layers} layers")
    idx, cnt = oracle.retained(wl.seg(0), wl.policy, max_keep)
    assert np.array_equal(db.count.cpu().numpy(), cnt)
    assert np.array_equal(db.idx.cpu().numpy(), idx)


@pytest.mark.parametrize("hq,hkv", [(4, 4), (16, 1)])
def test_ragged_split_ends_group_sizes(hq, hkv):
    from paper_2606_01483_amd.decode import DecodeBatch
    wl = ragged(EDGES, 2, hq, hkv)
    db = DecodeBatch(wl, out_dtype=M.MURMUR_DTYPE_F32, steps=[0], split_len=288)
    check(wl, db, lambda: db.step(0), f"{hq} query heads, {hkv} KV heads")


@pytest.mark.parametrize("split_len", [0, 96, 288])
def test_ring_passes_around_the_current_row(split_len):
    """Ring storage of 2 MiB a layer, where every pass addresses its rows one by one: rings of exactly the window,
    the current token's row (whose K/V come with the call) at their start, middle and end.  Streamed launches, which
    take consecutive rows beside it, are test_gpu_ring.py's."""
    from paper_2606_01483_amd.decode import RingBatch
    cap = 40
    seg0 = np.array([[5, 300, 0, 40 + d] for d in (0, 1, 7, 31, 38, 39)], dtype=np.int32)
    wl = W.build("ring", 78, 2, seg0, np.array([W.OFF, 0, 0, cap, 0]), 2, planted=False, hq=14, hkv=2)
    rb = RingBatch(wl, cap, out_dtype=M.MURMUR_DTYPE_F32, steps=[0, 1], split_len=split_len)
    for i in range(2):
        print(f"[case] ring split_len {split_len} step {i}", flush=True)
        rb.step(i)
        torch.cuda.synchronize()
        assert M.murmur_device_error() == 0
        idx, cnt = oracle.retained(wl.seg(i), wl.policy)
        ref, ref_lse = oracle.attend(wl.q(i), wl.k, wl.v, idx, cnt, scale=wl.scale)
        assert rel_err_fp32(rb.out.cpu().numpy(), ref) <= REL_TOL
        assert lse_err(rb.lse.cpu().numpy(), ref_lse) <= LSE_TOL


@pytest.mark.parametrize("rows", [2047, 2048, 2049])
def test_streamed_loads_on_both_sides_of_their_line(rows):
    """Launches just under and over 12 MiB of K/V per layer (6144 positions of 4 KV heads), where the loads' cache
    policy changes."""
    from paper_2606_01483_amd.decode import DecodeBatch
    wl = ragged([rows, rows, rows], 1, 28, 4)
    db = DecodeBatch(wl, out_dtype=M.MURMUR_DTYPE_F32, steps=[0])
    check(wl, db, lambda: db.step_fused(0), f"3 x {rows} positions")


@pytest.mark.parametrize("scale", [1e6, -1e6, 1e12, -1e12, 1e30])
@pytest.mark.parametrize("split_len,layers", [(96, 1), (288, 1), (288, 8)])
def test_logits_far_apart(split_len, layers, scale):
    """Logits whose spacing in fp32 is far above one: the weights are one-hot and every exponent stays in range.
    lse is the largest logit then, so the tolerances of ordinary logits hold."""
    from paper_2606_01483_amd.decode import DecodeBatch
    wl = ragged([64, 300, 577, 700], layers)
    wl.scale = scale
    db = DecodeBatch(wl, out_dtype=M.MURMUR_DTYPE_F32, steps=[0], split_len=split_len)
    check(wl, db, lambda: db.step_fused(0), f"scale {scale}, split_len {split_len}, {layers} layers")


def equal_logits(counts, layers):
    """Heads whose logits are the same at every position, of magnitudes 2^9 to 2^26 in log2 units, and one whose
    logits rise across 2^16 with the rank (their top value at the last positions of a sequence, over more than
    one pass of 32 wherever there is one)."""
    wl = ragged(counts, layers)
    k = np.zeros(wl.k.shape, dtype=np.float32)
    k[..., 0] = 1.3046875
    for b, n in enumerate(counts):
        k[:, b, :, :n, 1] = 2.0 ** np.minimum(np.arange(n) * 4 // max(1, n - 40), 3)
    past = wl.k == W.BF16_NAN
    wl.k = np.where(past, wl.k, W.f32_to_bf16_bits(k))
    q = np.zeros((layers, wl.batch, wl.hq, 128), dtype=np.float32)
    group = wl.hq // wl.hkv
    x = np.array([0.7 * 2**9, 1.3 * 2**14, 1.6 * 2**23, 1.7 * 2**24, -1.3 * 2**14, 0, 1])[:group]
    q[..., 0] = np.tile(x, wl.hkv)
    q[..., group - 2::group, 1] = 0.7 * 2**14  # x is 0 for this head
    bits = W.f32_to_bf16_bits(q)
    wl.q = lambda step: bits
    return wl


@pytest.mark.parametrize("scale", [1.0, -1.0, 0.0])
@pytest.mark.parametrize("split_len,layers", [(96, 1), (288, 1), (288, 8), (1024, 1)])
def test_equal_logits_weigh_the_same_in_every_pass(split_len, layers, scale):
    """A position's weight does not depend on the pass that holds it, whole or a sequence's last partial one, nor
    on the other heads of its group: with equal logits the output is the mean of V.  Bound: the weights carry 17
    bits (bf16 hi + lo) and cancel against their own sum, 2^-17 in relative terms, times four."""
    from paper_2606_01483_amd.decode import DecodeBatch
    counts = [33, 40, 47, 63, 95, 129, 300, 577, 1100]
    wl = equal_logits(counts, layers)
    wl.scale = scale
    for use_ranges in (True, False):
        db = DecodeBatch(wl, out_dtype=M.MURMUR_DTYPE_F32, steps=[0], split_len=split_len, use_ranges=use_ranges)
        idx, cnt = check(wl, db, lambda: db.step(0), f"equal logits, split_len {split_len}, scale {scale}")
        assert cnt.tolist() == counts
        ref, _ = oracle.attend(wl.q(0), wl.k, wl.v, idx, cnt, scale=wl.scale)
        err = rel_err_fp32(db.out.cpu().numpy(), ref)
        assert err <= 4 * 2.0**-17
