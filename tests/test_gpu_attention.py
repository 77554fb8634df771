"""GPU parity of the attention stage by itself: attention_forward (the kernels encoder_forward runs on
the output of its q | k | v BitLinear) against the oracle's causal_gqa_attention, element by element.

Five forms sit behind the entry point and every one is reached here in both layouts: attention_f32_kernel
(BRL_ATTN_F32), attn_pack_kernel + attention_frag_kernel (BRL_ATTN_MFMA), for states of at most 32 tokens
attention_short_kernel (a workgroup per query head) and attention_group_kernel (per four of them), and for heads of
128 and states of at most 64 tokens attention_rows_kernel.

Bound.  The oracle works in fp64 and rounds once.  The fp32 kernel accumulates dot products of
head_dim terms and the softmax sums in fp32; the matrix-core kernels carry every operand as an fp16
hi + lo pair (22 significant bits, the lo * lo term dropped) and accumulate in fp32.  With q, k, v of
unit scale a score then carries an absolute error of a few 1e-7 * sqrt(head_dim) before the
exponential, i.e. the probabilities a relative error of a few 1e-6, and the output (a convex
combination of v rows) the same relative to max|v|.  ATTN_REL below is that figure with a margin;
sharper softmaxes (inputs of three times the scale: nine times the score range) get nine times the
bound.
"""
import numpy as np
import pytest

from oracle import bitrl_oracle as O
from paper_2604_24273_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

ATTN_REL = 2e-6          # max |out - ref| / max |ref| per state, unit-scale inputs, either precision
                         # (largest seen over every case below: 5.3e-7 fp32, 4.1e-7 matrix cores; sharp case 3.5e-6)


def _mods():
    from paper_2604_24273_amd import binding as B
    from paper_2604_24273_amd import runtime as R
    B.lib()
    return B, R


def _run(B, R, qkv, lens, uniform_S, hq, hkv, dh, theta, prec, max_len=None):
    T = qkv.shape[0]
    nb = len(lens)
    out = torch.full((T, hq * dh), float("nan"), dtype=torch.float32, device="cuda")
    if uniform_S is not None:
        S, cu_dev, cu = uniform_S, None, None
    else:
        cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        cu_dev = R.dev(cu)
        S = max(lens) if max_len is None else max_len
    ws = R.Workspace(B.brl_attention_workspace_bytes(nb, S, hq, hkv, dh))
    B.attention_forward(R.dev(qkv), nb, S, cu_dev, cu, hq, hkv, dh, theta, prec, out, ws.buf)
    torch.cuda.synchronize()
    return out.cpu().numpy()


def _oracle(qkv, lens, hq, hkv, dh, theta):
    outs, r0 = [], 0
    for n in lens:
        rows = qkv[r0:r0 + n]
        q = rows[:, :hq * dh].reshape(n, hq, dh)
        k = rows[:, hq * dh:(hq + hkv) * dh].reshape(n, hkv, dh)
        v = rows[:, (hq + hkv) * dh:].reshape(n, hkv, dh)
        outs.append(O.causal_gqa_attention(q, k, v, theta))
        r0 += n
    return outs


def _check(got, refs, lens, rel):
    r0, worst = 0, 0.0
    for n, ref in zip(lens, refs):
        g = got[r0:r0 + n].astype(np.float64)
        assert np.all(np.isfinite(g)), "rows of a state were not written"
        err = np.abs(g - ref.astype(np.float64)).max() / np.abs(ref).max()
        worst = max(worst, err)
        r0 += n
    print("   worst max|d|/max|ref| over %d states: %.3e (bound %.1e)" % (len(lens), worst, rel), flush=True)
    assert worst <= rel, "attention error %.3e above %.1e" % (worst, rel)


CASES = [
    # (head_dim, n_heads, n_kv_heads, state lengths, uniform layout?, rope theta)
    (128, 20, 5, [128, 128, 128], True, 500000.0),          # the 2B shape, one state = one 128-token block row
    (128, 4, 1, [1], True, 500000.0),
    (128, 4, 1, [32, 32], True, 500000.0),                    # one key block, uniform: the one-kernel path
    (128, 4, 1, [33, 33], True, 500000.0),                    # one token into the second key block
    (100, 4, 4, [512], True, 10000.0),                        # the 3B head: 100 components padded to 128, 16 key blocks
    (100, 2, 2, [33, 7, 70], False, 10000.0),
    (100, 2, 2, [19, 32, 5], False, 10000.0),                 # short states, head_dim 100
    (16, 8, 1, [9, 40, 64], False, 10000.0),                  # eight query heads per key/value head
    (16, 8, 1, [9, 31], False, 10000.0),
    (32, 8, 8, [31, 17, 32], False, 10000.0),
    (64, 4, 2, [15, 40, 1, 32, 33, 27, 64, 31], False, 10000.0),
    (64, 8, 1, [15, 27, 1, 32, 8], False, 10000.0),           # 8:1 grouping, all short
    (128, 8, 2, [129, 2, 96, 18, 40], False, 500000.0),
]


@pytest.mark.parametrize("prec", ["f32", "mfma"])
@pytest.mark.parametrize("dh,hq,hkv,lens,uniform,theta", CASES)
def test_attention_stage_against_oracle(dh, hq, hkv, lens, uniform, theta, prec):
    B, R = _mods()
    print("attention_forward", dh, hq, hkv, lens, uniform, prec, flush=True)
    T = int(np.sum(lens))
    qkv = synth.normal(7, 600 + dh + len(lens), (T, (hq + 2 * hkv) * dh))
    p = B.BRL_ATTN_F32 if prec == "f32" else B.BRL_ATTN_MFMA
    got = _run(B, R, qkv, lens, lens[0] if uniform else None, hq, hkv, dh, theta, p)
    _check(got, _oracle(qkv, lens, hq, hkv, dh, theta), lens, ATTN_REL)
    if not uniform:
        # a larger bound on the lengths changes nothing, bit for bit
        again = _run(B, R, qkv, lens, None, hq, hkv, dh, theta, p, max_len=max(lens) + 37)
        assert np.array_equal(got, again)


@pytest.mark.parametrize("prec", ["f32", "mfma"])
def test_attention_sharp_softmax(prec):
    """Inputs of three times the scale: scores range over about +-30, the running-maximum form must hold."""
    B, R = _mods()
    dh, hq, hkv, lens = 128, 4, 2, [96, 40, 23]
    qkv = synth.normal(7, 650, (int(np.sum(lens)), (hq + 2 * hkv) * dh), 3.0)
    p = B.BRL_ATTN_F32 if prec == "f32" else B.BRL_ATTN_MFMA
    got = _run(B, R, qkv, lens, None, hq, hkv, dh, 500000.0, p)
    _check(got, _oracle(qkv, lens, hq, hkv, dh, 500000.0), lens, 9 * ATTN_REL)


def test_attention_many_short_states_take_the_two_kernel_path():
    """More than 1024 (state, key/value head) workgroups of short states: the pack + fragment kernels run
    with a single key block.  The same rows through the one-kernel path (few states per call) must agree with
    the oracle to the same bound; both are compared with it."""
    B, R = _mods()
    dh, hq, hkv = 64, 4, 4
    lens = [int(n) for n in synth.state_lengths(7, 660, 300, 1, 32)]       # 300 x 4 = 1200 workgroups
    qkv = synth.normal(7, 661, (int(np.sum(lens)), (hq + 2 * hkv) * dh))
    refs = _oracle(qkv, lens, hq, hkv, dh, 10000.0)
    got = _run(B, R, qkv, lens, None, hq, hkv, dh, 10000.0, B.BRL_ATTN_MFMA)
    _check(got, refs, lens, ATTN_REL)
    few = 40
    t_few = int(np.sum(lens[:few]))
    got_few = _run(B, R, qkv[:t_few], lens[:few], None, hq, hkv, dh, 10000.0, B.BRL_ATTN_MFMA)
    _check(got_few, refs[:few], lens[:few], ATTN_REL)
    # same block arithmetic in both kernels: identical bits
    assert np.array_equal(got[:t_few], got_few)


def test_attention_is_causal_and_state_local():
    """Changing the tokens behind a position, or another state, leaves that position's output unchanged bit
    for bit (a property that holds at any size; both precisions)."""
    B, R = _mods()
    dh, hq, hkv, lens = 128, 4, 1, [70, 45]
    T = int(np.sum(lens))
    qkv = synth.normal(7, 670, (T, (hq + 2 * hkv) * dh))
    other = qkv.copy()
    other[50:70] = synth.normal(7, 671, (20, qkv.shape[1]))     # the tail of state 0
    other[70:] = synth.normal(7, 672, (45, qkv.shape[1]))       # all of state 1
    for p in (B.BRL_ATTN_F32, B.BRL_ATTN_MFMA):
        a = _run(B, R, qkv, lens, None, hq, hkv, dh, 500000.0, p)
        b = _run(B, R, other, lens, None, hq, hkv, dh, 500000.0, p)
        assert np.array_equal(a[:50], b[:50])
        assert not np.array_equal(a[50:70], b[50:70])


def test_attention_argument_checks():
    B, R = _mods()
    qkv = R.dev(synth.normal(7, 680, (8, 3 * 64)))
    out = torch.empty((8, 64), dtype=torch.float32, device="cuda")
    ws = R.Workspace(B.brl_attention_workspace_bytes(1, 8, 1, 1, 64))
    with pytest.raises(B.BitrlError) as e:
        B.attention_forward(qkv, 1, 8, None, None, 1, 1, 48, 10000.0, B.BRL_ATTN_MFMA, out, ws.buf)
    assert e.value.status == B.BRL_EINVAL
    with pytest.raises(B.BitrlError) as e:
        B.attention_forward(qkv, 1, 8, None, None, 3, 2, 64, 10000.0, B.BRL_ATTN_MFMA, out, ws.buf)
    assert e.value.status == B.BRL_EINVAL
    cu = np.asarray([0, 9], dtype=np.int32)                   # longer than the bound S = 8
    with pytest.raises(B.BitrlError) as e:
        B.attention_forward(qkv, 1, 8, R.dev(cu), cu, 1, 1, 64, 10000.0, B.BRL_ATTN_MFMA, out, ws.buf)
    assert e.value.status == B.BRL_EINVAL
    small = R.Workspace(64)
    with pytest.raises(B.BitrlError) as e:
        B.attention_forward(qkv, 1, 8, None, None, 1, 1, 64, 10000.0, B.BRL_ATTN_MFMA, out, small.buf)
    assert e.value.status == B.BRL_ENOSPC


@pytest.mark.parametrize("hq,hkv,dh,S", [(8, 2, 128, 27), (8, 1, 100, 32), (8, 2, 64, 1), (8, 2, 16, 9)])
def test_short_state_kernels_meet_at_the_dispatch_line(hq, hkv, dh, S):
    """1024 and 1025 states of 8 heads: the states they share get the same bits, and the last one matches the oracle."""
    B, R = _mods()
    qkv = synth.normal(37, 5, (1025 * S, (hq + 2 * hkv) * dh))
    one = _run(B, R, qkv[:1024 * S], [S] * 1024, S, hq, hkv, dh, 10000.0, B.BRL_ATTN_MFMA)
    two = _run(B, R, qkv, [S] * 1025, S, hq, hkv, dh, 10000.0, B.BRL_ATTN_MFMA)
    assert np.array_equal(one, two[:1024 * S])
    ref = _oracle(qkv[1024 * S:], [S], hq, hkv, dh, 10000.0)[0]
    got = two[1024 * S:].reshape(ref.shape)
    assert np.abs(got - ref).max() <= ATTN_REL * np.abs(ref).max()


@pytest.mark.parametrize("hq,hkv,dh,batches", [
    (20, 5, 100, (1, 38, 39, 51, 52, 409, 410)),       # query head; query head | group | query head | pair
    (32, 4, 100, (24, 25, 32, 33, 127, 128)),          # two groups of four per key/value head
    (30, 6, 100, (1, 60, 300)),                        # groups of five: query head only
    (20, 5, 128, (1, 25, 26, 38, 39, 51, 52, 409, 410)),   # query head | rows
    (30, 6, 128, (1, 17, 18, 60, 300)),                # query head | rows, the second workgroup of a group with one head
    (30, 6, 128, (21, 22, 25, 26, 42, 43, 51, 52)),    # groups of five: rows | query head | rows | query head | rows
    (16, 8, 128, (48, 49, 64, 65, 80, 81)),            # groups of two: query head | rows | query head | rows
    (16, 16, 64, (1, 16, 17)),                         # group | query head
    (32, 4, 64, (1, 256, 257)),                        # group | pair
    (28, 4, 64, (1, 256, 257)),                        # the last wavefront of a group idle
    (16, 8, 64, (1, 128, 129)),                        # group | query head
    (30, 6, 64, (1, 85, 86, 273, 274)),                # groups of five: group | query head | pair
    (16, 4, 32, (1, 64, 65, 200)),                     # query head | group
    (24, 8, 16, (1, 42, 43)),
    (16, 8, 32, (1, 130)),                             # groups of two: query head only
])
def test_short_state_forms_give_the_same_bits(hq, hkv, dh, batches):
    """Batches on both sides of every line between the four forms of states of at most 32 tokens (a workgroup per query head,
    per group of four, the same from the fp32 rows, the pair of kernels), uniform and ragged: the states that they share get
    the same bits, first and last match the oracle."""
    B, R = _mods()
    n = batches[-1]
    for S, lens in ((19, [19] * n), (None, [1 + (11 * i + 30) % 32 for i in range(n)])):
        qkv = synth.normal(41, 5, (sum(lens), (hq + 2 * hkv) * dh))
        want = None
        for b in reversed(batches):
            rows = sum(lens[:b])
            print("short states", hq, hkv, dh, "uniform" if S else "ragged", b, flush=True)
            got = _run(B, R, qkv[:rows], lens[:b], S, hq, hkv, dh, 10000.0, B.BRL_ATTN_MFMA, max_len=None if S else 32)
            if want is None:
                want = got
                for i in (0, n - 1):
                    r0 = sum(lens[:i])
                    ref = _oracle(qkv[r0:r0 + lens[i]], lens[i:i + 1], hq, hkv, dh, 10000.0)[0]
                    assert np.abs(got[r0:r0 + lens[i]].reshape(ref.shape) - ref).max() <= ATTN_REL * np.abs(ref).max()
            assert np.array_equal(got, want[:rows]), b


@pytest.mark.parametrize("hq,hkv,longest,batches", [
    (20, 5, 64, (1, 70)), (12, 4, 64, (9,)), (16, 16, 64, (7, 70)),       # full groups, three of four, one head
    (7, 1, 64, (66,)), (30, 6, 64, (42, 43)),                             # last wavefront idle; groups of five: rows | pair
    (8, 2, 33, (5,)), (8, 2, 63, (64,)),
    (20, 5, 32, (25, 26)), (16, 8, 32, (32, 33)), (5, 1, 32, (102, 103)),  # one key block: query head | rows
    (16, 8, 32, (48, 49)),                                                # likewise, past one and a half workgroups per compute unit
    (16, 16, 32, (32, 33)),                                               # groups of one: query head
])
def test_states_of_two_key_blocks_give_the_bits_of_the_pair(hq, hkv, longest, batches):
    """Heads of 128, every state length up to two key blocks: a larger bound on the lengths (three key blocks, which run
    the pack and fragment kernels) changes no bit, a larger batch none of the states it shares, and single states match
    the oracle."""
    B, R = _mods()
    n, dh = batches[-1], 128
    for lens in ([1 + (27 * i + longest - 1) % longest for i in range(n)], [longest - 1] * n, [longest] * n):
        uniform = lens[0] if len(set(lens)) == 1 else None
        qkv = synth.normal(43, 5, (sum(lens), (hq + 2 * hkv) * dh))
        print("two key blocks", hq, hkv, n, "uniform" if uniform else "ragged", longest, flush=True)
        want = _run(B, R, qkv, lens, None, hq, hkv, dh, 10000.0, B.BRL_ATTN_MFMA, max_len=96)
        assert np.all(np.isfinite(want))
        for b in batches:
            rows = sum(lens[:b])
            got = _run(B, R, qkv[:rows], lens[:b], uniform, hq, hkv, dh, 10000.0, B.BRL_ATTN_MFMA, max_len=None if uniform else longest)
            assert np.array_equal(got, want[:rows]), b
        for i in (0, n - 1):
            r0 = sum(lens[:i])
            ref = _oracle(qkv[r0:r0 + lens[i]], lens[i:i + 1], hq, hkv, dh, 10000.0)[0]
            assert np.abs(want[r0:r0 + lens[i]].reshape(ref.shape) - ref).max() <= ATTN_REL * np.abs(ref).max()


@pytest.mark.parametrize("S,batches", [
    (384, (1, 24, 23)),                    # twelve chunks per head: their order turns from twelve heads per XCD on
    (1024, (1, 32, 31)),                   # thirty-two: from sixteen on
    (224, (2, 1)), (256, (2, 1)),          # seven never, eight always
])
def test_order_of_query_chunks_changes_no_bit(S, batches):
    """The order in which a head's chunks of queries are dispatched turns from head to head or not: states that two batches
    share get the same bits, and the last one matches the oracle."""
    B, R = _mods()
    hq, hkv, dh = 16, 4, 32
    n = max(batches)
    qkv = synth.normal(47, 5, (n * S, (hq + 2 * hkv) * dh))
    print("query chunks", S, batches, flush=True)
    want = _run(B, R, qkv, [S] * n, S, hq, hkv, dh, 10000.0, B.BRL_ATTN_MFMA)
    for b in batches:
        if b != n:
            assert np.array_equal(_run(B, R, qkv[:b * S], [S] * b, S, hq, hkv, dh, 10000.0, B.BRL_ATTN_MFMA), want[:b * S]), b
    ref = _oracle(qkv[(n - 1) * S:], [S], hq, hkv, dh, 10000.0)[0]
    assert np.abs(want[(n - 1) * S:].reshape(ref.shape) - ref).max() <= ATTN_REL * np.abs(ref).max()


def test_order_of_packing_changes_no_bit():
    """Heads of 128 whose fragments take just under and over 100 MB (133 and 134 states of three key blocks): the pack kernel's
    work goes by XCD or in plain order, the states they share get the same bits, and the last one matches the oracle."""
    B, R = _mods()
    hq, hkv, dh, S, n = 8, 8, 128, 96, 134
    qkv = synth.normal(53, 5, (n * S, (hq + 2 * hkv) * dh))
    two = _run(B, R, qkv, [S] * n, S, hq, hkv, dh, 10000.0, B.BRL_ATTN_MFMA)
    one = _run(B, R, qkv[:(n - 1) * S], [S] * (n - 1), S, hq, hkv, dh, 10000.0, B.BRL_ATTN_MFMA)
    assert np.array_equal(one, two[:(n - 1) * S])
    ref = _oracle(qkv[(n - 1) * S:], [S], hq, hkv, dh, 10000.0)[0]
    assert np.abs(two[(n - 1) * S:].reshape(ref.shape) - ref).max() <= ATTN_REL * np.abs(ref).max()
