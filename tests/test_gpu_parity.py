"""GPU parity: the HIP library, called through its C ABI, against the CPU oracle.

Integer stages (ternary codes, int8 activations, int32 accumulators) must be
bit-exact.  fp32 outputs of one BitLinear / RMSNorm / FFN stage must agree to
max relative error 1e-5; encoder outputs to cosine >= 0.999 per state.
Inputs are the seeded synthetic tensors of paper_2604_24273_amd.synth.
"""
import numpy as np
import pytest

from oracle import bitrl_oracle as O
from paper_2604_24273_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

REL = 1e-5


def _mods():
    from paper_2604_24273_amd import binding as B
    from paper_2604_24273_amd import runtime as R
    B.lib()       # fails loudly if the library has not been built
    return B, R


def assert_fp_close(got: np.ndarray, ref: np.ndarray, rel: float = REL):
    got = np.asarray(got, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    assert got.shape == ref.shape
    scale = np.abs(ref).max()
    if scale == 0:
        assert np.all(got == 0)
        return
    d = np.abs(got - ref)
    assert d.max() / scale <= rel, "max rel err %.3e" % (d.max() / scale)
    assert np.all(d <= rel * np.abs(ref) + 0.1 * rel * scale)


def cosine(a, b):
    a = np.asarray(a, np.float64).ravel(); b = np.asarray(b, np.float64).ravel()
    return float(a @ b / (np.linalg.norm(a) * np.linalg.norm(b)))


# ------------------------------------------------------------------ weights

@pytest.mark.parametrize("n,k", [(2048, 2048), (6912, 2560), (2560, 6912), (70, 200), (33, 8), (1, 128), (640, 2560)])
def test_quantize_weights_bit_exact(n, k):
    B, R = _mods()
    print("quantize_weights", n, k, flush=True)
    W = synth.normal(0, 1, (n, k), 0.02)
    codes_ref, beta_ref = O.ternary_quantize(W)
    pl = R.quantize_linear(W, want_codes=True)
    assert pl.packed.numel() == B.brl_packed_bytes(n, k)
    beta = pl.beta.cpu().numpy()[0]
    assert beta.view(np.uint32) == np.float32(beta_ref).view(np.uint32), (beta, beta_ref)
    assert np.array_equal(pl.codes.cpu().numpy(), codes_ref)
    out = torch.empty((n, k), dtype=torch.int8, device="cuda")
    B.brl_unpack_codes(pl.packed, n, k, out)
    assert np.array_equal(out.cpu().numpy(), codes_ref)
    # deterministic: a second run gives the same blob
    pl2 = R.quantize_linear(W)
    assert torch.equal(pl.packed, pl2.packed) and torch.equal(pl.beta, pl2.beta)


@pytest.mark.parametrize("n,k", [(1, 1), (31, 127), (33, 129), (32, 512), (40, 515), (65, 1030)])
def test_quantize_weights_block_edges(n, k):
    """Packing takes 32 rows x 512 columns per workgroup, four columns per load: sizes one below, at and above each,
    and rows that start at odd addresses.  Codes, scale and the packed blob's round trip are exact."""
    B, R = _mods()
    W = synth.normal(71, 3, (n, k), 0.02)
    codes_ref, beta_ref = O.ternary_quantize(W)
    pl = R.quantize_linear(W, want_codes=True)
    assert np.array_equal(pl.codes.cpu().numpy(), codes_ref) and np.float32(pl.beta.cpu().numpy()[0]) == beta_ref
    back = torch.full((n, k), 9, dtype=torch.int8, device="cuda")
    B.brl_unpack_codes(pl.packed, n, k, back)
    assert np.array_equal(back.cpu().numpy(), codes_ref)
    from oracle import critic_oracle as C
    c8_ref, s8_ref = C.int8_quantize(W)
    p8 = R.quantize_linear(W, want_codes=True, int8=True)
    assert np.array_equal(p8.codes.cpu().numpy(), c8_ref) and np.float32(p8.beta.cpu().numpy()[0]) == s8_ref
    B.brl_unpack_codes_int8(p8.packed, n, k, back)
    assert np.array_equal(back.cpu().numpy(), c8_ref)


@pytest.mark.parametrize("n,k", [(129, 16), (97, 640), (70, 700), (2097153, 8)])
def test_quantize_weights_super_blocks_through_the_blob(n, k):
    """A workgroup packs four consecutive super-blocks wherever they lie: several row blocks of a narrow matrix, row blocks
    that end inside a workgroup, and more row blocks than a second grid dimension has room for."""
    B, R = _mods()
    from oracle import critic_oracle as C
    print("quantize_weights", n, k, flush=True)
    W = synth.normal(73, 3, (n, k), 0.02)
    back = torch.empty((n, k), dtype=torch.int8, device="cuda")
    for int8, ref, unpack in ((False, O.ternary_quantize, B.brl_unpack_codes), (True, C.int8_quantize, B.brl_unpack_codes_int8)):
        codes_ref, scale_ref = ref(W)
        pl = R.quantize_linear(W, want_codes=True, int8=int8)
        assert np.float32(pl.beta.cpu().numpy()[0]) == scale_ref
        assert np.array_equal(pl.codes.cpu().numpy(), codes_ref)
        unpack(pl.packed, n, k, back.fill_(9))
        assert np.array_equal(back.cpu().numpy(), codes_ref)


def test_quantize_weights_special_matrices():
    B, R = _mods()
    for W in (np.zeros((40, 136), np.float32),                       # all zero: beta = eps, codes 0
              np.array([[3, -3, 1, -1, 3, -3, 1, -1]] * 2, np.float32),   # |w| == tau ties when eps = 0
              synth.normal(9, 1, (64, 256), 0.02) * np.float32(1e-4)):  # tiny scale: eps matters
        for eps in (1e-5, 0.0):
            c_ref, b_ref = O.ternary_quantize(W, eps)
            pl = R.quantize_linear(W, eps=eps, want_codes=True)
            assert np.float32(pl.beta.cpu().numpy()[0]).view(np.uint32) == np.float32(b_ref).view(np.uint32)
            assert np.array_equal(pl.codes.cpu().numpy(), c_ref)
    bad = np.ones((8, 16), np.float32); bad[1, 2] = np.inf
    with pytest.raises(B.BitrlError) as ei:
        R.quantize_linear(bad)
    assert ei.value.status == B.BRL_EINVAL


def test_quantising_thread_ends_without_waiting_for_the_device():
    """A loader thread that has quantised ends while a stream is still at work (about half a second of a kernel that spins)."""
    import os
    import threading
    import time
    B, R = _mods()
    W = R.dev(synth.normal(75, 1, (64, 256), 0.02))
    packed, beta, ws = R.device_bytes(B.brl_packed_bytes(64, 256)), torch.empty(1, device="cuda"), R.device_bytes(1 << 16)
    begin, end, done = (torch.cuda.Event(enable_timing=True) for _ in range(3))
    begin.record()
    torch.cuda._sleep(1000000)
    end.record()
    torch.cuda.synchronize()
    half_a_second = int(1000000 * 500.0 / max(begin.elapsed_time(end), 0.05))
    quantised, may_end = threading.Event(), threading.Event()

    def load():
        B.bitlinear_quantize_weights(W, 1e-5, packed, beta, None, ws)
        quantised.set()
        may_end.wait(60)

    t = threading.Thread(target=load)
    t.start()
    assert quantised.wait(60)
    task = "/proc/self/task/%d" % t.native_id
    torch.cuda._sleep(half_a_second)
    done.record()
    may_end.set()
    t.join(60)
    limit = time.monotonic() + 5
    while os.path.exists(task) and time.monotonic() < limit:     # join() returns before the thread's own clean-up
        time.sleep(0.001)
    ended_first = not done.query()
    torch.cuda.synchronize()
    assert not os.path.exists(task) and ended_first


def test_concurrent_quantising_threads_get_their_own_verdict():
    """More threads at once than the library has pinned words; every third has a bad weight, and only it hears of it."""
    import threading
    B, R = _mods()
    n, k, threads = 96, 640, 90
    W = [synth.normal(77, i, (n, k), 0.02) for i in range(threads)]
    for i in range(0, threads, 3):
        W[i][5, i] = np.nan if i % 2 else np.inf
    dev = [R.dev(w) for w in W]
    packed = [R.device_bytes(B.brl_packed_int8_bytes(n, k)) for _ in range(threads)]
    beta, ws = torch.empty((threads, 1), device="cuda"), [R.device_bytes(1 << 16) for _ in range(threads)]
    streams = [torch.cuda.Stream() for _ in range(4)]
    got, gate = [None] * threads, threading.Barrier(threads)
    torch.cuda.synchronize()

    def quantise(i):
        with torch.cuda.stream(streams[i % 4]):
            gate.wait(60)
            verdicts = []
            for r in range(5):
                try:
                    if i % 2:
                        B.bitlinear_quantize_weights(dev[i], 1e-5, packed[i], beta[i], None, ws[i])
                    else:
                        B.bitlinear_quantize_weights_int8(dev[i], 1e-5, 127, packed[i], beta[i], None, ws[i])
                    verdicts.append("good")
                except B.BitrlError as e:
                    verdicts.append("bad" if e.status == B.BRL_EINVAL else str(e))
            got[i] = verdicts

    ts = [threading.Thread(target=quantise, args=(i,)) for i in range(threads)]
    for t in ts:
        t.start()
    for t in ts:
        t.join(60)
    torch.cuda.synchronize()
    assert got == [["good" if i % 3 else "bad"] * 5 for i in range(threads)]


# ---------------------------------------------------------------- BitLinear

def _run_bitlinear(B, R, pl, X, residual=None, taps=True):
    m, k = X.shape
    n = pl.n_out
    y = torch.empty((m, n), dtype=torch.float32, device="cuda")
    xq = torch.zeros((m, k), dtype=torch.int8, device="cuda") if taps else None
    am = torch.zeros((m,), dtype=torch.float32, device="cuda") if taps else None
    acc = torch.zeros((m, n), dtype=torch.int32, device="cuda") if taps else None
    ws = R.Workspace(B.brl_bitlinear_workspace_bytes(m, n, k))
    B.bitlinear_forward(pl.packed, pl.beta, n, k, X, m, 1e-5, y, residual, xq, am, acc, ws.buf)
    torch.cuda.synchronize()
    return y, xq, am, acc, ws


@pytest.mark.parametrize("m,n,k", [
    (16, 2048, 2048),     # single-layer config
    (1, 6912, 2560), (1, 2560, 6912), (2, 2560, 6912), (3, 200, 264), (4, 6912, 2560),   # GEMV path
    (5, 96, 128), (33, 200, 264), (64, 2560, 2560), (100, 640, 2560), (300, 1000, 520),
    (256, 6912, 2560), (257, 2560, 6912), (1100, 3200, 3200),
    (600, 2560, 6912), (1300, 1000, 4608),                       # direct 32 x 64 tiles on eight wavefronts, long k (ragged N in the second)
    (200, 1000, 4608), (700, 264, 6912),                         # direct 32 x 32 tiles, k over sixteen wavefronts
    (2050, 8192, 264), (2048, 8200, 128),      # enough tiles for the 8-wavefront kernel, ragged edges
    (1024, 640, 2560), (1025, 640, 2560),      # last size of the one-workgroup-per-token quantiser, first of the one-wavefront-per-token one
    (1100, 64, 8640), (1030, 40, 8200),        # widest rows of the one-wavefront-per-token quantiser (34 chunks), ragged k
    (2100, 64, 6912), (6200, 32, 2560),        # 16-token groups (past 2048 tokens at 6912 wide, past 6144 at 2560 wide)
    (1100, 40, 9216),                          # the widest rows supported: four wavefronts per token
])
def test_bitlinear_forward_parity(m, n, k):
    B, R = _mods()
    print("bitlinear_forward", m, n, k, flush=True)
    case = synth.bitlinear_case(0, n, k, m)
    if m >= 3:
        case["X"][1] = 0.0                      # an all-zero token must give an all-zero row
        case["X"][2] *= np.float32(1e-7)        # a tiny token exercises the absmax floor
    codes, beta = O.ternary_quantize(case["W"])
    taps = {}
    y_ref = O.bitlinear_forward(case["X"], codes, beta, taps=taps)
    pl = R.quantize_linear(case["W"])
    y, xq, am, acc, _ = _run_bitlinear(B, R, pl, R.dev(case["X"]))
    assert np.array_equal(xq.cpu().numpy(), taps["xq"])
    assert np.array_equal(am.cpu().numpy().view(np.uint32), taps["absmax"].view(np.uint32))
    assert np.array_equal(acc.cpu().numpy(), taps["acc"])
    assert_fp_close(y.cpu().numpy(), y_ref)
    assert np.array_equal(y.cpu().numpy(), y_ref)          # same fp32 op order: identical in practice
    if m >= 3:
        assert np.all(y.cpu().numpy()[1] == 0)


@pytest.mark.parametrize("m,n,k", [
    (64, 4096, 136), (64, 4128, 136),           # 256 tiles of 32 x 32, one block more (32 x 64 tiles)
    (512, 1000, 136), (512, 1030, 136),         # ragged n: 512 tiles of 32 x 32, one block more
    (480, 4096, 264), (990, 1984, 264),         # 960 tiles of 32 x 64 on eight wavefronts, 961 on four
    (990, 1984, 4096), (990, 1990, 4088),       # ... with a longer k; ragged n and k
    (990, 1984, 5120), (990, 1990, 5112), (990, 1984, 4992),   # ... and on eight again from 40 super-blocks of k on
    (1600, 3200, 136), (1312, 3904, 136),       # 2500 tiles of 32 x 64; 2501: 128 x 128 on eight wavefronts
    (1920, 3840, 136), (1408, 5248, 136),       # 450 tiles of 128 x 128, 451
    (70, 40, 8), (200, 70, 1032),               # fewer super-blocks of k than wavefronts, a remainder of one
])
def test_bitlinear_dispatch_edges(m, n, k):
    """Both sides of every limit of the many-token dispatch, through both epilogue forms (taps / residual)."""
    B, R = _mods()
    print("dispatch edges", m, n, k, flush=True)
    case = synth.bitlinear_case(5, n, k, m)
    codes, beta = O.ternary_quantize(case["W"])
    taps = {}
    y_ref = O.bitlinear_forward(case["X"], codes, beta, taps=taps)
    pl = R.quantize_linear(case["W"])
    x = R.dev(case["X"])
    y, _, _, acc, ws = _run_bitlinear(B, R, pl, x)
    assert np.array_equal(acc.cpu().numpy(), taps["acc"])
    assert np.array_equal(y.cpu().numpy(), y_ref)
    res = synth.normal(5, 7, (m, n))
    y2 = torch.empty((m, n), dtype=torch.float32, device="cuda")
    B.bitlinear_forward(pl.packed, pl.beta, n, k, x, m, 1e-5, y2, R.dev(res), None, None, None, ws.buf)
    assert np.array_equal(y2.cpu().numpy(), O.bitlinear_forward(case["X"], codes, beta, residual=res))


@pytest.mark.parametrize("m,n,k,bf16", [
    (2, 64, 256, False), (3, 64, 256, False), (4, 33, 8, True), (15, 100, 1024, False),   # first token counts, ragged n, shortest k
    (16, 8192, 1032, True), (16, 8193, 1032, False),          # 256 workgroups; one more (two launches)
    (16, 70, 5120, False), (16, 70, 5128, False), (9, 40, 4104, True),                    # longest k at 16 tokens, past it
    (17, 96, 2560, False), (17, 96, 2568, True),              # (two launches)
    (32, 31, 2048, True), (17, 40, 2048, False), (32, 40, 2056, False),                   # longest k at 32 tokens, past it
    (31, 64, 1024, False), (32, 64, 520, False), (33, 64, 520, False),                    # most tokens, past them
])
def test_bitlinear_few_tokens_in_one_launch(m, n, k, bf16):
    """Both sides of every limit of the one-launch product for a few tokens, with taps, with a residual in place, through
    the entry point without a workspace, and with a result that overwrites the input."""
    B, R = _mods()
    print("few tokens", m, n, k, bf16, flush=True)
    case = synth.bitlinear_case(11, n, k, m)
    x = R.dev(case["X"])
    if bf16:
        x = x.to(torch.bfloat16)
    X = x.float().cpu().numpy()
    codes, beta = O.ternary_quantize(case["W"])
    taps = {}
    y_ref = O.bitlinear_forward(X, codes, beta, taps=taps)
    pl = R.quantize_linear(case["W"])
    y, xq, am, acc, ws = _run_bitlinear(B, R, pl, x)
    assert np.array_equal(xq.cpu().numpy(), taps["xq"])
    assert np.array_equal(am.cpu().numpy().view(np.uint32), taps["absmax"].view(np.uint32))
    assert np.array_equal(acc.cpu().numpy(), taps["acc"])
    assert np.array_equal(y.cpu().numpy(), y_ref)
    y2 = torch.empty_like(y)
    B.bitlinear_forward_static(pl.packed, pl.beta, n, k, x, m, 1e-5, y2, None, None, None, None)
    assert torch.equal(y2, y)
    res = synth.normal(11, 7, (m, n))
    y2.copy_(R.dev(res))
    B.bitlinear_forward(pl.packed, pl.beta, n, k, x, m, 1e-5, y2, y2, None, None, None, ws.buf)
    assert np.array_equal(y2.cpu().numpy(), O.bitlinear_forward(X, codes, beta, residual=res))
    if m > 4 and not bf16:                       # the result in the input's place (past the one-token path it always could be)
        both = torch.empty(m * max(n, k), dtype=torch.float32, device="cuda")
        both[:m * k].copy_(x.reshape(-1))
        out = both[:m * n].view(m, n)
        B.bitlinear_forward(pl.packed, pl.beta, n, k, both[:m * k].view(m, k), m, 1e-5, out, None, None, None, None, ws.buf)
        assert np.array_equal(out.cpu().numpy(), y_ref)


@pytest.mark.parametrize("m,n,k", [
    (1, 64, 256), (2, 70, 2560), (4, 64, 9216),       # one-launch kernels of a few tokens
    (16, 64, 264), (32, 40, 2560),
    (40, 64, 264), (1024, 32, 2560),                  # a workgroup per token
    (1100, 64, 264), (1100, 32, 6912),                # a wavefront per token
    (1100, 32, 9216),                                 # four of them
])
@pytest.mark.parametrize("bf16", [False, True])
def test_activation_codes_where_the_scale_overflows(m, n, k, bf16):
    """Rows whose largest value is below 127 / FLT_MAX under a floor that small: 127 / a is infinite and every code is +-127
    by its sign.  Rows just above have a finite scale, and other rows of the batch their usual codes.  (No zeros: the header
    leaves 0 x inf to NaN's code.)"""
    B, R = _mods()
    print("scale overflows", m, n, k, bf16, flush=True)
    case = synth.bitlinear_case(13, n, k, m)
    X = case["X"]
    X = np.where(X < 0, -1, 1).astype(np.float32) * np.maximum(np.abs(X), np.float32(0.5))      # (scaled below, still normal numbers)
    for t, a in {0: 2e-37, 1: 3.75e-37, m - 1: 1.5e-37}.items():
        if t < m:
            X[t] *= np.float32(a / np.abs(X[t]).max())
    if bf16:
        X = synth.bf16_bits_to_f32(synth.to_bf16_bits(X))
        x = R.bf16_from_bits(synth.to_bf16_bits(X))
    else:
        x = R.dev(X)
    eps = 1e-38
    codes, beta = O.ternary_quantize(case["W"])
    taps = {}
    with np.errstate(over="ignore", divide="ignore", under="ignore"):
        O.bitlinear_forward(X, codes, beta, eps=eps, taps=taps)
    assert np.array_equal(taps["xq"][m - 1], np.where(X[m - 1] > 0, 127, -127))
    pl = R.quantize_linear(case["W"])
    y = torch.empty((m, n), dtype=torch.float32, device="cuda")
    xq = torch.zeros((m, k), dtype=torch.int8, device="cuda")
    am = torch.zeros((m,), dtype=torch.float32, device="cuda")
    acc = torch.zeros((m, n), dtype=torch.int32, device="cuda")
    ws = R.Workspace(B.brl_bitlinear_workspace_bytes(m, n, k))
    B.bitlinear_forward(pl.packed, pl.beta, n, k, x, m, eps, y, None, xq, am, acc, ws.buf)
    assert np.array_equal(xq.cpu().numpy(), taps["xq"])
    assert np.array_equal(am.cpu().numpy().view(np.uint32), taps["absmax"].view(np.uint32))
    assert np.array_equal(acc.cpu().numpy(), taps["acc"])
    if m <= 4:                                        # the queued form has no taps: its results are the single call's
        def ptr(t):
            return torch.tensor([t.data_ptr()], dtype=torch.int64, device="cuda")
        y2 = torch.empty_like(y)
        B.bitlinear_forward_batch(ptr(pl.packed), ptr(pl.beta), n, k, ptr(x), B.BRL_BF16 if bf16 else B.BRL_F32, m, eps, ptr(y2), 1)
        assert torch.equal(y2, y)


@pytest.mark.parametrize("m,d,f", [
    (512, 136, 1024), (544, 136, 1000),         # 512 and 544 tiles of 32 tokens x 32 column pairs, the second ragged
    (1536, 136, 2048), (1664, 136, 2048),       # 192 and 208 wide tiles: 75 and 81 % of 256 compute units
    (20, 520, 40), (4000, 136, 1600), (3200, 136, 1920),   # smallest; past the direct kernel's last size (6250 and 6000 tiles)
])
def test_ffn_dispatch_edges(m, d, f):
    """Both sides of the limits of the gate | up dispatch."""
    B, R = _mods()
    print("ffn dispatch edges", m, d, f, flush=True)
    c = synth.ffn_case(0, m, d, f)
    x32 = synth.normal(0, 26, (m, d))
    T = O.TernaryLinear.from_fp32
    y_ref = O.ffn_block_forward(x32, O.FFNWeights(c["norm_g"], T(c["W_gate"]), T(c["W_up"]), c["subln_g"], T(c["W_down"])))
    hnd = R.FFNHandle(c["norm_g"], c["W_gate"], c["W_up"], c["subln_g"], c["W_down"])
    y = torch.empty((m, d), dtype=torch.float32, device="cuda")
    ws = R.Workspace(B.brl_ffn_workspace_bytes(m, d, f))
    B.ffn_block_forward(hnd.struct, R.dev(x32), m, d, f, 1e-5, 1e-5, y, ws.buf)
    assert_fp_close(y.cpu().numpy(), y_ref)


def test_bitlinear_forward_shape_sweep():
    """Seeded random shapes across the dispatch boundaries (1-4 token path, direct tiles with k over 16, 8 and 4
    wavefronts, narrow and wide LDS tiles): integer stages exact, outputs identical, with and without the taps
    (the two epilogue families) and with a residual."""
    B, R = _mods()
    rng = np.random.default_rng(20241)
    shapes = []
    for _ in range(28):
        m = int(rng.choice([rng.integers(1, 9), rng.integers(9, 200), rng.integers(200, 1400)]))
        n = int(rng.choice([rng.integers(1, 97), 32 * rng.integers(1, 130), rng.integers(97, 3000)]))
        k = 8 * int(rng.choice([rng.integers(1, 48), rng.integers(48, 400), rng.integers(400, 1153)]))
        shapes.append((m, n, k))
    for idx, (m, n, k) in enumerate(shapes):
        print("bitlinear_forward sweep", m, n, k, flush=True)
        case = synth.bitlinear_case(1000 + idx, n, k, m)
        codes, beta = O.ternary_quantize(case["W"])
        taps = {}
        y_ref = O.bitlinear_forward(case["X"], codes, beta, taps=taps)
        pl = R.quantize_linear(case["W"])
        x = R.dev(case["X"])
        y, xq, am, acc, ws = _run_bitlinear(B, R, pl, x)
        assert np.array_equal(xq.cpu().numpy(), taps["xq"]), (m, n, k)
        assert np.array_equal(acc.cpu().numpy(), taps["acc"]), (m, n, k)
        assert np.array_equal(y.cpu().numpy(), y_ref), (m, n, k)
        res = synth.normal(1000 + idx, 7, (m, n))
        y2 = R.dev(res)
        B.bitlinear_forward(pl.packed, pl.beta, n, k, x, m, 1e-5, y2, y2, None, None, None, ws.buf)
        assert np.array_equal(y2.cpu().numpy(), O.bitlinear_forward(case["X"], codes, beta, residual=res)), (m, n, k)


@pytest.mark.parametrize("m", [1, 4, 48])
def test_bitlinear_residual_bf16_and_no_taps(m):
    B, R = _mods()
    n, k = 320, 384
    case = synth.bitlinear_case(3, n, k, m)
    xb = synth.to_bf16_bits(case["X"])
    x32 = synth.bf16_bits_to_f32(xb)
    res = synth.normal(3, 7, (m, n))
    codes, beta = O.ternary_quantize(case["W"])
    y_ref = O.bitlinear_forward(x32, codes, beta, residual=res)
    pl = R.quantize_linear(case["W"])
    y, *_ = _run_bitlinear(B, R, pl, R.bf16_from_bits(xb), residual=R.dev(res), taps=False)
    assert np.array_equal(y.cpu().numpy(), y_ref)


def test_gemv_pair_decode_shape_repeated():
    """x[1, d] -> up -> (re-quantised) -> down, many calls on one workspace: identical every time."""
    B, R = _mods()
    c = synth.gemv_pair_case(0)
    up_c, up_b = O.ternary_quantize(c["W_up"]); dn_c, dn_b = O.ternary_quantize(c["W_down"])
    h_ref = O.bitlinear_forward(c["x"], up_c, up_b)
    y_ref = O.bitlinear_forward(h_ref, dn_c, dn_b)
    up, dn = R.quantize_linear(c["W_up"]), R.quantize_linear(c["W_down"])
    x = R.dev(c["x"])
    d, f = 2560, 6912
    h = torch.empty((1, f), dtype=torch.float32, device="cuda")
    y = torch.empty((1, d), dtype=torch.float32, device="cuda")
    ws = R.Workspace(max(B.brl_bitlinear_workspace_bytes(1, f, d), B.brl_bitlinear_workspace_bytes(1, d, f)))
    outs = []
    for it in range(50):
        B.bitlinear_forward(up.packed, up.beta, f, d, x, 1, 1e-5, h, None, None, None, None, ws.buf)
        B.bitlinear_forward(dn.packed, dn.beta, d, f, h, 1, 1e-5, y, None, None, None, None, ws.buf)
        if it in (0, 1, 49):
            outs.append((h.cpu().numpy().copy(), y.cpu().numpy().copy()))
    for hh, yy in outs:
        assert np.array_equal(hh, h_ref)
        assert np.array_equal(yy, y_ref)


@pytest.mark.parametrize("m,n,k,count,bf16", [(1, 6912, 2560, 9, False), (1, 2560, 6912, 7, False), (3, 100, 200, 5, True),
                                              (2, 264, 8200, 3, False), (4, 96, 128, 700, False),
                                              # so many row blocks per workgroup that a wavefront stores its parked
                                              # results more than once per problem
                                              (4, 400000, 128, 1, False), (2, 300100, 256, 2, True)])
def test_bitlinear_forward_batch(m, n, k, count, bf16):
    """Many independent few-token problems in one launch: each equals the oracle and the one-problem entry point."""
    B, R = _mods()
    n_w = min(count, 4)                       # weights and inputs repeat across the batch, outputs do not
    cases = [synth.bitlinear_case(100 + i, n, k, m) for i in range(n_w)]
    pls = [R.quantize_linear(c["W"]) for c in cases]
    xs_host = [synth.bf16_bits_to_f32(synth.to_bf16_bits(c["X"])) if bf16 else c["X"] for c in cases]
    xs = [R.bf16_from_bits(synth.to_bf16_bits(c["X"])) if bf16 else R.dev(c["X"]) for c in cases]
    ys = [torch.full((m, n), float("nan"), dtype=torch.float32, device="cuda") for _ in range(count)]
    order = [(3 * i + 1) % n_w for i in range(count)]

    def ptrs(ts):
        return torch.tensor([t.data_ptr() for t in ts], dtype=torch.int64, device="cuda")

    B.bitlinear_forward_batch(ptrs([pls[j].packed for j in order]), ptrs([pls[j].beta for j in order]), n, k,
                              ptrs([xs[j] for j in order]), B.BRL_BF16 if bf16 else B.BRL_F32, m, 1e-5, ptrs(ys), count)
    torch.cuda.synchronize()
    refs = []
    for j in range(n_w):
        codes, beta = O.ternary_quantize(cases[j]["W"])
        refs.append(O.bitlinear_forward(xs_host[j], codes, beta))
    ws = R.Workspace(B.brl_bitlinear_workspace_bytes(m, n, k))
    single = []
    for j in range(n_w):
        y1 = torch.empty((m, n), dtype=torch.float32, device="cuda")
        B.bitlinear_forward(pls[j].packed, pls[j].beta, n, k, xs[j], m, 1e-5, y1, None, None, None, None, ws.buf)
        single.append(y1.cpu().numpy())
    for i in range(count):
        got = ys[i].cpu().numpy()
        assert np.array_equal(got, single[order[i]]), i
        assert_fp_close(got, refs[order[i]])
    # an empty batch is a no-op
    B.bitlinear_forward_batch(ptrs(ys[:1]), ptrs(ys[:1]), n, k, ptrs(ys[:1]), B.BRL_F32, m, 1e-5, ptrs(ys[:1]), 0)


# ---------------------------------------------------------------------- FFN

@pytest.mark.parametrize("m,d,f,bf16", [(256, 2560, 6912, True), (37, 256, 392, False), (3, 128, 264, True), (130, 3200, 8640, False),
                                        (160, 256, 4224, False), (160, 4224, 512, False),    # long k in the down and in the gate|up (GLU) product
                                        # norms inside the one-wavefront-per-token quantiser: 34, 27 and 10 chunks per row,
                                        # groups of 8 tokens and (2100 at 6912 wide, 6200 at 2560 wide) of 16
                                        (1100, 128, 8640, False), (1100, 96, 6912, False), (2100, 96, 6912, False),
                                        (1200, 2560, 640, True), (6200, 2560, 64, False),
                                        (1100, 64, 9000, False)])      # four wavefronts per token, ragged k
def test_ffn_block_parity(m, d, f, bf16):
    B, R = _mods()
    print("ffn_block_forward", m, d, f, flush=True)
    c = synth.ffn_case(0, m, d, f)
    x32 = synth.bf16_bits_to_f32(c["x_bf16"]) if bf16 else synth.normal(0, 26, (m, d))
    w = O.FFNWeights(c["norm_g"], O.TernaryLinear.from_fp32(c["W_gate"]), O.TernaryLinear.from_fp32(c["W_up"]),
                     c["subln_g"], O.TernaryLinear.from_fp32(c["W_down"]))
    y_ref = O.ffn_block_forward(x32, w)
    hnd = R.FFNHandle(c["norm_g"], c["W_gate"], c["W_up"], c["subln_g"], c["W_down"])
    x = R.bf16_from_bits(c["x_bf16"]) if bf16 else R.dev(x32)
    y = torch.empty((m, d), dtype=torch.float32, device="cuda")
    ws = R.Workspace(B.brl_ffn_workspace_bytes(m, d, f))
    B.ffn_block_forward(hnd.struct, x, m, d, f, 1e-5, 1e-5, y, ws.buf)
    got = y.cpu().numpy()
    assert_fp_close(got, y_ref)
    # run again on the same workspace: bit-identical
    y2 = torch.empty_like(y)
    B.ffn_block_forward(hnd.struct, x, m, d, f, 1e-5, 1e-5, y2, ws.buf)
    assert torch.equal(y, y2)


# ------------------------------------------------------------------ encoder

def _oracle_encoder(shape, seed, layers_host):
    cfg = O.EncoderConfig(shape.n_layers, shape.d, shape.n_heads, shape.n_kv_heads, shape.head_dim, shape.f,
                          shape.vocab, shape.rope_theta)
    T = O.TernaryLinear.from_fp32
    layers = []
    for w in layers_host:
        layers.append(O.LayerWeights(w["attn_norm_g"], T(w["Wq"]), T(w["Wk"]), T(w["Wv"]), w["attn_subln_g"], T(w["Wo"]),
                                     O.FFNWeights(w["ffn_norm_g"], T(w["W_gate"]), T(w["W_up"]), w["ffn_subln_g"], T(w["W_down"]))))
    return cfg, layers


@pytest.mark.parametrize("kw,b,s", [
    (dict(n_layers=2, d=256, n_heads=4, n_kv_heads=2, head_dim=64, f=384, vocab=512), 5, 40),
    (dict(n_layers=3, d=128, n_heads=8, n_kv_heads=2, head_dim=16, f=264, vocab=300), 3, 70),
    (dict(n_layers=2, d=200, n_heads=2, n_kv_heads=2, head_dim=100, f=392, vocab=64), 2, 33),
    (dict(n_layers=1, d=256, n_heads=2, n_kv_heads=1, head_dim=128, f=512, vocab=1000), 4, 130),
    (dict(n_layers=2, d=64, n_heads=2, n_kv_heads=1, head_dim=32, f=128, vocab=50), 1, 1),
    (dict(n_layers=1, d=128, n_heads=4, n_kv_heads=4, head_dim=32, f=264, vocab=300), 2, 300),   # long multi-head states
    # states of at most 32 tokens: the one-kernel attention path
    (dict(n_layers=2, d=256, n_heads=4, n_kv_heads=2, head_dim=64, f=384, vocab=512), 5, 27),
    (dict(n_layers=2, d=200, n_heads=2, n_kv_heads=2, head_dim=100, f=392, vocab=64), 3, 32),
    (dict(n_layers=1, d=256, n_heads=2, n_kv_heads=1, head_dim=128, f=512, vocab=1000), 4, 19),
    (dict(n_layers=2, d=128, n_heads=8, n_kv_heads=1, head_dim=16, f=264, vocab=300), 2, 9),     # eight heads per k/v head
    (dict(n_layers=1, d=256, n_heads=8, n_kv_heads=8, head_dim=32, f=264, vocab=300), 3, 31),
])
@pytest.mark.parametrize("attn", ["mfma", "f32"])
def test_encoder_small_shapes(kw, b, s, attn):
    B, R = _mods()
    print("encoder_forward", kw, b, s, attn, flush=True)
    shape = synth.tiny_shape(**kw)
    host = []
    enc = R.EncoderHandle(shape, seed=1, layer_sink=lambda l, w: host.append(w),
                          attn_precision=B.BRL_ATTN_MFMA if attn == "mfma" else B.BRL_ATTN_F32)
    cfg, layers = _oracle_encoder(shape, 1, host)
    ids = synth.token_ids(1, 500, (b, s), shape.vocab)
    lengths = synth.state_lengths(1, 501, b, 1, s)
    emb = synth.embedding_bf16(1, shape)
    gfin = synth.final_norm_gain(1, shape)
    for ln in (None, lengths):
        h_ref = O.encoder_forward(ids, emb, layers, gfin, cfg, lengths=ln)
        h = enc.forward(R.dev(ids), None if ln is None else R.dev(ln)).cpu().numpy()
        for i in range(b):
            assert cosine(h[i], h_ref[i]) >= 0.999, (i, cosine(h[i], h_ref[i]))
        # An extra guard, not the bar: fp32-grade attention against fp64 attention differs in the last bits,
        # and where that flips one int8 rounding decision downstream the element moves by about 1/127 of its
        # token's absmax share, so no element-wise bound follows from the arithmetic; 5e-3 of the largest
        # output holds with a margin of two on every seeded case here.
        print("   guard ratio %.3e" % (np.abs(h - h_ref).max() / np.abs(h_ref).max()), flush=True)
        assert np.abs(h - h_ref).max() / np.abs(h_ref).max() < 5e-3
    # batch invariance and determinism, bit for bit
    h_all = enc.forward(R.dev(ids))
    assert torch.equal(h_all, enc.forward(R.dev(ids)))
    if b > 1:
        h_one = enc.forward(R.dev(ids[1:2]))
        assert torch.equal(h_all[1:2], h_one)


@pytest.mark.parametrize("kw,lens", [
    (dict(n_layers=2, d=256, n_heads=4, n_kv_heads=2, head_dim=64, f=384, vocab=512), [15, 40, 1, 32, 33, 27, 64, 31]),
    (dict(n_layers=2, d=200, n_heads=2, n_kv_heads=2, head_dim=100, f=392, vocab=64), [7, 70, 36]),
    (dict(n_layers=1, d=256, n_heads=8, n_kv_heads=2, head_dim=32, f=512, vocab=1000), [5]),
    (dict(n_layers=1, d=128, n_heads=2, n_kv_heads=1, head_dim=128, f=264, vocab=300), [129, 2, 96, 18, 40]),
    (dict(n_layers=2, d=256, n_heads=4, n_kv_heads=1, head_dim=64, f=384, vocab=512), [15, 27, 1, 32, 8]),   # all short
    (dict(n_layers=1, d=256, n_heads=2, n_kv_heads=2, head_dim=128, f=264, vocab=300), [27]),
])
@pytest.mark.parametrize("attn", ["mfma", "f32"])
def test_encoder_packed_variable_length(kw, lens, attn):
    """States of different lengths stored back to back: every state equals the oracle run on that state
    alone, and (bit for bit) the padded entry point with `lengths`."""
    B, R = _mods()
    print("encoder_forward_packed", kw, lens, attn, flush=True)
    shape = synth.tiny_shape(**kw)
    host = []
    enc = R.EncoderHandle(shape, seed=2, layer_sink=lambda l, w: host.append(w),
                          attn_precision=B.BRL_ATTN_MFMA if attn == "mfma" else B.BRL_ATTN_F32)
    cfg, layers = _oracle_encoder(shape, 2, host)
    emb = synth.embedding_bf16(2, shape)
    gfin = synth.final_norm_gain(2, shape)
    nb, smax = len(lens), max(lens)
    padded = synth.token_ids(2, 500, (nb, smax), shape.vocab)
    flat = np.concatenate([padded[i, :n] for i, n in enumerate(lens)]).astype(np.int32)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    h = enc.forward_packed(R.dev(flat), cu)
    # a larger bound on the lengths changes nothing
    assert torch.equal(h, enc.forward_packed(R.dev(flat), cu, max_len=smax + 29))
    h_pad = enc.forward(R.dev(padded), R.dev(np.asarray(lens, dtype=np.int32)))
    assert torch.equal(h, h_pad)
    hn = h.cpu().numpy()
    for i, n in enumerate(lens):
        h_ref = O.encoder_forward(padded[i:i + 1, :n], emb, layers, gfin, cfg)[0]
        assert cosine(hn[i], h_ref) >= 0.999, (i, n, cosine(hn[i], h_ref))
        print("   guard ratio %.3e" % (np.abs(hn[i] - h_ref).max() / np.abs(h_ref).max()), flush=True)
        assert np.abs(hn[i] - h_ref).max() / np.abs(h_ref).max() < 5e-3


def test_head_parity_and_variants():
    B, R = _mods()
    for hidden, act in (((256,), B.BRL_ACT_TANH), ((256, 128), B.BRL_ACT_TANH), ((64,), B.BRL_ACT_RELU), ((), B.BRL_ACT_TANH)):
        shape = synth.tiny_shape(d=2560, head_hidden=hidden, n_actions=18)
        hh = R.HeadHandle(shape, seed=0, act=act)
        h = synth.normal(0, 400, (64, 2560))
        logits, value = hh.forward(R.dev(h))
        name = "tanh" if act == B.BRL_ACT_TANH else "relu"
        lr, vr = O.policy_value_head(h, O.MLP(*hh.host["policy"], name), O.MLP(*hh.host["value"], name))
        assert_fp_close(logits.cpu().numpy(), lr)
        assert_fp_close(value.cpu().numpy(), vr)
        p = O.softmax(logits.cpu().numpy())
        assert np.allclose(p.sum(axis=1), 1.0)


def test_entry_points_replay_from_a_hip_graph():
    """encoder_forward_packed + policy_value_head enqueue kernels only: captured once (after one ordinary call),
    every replay - with eager calls and synchronisations in between - reproduces the eager result bit for bit."""
    B, R = _mods()
    shape = synth.tiny_shape(n_layers=2, d=128, n_heads=4, n_kv_heads=2, head_dim=32, f=264, vocab=300,
                             n_actions=6, head_hidden=(32,))
    enc = R.EncoderHandle(shape, seed=3)
    head = R.HeadHandle(shape, seed=3)
    lens = [17, 40, 5]
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ids = R.dev(synth.token_ids(3, 500, (int(cu[-1]),), shape.vocab))
    cu_dev = R.dev(cu)
    ws = R.Workspace(B.brl_encoder_packed_workspace_bytes(enc.struct, 3, int(cu[-1]), 40))
    hws = R.Workspace(B.brl_head_workspace_bytes(head.struct, 3))
    h = torch.empty((3, shape.d), dtype=torch.float32, device="cuda")
    logits = torch.empty((3, 6), dtype=torch.float32, device="cuda")
    value = torch.empty((3,), dtype=torch.float32, device="cuda")

    def call():
        B.encoder_forward_packed(enc.struct, ids, cu_dev, cu, 3, 40, h, ws.buf)
        B.policy_value_head(head.struct, h, 3, logits, value, hws.buf)

    call()
    torch.cuda.synchronize()
    ref = (h.clone(), logits.clone(), value.clone())
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    for _ in range(4):
        h.zero_(); logits.zero_(); value.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(h, ref[0]) and torch.equal(logits, ref[1]) and torch.equal(value, ref[2])
        call()                               # eager work between replays
        torch.cuda.synchronize()
        assert torch.equal(h, ref[0])
