"""GPU parity of the critic variants (int8-weight BitLinear, int8-weight encoder, ensemble of value
heads), through the C ABI, against oracle/critic_oracle.py.

Integer stages (int8 weight codes, int8 activations, int32 accumulators) must be bit-exact and the
weight scale equal; one int8 BitLinear output agrees to max relative error 1e-5 (in practice bit for
bit: the same fp32 operations in the same order); encoder outputs to cosine >= 0.999 per state;
ensemble members to the head tolerance, the mean exactly from the members."""
import numpy as np
import pytest

from oracle import bitrl_oracle as O
from oracle import critic_oracle as C
from paper_2604_24273_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _mods():
    from paper_2604_24273_amd import binding as B
    from paper_2604_24273_amd import runtime as R
    B.lib()
    return B, R


def _close(got, ref, rel=1e-5):
    got = np.asarray(got, np.float64); ref = np.asarray(ref, np.float64)
    scale = np.abs(ref).max()
    d = np.abs(got - ref)
    assert d.max() <= rel * scale, "max rel err %.3e" % (d.max() / max(scale, 1e-300))
    assert np.all(d <= rel * np.abs(ref) + 0.1 * rel * scale)


def cosine(a, b):
    a = np.asarray(a, np.float64).ravel(); b = np.asarray(b, np.float64).ravel()
    return float(a @ b / (np.linalg.norm(a) * np.linalg.norm(b)))


@pytest.mark.parametrize("n,k", [(96, 256), (100, 200), (33, 136), (640, 2560), (1, 8), (257, 6912)])
def test_int8_weight_quantisation_is_bit_exact(n, k):
    B, R = _mods()
    print("bitlinear_quantize_weights_int8", n, k, flush=True)
    W = synth.normal(3, 1, (n, k), synth.W_STD)
    codes_ref, s_ref = C.int8_quantize(W)
    pl = R.quantize_linear(W, want_codes=True, int8=True)
    assert pl.packed.numel() == B.brl_packed_int8_bytes(n, k)
    assert np.array_equal(pl.codes.cpu().numpy(), codes_ref)
    assert np.float32(pl.beta.item()) == s_ref
    un = torch.empty((n, k), dtype=torch.int8, device="cuda")
    B.brl_unpack_codes_int8(pl.packed, n, k, un)
    assert np.array_equal(un.cpu().numpy(), codes_ref)
    # padding of the blob is zero (it is multiplied by activation padding, but must not hold junk)
    assert int(pl.packed.view(torch.int8).to(torch.int64).abs().sum().item()) == int(np.abs(codes_ref.astype(np.int64)).sum())


@pytest.mark.parametrize("qmax", [7, 1, 100])
def test_weight_quantisation_on_other_grids(qmax):
    """qmax = 7 is the grid of the int4 critic; the layer built on it matches the oracle like the int8 one."""
    B, R = _mods()
    n, k, m = 200, 520, 37
    c = synth.bitlinear_case(8, n, k, m)
    codes_ref, s_ref = C.int8_quantize(c["W"], qmax=qmax)
    pl = R.quantize_linear(c["W"], want_codes=True, int8=True, qmax=qmax)
    assert np.array_equal(pl.codes.cpu().numpy(), codes_ref) and np.float32(pl.beta.item()) == s_ref
    assert int(pl.codes.abs().max().item()) == qmax
    y = torch.empty((m, n), dtype=torch.float32, device="cuda")
    acc = torch.empty((m, n), dtype=torch.int32, device="cuda")
    ws = R.Workspace(B.brl_bitlinear_workspace_bytes(m, n, k))
    B.bitlinear_int8_forward(pl.packed, pl.beta, n, k, R.dev(c["X"]), m, 1e-5, y, None, None, None, acc, ws.buf)
    taps = {}
    y_ref = C.int8_bitlinear_forward(c["X"], codes_ref, s_ref, taps=taps)
    assert np.array_equal(acc.cpu().numpy(), taps["acc"])
    _close(y.cpu().numpy(), y_ref)


def test_int8_weight_quantisation_special_cases():
    B, R = _mods()
    Z = np.zeros((40, 64), np.float32)
    pl = R.quantize_linear(Z, want_codes=True, int8=True)
    assert int(pl.codes.abs().sum().item()) == 0 and np.float32(pl.beta.item()) == np.float32(np.float32(1e-5) / np.float32(127))
    W = synth.normal(4, 1, (64, 128))
    a = R.quantize_linear(W, want_codes=True, int8=True)
    b = R.quantize_linear(W * np.float32(2.0 ** -9), want_codes=True, int8=True)
    assert torch.equal(a.codes, b.codes)
    Wbad = W.copy(); Wbad[5, 7] = np.nan
    with pytest.raises(B.BitrlError):
        R.quantize_linear(Wbad, int8=True)
    Wbad[5, 7] = -np.inf
    with pytest.raises(B.BitrlError):
        R.quantize_linear(Wbad, int8=True)


@pytest.mark.parametrize("n,k", [(96, 256), (100, 200), (520, 1024)])
@pytest.mark.parametrize("m", [1, 3, 37, 128, 300])
def test_int8_bitlinear_forward(n, k, m):
    B, R = _mods()
    print("bitlinear_int8_forward", n, k, m, flush=True)
    c = synth.bitlinear_case(5, n, k, m)
    codes, scale = C.int8_quantize(c["W"])
    taps = {}
    y_ref = C.int8_bitlinear_forward(c["X"], codes, scale, taps=taps)
    pl = R.quantize_linear(c["W"], int8=True)
    x = R.dev(c["X"])
    ws = R.Workspace(B.brl_bitlinear_workspace_bytes(m, n, k))
    y = torch.empty((m, n), dtype=torch.float32, device="cuda")
    xq = torch.empty((m, k), dtype=torch.int8, device="cuda")
    am = torch.empty((m,), dtype=torch.float32, device="cuda")
    acc = torch.empty((m, n), dtype=torch.int32, device="cuda")
    B.bitlinear_int8_forward(pl.packed, pl.beta, n, k, x, m, 1e-5, y, None, xq, am, acc, ws.buf)
    assert np.array_equal(xq.cpu().numpy(), taps["xq"])
    assert np.array_equal(am.cpu().numpy(), taps["absmax"])
    assert np.array_equal(acc.cpu().numpy(), taps["acc"])
    _close(y.cpu().numpy(), y_ref)
    # without taps (the 16-byte epilogue where the shape allows it), with a residual that aliases y
    r = synth.normal(5, 7, (m, n))
    y2 = R.dev(r)
    B.bitlinear_int8_forward(pl.packed, pl.beta, n, k, x, m, 1e-5, y2, y2, None, None, None, ws.buf)
    _close(y2.cpu().numpy(), C.int8_bitlinear_forward(c["X"], codes, scale, residual=r))
    y3 = torch.empty_like(y)
    B.bitlinear_int8_forward(pl.packed, pl.beta, n, k, x, m, 1e-5, y3, None, None, None, None, ws.buf)
    assert torch.equal(y3, y)          # both epilogues give the same bits
    # bf16 activations are widened exactly
    xb = x.to(torch.bfloat16)
    y4 = torch.empty_like(y)
    B.bitlinear_int8_forward(pl.packed, pl.beta, n, k, xb, m, 1e-5, y4, None, None, None, None, ws.buf)
    _close(y4.cpu().numpy(), C.int8_bitlinear_forward(xb.float().cpu().numpy(), codes, scale))


@pytest.mark.parametrize("m,n,k", [
    (64, 4096, 136), (64, 4100, 136), (20, 8224, 136),     # 256 tiles of 32 x 32, two more blocks, one token block of many columns
    (320, 4480, 136), (448, 3232, 136),                    # 700 tiles of 64 x 32, 707 (64 x 64)
    (1280, 3200, 136), (832, 4928, 136), (832, 4928, 4096),    # 1000 tiles of 64 x 64, 1001 (128 x 128), 1001 with a long k
])
def test_int8_dispatch_edges(m, n, k):
    """Both sides of every limit of the int8-weight dispatch, through both epilogue forms (tap / residual)."""
    B, R = _mods()
    print("int8 dispatch edges", m, n, k, flush=True)
    c = synth.bitlinear_case(9, n, k, m)
    codes, scale = C.int8_quantize(c["W"])
    pl = R.quantize_linear(c["W"], int8=True)
    ws = R.Workspace(B.brl_bitlinear_workspace_bytes(m, n, k))
    x, res = R.dev(c["X"]), synth.normal(9, 7, (m, n))
    y = torch.empty((m, n), dtype=torch.float32, device="cuda")
    acc = torch.empty((m, n), dtype=torch.int32, device="cuda")
    taps = {}
    y_ref = C.int8_bitlinear_forward(c["X"], codes, scale, taps=taps)
    B.bitlinear_int8_forward(pl.packed, pl.beta, n, k, x, m, 1e-5, y, None, None, None, acc, ws.buf)
    assert np.array_equal(acc.cpu().numpy(), taps["acc"])
    _close(y.cpu().numpy(), y_ref)
    B.bitlinear_int8_forward(pl.packed, pl.beta, n, k, x, m, 1e-5, y, R.dev(res), None, None, None, ws.buf)
    _close(y.cpu().numpy(), y_ref + res)


def test_int8_bitlinear_2b_layer_shape():
    B, R = _mods()
    n, k, m = 2560, 6912, 512
    print("bitlinear_int8_forward", n, k, m, flush=True)
    c = synth.bitlinear_case(6, n, k, m)
    codes, scale = C.int8_quantize(c["W"])
    y_ref = C.int8_bitlinear_forward(c["X"], codes, scale)
    pl = R.quantize_linear(c["W"], int8=True)
    ws = R.Workspace(B.brl_bitlinear_workspace_bytes(m, n, k))
    y = torch.empty((m, n), dtype=torch.float32, device="cuda")
    B.bitlinear_int8_forward(pl.packed, pl.beta, n, k, R.dev(c["X"]), m, 1e-5, y, None, None, None, None, ws.buf)
    _close(y.cpu().numpy(), y_ref)


@pytest.mark.parametrize("kw,b,s", [
    (dict(n_layers=2, d=256, n_heads=4, n_kv_heads=2, head_dim=64, f=384, vocab=512), 5, 40),
    (dict(n_layers=2, d=200, n_heads=2, n_kv_heads=2, head_dim=100, f=392, vocab=64), 2, 33),
    (dict(n_layers=1, d=128, n_heads=4, n_kv_heads=4, head_dim=32, f=264, vocab=300), 2, 150),
])
def test_int8_weight_encoder(kw, b, s):
    B, R = _mods()
    print("encoder_forward int8 weights", kw, b, s, flush=True)
    shape = synth.tiny_shape(**kw)
    host = []
    enc = R.EncoderHandle(shape, seed=1, layer_sink=lambda l, w: host.append(w), int8_weights=True)
    cfg = O.EncoderConfig(shape.n_layers, shape.d, shape.n_heads, shape.n_kv_heads, shape.head_dim, shape.f,
                          shape.vocab, shape.rope_theta)
    T = C.Int8Linear.from_fp32
    layers = [O.LayerWeights(w["attn_norm_g"], T(w["Wq"]), T(w["Wk"]), T(w["Wv"]), w["attn_subln_g"], T(w["Wo"]),
                             O.FFNWeights(w["ffn_norm_g"], T(w["W_gate"]), T(w["W_up"]), w["ffn_subln_g"], T(w["W_down"])))
              for w in host]
    ids = synth.token_ids(1, 500, (b, s), shape.vocab)
    lengths = synth.state_lengths(1, 501, b, 1, s)
    h_ref = O.encoder_forward(ids, synth.embedding_bf16(1, shape), layers, synth.final_norm_gain(1, shape), cfg, lengths=lengths)
    h = enc.forward(R.dev(ids), R.dev(lengths)).cpu().numpy()
    for i in range(b):
        assert cosine(h[i], h_ref[i]) >= 0.999, (i, cosine(h[i], h_ref[i]))
    assert np.abs(h - h_ref).max() / np.abs(h_ref).max() < 5e-3
    # the ternary encoder on the same master weights is a different function: the format flag is honoured
    enc_t = R.EncoderHandle(shape, seed=1)
    h_t = enc_t.forward(R.dev(ids), R.dev(lengths)).cpu().numpy()
    assert np.abs(h_t - h).max() > 1e-3 * np.abs(h).max()
    # packed variable-length entry point, same states
    cu = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    flat = np.concatenate([ids[i, :lengths[i]] for i in range(b)]).astype(np.int32)
    h_p = enc.forward_packed(R.dev(flat), cu).cpu().numpy()
    assert np.array_equal(h_p, h)


@pytest.mark.parametrize("f", [6400, 6392])
def test_int8_gate_up_tiles_give_the_same_bits(f):
    """The int8 gate | up product on both sides of its limits: up to 1024 blocks of 32 x 32 (1 and 2 states of 32 tokens),
    64 x 64 tiles up to 1000 of them (3 and 10 states), LDS tiles beyond (11).  Integer sums: the states that the batches
    share get the same bits.  Against the oracle as in the encoder test above; f off the blocks takes the ragged epilogue."""
    B, R = _mods()
    shape = synth.tiny_shape(n_layers=1, d=64, n_heads=2, n_kv_heads=1, head_dim=32, f=f, vocab=100)
    host = []
    enc = R.EncoderHandle(shape, seed=6, layer_sink=lambda l, w: host.append(w), int8_weights=True)
    ids = synth.token_ids(6, 500, (11, 32), shape.vocab)
    T, w = C.Int8Linear.from_fp32, host[0]
    layer = O.LayerWeights(w["attn_norm_g"], T(w["Wq"]), T(w["Wk"]), T(w["Wv"]), w["attn_subln_g"], T(w["Wo"]),
                           O.FFNWeights(w["ffn_norm_g"], T(w["W_gate"]), T(w["W_up"]), w["ffn_subln_g"], T(w["W_down"])))
    cfg = O.EncoderConfig(1, 64, 2, 1, 32, f, shape.vocab, shape.rope_theta)
    ref = O.encoder_forward(ids, synth.embedding_bf16(6, shape), [layer], synth.final_norm_gain(6, shape), cfg)
    want = None
    for b in (11, 10, 3, 2, 1):
        print("int8 gate | up", f, b, flush=True)
        h = enc.forward(R.dev(ids[:b]))
        if want is None:
            want = h
            got = h.cpu().numpy()
            assert min(cosine(got[i], ref[i]) for i in range(11)) >= 0.999
            assert np.abs(got - ref).max() <= 5e-3 * np.abs(ref).max()
        assert torch.equal(h, want[:b]), b


@pytest.mark.parametrize("m,n", [
    (4193, 3072), (4100, 3290), (8192, 2048),                   # 396 and 429 tiles of 128 x 256, rows and columns ending inside a tile; 512
    (4096, 3072), (4096, 3040),                                 # beside the rule: no more than three 128 x 128 tiles per compute unit,
    (4064, 2816), (8192, 2080),                                 # 0.69 and 1.13 rounds,
    (4065, 3330), (9000, 3200), (49152, 128), (24576, 320),     # padding: one tile in 27, one in 25, every other, one in three
])
def test_int8_wide_tile(m, n):
    """Both sides of the rule that takes the 128 x 256 tile on int8 weights, as in the dispatch test above."""
    test_int8_dispatch_edges(m, n, 136)


@pytest.mark.parametrize("m,n,k", [(8192, 3840, 1536), (8192, 3840, 1400), (15400, 1930, 1544), (15500, 1930, 1544)])
def test_int8_wide_tile_past_the_first_round(m, n, k):
    """Twelve super-blocks of k on 1.9 rounds of 128 x 256 tiles; eleven on 128 x 128.  Likewise 1.89 rounds with ragged rows
    and columns; 1.91 on 128 x 128, past nine tenths of the last one."""
    test_int8_dispatch_edges(m, n, k)


@pytest.mark.parametrize("f", [6400, 6392])
def test_int8_gate_up_on_the_wide_tile_gives_the_same_bits(f):
    """Gate | up on 450 wide tiles (36 states of 32 tokens), on narrow ones beside the rule (42 and 11): the same bits.
    (Against the oracle: the test above.)"""
    B, R = _mods()
    shape = synth.tiny_shape(n_layers=1, d=64, n_heads=2, n_kv_heads=1, head_dim=32, f=f, vocab=100)
    enc = R.EncoderHandle(shape, seed=6, int8_weights=True)
    ids = synth.token_ids(6, 500, (42, 32), shape.vocab)
    want = enc.forward(R.dev(ids))
    for b in (36, 11):
        print("int8 gate | up, wide tile", f, b, flush=True)
        assert torch.equal(enc.forward(R.dev(ids[:b])), want[:b]), b


@pytest.mark.parametrize("n_states,S", [(128, 128), (170, 96)])
def test_int8_qkv_product_writing_attention_operands_matches_two_step_path(n_states, S):
    """Uniform batches at head_dim 128 with enough rows: the int8-weight q | k | v product writes the attention operands
    itself.  The same states one per call and back to back take fp32 rows and the pack kernel: every bit agrees."""
    B, R = _mods()
    shape = synth.tiny_shape(n_layers=2, d=256, n_heads=4, n_kv_heads=2, head_dim=128, f=512, vocab=300, rope_theta=500000.0)
    enc = R.EncoderHandle(shape, seed=5, int8_weights=True)
    ids = synth.token_ids(5, 500, (n_states, S), shape.vocab)
    print("fused int8 q|k|v epilogue: %d states x %d tokens" % (n_states, S), flush=True)
    h = enc.forward(R.dev(ids))
    for b in (0, 1, n_states // 2, n_states - 1):
        assert torch.equal(h[b:b + 1], enc.forward(R.dev(ids[b:b + 1]))), b
    cu = (np.arange(n_states + 1) * S).astype(np.int32)
    assert torch.equal(h, enc.forward_packed(R.dev(ids.reshape(-1).astype(np.int32)), cu, max_len=S))


@pytest.mark.parametrize("dims,n_members,act,batch", [
    ([2560, 256, 1], 3, "tanh", 64),
    ([2560, 256, 1], 5, "tanh", 7),
    ([64, 32, 16, 1], 5, "relu", 33),
    ([48, 1], 8, "tanh", 5),
    ([96, 40, 1], 1, "relu", 2),
])
def test_value_ensemble(dims, n_members, act, batch):
    B, R = _mods()
    print("value_ensemble_forward", dims, n_members, act, batch, flush=True)
    members = [synth.mlp_params(9, 400 + 20 * e, dims) for e in range(n_members)]
    h = synth.normal(9, 399, (batch, dims[0]))
    ref_mean, ref_each = C.value_ensemble(h, [O.MLP(ws, bs, act) for ws, bs in members])
    code = B.BRL_ACT_TANH if act == "tanh" else B.BRL_ACT_RELU
    ens = R.ValueEnsemble(members, act=code)
    mean, each = ens.forward(R.dev(h))
    each_h, mean_h = each.cpu().numpy(), mean.cpu().numpy()
    assert np.abs(each_h - ref_each).max() <= 2e-6 * max(np.abs(ref_each).max(), 1.0)
    assert np.abs(mean_h - ref_mean).max() <= 2e-6 * max(np.abs(ref_each).max(), 1.0)
    # the mean is exactly the fp64 mean of the members' fp32 values, in member order
    t = np.zeros(batch, np.float64)
    for e in range(n_members):
        t = t + each_h[e].astype(np.float64)
    assert np.array_equal(mean_h, (t / n_members).astype(np.float32))
    # without the per-member output; and each member equals the single-head entry point bit for bit
    mean2, none = ens.forward(R.dev(h), want_each=False)
    assert none is None and torch.equal(mean2, mean)
    pw, pb = synth.mlp_params(9, 390, [dims[0], 4])
    for e in (0, n_members - 1):
        pol, k1 = B.make_mlp([R.dev(w) for w in pw], [R.dev(b) for b in pb], code)
        val, k2 = B.make_mlp([R.dev(w) for w in members[e][0]], [R.dev(b) for b in members[e][1]], code)
        head = B.brl_head(pol, val)
        logits = torch.empty((batch, 4), dtype=torch.float32, device="cuda")
        value = torch.empty((batch,), dtype=torch.float32, device="cuda")
        ws = R.Workspace(B.brl_head_workspace_bytes(head, batch))
        B.policy_value_head(head, R.dev(h), batch, logits, value, ws.buf)
        assert torch.equal(value, each[e])


@pytest.mark.parametrize("dims_p,dims_v,acts,batch", [
    ([2560, 256, 18], [2560, 256, 1], ("tanh", "tanh"), 1),
    ([2560, 256, 128, 18], [2560, 256, 1], ("relu", "relu"), 65),       # heads of unequal depth, one sample past a tile block
    ([37, 5], [37, 1], ("tanh", "tanh"), 67),                           # no hidden layer, inputs off every chunk
    ([130, 17, 33, 9], [130, 15, 1], ("tanh", "relu"), 64),             # different activations: one head after the other
    ([96, 2100, 700, 6], [96, 2050, 1], ("tanh", "tanh"), 5),           # too wide for a workgroup per sample: a launch per level
])
def test_policy_value_head_shapes(dims_p, dims_v, acts, batch):
    """fp64 sums rounded once: fp32 outputs within 1e-6 of the oracle's (2^-24 and the fp64 activation's last bits)."""
    B, R = _mods()
    codes = [B.BRL_ACT_TANH if a == "tanh" else B.BRL_ACT_RELU for a in acts]
    pw, pb = synth.mlp_params(23, 10, dims_p)
    vw, vb = synth.mlp_params(23, 40, dims_v)
    h = synth.normal(23, 70, (batch, dims_p[0]))
    pol, k1 = B.make_mlp([R.dev(w) for w in pw], [R.dev(b) for b in pb], codes[0])
    val, k2 = B.make_mlp([R.dev(w) for w in vw], [R.dev(b) for b in vb], codes[1])
    head = B.brl_head(pol, val)
    logits = torch.empty((batch, dims_p[-1]), dtype=torch.float32, device="cuda")
    value = torch.empty((batch,), dtype=torch.float32, device="cuda")
    ws = R.Workspace(B.brl_head_workspace_bytes(head, batch))
    B.policy_value_head(head, R.dev(h), batch, logits, value, ws.buf)
    l_ref, v_ref = O.policy_value_head(h, O.MLP(pw, pb, acts[0]), O.MLP(vw, vb, acts[1]))
    assert np.abs(logits.cpu().numpy() - l_ref).max() <= 1e-6 * np.abs(l_ref).max()
    assert np.abs(value.cpu().numpy() - np.asarray(v_ref).reshape(-1)).max() <= 1e-6 * max(np.abs(v_ref).max(), 1.0)


@pytest.mark.parametrize("dims", [[2560, 1], [2560, 256, 1], [1000, 40, 24, 1], [640, 512, 512, 1], [96, 2100, 1], [60, 700, 400, 1]])
def test_value_head_bits_do_not_depend_on_what_shares_the_call(dims):
    """A value head gives the same bits beside any policy head, in an ensemble of any size and in a batch of any size.
    The inputs of the first layer cancel to about 1e-9 of their size, so that another order of the fp64 sums would show
    in the fp32 results.  The last two: wide heads (a launch per level), alone and beside a policy head that is not."""
    B, R = _mods()
    rng = np.random.default_rng(7)
    d, n = dims[0], 8
    pairs = rng.permutation(d - 2).reshape(-1, 2)
    rest = [i for i in range(d) if i >= d - 2]

    def params(e):
        ws, bs = synth.mlp_params(31, 20 * e, dims)
        w = ws[0].copy()
        w[:, pairs[:, 1]] = -w[:, pairs[:, 0]]
        w[:, rest] *= np.float32(2.0 ** -30)
        return [w] + list(ws[1:]), [np.zeros_like(b) for b in bs]

    h = synth.normal(31, 399, (200, d))
    h[:, pairs[:, 1]] = h[:, pairs[:, 0]]
    h_dev = R.dev(h)
    members = [params(e) for e in range(n)]

    def value(e, policy_dims, batch):
        pw, pb = synth.mlp_params(31, 390, policy_dims)
        pol, k1 = B.make_mlp([R.dev(w) for w in pw], [R.dev(b) for b in pb], B.BRL_ACT_RELU)
        val, k2 = B.make_mlp([R.dev(w) for w in members[e][0]], [R.dev(b) for b in members[e][1]], B.BRL_ACT_RELU)
        head = B.brl_head(pol, val)
        logits = torch.empty((batch, policy_dims[-1]), dtype=torch.float32, device="cuda")
        out = torch.empty((batch,), dtype=torch.float32, device="cuda")
        ws = R.Workspace(B.brl_head_workspace_bytes(head, batch))
        B.policy_value_head(head, h_dev[:batch].contiguous(), batch, logits, out, ws.buf)
        p_ref = O.policy_value_head(h[:batch], O.MLP(pw, pb, "relu"), O.MLP(*members[e], "relu"))[0]
        assert np.abs(logits.cpu().numpy() - p_ref).max() <= 1e-6 * np.abs(p_ref).max()
        return out

    want = [value(e, [d, 4], 200) for e in (0, n - 1)]
    assert all(float(w.abs().max()) < 1e-3 for w in want)
    for policy_dims, batch in (([d, 4], 1), ([d, 4], 64), ([d, 700], 65), ([d, 256, 18], 64), ([d, 1200, 6], 129)):
        print("value head", dims, "beside", policy_dims, batch, flush=True)
        assert torch.equal(value(0, policy_dims, batch), want[0][:batch]), (policy_dims, batch)
    for members_n, batch in ((1, 64), (2, 200), (3, 64), (5, 65), (8, 1), (8, 200)):
        print("ensemble", dims, members_n, batch, flush=True)
        ens = R.ValueEnsemble(members[:members_n - 1] + members[-1:] if members_n > 1 else members[:1], act=B.BRL_ACT_RELU)
        mean, each = ens.forward(h_dev[:batch].contiguous())
        assert torch.equal(each[0], want[0][:batch]), (members_n, batch)
        if members_n > 1:
            assert torch.equal(each[-1], want[1][:batch]), (members_n, batch)


@pytest.mark.parametrize("d,batch", [(1000, 577), (2560, 640), (70, 520)])
def test_ensemble_of_many_tiles_gives_the_bits_of_few(d, batch):
    """Eight members of 256 units: beyond 1024 tiles of 16 units x 64 samples a workgroup takes all groups of inputs of its
    tile, up to there one of them.  Same bits, and the oracle's values."""
    B, R = _mods()
    members = [synth.mlp_params(33, 20 * e, [d, 256, 1]) for e in range(8)]
    h = synth.normal(33, 399, (batch, d))
    ens = R.ValueEnsemble(members, act=B.BRL_ACT_TANH)
    print("ensemble, many tiles", d, batch, flush=True)
    mean, each = ens.forward(R.dev(h))
    ref_mean, ref_each = C.value_ensemble(h, [O.MLP(ws, bs, "tanh") for ws, bs in members])
    assert np.abs(each.cpu().numpy() - ref_each).max() <= 2e-6 * max(np.abs(ref_each).max(), 1.0)
    for lo, hi in ((0, 64), (64, 65), (100, 300), (batch - 16, batch)):
        few_mean, few = ens.forward(R.dev(h[lo:hi]))
        assert torch.equal(few, each[:, lo:hi]) and torch.equal(few_mean, mean[lo:hi]), (lo, hi)
