"""Single kernels at the sizes where their tiles, splits and remainders can go wrong, against the oracle."""
import numpy as np
import pytest

import mt_synth as ms
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2107_05377_amd as mt  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    mt.lib()


def dev(x, dtype=None):
    t = torch.from_numpy(np.ascontiguousarray(x)).cuda()
    return t if dtype is None else t.to(dtype)


# one row, full and one-over row blocks, remainders of columns; K of the short-K kernel's forms and, from 256 on, of the block list, with as many slices as its
# rings hold and more, equal quarters and not
@pytest.mark.parametrize("M,N,K", [(1, 4, 64), (32, 100, 192), (33, 68, 64), (65, 64, 128), (31, 32, 832), (2113, 2052, 64), (70, 100, 128), (161, 228, 640),
                                   (385, 1056, 128), (700, 1000, 192)])
@pytest.mark.parametrize("act", [0, 1])
def test_gemm_f32_tiles(M, N, K, act):
    print(f"gemm_f32 {M}x{N}x{K} act {act}", flush=True)
    rng = np.random.default_rng(M + N + K)
    A, W = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((N, K)).astype(np.float32)
    b, r = rng.standard_normal(N).astype(np.float32), rng.standard_normal((M, N)).astype(np.float32)
    out = mt.op_linear(mt.MT_FP32_CHECK, dev(A), dev(W), dev(b), residual=dev(r), act=act).cpu().numpy()
    ref = oracle.linear(A, W, b)
    if act == 1:
        ref = oracle.gelu(ref)
    ref = ref + r
    assert np.abs(out - ref).max() <= 2e-5 * max(1.0, np.abs(ref).max())


# Short K: few blocks have K dealt out to wavefronts, many have not (the line is 512 blocks of 32 x 32, K = 192: 1536).  Quarters are added up in one order, so rows of a large launch
# are the bits of a small one; remainders of rows and columns on both sides.
@pytest.mark.parametrize("G,M,N,K,act", [(g, m, n, k, a) for k in (64, 128, 192) for g, m, n, a in ((1, 1, 4, 0), (1, 33, 36, 1), (2, 300, 804, 0), (1, 993, 516, 1), (8, 130, 420, 2), (3, 650, 804, 0))] +
                         [(8, 650, 900, 256, 1), (8, 650, 900, 320, 2)])      # K that takes this kernel beyond 4700 blocks only
def test_gemm_f32_short_k(G, M, N, K, act):
    print(f"gemm_f32, short K, {G} x {M} x {N} x {K} act {act}", flush=True)
    from scipy.special import erf
    rng = np.random.default_rng(G + M + N + K)
    A, W = rng.standard_normal((G, M, K)).astype(np.float32), rng.standard_normal((G, N, K)).astype(np.float32)
    b, r = rng.standard_normal((G, N)).astype(np.float32), rng.standard_normal((G, M, N)).astype(np.float32)
    out = torch.full((G * M + 1, N), 7.0, dtype=torch.float32, device="cuda")
    mt.op_linear_batched(mt.MT_FP32_CHECK, dev(A), dev(W), dev(b), residual=dev(r), act=act, out=out[:G * M].view(G, M, N))
    got = out.cpu().numpy()
    assert (got[G * M:] == 7.0).all()
    got = got[:G * M].reshape(G, M, N)
    few = min(M, 40)                                     # at most 512 blocks of each problem
    for i in range(G):
        one = mt.op_linear(mt.MT_FP32_CHECK, dev(A[i, -few:]), dev(W[i]), dev(b[i]), residual=dev(r[i, -few:]), act=act)
        assert np.array_equal(got[i, -few:], one.cpu().numpy()), i
    x = A.astype(np.float64) @ W.astype(np.float64).transpose(0, 2, 1) + b[:, None]
    # a quarter of K one after another, the four, the bias; GELU: slope below 1.13, 1e-6 for erff and tanhf
    bound = ((K + 128) / 4 + 8) * 2.0**-24 * (np.abs(A) @ np.abs(W).transpose(0, 2, 1) + np.abs(b[:, None]))      # (a quarter is whole slices)
    if act:
        x = x * 0.5 * (1 + (erf(x / 2**0.5) if act == 1 else np.tanh((2 / np.pi)**0.5 * (x + 0.044715 * x**3))))
        bound = 1.13 * bound + 1e-6 * (1 + np.abs(x))
    assert (np.abs(got - (x + r)) <= bound + 2.0**-23 * np.abs(r)).all()


# the block list of the float32 tile kernel: one block and several per workgroup (more than two per compute unit of 256), remainders of rows, columns and of the
# four K shares (equal and not), as few slices as the ring has and more, one problem and several
@pytest.mark.parametrize("G,M,N,K,act", [(1, 33, 36, 256, 0), (1, 64, 96, 320, 0), (3, 97, 100, 448, 0), (1, 3, 36, 256, 0), (8, 20, 100, 416, 0), (1, 1500, 1028, 256, 0), (8, 130, 516, 320, 0),
                                         (2, 700, 800, 768, 0), (5, 40, 64, 3072, 0), (1, 40, 64, 448, 3), (1, 1500, 1028, 256, 1), (8, 130, 516, 320, 2), (2, 700, 800, 768, 3)])
def test_gemm_f32_block_list(G, M, N, K, act):
    """With an activation also a residual: both wait, with the block's sums, for the second slice of the next block or, of a workgroup's last block, for the end."""
    print(f"gemm_f32, {G} x {M} x {N} x {K} act {act}", flush=True)
    from scipy.special import erf
    rng = np.random.default_rng(G + M + N + K)
    A, W = rng.standard_normal((G, M, K)).astype(np.float32), rng.standard_normal((G, N, K)).astype(np.float32)
    b = rng.standard_normal((G, N)).astype(np.float32)
    r = rng.standard_normal((G, M, N)).astype(np.float32) if act else np.zeros((G, M, N), np.float32)
    out = torch.full((G * M + 1, N), 7.0, dtype=torch.float32, device="cuda")
    mt.op_linear_batched(mt.MT_FP32_CHECK, dev(A), dev(W), dev(b), residual=dev(r) if act else None, act=act, out=out[:G * M].view(G, M, N))
    x = A.astype(np.float64) @ W.astype(np.float64).transpose(0, 2, 1) + b[:, None]
    # a quarter of K one after another, the four shares, the bias: each addition rounds at most by 2^-24 of the sum of magnitudes
    bound = (K / 4 + 8) * 2.0**-24 * (np.abs(A) @ np.abs(W).transpose(0, 2, 1) + np.abs(b[:, None]))
    if act in (1, 2):                                    # slope below 1.13, 1e-6 for erff and tanhf
        x = x * 0.5 * (1 + (erf(x / 2**0.5) if act == 1 else np.tanh((2 / np.pi)**0.5 * (x + 0.044715 * x**3))))
        bound = 1.13 * bound + 1e-6 * (1 + np.abs(x))
    elif act == 3:                                       # slope 1, 2^-21 for tanhf
        x, bound = np.tanh(x), bound + 2.0**-21
    if act:
        bound = bound + 2.0**-23 * np.abs(r)             # the last addition, of the residual
    got = out.cpu().numpy()
    assert (np.abs(got[:G * M].reshape(G, M, N) - (x + r)) <= bound).all()
    assert (got[G * M:] == 7.0).all()                    # nothing beyond the last row


@pytest.mark.parametrize("B,S,H,A", [(2, 1, 64, 1), (3, 31, 64, 2), (2, 33, 128, 2), (1, 130, 64, 1), (2, 257, 64, 2)])
def test_attention_f32_blocks(B, S, H, A):
    print(f"attention_f32 B={B} S={S} H={H} A={A}", flush=True)
    rng = np.random.default_rng(S)
    q, k, v = (rng.standard_normal((B, S, H)).astype(np.float32) for _ in range(3))
    mask = (np.arange(S)[None, :] < rng.integers(1, S + 1, B)[:, None]).astype(np.int32)
    mask[0] = 1
    if S > 8:
        mask[0, 3:7] = 0
    qkv = np.concatenate([q, k, v], axis=2).reshape(B * S, 3 * H)
    ctx = mt.op_attention(mt.MT_FP32_CHECK, dev(qkv), dev(mask), B, S, H, A).cpu().numpy().reshape(B, S, H)
    assert np.abs(ctx - oracle.attention(q, k, v, mask, A)).max() <= 2e-5


@pytest.mark.parametrize("S,H", [(33, 64), (35, 32), (64, 64)])
def test_attention_f32_infinite_value_of_the_last_key(S, H):
    """An infinite value makes its own column infinite and no NaN, also where the last key block is not full."""
    print(f"attention_f32 infinite value S={S} H={H}", flush=True)
    rng = np.random.default_rng(S)
    q, k, v = (rng.standard_normal((1, S, H)).astype(np.float32) for _ in range(3))
    ref = oracle.attention(q, k, v, np.ones((1, S), np.int32), 1)
    v[0, -1, 5] = np.inf
    ctx = mt.op_attention(mt.MT_FP32_CHECK, dev(np.concatenate([q, k, v], axis=2)[0]), dev(np.ones((1, S), np.int32)), 1, S, H, 1).cpu().numpy().reshape(1, S, H)
    rest = np.arange(H) != 5
    assert (ctx[..., 5] == np.inf).all() and np.abs(ctx[..., rest] - ref[..., rest]).max() <= 2e-5


# The panel layout through a whole model: ragged rows and the launch shapes that a rule on sizes chooses, put together (the kernels one by one:
# below).  Weights grow as the model gets narrower, so that a layer's output is of the size of its input at every width.
# Bound on the logits: bfloat16 operands (2^-8 each) through three layers give at most 2e-2 at logits of order 1.
@pytest.mark.parametrize("heads,ffn,batch,seq,lo", [
    (1, 64, 1, 1, 1),            # one row; K below one tile's ring
    (16, 192, 33, 65, 1),        # 16 heads; one sequence over a panel of first tokens; sequences that end one row into a key panel
    (2, 320, 2, 289, 280),       # key panels shared by two wavefronts, an odd number of them
    (10, 2112, 300, 9, 1),       # K split between wavefronts; a long K that no tile's slices divide
    (10, 2048, 720, 31, 17),     # pairs of workgroups per compute unit; tall tiles for the long K
    (12, 2048, 29, 70, 30),      # the trunk's long K in two ranges of tiles, 64 row panels by the bound
    (1, 16384, 2048, 33, 2),     # an operand of more than 2 GiB
])
def test_panel_layout_forms(heads, ffn, batch, seq, lo):
    print(f"panel layout: {heads} heads, ffn {ffn}, {batch} x {seq}", flush=True)
    spec = ms.MTSpec("panels", vocab=300, hidden=64 * heads, heads=heads, ffn=ffn, max_pos=seq + 1, n_trunk_layers=1,
                     tasks=(ms.TaskSpec(1, 2, 3), ms.TaskSpec(0, 1, 2), ms.TaskSpec(1, 0, 2)), precision="bf16", batch=batch, seq=seq,
                     len_lo=lo, len_hi=seq, input_seed=heads + seq)
    model, (trunk, tasks) = mt.load_synthetic(spec, keep_params=True, std=0.03 * max(1.0, (768 / spec.hidden)**0.5))
    ids, mask, _ = ms.make_inputs(spec)
    got = model.forward(dev(ids), dev(mask)).cpu().numpy()
    pick = np.unique(np.linspace(0, batch - 1, 7).astype(int))
    ref = oracle.Oracle(spec, trunk, tasks).mt_forward(ids[pick], mask[pick])
    err = np.abs(got[pick] - ref).max()
    print(f"  max |dlogit| {err:.3g}, logits up to {np.abs(ref).max():.3g}", flush=True)
    assert np.isfinite(got).all() and err <= 2e-2 * max(1.0, np.abs(ref).max())
    model.close()


def test_weight_layout_does_not_depend_on_a_handles_bounds():
    """Handles of different max_batch x max_seq share one weight arena (mt_share_weights), so its layout must be the same for all of them.  The
    owner's bound is beyond 65535 x 32 rows and takes more few-row workgroups along the rows than a grid has (65535 of 64 rows)."""
    batch, seq = 65535, 65
    spec = ms.MTSpec("bounds", vocab=300, hidden=64, heads=1, ffn=64, max_pos=seq, n_trunk_layers=1, tasks=(ms.TaskSpec(1, 2, 3), ms.TaskSpec(0, 1, 2)),
                     precision="bf16", batch=batch, seq=seq, len_lo=1, len_hi=seq, input_seed=5)
    owner, (trunk, tasks) = mt.load_synthetic(spec, keep_params=True, std=0.1)
    small = mt.Model(mt.make_config(spec, max_batch=5, max_seq=seq), bind=False)
    small.weights = owner.weights
    small.workspace = torch.empty(small.workspace_bytes(), dtype=torch.uint8, device="cuda")
    small._check(mt.lib().mt_bind(small.h, owner.weights.data_ptr(), owner.weights.numel(), small.workspace.data_ptr(), small.workspace.numel()))
    small._check(mt.lib().mt_share_weights(small.h, owner.h))
    ids, mask, _ = ms.make_inputs(spec)
    mask[-1] = 1                                   # the last panel of the bound is reached if every position before it is kept
    pick = np.array([0, 1, 31000, 65533, 65534])
    ref = oracle.Oracle(spec, trunk, tasks).mt_forward(ids[pick], mask[pick])
    bound = 2e-2 * max(1.0, np.abs(ref).max())     # bfloat16 operands through three layers, relative to the logits
    few = small.forward(dev(ids[pick]), dev(mask[pick])).cpu().numpy()
    print(f"replica: max |dlogit| {np.abs(few - ref).max():.3g}, logits up to {np.abs(ref).max():.3g}", flush=True)
    assert np.abs(few - ref).max() <= bound
    for m in (mask, np.ones_like(mask)):           # 2.1 and 4.3 million rows
        ref = oracle.Oracle(spec, trunk, tasks).mt_forward(ids[pick], m[pick])
        got = owner.forward(dev(ids), dev(m)).cpu().numpy()[pick]
        print(f"owner: max |dlogit| {np.abs(got - ref).max():.3g}", flush=True)
        assert np.abs(got - ref).max() <= bound
    small.close()
    owner.close()


def ragged_rows(lens, gap, rng):
    """(row0, total): sequences of these lengths behind one another with up to `gap` rows of no sequence between them."""
    row0, at = [], 0
    for n in lens:
        at += int(rng.integers(0, gap + 1))
        row0.append(at)
        at += int(n)
    return np.array(row0, np.int32), at + int(rng.integers(0, gap + 1))


def bf16(x):
    return torch.from_numpy(np.ascontiguousarray(x, np.float32)).to(torch.bfloat16).double().numpy()


# q~ and the weighted row sums against float64 on the same bf16 operands.  Rows of no sequence hold NaN; `late` puts each head's highest scores
# into the last key panel, 20 above the first ones, so that the running maximum has to follow.
# Bounds (bfloat16 rounds to 2^-8 of the value).  q~: the query (2^-8 of each q, so 2^-8 sum |Wk q|) and the result round once each.  Row sums:
# the result rounds once; the weights are float32 quantities: 2^-14 sum p |x| is what scores of |s| <= 50 summed in float32 (2^-24 sqrt(H) |s|)
# can shift them.
@pytest.mark.parametrize("heads,lens,late", [(1, [1, 32, 33], False), (2, [31, 65, 64, 1], True), (3, [200, 7], True), (5, [97] * 33, True), (11, [40, 128, 3], False),
                                             (12, [128, 127, 70], True), (16, [1, 257, 64], True)] + [(h, [33, 2, 70], True) for h in (4, 6, 7, 8, 9, 10, 13, 14, 15)] +
                         [(16, [2] * 545, False)])           # every width, and more panels of sequences than workgroups
def test_first_token_panels(heads, lens, late):
    print(f"first token: {heads} heads, {lens}, late {late}", flush=True)
    H, B, rng = 64 * heads, len(lens), np.random.default_rng(heads)
    row0, rows = ragged_rows(lens, 5, rng)
    first, Wq, Wk, bq = bf16(rng.standard_normal((B, H))), bf16(rng.standard_normal((H, H)) / H**0.5), bf16(rng.standard_normal((H, H)) / H**0.5), rng.standard_normal(H).astype(np.float32)
    panels = lambda x: mt.to_panels(torch.from_numpy(x).cuda(), torch.bfloat16)
    qt = mt.op_panel_first_query(panels(first), panels(Wq), dev(bq), panels(np.ascontiguousarray(Wk.T)), B, heads)
    q = (first @ Wq.T + bq).reshape(B, heads, 64)
    want = np.einsum("bad,adh->bah", q, Wk.reshape(heads, 64, H))
    bound = 1.01 * 2.0**-8 * np.abs(want) + 2.0**-8 * np.einsum("bad,adh->bah", np.abs(q), np.abs(Wk).reshape(heads, 64, H)) + 1e-30
    err = np.abs(qt[:, :heads].double().cpu().numpy() - want)
    print(f"  q~: {(err / bound).max():.3f} of the bound", flush=True)
    assert (err <= bound).all()

    x = np.full((rows, H), np.nan)
    qt16 = bf16(rng.standard_normal((B, 16, H)) * (60.0 / H**0.5 if late else 8.0 / H**0.5))
    for b, n in enumerate(lens):
        v = rng.standard_normal((n, H)) * 0.2
        if late:                              # rows lean towards the mean of the heads' q~, further from key to key
            d = qt16[b, :heads].sum(0)
            v += np.linspace(0.0, 1.0, n)[:, None] * d / (d @ d) * heads * 160.0
        x[row0[b]:row0[b] + n] = bf16(v)
    got = mt.op_panel_first_attend(panels(x), dev(qt16, torch.bfloat16), dev(row0), dev(np.array(lens, np.int32)), B, max(lens), heads).double().cpu().numpy()
    worst = 0.0
    for b, n in enumerate(lens):
        xb = x[row0[b]:row0[b] + n]
        s = qt16[b, :heads] @ xb.T / 8
        p = np.exp(s - s.max(1, keepdims=True))
        p /= p.sum(1, keepdims=True)
        want, bound = p @ xb, 1.01 * 2.0**-8 * np.abs(p @ xb) + 2.0**-14 * (p @ np.abs(xb))
        worst = max(worst, (np.abs(got[b] - want) / bound).max())
    print(f"  row sums: {worst:.3f} of the bound, scores of the last sequence up to {np.abs(s).max():.1f}, spread {np.ptp(s):.1f}", flush=True)
    assert worst <= 1.0


# Narrow models have one wavefront a sequence in large launches (the line is two sequences for each of 256 compute units) and four in small ones: the same bits.
@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("heads,B", [(1, 513), (2, 700)])
def test_first_token_panels_of_many_sequences(heads, B, fp8):
    print(f"first token, {B} sequences: {heads} heads, fp8 {fp8}", flush=True)
    H, rng = 64 * heads, np.random.default_rng(B)
    lens = rng.integers(1, 100, B).astype(np.int32)
    row0, rows = ragged_rows(lens, 5, rng)
    x = np.full((rows, H), np.nan)
    for b, n in enumerate(lens): x[row0[b]:row0[b] + n] = bf16(rng.standard_normal((n, H)))
    px, qt = mt.to_panels(torch.from_numpy(x).cuda(), torch.bfloat16), bf16(rng.standard_normal((B, 16, H)) * 8 / H**0.5)
    call = lambda lo, hi: mt.op_panel_first_attend(px, dev(qt[lo:hi], torch.bfloat16), dev(row0[lo:hi]), dev(lens[lo:hi]), hi - lo, 99, heads, fp8=fp8)
    many = call(0, B)
    assert not torch.isnan(many).any()
    for lo, hi in ((0, 37), (200, 512), (B - 64, B)):
        assert torch.equal(many[lo:hi], call(lo, hi)), (lo, hi)
    for b in (0, 31, 32, B // 2, B - 1):
        xb = x[row0[b]:row0[b] + lens[b]]
        s = qt[b, :heads] @ xb.T / 8
        p = np.exp(s - s.max(1, keepdims=True))
        p /= p.sum(1, keepdims=True)
        assert (np.abs(many[b].double().cpu().numpy() - p @ xb) <= 1.01 * 2.0**-8 * np.abs(p @ xb) + 2.0**-14 * (p @ np.abs(xb))).all(), b


# Row sums that cancel to 2^-18 of their terms show the bits of the weights: two keys of every sequence are chosen, column by column, against the
# sum of the others under one head's weights.  Weights of 24 bits from an exponential good to 2^-23 leave at most 2^-23 of sum p |x| (rms over the
# columns, independent from key to key); weights of 16 bits leave 2^-22 to 2^-20.  Scores come from one column alone, exactly.
@pytest.mark.parametrize("heads", [1, 5, 12, 16])
def test_first_token_panels_whole_weights(heads):
    lens = [4, 9, 33, 100]
    print(f"first token, whole weights: {heads} heads", flush=True)
    H, B, rng = 64 * heads, len(lens), np.random.default_rng(heads)
    row0, rows = ragged_rows(lens, 5, rng)
    qt = np.zeros((B, 16, H))
    qt[:, :, 0] = bf16(rng.uniform(2, 8, (B, 16)))
    x, ps = np.full((rows, H), np.nan), []
    for b, n in enumerate(lens):
        v = bf16(rng.standard_normal((n, H))).astype(np.float64)
        v[:, 0] = bf16(rng.uniform(-1, 1, n))
        s = qt[b, :heads, :1] * v[:, 0] / 8
        p = np.exp(s - s.max(1, keepdims=True))
        p /= p.sum(1, keepdims=True)
        own = p[np.arange(H) % heads]                      # [H][n]: the weights that column c is to cancel under
        v[n - 2:, 1:] = 0
        for k in (n - 2, n - 1):
            v[k, 1:] = bf16(-(own[1:] * v[:, 1:].T).sum(1) / own[1:, k])
        x[row0[b]:row0[b] + n] = v
        ps.append(own)
    got = mt.op_panel_first_attend(panels(x), dev(qt, torch.bfloat16), dev(row0), dev(np.array(lens, np.int32)), B, max(lens), heads, fp8=True).double().cpu().numpy()
    for b, n in enumerate(lens):
        terms = ps[b][1:] * x[row0[b]:row0[b] + n, 1:].T
        err = (got[b, np.arange(H) % heads, np.arange(H)][1:] - terms.sum(1)) / np.abs(terms).sum(1)
        print(f"  {n} keys: {np.sqrt((err**2).mean()) * 2**23:.3f} of the bound", flush=True)
        assert np.sqrt((err**2).mean()) <= 2.0**-23


def panels(x, dtype=None):
    """A float array [rows][width] in the panel layout on the device, rows of the last panel beyond it NaN."""
    return mt.to_panels(torch.from_numpy(np.ascontiguousarray(x)).cuda(), dtype or torch.bfloat16)


def nan_panels(rows, width, dtype):
    return torch.full(((rows + 31) // 32, width // 8, 32, 8), float("nan"), dtype=dtype, device="cuda")


def rows_of(p):
    return mt.from_panels(p).double().cpu().numpy()


def transposed_columns(x, first):
    """Columns from `first` on as an operand of a product over the rows: in blocks of 32 x 32, [16 rows][half][32 columns][8 rows]
    instead of [8 columns][32 rows] chunks; the array that stands at such addresses of an ordinary panel matrix."""
    rows, width = x.shape
    order = np.array([16 * r + 4 * h + (j & 3) + 8 * (j >> 2) for r in range(2) for h in range(2) for j in range(8)])     # rows of a run [r][h]
    out = x.copy()
    for p in range(0, rows, 32):
        for c in range(first, width, 32):
            runs = x[p:p + 32, c:c + 32][order].reshape(4, 8, 32)                # [run][8 rows][32 columns]
            out[p:p + 32, c:c + 32] = runs.transpose(2, 0, 1).reshape(32, 32)    # row of the chunk = column, chunk = run
    return out


ROWS_1X1, ROWS_2X1, ROWS_2X2, K2, PAIR, TALL = 1, 2, 3, 4, 5, 6


# Every form of the panel contraction and every tile height at remainders of rows, columns and K, against float64 on the same bf16 operands.
# `rows` of the M are present: what lies beyond is NaN.  Bound: K products summed in float32 in any order, K 2^-24 sum |a w| (+ bias), for
# bfloat16 results their rounding, 2^-8 of the value; GELU: slope below 1.13, 3e-5 for its fit; tanh: slope 1 and 2^-21 for tanhf.
@pytest.mark.parametrize("form,height,problems,M,rows,N,K,act,f32,splits", [
    (ROWS_1X1, 0, 1, 1, 1, 32, 64, 0, 1, 1), (ROWS_1X1, 0, 1, 70, 33, 96, 832, 1, 0, 1), (ROWS_1X1, 0, 3, 33, 33, 96, 768, 3, 1, 1),
    (ROWS_1X1, 0, 1, 40, 40, 64, 3072, 0, 1, 4), (ROWS_2X1, 0, 2, 97, 65, 96, 832, 2, 0, 1), (ROWS_2X1, 0, 1, 70, 70, 64, 1536, 0, 1, 2),
    (ROWS_2X2, 0, 1, 97, 97, 96, 128, 0, 0, 1), (ROWS_2X2, 0, 2, 65, 40, 160, 192, 1, 0, 1),
    (K2, 1, 1, 33, 33, 160, 640, 0, 1, 1), (K2, 2, 2, 97, 70, 288, 640, 1, 0, 1), (K2, 3, 1, 200, 193, 96, 896, 0, 0, 1), (K2, 4, 3, 290, 257, 160, 768, 0, 1, 1),
    (K2, 4, 1, 130, 130, 160, 3072, 0, 1, 2), (K2, 1, 3, 1024, 1010, 512, 640, 0, 0, 1),
    (PAIR, 1, 2, 65, 33, 288, 320, 2, 0, 1), (PAIR, 2, 1, 97, 97, 544, 448, 0, 1, 1), (PAIR, 3, 2, 200, 193, 96, 320, 1, 0, 1), (PAIR, 4, 1, 290, 257, 288, 384, 0, 0, 1),
    (PAIR, 4, 1, 130, 130, 288, 1536, 0, 1, 4), (PAIR, 1, 10, 1024, 1001, 512, 320, 1, 0, 1),
    (TALL, 5, 1, 170, 161, 288, 384, 0, 1, 1), (TALL, 6, 2, 390, 353, 96, 512, 0, 0, 1), (TALL, 7, 1, 230, 225, 288, 384, 0, 1, 1), (TALL, 8, 1, 300, 257, 544, 640, 0, 0, 1),
    (TALL, 5, 8, 1312, 1300, 1024, 384, 0, 1, 1), (TALL, 5, 3, 170, 161, 288, 384, 0, 1, 1), (TALL, 6, 3, 390, 353, 96, 640, 0, 1, 1), (TALL, 6, 1, 200, 190, 544, 384, 0, 0, 1),
    (0, 0, 3, 512, 290, 768, 3072, 0, 1, 1), (0, 0, 3, 384, 290, 768, 3072, 0, 1, 1), (0, 0, 2, 1376, 700, 768, 768, 0, 1, 1), (0, 0, 1, 2016, 1100, 768, 3072, 0, 1, 1),
    (0, 0, 12, 270, 257, 1024, 448, 3, 1, 1), (0, 0, 12, 288, 33, 1024, 256, 3, 1, 1), (0, 0, 1, 300, 171, 768, 768, 0, 0, 1), (0, 0, 8, 300, 171, 768, 768, 0, 1, 1), (0, 0, 1, 2080, 1900, 2304, 768, 1, 0, 1),
])
def test_panel_linear_forms(form, height, problems, M, rows, N, K, act, f32, splits):
    print(f"panel linear: form {form} height {height}, {problems} x {rows}/{M} x {N} x {K}, act {act}, f32 {f32}, splits {splits}", flush=True)
    from scipy.special import erf
    rng = np.random.default_rng(M + N + K + height)
    A, W = bf16(rng.standard_normal((problems, M, K))), bf16(rng.standard_normal((problems, N, K)) / K**0.5)
    b = rng.standard_normal((problems, N)).astype(np.float32)
    A[:, rows:] = np.nan
    pa, pw = torch.stack([panels(a) for a in A]), torch.stack([panels(w) for w in W])
    pc = torch.stack([nan_panels(M, N, torch.float32 if f32 else torch.bfloat16) for _ in range(problems * splits)])
    bias = torch.zeros((problems, (N + 63) // 64 * 64), device="cuda")           # a problem's bias starts at a multiple of 256 bytes
    bias[:, :N] = dev(b)
    size = lambda t: t[0].numel() * t.element_size()
    mt.op_panel_linear(pa, pw, bias, pc, M=M, N=N, K=K, rows=dev(np.array([rows], np.int32)), problems=problems, stride_A=size(pa), stride_W=size(pw),
                       stride_bias=size(bias), stride_C=size(pc) * splits, split_stride=pc[0].numel(), splits=splits, act_kind=act, out_f32=f32, form=form,
                       height=height)
    for i in range(problems):
        got = sum(rows_of(pc[i * splits + s])[:rows] for s in range(splits))
        a, w = A[i, :rows], W[i]
        x = a @ w.T + b[i]
        bound = K * 2.0**-24 * (np.abs(a) @ np.abs(w).T + np.abs(b[i])) + 1e-30
        if act in (1, 2):
            want = x * 0.5 * (1 + (erf(x / 2**0.5) if act == 1 else np.tanh((2 / np.pi)**0.5 * (x + 0.044715 * x**3))))
            bound = 1.13 * bound + 3e-5
        else:
            want, bound = (np.tanh(x), bound + 2.0**-21) if act == 3 else (x, bound)
        if not f32:
            bound = 1.01 * (bound + 2.0**-8 * np.abs(want))
        err = np.abs(got - want)
        assert (err <= bound).all(), (i, float((err / bound).max()))
    untouched = (rows + 31) // 32
    assert torch.isnan(pc[:, untouched:]).all()


# Poolers add K up in four quarters at any size (of the forms that take tanh): the same bits as one block per workgroup, on both sides of that form's line and
# far beyond it, K of both model widths.
@pytest.mark.parametrize("problems,M,N,K", [(3, 384, 1024, 2048), (4, 300, 1024, 2048), (21, 272, 768, 1536), (24, 128, 1024, 2048), (32, 33, 768, 1536)])
def test_panel_linear_poolers_sum_in_one_order(problems, M, N, K):
    print(f"panel linear, poolers: {problems} x {M} x {N} x {K}", flush=True)
    rng = np.random.default_rng(problems + M)
    pa = torch.stack([panels(rng.standard_normal((M, K)).astype(np.float32)) for _ in range(problems)])
    pw = torch.stack([panels(rng.standard_normal((N, K)).astype(np.float32) / K**0.5) for _ in range(problems)])
    bias = dev(rng.standard_normal((problems, N)).astype(np.float32))
    size = lambda t: t[0].numel() * t.element_size()
    auto, one = (mt.op_panel_linear(pa, pw, bias, torch.stack([nan_panels(M, N, torch.float32) for _ in range(problems)]), M=M, N=N, K=K, problems=problems, stride_A=size(pa),
                                    stride_W=size(pw), stride_bias=size(bias), stride_C=pa.shape[1] * 32 * N * 4, act_kind=3, out_f32=1, form=form) for form in (0, ROWS_1X1))
    for i in range(problems):
        assert np.array_equal(rows_of(auto[i])[:M], rows_of(one[i])[:M]), i


# the values' columns, stored transposed for the attention: the same numbers at other places
@pytest.mark.parametrize("form,height,M,K", [(ROWS_1X1, 0, 40, 64), (ROWS_2X1, 0, 70, 832), (ROWS_2X2, 0, 97, 128), (K2, 3, 97, 640), (PAIR, 4, 160, 384), (PAIR, 1, 33, 320), (TALL, 5, 200, 384)])
def test_panel_linear_transposed_columns(form, height, M, K):
    print(f"panel linear, transposed columns: form {form} height {height}, {M} x {K}", flush=True)
    rng, N, first = np.random.default_rng(M + K), 192, 128
    A, W, b = panels(rng.standard_normal((M, K))), panels(rng.standard_normal((N, K)) / K**0.5), dev(rng.standard_normal(N).astype(np.float32))
    full = (M + 31) // 32 * 32
    A[-1, :, M % 32 or 32:] = 0                                                  # (every row of the last panel is compared)
    plain, moved = (mt.op_panel_linear(A, W, b, nan_panels(M, N, torch.bfloat16), M=full, N=N, K=K, form=form, height=height, transposed_from=t) for t in (0, first))
    assert np.array_equal(rows_of(moved), transposed_columns(rows_of(plain), first))


@pytest.mark.parametrize("heads,B", [(3, 37), (12, 200), (12, 257), (8, 1200)])               # one block per workgroup, two by two, two by one
def test_panel_linear_parts(heads, B):
    """Problems of equal parts with operands of their own, as the contexts of the heads, over 2 problems."""
    print(f"panel linear, parts: {heads} heads, {B} rows", flush=True)
    rng, H = np.random.default_rng(5), heads * 64
    x, W, b = bf16(rng.standard_normal((2, heads, B, H))), bf16(rng.standard_normal((2, H, H)) / H**0.5), rng.standard_normal((2, H)).astype(np.float32)
    px, pw = torch.stack([panels(v) for p in x for v in p]), torch.stack([panels(w) for w in W])
    pc = torch.stack([nan_panels(B, H, torch.bfloat16) for _ in range(2)])
    bias = torch.zeros((2, max(256, H)), device="cuda")
    bias[:, :H] = dev(b)
    size = lambda t: t[0].numel() * t.element_size()
    mt.op_panel_linear(px, pw, bias, pc, M=B, N=64, K=H, ldc=H, problems=2, subs=heads, stride_A=size(px) * heads, stride_W=size(pw), stride_bias=size(bias),
                       stride_C=size(pc), sub_A=size(px), sub_W=64 * H * 2, sub_bias=256, sub_C=8 * 512)
    for p in range(2):
        for h in range(heads):
            w = W[p, h * 64:h * 64 + 64]
            want = x[p, h] @ w.T + b[p, h * 64:h * 64 + 64]
            bound = 1.01 * (2.0**-8 * np.abs(want) + H * 2.0**-24 * (np.abs(x[p, h]) @ np.abs(w).T + 3))
            assert (np.abs(rows_of(pc[p])[:B, h * 64:h * 64 + 64] - want) <= bound).all(), (p, h)


# heights, K and widths that no kernel takes are refused
@pytest.mark.parametrize("bad", [dict(form=ROWS_1X1, height=1), dict(form=K2, K=576), dict(form=K2, height=5), dict(form=K2, K=640, height=4), dict(form=PAIR, K=256),
                                 dict(form=PAIR, K=320, height=4), dict(form=TALL, K=320), dict(form=TALL, height=4), dict(form=TALL, act_kind=1), dict(form=TALL, height=9),
                                 dict(form=PAIR, subs=2), dict(N=48), dict(K=96), dict(transposed_from=32), dict(transposed_from=64, out_f32=1), dict(splits=2), dict(ldc=32), dict(form=7)])
def test_panel_linear_refuses(bad):
    t = torch.zeros(1 << 18, dtype=torch.bfloat16, device="cuda")
    with pytest.raises(mt.MTError) as e:
        mt.op_panel_linear(t, t, None, t, **{"M": 64, "N": 64, "K": 768, **bad})
    assert e.value.code == mt.MT_ERR_SHAPE


# Attention on the panels, each launch shape: one workgroup per sequence and head with up to four query panels, the fifth panel with and without
# a wavefront of its own, several workgroups per sequence, two wavefronts per query panel.  Rows of no sequence hold NaN in every column and are
# not written.  `late`: scores rise by 20 to the last key, so the running maximum follows panel after panel and the two halves of a query
# panel's keys meet with different maxima.  Bound: weights but the largest, which is 1, are rounded to bfloat16 before they are multiplied and
# before they are added up, so a rounding moves the context by 2^-8 p |v - context|; 2^-14 sum p |v| for scores summed in float32, as above;
# the result rounds once.
@pytest.mark.parametrize("heads,lens,seq,late", [
    (1, [1, 2, 31, 32, 33], 33, False), (3, [64, 65, 63, 96], 96, True), (2, [128, 127, 97, 3], 128, True), (16, [128] + [97, 128, 66] * 21, 128, True),
    (2, [200, 161, 5], 200, True), (5, [289, 288, 257, 4], 289, True), (1, [512, 509, 1], 512, False), (16, [289, 270, 33] * 4, 289, True), (2, [70, 64], 40, False),
    (2, [289, 1, 257, 33, 64] * 3, 289, True), (3, [51, 32, 1, 50, 33] * 17, 51, True), (3, [50, 32, 1, 49, 33] * 17, 50, False),      # many sequences: one wavefront a query panel and two, on both sides of the rule
])
def test_attention_panels(heads, lens, seq, late):
    print(f"attention: {heads} heads, {len(lens)} sequences of up to {max(lens)}, bound {seq}, late {late}", flush=True)
    H, rng = 64 * heads, np.random.default_rng(heads + seq)
    row0, rows = ragged_rows(lens, 5, rng)
    full = (rows + 31) // 32 * 32
    x = np.full((full, 3, heads, 64), np.nan)
    for r, n in zip(row0, lens):
        x[r:r + n] = rng.standard_normal((n, 3, heads, 64)) * np.array([2.0, 1.0, 1.0])[:, None, None]
        if late:
            u = rng.standard_normal((heads, 64))
            u /= np.linalg.norm(u, axis=1, keepdims=True)
            x[r:r + n, 0] += 5.0 * u
            x[r:r + n, 1] += 32.0 * u * np.linspace(0.0, 1.0, n)[:, None, None]
    x = bf16(x)
    qkv = panels(transposed_columns(x.reshape(full, 3 * H), 2 * H))
    got = rows_of(mt.op_panel_attention(qkv, dev(row0), dev(np.array(lens, np.int32)), len(lens), seq, heads)).reshape(full, heads, 64)
    worst, written = 0.0, np.zeros(full, bool)
    for r, n in zip(row0, np.minimum(lens, seq)):
        q, k, v = (x[r:r + n, i].transpose(1, 0, 2) for i in range(3))
        s = q @ k.transpose(0, 2, 1) / 8
        p = np.exp(s - s.max(2, keepdims=True))
        p /= p.sum(2, keepdims=True)
        want = p @ v
        rounded = np.where(p == p.max(2, keepdims=True), 0.0, p)
        spread = np.stack([(dev(rounded[a])[:, :, None] * (dev(v[a]) - dev(want[a])[:, None]).abs()).sum(1).cpu().numpy() for a in range(heads)])
        bound = 1.01 * 2.0**-8 * (np.abs(want) + spread) + 2.0**-14 * (p @ np.abs(v))
        worst = max(worst, (np.abs(got[r:r + n].transpose(1, 0, 2) - want) / bound).max())
        written[r:r + n] = True
    print(f"  {worst:.3f} of the bound, scores of the last sequence up to {np.abs(s).max():.1f}", flush=True)
    assert worst <= 1.0 and np.isnan(got[~written]).all()


# LayerNorm on the panels: remainders of the rows, each number of partial results, the three forms (up to 2048 rows, up to 16384, more), a residual
# that is looked up by row, the [hi | lo] operand.  Bound: float32 sums and a square root (2^-18 of the terms); the operand is the state rounded once, 2^-8
# of the value, and as [hi | lo] twice, 2^-16.
@pytest.mark.parametrize("M,rows,H,parts,look_up,split", [
    (1, 1, 64, 1, False, False), (33, 30, 768, 4, False, False), (70, 70, 832, 2, True, True), (2080, 2049, 64, 2, False, False), (2100, 2051, 1024, 4, False, False),
    (37, 37, 1024, 1, True, True), (2052, 2052, 128, 1, True, False), (64, 35, 320, 4, False, True),
    (2080, 2070, 768, 1, True, True), (16384, 16383, 256, 1, False, True), (16417, 16401, 768, 1, True, False), (16385, 16385, 256, 2, False, True),
    (16400, 16390, 384, 4, True, True),
])
def test_layernorm_panels(M, rows, H, parts, look_up, split):
    print(f"layernorm: {rows}/{M} x {H}, {parts} parts, look-up {look_up}, split {split}", flush=True)
    rng = np.random.default_rng(M + H)
    x = rng.standard_normal((parts, M, H)).astype(np.float32)
    x[:, rows:] = np.nan
    res_rows = 50 if look_up else M
    res = rng.standard_normal((res_rows, H)).astype(np.float32)
    index = rng.integers(0, res_rows, M).astype(np.int32)
    gamma, beta = 1 + 0.2 * rng.standard_normal(H).astype(np.float32), rng.standard_normal(H).astype(np.float32)
    of, ob = mt.op_panel_layernorm(torch.stack([panels(p, torch.float32) for p in x]), panels(res, torch.float32), dev(gamma), dev(beta), 1e-12, M, H,
                                   res_row=dev(index) if look_up else None, res_rows=res_rows if look_up else 0, split=split, rows=dev(np.array([rows], np.int32)))
    v = x[:, :rows].astype(np.float64).sum(0) + (res[index[:rows]] if look_up else res[:rows])
    n = (v - v.mean(1, keepdims=True)) / np.sqrt(v.var(1, keepdims=True) + 1e-12)
    want = gamma * n + beta
    got, operand = rows_of(of), rows_of(ob)
    assert (np.abs(got[:rows] - want) <= 2.0**-18 * (np.abs(gamma) * (1 + np.abs(n)) + np.abs(beta))).all()
    if split:
        operand = operand[:, :H] + operand[:, H:]
    assert (np.abs(operand[:rows] - got[:rows]) <= (2.0**-16 if split else 2.0**-8) * np.abs(got[:rows])).all()
    assert np.isnan(got[rows:]).all() and np.isnan(operand[rows:]).all()


@pytest.mark.parametrize("H,parts", [(64, 1), (128, 2), (192, 1), (256, 4), (384, 1), (640, 2), (704, 1), (768, 1), (768, 4), (896, 1), (1024, 2)])
def test_layernorm_panels_few_and_many_rows_give_the_same_bits(H, parts):
    """A launch of up to 2048 rows deals a row's columns out to several wavefronts (H / 64 a multiple of 4 or 2) before it knows the row count, one of up to
    16384 after, a larger one not."""
    rows = 1997
    print(f"layernorm, few and many rows: {rows} x {H}, {parts} parts", flush=True)
    rng = np.random.default_rng(H + parts)
    gamma, beta = 1 + 0.2 * rng.standard_normal(H).astype(np.float32), rng.standard_normal(H).astype(np.float32)
    x = (rng.standard_normal((parts, rows, H)) + 3 * rng.standard_normal((1, rows, 1))).astype(np.float32)
    res = rng.standard_normal((rows, H)).astype(np.float32)
    got = []
    for M in (2048, 2080, 16384, 16416):
        xm, rm = np.full((parts, M, H), np.nan, np.float32), np.full((M, H), np.nan, np.float32)
        xm[:, :rows], rm[:rows] = x, res
        of, ob = mt.op_panel_layernorm(torch.stack([panels(p, torch.float32) for p in xm]), panels(rm, torch.float32), dev(gamma), dev(beta), 1e-12, M, H,
                                       rows=dev(np.array([rows], np.int32)))
        got.append((rows_of(of)[:rows], rows_of(ob)[:rows]))
    assert all((got[0][0] == f).all() and (got[0][1] == b).all() for f, b in got[1:])
    v = x.astype(np.float64).sum(0) + res
    n = (v - v.mean(1, keepdims=True)) / np.sqrt(v.var(1, keepdims=True) + 1e-12)
    # the sums of up to 5 float32 values round at 2^-24 of values up to 4 standard deviations of the row's offset
    bound = 2.0**-18 * (np.abs(gamma) * (1 + np.abs(n)) + np.abs(beta)) * np.maximum(1, np.abs(v).max(1, keepdims=True) / v.std(1, keepdims=True))
    assert (np.abs(got[0][0] - (gamma * n + beta)) <= bound).all()


@pytest.mark.parametrize("M", [1500, 9000, 16500])
@pytest.mark.parametrize("H", [128, 192, 256, 384, 640, 768, 896, 1024])
def test_layernorm_panels_error_of_rows_far_from_zero(H, M):
    """Rows about 5: the error is that of the mean, whose parts are independent.  Its own rounding (values from 4 to 8 lie 2^-21 apart), and the last few
    additions of each share's sum, sqrt(1 + 1/2 + 1/4 + ..) roundings at the sum's size (a quarter of the columns where that is a multiple of 64, or
    half, or all); the result rounds at 2^-24 of itself.  A seventh more for the squares and the many smaller additions."""
    print(f"layernorm of rows about 5: {M} x {H}", flush=True)
    rng = np.random.default_rng(H + M)
    v = (rng.standard_normal((M, H)) + 5).astype(np.float32)
    of, _ = mt.op_panel_layernorm(panels(np.zeros_like(v), torch.float32)[None], panels(v, torch.float32), dev(np.ones(H, np.float32)), dev(np.zeros(H, np.float32)),
                                  1e-12, M, H)
    w = v.astype(np.float64)
    want = (w - w.mean(1, keepdims=True)) / w.std(1, keepdims=True)
    err = np.sqrt(((rows_of(of)[:M] - want)**2).mean())
    shares = 4 if H % 256 == 0 else 2 if H % 128 == 0 else 1
    cols = H // shares
    rounding = np.array([2.0**-21, np.sqrt(2.0) * np.spacing(np.float32(5 * cols)) / cols / np.sqrt(shares), 2.0**-23]) / np.sqrt(12)
    assert err <= 8 / 7 * np.sqrt((rounding**2).sum()), (err, rounding)


@pytest.mark.parametrize("mean", [0.0, 1e2, 1e4, 1e6, 4e6])
@pytest.mark.parametrize("H", [128, 384, 768, 896, 1024])
def test_layernorm_panels_error_against_one_float32_sum_over_the_row(H, mean):
    """Shares of a row put together are to be no further from float64 than one float32 sum over it (16 lanes, their values one after another, then pairwise),
    however far the row is from zero.  Two such orders differ by a few percent over 3000 rows: a tenth is allowed."""
    print(f"layernorm against one sum: rows about {mean:g}, {H} columns", flush=True)
    rng = np.random.default_rng(int(H + mean))
    v = (rng.standard_normal((3000, H)) + mean).astype(np.float32)
    w = v.astype(np.float64)
    want = (w - w.mean(1, keepdims=True)) / w.std(1, keepdims=True)

    def one_sum(x):
        x = x.reshape(len(x), H // 64, 16, 4)
        s = np.zeros((len(x), 16), np.float32)
        for i in range(H // 64):
            s = s + ((x[:, i, :, 0] + x[:, i, :, 1]) + (x[:, i, :, 2] + x[:, i, :, 3]))
        while s.shape[1] > 1:
            s = s[:, ::2] + s[:, 1::2]
        return s / np.float32(H)

    d = v - one_sum(v)
    ref = d * (np.float32(1) / np.sqrt(one_sum(d * d)))
    of, _ = mt.op_panel_layernorm(panels(np.zeros_like(v), torch.float32)[None], panels(v, torch.float32), dev(np.ones(H, np.float32)), dev(np.zeros(H, np.float32)),
                                  1e-12, len(v), H)
    err, bar = (np.sqrt(((x - want)**2).mean()) for x in (rows_of(of)[:len(v)], ref.astype(np.float64)))
    print(f"  {err:.3g}, one sum {bar:.3g}", flush=True)
    assert err <= 1.1 * bar


@pytest.mark.parametrize("batch,seq", [(9, 5), (60, 4), (70, 30)])
def test_heads_of_many_unequal_tasks(batch, seq):
    """18 tasks of 1 to 50 classes: the classifier's plain grid (9 sequences) and its list of classes; token heads of few and many positions; the row map in
    one launch (up to 2048 positions) and in two; first-token rows read in place (up to 8 sequences wanted) and gathered."""
    classes = (2, 3, 5, 8, 12, 1, 4, 30, 2, 6, 3, 2, 16, 4, 2, 9, 50, 7)
    tasks = tuple(ms.TaskSpec(1, 1 + t % 2, c, token_level=t in (7, 12)) for t, c in enumerate(classes))
    spec = ms.MTSpec("heads", vocab=300, hidden=256, heads=4, ffn=256, max_pos=64, n_trunk_layers=1, tasks=tasks, precision="bf16", batch=batch, seq=seq,
                     len_lo=1, len_hi=seq, input_seed=3)
    print(f"heads of 18 tasks: {batch} x {seq}", flush=True)
    model, (trunk, params) = mt.load_synthetic(spec, keep_params=True, std=0.05)
    ids, mask, _ = ms.make_inputs(spec)
    got, tok = model.forward_tokens(dev(ids), dev(mask))
    got, tok = got.cpu().numpy(), tok.cpu().numpy()
    rows = np.arange(batch)[-7:]
    ref, ref_tok = oracle.Oracle(spec, trunk, params).mt_forward(ids[rows], mask[rows], want_tokens=True)
    real = mask[rows].astype(bool)
    scale = max(1.0, np.abs(ref).max(), np.abs(ref_tok[real]).max())
    assert np.abs(got[rows] - ref).max() <= 2e-2 * scale and np.abs(tok[rows][real] - ref_tok[real]).max() <= 2e-2 * scale
    assert (tok[~mask.astype(bool)] == 0).all()
    for t, task in enumerate(tasks):             # alone, a task's classes are few enough for the plain grid; all of them go through the list from 60 sequences on
        if not task.token_level:
            at = slice(spec.logit_offset(t), spec.logit_offset(t) + task.n_classes)
            one = model.forward(dev(ids), dev(mask), task_mask=[u == t for u in range(len(tasks))]).cpu().numpy()
            assert np.array_equal(one[:, at], got[:, at]), t
    few = model.forward_tokens(dev(ids[:5].copy()), dev(mask[:5].copy()))[0].cpu().numpy()      # five sequences: in place
    assert np.abs(few - got[:5]).max() <= 1e-2 * scale
    model.close()
