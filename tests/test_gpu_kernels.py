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


# one row, full and one-over row blocks of the few-row kernel, of both tiles of the matrix-core kernel and of its large grid
@pytest.mark.parametrize("M,N,K", [(1, 4, 64), (32, 100, 192), (33, 68, 64), (65, 64, 128), (31, 32, 832), (2113, 2052, 64)])
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


# bfloat16 kernels of the panel layout through a whole model: ragged rows, both contractions' halves that a launch rule can choose.
# Bound on the logits: bfloat16 operands (2^-9 each) through three layers give at most 2e-2 at logits of order 1.
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
    model, (trunk, tasks) = mt.load_synthetic(spec, keep_params=True, std=0.03)
    ids, mask, _ = ms.make_inputs(spec)
    got = model.forward(dev(ids), dev(mask)).cpu().numpy()
    pick = np.unique(np.linspace(0, batch - 1, 7).astype(int))
    ref = oracle.Oracle(spec, trunk, tasks).mt_forward(ids[pick], mask[pick])
    err = np.abs(got[pick] - ref).max()
    print(f"  max |dlogit| {err:.3g}, logits up to {np.abs(ref).max():.3g}", flush=True)
    assert np.isfinite(got).all() and err <= 2e-2
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
                                             (12, [128, 127, 70], True), (16, [1, 257, 64], True)])
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
