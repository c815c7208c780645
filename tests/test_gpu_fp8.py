"""The FP8 variants (MT_FP8_FFN: the two feed-forward contractions of every all-rows layer in OCP E4M3; MT_FP8_LAYER: the
query/key/value and attention output projections too) against the oracle.

What each side consumes: the generator snaps the feed-forward matrices to the E4M3 grid under their power-of-two
storage scale (and everything else to the bfloat16 grid), so the float32 oracle and the library hold identical
weights; what the tolerance has to cover is the rounding of the two feed-forward OPERANDS (LayerNorm output, GELU
output) to E4M3, relative step 2^-4 against bfloat16's 2^-9 on the other operands.

Tolerance.  The bf16 path's measured error is about 2e-3 for a bar of 2e-2.  Two of a layer's four contraction
operands are now 32 times coarser, and they belong to the block whose output is a fraction (about a third at these
weights) of the residual stream it is added to: expected error about 32 * 0.5 * 2e-3 = 3e-2.  Bar: max |delta logit|
<= 8e-2 (four times the bf16 bar), and identical argmax on every (sequence, task) pair whose oracle margin exceeds
twice that.  MT_FP8_LAYER rounds all four contraction operands of a layer to E4M3 (the layer input, the attention
context, the LayerNorm output, the GELU output).  Independent roundings add in quadrature, so twice as many coarse
operands raise the expectation by sqrt(2), to about 4.2e-2: the same bar of 8e-2 is kept for both (relative to the
largest logit when that exceeds 1).
"""
import dataclasses
import sys

import numpy as np
import pytest

import mt_synth as ms
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2107_05377_amd as mt  # noqa: E402

TOL = {"fp8": 8e-2, "fp8_all": 8e-2}


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def e4m3_values(codes):
    return torch.from_numpy(np.ascontiguousarray(codes)).view(torch.float8_e4m3fn).float().numpy()


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    mt.lib()


@pytest.mark.parametrize("M,N,K", [(300, 392, 192), (2318, 768, 3072), (1560, 1300, 320)])
def test_fp8_contraction_vs_oracle(M, N, K):
    """Operands exactly representable in E4M3, so the oracle's float64 dot products are the exact result and only the
    float32 accumulation order differs; all three output kinds, ragged edges, a canary beyond them."""
    if K % 64:
        K = K // 64 * 64
    say(f"fp8 contraction {M}x{N}x{K}")
    rng = np.random.default_rng(M + N)
    a_codes = mt.e4m3_quantize(rng.standard_normal((M, K)).astype(np.float32) * 100)[1]          # scale 1 or 2: any codes do
    w_scale, w_codes = mt.e4m3_quantize((rng.standard_normal((N, K)) * 0.02).astype(np.float32))
    A, W = e4m3_values(a_codes), e4m3_values(w_codes) / np.float32(w_scale)
    bias = rng.standard_normal(N).astype(np.float32)
    res = rng.standard_normal((M, N)).astype(np.float32)
    ref = oracle.linear(A, W, bias)
    scale = max(1.0, float(np.abs(ref).max()))
    dA, dW, db, dr = dev(a_codes), dev(w_codes), dev(bias), dev(res)
    out = mt.op_linear_fp8(dA, dW, 1.0 / w_scale, db, None, 0, 1).cpu().numpy()
    assert np.abs(out - ref).max() <= 2e-4 * scale
    out = mt.op_linear_fp8(dA, dW, 1.0 / w_scale, db, dr, 0, 1).cpu().numpy()
    assert np.abs(out - (ref.astype(np.float64) + res)).max() <= 2e-4 * scale
    out = mt.op_linear_fp8(dA, dW, 1.0 / w_scale, db, None, 1, 0).float().cpu().numpy()
    g = oracle.gelu(ref)
    assert np.abs(out - g).max() <= 2 ** -8 * np.abs(g).max() + 1e-3
    # E4M3 output: the nearest code of the exact value, or a neighbour where the float32 value sits at a rounding boundary
    out8 = e4m3_values(mt.op_linear_fp8(dA, dW, 1.0 / w_scale, db, None, 1, 2, 0.5).cpu().numpy())
    want = np.clip(g * 0.5, -448, 448)
    assert np.all(np.abs(out8 - want) <= 2.0 ** -4 * np.abs(want) + 2.0 ** -9 + 1e-3)
    assert np.abs(out8 - want).mean() <= 2.0 ** -5 * np.abs(want).mean() + 2.0 ** -10
    big = torch.full((M + 1, N + 8), 7.0, dtype=torch.float32, device="cuda")
    rc = mt.lib().mt_op_linear_fp8(dA.data_ptr(), K, dW.data_ptr(), 1.0 / w_scale, db.data_ptr(), None, big.data_ptr(), N + 8, M, N, K, 0, 1, 1.0, None)
    assert rc == mt.MT_OK
    o = big.cpu().numpy()
    assert np.abs(o[:M, :N] - ref).max() <= 2e-4 * scale and (o[M] == 7.0).all() and (o[:, N:] == 7.0).all()


ROWS_1X1, PAIR = 1, 5


# Every form of the panel contraction on E4M3 operands and every tile height at remainders of rows, columns and K: the same bits as the row-major
# kernel, which test_fp8_contraction_vs_oracle holds to the oracle.
@pytest.mark.parametrize("form,height,problems,M,rows,N,K,act,out,w_std", [
    (ROWS_1X1, 0, 1, 1, 1, 32, 256, 0, 1, 0.02), (ROWS_1X1, 0, 2, 70, 33, 192, 3328, 1, 2, 0.02), (ROWS_1X1, 0, 1, 40, 40, 64, 768, 0, 0, 1e-9),
    (ROWS_1X1, 0, 2, 97, 65, 64, 896, 2, 2, 0.02), (ROWS_1X1, 0, 1, 70, 70, 160, 1536, 0, 1, 50.0), (ROWS_1X1, 0, 3, 33, 33, 96, 384, 0, 0, 0.02),
    (PAIR, 1, 2, 65, 33, 320, 768, 2, 2, 0.02), (PAIR, 2, 1, 97, 97, 544, 1408, 0, 1, 0.02), (PAIR, 4, 1, 290, 257, 288, 768, 0, 0, 0.02),
    (PAIR, 4, 2, 1024, 1001, 512, 1024, 1, 2, 0.02), (PAIR, 1, 3, 290, 257, 96, 640, 0, 0, 0.02),
    (0, 0, 1, 300, 171, 768, 768, 0, 1, 0.02), (0, 0, 8, 300, 171, 768, 3072, 0, 1, 0.02), (0, 0, 1, 2080, 1900, 3072, 768, 1, 2, 0.02),
])
def test_fp8_panel_linear_forms(form, height, problems, M, rows, N, K, act, out, w_std):
    say(f"fp8 panel linear: form {form} height {height}, {problems} x {rows}/{M} x {N} x {K}, act {act}, out {out}, weights {w_std}")
    rng = np.random.default_rng(M + N + K + height)
    bias = torch.zeros((problems, (N + 63) // 64 * 64), device="cuda")
    pa, pw, want = [], [], []
    for i in range(problems):
        a = mt.e4m3_quantize((rng.standard_normal((M, K)) * 200).astype(np.float32))[1]
        a[rows:] = 0x7F                                                          # NaN
        scale, w = mt.e4m3_quantize((rng.standard_normal((N, K)) * w_std).astype(np.float32))
        bias[i, :N] = dev((rng.standard_normal(N) * w_std).astype(np.float32))
        pa.append(mt.to_panels_e4m3(dev(a).view(torch.float8_e4m3fn)))
        slot = torch.full((256,), 127 - int(np.log2(scale)), dtype=torch.uint8, device="cuda")
        pw.append(torch.cat([slot, mt.to_panels_e4m3(dev(w).view(torch.float8_e4m3fn)).flatten()]))
        want.append(mt.op_linear_fp8(dev(a[:rows]), dev(w), 1.0 / scale, bias[i, :N].contiguous(), None, act, out).cpu())
    pa, pw = torch.stack(pa), torch.stack(pw)
    if out == 2:
        pc = torch.full((problems, (M + 31) // 32, N // 16, 32, 16), 0x7F, dtype=torch.uint8, device="cuda")
    else:
        pc = torch.full((problems, (M + 31) // 32, N // 8, 32, 8), float("nan"), dtype=torch.float32 if out else torch.bfloat16, device="cuda")
    size = lambda t: t[0].numel() * t.element_size()
    mt.op_panel_linear(pa, pw.flatten()[256:], bias, pc, fp8=True, M=M, N=N, K=K, rows=dev(np.array([rows], np.int32)), problems=problems, stride_A=size(pa),
                       stride_W=size(pw), stride_bias=size(bias), stride_C=size(pc), act_kind=act, out_f32=out, form=form, height=height)
    for i in range(problems):
        got = (mt.from_panels_e4m3(pc[i]).view(torch.uint8) if out == 2 else mt.from_panels(pc[i]))[:rows].cpu()
        assert torch.equal(got, want[i].view(got.dtype)), (i, int((got != want[i].view(got.dtype)).sum()))
    untouched = (rows + 31) // 32
    assert (pc[:, untouched:] == 0x7F).all() if out == 2 else torch.isnan(pc[:, untouched:]).all()


def to_e4m3(x):
    """E4M3 codes of a CPU tensor, saturating."""
    return x.float().clamp(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8)


# LayerNorm of the layers with E4M3 operands: the row-major kernel's bits (test_layernorm_vs_oracle holds that one to the oracle), whose E4M3 copy is of
# the bf16 values (a layer's output) or of the float32 ones (between the two halves of a layer).  Remainders of the rows, values that saturate.
@pytest.mark.parametrize("M,rows,H", [(1, 1, 256), (37, 33, 768), (300, 290, 1024), (2100, 2049, 512), (16500, 16401, 256)])
@pytest.mark.parametrize("want_b,want_q", [(True, True), (True, False), (False, True)])
def test_fp8_panel_layernorm_gives_the_row_major_bits(M, rows, H, want_b, want_q):
    say(f"fp8 panel layernorm: {rows}/{M} x {H}, bf16 {want_b}, E4M3 {want_q}")
    rng = np.random.default_rng(M + H)
    x, r = rng.standard_normal((2, M, H)).astype(np.float32)
    x += 2 * rng.standard_normal((M, 1)).astype(np.float32)
    x[rows:] = np.nan
    gamma, beta = 1 + 0.5 * rng.standard_normal(H).astype(np.float32), rng.standard_normal(H).astype(np.float32)
    gamma[::7] *= 200
    of, ob, oq = mt.op_panel_layernorm_fp8(mt.to_panels(dev(x), torch.float32), mt.to_panels(dev(r), torch.float32), dev(gamma), dev(beta), 1e-12, M, H, want_b, want_q,
                                           rows=dev(np.array([rows], np.int32)))
    wf, wb = mt.op_layernorm(dev(x[:rows] + r[:rows]), dev(gamma), dev(beta), 1e-12, want_bf16=True)
    assert torch.equal(mt.from_panels(of)[:rows], wf)
    assert not want_b or torch.equal(mt.from_panels(ob)[:rows].view(torch.int16), wb.view(torch.int16))
    if want_q:
        got, want = mt.from_panels_e4m3(oq).view(torch.uint8)[:rows].cpu(), to_e4m3((wb if want_b else wf).cpu())
        assert torch.equal(got, want), int((got != want).sum())
        assert (got & 0x7F).max() == 0x7E                                        # something saturates
        assert (oq[(rows + 31) // 32:] == 0x7F).all()


# The attention with an E4M3 context on panels: the row-major kernel's bits, and those are roundings of the bf16 form's values (which
# test_attention_bf16_vs_oracle holds to the oracle).  Sequences of part of a panel, of several, of more than one block of queries; rows of none hold NaN.
@pytest.mark.parametrize("heads,lens", [(4, [1, 33, 300]), (12, [128, 127, 2, 31]), (16, [65, 200]), (1, [32] * 9)])
def test_fp8_panel_attention_gives_the_row_major_bits(heads, lens):
    say(f"fp8 panel attention: {heads} heads, {lens}")
    rng, H = np.random.default_rng(heads), 64 * heads
    row0 = np.cumsum([3] + [n + 5 for n in lens[:-1]]).astype(np.int32)
    rows = int(row0[-1] + lens[-1] + 7)
    real = np.zeros(rows, bool)
    for a, n in zip(row0, lens):
        real[a:a + n] = True
    qkv = torch.full((rows, 3 * H), float("nan"), dtype=torch.bfloat16)
    qkv[torch.from_numpy(real)] = torch.from_numpy(rng.standard_normal((int(real.sum()), 3 * H)).astype(np.float32) * 2).to(torch.bfloat16)
    start, length, seq = dev(row0), dev(np.array(lens, np.int32)), max(lens)
    flat = mt.op_attention_fp8(qkv.cuda(), torch.full((rows, H), 0x7F, dtype=torch.uint8, device="cuda"), start, length, len(lens), seq, heads, False).cpu()
    ctx = torch.full(((rows + 31) // 32, H // 16, 32, 16), 0x7F, dtype=torch.uint8, device="cuda")
    mt.op_attention_fp8(mt.to_panels(qkv.cuda(), torch.bfloat16), ctx, start, length, len(lens), seq, heads, True)
    got = mt.from_panels_e4m3(ctx).view(torch.uint8)[:rows].cpu()
    assert torch.equal(got, flat), int((got != flat).sum())
    assert (flat[torch.from_numpy(~real)] == 0x7F).all()
    for b, n in enumerate(lens):
        alone = qkv[row0[b]:row0[b] + n].contiguous().cuda()
        want = mt.op_attention(mt.MT_BF16, alone, torch.ones((1, n), dtype=torch.int32, device="cuda"), 1, n, H, heads).float().cpu().view(n, H)
        have = flat[row0[b]:row0[b] + n].view(torch.float8_e4m3fn).float()
        assert ((have - want).abs() <= (2.0**-4 + 2.0**-8) * want.abs() + 2.0**-10).all()      # half a step of E4M3, half of the bf16 value


@pytest.mark.parametrize("hidden", [256, 768])
def test_fp8_embedding_gives_the_row_major_bits(hidden):
    """MT_FP8_FFN embeds with the row-major kernel."""
    states = []
    for precision in ("fp8", "fp8_all"):
        spec = dataclasses.replace(SMALL8, hidden=hidden, heads=hidden // 64, precision=precision)
        model, _ = mt.load_synthetic(spec, std=0.05)
        ids, mask, _ = ms.make_inputs(spec)
        model.forward_tokens(dev(ids), dev(mask))
        states.append(model.read_hidden(-1, 0, *ids.shape).cpu())
        model.close()
    say(f"fp8 embedding: {hidden} columns")
    assert states[0].abs().max() > 0 and torch.equal(*states)


SMALL8 = ms.MTSpec("small_fp8", vocab=500, hidden=256, heads=4, ffn=512, max_pos=64, n_trunk_layers=3,
                   tasks=(ms.TaskSpec(3, 2, 2), ms.TaskSpec(1, 1, 3), ms.TaskSpec(2, 0, 1), ms.TaskSpec(0, 2, 4, token_level=True),
                          ms.TaskSpec(3, 2, 2)),
                   precision="fp8", batch=7, seq=44, len_lo=5, len_hi=44, input_seed=5, weights_seed=99)


def _model(spec, stress=False, std=0.02, **kw):
    tr, tri = ms.make_trunk_params(spec, stress=stress, std=std)
    tps = [ms.make_task_params(spec, t, stress=stress, std=std) for t in range(spec.n_tasks)]
    model = mt.Model(mt.make_config(spec, **kw))
    model.load_params(-1, tr, len(tri))
    for t, (tp, tpi) in enumerate(tps):
        model.load_params(t, tp, len(tpi))
    return model, oracle.Oracle(spec, tr, [p for p, _ in tps])


def _safe_agreement(spec, got, ref, margin):
    col, n, agree = 0, 0, 0
    for t in spec.tasks:
        if t.token_level:
            continue
        if t.n_classes >= 2:
            g, o = got[:, col:col + t.n_classes], ref[:, col:col + t.n_classes]
            srt = np.sort(o, axis=1)
            safe = (srt[:, -1] - srt[:, -2]) > margin
            n += int(safe.sum())
            agree += int((g.argmax(1) == o.argmax(1))[safe].sum())
        col += t.n_classes
    return n, agree


@pytest.mark.parametrize("precision", ["fp8", "fp8_all"])
@pytest.mark.parametrize("stress", [False, True])
def test_fp8_small_model_whole_batches(stress, precision):
    """Heterogeneous forks, a task without own layers, a tagging task (all its layers on all rows, so its last layer is
    FP8 too), sequence tasks (last layer first-token-only, bf16), whole batches against the oracle."""
    spec = dataclasses.replace(SMALL8, precision=precision)
    model, orc = _model(spec, stress, 0.05)
    for bi in range(3):
        ids, mask, _ = ms.make_inputs(spec, batch_index=bi)
        ref, ref_tok = orc.mt_forward(ids, mask, want_tokens=True)
        got, tok = model.forward_tokens(dev(ids), dev(mask))
        got, tok = got.cpu().numpy(), tok.cpu().numpy()
        real = mask.astype(bool)
        err = max(float(np.abs(got - ref).max()), float(np.abs(tok[real] - ref_tok[real]).max()))
        bar = TOL[precision] * max(1.0, float(np.abs(ref).max()), float(np.abs(ref_tok[real]).max()))
        say(f"  {precision} small model stress={stress} batch {bi}: max |dlogit| {err:.4g} (bar {bar:.3g})")
        assert err <= bar
        n, agree = _safe_agreement(spec, got, ref, 2 * bar)
        assert agree == n
        assert (tok[~real] == 0).all()
    # the same checkpoints in the bf16 mode of the library are closer to the oracle: the FP8 path really ran
    spec_b = dataclasses.replace(spec, precision="bf16")
    mb = mt.Model(mt.make_config(spec_b))
    tr, tri = ms.make_trunk_params(spec, stress=stress, std=0.05)
    mb.load_params(-1, tr, len(tri))
    for t in range(spec.n_tasks):
        tp, tpi = ms.make_task_params(spec, t, stress=stress, std=0.05)
        mb.load_params(t, tp, len(tpi))
    ids, mask, _ = ms.make_inputs(spec)
    ref = orc.mt_forward(ids, mask)
    e_b = float(np.abs(mb.forward_tokens(dev(ids), dev(mask))[0].cpu().numpy() - ref).max())
    e_8 = float(np.abs(model.forward_tokens(dev(ids), dev(mask))[0].cpu().numpy() - ref).max())
    say(f"  same checkpoints: bf16 mode {e_b:.4g}, {precision} mode {e_8:.4g}")
    assert e_b <= 2e-2 and e_8 > e_b
    mb.close()
    model.close()


def test_fp8_panel_linear_of_more_row_panels_than_a_grid_takes():
    M, N, K = 65536 * 32 + 33, 32, 256
    say(f"fp8 panel linear: few-row form, {M} x {N} x {K}")
    gen = torch.Generator(device="cuda").manual_seed(3)
    pa = torch.randint(0, 0x38, ((M + 31) // 32, K // 16, 32, 16), dtype=torch.uint8, device="cuda", generator=gen)      # values of 0 to 0.94
    scale, w = mt.e4m3_quantize((np.random.default_rng(3).standard_normal((N, K)) * 0.02).astype(np.float32))
    slot = torch.full((256,), 127 - int(np.log2(scale)), dtype=torch.uint8, device="cuda")
    pw = torch.cat([slot, mt.to_panels_e4m3(dev(w).view(torch.float8_e4m3fn)).flatten()])
    pc = torch.full(((M + 31) // 32, N // 8, 32, 8), float("nan"), device="cuda")
    mt.op_panel_linear(pa, pw[256:], None, pc, fp8=True, M=M, N=N, K=K, out_f32=1, form=ROWS_1X1)
    for lo in (0, 32767, 32768, 65535, pc.shape[0] - 2):                         # panels: the first and last of a launch
        a = mt.from_panels_e4m3(pa[lo:lo + 2]).view(torch.uint8)
        assert torch.equal(mt.from_panels(pc[lo:lo + 2]).cpu(), mt.op_linear_fp8(a, dev(w), 1.0 / scale, None, None, 0, 1).cpu()), lo


@pytest.mark.parametrize("precision", ["fp8", "fp8_all"])
@pytest.mark.parametrize("hidden,ffn,batch,seq", [(192, 320, 5, 40), (256, 256, 3, 300), (512, 768, 40, 70)])
def test_fp8_layouts_and_attention_shapes(hidden, ffn, batch, seq, precision):
    """MT_FP8_FFN, and hidden or ffn not a multiple of 256: the row-major kernels; otherwise the panel layout, with sequences of few and many
    panels.  Plain and routed calls, a state that both an all-rows and a first-token layer read."""
    spec = dataclasses.replace(SMALL8, hidden=hidden, heads=hidden // 64, ffn=ffn, max_pos=seq, batch=batch, seq=seq, len_lo=3, len_hi=seq, precision=precision,
                               tasks=(ms.TaskSpec(3, 1, 2), ms.TaskSpec(1, 1, 3), ms.TaskSpec(1, 2, 5), ms.TaskSpec(2, 0, 1), ms.TaskSpec(0, 2, 4, token_level=True)))
    say(f"fp8 layouts: hidden {hidden}, ffn {ffn}, {batch} x {seq}, {precision}")
    model, orc = _model(spec, False, 0.05)
    ids, mask, _ = ms.make_inputs(spec)
    rows = np.arange(batch)[:6]
    ref, ref_tok = orc.mt_forward(ids[rows], mask[rows], want_tokens=True)
    got, tok = model.forward_tokens(dev(ids), dev(mask))
    got, tok = got.cpu().numpy(), tok.cpu().numpy()
    real = mask[rows].astype(bool)
    bar = TOL[precision] * max(1.0, float(np.abs(ref).max()), float(np.abs(ref_tok[real]).max()))
    err = max(float(np.abs(got[rows] - ref).max()), float(np.abs(tok[rows][real] - ref_tok[real]).max()))
    say(f"  max |dlogit| {err:.4g} (bar {bar:.3g})")
    assert err <= bar
    route = (np.arange(batch)[:, None] + np.arange(spec.n_tasks)) % 2 == 0
    route[:, 4] = False
    out = torch.full((batch, spec.n_logits), 7.0, device="cuda")
    model.forward_routed(dev(ids), dev(mask), route, out)
    out, col = out.cpu().numpy(), 0
    for t, task in enumerate(spec.tasks[:4]):
        o = out[:, col:col + task.n_classes]
        sel = route[rows, t]
        assert np.abs(o[rows][sel] - ref[sel, col:col + task.n_classes]).max() <= bar and (o[~route[:, t]] == 7.0).all()
        col += task.n_classes
    model.close()


@pytest.mark.parametrize("precision", ["fp8", "fp8_all"])
def test_fp8_base_workload_sampled_and_served(precision):
    """`base` shapes (B = 32, S = 128, 8 tasks) with E4M3 feed-forward matrices: sampled sequences against the oracle
    through mt_forward and through mt_forward_multi (8 request batches per call, the benchmark's configuration),
    replicas share the storage scales."""
    spec = dataclasses.replace(ms.get_config("base"), name="base_" + precision, precision=precision)
    model, orc = _model(spec, max_batch=8 * 32)
    ids, mask, lengths = ms.make_inputs(spec)
    rows = [0, int(np.argmin(lengths)), int(np.argmax(lengths)), 17]
    say("  oracle on rows", rows)
    ref = orc.mt_forward(ids[rows], mask[rows])
    got = model.forward(dev(ids), dev(mask)).cpu().numpy()
    assert np.isfinite(got).all()
    err = float(np.abs(got[rows] - ref).max())
    reqs = [(dev(ids), dev(mask))]
    for r in range(1, 8):
        i2, m2, _ = ms.make_inputs(spec, batch_index=r)
        reqs.append((dev(i2), dev(m2)))
    multi = model.forward_multi(reqs)[0].cpu().numpy()
    err_m = float(np.abs(multi[rows] - ref).max())
    rep = model.replica()
    again = rep.forward(dev(ids), dev(mask)).cpu().numpy()
    say(f"  {precision} base: max |dlogit| {err:.4g} (one request), {err_m:.4g} (eight per call); bar {TOL[precision]}")
    assert err <= TOL[precision] and err_m <= TOL[precision]
    assert np.array_equal(again, got)
    n, agree = _safe_agreement(spec, got[rows], ref, 2 * TOL[precision])
    assert agree == n
    rep.close()
    model.close()
