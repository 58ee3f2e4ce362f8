"""Projections on matrix-core fragments (bf16 weights, forwards of 17 rows and more) and prompts
prefilled in forwards of up to 512 rows.

Prompts whose lengths sit at the edges of the path: 16/17 rows (where it begins), 64/65 (the
first forward wider than the caller's rows can be), tile and row-block edges, 512/513 (one and
two forwards), appended to an empty or a non-empty context, with callers' row limits from 1 to
64.  Each prompt is checked against the float64 oracle (the last token's logits) and against the
same library with the K-split kernel (laser_model_set_gemm_kernel mode 1), which runs it in
chunks of the caller's rows: appended K/V within one rounding step of their storage type.
Tolerances are the parity protocol's (gpu_helpers)."""
import re

import numpy as np
import pytest
import torch

from gpu_helpers import LOGIT_TOL, compare_logits, make_pair, require_gpu
from oracle.transformer import SeqState
from paper_2606_31580_amd import laser as L
from paper_2606_31580_amd import synth
from paper_2606_31580_amd.configs import ModelShape

pytestmark = pytest.mark.gpu

HD64 = ModelShape("frag-hd64", 2, 256, 4, 2, 64, 352, 515, False, False, "bf16", 1.0e4, 1.0e-5)
HD128 = ModelShape("frag-hd128", 2, 384, 6, 2, 128, 1056, 1030, True, True, "bf16", 1.0e4, 1.0e-6)
FP8 = ModelShape("frag-fp8", 2, 384, 6, 2, 128, 1056, 1030, True, True, "bf16", 1.0e4, 1.0e-6, "fp8")


def _prefill(model, shape, kv, seq, prompt):
    lg = torch.zeros(shape.vocab, device="cuda")
    L.laser_prefill(model, kv, seq, prompt, lg)
    torch.cuda.synchronize()
    n = kv.seq_len(seq)
    dt = torch.float8_e4m3fn if shape.kv_storage == "fp8" else torch.bfloat16
    K = torch.empty((shape.n_layers, n, shape.n_kv_heads, shape.head_dim), dtype=dt, device="cuda")
    V = torch.empty_like(K)
    kv.export_kv(seq, K, V)
    torch.cuda.synchronize()
    return lg, K.float(), V.float()


@pytest.mark.parametrize("shape,max_rows,ctx,lengths", [
    (HD64, 64, 0, [16, 17, 32, 33, 64, 65, 129, 257]),
    (HD64, 1, 5, [1, 17, 80, 512, 513, 529]),
    (HD128, 16, 0, [17, 63, 97, 203, 300]),
    (HD128, 64, 37, [48, 49, 112, 161, 511, 520]),
    (FP8, 32, 250, [18, 40, 130]),
], ids=lambda v: v.name if isinstance(v, ModelShape) else None)
def test_prefill_edges(shape, max_rows, ctx, lengths):
    require_gpu()
    max_pos = 1024
    model, orc, _ = make_pair(shape, max_rows=max_rows, max_positions=max_pos, cache_oracle=True)
    k0, v0 = synth.make_prefill_kv(shape, ctx, 3) if ctx else (None, None)
    toks = synth.make_tokens(max(lengths), shape.vocab, 3007)
    st = SeqState.from_prefill(shape, synth.to_numpy(k0), synth.to_numpy(v0), max_pos) if ctx else SeqState(shape, max_pos)
    refs = {}
    for i, t in enumerate(toks):
        refs[i + 1] = orc.decode_token(st, int(t))
    # spacing of the storage type's values in [2^e, 2^(e+1)): 2^(e-7) for bf16 (8 significand bits),
    # 2^(e-3) for E4M3 (4), so neighbours differ by at most that fraction of the larger one
    step = 2.0 ** -3 if shape.kv_storage == "fp8" else 2.0 ** -7
    for n in lengths:
        got = {}
        for mode in (0, 1):
            model.set_gemm_kernel(mode)
            kv = L.KVCache(model, 2 * (max_pos // 16), 2, max_pos // 16, poison=True)
            kv.add_seq(0, ctx)
            if ctx:
                kv.import_kv(0, k0.cuda(), v0.cuda())
            got[mode] = _prefill(model, shape, kv, 0, toks[:n].cuda())
            kv.destroy()
        model.set_gemm_kernel(0)
        compare_logits(got[0][0].cpu().numpy(), refs[n], f"{shape.name} {n} tokens after {ctx}, max_rows {max_rows}")
        for a, b in zip(got[0][1:], got[1][1:]):
            assert torch.isfinite(a).all()
            lim = step * torch.maximum(torch.maximum(a.abs(), b.abs()), b.square().mean().sqrt())
            worst = float(((a - b).abs() / lim).max())
            assert worst <= 1.0, f"{shape.name} {n} tokens: appended K/V differ by {worst} rounding steps"
    model.destroy()


def test_probe_batches_and_mixed_steps():
    # probe chunks of 17-60 rows and mixed steps against the K-split kernel, with and without tiles
    # (bitwise), replayed from graphs with eager work in between
    require_gpu()
    shape = HD128
    w = {k: v.cuda() for k, v in synth.make_weights(shape).items()}
    w["final_norm"].fill_(8.0)
    model = L.Model(shape, w, max_rows=64, max_positions=1024, poison=True)
    suffix = synth.make_suffix(8, shape.vocab).cuda()
    for lens in ([300, 17, 45], [100, 16, 31, 250, 77, 400, 64], [50, 60, 70, 80]):
        B = len(lens)
        out = {}
        for mode, tiles in ((0, True), (0, False), (1, True)):
            model.set_gemm_kernel(mode)
            model.set_tiles(tiles)
            kv = L.KVCache(model, 256, B, 64, poison=True)
            for i, n in enumerate(lens):
                kv.add_seq(i, n)
                kv.import_kv(i, *synth.make_prefill_kv(shape, n, 90 + i, device="cuda"))
            lg = torch.zeros(B * 4, shape.vocab, device="cuda")
            conf, arg = torch.zeros(B, device="cuda"), torch.zeros(B * 4, dtype=torch.int32, device="cuda")
            reps = []
            for _ in range(3):
                L.laser_probe_confidence(model, kv, list(range(B)), suffix, 4, conf, arg, lg)
                torch.cuda.synchronize()
                reps.append((lg.clone(), conf.clone()))
                torch.zeros(1000, device="cuda").sum().item()
            for r in reps[1:]:
                assert torch.equal(r[0], reps[0][0]) and torch.equal(r[1], reps[0][1])
            tok = synth.make_tokens(B, shape.vocab, 83).cuda()
            nxt, p = torch.zeros(B, dtype=torch.int32, device="cuda"), torch.zeros(B, device="cuda")
            idx = list(range(0, B, 2))
            c2, a2 = torch.zeros(len(idx), device="cuda"), torch.zeros(len(idx) * 4, dtype=torch.int32, device="cuda")
            L.laser_step_mixed(model, kv, list(range(B)), tok, nxt, p, idx, suffix, 4, c2, a2)
            torch.cuda.synchronize()
            out[mode, tiles] = (reps[0][0], reps[0][1], p.clone(), c2.clone())
            kv.destroy()
        for a, b in zip(out[0, True], out[0, False]):
            assert torch.equal(a, b), "tiles change the results"
        first = out[0, True][0].view(B, 4, -1)[:, 0], out[1, True][0].view(B, 4, -1)[:, 0]  # (later rows follow their own tokens)
        assert float((first[0] - first[1]).abs().max()) <= 2e-2
        np.testing.assert_allclose(out[0, True][2].cpu(), out[1, True][2].cpu(), rtol=4e-2)
    model.destroy()


@pytest.mark.parametrize("shape,max_rows,rows", [(HD64, 20, 20), (HD128, 33, 33), (FP8, 17, 17), (HD64, 4, 65),
                                                 (HD128, 16, 129), (FP8, 64, 65)],
                         ids=lambda v: v.name if isinstance(v, ModelShape) else None)
def test_merge_in_attention(shape, max_rows, rows):
    # One-row attention groups that merge their splits inside the attention kernel, beside fragment
    # projections: decode batches from 17 rows, and the single row past the last 64 of a wide prefill,
    # whose splits have to fit that forward's partial slots.  Only the order of the fp32 merge differs.
    require_gpu()
    w = {k: v.cuda() for k, v in synth.make_weights(shape).items()}
    model = L.Model(shape, w, max_rows=max_rows, max_positions=1024, poison=True)
    decode = rows == max_rows
    lens = [40 + 45 * (i % 20) for i in range(rows)] if decode else [850]
    tok = synth.make_tokens(rows, shape.vocab, 29).cuda()
    out = []
    for fused in (False, True):
        model.set_attn_merge(fused, 128)
        kv = L.KVCache(model, 64 * len(lens), len(lens), 64, poison=True)
        for i, n in enumerate(lens):
            kv.add_seq(i, n)
            kv.import_kv(i, *synth.make_prefill_kv(shape, n, 7 + i, device="cuda"))
        if decode:
            lg, p = torch.zeros(rows, shape.vocab, device="cuda"), torch.zeros(rows, device="cuda")
            L.laser_decode_step(model, kv, list(range(rows)), tok, torch.zeros_like(tok), p, lg)
        else:
            lg = torch.zeros(shape.vocab, device="cuda")
            L.laser_prefill(model, kv, 0, tok, lg)
        torch.cuda.synchronize()
        out.append(lg)
        kv.destroy()
    assert torch.isfinite(out[1]).all()
    assert float((out[0] - out[1]).abs().max()) <= 2e-3
    model.destroy()


@pytest.mark.parametrize("group,hd", [(8, 128), (9, 128), (16, 128), (16, 64)])
def test_merge_in_attention_large_groups(group, hd):
    # One-row groups of up to 16 query heads per KV head, merged inside the attention kernel: group
    # x head dim / 4 chunks, more than its 256 threads above 8 heads of 128.  Against the merge
    # kernel; only the order of the fp32 merge differs.
    require_gpu()
    shape = ModelShape("merge-g%d" % group, 1, 64 * group, 2 * group, 2, hd, 352, 515, False, False, "bf16", 1.0e4, 1.0e-5)
    w = {k: v.cuda() for k, v in synth.make_weights(shape).items()}
    model = L.Model(shape, w, max_rows=3, max_positions=1024, poison=True)
    lens = [900, 350, 600]
    tok = synth.make_tokens(3, shape.vocab, 29).cuda()
    out = []
    for fused in (False, True):
        model.set_attn_merge(fused, 128)
        kv = L.KVCache(model, 192, 3, 64, poison=True)
        for i, n in enumerate(lens):
            kv.add_seq(i, n)
            kv.import_kv(i, *synth.make_prefill_kv(shape, n, 7 + i, device="cuda"))
        lg, p = torch.zeros(3, shape.vocab, device="cuda"), torch.zeros(3, device="cuda")
        L.laser_decode_step(model, kv, [0, 1, 2], tok, torch.zeros_like(tok), p, lg)
        torch.cuda.synchronize()
        out.append(lg)
        kv.destroy()
    assert torch.isfinite(out[1]).all()
    assert float((out[0] - out[1]).abs().max()) <= 2e-3
    model.destroy()


@pytest.mark.parametrize("shape,batch", [(HD64, 16), (HD64, 17), (HD64, 40), (FP8, 18)],
                         ids=lambda v: v.name if isinstance(v, ModelShape) else None)
def test_static_step_runs_the_same_kernels(shape, batch):
    # The allocation-free decode step on both sides of the row count where the fragment path begins:
    # the same kernels on the same splits as laser_decode_step, so the same bits.
    require_gpu()
    w = {k: v.cuda() for k, v in synth.make_weights(shape).items()}
    model = L.Model(shape, w, max_rows=batch, max_positions=512, poison=True)
    tok = synth.make_tokens(batch, shape.vocab, 31).cuda()
    out = []
    for step in (L.laser_decode_step, L.laser_decode_step_static):
        kv = L.KVCache(model, 32 * batch, batch, 32, poison=True)
        for i in range(batch):
            n = 30 + 23 * (i % 19)
            kv.add_seq(i, n)
            kv.import_kv(i, *synth.make_prefill_kv(shape, n, 5 + i, device="cuda"))
        lg, p = torch.zeros(batch, shape.vocab, device="cuda"), torch.zeros(batch, device="cuda")
        for _ in range(2):
            step(model, kv, list(range(batch)), tok, torch.zeros_like(tok), p, lg)
        torch.cuda.synchronize()
        out.append((lg, p))
        kv.destroy()
    assert torch.isfinite(out[1][0]).all()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    model.destroy()


@pytest.mark.parametrize("shape,what", [(HD64, "all"), (HD128, "all"), (FP8, "all"), (HD128, "tiles"), (HD128, "pools")],
                         ids=lambda v: getattr(v, "name", v))
def test_arrays_at_8_byte_boundaries(shape, what, monkeypatch):
    # Weights, workspace, weight tiles and page pools 8 bytes past a 16-byte boundary (tensors inside
    # one packed buffer): the copies straight to LDS ask for 16, so these calls take kernels that load
    # into registers.  A prompt, a decode step with runs of more than two pages per wave and a probe,
    # against the same on aligned arrays, which may take other kernels (tolerance: gpu_helpers).
    require_gpu()
    real = torch.empty

    def moved(n, dtype=torch.uint8, device="cuda"):
        return real(n + 24, dtype=dtype, device=device)[8:8 + n]

    def at8(t):
        out = moved(t.numel() * t.element_size()).view(t.dtype).view(t.shape)
        out.copy_(t)
        assert out.data_ptr() % 16 == 8
        return out

    w = {k: v.cuda() for k, v in synth.make_weights(shape).items()}
    n_seq, n, prompt = 20, 2000, 70  # (20 x 125 pages x 2 heads over 2,048 waves: 3 pages each)
    tok = synth.make_tokens(prompt, shape.vocab, 37).cuda()
    suffix = synth.make_suffix(8, shape.vocab).cuda()
    out = []
    for move in (False, True):
        with monkeypatch.context() as mp:  # what the binding allocates
            if move and what == "all":
                mp.setattr(torch, "empty", moved)
            model = L.Model(shape, {k: at8(v) for k, v in w.items()} if move and what == "all" else w, max_rows=24,
                            max_positions=2048, poison=True, tiles=False)
            if move and what == "tiles":
                mp.setattr(torch, "empty", moved)
            model.set_tiles(True)
            mp.setattr(torch, "empty", moved if move and what in ("all", "pools") else real)
            kv = L.KVCache(model, 128 * (n_seq + 1), n_seq + 1, 128, poison=True)
        assert model.workspace.data_ptr() % 16 == (8 if move and what == "all" else 0)
        assert model.tile_buf.data_ptr() % 16 == (8 if move and what != "pools" else 0)
        assert kv.k_pool.data_ptr() % 16 == (8 if move and what != "tiles" else 0)
        for i in range(n_seq):
            kv.add_seq(i, n - 7 * i)
            kv.import_kv(i, *synth.make_prefill_kv(shape, n - 7 * i, 11 + i, device="cuda"))
        kv.add_seq(n_seq, 0)
        lp = torch.zeros(shape.vocab, device="cuda")
        L.laser_prefill(model, kv, n_seq, tok, lp)
        lg, p = torch.zeros(n_seq, shape.vocab, device="cuda"), torch.zeros(n_seq, device="cuda")
        nxt = torch.zeros(n_seq, dtype=torch.int32, device="cuda")
        L.laser_decode_step(model, kv, list(range(n_seq)), tok, nxt, p, lg)
        conf, arg = torch.zeros(3, device="cuda"), torch.zeros(12, dtype=torch.int32, device="cuda")
        lq = torch.zeros(12, shape.vocab, device="cuda")
        L.laser_probe_confidence(model, kv, [0, 1, 2], suffix, 4, conf, arg, lq)
        torch.cuda.synchronize()
        out.append((lp, lg, lq.view(3, 4, -1)[:, 0]))
        kv.destroy()
        model.destroy()
    for a, b in zip(*out):
        assert torch.isfinite(b).all()
        assert float((a - b).abs().max()) <= LOGIT_TOL


@pytest.mark.parametrize("shape,max_rows", [(HD64, 1), (HD128, 16), (HD128, 40), (FP8, 64)], ids=lambda v: getattr(v, "name", v))
def test_workspace_without_wide_prefills(shape, max_rows, monkeypatch):
    # The smaller workspace that finalize takes: prompts in chunks of max_rows, no fragments, and
    # nothing written past its end.  Against the same calls with the full workspace, whose projections
    # sum in another order (tolerance: gpu_helpers).
    require_gpu()
    w = {k: v.cuda() for k, v in synth.make_weights(shape).items()}
    prompt = synth.make_tokens(97, shape.vocab, 43).cuda()
    tok = synth.make_tokens(max_rows, shape.vocab, 47).cuda()
    real, sizes, out = L._call, [], []

    def call(name, *a):
        if name != "laser_model_finalize":
            return real(name, *a)
        with pytest.raises(L.LaserError) as e:
            real(name, *a[:3], 16, *a[4:])
        full, small = (int(x) for x in re.findall(r"\d+", str(e.value).split("workspace of")[1])[:2])
        assert full == a[3] and small < full
        sizes.append(small)
        with pytest.raises(L.LaserError):
            real(name, *a[:3], small - 1, *a[4:])
        return real(name, *a[:3], small, *a[4:])

    for small in (False, True):
        with monkeypatch.context() as mp:
            if small:
                mp.setattr(L, "_call", call)
            model = L.Model(shape, w, max_rows=max_rows, max_positions=512, poison=True)
        kv = L.KVCache(model, 32 * (max_rows + 1), max_rows + 1, 32, poison=True)
        kv.add_seq(max_rows, 0)
        lp = torch.zeros(shape.vocab, device="cuda")
        L.laser_prefill(model, kv, max_rows, prompt, lp)
        for i in range(max_rows):
            kv.add_seq(i, 20 + 5 * i)
            kv.import_kv(i, *synth.make_prefill_kv(shape, 20 + 5 * i, 13 + i, device="cuda"))
        lg, p = torch.zeros(max_rows, shape.vocab, device="cuda"), torch.zeros(max_rows, device="cuda")
        L.laser_decode_step(model, kv, list(range(max_rows)), tok, torch.zeros_like(tok), p, lg)
        torch.cuda.synchronize()
        out.append((lp, lg))
        if small:
            assert bool((model.workspace[sizes[0]:] == 0xFF).all()), "written past the workspace's end"
        kv.destroy()
        model.destroy()
    for a, b in zip(*out):
        assert torch.isfinite(b).all()
        assert float((a - b).abs().max()) <= LOGIT_TOL
