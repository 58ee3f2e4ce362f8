"""Attention over long runs of pages (LDS rings) and two query tiles per item, for every KV type.

Decode batches wide enough that the planner lengthens the runs past two pages per wave (60
requests of 700 to 1,000 positions), with lengths that end in every part of a page pair; and
probe chunks of several 16-column tiles at long contexts, where items hold two tiles, with an odd
and an even number of tiles.  Checked row by row against the float64 oracle (tolerances of the
parity protocol)."""
import pytest
import torch

from gpu_helpers import check_prob, compare_logits, make_pair, require_gpu
from oracle.transformer import SeqState, lm_stats
from paper_2606_31580_amd import laser as L
from paper_2606_31580_amd import synth
from paper_2606_31580_amd.configs import ModelShape

pytestmark = pytest.mark.gpu


def _shape(kind, hd):
    return ModelShape(f"runs-{kind}-{hd}", 2, 256, 6, 2, hd, 352, 515, False, True, "f32" if kind == "f32" else "bf16", 1.0e4,
                      1.0e-5, "fp8" if kind == "fp8" else "")


def _filled(model, shape, lens, extra, max_pos):
    pages = sum((n + extra) // 16 + 2 for n in lens)
    kv = L.KVCache(model, pages, len(lens), max_pos // 16, poison=True)
    for i, n in enumerate(lens):
        kv.add_seq(i, n)
        k, v = synth.make_prefill_kv(shape, n, i)
        kv.import_kv(i, k.cuda(), v.cuda())
    return kv


def _state(shape, n, i, max_pos):
    k, v = synth.make_prefill_kv(shape, n, i)
    return SeqState.from_prefill(shape, synth.to_numpy(k), synth.to_numpy(v), max_pos)


@pytest.mark.parametrize("kind", ["f32", "bf16", "fp8"])
@pytest.mark.parametrize("hd", [64, 128])
def test_long_runs(kind, hd):
    require_gpu()
    shape, max_pos, B = _shape(kind, hd), 1056, 60
    model, orc, _ = make_pair(shape, max_rows=64, max_positions=max_pos, cache_oracle=True)
    lens = [700 + (37 * i) % 301 for i in range(B)]
    lens[:6] = [1000, 991, 992, 993, 1, 17]
    kv = _filled(model, shape, lens, 8, max_pos)
    tok = synth.make_tokens(B, shape.vocab, 3100)
    d_tok, nxt, p = tok.cuda(), torch.zeros(B, dtype=torch.int32, device="cuda"), torch.zeros(B, device="cuda")
    lg = torch.zeros(B, shape.vocab, device="cuda")
    L.laser_decode_step(model, kv, list(range(B)), d_tok, nxt, p, lg)
    torch.cuda.synchronize()
    for b in list(range(8)) + [31, 59]:
        ref = orc.decode_token(_state(shape, lens[b], b, max_pos), int(tok[b]))
        compare_logits(lg[b].cpu().numpy(), ref, f"{shape.name} request {b} ({lens[b]} positions)")
        check_prob(p[b].item(), lm_stats(ref)[1], f"{shape.name} request {b}")
    kv.destroy()
    model.destroy()


@pytest.mark.parametrize("kind,hd,S", [("bf16", 128, 6), ("bf16", 128, 11), ("fp8", 128, 9), ("bf16", 64, 8)])
def test_two_tiles_per_item(kind, hd, S):
    # G = 3: S = 6, 9, 11 rows are 18, 27, 33 columns (two tiles, two, three), S = 8 is 24
    require_gpu()
    shape, max_pos = _shape(kind, hd), 16640
    model, orc, _ = make_pair(shape, max_rows=64, max_positions=max_pos, cache_oracle=True)
    lens = [16000, 15993, 15007, 14001, 13000]
    kv = _filled(model, shape, lens, S + 8, max_pos)
    suffix = synth.make_suffix(S, shape.vocab)
    B = len(lens)
    conf, arg = torch.zeros(B, device="cuda"), torch.zeros(B, dtype=torch.int32, device="cuda")
    lg = torch.zeros(B, shape.vocab, device="cuda")
    L.laser_probe_confidence(model, kv, list(range(B)), suffix.cuda(), 1, conf, arg, lg)
    torch.cuda.synchronize()
    for b in (0, 1, 4):
        res = orc.probe(_state(shape, lens[b], b, max_pos), [int(t) for t in suffix], 1, keep_logits=True)
        compare_logits(lg[b].cpu().numpy(), res.logits[0], f"{shape.name} probe of request {b}")
        check_prob(conf[b].item(), res.confidence, f"{shape.name} confidence of request {b}")
    kv.destroy()
    model.destroy()


@pytest.mark.parametrize("kind", ["bf16", "fp8"])
@pytest.mark.parametrize("lens", [[100 + i % 5 for i in range(40)] + [14000] + [90] * 23, [1500 + i % 9 for i in range(64)]],
                         ids=["one-long", "even"])
def test_batches_of_64(kind, lens):
    # one long request among many short ones (short runs), and an even batch whose every request is one
    # workgroup per KV head (runs of 24 pages)
    require_gpu()
    shape = ModelShape(f"runs64-{kind}", 1, 256, 16, 8, 64, 352, 515, False, True, "bf16", 1.0e4, 1.0e-5,
                       "fp8" if kind == "fp8" else "")
    max_pos, B = 14336, len(lens)
    model, orc, _ = make_pair(shape, max_rows=64, max_positions=max_pos, cache_oracle=True)
    kv = _filled(model, shape, lens, 8, max_pos)
    tok = synth.make_tokens(B, shape.vocab, 3200)
    d_tok, nxt, p = tok.cuda(), torch.zeros(B, dtype=torch.int32, device="cuda"), torch.zeros(B, device="cuda")
    lg = torch.zeros(B, shape.vocab, device="cuda")
    L.laser_decode_step(model, kv, list(range(B)), d_tok, nxt, p, lg)
    torch.cuda.synchronize()
    assert torch.isfinite(lg).all()
    for b in (0, 3, 39, 40, 41, 63):
        ref = orc.decode_token(_state(shape, lens[b], b, max_pos), int(tok[b]))
        compare_logits(lg[b].cpu().numpy(), ref, f"{shape.name} request {b} ({lens[b]} positions)")
        check_prob(p[b].item(), lm_stats(ref)[1], f"{shape.name} request {b}")
    kv.destroy()
    model.destroy()


@pytest.mark.parametrize("lens", [[14000] * 24, [6000 - i for i in range(16)]], ids=["longest-runs", "two-per-xcd"])
def test_few_items_per_head(lens):
    # 32 KV heads, every request one workgroup per head: runs of 219 pages a wave, and of 94
    require_gpu()
    shape = ModelShape("runs-mha", 1, 256, 32, 32, 64, 352, 515, False, False, "bf16", 1.0e4, 1.0e-5)
    max_pos, B = 14336, len(lens)
    model, orc, _ = make_pair(shape, max_rows=64, max_positions=max_pos, cache_oracle=True)
    kv = L.KVCache(model, sum((n + 24) // 16 + 1 for n in lens), B, max_pos // 16, poison=True)
    k, v = synth.make_prefill_kv(shape, max(lens), 0)
    for i, n in enumerate(lens):
        kv.add_seq(i, n)
        kv.import_kv(i, k[:, :n].contiguous().cuda(), v[:, :n].contiguous().cuda())
    tok = synth.make_tokens(B, shape.vocab, 3300)
    d_tok, nxt, p = tok.cuda(), torch.zeros(B, dtype=torch.int32, device="cuda"), torch.zeros(B, device="cuda")
    lg = torch.zeros(B, shape.vocab, device="cuda")
    L.laser_decode_step(model, kv, list(range(B)), d_tok, nxt, p, lg)
    torch.cuda.synchronize()
    assert torch.isfinite(lg).all()
    for b in (0, B - 1):
        n = lens[b]
        st = SeqState.from_prefill(shape, synth.to_numpy(k[:, :n].contiguous()), synth.to_numpy(v[:, :n].contiguous()), max_pos)
        ref = orc.decode_token(st, int(tok[b]))
        compare_logits(lg[b].cpu().numpy(), ref, f"{shape.name} request {b} ({n} positions)")
        check_prob(p[b].item(), lm_stats(ref)[1], f"{shape.name} request {b}")
    kv.destroy()
    model.destroy()
