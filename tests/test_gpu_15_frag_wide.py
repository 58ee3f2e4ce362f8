"""The fragment projections at the projections' real widths, whose wide forwards run workgroups of
several row waves (frag_shape: 256 compute units).

Two layers of the 1.5B, 7B and 8B shapes with a small vocabulary, prompts of 65 to 511 rows in one
forward.  Over these row counts every entry of LASER_FRAG_SHAPES with more than one row wave is chosen
for each projection that ever takes it, with K shares from 1 to 8, with row blocks and group blocks that
are full and that end early: 3 x 4 (7B residual at 65, QKV at 257; 8B gate/up at 65), 4 x 3 (8B QKV at
203, 1.5B residual at 203), 4 x 4 (7B residual at 122 and 250, QKV at 300; 8B gate/up at 340), 4 x 5 (7B
gate/up at 65 and 257, QKV at 449; 1.5B gate/up at 203), eight-wave 4 x 4 (8B gate/up at 130, residual at
203, QKV at 490) and 4 x 5 (7B gate/up at 250 and 449, 1.5B at 257).

Against the K-split kernel (set_gemm_kernel mode 1, itself checked against the oracle at these widths),
which runs the prompt in chunks of 64 rows: the last token's logits, and every row's appended K/V.
Those of the second layer follow every projection of the first, row by row, so a wrong row or column
of any of them shows."""
from dataclasses import replace

import pytest
import torch

from gpu_helpers import LOGIT_TOL, require_gpu
from paper_2606_31580_amd import laser as L
from paper_2606_31580_amd import synth
from paper_2606_31580_amd.configs import LLAMA_8B, QWEN_1P5B, QWEN_7B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,rows", [(QWEN_1P5B, [203, 257]), (QWEN_7B, [65, 122, 250, 257, 300, 449, 511]),
                                        (LLAMA_8B, [65, 130, 203, 340, 490, 511])], ids=lambda v: getattr(v, "name", None))
def test_wide_prefill(shape, rows):
    require_gpu()
    shape = replace(shape, n_layers=2, vocab=515)
    model = L.Model(shape, synth.make_weights(shape, device="cuda"), max_rows=64, max_positions=512, poison=True)
    tok = synth.make_tokens(max(rows), shape.vocab, 41).cuda()
    for n in rows:
        got = []
        for mode in (0, 1):
            model.set_gemm_kernel(mode)
            kv = L.KVCache(model, 32, 1, 32, poison=True)
            kv.add_seq(0, 0)
            lg = torch.zeros(shape.vocab, device="cuda")
            L.laser_prefill(model, kv, 0, tok[:n], lg)
            K = torch.empty((2, n, shape.n_kv_heads, shape.head_dim), dtype=torch.bfloat16, device="cuda")
            V = torch.empty_like(K)
            kv.export_kv(0, K, V)
            torch.cuda.synchronize()
            got.append((lg, K.float(), V.float()))
            kv.destroy()
        (la, *kva), (lb, *kvb) = got
        assert torch.isfinite(la).all()
        err = float((la - lb).abs().max())
        assert err <= LOGIT_TOL, f"{shape.name} {n} rows: logits differ by {err}"
        for a, b in zip(kva, kvb):
            assert torch.isfinite(a).all()
            # one step of bf16 (neighbours differ by at most 2^-7 of the larger), of a row mean
            # square for values near zero, as for the narrow shapes
            lim = 2.0 ** -7 * torch.maximum(torch.maximum(a.abs(), b.abs()), b.square().mean().sqrt())
            worst = float(((a - b).abs() / lim).max())
            assert worst <= 1.0, f"{shape.name} {n} rows: appended K/V differ by {worst} rounding steps"
        print(f"{shape.name} {n} rows: logits within {err:.2g}", flush=True)
    model.destroy()
