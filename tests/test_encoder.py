"""Encode stage: host logic without a GPU, and GPU parity with the float64 oracle through the
C ABI (tolerances as for the denoising step: max-abs 2e-2, rel-L2 1e-2 on an output of rms ~1)."""
import os
import re

import numpy as np
import pytest

import synth
from helpers import rel_l2, max_abs
from oracle import encoder_oracle as E

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ARCH = synth.ENCODERS["t5_tiny"]


@pytest.fixture(scope="module")
def X():
    from paper_2510_02838_amd import encoder
    return encoder


@pytest.fixture(scope="module")
def torch():
    import torch
    torch.cuda.set_device(0)
    return torch


def test_library_exports_every_declared_encoder_symbol(X):
    hdr = open(os.path.join(ROOT, "include", "encoder.h")).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    declared = set(re.findall(r"\b(enc_[a-z_0-9]+)\s*\(", hdr))
    assert declared == set(X.EXPORTS) and len(declared) == 14


@pytest.mark.parametrize("name", list(synth.ENCODERS))
def test_encoder_tensor_table_matches_oracle_parameter_list(X, name):
    arch = synth.ENCODERS[name]
    m = X.Encoder(arch, bind=False)
    shapes = E.param_shapes(arch)
    table = m.tensors()
    assert [t[0] for t in table] == list(shapes)
    kinds = {"matrix": 0, "gain": 2, "table": 3}
    for tname, r, c, k in table:
        shape, kind = shapes[tname]
        assert k == kinds[kind]
        assert (r, c) == (tuple(shape) if len(shape) == 2 else (1, shape[0]))
    n_params = sum(int(np.prod(s)) for s, _ in shapes.values())
    assert 2 * n_params <= m.weight_bytes() <= 2.3 * n_params + (1 << 22) + 2 * arch["vocab"] * arch["d_model"]
    m.close()


def test_encoder_rejects_bad_configurations_and_lengths(X):
    for bad in (dict(ARCH, d_model=200), dict(ARCH, head_dim=96), dict(ARCH, d_ff=500), dict(ARCH, n_layers=0),
                dict(ARCH, n_heads=3), dict(ARCH, vocab=0)):
        with pytest.raises(Exception):
            X.Encoder(bad, bind=False)
    m = X.Encoder(ARCH, bind=False)
    a = m.workspace_bytes([30])
    b = m.workspace_bytes([30, 500])
    assert 0 < a < b
    assert m.workspace_bytes([0]) == 0 and m.workspace_bytes([]) == 0 and m.workspace_bytes([1025]) == 0
    m.close()


# --------------------------------------------------------------------------------- GPU
def _case(torch, X, arch, lens, std=0.05, gain_std=0.1, bias_scale=1.0):
    params = synth.make_params(E.param_shapes(arch), 1, std, 0.0, gain_std)
    params["rel_bias"] = synth.round_bf16(params["rel_bias"] * bias_scale / std)       # O(bias_scale) biases
    params["embed"] = synth.round_bf16(params["embed"] / std)                          # O(1) embeddings
    toks = synth.make_tokens(lens, arch["vocab"])
    m = X.Encoder(arch)
    m.ensure_workspace(lens)
    m.init_weights(0, 0.0)
    m.set_params(params)
    d_tok = torch.from_numpy(np.concatenate(toks)).cuda()
    return params, toks, m, d_tok


@pytest.mark.gpu
@pytest.mark.parametrize("lens", [[1], [30], [64, 7, 300], [129, 500, 65]])
def test_encoder_forward_against_oracle(torch, X, lens):
    params, toks, m, d_tok = _case(torch, X, ARCH, lens, bias_scale=2.0)
    n = sum(lens)
    out16 = torch.full((n, ARCH["d_model"]), float("nan"), dtype=torch.bfloat16, device="cuda")
    out32 = torch.full((n, ARCH["d_model"]), float("nan"), dtype=torch.float32, device="cuda")
    m.forward(lens, d_tok, out16, out32)
    torch.cuda.synchronize()
    got32, got16 = out32.cpu().numpy(), out16.to(torch.float32).cpu().numpy()
    ora = E.EncoderOracle(ARCH, params)
    o = 0
    for s, L in enumerate(lens):
        ref = ora.forward(toks[s])
        g = got32[o:o + L]
        assert np.isfinite(g).all()
        assert max_abs(g, ref) <= 2e-2 * max(1.0, np.abs(ref).max()), (s, max_abs(g, ref))
        assert rel_l2(g, ref) <= 1e-2, (s, rel_l2(g, ref))
        assert rel_l2(got16[o:o + L], ref) <= 1e-2
        o += L
    m.close()


@pytest.mark.gpu
@pytest.mark.parametrize("lens", [[1], [33], [64], [65], [300, 77]])
def test_encoder_benchmark_width_few_rows(torch, X, lens):
    """The 32x128 tiles for few rows, split over K (one row of tiles in every product; two in the attention output product
    up to 64 rows), the 128-row tiles from there on, and the norm with a workgroup per row: one layer of the benchmark
    width, same bounds as the other encoder tests."""
    arch = dict(synth.ENCODERS["t5_xxl"], n_layers=1, vocab=512)
    params, toks, m, d_tok = _case(torch, X, arch, lens, std=0.0125, bias_scale=2.0)
    out32 = torch.full((sum(lens), arch["d_model"]), float("nan"), dtype=torch.float32, device="cuda")
    m.forward(lens, d_tok, None, out32)
    torch.cuda.synchronize()
    got, ora, o = out32.cpu().numpy(), E.EncoderOracle(arch, params), 0
    for s, L in enumerate(lens):
        ref = ora.forward(toks[s])
        assert np.isfinite(got[o:o + L]).all()
        assert rel_l2(got[o:o + L], ref) <= 1e-2, (s, rel_l2(got[o:o + L], ref))
        o += L
    m.close()


@pytest.mark.gpu
@pytest.mark.parametrize("lens", [[32], [500, 7]])
def test_encoder_benchmark_width_one_layer(torch, X, lens):
    """The T5-XXL width the stage tables are timed at (d_model 4096, 64 heads, d_ff 10240), one
    layer, vocabulary cut to 2048 rows (the lookup does not depend on the width of the table's
    other dimension): three-product q/k/v launches, K = 10240 in the MLP's output product and, for
    the short prompts, the split-K form, none of which the 256-wide test model reaches."""
    arch = dict(synth.ENCODERS["t5_xxl"], n_layers=1, vocab=2048)
    params, toks, m, d_tok = _case(torch, X, arch, lens, std=0.0125, bias_scale=2.0)
    n = sum(lens)
    out32 = torch.full((n, arch["d_model"]), float("nan"), dtype=torch.float32, device="cuda")
    m.forward(lens, d_tok, None, out32)
    torch.cuda.synchronize()
    got32 = out32.cpu().numpy()
    ora = E.EncoderOracle(arch, params)
    o = 0
    for s, L in enumerate(lens):
        ref = ora.forward(toks[s])
        g = got32[o:o + L]
        assert np.isfinite(g).all()
        assert max_abs(g, ref) <= 2e-2 * max(1.0, np.abs(ref).max()), (s, max_abs(g, ref))
        assert rel_l2(g, ref) <= 1e-2, (s, rel_l2(g, ref))
        o += L
    m.close()


@pytest.mark.gpu
def test_encoder_intermediates_and_batch_independence(torch, X):
    lens = [40, 200]
    params, toks, m, d_tok = _case(torch, X, ARCH, lens, bias_scale=3.0)
    n, d, inner, dff = sum(lens), ARCH["d_model"], ARCH["n_heads"] * ARCH["head_dim"], ARCH["d_ff"]
    bufs = {"l0.ln1": torch.zeros((n, d), dtype=torch.bfloat16, device="cuda"),
            "l0.attn": torch.zeros((n, inner), dtype=torch.bfloat16, device="cuda"),
            "l0.x_attn": torch.zeros((n, d), dtype=torch.float32, device="cuda"),
            "l0.act": torch.zeros((n, dff), dtype=torch.bfloat16, device="cuda"),
            "l1.x_out": torch.zeros((n, d), dtype=torch.float32, device="cuda")}
    for name, t in bufs.items():
        m.set_tap(name, t)
    out32 = torch.empty((n, d), dtype=torch.float32, device="cuda")
    m.forward(lens, d_tok, None, out32)
    torch.cuda.synchronize()
    ora = E.EncoderOracle(ARCH, params)
    taps = [dict(), dict()]
    for s in range(2):
        ora.forward(toks[s], taps[s])
    for name, t in bufs.items():
        ref = np.concatenate([taps[0][name], taps[1][name]])
        got = t.to(torch.float32).cpu().numpy()
        assert rel_l2(got, ref) <= 1e-2, (name, rel_l2(got, ref))
    # a sequence's output does not depend on its batch mates
    m.clear_taps()
    solo = torch.empty((lens[1], d), dtype=torch.float32, device="cuda")
    m.forward([lens[1]], d_tok[lens[0]:], None, solo)
    torch.cuda.synchronize()
    assert np.array_equal(solo.cpu().numpy(), out32[lens[0]:].cpu().numpy())
    m.close()


@pytest.mark.gpu
@pytest.mark.parametrize("lens", [[31], [33, 61], [77, 130, 125], [77, 200, 33, 131, 97, 500, 51], [500, 431, 351, 287, 255, 201, 163, 127, 97, 77, 77, 64, 51, 43, 33, 31]])
def test_encoder_benchmark_widths_over_the_tiles(torch, X, lens):
    """One layer of the benchmark widths, from the split tiles for few rows to the 8-wave tiles, with prompts of odd length
    (the transposed values of a product's rows then start anywhere, break inside a tile and leave pad columns between
    the prompts): every prompt against the oracle."""
    arch = dict(synth.ENCODERS["t5_xxl"], n_layers=1, vocab=1024)
    m = X.Encoder(arch)
    m.ensure_workspace(lens)
    m.workspace.fill_(0xFF)                              # NaN in whatever is read without having been written
    m.init_weights(3, 0.008)
    shapes = E.param_shapes(arch)
    params = {n: m.get_tensor(n, shapes[n][0]) for n in shapes}
    toks = synth.make_tokens(lens, arch["vocab"])
    out = torch.empty((sum(lens), arch["d_model"]), dtype=torch.float32, device="cuda")
    m.forward(lens, torch.from_numpy(np.concatenate(toks)).cuda(), None, out)
    torch.cuda.synchronize()
    got, ora, at = out.cpu().numpy(), E.EncoderOracle(arch, params), 0
    assert np.isfinite(got).all()
    for n, t in zip(lens, toks):
        ref = ora.forward(t)
        assert rel_l2(got[at:at + n], ref) <= 1e-2, (n, rel_l2(got[at:at + n], ref))
        at += n
    m.close()


@pytest.mark.gpu
def test_encoder_device_init_matches_host_generator_and_feeds_the_denoiser(torch, X):
    """Weights from the device generator equal the host recipe bit for bit; the bf16 output has
    the layout the denoising step takes as its condition."""
    m = X.Encoder(ARCH)
    lens = [16]
    m.ensure_workspace(lens)
    m.init_weights(1, 0.05)
    shapes = E.param_shapes(ARCH)
    host = synth.make_params(shapes, 1, 0.05)
    for name in ("embed", "rel_bias", "l0.q.w", "l1.wo.w", "l0.ln1.g", "final.g"):
        got = m.get_tensor(name, shapes[name][0])
        assert np.array_equal(got, host[name].reshape(shapes[name][0])), name
    toks = synth.make_tokens(lens, ARCH["vocab"])
    d_tok = torch.from_numpy(toks[0]).cuda()
    cond = torch.empty((16, ARCH["d_model"]), dtype=torch.bfloat16, device="cuda")
    m.forward(lens, d_tok, cond, None)
    torch.cuda.synchronize()
    ref = E.EncoderOracle(ARCH, host).forward(toks[0])
    # (raw N(0, 0.05^2) embeddings make the residual stream as small as the branch outputs, so the
    # bf16 noise of four branches shows at full size; the parity tests above use O(1) embeddings)
    assert rel_l2(cond.to(torch.float32).cpu().numpy(), ref) <= 3e-2
    # tiny denoiser with cond_dim == d_model == 256 consumes it directly
    from paper_2510_02838_amd import binding as B
    arch = synth.CONFIGS["tiny"]["arch"]
    dit = B.DiT(arch)
    reqs = [(1, 16, 16, 16)]
    dit.ensure_workspace(reqs, 1)
    dit.init_weights(1, 0.02)
    lat = torch.randn(4 * 16 * 16, device="cuda")
    dit.sample(reqs, lat, cond, synth.default_sigmas(1)[None, :])
    torch.cuda.synchronize()
    assert torch.isfinite(lat).all()
    m.close()
