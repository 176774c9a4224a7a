"""GPU parity, kernel by kernel: every step of the hot path is fed the SAME inputs as the CPU
oracle and compared element by element through the C ABI.

Bars: integer codes and scales of the quantiser bit-exact; floats rel-L2 <= 1e-5 on the fp32
paths (DLCX_MMA_FMA, DLCX_MMA_F32) and <= 2e-3 on the bf16 MFMA path.
"""
import ctypes as C

import numpy as np
import pytest
import torch

import paper_2506_21263_amd as dlcx
import synth
from oracle import ref
from gpu_util import DEV, GUARD, close, payload_buffers, rel_l2, to_dev, to_np, ws_for

pytestmark = pytest.mark.gpu

TOL = GUARD
MODES = [dlcx.MMA_FMA, dlcx.MMA_F32, dlcx.MMA_BF16]
MODE_IDS = ["mma_fma", "mma_f32", "mma_bf16"]


def rng(seed):
    return np.random.default_rng(seed)


# ------------------------------------------------------------------ streaming kernels
@pytest.mark.parametrize("numel", [0, 1, 3, 4, 1023, 4096, 4099, 1 << 20, (1 << 20) + 7])
@pytest.mark.parametrize("kind", ["f32", "bf16"])
def test_delta_ef(numel, kind):
    g = rng(numel + 11)
    pad = numel + 8
    tg = (0.02 * g.standard_normal(pad)).astype(np.float32)
    e = (1e-3 * g.standard_normal(pad)).astype(np.float32)
    tl32 = (tg - 1e-3 * g.standard_normal(pad)).astype(np.float32)
    tl = synth.f32_to_bf16_bits(tl32) if kind == "bf16" else tl32
    want = ref.delta_ef(tg[:numel], tl[:numel], e[:numel]) if numel else np.zeros(0, np.float32)
    d_e = to_dev(e)
    dlcx.dlcx_delta_ef(to_dev(tg), to_dev(tl), d_e, numel=numel)
    got = to_np(d_e)
    assert np.array_equal(got[numel:], e[numel:]), "wrote past numel"
    if numel:  # (theta - theta_l) + e summed in fp64 and rounded once on both sides
        assert np.array_equal(got[:numel].view(np.uint32), want.view(np.uint32))


@pytest.mark.parametrize("numel", [0, 4, 5, 4096, (1 << 20) + 3])
def test_outer_nesterov(numel):
    g = rng(numel + 5)
    pad = numel + 8
    th = (0.02 * g.standard_normal(pad)).astype(np.float32)
    v = (1e-3 * g.standard_normal(pad)).astype(np.float32)
    gr = (1e-3 * g.standard_normal(pad)).astype(np.float32)
    th_w, v_w = th[:numel].copy(), v[:numel].copy()
    if numel:
        ref.outer_nesterov(th_w, v_w, gr[:numel].copy(), synth.LR, synth.MU)
    d_th, d_v = to_dev(th), to_dev(v)
    dlcx.dlcx_outer_nesterov(d_th, d_v, to_dev(gr), synth.LR, synth.MU, numel=numel)
    got_th, got_v = to_np(d_th), to_np(d_v)
    assert np.array_equal(got_th[numel:], th[numel:]) and np.array_equal(got_v[numel:], v[numel:])
    if numel:
        assert rel_l2(got_th[:numel], th_w) <= 1e-6 and rel_l2(got_v[:numel], v_w) <= 1e-6


def test_outer_nesterov_three_steps_closed_form(golden):
    g = golden("nesterov_closed_form.txt")
    th = torch.zeros(8, device=DEV)
    v = torch.zeros(8, device=DEV)
    gr = torch.ones(8, device=DEV)
    for want in g["theta_t1_t2_t3"]:
        dlcx.dlcx_outer_nesterov(th, v, gr, g["lr"][0], g["mu"][0])
        assert np.allclose(to_np(th), want, rtol=3e-7)


# ------------------------------------------------------------------ quantiser
@pytest.mark.parametrize("qbits", [4, 8])
@pytest.mark.parametrize("group", [16, 32, 64, 128, 256])
def test_quantize_codes_and_scales_bit_exact(qbits, group):
    g = rng(qbits * 1000 + group)
    count = group * 1031  # ragged against the 1024-element workgroup
    x = (g.standard_normal(count) * np.exp(2 * g.standard_normal(count))).astype(np.float32)
    x[3 * group:4 * group] = 0.0                       # all-zero group
    x[5 * group:6 * group] = 1e-40                      # denormal group (below the cut)
    qmax = 2 ** (qbits - 1) - 1
    x[7 * group] = float(qmax)                          # exact ties: x * inv on .5 boundaries
    x[7 * group + 1:8 * group] = 0.0
    x[7 * group + 1:7 * group + 7] = [0.5, 1.5, 2.5, -0.5, -1.5, -2.5]
    codes_w, scales_w = ref.quantize(x, qbits, group)
    codes = torch.zeros(codes_w.size, device=DEV, dtype=torch.uint8)
    scales = torch.zeros(scales_w.size, device=DEV, dtype=torch.float32)
    dlcx.dlcx_quantize(to_dev(x), qbits, group, codes, scales)
    assert np.array_equal(to_np(scales).view(np.uint32), scales_w.view(np.uint32))
    assert np.array_equal(to_np(codes), codes_w)


@pytest.mark.parametrize("qbits,group,K", [(4, 64, 2), (4, 128, 4), (8, 64, 8), (4, 16, 1), (8, 256, 16),
                                           (4, 32, 3), (8, 128, 7)])
def test_dequant_average(qbits, group, K):
    g = rng(K * 7 + qbits)
    count = group * 517
    payloads = [ref.quantize((g.standard_normal(count) * (1 + k)).astype(np.float32), qbits, group)
                for k in range(K)]
    want = ref.dequant_average([p[0] for p in payloads], [p[1] for p in payloads], count, qbits, group)
    out = torch.zeros(count, device=DEV)
    dlcx.dlcx_dequant_average([to_dev(p[0]) for p in payloads], [to_dev(p[1]) for p in payloads],
                              count, qbits, group, out)
    # fp64 sum of exact products in worker order, one rounding: the same bits on both sides
    assert np.array_equal(to_np(out).view(np.uint32), want.view(np.uint32))


# ------------------------------------------------------------------ rank-r products
SHAPES = [  # (m, n, r, K, group): several tiles and ragged tails in both dimensions
    (512, 512, 8, 2, 64),
    (528, 336, 5, 3, 16),
    (208, 1040, 33, 1, 16),
    (1024, 768, 64, 4, 128),
    (640, 2048, 96, 2, 128),
    (2048, 512, 256, 1, 64),
    (4096, 320, 200, 8, 64),     # enough workgroups for the 128-row form of the P kernel
    # the two-role kernels with ragged rows and columns, a partial last stage and a partial last
    # basis block, at 2, 4 and 8 basis blocks
    (4240, 208, 40, 8, 16),
    (4112, 336, 72, 8, 16),
    (4112, 336, 130, 8, 16),
    # the smallest sizes the descriptor admits (one group per side, rank 1), the largest number
    # of workers, a rank equal to the smaller side
    (16, 16, 1, 1, 16),
    (32, 48, 16, 16, 16),
    (64, 48, 40, 2, 16),
]


def _lowrank_inputs(m, n, r, K, seed):
    inp = synth.MatrixInputs(m, n, K, r, seed=seed, sigma=1e-3, alpha=1.0)
    deltas = [inp.raw_pseudo_gradient(1, k).astype(np.float32) for k in range(K)]
    return inp, deltas


@pytest.mark.parametrize("mma", MODES, ids=MODE_IDS)
@pytest.mark.parametrize("m,n,r,K,group", SHAPES)
def test_project_p_and_q(mma, m, n, r, K, group):
    inp, deltas = _lowrank_inputs(m, n, r, K, seed=m + n + r)
    d = dlcx.desc(m, n, r, 4, group, mma)
    ws = ws_for(d, K)
    d_deltas = [to_dev(x) for x in deltas]
    # P phase with the round-1 Gaussian basis
    want_p = [ref.project_p(x, inp.q_in) for x in deltas]
    outs = [torch.zeros(r, m, device=DEV) for _ in range(K)]
    dlcx.dlcx_project(d, dlcx.PHASE_P, d_deltas, to_dev(inp.q_in), outs, ws)
    for k in range(K):
        assert close(to_np(outs[k]), want_p[k], TOL[mma]), ("P", k)
    # Q phase with the oracle's orthonormal basis
    p_hat = ref.orthonormalize(np.mean(want_p, axis=0).astype(np.float32))
    want_q = [ref.project_q(x, p_hat) for x in deltas]
    outs = [torch.zeros(r, n, device=DEV) for _ in range(K)]
    dlcx.dlcx_project(d, dlcx.PHASE_Q, d_deltas, to_dev(p_hat), outs, ws)
    for k in range(K):
        assert close(to_np(outs[k]), want_q[k], TOL[mma]), ("Q", k)


@pytest.mark.parametrize("mma", [dlcx.MMA_F32, dlcx.MMA_BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("m,n,r,K", [
    (1040, 3184, 24, 1), (144, 4112, 48, 2), (1296, 2064, 100, 3), (528, 1808, 200, 1),  # P split by columns
    (1040, 784, 100, 2), (336, 1008, 200, 3), (2096, 272, 145, 1),  # short rows: 64 per workgroup
    (3184, 1040, 24, 1), (4112, 144, 48, 2), (2064, 1296, 100, 3), (1808, 528, 200, 1),  # Q split by rows
    (1040, 1264, 48, 15), (1040, 1264, 100, 15), (1264, 1040, 48, 15),  # more than one workgroup per unit
])
def test_projections_split_along_the_reduction(mma, m, n, r, K):
    # Few rows (columns) of output: the reduction is split and the partial sums are added behind it, by
    # the projection itself or by the quantiser.  Stages of 64 that do not divide into the splits, a
    # last stage that is partial, every number of basis blocks.
    inp, deltas = _lowrank_inputs(m, n, r, K, seed=7 * m + n + r)
    d = dlcx.desc(m, n, r, 8, 16, mma)
    ws = ws_for(d, K + 1)  # a workspace sized for more workers serves fewer
    d_deltas = [to_dev(x) for x in deltas]
    p_hat = ref.orthonormalize(rng(r).standard_normal((r, m)).astype(np.float32))
    for phase, basis, L, want in ((dlcx.PHASE_P, inp.q_in, m, ref.project_p), (dlcx.PHASE_Q, p_hat, n, ref.project_q)):
        ws.fill_(255)  # NaN in whatever is not written
        outs = [torch.zeros(r, L, device=DEV) for _ in range(K)]
        dlcx.dlcx_project(d, phase, d_deltas, to_dev(basis), outs, ws)
        codes, scales = payload_buffers(d, phase, K)
        ws.fill_(255)
        dlcx.dlcx_compress_batched(d, phase, d_deltas, to_dev(basis), codes, scales, ws)
        factors = ws[: K * r * L * 4].view(torch.float32).view(K, r, L)
        for k in range(K):
            assert close(to_np(outs[k]), want(deltas[k], basis), TOL[mma]), (phase, k)
            assert torch.equal(factors[k], outs[k])  # the same additions in the same order
            cw, sw = ref.quantize(to_np(outs[k]), 8, 16)
            assert np.array_equal(to_np(codes[k]), cw)
            assert np.array_equal(to_np(scales[k]).view(np.uint32), sw.view(np.uint32))


@pytest.mark.parametrize("mma", [dlcx.MMA_F32, dlcx.MMA_BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("m,n,r,K", [
    (2064, 16, 16, 16), (2064, 80, 31, 16), (1776, 208, 12, 16), (4000, 144, 32, 9),  # one-role: 64 rows
    (2048, 4112, 20, 16), (2048, 4096, 20, 16),  # one workgroup for every unit: two-role if long, one-role if not
])
def test_project_p_of_one_basis_block_with_a_workgroup_per_unit(mma, m, n, r, K):
    # Ranks up to 32 and at least 224 workgroups of 128 rows: rows that do not divide into 64, one and
    # two stages of 64 columns, a stage that is partial, both sides of the rule between the kernels.
    g = torch.Generator(device=DEV)
    g.manual_seed(m + n)
    deltas = [torch.randn(m, n, generator=g, device=DEV) for _ in range(2)]
    basis = torch.randn(r, n, generator=g, device=DEV)
    d = dlcx.desc(m, n, r, 8, 16, mma)
    outs = [torch.full((r, m), float("nan"), device=DEV) for _ in range(K)]
    dlcx.dlcx_project(d, dlcx.PHASE_P, [deltas[k % 2] for k in range(K)], basis, outs, ws_for(d, K))
    for k in (0, 1):
        want = to_np(basis).astype(np.float64) @ to_np(deltas[k]).astype(np.float64).T
        assert close(to_np(outs[k]), want, TOL[mma]), k
    for k in range(2, K):
        assert torch.equal(outs[k], outs[k % 2]), k


@pytest.mark.parametrize("mma", [dlcx.MMA_FMA, dlcx.MMA_F32, dlcx.MMA_BF16, dlcx.MMA_F16],
                         ids=["fma", "f32", "bf16", "f16"])
@pytest.mark.parametrize("m,n,r,K,k", [(512, 8256, 16, 8, 7), (1024, 8720, 96, 4, 3), (8720, 528, 96, 4, 3)])
def test_fewer_workers_stay_inside_a_larger_workspace(mma, m, n, r, K, k):
    # Fewer workers may be split further (8 workers at 8256 columns not at all, 7 in two): the
    # bytes behind a workspace sized for K workers stay as they were when k of them are run.
    guard = 1 << 20
    size = dlcx.dlcx_workspace_bytes(dlcx.desc(m, n, r, 4, 16, mma), K)
    buf = torch.full((size + guard,), 165, device=DEV, dtype=torch.uint8)
    g = torch.Generator(device=DEV)
    g.manual_seed(r)
    delta = torch.randn(m, n, generator=g, device=DEV)
    d = dlcx.desc(m, n, r, 4, 16, mma)
    for phase, L in ((dlcx.PHASE_P, n), (dlcx.PHASE_Q, m)):
        basis = torch.randn(r, L, generator=g, device=DEV)
        codes, scales = payload_buffers(d, phase, k)
        dlcx.dlcx_compress_batched(d, phase, [delta] * k, basis, codes, scales, buf[:size])
        assert bool((buf[size:] == 165).all()), phase
        assert all(torch.equal(c, codes[0]) for c in codes) and bool((codes[0] != 0).any())


@pytest.mark.parametrize("m,n,r,K", [
    (16, 16, 16, 1), (48, 272, 17, 3), (272, 80, 31, 2),      # fewer steps than wavefronts, ragged tiles
    (1040, 208, 65, 1), (320, 336, 128, 2), (272, 528, 129, 1), (512, 256, 256, 1),
    (8208, 64, 20, 2), (8208, 80, 48, 2), (48, 128, 20, 1),   # two row blocks per wavefront in P; narrow
])
def test_fp64_products_at_tile_edges(m, n, r, K):
    # The fp64-accumulating form: products of fp32 values are exact and their sums carry 2^-53 per
    # addition, so P and the reconstruction are the 64-bit result rounded once (2^-24 relative).  Q is
    # rounded to fp32 in every slab (up to 64 of them), added up in fp64 and rounded once more: errors
    # of 2^-24 of each partial sum, which in norm are 2^-24 of the result for sums of random signs.
    g = rng(m + 3 * n + r)
    deltas = [g.standard_normal((m, n)).astype(np.float32) for _ in range(K)]
    p, q = g.standard_normal((r, m)).astype(np.float32), g.standard_normal((r, n)).astype(np.float32)
    d = dlcx.desc(m, n, r, 4, 16, dlcx.MMA_FMA)
    ws = ws_for(d, K)
    for phase, basis, L in ((dlcx.PHASE_P, q, m), (dlcx.PHASE_Q, p, n)):
        outs = [torch.zeros(r, L, device=DEV) for _ in range(K)]
        dlcx.dlcx_project(d, phase, [to_dev(x) for x in deltas], to_dev(basis), outs, ws)
        for k in range(K):
            x = deltas[k].astype(np.float64)
            want = basis.astype(np.float64) @ (x.T if phase == dlcx.PHASE_P else x)
            assert close(to_np(outs[k]), want, 2.0 ** -23), (phase, k)
    out = torch.zeros(m, n, device=DEV)
    dlcx.dlcx_decompress(d, to_dev(p), to_dev(q), out, workspace=ws)
    assert close(to_np(out), p.astype(np.float64).T @ q.astype(np.float64), 2.0 ** -23)


@pytest.mark.parametrize("steps", [1, 3, 5, 8, 9, 12, 13, 24, 25, 28, 48, 49, 50, 52, 53, 57, 61, 65, 69])
@pytest.mark.parametrize("m,r", [(48, 20), (4128, 9), (8224, 7), (16, 100), (32, 200)])
def test_fp64_products_over_every_length_of_the_operand_pipeline(m, r, steps):
    # Reductions of `steps` times 16: a wavefront's share is none, one, or any remainder of the two or three sets of
    # operands that it keeps (P: three from 49 on, but two with one basis block and more than 8192 rows; Q: two).
    # Tolerance as above.
    n = 16 * steps
    g = rng(m + r + steps)
    x = g.standard_normal((m, n)).astype(np.float32)
    b = g.standard_normal((r, n)).astype(np.float32)
    want = b.astype(np.float64) @ x.T.astype(np.float64)
    for phase, delta in ((dlcx.PHASE_P, x), (dlcx.PHASE_Q, np.ascontiguousarray(x.T))):
        d = dlcx.desc(*delta.shape, min(r, *delta.shape), 4, 16, dlcx.MMA_FMA)
        out = torch.zeros(d.r, m, device=DEV)
        dlcx.dlcx_project(d, phase, [to_dev(delta)], to_dev(b[: d.r]), [out], ws_for(d, 1))
        assert close(to_np(out), want[: d.r], 2.0 ** -23), phase


@pytest.mark.parametrize("steps", [32, 33, 34, 35, 36, 37, 40, 44, 48])
@pytest.mark.parametrize("r", [20, 50, 100, 200])
def test_fp64_q_projection_of_many_workers_over_long_reductions(r, steps):
    # 16 workers of 4112 columns leave the rows in one piece, and from more than 512 of them on a wavefront keeps
    # three sets of operands.  Tolerance as above.
    m, n, K = 16 * steps, 4112, 16
    g = rng(r + steps)
    x = g.standard_normal((m, n)).astype(np.float32)
    b = g.standard_normal((r, m)).astype(np.float32)
    d = dlcx.desc(m, n, r, 4, 16, dlcx.MMA_FMA)
    outs = [torch.zeros(r, n, device=DEV) for _ in range(K)]
    dlcx.dlcx_project(d, dlcx.PHASE_Q, [to_dev(x)] * K, to_dev(b), outs, ws_for(d, K))
    assert close(to_np(outs[0]), b.astype(np.float64) @ x.astype(np.float64), 2.0 ** -23)
    assert all(torch.equal(o, outs[0]) for o in outs)


@pytest.mark.parametrize("mma", MODES, ids=MODE_IDS)
@pytest.mark.parametrize("value", [np.nan, np.inf], ids=["nan", "inf"])
@pytest.mark.parametrize("m,n,r", [(48, 80, 17), (272, 144, 100)])
def test_what_is_not_finite_stays_in_its_row_and_column(mma, value, m, n, r):
    # Padding of tiles and lanes past the matrix must not meet a NaN or an infinity, and a product
    # with one reaches the outputs that contain it, no others.
    g = rng(m)
    delta = g.standard_normal((m, n)).astype(np.float32)
    p, q = g.standard_normal((r, m)).astype(np.float32), g.standard_normal((r, n)).astype(np.float32)
    i, j, c = m - 1, n - 1, r - 1
    d = dlcx.desc(m, n, r, 8, 16, mma)
    ws = ws_for(d, 1)

    def products(delta, p, q):
        P, Q, D = torch.zeros(r, m, device=DEV), torch.zeros(r, n, device=DEV), torch.zeros(m, n, device=DEV)
        dlcx.dlcx_project(d, dlcx.PHASE_P, [to_dev(delta)], to_dev(q), [P], ws)
        dlcx.dlcx_project(d, dlcx.PHASE_Q, [to_dev(delta)], to_dev(p), [Q], ws)
        dlcx.dlcx_decompress(d, to_dev(p), to_dev(q), D, workspace=ws)
        return to_np(P), to_np(Q), to_np(D)

    clean = products(delta, p, q)
    delta2, p2, q2 = delta.copy(), p.copy(), q.copy()
    delta2[i, j] = p2[c, i] = q2[c, j] = value
    hit = [np.zeros(x.shape, bool) for x in clean]
    hit[0][:, i] = hit[0][c, :] = True   # P = delta q: row i of delta, column c of the basis
    hit[1][:, j] = hit[1][c, :] = True
    hit[2][i, :] = hit[2][:, j] = True
    for got, want, h in zip(products(delta2, p2, q2), clean, hit):
        assert not np.isfinite(got[h]).any()
        assert np.isfinite(got[~h]).all()
        assert np.array_equal(got[~h], want[~h])


# ranks above 64 in the fp16 form: (Q only: few rows) / (P and Q: the two-role P kernel is used)
SHAPES_F16 = [(640, 2048, 96, 2, 128), (2048, 512, 256, 1, 64), (4096, 320, 200, 8, 64),
              (4112, 336, 72, 8, 16), (4112, 336, 130, 8, 16)]


@pytest.mark.parametrize("m,n,r,K,group", SHAPES_F16)
def test_project_p_and_q_fp16_form(m, n, r, K, group):
    test_project_p_and_q(dlcx.MMA_F16, m, n, r, K, group)


@pytest.mark.parametrize("n", [8176, 8192, 8208, 8256, 8320])
def test_project_p_fp16_form_with_three_stages_ahead(n):
    # From 8192 columns on the producers of the fp16 P projection at 8 basis blocks hold three stages: numbers of
    # stages of 64 columns that leave 0, 1 and 2 over, a ragged one, and the size before the line.  Operands
    # rounded to 11 bits once, sums in random order: 2^-12 x sqrt(2) of the result, twice that is allowed; the
    # rounding, about 2^-12 in the mean, has to show (the stand-by's result is an order closer), and with an
    # element out of range in the last stage the result has to be the stand-by's, that is the bf16 mode's.
    m, r, K = 4096, 130, 8
    g = torch.Generator(device=DEV)
    g.manual_seed(n)
    deltas = [1e-2 * torch.randn(m, n, generator=g, device=DEV) for _ in range(K)]
    basis = torch.randn(r, n, generator=g, device=DEV)

    def project(mma):
        out = [torch.zeros(r, m, device=DEV) for _ in range(K)]
        d = dlcx.desc(m, n, r, 4, 16, mma)
        dlcx.dlcx_project(d, dlcx.PHASE_P, deltas, basis, out, ws_for(d, K))
        return out

    for x, y in zip(deltas, project(dlcx.MMA_F16)):
        want = basis.double() @ x.double().T.contiguous()
        rms = want.square().mean().sqrt()
        assert 5e-5 <= float((y.double() - want).norm() / want.norm()) <= 7e-4
        assert float(((y.double() - want).abs() / torch.maximum(want.abs(), rms)).max()) <= 8 * 7e-4
    deltas[-1][m - 1, n - 1] = 1e3
    assert all(torch.equal(x, y) for x, y in zip(project(dlcx.MMA_F16), project(dlcx.MMA_BF16)))


def test_fp16_form_is_the_bf16_form_up_to_rank_64():
    m, n, r, K, group = 1024, 768, 64, 4, 128
    inp, deltas = _lowrank_inputs(m, n, r, K, seed=5)
    basis_q = rng(9).standard_normal((r, m)).astype(np.float32)
    outs = {}
    for mma in (dlcx.MMA_BF16, dlcx.MMA_F16):
        d = dlcx.desc(m, n, r, 4, group, mma)
        po = [torch.zeros(r, m, device=DEV) for _ in range(K)]
        qo = [torch.zeros(r, n, device=DEV) for _ in range(K)]
        dd = [to_dev(x) for x in deltas]
        dlcx.dlcx_project(d, dlcx.PHASE_P, dd, to_dev(inp.q_in), po, ws_for(d, K))
        dlcx.dlcx_project(d, dlcx.PHASE_Q, dd, to_dev(basis_q), qo, ws_for(d, K))
        outs[mma] = [to_np(x) for x in po + qo]
    for a, b in zip(outs[dlcx.MMA_BF16], outs[dlcx.MMA_F16]):
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))


@pytest.mark.parametrize("case", ["in-range", "huge-element", "tiny", "zero"])
def test_fp16_form_stands_by_outside_its_range(case):
    """The fp16 launch records the largest |delta|; outside [2^-14, 15.99) the stand-by launch
    redoes the projection in the bf16 arithmetic, so the result is then that of DLCX_MMA_BF16 bit
    for bit -- a single element of 1e3 among values of 1e-3, a matrix of values around 1e-9, an
    all-zero matrix.  In range, the result is the fp16 one (close to, not equal to, the bf16 one)."""
    m, n, r, K, group = 4096, 320, 200, 8, 64
    inp, deltas = _lowrank_inputs(m, n, r, K, seed=77)
    if case == "huge-element":
        deltas[3][1234, 77] = 1.0e3
    elif case == "tiny":
        deltas = [(x * 1e-7).astype(np.float32) for x in deltas]
    elif case == "zero":
        deltas = [np.zeros_like(x) for x in deltas]
    d_deltas = [to_dev(x) for x in deltas]
    p_hat = ref.orthonormalize(ref.project_p(deltas[0] if case != "zero" else inp.theta_g, inp.q_in))
    res = {}
    for mma in (dlcx.MMA_BF16, dlcx.MMA_F16):
        d = dlcx.desc(m, n, r, 4, group, mma)
        ws = ws_for(d, K)
        po = [torch.zeros(r, m, device=DEV) for _ in range(K)]
        qo = [torch.zeros(r, n, device=DEV) for _ in range(K)]
        dlcx.dlcx_project(d, dlcx.PHASE_P, d_deltas, to_dev(inp.q_in), po, ws)
        dlcx.dlcx_project(d, dlcx.PHASE_Q, d_deltas, to_dev(p_hat), qo, ws)
        res[mma] = [to_np(x) for x in po + qo]
    same = all(np.array_equal(a.view(np.uint32), b.view(np.uint32))
               for a, b in zip(res[dlcx.MMA_BF16], res[dlcx.MMA_F16]))
    if case == "in-range":
        assert not same
        for a, b in zip(res[dlcx.MMA_BF16], res[dlcx.MMA_F16]):
            assert close(b, a, TOL[dlcx.MMA_F16])
        want = ref.project_q(deltas[2], p_hat)
        assert close(res[dlcx.MMA_F16][K + 2], want, TOL[dlcx.MMA_F16])
    else:
        assert same
        if case != "zero":
            want = ref.project_q(deltas[3], p_hat)
            assert rel_l2(res[dlcx.MMA_F16][K + 3], want) <= TOL[dlcx.MMA_BF16]


@pytest.mark.parametrize("m,n,r,K", [(4096, 320, 200, 8), (2064, 1296, 100, 3), (3072, 3072, 140, 1)])
@pytest.mark.parametrize("huge", [False, True], ids=["in-range", "stand-by"])
def test_fp16_form_and_its_stand_by_are_split_each_in_its_own_way(m, n, r, K, huge):
    """The two launches leave different numbers of partial sums; the quantiser and the sum behind a
    projection read from the record how many count."""
    g = torch.Generator(device=DEV)
    g.manual_seed(m + r)
    deltas = [0.1 * torch.randn(m, n, generator=g, device=DEV) for _ in range(K)]
    if huge:
        deltas[K - 1][m - 1, n - 1] = 1.0e3
    for phase, L, lb in ((dlcx.PHASE_P, m, n), (dlcx.PHASE_Q, n, m)):
        basis = torch.randn(r, lb, generator=g, device=DEV)
        got = {}
        for mma in (dlcx.MMA_BF16, dlcx.MMA_F16):
            d = dlcx.desc(m, n, r, 8, 16, mma)
            ws = ws_for(d, K)
            outs = [torch.empty(r, L, device=DEV) for _ in range(K)]
            ws.fill_(255)
            dlcx.dlcx_project(d, phase, deltas, basis, outs, ws)
            codes, scales = payload_buffers(d, phase, K)
            ws.fill_(255)
            dlcx.dlcx_compress_batched(d, phase, deltas, basis, codes, scales, ws)
            factors = ws[: K * r * L * 4].view(torch.float32).view(K, r, L)
            assert all(torch.equal(factors[k], outs[k]) for k in range(K)), (phase, mma)
            got[mma] = outs, codes
        for k in range(K):
            want = to_np(basis.double() @ (deltas[k].double().T if phase == dlcx.PHASE_P else deltas[k].double()).contiguous())
            assert close(to_np(got[dlcx.MMA_F16][0][k]), want, TOL[dlcx.MMA_BF16 if huge else dlcx.MMA_F16])
            if huge:
                assert all(torch.equal(a[k], b[k]) for a, b in zip(got[dlcx.MMA_BF16], got[dlcx.MMA_F16])), (phase, k)


@pytest.mark.parametrize("mma", MODES, ids=MODE_IDS)
@pytest.mark.parametrize("m,n,r,K,group", SHAPES)
def test_decompress_and_error_buffer(mma, m, n, r, K, group):
    g = rng(m * 3 + n)
    p_hat = ref.orthonormalize(g.standard_normal((r, m)).astype(np.float32))
    q_bar = (g.standard_normal((r, n)) * np.arange(1, r + 1)[:, None] ** -1.0).astype(np.float32)
    deltas = [g.standard_normal((m, n)).astype(np.float32) * 0.1 for _ in range(K)]
    want = ref.reconstruct(p_hat, q_bar)
    want_e = [ref.ef_update(x.copy().reshape(-1), want.reshape(-1)).reshape(m, n) for x in deltas]
    d = dlcx.desc(m, n, r, 4, group, mma)
    out = torch.zeros(m, n, device=DEV)
    efs = [to_dev(x) for x in deltas]
    ws = ws_for(d, max(K, 1))
    dlcx.dlcx_decompress(d, to_dev(p_hat), to_dev(q_bar), out, efs, workspace=ws)
    assert close(to_np(out), want, TOL[mma])
    for k in range(K):
        # e = delta - delta_hat: compare the correction, not the (larger) buffer
        assert close(deltas[k] - to_np(efs[k]), deltas[k] - want_e[k], TOL[mma])
    # error buffers only (no materialised delta_hat) gives the same buffers
    efs2 = [to_dev(x) for x in deltas]
    dlcx.dlcx_decompress(d, to_dev(p_hat), to_dev(q_bar), None, efs2, workspace=ws)
    for k in range(K):
        assert torch.equal(efs2[k], efs[k])
    # fused with the outer update: same error buffers, and (theta, v) as the separate kernels give
    g2 = rng(7)
    th = (0.02 * g2.standard_normal((m, n))).astype(np.float32)
    v = (1e-3 * g2.standard_normal((m, n))).astype(np.float32)
    th_w, v_w = th.copy(), v.copy()
    ref.outer_nesterov(th_w.reshape(-1), v_w.reshape(-1), want.reshape(-1), synth.LR, synth.MU)
    efs3 = [to_dev(x) for x in deltas]
    d_th, d_v = to_dev(th), to_dev(v)
    dlcx.dlcx_decompress_apply(d, to_dev(p_hat), to_dev(q_bar), efs3, d_th, d_v, synth.LR, synth.MU,
                               workspace=ws)
    for k in range(K):
        assert torch.equal(efs3[k], efs[k])
    assert close(th - to_np(d_th), th - th_w, TOL[mma])
    assert close(to_np(d_v), v_w, TOL[mma])


# ------------------------------------------------------------------ compress = project + quantise
@pytest.mark.parametrize("mma", MODES, ids=MODE_IDS)
@pytest.mark.parametrize("qbits", [4, 8])
def test_compress_codes_are_the_quantiser_of_its_own_factor(mma, qbits):
    m, n, r, K, group = 1024, 768, 32, 3, 128
    inp, deltas = _lowrank_inputs(m, n, r, K, seed=99)
    d = dlcx.desc(m, n, r, qbits, group, mma)
    ws = ws_for(d, K)
    for phase, basis, L in ((dlcx.PHASE_P, inp.q_in, m),
                            (dlcx.PHASE_Q, ref.orthonormalize(rng(1).standard_normal((r, m)).astype(np.float32)), n)):
        codes, scales = payload_buffers(d, phase, K)
        dlcx.dlcx_compress_batched(d, phase, [to_dev(x) for x in deltas], to_dev(basis), codes, scales, ws)
        torch.cuda.synchronize()
        factors = to_np(ws[: K * r * L * 4].view(torch.float32)).reshape(K, r, L)
        for k in range(K):
            want_f = (ref.project_p if phase == dlcx.PHASE_P else ref.project_q)(deltas[k], basis)
            assert close(factors[k], want_f, TOL[mma])
            cw, sw = ref.quantize(factors[k], qbits, group)   # oracle quantiser on the GPU's factor
            assert np.array_equal(to_np(codes[k]), cw)
            assert np.array_equal(to_np(scales[k]).view(np.uint32), sw.view(np.uint32))
        # the single-worker entry point writes the same payload
        c1, s1 = payload_buffers(d, phase, 1)
        dlcx.dlcx_compress(d, phase, to_dev(deltas[1]), to_dev(basis), c1[0], s1[0], ws)
        assert torch.equal(c1[0], codes[1]) and torch.equal(s1[0], scales[1])


# ------------------------------------------------------------------ orthonormalisation
@pytest.mark.parametrize("L,r", [(64, 1), (512, 8), (528, 5), (2048, 64), (1040, 33), (4096, 128),
                                  (1024, 200), (2048, 256)])
def test_orthonormalize_matches_oracle(L, r):
    g = rng(L + r)
    # columns with very different norms and a decaying spectrum (warm-started basis)
    U = synth.orthonormal_columns(g, L, r)
    W = synth.orthonormal_columns(g, r, r)
    s = np.arange(1, r + 1, dtype=np.float64) ** -1.5
    A = ((U * s) @ W.T * (np.arange(1, r + 1) ** -2.0)).T.astype(np.float32)
    A = np.ascontiguousarray(A)
    want = ref.orthonormalize(A)
    d_A = to_dev(A)
    ws = torch.empty(dlcx.dlcx_workspace_bytes(dlcx.desc(L, L, r, 4, 16), 1), device=DEV, dtype=torch.uint8)
    dlcx.dlcx_orthonormalize(L, r, d_A, ws)
    got = to_np(d_A).astype(np.float64)
    assert np.abs(got @ got.T - np.eye(r)).max() <= 1e-5
    cond = np.linalg.cond(A.astype(np.float64))
    assert rel_l2(got, want) <= max(1e-5, 4e-7 * cond), cond


@pytest.mark.parametrize("L,r", [(16, 16), (32, 17), (528, 15), (1040, 32), (2064, 33), (512, 80),
                                  (656, 81), (1536, 144), (1040, 145), (1024, 255), (272, 256)])
@pytest.mark.parametrize("cond", [3.0, 1e5])
def test_orthonormalize_block_edges_both_rounds(L, r, cond):
    # Ranks around the edges of the 16 x 16 blocks and of the launch shapes, lengths around those
    # of the 512-element sums and 64-element tiles.  cond 3: the first round is enough and the
    # second returns at once; cond 1e5: both run.  All sums are in 64 bits, so what is left is the
    # rounding to fp32 after each round: 2^-24 of every element, at most 2 x 2^-24 in norm, times
    # the 1 + cond 2^-53 ... of the 64-bit steps; twice that is allowed.
    g = rng(L * 7 + r)
    U = synth.orthonormal_columns(g, L, r)
    W = synth.orthonormal_columns(g, r, r)
    A = np.ascontiguousarray(((U * np.logspace(0, -np.log10(cond), r)) @ W.T).T.astype(np.float32))
    q, t = np.linalg.qr(A.T.astype(np.float64))
    want = (q * np.sign(np.diag(t))).T
    d_A = to_dev(A)
    ws = torch.empty(dlcx.dlcx_workspace_bytes(dlcx.desc(L, L, r, 4, 16), 1), device=DEV, dtype=torch.uint8)
    dlcx.dlcx_orthonormalize(L, r, d_A, ws)
    assert rel_l2(to_np(d_A), want) <= 2.4e-7


@pytest.mark.parametrize("L,r", [(64, 1), (272, 20), (1040, 33), (528, 100), (1024, 256)])
@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf], ids=["nan", "inf", "-inf"])
def test_orthonormalize_leaves_the_columns_before_one_that_is_not_finite(L, r, value):
    # Column c of a thin QR hangs on the columns up to c alone: those before the first column that is
    # not finite are what they are without the rest, that column and those after it are NaN.
    g = rng(L + r)
    A = g.standard_normal((r, L)).astype(np.float32)
    ws = torch.empty(dlcx.dlcx_workspace_bytes(dlcx.desc(L, L, r, 4, 16), 1), device=DEV, dtype=torch.uint8)
    for col in sorted({0, r // 3, 17 * r // 20, r - 1}):
        B = A.copy()
        B[col, L // 2] = value
        B[r - 1, 0] = np.nan if col < r - 1 else B[r - 1, 0]
        d_B = to_dev(B)
        dlcx.dlcx_orthonormalize(L, r, d_B, ws)
        got = to_np(d_B)
        assert np.isnan(got[col:]).all(), col
        if col:
            q, t = np.linalg.qr(A[:col].T.astype(np.float64))
            assert rel_l2(got[:col], (q * np.sign(np.diag(t))).T) <= 2.4e-7, col


@pytest.mark.parametrize("L,r", [(16, 1), (16, 16), (48, 3), (512, 8), (528, 15), (1024, 16), (1040, 9), (1520, 16),
                                 (1536, 16), (2048, 7), (2064, 2)])
@pytest.mark.parametrize("cond", [3.0, 1e5])
def test_small_factors_alone_and_in_a_batch_with_large_ones(L, r, cond):
    # A batch of factors of at most 16 columns that fit in LDS is orthonormalised, and measured, by one launch; in
    # a batch with a larger one they take the general kernels.  Same sums in the same order: the same bits; and
    # against a 64-bit QR what is left is the rounding to fp32 after each round, as above.
    g = rng(L * 5 + r)
    U, W = synth.orthonormal_columns(g, L, r), synth.orthonormal_columns(g, r, r)
    A = np.ascontiguousarray(((U * np.logspace(0, -np.log10(cond), r)) @ W.T).T.astype(np.float32))
    big = g.standard_normal((20, 64)).astype(np.float32)
    descs = [dlcx.desc(L, L, r, 4, 16), dlcx.desc(64, 64, 20, 4, 16)]
    ws = torch.empty(dlcx.dlcx_batched_workspace_bytes(descs), device=DEV, dtype=torch.uint8)
    got, ranks = [], []
    for n in (1, 2):
        f, out = [to_dev(A), to_dev(big)][:n], torch.full((2,), -1, device=DEV, dtype=torch.int32)
        dlcx.dlcx_effective_rank_batched(descs[:n], f, 0.999, out, ws)
        dlcx.dlcx_orthonormalize_batched(descs[:n], f, ws)
        got.append(to_np(f[0]))
        ranks.append(int(out[0].item()))
    assert np.array_equal(got[0].view(np.uint32), got[1].view(np.uint32))
    assert ranks[0] == ranks[1] == ref.effective_rank(A, 0.999)
    q, t = np.linalg.qr(A.T.astype(np.float64))
    assert rel_l2(got[0], (q * np.sign(np.diag(t))).T) <= 2.4e-7


@pytest.mark.parametrize("r", [2, 9, 16])
def test_small_factors_take_the_second_round_alone_or_in_a_batch(r):
    # Whether the second round runs hangs on ||R^-1||_F^2 of the unit-diagonal Gram matrix (4e6 is the line): two
    # columns at an angle of e put 2 / e^2 there.  Up to rank 16 it is one wavefront's sum in every form, so factors
    # on either side of the line, and as close to it as fp32 inputs get, have the same bits alone and in a batch.
    L, n = 512, 24
    g = rng(r)
    Q = synth.orthonormal_columns(g, L, r + 1).T
    big = g.standard_normal((20, 64)).astype(np.float32)
    angles = np.sqrt(2.0 / 4e6) * (1 + 2.0 ** -np.arange(2, n + 2) * np.where(np.arange(n) % 2, 1, -1))
    for e in angles:
        A = Q[:r].copy()
        A[r - 1] = Q[0] * np.cos(e) + Q[r] * np.sin(e)
        A = A.astype(np.float32)
        descs = [dlcx.desc(L, L, r, 4, 16), dlcx.desc(64, 64, 20, 4, 16)]
        ws = torch.empty(dlcx.dlcx_batched_workspace_bytes(descs), device=DEV, dtype=torch.uint8)
        alone, batch = [to_dev(A)], [to_dev(A), to_dev(big)]
        dlcx.dlcx_orthonormalize_batched(descs[:1], alone, ws)
        dlcx.dlcx_orthonormalize_batched(descs, batch, ws)
        assert torch.equal(alone[0], batch[0]), e


@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_small_factor_that_is_not_finite_or_has_no_rank(value):
    L, r = 528, 12
    A = rng(77).standard_normal((r, L)).astype(np.float32)
    A[3] = 0.0
    A[6] = 2.0 * A[1]
    ws = torch.empty(dlcx.dlcx_workspace_bytes(dlcx.desc(L, L, r, 4, 16), 1), device=DEV, dtype=torch.uint8)
    d_A = to_dev(A)
    dlcx.dlcx_orthonormalize(L, r, d_A, ws)
    want = to_np(d_A)
    assert not want[3].any() and not want[6].any()
    assert rel_l2(want, ref.orthonormalize(A)) <= 1e-5
    A[9, 100] = value
    d_A = to_dev(A)
    dlcx.dlcx_orthonormalize(L, r, d_A, ws)
    got = to_np(d_A)
    assert np.isnan(got[9:]).all() and rel_l2(got[:9], want[:9]) <= 2.4e-7


@pytest.mark.parametrize("r", [65, 240, 241, 256])
def test_sturm_table_ends_behind_all_that_is_read_of_it(r):
    # Above rank 64 the eigenvalues are found from a table in the workspace, read in whole blocks of 16 terms and
    # half a block further while other wavefronts write their eigenvalues there: all that is read has to be terms,
    # those past the matrix (4, 0), and none of them an eigenvalue.
    L = 256
    A = rng(r).standard_normal((r, L)).astype(np.float32)
    ws = torch.full((dlcx.dlcx_workspace_bytes(dlcx.desc(L, L, r, 4, 16), 1),), 165, device=DEV, dtype=torch.uint8)
    out = torch.zeros(1, device=DEV, dtype=torch.int32)
    dlcx.dlcx_effective_rank(L, r, to_dev(A), 1.0, out, ws)
    g = to_np(ws)[(r * r + 1) // 2 * 16:].view(np.float64)  # behind the partial sums, one chunk
    last = (r + 15) // 16 * 16 + 8
    table = g[:2 * last].reshape(last, 2)
    assert (np.abs(table[:r, 0]) <= 1).all() and (table[:r, 1] <= 0).all()
    assert (table[r:] == (4.0, 0.0)).all()
    assert int(out.item()) == r


@pytest.mark.parametrize("L,r", [
    (8192, 8), (7696, 16), (3600, 17), (4112, 24), (8192, 32), (3088, 33), (2048, 64), (1024, 90),  # 16 .. 2 chunks,
    (8208, 32), (2064, 64), (1040, 90),  # .. added up by the kernels that use them; past the lines: beforehand
])
def test_sums_over_many_chunks(L, r):
    # The partial sums of 512 elements each are requested several at a time.  Most of row k lies in chunk k modulo
    # their number: a sum that is left out or counted twice takes or doubles whole rows.
    g = rng(L + 11 * r)
    chunks = -(-L // 512)
    A = 0.1 * g.standard_normal((r, L))
    for k in range(r):
        c = k % chunks
        A[k, 512 * c: 512 * c + 512] += g.standard_normal(min(512, L - 512 * c))
    A = np.ascontiguousarray((A * np.arange(1, r + 1)[:, None] ** -0.3).astype(np.float32))
    ws = torch.empty(dlcx.dlcx_workspace_bytes(dlcx.desc(L, L, r, 4, 16), 1), device=DEV, dtype=torch.uint8)
    out = torch.full((1,), -1, device=DEV, dtype=torch.int32)
    d_A = to_dev(A)
    for tau in np.arange(0.05, 1.0, 0.1):
        dlcx.dlcx_effective_rank(L, r, d_A, tau, out, ws)
        assert int(out.item()) == ref.effective_rank(A, tau), tau
    dlcx.dlcx_orthonormalize(L, r, d_A, ws)
    q, t = np.linalg.qr(A.T.astype(np.float64))
    assert rel_l2(to_np(d_A), (q * np.sign(np.diag(t))).T) <= 2.4e-7


@pytest.mark.parametrize("L,ranks", [
    (1040, [20, 3, 33]),                  # equal lengths: a row of the grid each
    (4096, [33, 20, 64, 7, 40, 33, 33, 33]),    # .. of whole groups of eight chunks
    (5120, [33, 40, 17, 64, 33, 33, 130]),      # 70 chunks, not in groups of eight: looked up
    (36880, [17]),                        # a row that ends within a group
])
def test_batches_of_equal_lengths_are_their_factors_one_by_one(L, ranks):
    g = rng(L)
    descs = [dlcx.desc(L, L, r, 4, 16) for r in ranks]
    ws = torch.empty(dlcx.dlcx_batched_workspace_bytes(descs), device=DEV, dtype=torch.uint8)
    A = [g.standard_normal((r, L)).astype(np.float32) for r in ranks]
    f, out = [to_dev(a) for a in A], torch.zeros(len(ranks), device=DEV, dtype=torch.int32)
    dlcx.dlcx_effective_rank_batched(descs, f, 0.9, out, ws)
    dlcx.dlcx_orthonormalize_batched(descs, f, ws)
    for i, r in enumerate(ranks):
        one, alone = torch.zeros(1, device=DEV, dtype=torch.int32), to_dev(A[i])
        dlcx.dlcx_effective_rank(L, r, alone, 0.9, one, ws)
        dlcx.dlcx_orthonormalize(L, r, alone, ws)
        assert torch.equal(alone, f[i]) and int(one.item()) == int(out[i].item()), i
        q, t = np.linalg.qr(A[i].T.astype(np.float64))
        assert rel_l2(to_np(f[i]), (q * np.sign(np.diag(t))).T) <= 2.4e-7, i
        assert int(out[i].item()) == ref.effective_rank(A[i], 0.9), i


def test_a_very_long_factor_in_a_batch_with_one_of_large_rank():
    # The launches have as many workgroups as the long factor has chunks, each as many threads as the high rank
    # asks for, more than 2^32 threads together: the Gram sums of r' and of the orthonormalisation, and P W.
    L = (1 << 29) + 16
    descs = [dlcx.desc(L, L, 1, 4, 16), dlcx.desc(256, 256, 256, 4, 16)]
    ws = torch.empty(dlcx.dlcx_batched_workspace_bytes(descs), device=DEV, dtype=torch.uint8)
    g = torch.Generator(device=DEV)
    g.manual_seed(29)
    f = [torch.randn(1, L, generator=g, device=DEV), torch.randn(256, 256, generator=g, device=DEV)]
    want = f[0] / torch.linalg.vector_norm(f[0], dtype=torch.float64)
    small = f[1].clone()
    out = torch.zeros(2, device=DEV, dtype=torch.int32)
    dlcx.dlcx_effective_rank_batched(descs, f, 1.0, out, ws)
    dlcx.dlcx_orthonormalize_batched(descs, f, ws)
    dlcx.dlcx_orthonormalize_batched(descs[1:], [small], ws)
    assert out.tolist() == [1, 256]
    assert float(torch.linalg.vector_norm(f[0] - want)) <= 2.4e-7  # the rounding to fp32, as above
    assert torch.equal(f[1], small)


def test_orthonormalize_degenerate_columns():
    L, r = 256, 6
    g = rng(3)
    A = g.standard_normal((r, L)).astype(np.float32)
    A[1] = 0.0
    A[4] = -3.0 * A[2]
    want = ref.orthonormalize(A)
    d_A = to_dev(A)
    ws = torch.empty(dlcx.dlcx_workspace_bytes(dlcx.desc(L, L, r, 4, 16), 1), device=DEV, dtype=torch.uint8)
    dlcx.dlcx_orthonormalize(L, r, d_A, ws)
    got = to_np(d_A)
    assert np.all(got[1] == 0) and np.all(got[4] == 0)
    assert rel_l2(got, want) <= 1e-5
    z = torch.zeros(3, L, device=DEV)
    dlcx.dlcx_orthonormalize(L, 3, z, ws)
    assert not to_np(z).any()


# ------------------------------------------------------------------ effective rank
@pytest.mark.parametrize("alpha,want", [(0.5, 241), (1.0, 49), (2.0, 3)])
def test_effective_rank_prescribed_spectra(alpha, want):
    n, r = 512, 256
    V = synth.orthonormal_columns(rng(1), n, r)
    W = synth.orthonormal_columns(rng(2), r, r)          # rotate: Gram is dense
    sig = np.arange(1, r + 1, dtype=np.float64) ** (-alpha)
    q_bar = np.ascontiguousarray(((V * sig) @ W.T).T.astype(np.float32))
    assert ref.effective_rank(q_bar, 0.99) == want
    out = torch.zeros(1, device=DEV, dtype=torch.int32)
    ws = torch.empty(dlcx.dlcx_workspace_bytes(dlcx.desc(n, n, r, 4, 16), 1), device=DEV, dtype=torch.uint8)
    dlcx.dlcx_effective_rank(n, r, to_dev(q_bar), 0.99, out, ws)
    assert int(out.item()) == want


@pytest.mark.parametrize("n,r", [(64, 1), (128, 7), (528, 33), (1024, 64), (768, 128), (512, 129),
                                 (512, 130), (1024, 192), (512, 255), (768, 256)])
def test_effective_rank_random_and_zero(n, r):
    g = rng(n + r)
    q = (g.standard_normal((r, n)) * (np.arange(1, r + 1)[:, None] ** -1.2)).astype(np.float32)
    ws = torch.empty(dlcx.dlcx_workspace_bytes(dlcx.desc(n, n, r, 4, 16), 1), device=DEV, dtype=torch.uint8)
    out = torch.full((1,), -1, device=DEV, dtype=torch.int32)
    for tau in (0.5, 0.9, 0.99, 1.0):
        dlcx.dlcx_effective_rank(n, r, to_dev(q), tau, out, ws)
        assert int(out.item()) == ref.effective_rank(q, tau), tau
    dlcx.dlcx_effective_rank(n, r, torch.zeros(r, n, device=DEV), 0.99, out, ws)
    assert int(out.item()) == 0
    if r >= 8:  # rank-deficient Gram: repeated, zero and low-rank columns
        q2 = q.copy()
        q2[5] = q2[3]
        q2[6] = 0.0
        q2[r // 2:] = (g.standard_normal((r - r // 2, 3)) @ g.standard_normal((3, n))).astype(np.float32)
        for tau in (0.9, 0.999, 1.0):
            dlcx.dlcx_effective_rank(n, r, to_dev(q2), tau, out, ws)
            want = ref.effective_rank(q2, tau)
            # at tau = 1 the count depends on eigenvalues at rounding level: not compared
            if tau < 1.0:
                assert int(out.item()) == want, tau


@pytest.mark.parametrize("r", [2, 3, 15, 16, 17, 48, 63, 65, 127, 191, 193, 240, 254])
@pytest.mark.parametrize("kind", ["dense", "diagonal", "blocks"])
def test_effective_rank_tile_edges_and_decoupled_rows(r, kind):
    # Ranks around the edges of the 16 x 16 tiles and of the launch shapes.  "diagonal": columns
    # with disjoint supports (S is diagonal bit for bit, no row is ever reflected, eigenvalues
    # coincide); "blocks": half of the rows decoupled from the rest, with equal columns among them.
    n = 768 if r <= 254 else 1024
    g = rng(31 * r + len(kind))
    q = (g.standard_normal((r, n)) * (np.arange(1, r + 1)[:, None] ** -0.8)).astype(np.float32)
    if kind == "diagonal":
        q = np.zeros((r, n), np.float32)
        for c in range(r):
            q[c, 3 * c: 3 * c + 3] = np.float32(2.0 ** -(c // 7))
    elif kind == "blocks":
        h = r // 2
        q[:h, n // 2:] = 0.0
        q[h:, : n // 2] = 0.0
        q[h:] = q[h]
    ws = torch.empty(dlcx.dlcx_workspace_bytes(dlcx.desc(n, n, r, 4, 16), 1), device=DEV, dtype=torch.uint8)
    out = torch.full((1,), -1, device=DEV, dtype=torch.int32)
    for tau in (0.3, 0.9, 0.99, 0.9999):
        dlcx.dlcx_effective_rank(n, r, to_dev(q), tau, out, ws)
        assert int(out.item()) == ref.effective_rank(q, tau), tau


@pytest.mark.parametrize("r,norms2", [
    (32, [1] * 18 + [0] * 13 + [9]), (64, [1] * 18 + [0] * 45 + [5]), (64, [5] + [1] * 41 + [0] * 22),
    (100, [1] * 18 + [65] + [0] * 81), (250, [1] * 101 + [65] + [0] * 148),
])
def test_effective_rank_on_runs_of_equal_decoupled_rows(r, norms2):
    # S is diagonal, the largest element G + 1 times the others for the G points that a round of the
    # multisection takes (4, 8, 64): the first point is the repeated eigenvalue to the last bit, and
    # every other term of the Sturm sequence there is exactly zero.  (No share of the trace falls on a whole
    # number of eigenvalues.)
    n = 768
    q = np.zeros((r, n), np.float32)
    for c, x in enumerate(norms2):  # x = a^2 + b^2 + ..: small integers, squares and sums are exact
        for k in range(3):
            a = int(np.sqrt(x))
            q[c, 3 * c + k] = a
            x -= a * a
        assert x == 0
    ws = torch.empty(dlcx.dlcx_workspace_bytes(dlcx.desc(n, n, r, 4, 16), 1), device=DEV, dtype=torch.uint8)
    out = torch.full((1,), -1, device=DEV, dtype=torch.int32)
    for tau in (0.3, 0.6, 0.9, 0.99):
        dlcx.dlcx_effective_rank(n, r, to_dev(q), tau, out, ws)
        assert int(out.item()) == ref.effective_rank(q, tau), tau


@pytest.mark.parametrize("r", [1, 2, 5, 8, 17, 24, 31, 32, 33, 40, 55, 64, 65, 100, 129, 200, 256])
def test_effective_rank_counts_no_zero_column_at_tau_one(r):
    # Exactly zero columns (what the orthonormalisation makes of dead ones, and Q_bar inherits) hold
    # no share of the trace: at tau = 1 r' is the number of the others, wherever they stand.
    n = 512
    g = rng(r)
    ws = torch.empty(dlcx.dlcx_workspace_bytes(dlcx.desc(n, n, r, 4, 16), 1), device=DEV, dtype=torch.uint8)
    out = torch.full((1,), -1, device=DEV, dtype=torch.int32)
    for trial in range(12):
        q = (g.standard_normal((r, n)) * (np.arange(1, r + 1)[:, None] ** -0.7)).astype(np.float32)
        dead = g.permutation(r)[: g.integers(0, r + 1)] if trial else np.arange(1, r)
        q[dead] = 0.0
        dlcx.dlcx_effective_rank(n, r, to_dev(q), 1.0, out, ws)
        assert int(out.item()) == r - len(dead), (trial, sorted(dead))
        for tau in (0.9, 0.99):
            dlcx.dlcx_effective_rank(n, r, to_dev(q), tau, out, ws)
            assert int(out.item()) == ref.effective_rank(q, tau), (trial, tau)
    dlcx.dlcx_effective_rank(n, r, torch.zeros(r, n, device=DEV), 1.0, out, ws)
    assert int(out.item()) == 0


@pytest.mark.parametrize("r", [16, 31, 60, 120, 250])
def test_effective_rank_at_tau_one_stops_where_the_sum_does(r):
    # Orthogonal columns with squared norms 4^-k: their sum in 64 bits, largest first, ends with
    # 4^-26 (4^-27 = 2^-54 is less than half a unit in the last place of 4 / 3).
    n = 256
    q = np.zeros((r, n), np.float32)
    q[np.arange(r), np.arange(r)] = 2.0 ** -np.minimum(np.arange(r), 60.0)
    ws = torch.empty(dlcx.dlcx_workspace_bytes(dlcx.desc(n, n, r, 4, 16), 1), device=DEV, dtype=torch.uint8)
    out = torch.full((1,), -1, device=DEV, dtype=torch.int32)
    dlcx.dlcx_effective_rank(n, r, to_dev(q), 1.0, out, ws)
    assert int(out.item()) == min(r, 27) == ref.effective_rank(q, 1.0)


@pytest.mark.parametrize("r", [3, 4, 7, 8, 14, 16, 18, 30, 32, 34, 47, 62, 64, 66, 127, 128, 190, 191, 255, 256])
@pytest.mark.parametrize("kind", ["dense", "equal"])
def test_effective_rank_where_a_share_is_reached_by_a_hair(r, kind):
    # tau 1e-9 below and above the share of the j largest eigenvalues: eigenvalues to 2^-56 (of sums of at most 256)
    # tell on which side it falls, the bounds before them (2^-19 .. 2^-23 up to rank 64, 2^-29 above) as a rule do not.
    # "equal": all but two eigenvalues coincide, with room around them in the interval that the search starts from.
    n = 512
    q = (rng(7 * r).standard_normal((r, n)) * (np.arange(1, r + 1)[:, None] ** -0.6)).astype(np.float32)
    if kind == "equal":
        q = np.zeros((r, n), np.float32)
        q[np.arange(r), np.arange(r)] = 1.0
        q[0, 0], q[1, 0] = 2.0, 0.5
    s = np.cumsum(np.linalg.eigvalsh(q.astype(np.float64) @ q.T.astype(np.float64))[::-1])
    ws = torch.empty(dlcx.dlcx_workspace_bytes(dlcx.desc(n, n, r, 4, 16), 1), device=DEV, dtype=torch.uint8)
    out = torch.full((1,), -1, device=DEV, dtype=torch.int32)
    for j in sorted({1, r // 3, r // 2, r - 1}):
        for tau, want in ((s[j - 1] / s[-1] - 1e-9, j), (s[j - 1] / s[-1] + 1e-9, j + 1)):
            dlcx.dlcx_effective_rank(n, r, to_dev(q), tau, out, ws)
            assert int(out.item()) == want == ref.effective_rank(q, tau), (j, tau)


@pytest.mark.parametrize("r,live", [(66, 1), (100, 31), (100, 33), (128, 64), (128, 65), (129, 66), (130, 80),
                                    (192, 81), (193, 96), (250, 97), (256, 128), (256, 193)])
def test_effective_rank_where_one_wavefront_takes_the_last_rows(r, live):
    # Above rank 64 the last 64 of the columns that are not zero are left to one wavefront: none, one or many before
    # them, and fewer than 64 in all.
    n = 512
    g = rng(r * live)
    q = (g.standard_normal((r, n)) * (np.arange(1, r + 1)[:, None] ** -0.6)).astype(np.float32)
    q[g.permutation(r)[live:]] = 0.0
    ws = torch.empty(dlcx.dlcx_workspace_bytes(dlcx.desc(n, n, r, 4, 16), 1), device=DEV, dtype=torch.uint8)
    out = torch.full((1,), -1, device=DEV, dtype=torch.int32)
    for tau in (0.3, 0.9, 0.99, 0.9999):
        dlcx.dlcx_effective_rank(n, r, to_dev(q), tau, out, ws)
        assert int(out.item()) == ref.effective_rank(q, tau), tau


@pytest.mark.parametrize("r", [128, 192, 256])  # one for each form of the reduction above rank 64
def test_effective_rank_of_the_last_rows_at_every_cut(r):
    # The 64 rows left to one wavefront begin anywhere in a 16 x 16 tile and in a group of four tiles: every number
    # of columns that are not zero from 65 on, with eigenvalues that hardly fall.  tau 1e-9 below and above the
    # share of the j largest, so that an eigenvalue that is off by 1e-8 of the sum is another r' (fp64 here and
    # there: sums of at most 256 eigenvalues good to about 256 2^-52 of the largest, 1e-13).
    n = 512
    g = rng(r)
    ws = torch.empty(dlcx.dlcx_workspace_bytes(dlcx.desc(n, n, r, 4, 16), 1), device=DEV, dtype=torch.uint8)
    out = torch.full((1,), -1, device=DEV, dtype=torch.int32)
    wrong = []
    for live in range(65, r + 1):
        q = g.standard_normal((r, n)).astype(np.float32)
        q[g.permutation(r)[live:]] = 0.0
        s = np.cumsum(np.linalg.eigvalsh(q.astype(np.float64) @ q.T.astype(np.float64))[::-1])
        for j in (1, live // 2, live - 1):
            for side in (0, 1):
                dlcx.dlcx_effective_rank(n, r, to_dev(q), s[j - 1] / s[-1] + (side - 0.5) * 2e-9, out, ws)
                if int(out.item()) != j + side:
                    wrong.append((live, j, side, int(out.item())))
    assert not wrong, wrong


@pytest.mark.parametrize("r", [1, 3, 16, 31, 32, 33, 64, 65, 130, 256])
def test_effective_rank_of_a_factor_that_is_not_finite(r):
    # A NaN anywhere: no eigenvalue is a number and no share is ever reached, r' = 0.  An infinity: up
    # to rank 31 every column of S is infinite and the first one holds every share (where an element
    # beside it is zero, S has a NaN); above that no eigenvalue is found, 0.
    n = 512
    g = rng(r)
    ws = torch.empty(dlcx.dlcx_workspace_bytes(dlcx.desc(n, n, r, 4, 16), 1), device=DEV, dtype=torch.uint8)
    out = torch.full((1,), -1, device=DEV, dtype=torch.int32)
    for col in sorted({0, r // 2, r - 1}):
        for value, beside, want in ((np.nan, 1.0, 0), (np.inf, 1.0, 1 if r < 32 else 0),
                                    (-np.inf, 1.0, 1 if r < 32 else 0), (np.inf, 0.0, 1 if r == 1 else 0)):
            q = g.standard_normal((r, n)).astype(np.float32)
            q[:, n // 3] = beside
            q[col, n // 3] = value
            dlcx.dlcx_effective_rank(n, r, to_dev(q), 0.99, out, ws)
            assert int(out.item()) == want, (col, value, beside)


def test_select_rank_stage_value_and_window():
    # three matrices with known r' (3, 49, zero matrix -> rmin 4): mean 56/3 = 18.67 -> 19
    n, r = 512, 64
    mats = []
    for alpha in (2.0, 1.0):
        V = synth.orthonormal_columns(rng(5), n, 256)
        sig = np.arange(1, 257, dtype=np.float64) ** (-alpha)
        mats.append(np.ascontiguousarray((V * sig).T.astype(np.float32)))
    descs = [dlcx.desc(n, n, 256, 4, 16), dlcx.desc(n, n, 256, 4, 16), dlcx.desc(n, n, r, 4, 16)]
    q_bars = [to_dev(mats[0]), to_dev(mats[1]), torch.zeros(r, n, device=DEV)]
    assert [ref.effective_rank(x, 0.99) for x in mats] == [3, 49]
    ws = torch.empty(dlcx.dlcx_select_rank_workspace_bytes(descs), device=DEV, dtype=torch.uint8)
    hist = (C.c_int32 * 5)(256, 256, 256, 256, 0)
    rp, r_next, H = dlcx.dlcx_select_rank(descs, q_bars, 0.99, hist, 5, 5, 256, 4, 256, 125, workspace=ws)
    assert rp == 19
    want_r, want_H = ref.adagradcmp([256, 256, 256, 256, 19], 5, 5, 256, 4, 256, 125)
    assert (r_next, H) == (want_r, want_H)


def test_batched_orthonormalize_and_rank_mixed_shapes():
    # 70 factors of different lengths and ranks in one call (more than one launch chunk of 64):
    # same results as the one-matrix entry points, which are checked against the oracle above.
    g = rng(4242)
    shapes = [(256 + 16 * (i % 9), 8 + (i * 7) % 57) for i in range(70)]      # (L, r)
    shapes[3] = (2048, 200)                                                   # global-memory path
    descs, ps, qs, ps_single = [], [], [], []
    for L, r in shapes:
        descs.append(dlcx.desc(L, L, r, 4, 16))
        a = (g.standard_normal((r, L)) * (np.arange(1, r + 1)[:, None] ** -1.0)).astype(np.float32)
        ps.append(to_dev(a))
        ps_single.append(to_dev(a))
        qs.append(to_dev(a))
    ws = torch.empty(dlcx.dlcx_batched_workspace_bytes(descs), device=DEV, dtype=torch.uint8)
    out = torch.zeros(len(descs), device=DEV, dtype=torch.int32)
    dlcx.dlcx_effective_rank_batched(descs, qs, 0.9, out, ws)
    dlcx.dlcx_orthonormalize_batched(descs, ps, ws)
    one = torch.zeros(1, device=DEV, dtype=torch.int32)
    for i, (L, r) in enumerate(shapes):
        w1 = torch.empty(dlcx.dlcx_workspace_bytes(descs[i], 1), device=DEV, dtype=torch.uint8)
        dlcx.dlcx_orthonormalize(L, r, ps_single[i], w1)
        assert torch.equal(ps[i], ps_single[i]), i
        dlcx.dlcx_effective_rank(L, r, qs[i], 0.9, one, w1)
        assert int(one.item()) == int(out[i].item()), i
    for i in (0, 3, 17, 69):
        assert int(out[i].item()) == ref.effective_rank(to_np(qs[i]), 0.9)
        assert rel_l2(to_np(ps[i]), ref.orthonormalize(to_np(qs[i]))) <= 1e-5


@pytest.mark.parametrize("mma", [dlcx.MMA_FMA, dlcx.MMA_F32, dlcx.MMA_BF16, dlcx.MMA_F16])
@pytest.mark.parametrize("m,n,r,K,qbits,group", [
    (16, 16, 1, 1, 4, 16),          # one group
    (272, 528, 3, 2, 8, 16),        # a last wavefront that is partly idle
    (512, 512, 8, 3, 4, 64), (512, 768, 33, 5, 8, 256), (1024, 256, 70, 4, 4, 32), (256, 1280, 130, 16, 4, 128),
    (256, 512, 100, 3, 4, 16),      # three workers: 1e3 times larger, beyond what the fp16 form above rank 64 takes
])
def test_quantise_and_average_in_one_launch_is_both(mma, m, n, r, K, qbits, group):
    # Codes, scales, factors and mean bit for bit those of the two calls: with and without partial sums, with
    # the fp16 form in and out of its range, payloads with zeros, infinities and NaN.
    g = rng(m + n + r + K)
    d = dlcx.desc(m, n, r, qbits, group, mma)
    scale = 1e3 if K == 3 else 1.0
    deltas = [to_dev((scale * g.standard_normal((m, n))).astype(np.float32)) for _ in range(K)]
    deltas[0][:, : n // 2] = 0.0
    deltas[0][: m // 2] = 0.0
    if K == 2:
        deltas[1][0, 0], deltas[1][m - 1, n - 1] = float("inf"), float("nan")
    ws = torch.zeros(dlcx.dlcx_workspace_bytes(d, K), device=DEV, dtype=torch.uint8)
    for phase, length, other in ((dlcx.PHASE_P, m, n), (dlcx.PHASE_Q, n, m)):
        basis = to_dev(g.standard_normal((r, other)).astype(np.float32))
        got = []
        for fused in (False, True):
            codes, scales = payload_buffers(d, phase, K)
            mean = torch.full((r, length), -1.0, device=DEV)
            ws.fill_(255)
            if fused:
                dlcx.dlcx_compress_average(d, phase, deltas, basis, codes, scales, mean, ws)
            else:
                dlcx.dlcx_compress_batched(d, phase, deltas, basis, codes, scales, ws)
                dlcx.dlcx_dequant_average(codes, scales, r * length, qbits, group, mean)
            got.append([to_np(x).view(np.uint8) for x in codes + scales + [mean, ws[: 4 * K * r * length]]])
        for a, b in zip(*got):
            assert np.array_equal(a, b), phase


@pytest.mark.parametrize("mma", [dlcx.MMA_FMA, dlcx.MMA_F32, dlcx.MMA_BF16, dlcx.MMA_F16])
@pytest.mark.parametrize("m,n,r,r_prev,K,dtype", [
    (48, 80, 5, 0, 2, torch.float32), (272, 528, 8, 8, 3, torch.bfloat16), (512, 256, 64, 20, 1, torch.float32),
    (256, 512, 33, 70, 5, torch.bfloat16), (256, 272, 100, 64, 16, torch.float32),   # above rank 64: two passes
])
def test_round_with_the_average_is_the_two_calls(mma, m, n, r, r_prev, K, dtype):
    # State, codes, scales and mean bit for bit those of the round and the average of its payloads, the mean written
    # over the factor of the round before, of the same rank, a lower one or a higher one.
    g = rng(m + n + r + K)
    d = dlcx.desc(m, n, r, 4, 16, mma)
    up = lambda *shape: to_dev(g.standard_normal(shape).astype(np.float32))
    theta_l = [up(m, n).to(dtype) for _ in range(K)]
    state = [up(m, n) for _ in range(K + 2)]   # error buffers, theta, momentum
    factor, q_bar, basis = up(max(r, r_prev, 1), m), up(max(r_prev, 1), n), up(r, n)
    ws = torch.zeros(max(dlcx.dlcx_workspace_bytes(d, K), dlcx.dlcx_workspace_bytes(dlcx.desc(m, n, max(r_prev, 1), 4, 16, mma), K)),
                     device=DEV, dtype=torch.uint8)
    got = []
    for one in (False, True):
        codes, scales = payload_buffers(d, dlcx.PHASE_P, K)
        *ef, theta, v = [x.clone() for x in state]
        p_hat = factor.clone()
        ws.fill_(255)
        args = (d, r_prev, p_hat, q_bar, theta_l, ef, theta, v, 0.7, 0.9, basis, codes, scales)
        if one:
            dlcx.dlcx_ef_delta_apply_compress_average(*args, p_hat, ws)
        else:
            dlcx.dlcx_ef_delta_apply_compress(*args, ws)
            dlcx.dlcx_dequant_average(codes, scales, r * m, 4, 16, p_hat)
        got.append([to_np(x).view(np.uint8) for x in codes + scales + ef + [theta, v, p_hat]])
    for i, (a, b) in enumerate(zip(*got)):
        assert np.array_equal(a, b), i
