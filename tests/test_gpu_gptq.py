"""GPU parity of the error-compensated quantizer (paper Sec. 5: GPTQ as the base
quantizer) against the CPU oracle: the column sweep bit for bit, given the same
inverse-Hessian factor."""
import numpy as np
import pytest
import torch

from oracle import dymoe_oracle as O
from paper_2603_19172_amd import binding as B
from paper_2603_19172_amd import synth
from gpu_helpers import DEV, bits_of, subnormal_sweep_inputs, to_bf16

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = B.Context(0)
    yield c
    c.close()


def _case(cid, N, K, n=None):
    xb = synth.calibration_inputs(cid, n or max(256, 2 * K), K)
    wb = synth.normal_bf16(cid, 77, (N, K), 0.02)
    U = O.gptq_factor(O.gptq_hessian(xb)).astype(np.float32)
    return xb, wb, U


def _same(got, want):
    codes, scale, zero = got
    torch.cuda.synchronize()
    return (np.array_equal(codes.cpu().numpy(), want[0]) and np.array_equal(bits_of(scale), want[1])
            and np.array_equal(bits_of(zero), want[2]))


# rows: fewer than a workgroup's 32, a ragged tail, several workgroups; columns: one group (no
# trailing update), a ragged 128-column trail tile, many steps
@pytest.mark.parametrize("N,K", [(24, 64), (24, 192), (130, 320), (64, 1024), (257, 2048)])
@pytest.mark.parametrize("bits", [2, 4, 8])
def test_gptq_sweep_is_bit_exact(ctx, N, K, bits):
    if K == 2048 and bits != 4:
        pytest.skip("the largest case runs once")
    _, wb, U = _case(700 + N, N, K)
    want = O.gptq_quantize_pack(wb, U, bits)
    got = ctx.gptq_quantize_pack(to_bf16(wb), torch.from_numpy(U).to(DEV), bits)
    torch.cuda.synchronize()
    codes = got[0].cpu().numpy()
    print("N=%d K=%d bits=%d: code bytes equal %.6f" % (N, K, bits, (codes == want[0]).mean()))
    assert _same(got, want)
    # and it is not the plain quantizer's answer
    plain = O.quantize_pack(wb, bits)
    assert K == 64 or not np.array_equal(want[0], plain[0])


def test_gptq_identity_factor_gives_the_plain_quantizer(ctx):
    _, wb, _ = _case(720, 100, 256)
    w = to_bf16(wb)
    eye = torch.eye(256, dtype=torch.float32, device=DEV)
    for bits in (2, 4, 8):
        a = ctx.gptq_quantize_pack(w, eye, bits)
        b = ctx.quantize_pack(w, bits)
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(a, b))


def test_gptq_reuses_a_dirty_workspace_and_lowers_the_output_error(ctx):
    xb, wb, U = _case(730, 96, 512, n=1024)
    w, u = to_bf16(wb), torch.from_numpy(U).to(DEV)
    need = int(B.lib.dymoe_gptq_workspace_bytes(96, 512))
    ws = torch.full((need + 512,), 0xFF, dtype=torch.uint8, device=DEV)
    first = ctx.gptq_quantize_pack(w, u, 4, workspace=ws)
    second = ctx.gptq_quantize_pack(w, u, 4, workspace=ws)
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(first, second))
    assert _same(first, O.gptq_quantize_pack(wb, U, 4))
    H = O.gptq_hessian(xb)
    wf = synth.bf16_bits_to_f32(wb).astype(np.float64)
    deq = O.dequantize(first[0].cpu().numpy(), bits_of(first[1]), bits_of(first[2]), 4)
    plain = O.dequantize(*O.quantize_pack(wb, 4), 4)
    assert O.output_error(wf, deq, H) < 0.5 * O.output_error(wf, plain, H)


# samples: fewer than a step's 64, ragged, several steps; columns: one tile, a ragged last tile, several tiles
@pytest.mark.parametrize("n,K", [(9, 64), (300, 320), (1000, 512), (64, 1024)])
def test_gptq_hessian_matches_the_oracle(ctx, n, K):
    xb = synth.calibration_inputs(740 + K, n, K)
    want = O.gptq_hessian(xb)
    x = to_bf16(xb)
    got = ctx.gptq_hessian(x)
    torch.cuda.synchronize()
    g = got.cpu().numpy().astype(np.float64)
    scale = np.sqrt(np.outer(np.diag(want), np.diag(want)))
    err = np.abs(g - want) / scale
    print("n=%d K=%d: max |dH| / sqrt(Hii Hjj) = %.2e" % (n, K, err.max()))
    assert err.max() < 1e-5 and np.array_equal(g, g.T)
    # a second batch added on top
    both = ctx.gptq_hessian(x, out=got, accumulate=True)
    torch.cuda.synchronize()
    assert np.abs(both.cpu().numpy() - 2.0 * want).max() <= 2e-5 * scale.max()


@pytest.mark.parametrize("K", [64, 192, 1024])
def test_gptq_factor_matches_the_oracle(ctx, K):
    xb = synth.calibration_inputs(760 + K, 2 * K, K)
    H = O.gptq_hessian(xb)
    H[:, 5] = 0.0                      # a column no input reached
    H[5, :] = 0.0
    want = O.gptq_factor(H, damp=0.01)
    got = ctx.gptq_factor(torch.from_numpy(H.astype(np.float32)).to(DEV), damp=0.01)
    torch.cuda.synchronize()
    U = got.cpu().numpy().astype(np.float64)
    assert np.isfinite(U).all() and np.array_equal(U, np.triu(U)) and (np.diag(U) > 0).all()
    rel = np.abs(U - want).max(axis=1) / np.abs(want).max(axis=1)
    Hd = O.gptq_damped(H, 0.01)
    resid = np.abs(U.T @ U @ Hd - np.eye(K)).max()
    print("K=%d: max row-relative error %.2e, |U^T U Hd - I| = %.2e" % (K, rel.max(), resid))
    assert rel.max() < 2e-4 and resid < 2e-3


def test_gptq_chain_on_the_device(ctx):
    """Hessian, factor and sweep all on the device; the result is as good as the oracle's own chain (the
    factors differ in the last fp32 digits, so a code may differ here and there)."""
    N, K = 128, 512
    xb = synth.calibration_inputs(780, 1024, K)
    wb = synth.normal_bf16(780, 77, (N, K), 0.02)
    H = O.gptq_hessian(xb)
    want = O.gptq_quantize_pack(wb, O.gptq_factor(H), 4)
    hess = ctx.gptq_hessian(to_bf16(xb))
    u = ctx.gptq_factor(hess)
    got = ctx.gptq_quantize_pack(to_bf16(wb), u, 4)
    torch.cuda.synchronize()
    wf = synth.bf16_bits_to_f32(wb).astype(np.float64)
    d_got = O.dequantize(got[0].cpu().numpy(), bits_of(got[1]), bits_of(got[2]), 4)
    d_want = O.dequantize(*want, 4)
    e_got, e_want = O.output_error(wf, d_got, H), O.output_error(wf, d_want, H)
    e_plain = O.output_error(wf, O.dequantize(*O.quantize_pack(wb, 4), 4), H)
    same = (d_got == d_want).mean()
    print("same dequantised values %.4f; output error device %.4e oracle %.4e plain %.4e" % (same, e_got, e_want, e_plain))
    assert same > 0.98 and abs(e_got - e_want) <= 0.02 * e_want and e_got < 0.5 * e_plain


def test_gptq_mixtral_sized_matrix(ctx):
    """The first expert matrix of the Mixtral-shaped layer at full size (14336 x 4096), 1024 calibration
    tokens.  Rows are independent in the sweep, so the oracle checks a seeded sample of them bit for bit;
    the factor is compared in full."""
    N, K, n = 14336, 4096, 1024
    cfg = synth.CONFIGS["mixtral_decode"]
    wb = synth.expert_matrix(cfg, 0, 0)
    assert wb.shape == (N, K)
    xb = synth.calibration_inputs(790, n, K)
    H = O.gptq_hessian(xb)
    U = O.gptq_factor(H)
    x = to_bf16(xb)
    hess = ctx.gptq_hessian(x)
    u_dev = ctx.gptq_factor(hess)
    torch.cuda.synchronize()
    Ud = u_dev.cpu().numpy().astype(np.float64)
    rel = np.abs(Ud - U).max(axis=1) / np.abs(U).max(axis=1)
    print("factor K=%d: max row-relative error %.2e" % (K, rel.max()))
    assert np.isfinite(Ud).all() and rel.max() < 5e-4
    del Ud
    # the sweep with the oracle's own factor, so that the comparison is bit for bit
    U32 = U.astype(np.float32)
    got = ctx.gptq_quantize_pack(to_bf16(wb), torch.from_numpy(U32).to(DEV), 4)
    torch.cuda.synchronize()
    rows = np.sort(np.random.default_rng(790).choice(N, size=24, replace=False))
    rows[0], rows[-1] = 0, N - 1
    want = O.gptq_quantize_pack(wb[rows], U32, 4)
    assert np.array_equal(got[0].cpu().numpy()[rows], want[0])
    assert np.array_equal(bits_of(got[1])[rows], want[1]) and np.array_equal(bits_of(got[2])[rows], want[2])
    # the sampled rows' output error against the plain quantizer's
    wf = synth.bf16_bits_to_f32(wb[rows]).astype(np.float64)
    e_comp = O.output_error(wf, O.dequantize(*want, 4), H)
    e_plain = O.output_error(wf, O.dequantize(*O.quantize_pack(wb[rows], 4), 4), H)
    print("output error on 24 rows: compensated %.4e, plain %.4e" % (e_comp, e_plain))
    assert e_comp < 0.7 * e_plain


def test_gptq_experts_feed_the_mixed_ffn(ctx):
    """The compensated quantizer writes the plain quantizer's formats: the FFN reads its experts unchanged.
    Two experts (int4 and int2) quantised on the device with calibration inputs for [F,H] and [H,F]; the
    FFN's output against the oracle's FFN over the oracle's own compensated codes."""
    cfg = synth.scaled(synth.CONFIGS["tiny"], T=3, H=256, F=512, E=2, k=2, config_id=83)
    x, _ = synth.activations(cfg)
    hw = {e: synth.expert_weights(cfg, e) for e in range(cfg.E)}
    cal = {cfg.H: synth.calibration_inputs(83, 1024, cfg.H), cfg.F: synth.calibration_inputs(84, 1024, cfg.F)}
    U = {K: O.gptq_factor(O.gptq_hessian(cal[K])).astype(np.float32) for K in cal}
    Ud = {K: torch.from_numpy(U[K]).to(DEV) for K in U}
    bits_np = np.array([4, 2], dtype=np.uint8)
    experts_dev, experts_ref = [], []
    for e in range(cfg.E):
        b = int(bits_np[e])
        experts_dev.append({"q%d" % b: [ctx.gptq_quantize_pack(to_bf16(m), Ud[m.shape[1]], b) for m in hw[e]]})
        experts_ref.append({"q": [O.gptq_quantize_pack(m, U[m.shape[1]], b) for m in hw[e]]})
    table, keep = B.make_expert_table(experts_dev, DEV)
    idx_np = np.array([[0, 1], [1, 0], [0, 1]], dtype=np.int32)
    w_np = np.array([[0.6, 0.4], [0.3, 0.7], [0.5, 0.5]], dtype=np.float32)
    y = ctx.moe_ffn_mixed(to_bf16(x), torch.from_numpy(idx_np).to(DEV), torch.from_numpy(w_np).to(DEV),
                          torch.from_numpy(bits_np).to(DEV), table, cfg.F, out_dtype=B.OUT_F32)
    torch.cuda.synchronize()
    ref = O.moe_ffn_mixed(x, idx_np, w_np.astype(np.float64), bits_np, experts_ref)
    rms = np.sqrt((ref ** 2).mean(axis=1, keepdims=True))
    err = float((np.abs(y.cpu().numpy() - ref) / rms).max())
    print("FFN over compensated experts: max err / rms = %.2e" % err)
    assert err <= 2e-2


def test_code_tiles_from_rowmajor_equal_the_quantizers_own_tiles(ctx):
    """dymoe_pack_code_tiles is the permutation between the two layouts the plain quantizer can write."""
    from paper_2603_19172_amd.layer import ExpertStore
    cfg = synth.scaled(synth.CONFIGS["tiny"], H=384, F=256, E=3, k=2, config_id=85)
    hw = {e: synth.expert_weights(cfg, e) for e in range(cfg.E)}
    store = ExpertStore([[to_bf16(m) for m in hw[e]] for e in range(cfg.E)], cfg.H, cfg.F, DEV, formats=(8, 4, 2))
    bits = torch.tensor([8, 4, 2], dtype=torch.uint8, device=DEV)
    ones = torch.ones((cfg.E,), dtype=torch.int32, device=DEV)
    ctx.quantize_experts(store.table, bits, ones, cfg.E, cfg.H, cfg.F, layout=B.LAYOUT_TILE)
    for e, b in enumerate((8, 4, 2)):
        for i in range(3):
            tiles = ctx.pack_code_tiles(ctx.quantize_pack(store.w[e][i], b), b)
            torch.cuda.synchronize()
            # scale and zero of a tile are 64 fp16 in lane order: compare as flat arrays
            assert torch.equal(tiles[0].flatten(), store.q[b][e][i][0].flatten())
            assert torch.equal(tiles[1].flatten(), store.q[b][e][i][1].flatten())
            assert torch.equal(tiles[2].flatten(), store.q[b][e][i][2].flatten())


def test_gptq_experts_feed_the_grouped_gemm(ctx):
    """Compensated experts, re-packed into tiles, through the MFMA path (8 tokens) against the oracle's FFN."""
    cfg = synth.scaled(synth.CONFIGS["tiny"], T=8, H=256, F=512, E=2, k=2, config_id=86)
    x, _ = synth.activations(cfg)
    hw = {e: synth.expert_weights(cfg, e) for e in range(cfg.E)}
    cal = {cfg.H: synth.calibration_inputs(86, 1024, cfg.H), cfg.F: synth.calibration_inputs(87, 1024, cfg.F)}
    U = {K: O.gptq_factor(O.gptq_hessian(cal[K])).astype(np.float32) for K in cal}
    Ud = {K: torch.from_numpy(U[K]).to(DEV) for K in U}
    bits_np = np.array([4, 2], dtype=np.uint8)
    experts_dev, experts_ref = [], []
    for e in range(cfg.E):
        b = int(bits_np[e])
        rm = [ctx.gptq_quantize_pack(to_bf16(m), Ud[m.shape[1]], b) for m in hw[e]]
        experts_dev.append({"q%d" % b: [ctx.pack_code_tiles(t, b) for t in rm]})
        experts_ref.append({"q": [O.gptq_quantize_pack(m, U[m.shape[1]], b) for m in hw[e]]})
    table, keep = B.make_expert_table(experts_dev, DEV)
    rng = np.random.default_rng(86)
    idx_np = np.stack([rng.permutation(2) for _ in range(cfg.T)]).astype(np.int32)
    w_np = rng.uniform(0.2, 0.8, size=(cfg.T, 1)).astype(np.float32)
    w_np = np.concatenate([w_np, 1.0 - w_np], axis=1)
    y = ctx.moe_ffn_mixed(to_bf16(x), torch.from_numpy(idx_np).to(DEV), torch.from_numpy(w_np).to(DEV),
                          torch.from_numpy(bits_np).to(DEV), table, cfg.F, out_dtype=B.OUT_F32, path=B.PATH_GEMM)
    torch.cuda.synchronize()
    ref = O.moe_ffn_mixed(x, idx_np, w_np.astype(np.float64), bits_np, experts_ref)
    rms = np.sqrt((ref ** 2).mean(axis=1, keepdims=True))
    err = float((np.abs(y.cpu().numpy() - ref) / rms).max())
    print("grouped GEMM over compensated experts: max err / rms = %.2e" % err)
    assert err <= 2e-2


def test_gptq_factor_with_fewer_samples_than_columns(ctx):
    """64 calibration tokens for 512 columns: the Hessian has rank 64 and only the damping keeps it
    positive definite (condition number about 1e4), the case fp32 Cholesky has least room for."""
    K = 512
    H = O.gptq_hessian(synth.calibration_inputs(864, 64, K))
    want = O.gptq_factor(H)
    got = ctx.gptq_factor(torch.from_numpy(H.astype(np.float32)).to(DEV))
    torch.cuda.synchronize()
    U = got.cpu().numpy().astype(np.float64)
    rel = np.abs(U - want).max(axis=1) / np.abs(want).max(axis=1)
    print("rank-deficient Hessian: max row-relative error %.2e" % rel.max())
    assert np.isfinite(U).all() and rel.max() < 5e-4


def test_gptq_sweep_edge_rows(ctx):
    """One row; a group of equal weights (scale 0: every code 0, the whole value becomes error and is passed
    on); a group of zeros; values at the top of the bf16 range the plain quantizer accepts."""
    K = 256
    _, wb, U = _case(741, 4, K)
    w = synth.bf16_bits_to_f32(wb).copy()
    w[1, 64:128] = 0.01953125          # one bf16 value through a whole group
    w[2, 0:64] = 0.0
    w[3, 128:192] *= 1.0e6             # ~2e4: near the fp16 range of scale and zero
    wb = synth.f32_to_bf16_bits(w)
    for rows in (slice(0, 1), slice(0, 4)):
        for bits in (2, 4, 8):
            want = O.gptq_quantize_pack(wb[rows], U, bits)
            got = ctx.gptq_quantize_pack(to_bf16(wb[rows]), torch.from_numpy(U).to(DEV), bits)
            assert _same(got, want)
    # one calibration token
    xb = synth.calibration_inputs(742, 1, 128)
    h = ctx.gptq_hessian(to_bf16(xb))
    torch.cuda.synchronize()
    assert np.allclose(h.cpu().numpy(), O.gptq_hessian(xb), rtol=1e-6, atol=0)


# a panel is four groups of 64 columns, a row block 32 rows, a workgroup of the columns behind takes 64 rows by 64 columns or 128 by 128: rows
# below, at and beyond each edge (below 64 rows panels are two groups wide), columns that end inside a panel and inside a pair of groups
@pytest.mark.parametrize("N,K,bits", [(63, 320, 4), (64, 512, 2), (65, 576, 8), (127, 256, 4), (129, 832, 2), (200, 704, 4)])
def test_gptq_sweep_panel_edges(ctx, N, K, bits):
    _, wb, U = _case(800 + N, N, K)
    want = O.gptq_quantize_pack(wb, U, bits)
    got = ctx.gptq_quantize_pack(to_bf16(wb), torch.from_numpy(U).to(DEV), bits)
    assert _same(got, want)


# row blocks of 32 whose errors outlive the launch that makes them: one ragged block, a whole and a ragged one, two whole ones, three and a
# half; half panels below 64 rows, last panels of every number of groups
@pytest.mark.parametrize("N,K,bits", [(1, 704, 4), (31, 832, 8), (32, 640, 4), (33, 1152, 2), (63, 1088, 4), (95, 1344, 4), (96, 896, 2),
                                      (97, 1216, 8), (128, 1536, 4), (161, 1024, 4)])
def test_gptq_sweep_row_blocks(ctx, N, K, bits):
    _, wb, U = _case(1200 + N, N, K)
    assert _same(ctx.gptq_quantize_pack(to_bf16(wb), torch.from_numpy(U).to(DEV), bits), O.gptq_quantize_pack(wb, U, bits))


# more row blocks than compute units, whose chains then lie on other wavefronts: one panel, a last panel of one group, of two (two
# wavefronts share a group's values) and of three, whole and ragged last row blocks
@pytest.mark.parametrize("N,K,bits", [(8193, 64, 2), (8224, 256, 8), (8225, 320, 4), (8287, 384, 2), (8256, 448, 4)])
def test_gptq_sweep_more_row_blocks_than_compute_units(ctx, N, K, bits):
    _, wb, U = _case(1500 + N, N, K)
    assert _same(ctx.gptq_quantize_pack(to_bf16(wb), torch.from_numpy(U).to(DEV), bits), O.gptq_quantize_pack(wb, U, bits))


@pytest.mark.parametrize("bits", [2, 4, 8])
def test_gptq_sweep_subnormal_errors(ctx, bits):
    """Rows so small that rest / U[c,c] is subnormal, beside ordinary ones in the same groups: the ordinary rows' codes, and
    scale and zero of the small ones.  (Scale 0 makes every code of the small rows 0: what their errors are cannot be seen
    here, but in the test below.)"""
    N, K = 66, 320
    _, wb, U = _case(850, N, K)
    w = synth.bf16_bits_to_f32(wb).copy()
    w[3] *= 1e-37
    w[20] *= 3e-36
    w[64, 64:128] = 0.0
    w[65] = 1e-39
    wb = synth.f32_to_bf16_bits(w)
    for scale in (1.0, 1e3):
        u = (U * np.float32(scale)).astype(np.float32)
        want = O.gptq_quantize_pack(wb, u, bits)
        got = ctx.gptq_quantize_pack(to_bf16(wb), torch.from_numpy(u).to(DEV), bits)
        assert _same(got, want)


# every error subnormal, at a size with panels of two groups and one with a whole panel and a ragged row block; on the
# halfway inputs a reciprocal in the place of the division changes up to 59 code bytes, a flush of subnormal numbers more
# than 1000 (tests/test_oracle_pins.py makes both mistakes)
@pytest.mark.parametrize("halfway", [False, True])
@pytest.mark.parametrize("N,K", [(24, 192), (66, 320)])
@pytest.mark.parametrize("bits", [2, 4, 8])
def test_gptq_sweep_subnormal_errors_reach_the_codes(ctx, N, K, bits, halfway):
    wb, u = subnormal_sweep_inputs(1, N, K, halfway)
    want = O.gptq_quantize_pack(wb, u, bits)
    got = ctx.gptq_quantize_pack(to_bf16(wb), torch.from_numpy(u).to(DEV), bits)
    assert _same(got, want)


# blocks of 64, brought forward two steps at a time in pairs of blocks: one to ten of them and a few odd numbers beyond, and pivots
# outside the range of the estimate's steps
@pytest.mark.parametrize("K,size", [(128, 1.0), (320, 1.0), (704, 1.0), (192, 1e-34), (192, 1e32), (256, 1.0), (384, 1.0), (448, 1.0),
                                    (512, 1.0), (576, 1.0), (640, 1.0), (1088, 1.0)])
def test_gptq_factor_block_edges(ctx, K, size):
    xb = synth.calibration_inputs(870 + K, 2 * K, K)
    H = O.gptq_hessian(xb)
    H32 = (H * size / np.diag(H).mean()).astype(np.float32)
    want = O.gptq_factor(H32.astype(np.float64))
    u = ctx.gptq_factor(torch.from_numpy(H32).to(DEV))
    torch.cuda.synchronize()
    U = u.cpu().numpy().astype(np.float64)
    rel = np.abs(U - want).max(axis=1) / np.abs(want).max(axis=1)
    print("K=%d size %.0e: max row-relative error %.2e" % (K, size, rel.max()))
    # the same bound as for the other sizes: fp32 Cholesky of a matrix with a condition number of about 1e3
    assert np.array_equal(U, np.triu(U)) and rel.max() < 2e-4


# workspaces of exactly the bytes asked for, one value everywhere before and behind them: what lies behind stays, and the
# results do not depend on what lay inside
@pytest.mark.parametrize("N,K", [(24, 192), (64, 320), (65, 64), (130, 576)])
def test_gptq_workspaces_are_as_large_as_asked_for(ctx, N, K):
    _, wb, _ = _case(900 + N, N, K)
    hess = ctx.gptq_hessian(to_bf16(synth.calibration_inputs(900 + N, 2 * K, K)))
    want_u = ctx.gptq_factor(hess)
    want = ctx.gptq_quantize_pack(to_bf16(wb), want_u, 4)
    for fill in (0x00, 0xFF):
        need = int(B.lib.dymoe_gptq_factor_workspace_bytes(K))
        ws = torch.full((need + 4096,), fill, dtype=torch.uint8, device=DEV)
        u = ctx.gptq_factor(hess, workspace=ws[:need])
        assert torch.equal(u, want_u) and (ws[need:] == fill).all()
        need = int(B.lib.dymoe_gptq_workspace_bytes(N, K))
        ws = torch.full((need + 65536,), fill, dtype=torch.uint8, device=DEV)
        got = ctx.gptq_quantize_pack(to_bf16(wb), want_u, 4, workspace=ws[:need])
        assert all(torch.equal(a, b) for a, b in zip(got, want)) and (ws[need:] == fill).all()


# corrections behind a panel: both kernels on either side of the rule (192 workgroups of 128 x 128 on 256 compute units), their values from the
# matrix itself and from the working copy; an odd number of 64-row blocks, last ones of 1, 32 and 42 rows, last pairs of column
# blocks that are one; and panels with nothing behind them
CORRECTIONS = {"small": [(12288, 704, 4), (6144, 832, 4), (6273, 768, 4)],
               "large": [(12353, 704, 2), (12458, 704, 8), (12448, 960, 4), (12353, 960, 4)],
               "none": [(12288, 512, 4), (12289, 512, 4)]}


# rows are independent: a few of them alone give the same codes, and the oracle's
@pytest.mark.parametrize("N,K,bits", [c for v in CORRECTIONS.values() for c in v])
def test_gptq_corrections_of_few_and_many_workgroups(ctx, N, K, bits):
    g = torch.Generator(device=DEV).manual_seed(N)
    w = (torch.randn((N, K), generator=g, device=DEV) * 0.02).bfloat16()
    x = torch.randn((2 * K, K), generator=g, device=DEV)
    u = ctx.gptq_factor(ctx.gptq_hessian((x + torch.randn((2 * K, 1), generator=g, device=DEV)).bfloat16()))
    whole = ctx.gptq_quantize_pack(w, u, bits)
    for rows in (slice(0, 70), slice(N - 131, N)):
        part = ctx.gptq_quantize_pack(w[rows].contiguous(), u, bits)
        for a, b in zip(whole, part):
            assert torch.equal(a[rows].contiguous().view(torch.uint8), b.view(torch.uint8))
    for rows in (slice(60, 68), slice(N - 45, N)):
        wb = w[rows].contiguous().view(torch.int16).cpu().numpy().view(np.uint16)
        assert _same(tuple(a[rows].contiguous() for a in whole), O.gptq_quantize_pack(wb, u.cpu().numpy(), bits))


@pytest.mark.gpu
@pytest.mark.parametrize("n,K", [(512, 136), (513, 136), (576, 8), (640, 2816), (641, 2824), (1345, 264)])
def test_gptq_hessian_of_few_and_many_tiles(ctx, n, K):
    # the split of the samples between the halves of a workgroup: last steps of one or both halves, remainders of 64 samples.
    # 16-bit inputs multiply exactly; a sum of n terms in fp32, in any order, is off by at most n 2^-24 of the sum of its magnitudes
    x = to_bf16(synth.calibration_inputs(910 + n, n, K))
    exact = x.double().t() @ x.double()
    bound = (n + 1) * 2.0**-24 * (x.double().abs().t() @ x.double().abs())
    got = ctx.gptq_hessian(x)
    assert bool(((got.double() - exact).abs() <= bound).all())
    assert torch.equal(got, got.t())
    twice = ctx.gptq_hessian(x, out=got.clone(), accumulate=True)
    assert torch.equal(twice, got + got)


# tiles dealt out over several rounds: workgroups on the compute units that the solvers leave (61 blocks of columns) and also
# behind the solvers (81), both with a last pair of blocks that is not whole; more solvers than compute units (257)
@pytest.mark.parametrize("K", [3904, 5184, 16448])
def test_gptq_factor_of_many_tiles(ctx, K):
    g = torch.Generator(device=DEV).manual_seed(K)
    x = torch.randn((2 * K, K), generator=g, device=DEV)
    if K < 16384:                                           # (the condition number grows with K where columns share a direction)
        x += 1.5 * torch.randn((2 * K, 1), generator=g, device=DEV)
    H = (x.T @ x).contiguous()
    u = ctx.gptq_factor(H, damp=0.01).double()
    torch.cuda.synchronize()
    Hd = H.double()
    Hd.diagonal().add_(0.01 * H.double().diagonal().mean())
    eye = torch.eye(K, dtype=torch.float64, device=DEV)
    assert torch.equal(u, u.triu())
    # (U^T U)^-1 = Hd, so U Hd U^T = I: what binary32 leaves of that is its epsilon times the condition number (about a thousand)
    err = (u @ Hd @ u.T - eye).abs().max().item()
    print("K=%d: |U Hd U^T - I| = %.2e" % (K, err))
    assert err < 1e3 * 2.0 ** -23


def test_gptq_sweep_of_more_rows_than_one_launch_holds(ctx):
    """A dimension of a launch holds fewer than 2^32 threads, 2^29 rows of a panel: one row block more, ragged, on top of that."""
    K, bits, rows, N = 64, 2, 1 << 20, (1 << 29) + 65
    torch.cuda.empty_cache()
    need = N * K * 2 + N * K * bits // 8 + N * 4 + int(B.lib.dymoe_gptq_workspace_bytes(N, K)) + (8 << 30)
    if torch.cuda.mem_get_info()[0] < need:
        pytest.skip("needs %d GB of free device memory" % (need >> 30))
    g = torch.Generator(device=DEV).manual_seed(29)
    some = (torch.randn((rows, K), generator=g, device=DEV) * 0.02).bfloat16()
    u = (torch.eye(K, device=DEV) + 0.1 * torch.randn((K, K), generator=g, device=DEV).triu(1)).contiguous()
    want = ctx.gptq_quantize_pack(some, u, bits)
    w = torch.empty((N, K), dtype=torch.bfloat16, device=DEV)
    for r in range(0, N, rows):
        w[r:r + rows] = some[:min(rows, N - r)]
    ws = torch.empty((int(B.lib.dymoe_gptq_workspace_bytes(N, K)),), dtype=torch.uint8, device=DEV)
    out = tuple(torch.full(s, 0, dtype=t, device=DEV) for s, t in (((N, K * bits // 8), torch.uint8), ((N, 1), torch.float16), ((N, 1), torch.float16)))
    got = ctx.gptq_quantize_pack(w, u, bits, out=out, workspace=ws)
    torch.cuda.synchronize()
    same = all(torch.equal(a[r:r + rows], b[:min(rows, N - r)]) for r in range(0, N, rows) for a, b in zip(got, want))
    del w, ws, out, got
    torch.cuda.empty_cache()
    assert same
