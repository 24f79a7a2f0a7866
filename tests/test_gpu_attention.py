"""GPU parity of the attention-derived token score (paper Sec. 4.2.1, first
equation) against the CPU oracle, and its hand-over to the importance step."""
import numpy as np
import pytest
import torch

from oracle import dymoe_oracle as O
from paper_2603_19172_amd import binding as B
from paper_2603_19172_amd import synth
from gpu_helpers import DEV

pytestmark = pytest.mark.gpu

# fp32 accumulation of exact bf16 products over d <= 128 terms, v_exp_f32 on arguments of
# magnitude <= ~40, sums of <= 2048 probabilities: a few 1e-6 relative on every score
RTOL, ATOL = 2e-5, 1e-9


@pytest.fixture(scope="module")
def ctx():
    c = B.Context(0)
    yield c
    c.close()


def _dev3(bits):
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).to(DEV).view(torch.bfloat16)


def _run(ctx, q, k, causal, scale=0.0):
    s = ctx.token_score_attention(_dev3(q), _dev3(k), causal=causal, scale=scale)
    torch.cuda.synchronize()
    return s.cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("T,Hh,Hkv,d", [(16, 2, 2, 64), (77, 4, 2, 128), (1, 2, 1, 64), (33, 3, 3, 64),
                                        (160, 8, 2, 128), (512, 32, 8, 128),
                                        # many tokens, few heads (operands straight from memory, but for the last and for 2048
                                        # unmasked): ragged ends, a head count the XCD mapping does not divide, both head sizes
                                        (993, 8, 2, 128), (1100, 3, 3, 64), (1057, 5, 1, 128), (2048, 8, 8, 64),
                                        (4100, 2, 1, 128)])
@pytest.mark.parametrize("causal", [True, False])
def test_attention_score_matches_the_oracle(ctx, T, Hh, Hkv, d, causal):
    cfg = synth.scaled(synth.CONFIGS["mixtral_prefill"], T=T, k_hh=max(1, T // 20), config_id=60 + T)
    q, k, heavy = synth.attention_inputs(cfg, Hh, Hkv, d, boost=1.0)
    ref = O.token_score_attention(q, k, Hh, Hkv, causal=causal)
    got = _run(ctx, q, k, causal)
    assert np.isfinite(got).all()
    err = np.abs(got - ref) / (np.abs(ref) + ATOL / RTOL)
    print("T=%d heads=%d/%d d=%d causal=%d: max rel err %.2e, sum %.8f" % (T, Hh, Hkv, d, causal, err.max(), got.sum()))
    assert np.allclose(got, ref, rtol=RTOL, atol=ATOL)
    assert abs(got.sum() - 1.0) < 1e-5                      # every query hands out one unit of attention


# the LDS-staged kernels: stages of the stream that end whole, half and ragged, head counts that the XCD mapping divides and does not
@pytest.mark.parametrize("T,Hh,Hkv,d", [(1024, 16, 4, 128), (1025, 16, 4, 128), (1057, 17, 1, 64), (1088, 24, 6, 64),
                                        (1120, 20, 5, 128), (2111, 8, 2, 128), (1100, 32, 8, 128), (1500, 32, 8, 128),
                                        (1500, 32, 8, 64), (4200, 8, 2, 64)])
@pytest.mark.parametrize("causal", [True, False])
def test_attention_score_staged_kernels(ctx, T, Hh, Hkv, d, causal):
    cfg = synth.scaled(synth.CONFIGS["mixtral_prefill"], T=T, k_hh=max(1, T // 20), config_id=160 + T)
    q, k, heavy = synth.attention_inputs(cfg, Hh, Hkv, d, boost=1.0)
    ref = O.token_score_attention(q, k, Hh, Hkv, causal=causal)
    got = _run(ctx, q, k, causal)
    assert np.allclose(got, ref, rtol=RTOL, atol=ATOL) and abs(got.sum() - 1.0) < 1e-5


# on both sides of where the rule changes (attention_rule.hpp): the last size of one form and, a fragment of one token more, the first of the
# next; forms as tokens per block in units of 64 (0: operands straight from memory) and wavefronts
AROUND_THE_LINES = [(128, True, 5, 1, 1536, (0, 4), (2, 8)), (128, True, 20, 5, 416, (0, 4), (2, 8)), (128, False, 8, 2, 1024, (0, 4), (2, 8)),
                    (128, True, 32, 8, 288, (0, 4), (2, 4)), (128, True, 32, 8, 1536, (2, 8), (2, 4)), (128, False, 32, 8, 1024, (2, 8), (4, 8)),
                    (128, False, 32, 8, 2048, (4, 8), (2, 4)), (128, True, 32, 8, 3456, (2, 4), (4, 8)), (128, False, 32, 8, 320, (2, 4), (2, 8)),
                    (64, True, 20, 5, 2944, (2, 8), (2, 4)), (64, False, 8, 8, 1280, (0, 4), (2, 8)), (64, True, 8, 2, 2592, (0, 4), (2, 8)),
                    (64, False, 5, 5, 1632, (0, 4), (2, 8)), (64, False, 20, 5, 1536, (2, 8), (2, 4)), (64, True, 33, 11, 1408, (2, 8), (2, 4))]


@pytest.mark.parametrize("d,causal,Hh,Hkv,T,form,form_behind", AROUND_THE_LINES)
def test_attention_score_around_the_lines(ctx, d, causal, Hh, Hkv, T, form, form_behind):
    for tokens in (T, T + 1):
        cfg = synth.scaled(synth.CONFIGS["mixtral_prefill"], T=tokens, k_hh=max(1, T // 20), config_id=560 + tokens)
        q, k, heavy = synth.attention_inputs(cfg, Hh, Hkv, d, boost=1.0)
        ref = O.token_score_attention(q, k, Hh, Hkv, causal=causal)
        got = _run(ctx, q, k, causal)
        assert np.allclose(got, ref, rtol=RTOL, atol=ATOL) and abs(got.sum() - 1.0) < 1e-5


# heads of 64 values in blocks of 128 tokens by eight wavefronts
@pytest.mark.parametrize("T,Hh,Hkv", [(1024, 24, 8), (1025, 24, 8), (6113, 4, 4), (2975, 8, 2)])
@pytest.mark.parametrize("causal", [True, False])
def test_attention_score_small_heads(ctx, T, Hh, Hkv, causal):
    cfg = synth.scaled(synth.CONFIGS["mixtral_prefill"], T=T, k_hh=max(1, T // 20), config_id=260 + T)
    q, k, heavy = synth.attention_inputs(cfg, Hh, Hkv, 64, boost=1.0)
    ref = O.token_score_attention(q, k, Hh, Hkv, causal=causal)
    got = _run(ctx, q, k, causal)
    assert np.allclose(got, ref, rtol=RTOL, atol=ATOL) and abs(got.sum() - 1.0) < 1e-5


# the staged kernels' blocks of 128 tokens; last blocks of one token, one fragment and a fragment and a bit; trips of the stream that end
# whole and in every remainder; wavefronts whose tokens lie past the end
@pytest.mark.parametrize("T,Hh,Hkv,d", [(321, 30, 5, 128), (353, 32, 8, 128), (385, 32, 8, 128), (449, 24, 24, 128), (513, 20, 5, 128),
                                        (1537, 5, 5, 128), (1665, 5, 1, 128), (2048, 32, 8, 128), (1900, 34, 17, 128), (2561, 24, 4, 128),
                                        (673, 32, 8, 64), (705, 30, 10, 64), (1025, 21, 3, 64), (3073, 5, 5, 64), (2049, 32, 4, 64)])
@pytest.mark.parametrize("causal", [True, False])
def test_attention_score_staged_blocks(ctx, T, Hh, Hkv, d, causal):
    cfg = synth.scaled(synth.CONFIGS["mixtral_prefill"], T=T, k_hh=max(1, T // 20), config_id=360 + T)
    q, k, heavy = synth.attention_inputs(cfg, Hh, Hkv, d, boost=1.0)
    ref = O.token_score_attention(q, k, Hh, Hkv, causal=causal)
    got = _run(ctx, q, k, causal)
    assert np.allclose(got, ref, rtol=RTOL, atol=ATOL) and abs(got.sum() - 1.0) < 1e-5


# blocks of 256 tokens, under the mask and without it: last blocks of one token, one fragment, a fragment and a bit, all but one token, and
# wavefronts whose tokens lie past the end; the stream of two sharing wavefronts ends in every remainder
BLOCKS_OF_256 = [(5121, 21, 7, True), (5185, 21, 21, True), (3457, 32, 8, True), (3560, 30, 10, True), (257, 88, 8, False), (290, 88, 11, False),
                 (400, 68, 4, False), (1025, 32, 8, False), (1312, 32, 4, False), (929, 64, 16, False), (1313, 32, 8, False), (900, 33, 3, False)]


@pytest.mark.parametrize("T,Hh,Hkv,causal", BLOCKS_OF_256)
def test_attention_score_blocks_of_256(ctx, T, Hh, Hkv, causal):
    cfg = synth.scaled(synth.CONFIGS["mixtral_prefill"], T=T, k_hh=max(1, T // 20), config_id=660 + T)
    q, k, heavy = synth.attention_inputs(cfg, Hh, Hkv, 128, boost=1.0)
    ref = O.token_score_attention(q, k, Hh, Hkv, causal=causal)
    got = _run(ctx, q, k, causal)
    assert np.allclose(got, ref, rtol=RTOL, atol=ATOL) and abs(got.sum() - 1.0) < 1e-5


# heads of 128 values in blocks of 128 tokens by four wavefronts, two workgroups of which share a compute unit: last blocks of one token, a
# fragment and a bit, three fragments, all but one token; trips of four fragments that end in every remainder
TWO_ON_A_UNIT = [(257, 64, 8, True), (300, 64, 16, True), (900, 64, 8, True), (1025, 64, 8, True), (1056, 64, 16, True), (1070, 64, 64, True),
                 (1279, 64, 8, True), (1536, 64, 4, True), (2600, 33, 11, True), (2625, 32, 8, True), (257, 64, 64, False), (300, 64, 8, False),
                 (1089, 64, 64, False), (1120, 64, 8, False), (1409, 64, 4, False), (1535, 64, 8, False), (2049, 32, 8, False)]


@pytest.mark.parametrize("T,Hh,Hkv,causal", TWO_ON_A_UNIT)
def test_attention_score_two_workgroups_on_a_unit(ctx, T, Hh, Hkv, causal):
    cfg = synth.scaled(synth.CONFIGS["mixtral_prefill"], T=T, k_hh=max(1, T // 20), config_id=760 + T)
    q, k, heavy = synth.attention_inputs(cfg, Hh, Hkv, 128, boost=1.0)
    ref = O.token_score_attention(q, k, Hh, Hkv, causal=causal)
    got = _run(ctx, q, k, causal)
    assert np.allclose(got, ref, rtol=RTOL, atol=ATOL) and abs(got.sum() - 1.0) < 1e-5


# heads of 64 values in so many blocks of 128 tokens that three workgroups of four wavefronts share a compute unit: last blocks of one
# token, a fragment, a fragment and a bit and all but one token, trips of four fragments that end in every remainder
THREE_ON_A_UNIT = [(897, 64, 8, 64), (929, 64, 8, 64), (970, 64, 16, 64), (1023, 64, 64, 64), (1089, 49, 7, 64), (2625, 32, 8, 64)]


@pytest.mark.parametrize("T,Hh,Hkv,d", THREE_ON_A_UNIT)
@pytest.mark.parametrize("causal", [True, False])
def test_attention_score_three_workgroups_on_a_unit(ctx, T, Hh, Hkv, d, causal):
    cfg = synth.scaled(synth.CONFIGS["mixtral_prefill"], T=T, k_hh=max(1, T // 20), config_id=460 + T)
    q, k, heavy = synth.attention_inputs(cfg, Hh, Hkv, d, boost=1.0)
    ref = O.token_score_attention(q, k, Hh, Hkv, causal=causal)
    got = _run(ctx, q, k, causal)
    assert np.allclose(got, ref, rtol=RTOL, atol=ATOL) and abs(got.sum() - 1.0) < 1e-5


@pytest.mark.parametrize("T,Hh,d", [(900, 24, 128), (900, 64, 128), (900, 24, 64), (900, 64, 64)])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("rise", [90.0, -90.0])
def test_attention_score_logits_that_rise_along_the_keys(ctx, T, Hh, d, causal, rise):
    """The staged kernels raise their reference exponent only when a sum outgrows it: logits that climb (and fall) by 90 from the
    first key to the last, so that it is raised many times, or never after the first fragment."""
    q, k = (synth.normal_bf16(77 + T, 9200 + i, (T, Hh, d), 0.5) for i in range(2))
    def values(bits):
        return (bits.astype(np.uint32) << 16).view(np.float32)
    def bf16(x):
        return (np.ascontiguousarray(x, np.float32).view(np.uint32) >> 16).astype(np.uint16)
    qf, kf = values(q).copy(), values(k).copy()
    qf[:, :, 0] = np.sqrt(d)
    kf[:, :, 0] = rise * np.arange(T)[:, None] / T
    q, k = bf16(qf), bf16(kf)
    ref = O.token_score_attention(q, k, Hh, Hh, causal=causal)
    got = _run(ctx, q, k, causal)
    # arguments of the exponentials of up to 130 in base 2: a rounding of 2^-18 there is 5e-6 of a probability
    assert np.allclose(got, ref, rtol=RTOL, atol=ATOL) and abs(got.sum() - 1.0) < 1e-5


@pytest.mark.parametrize("T,Hh,d", [(900, 24, 128), (900, 64, 128), (900, 24, 64), (1025, 32, 128), (3457, 32, 128), (900, 64, 64)])
def test_attention_score_a_query_that_is_no_number_spoils_the_keys_it_sees(ctx, T, Hh, d):
    q, k = (synth.normal_bf16(277 + T, 9300 + i, (T, Hh, d), 1.0) for i in range(2))
    ref = O.token_score_attention(q, k, Hh, Hh, causal=True)
    bad = T // 2 + 5
    q[bad, 3, 7] = 0x7FC0
    got = _run(ctx, q, k, True)
    assert np.isnan(got[:bad + 1]).all()
    assert np.allclose(got[bad + 1:], ref[bad + 1:], rtol=RTOL, atol=ATOL)


# the sum over heads: one or two of them, batches of sixteen, whole, short by one and with one head left
@pytest.mark.parametrize("Hh", [1, 2, 3, 15, 16, 17, 31, 32, 33])
def test_attention_score_sums_every_head_once(ctx, Hh):
    T, d = 70, 64
    q, k = (synth.normal_bf16(180 + Hh, 9100 + i, (T, Hh, d), 1.0) for i in range(2))
    ref = O.token_score_attention(q, k, Hh, Hh, causal=True)
    got = _run(ctx, q, k, True)
    assert np.allclose(got, ref, rtol=RTOL, atol=ATOL)


def test_attention_score_explicit_scale_and_determinism(ctx):
    cfg = synth.scaled(synth.CONFIGS["mixtral_prefill"], T=200, k_hh=10, config_id=71)
    q, k, _ = synth.attention_inputs(cfg, 4, 4, 64)
    ref = O.token_score_attention(q, k, 4, 4, causal=True, scale=0.05)
    a = _run(ctx, q, k, True, scale=0.05)
    b = _run(ctx, q, k, True, scale=0.05)
    assert np.allclose(a, ref, rtol=RTOL, atol=ATOL)
    assert np.array_equal(a, b)                              # fixed summation order, no atomics


def test_attention_score_uniform_closed_form(ctx):
    T, Hh, d = 45, 2, 64
    k = synth.normal_bf16(3, 9001, (T, Hh, d), 1.0)
    q = np.zeros((T, Hh, d), np.uint16)
    got = _run(ctx, q, k, True)
    harm = np.concatenate([[0.0], np.cumsum(1.0 / np.arange(1, T + 1))])
    want = (harm[T] - harm[:T]) / T
    assert np.allclose(got, want, rtol=1e-6)
    assert np.allclose(_run(ctx, q, k, False), 1.0 / T, rtol=1e-6)


def test_attention_score_feeds_the_importance_step(ctx):
    """Eq. 1 -> Eq. 2: heavy hitters found by the attention they receive; the expert importance
    computed from the device's scores equals the oracle's from its own."""
    cfg = synth.scaled(synth.CONFIGS["mixtral_prefill"], T=256, k_hh=13, config_id=41)
    q, k, heavy = synth.attention_inputs(cfg, 8, 2, 64, boost=1.5)
    x, _ = synth.activations(cfg)
    wg, bias = synth.router(cfg)
    ridx, _, _, _ = O.route_topk(x, wg, bias, cfg.k)
    rscore = O.token_score_attention(q, k, 8, 2, causal=False)
    rimp, rload, rheavy = O.expert_importance_prefill(ridx, rscore, cfg.E, cfg.k_hh)
    assert set(np.nonzero(rheavy)[0].tolist()) == set(heavy.tolist())
    score = ctx.token_score_attention(_dev3(q), _dev3(k), causal=False)
    idx = torch.from_numpy(ridx).to(DEV)
    imp, load = ctx.expert_importance(B.PHASE_PREFILL, idx, cfg.E, k_hh=cfg.k_hh, token_score=score)
    torch.cuda.synchronize()
    assert np.array_equal(imp.cpu().numpy(), rimp) and np.array_equal(load.cpu().numpy(), rload)
