"""GPU parity of the retention-gate forward (Sec. 4.1, weight-tied gates) against the fp64 oracle.

The path is floating point throughout: bf16 weights and inputs, fp32 accumulation on the matrix
cores, the hidden activations carried to 16 mantissa bits into the second layer.  Tolerance:
|log beta_gpu - log beta_ref| <= 2e-4 |log beta_ref|: d(log beta)/dz = sigmoid(-z) <= |log beta|, so
the relative error of log beta is at most the absolute error of the gate logit z, and fp32
accumulation over <= 4608 products (about sqrt(n) 2^-24 of the summed magnitudes) plus the 2^-17
split keep that near 1e-5 for the logits of the synthetic gates (|z| < 20); the tests print what
they measure (1e-6 .. 2e-5).
"""
import numpy as np
import pytest
import torch

import kvtrim_inputs as ki
import oracle
import paper_2605_09649_amd as kv
from helpers import bf16_bits

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
RTOL = 2e-4


def run_both(L, H, d_model, d_g, d_p, n_tok, b_g=3.5, layer_begin=0, layer_end=None, horizon=None, salt=0, pick=None):
    """GPU on all n_tok tokens; the oracle on all of them, or on the tokens listed in `pick` (a token's
    gates do not depend on the other tokens of the call) - the GPU rows are then cut to the same list."""
    layer_end = L if layer_end is None else layer_end
    w = ki.gate_weights(L, H, d_model, d_g, d_p, b_g=b_g, seed=1234 + salt)
    x = ki.gate_inputs(L, n_tok, d_model, salt=salt)[layer_begin:layer_end].contiguous()
    og = oracle.Gate(bf16_bits(w["w1"]), w["c1"].numpy(), bf16_bits(w["w2"]), w["c2"].numpy(), w["w_g"].numpy(), b_g)
    x_ref = x if pick is None else x[:, pick].contiguous()
    z_ref, lb_ref, lt_ref = oracle.gate_forward(og, bf16_bits(x_ref), layer_begin, layer_end, horizon)
    ctx = kv.Context(1, L, H, H, 64, 1024)
    gate = kv.Gate.from_dict(w, DEV)
    nl = layer_end - layer_begin
    scratch = torch.empty(kv.kvtrim_gate_scratch_bytes(gate, n_tok, nl) // 4, dtype=torch.float32, device=DEV)
    lb = torch.full((n_tok, L, H), float("nan"), dtype=torch.float32, device=DEV)
    lt = torch.full((n_tok, L, H), float("nan"), dtype=torch.float32, device=DEV) if horizon is not None else None
    kv.kvtrim_gate_forward(ctx, gate, x.to(DEV), n_tok, layer_begin, layer_end, 0 if horizon is None else horizon,
                           scratch, lb, lt)
    assert kv.kvtrim_poll_error(ctx) == 0
    if pick is not None:
        lb = lb[pick]
        lt = None if lt is None else lt[pick]
    return z_ref, lb_ref, lt_ref, lb.cpu().numpy(), None if lt is None else lt.cpu().numpy()


def rel_err(got, ref):
    return float(np.max(np.abs(got.astype(np.float64) - ref) / np.abs(ref)))


@pytest.mark.parametrize("L,H,d_model,d_g,d_p,n_tok", [
    (2, 2, 256, 64, 1, 1),            # smallest legal sizes, scalar projection: per-token kernels
    (3, 2, 512, 128, 7, 5),           # ... d_p not a multiple of the 16-row tile
    (2, 4, 1024, 512, 128, 16),       # ... the paper's hidden width, one full token tile
    (2, 2, 256, 576, 40, 17),         # folded, sliced kernel: hidden width above 512, token tail of one
    (1, 2, 512, 64, 33, 20),          # ... two token tiles per block
    (1, 2, 512, 64, 33, 64),          # ... four token tiles in one block
    (1, 2, 512, 64, 33, 150),         # ... three blocks along the tokens, ragged tail
    (2, 2, 256, 192, 16, 300),        # ... hidden width not a multiple of 128
    (1, 2, 256, 576, 8, 256),         # ... full token tiles, hidden width above 512
    (1, 1, 1024, 512, 128, 257),      # ... the paper's hidden width, one token beyond four 64-token blocks
    (2, 3, 512, 128, 20, 300),        # folded prefill kernel: one 16-row tile per wavefront, three heads, W1 from its copy in the scratch
    (9, 2, 256, 256, 16, 260),        # ... nine layers: the second round of the layer-to-XCD dealing is partly empty
    (1, 8, 256, 384, 5, 513),         # sliced kernel: eight heads, token tail of one
    (3, 2, 256, 512, 1, 256),         # ... scalar projection
    (2, 2, 512, 128, 9, 129),         # folded prefill kernel: 32-token blocks, a tail of one, W1 straight from its rows
    (2, 2, 256, 512, 16, 300),        # sliced kernel: the paper's hidden width, short rows
    (32, 2, 1280, 128, 8, 520),       # folded prefill kernel: 64-token blocks (32 layers x 9 tiles), W1 straight from its rows
])
def test_gate_forward_matches_the_oracle(L, H, d_model, d_g, d_p, n_tok):
    z_ref, lb_ref, _, lb, _ = run_both(L, H, d_model, d_g, d_p, n_tok, salt=d_p)
    assert np.isfinite(lb).all() and (lb <= 0).all()
    err = rel_err(lb, lb_ref)
    print(f"max relative error of log beta: {err:.2e} (logits {z_ref.min():.2f} .. {z_ref.max():.2f})")
    assert err <= RTOL


def test_layer_range_leaves_other_layers_alone():
    _, lb_ref, _, lb, _ = run_both(4, 2, 256, 64, 16, 3, layer_begin=1, layer_end=3)
    assert np.isnan(lb[:, 0, :]).all() and np.isnan(lb[:, 3, :]).all()
    assert rel_err(lb[:, 1:3, :], lb_ref[:, 1:3, :]) <= RTOL


@pytest.mark.parametrize("horizon", [1, 2, 5, 0])
def test_horizon_tail_constant(horizon):
    # Eq. global_score: the factor sum_{k<H} beta^k, cached in log form with log beta
    _, lb_ref, lt_ref, lb, lt = run_both(2, 2, 256, 128, 32, 9, b_g=1.0, horizon=horizon)
    assert rel_err(lb, lb_ref) <= RTOL
    assert np.max(np.abs(lt - lt_ref)) <= 1e-3 * np.max(np.abs(lt_ref)) + 1e-6
    if horizon == 1:
        assert np.array_equal(lt, np.zeros_like(lt))


def test_prefill_sized_call_with_a_layer_range_and_a_horizon():
    # the folded prefill kernel: layers outside the range stay untouched, the tail constant follows log beta
    _, lb_ref, lt_ref, lb, lt = run_both(5, 2, 256, 128, 12, 300, b_g=1.0, layer_begin=1, layer_end=4, horizon=2)
    assert np.isnan(lb[:, 0, :]).all() and np.isnan(lb[:, 4, :]).all()
    assert np.isnan(lt[:, 0, :]).all() and np.isnan(lt[:, 4, :]).all()
    assert rel_err(lb[:, 1:4, :], lb_ref[:, 1:4, :]) <= RTOL
    assert np.max(np.abs(lt[:, 1:4, :] - lt_ref[:, 1:4, :])) <= 1e-3 * np.max(np.abs(lt_ref[:, 1:4, :])) + 1e-6


def test_both_paths_agree_across_the_token_threshold():
    # 16 tokens run the per-token kernels, more the folded ones: the shared tokens get the same gates to rounding
    L, H, d_model, d_g, d_p = 2, 2, 512, 256, 24
    w = ki.gate_weights(L, H, d_model, d_g, d_p, b_g=3.5, seed=77)
    x = ki.gate_inputs(L, 128, d_model, salt=3)
    og = oracle.Gate(bf16_bits(w["w1"]), w["c1"].numpy(), bf16_bits(w["w2"]), w["c2"].numpy(), w["w_g"].numpy(), 3.5)
    _, lb_ref, _ = oracle.gate_forward(og, bf16_bits(x), 0, L, None)
    ctx = kv.Context(1, L, H, H, 64, 1024)
    gate = kv.Gate.from_dict(w, DEV)
    got = {}
    for n_tok in (16, 17, 127, 128):
        xd = x[:, :n_tok].contiguous().to(DEV)
        scratch = torch.empty(kv.kvtrim_gate_scratch_bytes(gate, n_tok, L) // 4, dtype=torch.float32, device=DEV)
        lb = torch.full((n_tok, L, H), float("nan"), dtype=torch.float32, device=DEV)
        kv.kvtrim_gate_forward(ctx, gate, xd, n_tok, 0, L, 1, scratch, lb, None)
        assert kv.kvtrim_poll_error(ctx) == 0
        got[n_tok] = lb.cpu().numpy()
        assert rel_err(got[n_tok], lb_ref[:n_tok]) <= RTOL
    for n_tok in (16, 17, 127):
        assert np.max(np.abs(got[n_tok] - got[128][:n_tok]) / np.abs(lb_ref[:n_tok])) <= RTOL


@pytest.mark.parametrize("d_g,n_tok", [(64, 4), (128, 130)])     # per-token kernels; folded kernel
def test_initial_bias_of_eighteen_keeps_beta_next_to_one(d_g, n_tok):
    # Sec. 5.1: b_g starts at 18.0 - log beta is about -1.5e-8 and must not flush to 0 or lose its digits
    z_ref, lb_ref, _, lb, _ = run_both(2, 2, 256, d_g, 16, n_tok, b_g=18.0)
    assert (lb < 0).all() and rel_err(lb, lb_ref) <= 2e-3 * np.max(np.abs(z_ref))   # d(log beta)/log beta = -dz here


def test_full_size_gate_one_token_and_sixteen():
    # the benchmark model: 32 layers x 8 KV heads, d_model 4096, hidden width 512 (Sec. 5.1), d_p 128
    for n_tok in (1, 16):
        z_ref, lb_ref, _, lb, _ = run_both(32, 8, 4096, 512, 128, n_tok, salt=n_tok)
        err = rel_err(lb, lb_ref)
        print(f"n_tok {n_tok}: max relative error of log beta {err:.2e}")
        assert err <= RTOL


def test_full_size_gate_prefill_chunk_on_sampled_tokens():
    # a 2048-token chunk through the benchmark model; the oracle takes 12 of its tokens (tile edges and interiors)
    pick = [0, 1, 15, 16, 127, 128, 1000, 1023, 1024, 1500, 2046, 2047]
    z_ref, lb_ref, _, lb, _ = run_both(32, 8, 4096, 512, 128, 2048, salt=7, pick=pick)
    err = rel_err(lb, lb_ref)
    print(f"2048 tokens, {len(pick)} sampled: max relative error of log beta {err:.2e}")
    assert err <= RTOL


@pytest.mark.parametrize("L,H,d_model,d_g,d_p,n_toks", [
    (3, 2, 256, 64, 7, (1, 5, 20, 150)),          # sliced kernel; hidden width not for the prefill kernel
    (2, 3, 512, 128, 20, (16, 23, 24, 127, 300)),  # sliced kernel, then the prefill kernel's 32-token blocks from the prepared tiles
    (32, 2, 1280, 128, 8, (520,)),                 # 64-token blocks from the prepared tiles
    (2, 8, 256, 512, 16, (1, 7, 16, 64, 513, 1100)),   # the paper's hidden width, eight heads: slices, then prefill blocks
    (2, 17, 256, 64, 4, (3,)),                     # more than 16 heads: slices of 32 units, whose parts fit the scratch buffer
    (2, 2, 256, 576, 8, (256,)),                   # hidden width above 512
])
def test_prepared_gate_matches_the_oracle_and_is_reusable(L, H, d_model, d_g, d_p, n_toks):
    w = ki.gate_weights(L, H, d_model, d_g, d_p, b_g=3.5, seed=99 + d_p)
    og = oracle.Gate(bf16_bits(w["w1"]), w["c1"].numpy(), bf16_bits(w["w2"]), w["c2"].numpy(), w["w_g"].numpy(), 3.5)
    ctx = kv.Context(1, L, H, H, 64, 1024)
    gate = kv.Gate.from_dict(w, DEV)
    nbytes = kv.kvtrim_gate_prepared_bytes(gate, L, H)
    assert nbytes >= L * d_g * d_model * 2 + L * H * (d_g + 1) * 4
    prepared = torch.empty(nbytes // 4, dtype=torch.float32, device=DEV)
    kv.kvtrim_gate_prepare(ctx, gate, prepared)                   # once; every call below reuses it
    for n_tok in n_toks:
        x = ki.gate_inputs(L, n_tok, d_model, salt=n_tok)
        pick = None if n_tok * L * d_g * d_model < 3e9 else sorted({0, 1, 63, 64, n_tok // 2, n_tok - 1})
        x_ref = x if pick is None else x[:, pick].contiguous()
        for lo, hi in ((0, L), (L // 2, L)):
            _, lb_ref, lt_ref = oracle.gate_forward(og, bf16_bits(x_ref[lo:hi].contiguous()), lo, hi, 2)
            scratch = torch.empty(kv.kvtrim_gate_scratch_bytes(gate, n_tok, hi - lo) // 4, dtype=torch.float32, device=DEV)
            lb = torch.full((n_tok, L, H), float("nan"), dtype=torch.float32, device=DEV)
            lt = torch.full((n_tok, L, H), float("nan"), dtype=torch.float32, device=DEV)
            kv.kvtrim_gate_forward_prepared(ctx, gate, prepared, x[lo:hi].contiguous().to(DEV), n_tok, lo, hi, 2, scratch, lb, lt)
            assert kv.kvtrim_poll_error(ctx) == 0
            if n_tok <= 16:                                       # (the last block of a layer adds the parts of the readout: always in the same order)
                lb2 = torch.full((n_tok, L, H), float("nan"), dtype=torch.float32, device=DEV)
                kv.kvtrim_gate_forward_prepared(ctx, gate, prepared, x[lo:hi].contiguous().to(DEV), n_tok, lo, hi, 2, scratch, lb2, None)
                assert torch.equal(lb[:, lo:hi], lb2[:, lo:hi])
            lb_h, lt_h = lb.cpu().numpy(), lt.cpu().numpy()
            assert np.isnan(lb_h[:, :lo, :]).all()                # layers outside the range stay untouched
            if pick is not None:
                lb_h, lt_h = lb_h[pick], lt_h[pick]
            assert rel_err(lb_h[:, lo:hi], lb_ref[:, lo:hi]) <= RTOL, (n_tok, lo, hi)
            assert np.max(np.abs(lt_h[:, lo:hi] - lt_ref[:, lo:hi])) <= 1e-3 * np.max(np.abs(lt_ref[:, lo:hi])) + 1e-6


def test_host_side_argument_checks_of_the_gate():
    L, H = 2, 2
    w = ki.gate_weights(L, H, 256, 64, 8)
    ctx = kv.Context(1, L, H, H, 64, 1024)
    gate = kv.Gate.from_dict(w, DEV)
    x = ki.gate_inputs(L, 2, 256).to(DEV)
    scratch = torch.empty(2 * L * 64, dtype=torch.float32, device=DEV)
    lb = torch.zeros(2, L, H, dtype=torch.float32, device=DEV)
    with pytest.raises(kv.KvtrimError):
        kv.kvtrim_gate_forward(ctx, gate, x, 0, 0, L, 1, scratch, lb)              # no token
    with pytest.raises(kv.KvtrimError):
        kv.kvtrim_gate_forward(ctx, gate, x, 2, 0, L + 1, 1, scratch, lb)          # layer range beyond the model
    with pytest.raises(kv.KvtrimError):
        kv.kvtrim_gate_forward(ctx, gate, x, 2, 0, L, 5000, scratch, lb)           # horizon out of range
    with pytest.raises(kv.KvtrimError):
        kv.kvtrim_gate_forward(ctx, gate, x, 2, 0, L, 1, None, lb)                 # no scratch
    w_bad = ki.gate_weights(L, H, 128, 64, 8)
    with pytest.raises(kv.KvtrimError):                                            # d_model not a multiple of 256
        kv.kvtrim_gate_forward(ctx, kv.Gate.from_dict(w_bad, DEV), x, 2, 0, L, 1, scratch, lb)
    assert kv.kvtrim_gate_scratch_bytes(gate, 2, L) == 2 * L * 64 * 4
    assert kv.kvtrim_gate_scratch_bytes(gate, 0, L) == 0
    assert kv.kvtrim_gate_prepared_bytes(gate, 0, H) == 0 and kv.kvtrim_gate_prepared_bytes(gate, L, H) > 0
    with pytest.raises(kv.KvtrimError):
        kv.kvtrim_gate_prepare(ctx, gate, None)                                    # no buffer
    prepared = torch.empty(kv.kvtrim_gate_prepared_bytes(gate, L, H) // 4, dtype=torch.float32, device=DEV)
    kv.kvtrim_gate_prepare(ctx, gate, prepared)
    with pytest.raises(kv.KvtrimError):
        kv.kvtrim_gate_forward_prepared(ctx, gate, None, x, 2, 0, L, 1, scratch, lb)   # no prepared buffer
    with pytest.raises(kv.KvtrimError):
        kv.kvtrim_gate_forward_prepared(ctx, gate, prepared, x, 2, 1, 1, 1, scratch, lb)   # empty layer range
    kv.kvtrim_gate_forward_prepared(ctx, gate, prepared, x, 2, 0, L, 1, scratch, lb)
    assert kv.kvtrim_poll_error(ctx) == 0


@pytest.mark.parametrize("L,H,d_model,d_g,n_tok,prepared,kernel", [
    (2, 3, 256, 64, 1, True, "k_gate_slice"),        # slices of 16 units, eight shares of four steps: half of them have none
    (2, 9, 768, 192, 15, True, "k_gate_slice"),      # twelve steps in eight shares, more heads than wavefronts
    (2, 32, 256, 128, 16, True, "k_gate_slice"),     # the most heads, a full token tile
    (2, 33, 256, 128, 16, True, "k_gate_hidden"),    # ... one more: the two-kernel path
    (1, 33, 512, 64, 20, True, "k_gate_hidden"),     # ... with two token tiles per block
    (1, 33, 512, 64, 64, True, "k_gate_hidden"),     # ... with four
    (1, 33, 512, 64, 150, True, "k_gate_hidden"),    # ... three blocks along the tokens
    (2, 33, 256, 192, 300, True, "k_gate_hidden"),   # ... its LDS-tiled first layer: 1.5 row tiles, 2.3 token tiles
    (1, 33, 512, 64, 20, False, "k_gate_hidden"),    # the same without prepared weights, second layer on the matrix cores
    (1, 33, 512, 64, 64, False, "k_gate_hidden"),
    (1, 33, 512, 64, 150, False, "k_gate_hidden"),
    (2, 33, 256, 192, 300, False, "k_gate_hidden"),
    (1, 33, 256, 576, 256, False, "k_gate_hidden"),  # hidden width beyond one staged chunk of the readout
    (6, 2, 256, 512, 33, True, "k_gate_slice"),      # four token tiles, slices of 32 units
    (9, 2, 512, 512, 31, True, "k_gate_slice"),      # two token tiles, slices of 32 units
    (33, 2, 256, 512, 17, True, "k_gate_slice"),     # two token tiles, slices of 64 units, more blocks than compute units
    (33, 1, 256, 512, 2, True, "k_gate_slice"),      # one token tile, slices of 64 units
    (20, 9, 256, 512, 65, True, "k_gate_slice"),     # two blocks of 64 tokens or one of 128, a tail of one
    (33, 2, 1024, 576, 130, True, "k_gate_slice"),   # 128-token blocks, hidden width above 512
    (1, 2, 256, 64, 700, True, "k_gate_slice"),      # eleven 64-token blocks along the tokens
    (2, 8, 1024, 192, 1025, True, "k_gate_slice"),   # seventeen 64-token blocks, for sixteen counters: 128-token blocks
    (1, 2, 256, 64, 2048, True, "k_gate_slice"),     # sixteen 128-token blocks
    (1, 2, 256, 64, 8193, True, "k_gate_hidden"),    # more token tiles than there are counters
    (3, 2, 256, 192, 40, False, "k_gate_slice"),     # vectors folded in the call, W1 straight from its rows
    (2, 8, 256, 64, 17, False, "k_gate_slice"),      # ... the scratch buffer just holds vectors and parts
    (2, 16, 256, 64, 17, False, "k_gate_hidden"),    # ... and with twice the heads it does not
    (2, 16, 512, 512, 22, False, "k_gate_slice"),    # ... holds them with slices of 64 units only
    (2, 16, 512, 512, 21, False, "k_gate_hidden"),   # ... and not even then
    (8, 2, 1024, 384, 519, True, "k_gate_prefill"),  # 32-token blocks
    (4, 2, 256, 128, 2049, True, "k_gate_prefill"),  # 32-token blocks of 128 units, a little over one per compute unit
    (40, 1, 256, 512, 641, True, "k_gate_prefill"),  # 64- or 128-token blocks
    (40, 1, 256, 512, 900, False, "k_gate_prefill"),  # 128-token blocks, everything derived in the call
])
def test_gate_path_by_tokens_heads_and_widths(L, H, d_model, d_g, n_tok, prepared, kernel):
    # every path a call can take, at the sizes where its tiles, shares and slices end
    w = ki.gate_weights(L, H, d_model, d_g, 5, b_g=3.5, seed=31 + n_tok)
    og = oracle.Gate(bf16_bits(w["w1"]), w["c1"].numpy(), bf16_bits(w["w2"]), w["c2"].numpy(), w["w_g"].numpy(), 3.5)
    x = ki.gate_inputs(L, n_tok, d_model, salt=n_tok)
    pick = sorted({i for i in (0, 1, 15, 16, 63, 64, 127, 128, n_tok // 2, n_tok - 2, n_tok - 1) if 0 <= i < n_tok})
    ctx = kv.Context(1, L, H, H, 64, 1024)
    gate = kv.Gate.from_dict(w, DEV)
    scratch = torch.empty(kv.kvtrim_gate_scratch_bytes(gate, n_tok, L) // 4, dtype=torch.float32, device=DEV)
    prep = torch.empty(kv.kvtrim_gate_prepared_bytes(gate, L, H) // 4, dtype=torch.float32, device=DEV)
    if prepared:
        kv.kvtrim_gate_prepare(ctx, gate, prep)
    names = [kv.kvtrim_kernel_name(i) for i in range(40)]
    mask = sum(1 << i for i, n in enumerate(names) if n.startswith("k_gate"))
    _, lb_ref, lt_ref = oracle.gate_forward(og, bf16_bits(x[:, pick].contiguous()), 0, L, 2)
    outs = []
    for again in range(2):                                        # (the arrival counters are back at zero; same bits)
        lb = torch.full((n_tok, L, H), float("nan"), dtype=torch.float32, device=DEV)
        lt = torch.full((n_tok, L, H), float("nan"), dtype=torch.float32, device=DEV)
        kv.kvtrim_profile_begin(ctx, mask)
        if prepared:
            kv.kvtrim_gate_forward_prepared(ctx, gate, prep, x.to(DEV), n_tok, 0, L, 2, scratch, lb, lt)
        else:
            kv.kvtrim_gate_forward(ctx, gate, x.to(DEV), n_tok, 0, L, 2, scratch, lb, lt)
        assert kernel in kv.kvtrim_profile_end(ctx)
        outs.append(lb.cpu())
        assert torch.isfinite(lb).all() and torch.isfinite(lt).all()
        assert rel_err(lb[pick].cpu().numpy(), lb_ref) <= RTOL
        assert np.max(np.abs(lt[pick].cpu().numpy() - lt_ref)) <= 1e-3 * np.max(np.abs(lt_ref)) + 1e-6
    assert torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("n_tok", [12, 64])
def test_sliced_kernel_is_as_exact_as_the_two_kernels(n_tok):
    # 32 heads take k_gate_slice, 33 k_gate_hidden + k_gate_dot, which sum a pre-activation in four chains and add a
    # readout's constant last: the gates that both compute must be as close to 64 bits either way.  (17 layers: slices of
    # 64 units, with the fewest shares of the contraction.  Errors are those of some thousand sums, so their 2-norms vary
    # by a few per cent; two chains instead of four gave 1.3 times the error.)
    L, d_model, d_g = 17, 2048, 512
    w = ki.gate_weights(L, 33, d_model, d_g, 4, b_g=3.5, seed=5)
    og = oracle.Gate(bf16_bits(w["w1"]), w["c1"].numpy(), bf16_bits(w["w2"]), w["c2"].numpy(), w["w_g"].numpy(), 3.5)
    x = ki.gate_inputs(L, n_tok, d_model, salt=6)
    pick = list(range(0, n_tok, max(1, n_tok // 16)))
    _, ref, _ = oracle.gate_forward(og, bf16_bits(x[:, pick].contiguous()), 0, L, None)
    names = [kv.kvtrim_kernel_name(i) for i in range(40)]
    mask = sum(1 << i for i, n in enumerate(names) if n.startswith("k_gate"))
    err = {}
    for H, kernel in ((33, "k_gate_hidden"), (32, "k_gate_slice")):
        wh = dict(w, w2=w["w2"][:, :H].contiguous(), c2=w["c2"][:, :H].contiguous())
        ctx = kv.Context(1, L, H, H, 64, 1024)
        gate = kv.Gate.from_dict(wh, DEV)
        prep = torch.empty(kv.kvtrim_gate_prepared_bytes(gate, L, H) // 4, dtype=torch.float32, device=DEV)
        scratch = torch.empty(kv.kvtrim_gate_scratch_bytes(gate, n_tok, L) // 4, dtype=torch.float32, device=DEV)
        lb = torch.zeros(n_tok, L, H, dtype=torch.float32, device=DEV)
        kv.kvtrim_gate_prepare(ctx, gate, prep)
        kv.kvtrim_profile_begin(ctx, mask)
        kv.kvtrim_gate_forward_prepared(ctx, gate, prep, x.to(DEV), n_tok, 0, L, 1, scratch, lb)
        assert kernel in kv.kvtrim_profile_end(ctx)
        d = lb[pick][:, :, :32].cpu().numpy().astype(np.float64) - ref[:, :, :32]
        err[H] = np.linalg.norm(d) / np.linalg.norm(ref[:, :, :32])
    print(f"two kernels {err[33]:.2e}, sliced {err[32]:.2e}")
    assert err[32] <= 1.1 * err[33]


# W1 prepared or copied in the call (+ 1000), or straight from its rows; every width that the kernel has
@pytest.mark.parametrize("L,n_tok,d_model,d_g,prepared,w1", [
    (24, 4090, 2048, 512, True, 1000), (16, 3113, 4096, 128, False, 1000), (32, 1577, 4096, 128, False, 0), (34, 1205, 4096, 256, False, 0),
    (22, 3001, 3072, 384, False, 1000)])
def test_calls_whose_rows_bypass_the_caches_give_the_same_bits(L, n_tok, d_model, d_g, prepared, w1):
    # more than 300 MB of token rows are loaded past the caches; the same layers in two calls are not.  Both in blocks of 128
    # tokens, as the library's own plan says.
    for layers, rows in ((L, 2000), (L // 2, 0)):
        assert kv.load_library().kvtrim_internal_gate_prefill(2, d_model, d_g, n_tok, layers, int(prepared)) == 128 + w1 + rows
    g = torch.Generator(device=DEV).manual_seed(n_tok)
    H = 2
    w = {k: v.to(DEV) for k, v in ki.gate_weights(L, H, d_model, d_g, 4, b_g=3.5, seed=9).items() if torch.is_tensor(v)}
    gate = kv.Gate(w["w1"], w["c1"], w["w2"], w["c2"], w["w_g"], 3.5)
    x = torch.randn(L, n_tok, d_model, generator=g, device=DEV, dtype=torch.bfloat16)
    assert x.numel() * 2 > 300 << 20 and x[:L // 2].numel() * 2 <= 300 << 20
    ctx = kv.Context(1, L, H, H, 64, 1024)
    scratch = torch.empty(kv.kvtrim_gate_scratch_bytes(gate, n_tok, L), dtype=torch.uint8, device=DEV)
    prep = torch.empty(kv.kvtrim_gate_prepared_bytes(gate, L, H), dtype=torch.uint8, device=DEV)
    kv.kvtrim_gate_prepare(ctx, gate, prep)
    one, two = (torch.full((n_tok, L, H), float("nan"), device=DEV) for _ in range(2))
    for out, ranges in ((one, [(0, L)]), (two, [(0, L // 2), (L // 2, L)])):
        for lo, hi in ranges:
            part = x[lo:hi].contiguous()
            if prepared:
                kv.kvtrim_gate_forward_prepared(ctx, gate, prep, part, n_tok, lo, hi, 1, scratch, out, None)
            else:
                kv.kvtrim_gate_forward(ctx, gate, part, n_tok, lo, hi, 1, scratch, out, None)
    assert kv.kvtrim_poll_error(ctx) == 0 and torch.isfinite(one).all()
    assert torch.equal(one, two)
    pick = torch.tensor([0, 15, 16, n_tok - 1], device=DEV)
    for layer in (0, L - 1):
        u = x[layer, pick].double() @ w["w1"][layer].double().t() + w["c1"][layer].double()
        p = torch.einsum("tu,hpu->thp", u * torch.sigmoid(u), w["w2"][layer].double()) + w["c2"][layer].double()
        ref = torch.nn.functional.logsigmoid(p @ w["w_g"].double() + 3.5)
        assert rel_err(one[pick, layer].cpu().numpy(), ref.cpu().numpy()) <= RTOL
