"""Mixture-of-experts prefill (Section 7: the `gate` and `experts` operators) through the C ABI
against the oracle.  The router turns floating point into an integer decision: the GPU decides on
fp32 probabilities of bf16 activations, so where two experts are a rounding error apart its choice
may differ from the fp64 oracle's.  The tests therefore read the GPU's selection back, check that
it is a top-k set of the oracle's own probabilities to within that rounding error, and let the
oracle evaluate the experts the GPU chose (with the oracle's own weights for them)."""
import pytest
import torch

from oracle import prefill_oracle as O
from paper_2602_16603_amd import inputs as I
from tests.util import TOL, fro_rel_err, max_rel_err, oracle_layers, oracle_shape

pytestmark = pytest.mark.gpu


def _mods():
    from paper_2602_16603_amd import binding, runner
    return binding, runner


def run_and_check(spec, lengths, seed, pool_blocks):
    B, R = _mods()
    total = sum(lengths)
    weights = I.make_weights(spec, seed, torch.bfloat16, "cpu")
    I.randomize_gains(weights, seed)
    model = R.PrefillModel(spec, weights, B.FP_DTYPE_BF16, pool_blocks, max(max(lengths), 16))
    hidden = I.make_hidden(total, spec.hidden, seed, torch.bfloat16, "cpu")
    task = model.begin(hidden.cuda(), lengths)
    task.run_to_completion()
    got = task.hidden()
    forced = [task.moe_routing(l)[0].cpu() for l in range(spec.n_layers)]
    gpu_wts = [task.moe_routing(l)[1].cpu() for l in range(spec.n_layers)]
    for ids, wts in zip(forced, gpu_wts):
        assert int(ids.min()) >= 0 and int(ids.max()) < spec.n_experts
        srt = torch.sort(ids, dim=-1).values
        assert bool((srt[:, 1:] != srt[:, :-1]).all())                                            # distinct experts, every row
        assert torch.allclose(wts.sum(dim=-1), torch.ones(total), atol=1e-5)
        assert bool((wts[:, :-1] >= wts[:, 1:]).all())                                            # most probable first
    shortfall, ref_wts = [], []
    x_ref, cache_ref = O.prefill(oracle_shape(spec), oracle_layers(weights), hidden, I.cu_seqlens_of(lengths),
                                 forced_ids=forced, shortfall_out=shortfall, weights_out=ref_wts)
    absolute, relative = shortfall[0::2], shortfall[1::2]      # per layer: absolute, then relative to the k-th probability
    worst = max(float(s.max()) for s in absolute) if total else 0.0
    worst_rel = max(float(s.max()) for s in relative) if total else 0.0
    flipped = sum(int((s > 0).sum()) for s in absolute) / max(1, total * spec.n_layers)
    e = max_rel_err(got, x_ref)
    # The GPU's renormalised weights against the oracle's own probabilities of the same experts,
    # element by element (fp32 softmax of bf16 activations against fp64 of fp64 activations).
    w_err = max((float((g.double() - r).abs().max()) for g, r in zip(gpu_wts, ref_wts)), default=0.0) if total else 0.0
    w_fro = max((fro_rel_err(g, r) for g, r in zip(gpu_wts, ref_wts)), default=0.0) if total else 0.0
    print(f"  hidden: E={e:.3e} fro={fro_rel_err(got, x_ref):.3e}; router: worst shortfall {worst:.2e} "
          f"({worst_rel:.2e} of the k-th probability), "
          f"{100 * flipped:.2f}% of token-layers decided the other way; weights: max abs err {w_err:.2e}, "
          f"fro {w_fro:.2e}", flush=True)
    # Only near-ties may differ.  The GPU's router reads the bf16-stored activations (2^-9 relative
    # rounding per element, on top of the layer's accumulated bf16 error), which moves a logit by
    # about 0.2 * sqrt(hidden) * 2^-9 / sqrt(3): 0.004 (hidden 256) to 0.01 (hidden 2048) standard
    # deviations, and the difference of two logits by sqrt(2) of that.  Two experts can change
    # places when their probabilities are within about four such deviations of each other: a
    # relative gap of 6e-2 at the largest shape tested.  Observed: 4.1e-2 there (6.3e-5 absolute:
    # the 8th of 128 probabilities is small), 0.6 % at the 8-expert shape (6.1e-4 absolute).
    assert worst <= 1e-3 and worst_rel <= 6e-2 and flipped <= 0.02
    assert w_err <= 3e-2 and w_fro <= 1e-2
    assert e <= TOL["bf16"]
    for layer in range(spec.n_layers):
        for s in range(len(lengths)):
            k, v = task.kv(layer, s)
            assert max_rel_err(k, cache_ref.k[layer][s]) <= TOL["bf16"]
            assert max_rel_err(v, cache_ref.v[layer][s]) <= TOL["bf16"]
    return model, task, hidden, got


def test_tiny_moe_ragged_batch_matches_oracle_and_repeats_bit_for_bit():
    spec = I.TINY_MOE
    lengths = [300, 17, 0, 513, 64]
    model, task, hidden, got = run_and_check(spec, lengths, 51, pool_blocks=256)
    again = model.begin(hidden.cuda(), lengths)
    again.run_to_completion()
    assert torch.equal(again.hidden(), got)       # slot order inside an expert varies; results must not
    again.end()
    task.end()
    model.close()


def test_moe_preempt_at_every_boundary_resumes_bit_identically():
    B, R = _mods()
    spec = I.TINY_MOE
    lengths = [200, 77]
    weights = I.make_weights(spec, 52, torch.bfloat16, "cuda")
    model = R.PrefillModel(spec, weights, B.FP_DTYPE_BF16, 64, 256)
    hidden = I.make_hidden(sum(lengths), spec.hidden, 52, torch.bfloat16, "cuda")
    ref = model.begin(hidden, lengths)
    ref.run_to_completion()
    want = ref.hidden()
    want_kv = [t for layer in range(spec.n_layers) for t in ref.kv(layer, 0)]
    n_ops = spec.n_layers * B.FP_OPS_PER_LAYER
    for stop in range(1, n_ops):
        task = model.begin(hidden, lengths)
        status, done = task.advance(stop)
        assert status == B.FP_OK and done == stop
        assert task.preempt() == B.FP_PREEMPTED           # idle between advances: parks at once
        assert task.cursor() == (stop // 9, stop % 9)
        task.resume()
        task.run_to_completion()
        assert torch.equal(task.hidden(), want), f"resume after {stop} operators changed the result"
        got_kv = [t for layer in range(spec.n_layers) for t in task.kv(layer, 0)]
        assert all(torch.equal(a, b) for a, b in zip(got_kv, want_kv))
        task.end()
    ref.end()
    model.close()


def test_qwen3_30b_a3b_shaped_layer_matches_oracle():
    """One layer of the 30B-A3B shape (hidden 2048, 32/4 heads of 128, 128 experts of width 768,
    8 per token), 2048 tokens in two prompts: the grouped GEMMs run with ~128 tokens per expert."""
    spec = I.QWEN3_30B_A3B.with_layers(1)
    model, task, _, _ = run_and_check(spec, [1500, 548], 53, pool_blocks=256)
    task.end()
    model.close()


@pytest.mark.parametrize("lengths", [[3], [0], [1, 0, 2]])
def test_moe_with_almost_no_tokens(lengths):
    """Three tokens over eight experts leave most experts without a row (no row tile at all);
    an empty batch launches nothing."""
    B, R = _mods()
    spec = I.TINY_MOE
    if sum(lengths) == 0:
        weights = I.make_weights(spec, 54, torch.bfloat16, "cuda")
        model = R.PrefillModel(spec, weights, B.FP_DTYPE_BF16, 16, 16)
        task = model.begin(torch.empty((0, spec.hidden), dtype=torch.bfloat16, device="cuda"), lengths)
        status, _ = task.advance()
        assert status == B.FP_DONE
        task.end()
        model.close()
        return
    model, task, _, _ = run_and_check(spec, lengths, 54, pool_blocks=16)
    task.end()
    model.close()


def test_moe_shape_validation():
    B, R = _mods()
    import dataclasses
    weights = I.make_weights(I.TINY_MOE, 55, torch.bfloat16, "cuda")
    for bad in (dataclasses.replace(I.TINY_MOE, top_k=0), dataclasses.replace(I.TINY_MOE, top_k=9),
                dataclasses.replace(I.TINY_MOE, n_experts=12, top_k=2)):
        with pytest.raises(B.FlowPrefillError):
            R.PrefillModel(bad, weights, B.FP_DTYPE_BF16, 16, 16)
    with pytest.raises(B.FlowPrefillError):                       # fp32 debug path has no MoE
        R.PrefillModel(I.TINY_MOE, I.make_weights(I.TINY_MOE, 55, torch.float32, "cuda"), B.FP_DTYPE_F32, 16, 16)
    dense = R.PrefillModel(I.TINY, I.make_weights(I.TINY, 55, torch.bfloat16, "cuda"), B.FP_DTYPE_BF16, 16, 16)
    t = dense.begin(I.make_hidden(4, I.TINY.hidden, 1, torch.bfloat16, "cuda"), [4])
    t.run_to_completion()
    with pytest.raises(B.FlowPrefillError):                       # dense model has no routing to report
        t.moe_routing(0)
    t.end()
    dense.close()


@pytest.mark.parametrize("tokens", [40, 150, 300, 500])
def test_expert_row_tiles_of_every_size(tokens):
    """10, 37, 75 and 125 rows per expert on average: the experts' GEMMs run on row tiles of 32, 64, 128
    and 256; the routing is uneven, so some experts open a second tile."""
    model, task, _, _ = run_and_check(I.TINY_MOE, [tokens], 56, pool_blocks=64)
    task.end()
    model.close()


def test_a_router_logit_beyond_the_fp32_range_is_not_hidden():
    """A logit of +inf makes the softmax NaN: that token's weights and output row are NaN, every other row is the
    one of a run without it."""
    B, R = _mods()
    spec = I.TINY_MOE.with_layers(1)
    tokens, row, expert, channel = 70, 33, 3, 5
    weights = I.make_weights(spec, 57, torch.bfloat16, "cpu")
    weights[0]["w_o"].zero_()                          # the router sees the norm of the input itself
    hidden = I.make_hidden(tokens, spec.hidden, 57, torch.bfloat16, "cpu")
    hidden[:, channel] = 0
    hidden[row, channel] = 4.0
    outs = []
    for big in (False, True):
        weights[0]["w_router"][expert] = 0
        weights[0]["w_router"][expert, channel] = 3e38 if big else 0.0
        model = R.PrefillModel(spec, weights, B.FP_DTYPE_BF16, 16, 128)
        task = model.begin(hidden.cuda(), [tokens])
        task.run_to_completion()
        outs.append((task.hidden().cpu(), *(t.cpu() for t in task.moe_routing(0))))
        task.end()
        model.close()
    others = torch.arange(tokens) != row
    (x0, ids0, wts0), (x1, ids1, wts1) = outs
    assert int(ids1.min()) >= 0 and int(ids1.max()) < spec.n_experts
    assert torch.isnan(wts1[row]).all() and torch.isnan(x1[row]).all()
    assert torch.isfinite(x0).all() and torch.equal(ids1[others], ids0[others])
    assert torch.equal(wts1[others], wts0[others]) and torch.equal(x1[others], x0[others])


@pytest.mark.parametrize("ffn,seed", [(192, 61), (128, 62)])
def test_experts_of_unlike_sizes_run_on_large_tiles_of_every_height(ffn, seed):
    """A router that favours some of its 32 experts: from a few rows to several hundred each, so the large tile of the
    experts' GEMMs multiplies 64 to 256 rows in steps of 32, alone and as one of an expert's evenly filled tiles (odd
    multiples of 32 among them; five k-tiles, and three or two; a last column tile that is half outside)."""
    B, R = _mods()
    spec = I.ShapeSpec(1, 320, 4, 2, 64, ffn, 1e-5, 10000.0, n_experts=32, top_k=4)
    n = 1100
    weights = I.make_weights(spec, seed, torch.bfloat16, "cpu")
    weights[0]["w_router"] *= torch.linspace(0.3, 1.6, 32)[:, None].to(torch.bfloat16)
    hidden = I.make_hidden(n, spec.hidden, seed, torch.bfloat16, "cpu")
    model = R.PrefillModel(spec, weights, B.FP_DTYPE_BF16, 128, n)
    print(f"experts of unlike sizes ffn={ffn}", flush=True)
    task = model.begin(hidden.cuda(), [n])
    task.run_to_completion()
    got, ids = task.hidden(), task.moe_routing(0)[0].cpu()
    rows = torch.bincount(ids.flatten().long(), minlength=32).tolist()
    heights = {max(2, -(-(-(-r // -(-r // 256))) // 32)) for r in rows if r}
    assert heights == set(range(2, 9)), rows
    assert max(rows) > 256                                # ... and an expert of more than one tile
    x_ref, _ = O.prefill(oracle_shape(spec), oracle_layers(weights), hidden, [0, n], forced_ids=[ids])
    # Eight intermediates rounded to bf16 (2^-9 each): 1.2e-2 at most, and 1e-2 for their mean square.
    assert fro_rel_err(got, x_ref) <= 1e-2 and max_rel_err(got, x_ref) <= TOL["bf16"]
    task.end()
    model.close()


@pytest.mark.parametrize("ffn,seed", [(192, 61), (128, 62)])
@pytest.mark.parametrize("n", [100, 300, 600, 1100])
def test_what_experts_add_to_each_token(n, ffn, seed):
    """The experts' contribution by itself, token by token and 32 columns at a time, against its definition in 64 bits: 32 to 256-row
    tiles (n / 8 rows per expert on average, from a few to several hundred at n = 1100), every (expert, column tile) starting at
    another of its five, three or two k-tiles.  Attention adds nothing here, so what the layer adds is the experts' sum."""
    B, R = _mods()
    spec = I.ShapeSpec(1, 320, 4, 2, 64, ffn, 1e-5, 10000.0, n_experts=32, top_k=4)
    weights = I.make_weights(spec, seed, torch.bfloat16, "cuda")
    w = weights[0]
    w["w_o"].zero_()
    w["w_router"] *= torch.linspace(0.3, 1.6, 32, device="cuda")[:, None].to(torch.bfloat16)
    x = I.make_hidden(n, spec.hidden, seed, torch.bfloat16, "cuda")
    model = R.PrefillModel(spec, weights, B.FP_DTYPE_BF16, 128, n)
    print(f"experts' contribution n={n} ffn={ffn}", flush=True)
    task = model.begin(x, [n])
    task.run_to_completion()
    ids, wts = task.moe_routing(0)
    h = torch.empty_like(x)
    x32 = x.float()
    torch.cuda.synchronize()
    B.fp_op_rmsnorm(1, x32.data_ptr(), w["mlp_norm"].data_ptr(), h.data_ptr(), n, spec.hidden, spec.rms_eps)
    torch.cuda.synchronize()
    ref = torch.zeros(n, spec.hidden, dtype=torch.float64, device="cuda")
    for e in range(spec.n_experts):
        token, slot = (ids == e).nonzero(as_tuple=True)
        g, u = (h[token].double() @ w["w_gate_up"][e].double().T).split(ffn, dim=1)
        y = (torch.nn.functional.silu(g) * u) @ w["w_down"][e].double().T
        ref.index_add_(0, token, wts[token, slot, None].double() * y)
    off = task.hidden().double() - x.double() - ref
    # Four roundings to bf16 (gate, up, their product, the expert's output), 2^-8 / sqrt(3) in the mean square each, the gate's
    # up to doubled: 6e-3 of a token's contribution, 8e-3 of 32 of its columns at most (computed on the CPU); twice that.  One
    # k-tile left out of one expert's last eight columns is 0.2 and 0.25, a lost row or column tile more.
    assert (off.norm(dim=1) / ref.norm(dim=1)).max().item() <= 1.2e-2
    blocks = (n, spec.hidden // 32, 32)
    assert (off.view(blocks).norm(dim=2) / ref.view(blocks).norm(dim=2)).max().item() <= 1.6e-2
    task.end()
    model.close()


@pytest.mark.parametrize("experts,top_k", [(8, 2), (256, 8)])
@pytest.mark.parametrize("n", [1, 7, 8, 9, 15, 16, 17, 1040, 2047, 2048, 2049, 8192, 8193, 16384, 16385])
def test_every_pair_has_its_row(n, experts, top_k):
    """Route workgroups of 8, 32 and 64 tokens, the last of one token, of all but one and full; their counts added up by every workgroup
    of the plan, or (16385 tokens and more) by one: what the layer adds to every token is its experts' weighted sum."""
    B, R = _mods()
    spec = I.ShapeSpec(1, 192, 2, 1, 64, 64, 1e-5, 10000.0, n_experts=experts, top_k=top_k)
    weights = I.make_weights(spec, 63, torch.bfloat16, "cuda")
    w = weights[0]
    w["w_o"].zero_()
    w["w_router"] *= torch.linspace(0.5, 1.5, experts, device="cuda")[:, None].to(torch.bfloat16)
    x = I.make_hidden(n, spec.hidden, 63, torch.bfloat16, "cuda")
    lengths = [512] * (n // 512) + ([n % 512] if n % 512 else [])
    model = R.PrefillModel(spec, weights, B.FP_DTYPE_BF16, n // 16 + len(lengths) + 8, 512)
    print(f"pairs' rows n={n} experts={experts}", flush=True)
    task = model.begin(x, lengths)
    task.run_to_completion()
    ids, wts = task.moe_routing(0)
    h, x32 = torch.empty_like(x), x.float()
    torch.cuda.synchronize()
    B.fp_op_rmsnorm(1, x32.data_ptr(), w["mlp_norm"].data_ptr(), h.data_ptr(), n, spec.hidden, spec.rms_eps)
    torch.cuda.synchronize()
    ref = torch.zeros(n, spec.hidden, dtype=torch.float64, device="cuda")
    for e in range(experts):
        token, slot = (ids == e).nonzero(as_tuple=True)
        g, u = (h[token].double() @ w["w_gate_up"][e].double().T).split(spec.ffn, dim=1)
        ref.index_add_(0, token, wts[token, slot, None].double() * ((torch.nn.functional.silu(g) * u) @ w["w_down"][e].double().T))
    off = task.hidden().double() - x.double() - ref
    # Four roundings to bf16, 2^-8 / sqrt(3) in the mean square each, the gate's up to doubled, over 64 products: 1.2e-2 of a token's
    # contribution at most; a pair on a row that is not its own is 0.3 of it or more.
    assert (off.norm(dim=1) / ref.norm(dim=1)).max().item() <= 2.4e-2
    task.end()
    model.close()


def test_a_marker_stands_for_the_last_kernel_of_its_operator():
    """One operator in flight: when operator i is launched, all kernels of operator i - 1 are done.  experts_down's second kernel, the
    combine, takes most of its time here (16384 tokens of 8 choices over 16 narrow experts), and layer 1's qkv projection, which
    does not touch the residual, long enough to look at it: once the cursor says that the operator behind experts_down has been
    launched, the residual's rows, read on another stream, are those of a task that stopped there.  (Read one operator earlier,
    with experts_down in flight, they were not in any of 39 looks.)"""
    import ctypes
    import threading
    B, R = _mods()
    spec = I.ShapeSpec(2, 2048, 32, 32, 128, 64, 1e-5, 10000.0, n_experts=16, top_k=8)
    n, rows = 16384, 64
    stream, side = torch.cuda.Stream(), torch.cuda.Stream()
    model = R.PrefillModel(spec, I.make_weights(spec, 71, torch.bfloat16, "cuda"), B.FP_DTYPE_BF16, n // 16 + 8, 512, stream)
    x = I.make_hidden(n, spec.hidden, 71, torch.bfloat16, "cuda")
    lengths = [512] * (n // 512)
    task = model.begin(x, lengths)
    assert task.advance(9) == (B.FP_OK, 9)
    want = task.hidden()[-rows:].clone()
    task.end()
    hip = ctypes.CDLL("libamdhip64.so")
    hip.hipMemcpyAsync.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int, ctypes.c_void_p]
    looked = 0
    for attempt in range(20):
        got = torch.zeros_like(want)
        torch.cuda.synchronize()
        task = model.begin(x, lengths)
        B.fp_prefill_set_launch_ahead(task.handle, 1)
        at = B.fp_prefill_hidden(task.handle) + (n - rows) * spec.hidden * 4
        th = threading.Thread(target=task.run_to_completion)
        th.start()
        while th.is_alive() and task.cursor() < (1, 1):
            pass
        rc = hip.hipMemcpyAsync(got.data_ptr(), at, got.numel() * 4, 3, side.cuda_stream)
        side.synchronize()
        in_time = task.cursor() <= (1, 3)              # (the o_proj, which adds to the residual, is operator 4)
        th.join()
        assert rc == 0 and task.cursor() == (2, 0)
        task.end()
        if in_time:
            looked += 1
            assert torch.equal(got, want), f"attempt {attempt}"
    model.close()
    assert looked >= 5
