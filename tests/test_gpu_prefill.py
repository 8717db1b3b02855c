"""End-to-end parity of the HIP prefill path (through the C ABI) against the CPU oracle on the
same seeded inputs: final residual stream and every layer's K (rotated) and V, element by
element; plus the GPU-side invariants (chunked == one-shot, packed == alone, any block-table
permutation)."""
import numpy as np
import pytest
import torch

from oracle import prefill_oracle as O
from paper_2602_16603_amd import inputs as I
from tests.util import TOL, fro_rel_err, max_rel_err, oracle_layers, oracle_shape

pytestmark = pytest.mark.gpu

DT = {"fp32": (0, torch.float32), "bf16": (1, torch.bfloat16)}


def _runner():
    from paper_2602_16603_amd import runner
    return runner


def build(spec, seed, name, pool_blocks=None, max_position=None, total_tokens=0, random_gains=False):
    R = _runner()
    code, td = DT[name]
    weights = I.make_weights(spec, seed, td, "cpu")
    if random_gains:
        I.randomize_gains(weights, seed)
    pool_blocks = pool_blocks or (total_tokens // 16 + 64)
    model = R.PrefillModel(spec, weights, code, pool_blocks, max_position or max(total_tokens, 16))
    return model, weights


def check_against_oracle(spec, weights, hidden_cpu, lengths, task, name, cache=None):
    x_ref, cache_ref = O.prefill(oracle_shape(spec), oracle_layers(weights), hidden_cpu,
                                 I.cu_seqlens_of(lengths), cache)
    tol = TOL[name]
    got = task.hidden()
    e = max_rel_err(got, x_ref)
    print(f"  hidden: E={e:.3e} fro={fro_rel_err(got, x_ref):.3e}", flush=True)
    assert e <= tol, f"hidden states off by {e}"
    for layer in range(spec.n_layers):
        for s in range(len(lengths)):
            k, v = task.kv(layer, s)
            ek = max_rel_err(k, cache_ref.k[layer][s])
            ev = max_rel_err(v, cache_ref.v[layer][s])
            assert ek <= tol and ev <= tol, f"layer {layer} seq {s}: K {ek} V {ev}"
    return cache_ref


@pytest.mark.parametrize("name", ["fp32", "bf16"])
def test_cfg1_tiny_prompt(name):
    """cfg1: 2 layers, hidden 256, 4/2 heads of 64, FFN 704, one 256-token prompt."""
    cfg = I.CONFIGS["cfg1"]
    spec, n = cfg["shape"], cfg["lengths"][0]
    model, weights = build(spec, cfg["seed"], name, total_tokens=n)
    hidden = I.make_hidden(n, spec.hidden, cfg["seed"], DT[name][1], "cpu")
    task = model.begin(hidden.cuda(), [n])
    task.run_to_completion()
    assert task.cursor() == (spec.n_layers, 0)
    check_against_oracle(spec, weights, hidden, [n], task, name)
    task.end()
    model.close()


@pytest.mark.parametrize("name", ["fp32", "bf16"])
def test_ragged_packed_batch_with_permuted_blocks_and_random_gains(name):
    """Packed varlen batch (lengths straddle the 16-token block, the 64-key tile and the
    256-row query tile), block table = seeded permutation of the pool, norm gains != 1."""
    spec = I.TINY
    lengths = [1, 300, 17, 64, 0, 255, 513, 16]
    total = sum(lengths)
    model, weights = build(spec, 21, name, pool_blocks=256, max_position=1024, random_gains=True)
    hidden = I.make_hidden(total, spec.hidden, 21, DT[name][1], "cpu")
    table, _ = I.permuted_block_tables(lengths, None, 16, 256, seed=5)
    task = model.begin(hidden.cuda(), lengths, cached=[0] * len(lengths), block_tables=table)
    task.run_to_completion()
    check_against_oracle(spec, weights, hidden, lengths, task, name)
    # Same batch with library-allocated (identity-ordered) blocks must give the same bits.
    task2 = model.begin(hidden.cuda(), lengths)
    task2.run_to_completion()
    assert torch.equal(task.hidden(), task2.hidden())
    task.end()
    task2.end()
    model.close()


@pytest.mark.parametrize("name", ["fp32", "bf16"])
@pytest.mark.parametrize("chunk", [16, 100, 257])
def test_chunked_prefill_reads_cached_prefix(name, chunk):
    """A prompt run chunk by chunk, every chunk attending to the KV its predecessors left in the
    paged cache (Section 3.1), equals the oracle's one-shot prefill."""
    spec = I.TINY
    n = 600
    model, weights = build(spec, 22, name, pool_blocks=64, max_position=n, random_gains=True)
    hidden = I.make_hidden(n, spec.hidden, 22, DT[name][1], "cpu")
    x_ref, cache_ref = O.prefill(oracle_shape(spec), oracle_layers(weights), hidden, [0, n])
    from paper_2602_16603_amd import binding as B
    blocks = B.fp_kv_alloc(model.handle, (n + 15) // 16)
    table = np.asarray(blocks, dtype=np.int32).reshape(1, -1)
    outs, last = [], None
    for lo in range(0, n, chunk):
        hi = min(n, lo + chunk)
        task = model.begin(hidden[lo:hi].contiguous().cuda(), [hi - lo], cached=[lo],
                           block_tables=table, boundary_mask=B.FP_BOUNDARY_NONE)
        task.run_to_completion()
        outs.append(task.hidden())
        if last is not None:
            last.end()
        last = task
    got = torch.cat(outs)
    assert max_rel_err(got, x_ref) <= TOL[name]
    for layer in range(spec.n_layers):
        k, v = last.kv(layer, 0)
        assert max_rel_err(k, cache_ref.k[layer][0]) <= TOL[name]
        assert max_rel_err(v, cache_ref.v[layer][0]) <= TOL[name]
    last.end()
    B.fp_kv_free(model.handle, blocks)
    model.close()


def test_8b_head_shapes_small_twin_bf16():
    """Llama-3-8B head/hidden/FFN shapes, 2 layers, ragged lengths (shrunken twin of cfg2/cfg3):
    exercises head_dim 128, GQA 32/8, K = 14336 and the 256x256 GEMM tiles."""
    spec = I.LLAMA3_8B.with_layers(2)
    lengths = [700, 130, 333]
    total = sum(lengths)
    model, weights = build(spec, 23, "bf16", total_tokens=total, max_position=1024)
    hidden = I.make_hidden(total, spec.hidden, 23, torch.bfloat16, "cpu")
    task = model.begin(hidden.cuda(), lengths)
    task.run_to_completion()
    check_against_oracle(spec, weights, hidden, lengths, task, "bf16")
    task.end()
    model.close()


@pytest.mark.parametrize("lengths", [[128], [512, 40], [1024]])
def test_short_requests_8b_shape_use_split_k(lengths):
    """The 128..1024-token requests of the preemption workload: too few output tiles to fill the
    chip, so the projections run on the 128-column tile (up to 512 tokens), are split over K and
    reduced in a fixed order by kernels that also carry the small operator that follows."""
    spec = I.LLAMA3_8B.with_layers(1)
    total = sum(lengths)
    model, weights = build(spec, 26, "bf16", total_tokens=total, max_position=1024)
    hidden = I.make_hidden(total, spec.hidden, 26, torch.bfloat16, "cpu")
    task = model.begin(hidden.cuda(), lengths)
    task.run_to_completion()
    check_against_oracle(spec, weights, hidden, lengths, task, "bf16")
    again = model.begin(hidden.cuda(), lengths)          # fixed reduction order: same bits every run
    again.run_to_completion()
    assert torch.equal(task.hidden(), again.hidden())
    task.end()
    again.end()
    model.close()


def test_packed_equals_alone_on_gpu_bf16():
    spec = I.TINY
    lengths = [90, 270, 33]
    model, _ = build(spec, 24, "bf16", pool_blocks=128, max_position=512)
    hidden = I.make_hidden(sum(lengths), spec.hidden, 24, torch.bfloat16, "cuda")
    packed = model.begin(hidden, lengths)
    packed.run_to_completion()
    out = packed.hidden()
    cu = I.cu_seqlens_of(lengths)
    for s, n in enumerate(lengths):
        alone = model.begin(hidden[cu[s]:cu[s + 1]].contiguous(), [n])
        alone.run_to_completion()
        # different M changes no per-row arithmetic order in these kernels: bit-equal
        assert torch.equal(alone.hidden(), out[cu[s]:cu[s + 1]])
        alone.end()
    packed.end()
    model.close()


def test_empty_batch_and_invalid_arguments():
    from paper_2602_16603_amd import binding as B
    spec = I.TINY
    model, _ = build(spec, 25, "bf16", pool_blocks=8, max_position=64)
    hidden = I.make_hidden(16, spec.hidden, 25, torch.bfloat16, "cuda")
    empty = model.begin(hidden[:0].contiguous(), [0])
    st, _ = empty.advance()
    assert st == B.FP_DONE
    empty.end()
    with pytest.raises(B.FlowPrefillError):          # beyond max_position
        model.begin(I.make_hidden(80, spec.hidden, 1, torch.bfloat16, "cuda"), [80])
    with pytest.raises(B.FlowPrefillError):          # pool exhausted (8 blocks = 128 tokens)
        a = model.begin(I.make_hidden(64, spec.hidden, 1, torch.bfloat16, "cuda"), [64])
        b = model.begin(I.make_hidden(64, spec.hidden, 1, torch.bfloat16, "cuda"), [64])
        try:
            model.begin(I.make_hidden(16, spec.hidden, 1, torch.bfloat16, "cuda"), [16])
        finally:
            a.end()
            b.end()
    with pytest.raises(B.FlowPrefillError):          # block id outside the pool
        model.begin(hidden, [16], cached=[0], block_tables=np.array([[99]], dtype=np.int32))
    model.close()


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("new,cached", [([1], [1023]), ([257, 40], [1008, 3000]), ([700], [2400]), ([2100], [0]),
                                        ([1], [0]), ([1], [64]), ([65], [0]), ([129], [50]), ([300, 40], [7, 100]), ([640], [63])])
def test_attention_cut_over_its_keys(head_dim, new, cached):
    """Few query tiles over many keys: the launch is cut over the keys and the parts are merged (the
    last part holds the diagonal; a tile of one row, of a full and a nearly empty tile, of two
    sequences of unlike length), and left whole over few keys.  Against the oracle's one-shot prefill."""
    spec = I.ShapeSpec(1, 256, 4, 2, head_dim, 704, 1e-5, 10000.0)
    full = [n + c for n, c in zip(new, cached)]
    model, weights = build(spec, 27, "bf16", pool_blocks=512, max_position=max(full), random_gains=True)
    rows = [I.make_hidden(n, spec.hidden, 27 + i, torch.bfloat16, "cpu") for i, n in enumerate(full)]
    table, _ = I.permuted_block_tables(full, None, 16, 512, seed=6)
    if any(cached):
        first = model.begin(torch.cat([r[:c] for r, c in zip(rows, cached)]).cuda(), cached, [0] * len(full), table)
        first.run_to_completion()
        first.end()
    print(f"attention parts head_dim={head_dim} new={new} cached={cached}", flush=True)
    last = torch.cat([r[c:] for r, c in zip(rows, cached)]).cuda()
    task = model.begin(last, new, cached, table)
    task.run_to_completion()
    got = task.hidden()
    x_ref, _ = O.prefill(oracle_shape(spec), oracle_layers(weights), torch.cat(rows), I.cu_seqlens_of(full))
    x_ref = torch.cat([x[c:] for x, c in zip(x_ref.split(full), cached)])
    assert max_rel_err(got, x_ref) <= TOL["bf16"]
    # With one-layer models attention reaches the output through o_proj only: without a wrong part the
    # error stays at the storage rounding (2^-9 per intermediate, six of them: 1e-2 at most).
    assert fro_rel_err(got, x_ref) <= 1e-2
    again = model.begin(last, new, cached, table)
    again.run_to_completion()
    assert torch.equal(again.hidden(), got)               # parts are merged in a fixed order
    task.end()
    again.end()
    model.close()


@pytest.mark.parametrize("hidden,ffn,lengths", [(256, 704, [200]), (256, 704, [1]), (264, 200, [33, 64]), (320, 1032, [700])])
def test_small_models_fuse_gate_up(hidden, ffn, lengths):
    """A stack whose gate_up projection is far from filling the chip runs it on small tiles with
    SiLU(gate)*up in the epilogue (rows and columns that leave partly filled tiles, K with a tail): against the
    oracle, and operator 7 launches nothing."""
    from paper_2602_16603_amd import binding as B
    spec = I.ShapeSpec(2, hidden, 4, 2, 64, ffn, 1e-5, 10000.0)
    total = sum(lengths)
    model, weights = build(spec, 28, "bf16", total_tokens=total, max_position=1024, random_gains=True)
    rows = I.make_hidden(total, hidden, 28, torch.bfloat16, "cpu")
    task = model.begin(rows.cuda(), lengths)
    B.fp_prefill_set_timing(task.handle, True)
    task.run_to_completion()
    assert B.fp_prefill_op_times(task.handle, 18)[7] == 0.0
    check_against_oracle(spec, weights, rows, lengths, task, "bf16")
    task.end()
    model.close()


@pytest.mark.parametrize("new,cached", [([1], [0]), ([37], [5]), ([100, 28], [3, 16]), ([300, 7, 64], [9, 30, 0])])
def test_rope_adds_up_the_projection_of_a_short_request(new, cached):
    """A short request's qkv projection is cut over K and RoPE + KV write adds the partial sums: few rows, one
    and two row tiles, first and last cache blocks that are partly old and partly filled.  The slots of
    tokens that are not new keep their bits."""
    spec = I.ShapeSpec(1, 1024, 32, 8, 128, 256, 1e-5, 10000.0)
    from paper_2602_16603_amd import binding as B
    assert B.fp_op_gemm_workspace_bytes(1, sum(new), spec.qkv_width, spec.hidden) > 0
    full = [n + c for n, c in zip(new, cached)]
    model, weights = build(spec, 29, "bf16", pool_blocks=64, max_position=max(full), random_gains=True)
    rows = [I.make_hidden(n, spec.hidden, 29 + i, torch.bfloat16, "cpu") for i, n in enumerate(full)]
    table, _ = I.permuted_block_tables(full, None, 16, 64, seed=7)
    before = None
    if any(cached):
        first = model.begin(torch.cat([r[:c] for r, c in zip(rows, cached)]).cuda(), cached, [0] * len(full), table)
        first.run_to_completion()
        before = [first.kv(0, s) for s in range(len(full))]
        first.end()
    task = model.begin(torch.cat([r[c:] for r, c in zip(rows, cached)]).cuda(), new, cached, table)
    task.run_to_completion()
    x_ref, cache_ref = O.prefill(oracle_shape(spec), oracle_layers(weights), torch.cat(rows), I.cu_seqlens_of(full))
    x_ref = torch.cat([x[c:] for x, c in zip(x_ref.split(full), cached)])
    assert max_rel_err(task.hidden(), x_ref) <= TOL["bf16"]
    for s in range(len(full)):
        k, v = task.kv(0, s)
        assert max_rel_err(k, cache_ref.k[0][s]) <= TOL["bf16"] and max_rel_err(v, cache_ref.v[0][s]) <= TOL["bf16"]
        if before is not None and cached[s]:
            assert torch.equal(k[:cached[s]], before[s][0]) and torch.equal(v[:cached[s]], before[s][1])
    task.end()
    model.close()


@pytest.mark.parametrize("lengths", [[5], [16, 3], [37], [300, 21]])
def test_fp32_slots_of_an_earlier_request_do_not_matter(lengths):
    """The slots behind a sequence's last token still hold what an earlier request left in the block, here
    NaN in every slot of the pool: a later request's results have the bits they have in a pool that was never used."""
    model, _ = build(I.TINY, 61, "fp32", pool_blocks=32, max_position=512)
    hidden = I.make_hidden(sum(lengths), I.TINY.hidden, 61, torch.float32, "cuda")
    print(f"fp32 reused blocks {lengths}", flush=True)

    def outputs():
        task = model.begin(hidden, lengths)
        task.run_to_completion()
        out = [task.hidden()] + [t for layer in range(2) for s in range(len(lengths)) for t in task.kv(layer, s)]
        task.end()
        return out

    want = outputs()
    poison = model.begin(torch.full((512, I.TINY.hidden), float("nan"), device="cuda"), [512])   # every block of the pool
    poison.run_to_completion()
    assert not torch.isfinite(poison.kv(1, 0)[1]).any()
    poison.end()
    got = outputs()
    assert all(torch.isfinite(t).all() for t in want)
    assert all(torch.equal(a, b) for a, b in zip(got, want))


@pytest.mark.parametrize("head_dim", [16, 128])
@pytest.mark.parametrize("new,cached,at", [(40, 0, 33), (40, 0, 20), (21, 0, 20), (30, 5, 17), (90, 27, 70)])
def test_fp32_tokens_see_no_later_token_that_is_not_finite(head_dim, new, cached, at):
    """Causality holds for NaN too: tokens in front of a NaN one, its own cache block's among them, have the bits
    they have when that token is an ordinary one; from that token on every row is NaN."""
    spec = I.ShapeSpec(1, 64, 6, 3, head_dim, 64, 1e-5, 10000.0)
    model, _ = build(spec, 62, "fp32", pool_blocks=32, max_position=256)
    hidden = I.make_hidden(cached + new, spec.hidden, 62, torch.float32, "cuda")
    table, _ = I.permuted_block_tables([new], [cached], 16, 32, seed=62)
    if cached:
        first = model.begin(hidden[:cached].contiguous(), [cached], [0], table)
        first.run_to_completion()
        first.end()
    print(f"fp32 causality head_dim={head_dim} new={new} cached={cached} at={at}", flush=True)
    out = []
    for value in (None, float("nan")):
        rows = hidden[cached:].clone()
        if value is not None:
            rows[at] = value
        task = model.begin(rows, [new], [cached], table)
        task.run_to_completion()
        out.append(task.hidden())
        task.end()
    assert torch.isfinite(out[0]).all()
    assert torch.equal(out[1][:at], out[0][:at])
    assert torch.isnan(out[1][at:]).all()


@pytest.mark.parametrize("head_dim", [64, 128])
def test_attention_parts_whose_first_keys_score_minus_infinity(head_dim):
    """Scores below the fp32 range are -inf and weigh nothing.  Keys 128 to 1327 are such for all 32 queries, so the
    second part of the cut launch opens with tiles that hold nothing but -inf (and the launch as a whole does not)."""
    hidden, first, far, last = 64, 128, 1200, 32
    spec = I.ShapeSpec(1, hidden, 4, 2, head_dim, 64, 1e-5, 1e30)
    weights = I.make_weights(spec, 63, torch.bfloat16, "cpu")
    w = weights[0]["w_qkv"]
    q_rows, k_rows = 4 * head_dim, 6 * head_dim
    w[:k_rows] = 0
    # Two kinds of token, told apart by their one non-zero channel (8 after the norm): kind 1 asks, and scores
    # -1e40 on kind 0's keys.  Only channels that the rotation leaves alone over 1360 positions are used.
    turning = (torch.arange(k_rows) % (head_dim // 2)) < head_dim // 4
    q, k = w[:q_rows], w[q_rows:k_rows]
    q[:, 1] = 1e19
    k[:, 0] = -1e19
    k[:, 1] = 1e-21
    w[:k_rows][turning] = 0
    R = _runner()
    model = R.PrefillModel(spec, weights, 1, 128, 2048)
    kind = torch.tensor([1] * first + [0] * far + [1] * last)
    rows = torch.nn.functional.one_hot(kind, hidden).to(torch.bfloat16)
    cached = first + far
    table, _ = I.permuted_block_tables([last], [cached], 16, 128, seed=63)
    print(f"attention parts over -inf, head_dim={head_dim}", flush=True)
    task = model.begin(rows[:cached].cuda(), [cached], [0], table)
    task.run_to_completion()
    task.end()
    task = model.begin(rows[cached:].cuda(), [last], [cached], table)
    task.run_to_completion()
    got = task.hidden()
    x_ref, _ = O.prefill(oracle_shape(spec), oracle_layers(weights), rows, [0, cached + last])
    assert torch.isfinite(got).all()
    assert max_rel_err(got, x_ref[cached:]) <= TOL["bf16"]
    task.end()
    model.close()


@pytest.mark.parametrize("name", ["fp32", "bf16"])
def test_model_on_a_stream_of_its_own(name):
    """begin() and kv() of a model whose kernels run on another stream than torch's: inputs that torch is still
    producing are waited for, and memory that torch is still using is not written early."""
    R = _runner()
    code, td = DT[name]
    spec, lengths = I.TINY, [37, 200]
    weights = I.make_weights(spec, 64, td, "cpu")
    hidden = I.make_hidden(sum(lengths), spec.hidden, 64, td, "cuda")

    def outputs(model):
        busy = torch.randn(4096, 4096, device="cuda")
        for _ in range(20):
            busy = busy @ busy.T * 1e-4                # torch's stream is some way behind the host
        rows = hidden + (busy[:1, :1] * 0).nan_to_num().to(td)
        task = model.begin(rows, lengths)
        task.run_to_completion()
        out = [task.hidden()]
        for layer in range(spec.n_layers):
            for s in range(len(lengths)):
                garbage = torch.full((lengths[s], spec.n_kv_heads, spec.head_dim), 7.0, dtype=td, device="cuda")
                del garbage                            # its memory goes to the next kv(), its fill may still be queued
                out += task.kv(layer, s)
        task.end()
        return out

    same = R.PrefillModel(spec, weights, code, 64, 256)
    own = R.PrefillModel(spec, weights, code, 64, 256, stream=torch.cuda.Stream())
    want = outputs(same)
    for _ in range(3):
        assert all(torch.equal(a, b) for a, b in zip(outputs(own), want))
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):                      # torch on a stream of its own, the model on the default one
        side.wait_stream(torch.cuda.default_stream())
        assert all(torch.equal(a, b) for a, b in zip(outputs(same), want))
    torch.cuda.synchronize()
    same.close()
    own.close()


GATE_UP_OF_ONE_ROW_TILE = ([(6152, hidden, n) for hidden in (64, 192, 1088) for n in (1, 32, 33, 64, 65, 128, 129, 161, 193, 256)] +
                           [(20488, hidden, n) for hidden in (64, 576) for n in (65, 129, 161, 193, 256)])


@pytest.mark.parametrize("ffn,hidden,n", GATE_UP_OF_ONE_ROW_TILE)
def test_gate_up_of_one_row_tile(ffn, hidden, n):
    """The fused gate_up projection of up to 256 tokens (row tiles of the few-rows kernel, then the 128-column tile and,
    where its columns fill the chip, the 256-column one; one k-tile, fewer than the stages hold, a number
    that is no multiple of them; a last column tile of eight outputs)."""
    spec = I.ShapeSpec(1, hidden, 2, 1, 64, ffn, 1e-5, 10000.0)
    model, weights = build(spec, 31, "bf16", total_tokens=n, random_gains=True)
    x = I.make_hidden(n, hidden, 31, torch.bfloat16, "cpu")
    print(f"gate_up of one row tile n={n} hidden={hidden} ffn={ffn}", flush=True)
    task = model.begin(x.cuda(), [n])
    task.run_to_completion()
    x_ref, _ = O.prefill(oracle_shape(spec), oracle_layers(weights), x, [0, n])
    # Six intermediates rounded to bf16 (2^-9 each): 1e-2 at most.  (Of the residual: the projection alone is checked below.)
    assert fro_rel_err(task.hidden(), x_ref) <= 1e-2
    task.end()
    model.close()


@pytest.mark.parametrize("ffn,hidden,n", GATE_UP_OF_ONE_ROW_TILE)
def test_gate_up_of_a_short_request_has_the_operators_bits(ffn, hidden, n):
    """The prefill path launches the kernels of the single-operator entry points: with nothing coming from attention, the
    residual is that of rmsnorm, gemm_swiglu and gemm called one by one, bit for bit; gemm_swiglu has the bits of gemm and
    silu_mul, and every value of it is as near its definition as its three bf16 roundings are."""
    from paper_2602_16603_amd import binding as B
    spec = I.ShapeSpec(1, hidden, 2, 1, 64, ffn, 1e-5, 10000.0)
    weights = I.make_weights(spec, 32, torch.bfloat16, "cuda")
    I.randomize_gains(weights, 32)
    w = weights[0]
    w["w_o"].zero_()
    rows = I.make_hidden(n, hidden, 32, torch.bfloat16, "cuda")
    model = _runner().PrefillModel(spec, weights, 1, 64, 256)
    print(f"gate_up against its operators n={n} hidden={hidden} ffn={ffn}", flush=True)
    task = model.begin(rows, [n])
    task.run_to_completion()
    got = task.hidden()
    x = rows.float()
    h, gu, two, act = (torch.empty(n, width, dtype=torch.bfloat16, device="cuda") for width in (hidden, 2 * ffn, ffn, ffn))
    ws_bytes = B.fp_op_gemm_workspace_bytes(1, n, hidden, ffn)
    ws = torch.empty(max(ws_bytes, 256), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    B.fp_op_rmsnorm(1, x.data_ptr(), w["mlp_norm"].data_ptr(), h.data_ptr(), n, hidden, spec.rms_eps)
    B.fp_op_gemm(1, h.data_ptr(), w["w_gate_up"].data_ptr(), gu.data_ptr(), n, 2 * ffn, hidden, False)
    B.fp_op_silu_mul(1, gu.data_ptr(), two.data_ptr(), n, ffn)
    B.fp_op_gemm_swiglu(h.data_ptr(), w["w_gate_up"].data_ptr(), act.data_ptr(), n, ffn, hidden)
    B.fp_op_gemm_ws(1, act.data_ptr(), w["w_down"].data_ptr(), x.data_ptr(), n, hidden, ffn, True, ws.data_ptr(), ws_bytes)
    torch.cuda.synchronize()
    assert torch.equal(act, two)
    gate, up = (h.double() @ w["w_gate_up"].double().T).split(ffn, dim=1)
    ref = torch.nn.functional.silu(gate) * up
    # gate, up and their product each rounded to bf16, whose eight significant bits are off by up to 2^-8 of the value
    # (silu's slope is at most 1.1; 2 % for the terms of second order); sums of up to 1088 products of about 0.02 in fp32: 1e-5 at most.
    bound = 2.0 ** -8 * 1.02 * (1.1 * (gate * up).abs() + 2 * ref.abs()) + 1e-5 * (1 + gate.abs() + up.abs())
    assert torch.all((act.double() - ref).abs() <= bound), ((act.double() - ref).abs() / bound).max().item()
    assert torch.equal(got, x)
    task.end()
    model.close()
