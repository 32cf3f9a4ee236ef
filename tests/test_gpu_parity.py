"""GPU parity: the HIP path through the C ABI against the CPU oracle on the same seeded inputs."""
import numpy as np
import pytest

import paper_2608_11226_amd as R
import workload as W
from gpu_helpers import TILE_ROWS, check_rows, guarded_token_compare, log, one_token_logits, shape_of, to_dev
from oracle import OracleModel, bf16_round, grpo_advantages, rollout, sample_row

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a ROCm GPU"
    yield
    torch.cuda.synchronize()


# ---------------------------------------------------------------------------
# group-relative advantages
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("G", [1, 2, 3, 8, 16, 64, 100, 257])
@pytest.mark.parametrize("ddof,eps", [(1, 0.0), (0, 0.0), (1, 1e-4)])
def test_grpo_advantages_match_oracle(G, ddof, eps):
    log(f"grpo G={G} ddof={ddof} eps={eps}")
    n_groups = 37
    r = W.rewards(n_groups * G, seed=3)
    r[: 2 * G] = 0.9  # two all-equal groups
    r[5 * G: 6 * G] = np.float32(0.25)
    want, zv = grpo_advantages(r, G, eps=eps, ddof=ddof)
    dr = to_dev(r, torch)
    adv = torch.empty(n_groups * G, dtype=torch.float32, device="cuda:0")
    cnt = torch.full((1,), -7, dtype=torch.int32, device="cuda:0")
    R.grpo_advantages(dr, n_groups, G, eps, ddof, adv, cnt, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    got = adv.cpu().numpy()
    assert np.max(np.abs(got - want)) <= 1e-5
    assert int(cnt.item()) == zv
    assert np.all(got[: 2 * G] == 0)


def test_grpo_advantages_at_full_size():
    # the 7B workload's 8 groups of 8, and a large batch of groups
    for n_groups, G in ((8, 8), (4096, 16)):
        r = W.rewards(n_groups * G, seed=3)
        want, zv = grpo_advantages(r, G)
        adv = torch.empty(n_groups * G, dtype=torch.float32, device="cuda:0")
        R.grpo_advantages(to_dev(r, torch), n_groups, G, 0.0, 1, adv, None, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert np.max(np.abs(adv.cpu().numpy() - want)) <= 1e-5


# ---------------------------------------------------------------------------
# weights synthesised on the device equal the seeded generator's, bit for bit
# ---------------------------------------------------------------------------
SMALL_BF16 = (2, 256, 8, 2, 64, 512, 2048, 1e6)


@pytest.mark.parametrize("dtype,shape", [(R.DTYPE_FP32, "tiny"), (R.DTYPE_BF16, SMALL_BF16)])
def test_weights_bit_exact(dtype, shape):
    cfg = R.model_config(shape, dtype, 16, 8, 4)
    log(f"weights dtype={dtype} shape={shape}")
    eng = R.Engine(cfg)
    sh = shape_of(cfg)
    ids = [(0, "embed"), (W.tensor_id_lm_head(sh), "lm_head")]
    for l in range(sh.n_layers):
        for slot in (W.WQ, W.WK, W.WV, W.WO, W.WGATE, W.WUP, W.WDOWN):
            ids.append((W.tensor_id_layer(l, slot), W.LAYER_SLOTS[slot]))
    for tid, name in ids:
        rows, cols = W.logical_shape(sh, name)
        out = torch.empty(rows * cols, dtype=torch.float32, device="cuda:0")
        R.rollout_export_weight(eng.ctx, tid, out)
        eng.synchronize()
        want = W.weight_matrix(0, tid, rows, cols).reshape(-1)
        if dtype == R.DTYPE_BF16:
            want = bf16_round(want).astype(np.float32)
        got = out.cpu().numpy()
        assert np.array_equal(got.view(np.uint32), want.view(np.uint32)), f"tensor {tid} ({name})"
    eng.close()


# ---------------------------------------------------------------------------
# sampler on identical logits
# ---------------------------------------------------------------------------
# vocabularies: one chunk; 152064 (38 chunks of 4096 ids, the last of 512); 300000 (above 64 x 4096: chunks
# of two 4096-id batches).  Widths that are not a multiple of 16 go through rollout_sample_noalloc.
@pytest.mark.parametrize("V", [1024, 2048, 152064, 300000])
@pytest.mark.parametrize("temperature,top_p", [(0.0, 1.0), (1.0, 1.0), (0.9, 0.95), (0.7, 0.5), (1.0, 1e-6)])
def test_sampler_matches_oracle(V, temperature, top_p):
    log(f"sampler V={V} T={temperature} top_p={top_p}")
    S = 48 if V < 10**5 else 128
    rng = np.random.default_rng(V + int(temperature * 10) + int(top_p * 100))
    z = (rng.standard_normal((S, V)) * 2.0).astype(np.float32)
    z[:8] = np.round(z[:8], 1)  # ties in value
    z[8, :] = 0.5  # a flat row
    u = W.uniforms(S, 1, seed=9)[:, 0]
    cfg = R.model_config("tiny", R.DTYPE_FP32, 16, 8, 4)
    cfg.vocab = V  # the sampler takes the row width from the context
    eng = R.Engine(cfg)
    dz = to_dev(z, torch)
    du = to_dev(u, torch)
    out = torch.full((S,), -1, dtype=torch.int32, device="cuda:0")
    R.rollout_sample(eng.ctx, dz, S, temperature, top_p, du, out)
    eng.synchronize()
    got = out.cpu().numpy()
    # Same logits on both sides: the decision values differ only by exp() rounding
    # (about 1e-7 relative) and the 2^-40 fixed-point mass, so a draw is compared
    # unless it lies within 1e-6 of the kept mass from flipping.  At V = 152064 a
    # token's CDF bucket averages 1/V = 6.6e-6 of the mass, so many draws sit
    # that close to an edge; the row count is raised there to keep coverage.
    checked = 0
    for s in range(S):
        tok, margin = sample_row(z[s], temperature, top_p, float(u[s]))
        if margin < 1e-6:
            continue
        assert got[s] == tok, f"row {s}: gpu {got[s]} oracle {tok} margin {margin}"
        checked += 1
    log(f"  compared {checked} of {S} draws")
    assert checked >= (S - 4 if V < 10**5 else S // 2)
    eng.close()


@pytest.mark.parametrize("V", [1024, 2064, 152064, 262144])
@pytest.mark.parametrize("temperature,top_p", [(1.0, 1.0), (0.9, 0.95), (0.7, 0.5), (1.0, 1e-6)])
def test_sampler_row_kernel_equals_chunked_kernels(V, temperature, top_p, monkeypatch):
    """The one-workgroup-per-row sampler and the chunked kernels draw the same token from the same logits
    (same integer masses, digits, tie rule and draw), including value ties and a flat row."""
    log(f"sampler paths V={V} T={temperature} top_p={top_p}")
    S = 64
    rng = np.random.default_rng(V + 7)
    z = (rng.standard_normal((S, V)) * 2.0).astype(np.float32)
    z[:8] = np.round(z[:8], 1)
    z[8, :] = 0.5
    z[9, : V // 2] = 3.0  # a tie at the maximum over half the row
    u = W.uniforms(S, 1, seed=11)[:, 0]
    u[10] = 0.0
    u[11] = np.float32(1.0) - np.float32(2.0**-24)
    cfg = R.model_config("tiny", R.DTYPE_FP32, 16, 8, 4)
    cfg.vocab = V
    eng = R.Engine(cfg)
    dz = to_dev(z, torch)
    du = to_dev(u, torch)
    got = {}
    for path in ("row", "chunked"):
        monkeypatch.setenv("ROLLOUT_SAMPLE_PATH", path)
        out = torch.full((S,), -1, dtype=torch.int32, device="cuda:0")
        R.rollout_sample(eng.ctx, dz, S, temperature, top_p, du, out)
        eng.synchronize()
        got[path] = out.cpu().numpy()
    monkeypatch.delenv("ROLLOUT_SAMPLE_PATH", raising=False)
    assert (got["row"] >= 0).all() and (got["row"] < V).all()
    assert np.array_equal(got["row"], got["chunked"]), np.nonzero(got["row"] != got["chunked"])
    eng.close()


@pytest.mark.parametrize("V", [1024, 2064, 20016])
@pytest.mark.parametrize("top_p", [1.0, 0.95])
def test_sampler_chunked_loads_by_alignment(V, top_p, monkeypatch):
    """The chunked kernels draw the same tokens by 16-byte loads (aligned logits) and by 4-byte loads (logits
    one float further on), with masked ids (-inf) in the rows."""
    log(f"sampler chunked loads V={V} top_p={top_p}")
    S = 16
    rng = np.random.default_rng(V)
    z = (rng.standard_normal((S, V)) * 2.0).astype(np.float32)
    z[:4, V // 2:] = -np.inf
    buf = torch.empty((S * V + 1,), dtype=torch.float32, device="cuda:0")
    du = to_dev(W.uniforms(S, 1, seed=13)[:, 0], torch)
    cfg = R.model_config("tiny", R.DTYPE_FP32, 16, 8, 4)
    cfg.vocab = V
    eng = R.Engine(cfg)
    monkeypatch.setenv("ROLLOUT_SAMPLE_PATH", "chunked")
    got = []
    for off in (0, 1):
        dz = buf[off:off + S * V].view(S, V)
        dz.copy_(to_dev(z, torch))
        torch.cuda.synchronize()
        out = torch.full((S,), -1, dtype=torch.int32, device="cuda:0")
        R.rollout_sample(eng.ctx, dz, S, 0.9, top_p, du, out)
        eng.synchronize()
        got.append(out.cpu().numpy())
    assert (got[0] >= 0).all() and (got[0] < V).all() and (got[0][:4] < V // 2).all()
    assert np.array_equal(got[0], got[1])
    eng.close()


# ---------------------------------------------------------------------------
# tiny fp32 model: the whole rollout
# ---------------------------------------------------------------------------
def _tiny_engine(P=16, N=16, S=8, blk=16):
    cfg = R.model_config("tiny", R.DTYPE_FP32, P, N, S, kv_block_size=blk)
    return R.Engine(cfg), cfg


@pytest.mark.parametrize("P,blk,G,n_prompts", [(16, 16, 4, 2), (13, 8, 4, 2), (16, 16, 1, 3), (5, 16, 3, 2)])
def test_tiny_fp32_teacher_forced_logits(P, blk, G, n_prompts):
    log(f"tiny fp32 teacher forced P={P} blk={blk} G={G} prompts={n_prompts}")
    N = 16
    S = n_prompts * G
    eng, cfg = _tiny_engine(P, N, S, blk)
    model = OracleModel(shape_of(cfg), mode="fp32")
    prompts = W.prompts(n_prompts, P, cfg.vocab)
    u = W.uniforms(S, N)
    ref = rollout(model, prompts, G, N, 1.0, 1.0, u)
    logits = torch.empty((S, cfg.vocab), dtype=torch.float32, device="cuda:0")
    R.rollout_prefill(eng.ctx, to_dev(prompts, torch), n_prompts, P, G, logits)
    eng.synchronize()
    err = [float(np.max(np.abs(logits.cpu().numpy() - ref["logits"][0])))]
    for t in range(1, N):
        R.rollout_decode_step(eng.ctx, to_dev(ref["tokens"][:, t - 1], torch), logits)
        eng.synchronize()
        err.append(float(np.max(np.abs(logits.cpu().numpy() - ref["logits"][t]))))
    log(f"  max abs logit error per step: {max(err):.3g}")
    assert max(err) <= 1e-4
    eng.close()


def test_tiny_fp32_generate_matches_oracle_tokens():
    log("tiny fp32 generate (the tiny workload: 2 prompts x 16, G=4, 16 new tokens, T=1, top-p 1)")
    eng, cfg = _tiny_engine()
    model = OracleModel(shape_of(cfg), mode="fp32")
    prompts = W.prompts(2, 16, cfg.vocab)
    u = W.uniforms(8, 16)
    ref = rollout(model, prompts, 4, 16, 1.0, 1.0, u, keep_logits=False)
    out = torch.full((8, 16), -1, dtype=torch.int32, device="cuda:0")
    R.rollout_generate(eng.ctx, to_dev(prompts, torch), 2, 16, 4, 8, 16, 1.0, 1.0, to_dev(u, torch), out)
    eng.synchronize()
    compared, skipped = guarded_token_compare(out.cpu().numpy(), ref["tokens"], ref["margins"])
    log(f"  compared {compared} tokens, skipped {skipped} after near-ties")
    assert compared >= 100


@pytest.mark.parametrize("temperature,top_p,seqs", [(0.0, 1.0, 8), (0.8, 0.9, 4), (1.0, 1.0, 2)])
def test_tiny_fp32_generate_waves_and_knobs(temperature, top_p, seqs):
    log(f"tiny fp32 generate T={temperature} top_p={top_p} seqs_in_flight={seqs}")
    eng, cfg = _tiny_engine(S=8)
    model = OracleModel(shape_of(cfg), mode="fp32")
    prompts = W.prompts(4, 16, cfg.vocab, seed=21)
    u = W.uniforms(8, 12, seed=22)
    ref = rollout(model, prompts, 2, 12, temperature, top_p, u, keep_logits=False)
    out = torch.full((8, 12), -1, dtype=torch.int32, device="cuda:0")
    R.rollout_generate(eng.ctx, to_dev(prompts, torch), 4, 16, 2, seqs, 12, temperature, top_p, to_dev(u, torch), out)
    eng.synchronize()
    compared, _ = guarded_token_compare(out.cpu().numpy(), ref["tokens"], ref["margins"])
    assert compared >= 60


def test_generate_is_deterministic():
    eng, cfg = _tiny_engine()
    prompts = to_dev(W.prompts(2, 16, cfg.vocab), torch)
    u = to_dev(W.uniforms(8, 16), torch)
    outs = []
    for _ in range(2):
        out = torch.full((8, 16), -1, dtype=torch.int32, device="cuda:0")
        R.rollout_generate(eng.ctx, prompts, 2, 16, 4, 8, 16, 0.9, 0.95, u, out)
        eng.synchronize()
        outs.append(out.cpu().numpy())
    assert np.array_equal(outs[0], outs[1])


# ---------------------------------------------------------------------------
# bf16 path on a small GQA model
# ---------------------------------------------------------------------------
# Decode-attention path switches (read by the library per call): the shared-prefix pass (0 never, 1 by
# size, 2 always) and the waves per attention workgroup (4 or 8; unset = by grid size).
ATTN_KNOBS = [("1", None), ("2", "8"), ("2", "4"), ("0", "4")]


def set_attn_knobs(monkeypatch, shared, waves):
    monkeypatch.setenv("ROLLOUT_SHARED_PREFIX", shared)
    if waves is None:
        monkeypatch.delenv("ROLLOUT_ATTN_WAVES", raising=False)
    else:
        monkeypatch.setenv("ROLLOUT_ATTN_WAVES", waves)


@pytest.mark.parametrize("shared,waves", ATTN_KNOBS)
@pytest.mark.parametrize("n_prompts,G,P", [(3, 4, 32), (1, 16, 48), (5, 1, 20)])
def test_bf16_small_teacher_forced_logits(n_prompts, G, P, shared, waves, monkeypatch):
    set_attn_knobs(monkeypatch, shared, waves)
    log(f"bf16 small GQA teacher forced prompts={n_prompts} G={G} P={P} shared={shared} waves={waves}")
    N = 8
    S = n_prompts * G
    cfg = R.model_config(SMALL_BF16, R.DTYPE_BF16, 64, N, S)
    eng = R.Engine(cfg)
    model = OracleModel(shape_of(cfg), mode="bf16")
    prompts = W.prompts(n_prompts, P, cfg.vocab, seed=31)
    u = W.uniforms(S, N, seed=32)
    ref = rollout(model, prompts, G, N, 1.0, 1.0, u)
    logits = torch.empty((S, cfg.vocab), dtype=torch.float32, device="cuda:0")
    R.rollout_prefill(eng.ctx, to_dev(prompts, torch), n_prompts, P, G, logits)
    eng.synchronize()
    err = [float(np.max(np.abs(logits.cpu().numpy() - ref["logits"][0])))]
    for t in range(1, N):
        R.rollout_decode_step(eng.ctx, to_dev(ref["tokens"][:, t - 1], torch), logits)
        eng.synchronize()
        err.append(float(np.max(np.abs(logits.cpu().numpy() - ref["logits"][t]))))
    log(f"  max abs logit error per step: {[round(e, 5) for e in err]}")
    assert max(err) <= 3e-2
    eng.close()


GQA7_BF16 = (2, 256, 14, 2, 128, 512, 2048, 1e6)  # 7 query heads per KV head, head_dim 128 (the 7B ratio)


@pytest.mark.parametrize("shared,waves", ATTN_KNOBS)
@pytest.mark.parametrize("blk,n_prompts,G,P", [(16, 2, 8, 40), (8, 3, 2, 37), (32, 1, 4, 70), (16, 9, 1, 33)])
def test_bf16_gqa7_teacher_forced_logits(blk, n_prompts, G, P, shared, waves, monkeypatch):
    set_attn_knobs(monkeypatch, shared, waves)
    log(f"bf16 GQA 14/2 x 128 teacher forced blk={blk} prompts={n_prompts} G={G} P={P} shared={shared} waves={waves}")
    N = 6
    S = n_prompts * G
    cfg = R.model_config(GQA7_BF16, R.DTYPE_BF16, 80, N, S, kv_block_size=blk)
    eng = R.Engine(cfg)
    model = OracleModel(shape_of(cfg), mode="bf16")
    prompts = W.prompts(n_prompts, P, cfg.vocab, seed=41)
    u = W.uniforms(S, N, seed=42)
    ref = rollout(model, prompts, G, N, 1.0, 1.0, u)
    logits = torch.empty((S, cfg.vocab), dtype=torch.float32, device="cuda:0")
    R.rollout_prefill(eng.ctx, to_dev(prompts, torch), n_prompts, P, G, logits)
    eng.synchronize()
    err = [float(np.max(np.abs(logits.cpu().numpy() - ref["logits"][0])))]
    for t in range(1, N):
        R.rollout_decode_step(eng.ctx, to_dev(ref["tokens"][:, t - 1], torch), logits)
        eng.synchronize()
        err.append(float(np.max(np.abs(logits.cpu().numpy() - ref["logits"][t]))))
    log(f"  max abs logit error per step: {[round(e, 5) for e in err]}")
    assert max(err) <= 3e-2
    eng.close()


# prefill attention: tiles of 128 (token, head) columns and 64 keys.  Prompts of one token, around a key tile
# and around two, column tiles that end inside a token's heads (7 and 5 heads per KV head, 16 with one token
# left over) and head_dim 64, block sizes 8, 16 and 32, several prompts per launch.
PREFILL_ATTN = [
    # (model shape, block size, prompts, prompt length)
    ((1, 256, 14, 2, 128, 256, 2048, 1e6), 16, 2, 1), ((1, 256, 14, 2, 128, 256, 2048, 1e6), 16, 3, 63),
    ((1, 256, 14, 2, 128, 256, 2048, 1e6), 8, 1, 64), ((1, 256, 14, 2, 128, 256, 2048, 1e6), 32, 2, 65),
    ((2, 256, 10, 2, 128, 256, 2048, 1e6), 16, 2, 203), ((1, 256, 16, 1, 64, 256, 2048, 1e6), 8, 3, 129),
    ((1, 256, 3, 3, 64, 256, 2048, 1e6), 32, 1, 127),
]


@pytest.mark.parametrize("shape,blk,n_prompts,P", PREFILL_ATTN)
def test_bf16_prefill_attention_tiles(shape, blk, n_prompts, P):
    log(f"bf16 prefill attention shape={shape} blk={blk} prompts={n_prompts} P={P}")
    G, N = 2, 3
    S = n_prompts * G
    cfg = R.model_config(shape, R.DTYPE_BF16, P, N, S, kv_block_size=blk)
    eng = R.Engine(cfg)
    model = OracleModel(shape_of(cfg), mode="bf16")
    prompts = W.prompts(n_prompts, P, cfg.vocab, seed=47)
    ref = rollout(model, prompts, G, N, 1.0, 1.0, W.uniforms(S, N, seed=48))
    logits = torch.empty((S, cfg.vocab), dtype=torch.float32, device="cuda:0")
    # stale values (NaN bit patterns) in the pool must not reach a prompt's outputs
    eng.arena[eng.plan.arena_bytes - eng.plan.kv_bytes:].fill_(255)
    torch.cuda.synchronize()
    R.rollout_prefill(eng.ctx, to_dev(prompts, torch), n_prompts, P, G, logits)
    eng.synchronize()
    err = [float(np.max(np.abs(logits.cpu().numpy() - ref["logits"][0])))]
    for t in range(1, N):
        R.rollout_decode_step(eng.ctx, to_dev(ref["tokens"][:, t - 1], torch), logits)
        eng.synchronize()
        err.append(float(np.max(np.abs(logits.cpu().numpy() - ref["logits"][t]))))
    log(f"  max abs logit error per step: {[round(e, 5) for e in err]}")
    assert max(err) <= 3e-2  # the bf16 contract's bound, as in the tests above
    eng.close()


# The same tiles, every token observed: the second layer's keys and values of a token follow from all that the first
# layer did with it, and are read from the pool ([layer][block][KV head][K: blk x hd | V: hd x blk], blocks in order).
@pytest.mark.parametrize("heads,nkv,hd,blk,P", [(14, 2, 128, 16, 203), (10, 2, 128, 8, 129), (16, 1, 64, 8, 65),
                                                (3, 3, 64, 32, 257), (7, 1, 128, 32, 300)])
def test_bf16_prefill_every_token(heads, nkv, hd, blk, P):
    log(f"bf16 prefill, every token: {heads} heads, {nkv} KV heads of {hd}, blk={blk} P={P}")
    cfg = R.model_config((2, 256, heads, nkv, hd, 256, 2048, 1e6), R.DTYPE_BF16, P, 1, 2, kv_block_size=blk)
    eng = R.Engine(cfg)
    model = OracleModel(shape_of(cfg), mode="bf16")
    prompts = W.prompts(2, P, cfg.vocab, seed=65)
    logits = torch.empty((2, cfg.vocab), dtype=torch.float32, device="cuda:0")
    eng.arena[eng.plan.arena_bytes - eng.plan.kv_bytes:].fill_(255)  # stale NaN bit patterns
    torch.cuda.synchronize()
    R.rollout_prefill(eng.ctx, to_dev(prompts, torch), 2, P, 1, logits)
    eng.synchronize()
    pool = eng.arena[eng.plan.arena_bytes - eng.plan.kv_bytes:].view(torch.bfloat16).float().cpu().numpy()
    pool = pool.reshape(2, eng.plan.kv_blocks, nkv, 2, blk * hd)[1]
    eng.close()
    per = (P + 1 + blk - 1) // blk  # blocks of a sequence (P tokens and one more)
    worst = 0.0
    for s in range(2):
        blocks = pool[s * per:(s + 1) * per]
        k = blocks[:, :, 0].reshape(per, nkv, blk, hd).transpose(0, 2, 1, 3).reshape(per * blk, nkv, hd)[:P]
        v = blocks[:, :, 1].reshape(per, nkv, hd, blk).transpose(0, 3, 1, 2).reshape(per * blk, nkv, hd)[:P]
        (_, (wk, wv)), want = model.prefill(prompts[s])
        for got, ref in ((k, wk), (v, wv)):
            row = np.sqrt(((got - ref) ** 2).sum((1, 2)) / (ref ** 2).sum((1, 2)))
            # nine bf16 roundings on the way (three norms, q, k, v, attention, silu(g) * u, the result), as in check_rows
            assert row.max() <= 3 / 128, f"prompt {s} token {int(np.nanargmax(row))}: {row.max():.3g}"
            worst = max(worst, float(row.max()))
        assert np.max(np.abs(logits.cpu().numpy()[s] - want)) <= 3e-2
    log(f"  worst token {worst:.3g} of its norm")


# the LM head after a prefill stores a prompt's row for every member that is not a copy in its operand: 40 rows three
# times, one row 67 times, 70 rows (more than 64) twice, 8 prompts of 7 members copied as far as 64 rows go
@pytest.mark.parametrize("dtype,mode,shape,tol", [(R.DTYPE_FP32, "fp32", "tiny", 1e-4), (R.DTYPE_BF16, "bf16", SMALL_BF16, 3e-2)])
@pytest.mark.parametrize("n_prompts,G", [(40, 3), (1, 67), (70, 2), (8, 7)])
def test_prefill_logits_of_every_member(n_prompts, G, dtype, mode, shape, tol):
    log(f"prefill logits of every member: {mode}, {n_prompts} prompts, G={G}")
    P = 3
    cfg = R.model_config(shape, dtype, P, 1, n_prompts * G)
    eng = R.Engine(cfg, group_size=G)
    model = OracleModel(shape_of(cfg), mode=mode)
    prompts = W.prompts(n_prompts, P, cfg.vocab, seed=67)
    want = np.stack([model.prefill(p)[1] for p in prompts])
    logits = torch.full((n_prompts, G, cfg.vocab), float("nan"), dtype=torch.float32, device="cuda:0")
    R.rollout_prefill(eng.ctx, to_dev(prompts, torch), n_prompts, P, G, logits)
    eng.synchronize()
    eng.close()
    got = logits.cpu().numpy()
    assert np.max(np.abs(got - want[:, None])) <= tol
    assert np.array_equal(got, np.repeat(got[:, :1], G, axis=1))  # rows of a group are equal


@pytest.mark.parametrize("name", [n for n, t in TILE_ROWS.items() if t[0]])
def test_bf16_tile_gemm_rows(name):
    rows, _, shape = TILE_ROWS[name]
    cfg = R.model_config(shape, R.DTYPE_BF16, 1, 1, max(rows))
    eng = R.Engine(cfg)
    model = OracleModel(shape_of(cfg), mode="bf16")
    tokens = W.prompts(max(rows), 1, cfg.vocab, seed=49)
    want = one_token_logits(model, tokens[:, 0])
    for n in rows:
        log(f"bf16 tile GEMM, {name}: {n} rows")
        logits = torch.empty((n, cfg.vocab), dtype=torch.float32, device="cuda:0")
        R.rollout_prefill(eng.ctx, to_dev(tokens[:n], torch), n, 1, 1, logits)
        eng.synchronize()
        check_rows(logits.cpu().numpy(), want[:n])
    eng.close()


# decode rows whose context is shared out over workgroups (from position 384 on in small batches): the step that
# begins to, a last part of one token, 5 to 16 parts of one tile a wave and more, one and seven column groups
PARTS_ATTN = [
    # (model shape, block size, prompts, G, prompt length)
    ((1, 256, 14, 2, 128, 256, 2048, 1e6), 16, 1, 2, 382), ((1, 256, 14, 2, 128, 256, 2048, 1e6), 8, 3, 1, 513),
    ((1, 256, 4, 1, 64, 256, 2048, 1e6), 32, 1, 3, 385), ((1, 256, 4, 1, 128, 256, 2048, 1e6), 16, 2, 2, 1027),
]


@pytest.mark.parametrize("shape,blk,n_prompts,G,P", PARTS_ATTN)
def test_bf16_decode_attention_parts(shape, blk, n_prompts, G, P, monkeypatch):
    set_attn_knobs(monkeypatch, "1", None)
    log(f"bf16 decode attention in parts shape={shape} blk={blk} prompts={n_prompts} G={G} P={P}")
    S, N = n_prompts * G, 4
    cfg = R.model_config(shape, R.DTYPE_BF16, P, N, S, kv_block_size=blk)
    eng = R.Engine(cfg)
    model = OracleModel(shape_of(cfg), mode="bf16")
    prompts = W.prompts(n_prompts, P, cfg.vocab, seed=61)
    ref = rollout(model, prompts, G, N, 1.0, 1.0, W.uniforms(S, N, seed=62))
    logits = torch.empty((S, cfg.vocab), dtype=torch.float32, device="cuda:0")
    # stale values (NaN bit patterns) in the pool must not reach the outputs
    eng.arena[eng.plan.arena_bytes - eng.plan.kv_bytes:].fill_(255)
    torch.cuda.synchronize()
    R.rollout_prefill(eng.ctx, to_dev(prompts, torch), n_prompts, P, G, logits)
    eng.synchronize()
    err = [float(np.max(np.abs(logits.cpu().numpy() - ref["logits"][0])))]
    for t in range(1, N):
        R.rollout_decode_step(eng.ctx, to_dev(ref["tokens"][:, t - 1], torch), logits)
        eng.synchronize()
        err.append(float(np.max(np.abs(logits.cpu().numpy() - ref["logits"][t]))))
    log(f"  max abs logit error per step: {[round(e, 5) for e in err]}")
    assert max(err) <= 3e-2  # the bf16 contract's bound, as in the tests above
    eng.close()


@pytest.mark.parametrize("shared", ["0", "2"])
def test_bf16_gqa7_context_beyond_4096_tokens_teacher_forced(shared, monkeypatch):
    # A context of more than 256 blocks of 16 (4,096 tokens): the decode attention's workgroup of 256
    # threads then copies the sequence's block table in more than one pass, and the prefill attention reads
    # a 4,090-token prompt.  The decode steps cross from 256 to 257 blocks; with the shared-prefix path the
    # prompt's 255 full blocks go to the prefix pass and the suffix pass starts at block 255.
    set_attn_knobs(monkeypatch, shared, None)
    n_prompts, G, P, N = 1, 2, 4090, 12
    log(f"bf16 GQA 14/2 x 128 teacher forced, context {P} .. {P + N - 1} (beyond 256 blocks), shared={shared}")
    S = n_prompts * G
    cfg = R.model_config(GQA7_BF16, R.DTYPE_BF16, P, N, S)
    eng = R.Engine(cfg, group_size=G)
    model = OracleModel(shape_of(cfg), mode="bf16")
    prompts = W.prompts(n_prompts, P, cfg.vocab, seed=45)
    u = W.uniforms(S, N, seed=46)
    ref = rollout(model, prompts, G, N, 1.0, 1.0, u)
    log("  oracle done")
    logits = torch.empty((S, cfg.vocab), dtype=torch.float32, device="cuda:0")
    R.rollout_prefill(eng.ctx, to_dev(prompts, torch), n_prompts, P, G, logits)
    eng.synchronize()
    err = [float(np.max(np.abs(logits.cpu().numpy() - ref["logits"][0])))]
    for t in range(1, N):
        R.rollout_decode_step(eng.ctx, to_dev(ref["tokens"][:, t - 1], torch), logits)
        eng.synchronize()
        err.append(float(np.max(np.abs(logits.cpu().numpy() - ref["logits"][t]))))
    log(f"  max abs logit error per step: {[round(e, 5) for e in err]}")
    assert max(err) <= 3e-2
    eng.close()


def test_bf16_gqa7_large_batch_teacher_forced_logits(monkeypatch):
    # 32 groups of 8: 512 (row, KV head) attention workgroups, where the library picks four waves by itself;
    # G x shared prompt = 8 x 64 keeps the shared-prefix pass off by size, so it is forced on here as well
    for shared in ("1", "2"):
        set_attn_knobs(monkeypatch, shared, None)
        log(f"bf16 GQA 14/2 x 128 teacher forced, 32 prompts x G=8, P=70, shared={shared}")
        n_prompts, G, P, N = 32, 8, 70, 3
        S = n_prompts * G
        cfg = R.model_config(GQA7_BF16, R.DTYPE_BF16, 80, N, S)
        eng = R.Engine(cfg)
        model = OracleModel(shape_of(cfg), mode="bf16")
        prompts = W.prompts(n_prompts, P, cfg.vocab, seed=43)
        u = W.uniforms(S, N, seed=44)
        ref = rollout(model, prompts, G, N, 1.0, 1.0, u)
        logits = torch.empty((S, cfg.vocab), dtype=torch.float32, device="cuda:0")
        R.rollout_prefill(eng.ctx, to_dev(prompts, torch), n_prompts, P, G, logits)
        eng.synchronize()
        err = [float(np.max(np.abs(logits.cpu().numpy() - ref["logits"][0])))]
        for t in range(1, N):
            R.rollout_decode_step(eng.ctx, to_dev(ref["tokens"][:, t - 1], torch), logits)
            eng.synchronize()
            err.append(float(np.max(np.abs(logits.cpu().numpy() - ref["logits"][t]))))
        log(f"  max abs logit error per step: {[round(e, 5) for e in err]}")
        assert max(err) <= 3e-2
        eng.close()


# Shapes whose GEMMs have odd k-step counts and ragged weight groups: d_model 32 (one 32-wide k-step, so
# the second wave of a two-wave decode workgroup has none), d_model 96 / d_ff 160 (3 and 5 k-steps, split
# unevenly between the two waves), and row counts (QKV 160 = 10 blocks, vocab 208 = 13 blocks) that leave
# the last four-block weight group short.  Prefill (72 rows) takes the tile GEMM, decode the ring.
ODD_BF16 = [(1, 32, 1, 1, 32, 32, 64, 1e4), (2, 96, 3, 1, 32, 160, 208, 1e4),
            # gate/up of 2 x 9248 rows = 1156 blocks: the balanced decode grid (one workgroup per CU, 4 or 5
            # blocks each, the two waves splitting K); a vocabulary of 75,008 = 4688 blocks: the balanced LM
            # head (four one-wave workgroups per CU, 4 or 5 blocks each)
            (1, 128, 4, 2, 32, 9248, 75008, 1e4)]


@pytest.mark.parametrize("shape", ODD_BF16)
def test_bf16_odd_k_steps_teacher_forced_logits(shape):
    log(f"bf16 odd shape {shape} teacher forced")
    n_prompts, G, P, N = 3, 4, 24, 5
    S = n_prompts * G
    cfg = R.model_config(shape, R.DTYPE_BF16, P, N, S)
    eng = R.Engine(cfg)
    model = OracleModel(shape_of(cfg), mode="bf16")
    prompts = W.prompts(n_prompts, P, cfg.vocab, seed=51)
    u = W.uniforms(S, N, seed=52)
    ref = rollout(model, prompts, G, N, 1.0, 1.0, u)
    logits = torch.empty((S, cfg.vocab), dtype=torch.float32, device="cuda:0")
    R.rollout_prefill(eng.ctx, to_dev(prompts, torch), n_prompts, P, G, logits)
    eng.synchronize()
    err = [float(np.max(np.abs(logits.cpu().numpy() - ref["logits"][0])))]
    for t in range(1, N):
        R.rollout_decode_step(eng.ctx, to_dev(ref["tokens"][:, t - 1], torch), logits)
        eng.synchronize()
        err.append(float(np.max(np.abs(logits.cpu().numpy() - ref["logits"][t]))))
    scale = float(np.max(np.abs(np.asarray(ref["logits"]))))
    log(f"  max abs logit error per step: {['%.2e' % e for e in err]} (logits up to {scale:.3f})")
    assert scale > 1e-2  # the comparison is not between near-zero logits
    assert max(err) <= 3e-2
    eng.close()


# Decode batches of more than 64 rows take the tile GEMM: 170 rows are two activation tiles of 128 rows for the split
# projections and one of 256 for gate/up and the LM head, the last 16-row block ragged; the 512- and 1536-wide
# K dimensions split into 2 and 6 partials.
TALL_BF16 = (1, 512, 8, 2, 64, 1536, 2048, 1e6)


def test_bf16_tall_decode_batch_teacher_forced_logits():
    log("bf16 tall decode batch: 10 prompts x G=17 (170 rows) teacher forced")
    n_prompts, G, P, N = 10, 17, 24, 4
    S = n_prompts * G
    cfg = R.model_config(TALL_BF16, R.DTYPE_BF16, P, N, S)
    eng = R.Engine(cfg)
    model = OracleModel(shape_of(cfg), mode="bf16")
    prompts = W.prompts(n_prompts, P, cfg.vocab, seed=57)
    u = W.uniforms(S, N, seed=58)
    ref = rollout(model, prompts, G, N, 1.0, 1.0, u)
    logits = torch.empty((S, cfg.vocab), dtype=torch.float32, device="cuda:0")
    R.rollout_prefill(eng.ctx, to_dev(prompts, torch), n_prompts, P, G, logits)
    eng.synchronize()
    err = [float(np.max(np.abs(logits.cpu().numpy() - ref["logits"][0])))]
    for t in range(1, N):
        R.rollout_decode_step(eng.ctx, to_dev(ref["tokens"][:, t - 1], torch), logits)
        eng.synchronize()
        err.append(float(np.max(np.abs(logits.cpu().numpy() - ref["logits"][t]))))
    log(f"  max abs logit error per step: {[round(e, 5) for e in err]}")
    assert max(err) <= 3e-2
    eng.close()


# The shared-prefix pass at many groups (384 and 640 rows, decode on the tile GEMM) with eight query heads
# per KV head: 64 groups of 6 (three full 16-column tiles per group and KV head) and 128 groups of 5 (40
# columns, the last tile half filled).
WIDE_PREFIX_BF16 = (1, 512, 16, 2, 64, 512, 2048, 1e6)


@pytest.mark.parametrize("n_prompts,G", [(64, 6), (128, 5)])
def test_bf16_shared_prefix_wide_workgroups_teacher_forced(n_prompts, G, monkeypatch):
    set_attn_knobs(monkeypatch, "2", None)
    log(f"bf16 shared prefix, {n_prompts} prompts x G={G}, 8 query heads per KV head, teacher forced")
    P, N = 40, 3
    S = n_prompts * G
    cfg = R.model_config(WIDE_PREFIX_BF16, R.DTYPE_BF16, P, N, S)
    eng = R.Engine(cfg, group_size=G)
    model = OracleModel(shape_of(cfg), mode="bf16")
    prompts = W.prompts(n_prompts, P, cfg.vocab, seed=63)
    u = W.uniforms(S, N, seed=64)
    ref = rollout(model, prompts, G, N, 1.0, 1.0, u)
    logits = torch.empty((S, cfg.vocab), dtype=torch.float32, device="cuda:0")
    R.rollout_prefill(eng.ctx, to_dev(prompts, torch), n_prompts, P, G, logits)
    eng.synchronize()
    err = [float(np.max(np.abs(logits.cpu().numpy() - ref["logits"][0])))]
    for t in range(1, N):
        R.rollout_decode_step(eng.ctx, to_dev(ref["tokens"][:, t - 1], torch), logits)
        eng.synchronize()
        err.append(float(np.max(np.abs(logits.cpu().numpy() - ref["logits"][t]))))
    log(f"  max abs logit error per step: {[round(e, 5) for e in err]}")
    assert max(err) <= 3e-2
    eng.close()


def test_device_error_flag_on_bad_token():
    eng, cfg = _tiny_engine()
    prompts = W.prompts(2, 16, cfg.vocab)
    prompts[1, 3] = cfg.vocab + 5  # outside the vocabulary: the kernel clamps and flags it
    logits = torch.empty((8, cfg.vocab), dtype=torch.float32, device="cuda:0")
    R.rollout_prefill(eng.ctx, to_dev(prompts, torch), 2, 16, 4, logits)
    with pytest.raises(R.RolloutError) as e:
        eng.synchronize()
    assert e.value.code == R.EINVAL and "token id" in str(e.value)
    eng.synchronize()  # the flag was cleared
    with pytest.raises(R.RolloutError) as e:
        R.rollout_decode_step(eng.ctx, to_dev(np.zeros(8, np.int32), torch), logits)
        for _ in range(20):
            R.rollout_decode_step(eng.ctx, to_dev(np.zeros(8, np.int32), torch), logits)
    assert e.value.code == R.ESTATE
    eng.close()
