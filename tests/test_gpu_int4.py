"""GPU parity of the int4 weight-only path (ROLLOUT_DTYPE_INT4) against the oracle's int4 mode.

The library quantises the layer projections on the device from the same seeded fp32 weights; the exported
dequantised values (q - z) * s in fp32 must equal the oracle's quantiser bit for bit, and logits must stay
within the bf16 tolerance of the oracle run over the exact dequantised weights.  Decode batches up to 64
rows take the group-scaled int4 ring GEMM, larger batches (prefill chunks, 256-row decode) write the integers
q - z out as bf16 fragments and take the tile GEMM with the groups' scales.
"""
import numpy as np
import pytest

import paper_2608_11226_amd as R
import workload as W
from gpu_helpers import TILE_ROWS, check_rows, log, one_token_logits, shape_of, to_dev
from oracle import OracleModel, bf16_round, rollout
from oracle.quant import dequantize_int4, quantize_int4

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# (layers, d_model, heads, kv heads, head_dim, d_ff, vocab, rope theta)
INT4_SMALL = (2, 256, 8, 2, 64, 512, 2048, 1e6)
INT4_RAGGED = (2, 256, 8, 1, 32, 384, 2048, 1e4)    # q/k/v rows 320 = 20 weight blocks: a ragged ring group
INT4_SPLITS = (2, 512, 8, 2, 64, 1536, 2048, 1e6)   # down projection over 1536 inputs: six K splits of 256
INT4_GQA7 = (2, 256, 14, 2, 128, 512, 2048, 1e6)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    assert torch.cuda.is_available(), "GPU tests need a ROCm GPU"
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("shape", [INT4_SMALL, INT4_RAGGED, INT4_SPLITS])
def test_int4_weights_bit_exact(shape):
    cfg = R.model_config(shape, R.DTYPE_INT4, 16, 8, 4)
    log(f"int4 weights shape={shape}")
    eng = R.Engine(cfg)
    sh = shape_of(cfg)
    ids = [(0, "embed", False), (W.tensor_id_lm_head(sh), "lm_head", False)]
    for l in range(sh.n_layers):
        for slot in (W.WQ, W.WK, W.WV, W.WO, W.WGATE, W.WUP, W.WDOWN):
            ids.append((W.tensor_id_layer(l, slot), W.LAYER_SLOTS[slot], True))
    for tid, name, q4 in ids:
        rows, cols = W.logical_shape(sh, name)
        out = torch.empty(rows * cols, dtype=torch.float32, device="cuda:0")
        R.rollout_export_weight(eng.ctx, tid, out)
        eng.synchronize()
        w = W.weight_matrix(0, tid, rows, cols)
        want = (dequantize_int4(*quantize_int4(w)) if q4 else bf16_round(w).astype(np.float32)).reshape(-1)
        got = out.cpu().numpy()
        bad = np.flatnonzero(got.view(np.uint32) != want.view(np.uint32))
        assert bad.size == 0, f"tensor {tid} ({name}): {bad.size} differ, first at {bad[0]}: " \
                              f"{got[bad[0]]} vs {want[bad[0]]}"
    eng.close()


def _teacher_forced(shape, n_prompts, G, P, N, blk=16, seed=51):
    S = n_prompts * G
    cfg = R.model_config(shape, R.DTYPE_INT4, max(P, 16), N, S, kv_block_size=blk)
    eng = R.Engine(cfg)
    model = OracleModel(shape_of(cfg), mode="int4")
    prompts = W.prompts(n_prompts, P, cfg.vocab, seed=seed)
    u = W.uniforms(S, N, seed=seed + 1)
    ref = rollout(model, prompts, G, N, 1.0, 1.0, u)
    logits = torch.empty((S, cfg.vocab), dtype=torch.float32, device="cuda:0")
    R.rollout_prefill(eng.ctx, to_dev(prompts, torch), n_prompts, P, G, logits)
    eng.synchronize()
    err = [float(np.max(np.abs(logits.cpu().numpy() - ref["logits"][0])))]
    for t in range(1, N):
        R.rollout_decode_step(eng.ctx, to_dev(ref["tokens"][:, t - 1], torch), logits)
        eng.synchronize()
        err.append(float(np.max(np.abs(logits.cpu().numpy() - ref["logits"][t]))))
    eng.close()
    return err


def _one_token_rows(what, shape, rows):
    """Prompts of one token, so that every row of every GEMM has logits of its own to compare."""
    cfg = R.model_config(shape, R.DTYPE_INT4, 1, 1, max(rows))
    eng = R.Engine(cfg)
    model = OracleModel(shape_of(cfg), mode="int4")
    tokens = W.prompts(max(rows), 1, cfg.vocab, seed=57)
    want = one_token_logits(model, tokens[:, 0])
    for n in rows:
        log(f"{what}: {n} rows")
        logits = torch.empty((n, cfg.vocab), dtype=torch.float32, device="cuda:0")
        R.rollout_prefill(eng.ctx, to_dev(tokens[:n], torch), n, 1, 1, logits)
        eng.synchronize()
        check_rows(logits.cpu().numpy(), want[:n])
    eng.close()


# prefill rows n_prompts x P above or below 64 (dequantise + tile GEMM, or the int4 ring), decode rows S
@pytest.mark.parametrize("shape,n_prompts,G,P", [
    (INT4_SMALL, 3, 4, 32),     # prefill 96 rows (tile), decode 12 rows (ring, one 16-row block)
    (INT4_SMALL, 1, 16, 48),    # prefill 48 rows (ring, three blocks), decode 16
    (INT4_RAGGED, 2, 8, 20),    # ragged weight blocks, decode 16 rows
    (INT4_SPLITS, 5, 12, 13),   # prefill 65 rows (tile), decode 60 rows (ring, four blocks), K splits
    (INT4_GQA7, 2, 8, 40),
])
def test_int4_teacher_forced_logits(shape, n_prompts, G, P):
    log(f"int4 teacher forced shape={shape} prompts={n_prompts} G={G} P={P}")
    err = _teacher_forced(shape, n_prompts, G, P, N=6)
    log(f"  max abs logit error per step: {[round(e, 5) for e in err]}")
    assert max(err) <= 3e-2


def test_int4_large_batch_decode_logits():
    # 256 decode rows: every projection of a decode step writes its integers q - z out and takes the tile GEMM
    log("int4 teacher forced, 32 prompts x G=8, P=24 (256-row decode)")
    err = _teacher_forced(INT4_SMALL, 32, 8, 24, N=3, seed=53)
    log(f"  max abs logit error per step: {[round(e, 5) for e in err]}")
    assert max(err) <= 3e-2


@pytest.mark.parametrize("name", [n for n, t in TILE_ROWS.items() if t[1]])
def test_int4_tile_gemm_rows(name):
    _, rows, shape = TILE_ROWS[name]
    _one_token_rows(f"int4 tile GEMM, {name}", shape, rows)


# the ring GEMM at one to four 16-row blocks: one group (a set of waves without any), five (an odd share) and
# eleven over K splits; 26368 gate/up features are enough blocks for the form whose waves all share a group
@pytest.mark.parametrize("d,d_ff", [(128, 384), (640, 1408), (640, 26368)])
def test_int4_ring_gemm_rows(d, d_ff):
    heads = d // 64 if d > 128 else 2
    _one_token_rows(f"int4 ring GEMM d={d} d_ff={d_ff}", (1, d, heads, 2, 64, d_ff, 2064, 1e6), (1, 16, 17, 33, 64))
