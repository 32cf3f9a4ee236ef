"""Shared helpers of the GPU parity tests (inputs come from the seeded workload;
expected values come from the oracle only)."""
import sys

import numpy as np

import workload as W


def log(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def to_dev(arr, torch, device="cuda:0"):
    return torch.from_numpy(np.ascontiguousarray(arr)).to(device)


def shape_of(cfg):
    return W.ModelShape(cfg.n_layers, cfg.d_model, cfg.n_heads, cfg.n_kv_heads, cfg.head_dim, cfg.d_ff, cfg.vocab,
                        cfg.rms_eps, cfg.rope_theta)


def one_token_logits(model, tokens):
    """Oracle logits [n, V] of n one-token prompts together: position 0, and attention over one key is its value."""
    x = model.embed[tokens].astype(np.float64)
    pos = np.zeros(len(tokens))
    for lw in model.layers:
        _, _, v = model._qkv(lw, x, pos)
        x = model._post_attn(lw, x, np.repeat(v, model.n_rep, axis=1))
    return model.logits_from_hidden(x)


def check_rows(got, want):
    """Every row of bf16-contract logits.  Both sides round the same values to bf16 at five points (two norms, v, the
    attention's output, silu(g) * u), and a rounding that falls the other way moves an element by one spacing, at most
    2^-7 of it: a row differs by at most sqrt(5) 2^-7 of its norm even if all of them did.  Single logits: the
    contract's 3e-2 for logits of unit size."""
    err = np.abs(got - want)
    row = np.sqrt((err ** 2).sum(1) / (want ** 2).sum(1))
    rms = float(np.sqrt((want ** 2).mean()))
    log(f"  max abs logit error {err.max():.4g} (logits of rms {rms:.3g}), worst row {row.max():.3g} of its norm")
    assert row.max() <= np.sqrt(5) / 128, f"row {int(row.argmax())}"
    assert err.max() <= 3e-2 * max(1.0, rms)


# Models and row counts of the row tests of the GEMM for more than 64 rows (one-token prompts, so that every row has
# logits of its own).  Row counts around its tile choices (128- and 256-row activation tiles, one to three of them),
# most of them ragged; K and N that leave odd k-steps, short K splits and partial weight tiles; gate/up and LM head wide
# enough for the large tiles; O and down of one split, which add to the residual stream.
TILE_ROWS = {
    # name: (bf16 rows, int4 rows, (layers, d_model, heads, kv heads, head_dim, d_ff, vocab, rope theta))
    "odd k-steps": ((65, 128, 129, 256, 257, 385, 513, 1053), (), (1, 544, 10, 2, 64, 1056, 2064, 1e6)),
    "ragged tiles": ((), (65, 129, 256, 257, 385, 513), (1, 640, 10, 2, 64, 1408, 2064, 1e6)),
    "one split": ((65, 129, 257, 385), (65, 129, 257), (1, 640, 6, 2, 64, 384, 2064, 1e6)),
    "wide": ((65, 129, 257, 513), (65, 129, 257, 385), (1, 640, 6, 2, 64, 26368, 52736, 1e6)),
    "half as wide": ((385, 513), (513,), (1, 640, 6, 2, 64, 6656, 20480, 1e6)),
    "wide residual": ((385, 513), (129, 513), (1, 26624, 6, 2, 64, 384, 2064, 1e6)),
}


def guarded_token_compare(gpu_tokens, oracle_tokens, oracle_margins, guard=1e-5):
    """Compare free-running token streams sequence by sequence.

    Tokens must agree up to and including the first draw whose oracle margin is
    below ``guard`` (a legitimate near-tie); a mismatch exactly at that draw is
    allowed and later draws are not compared.  Returns (compared, skipped).
    """
    compared = skipped = 0
    for s in range(oracle_tokens.shape[0]):
        for t in range(oracle_tokens.shape[1]):
            near_tie = oracle_margins[s, t] < guard
            if gpu_tokens[s, t] != oracle_tokens[s, t]:
                assert near_tie, f"sequence {s} step {t}: gpu {gpu_tokens[s, t]} oracle {oracle_tokens[s, t]} " \
                                 f"(margin {oracle_margins[s, t]:.3g})"
                skipped += oracle_tokens.shape[1] - t
                break
            compared += 1
            if near_tie:
                skipped += oracle_tokens.shape[1] - t - 1
                break
    return compared, skipped
