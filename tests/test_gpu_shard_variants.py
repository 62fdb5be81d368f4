"""The sharded loss at the row lengths where its kernel changes (512 and 1,600 vectors of 16 bytes, whole and ragged), at
shard counts below, at and above a wave's 64 lanes, records of fully masked shards among them, against the oracle over the
whole rows with the gates of tests/gpu_parity.py."""
import numpy as np
import pytest
import torch

import oracle
from synth.rollouts import Config, make_batch
from tests.gpu_parity import LOSS_RTOL, check_dlogits, dl_to_f64, gpu_norm, oracle_inputs, to_np_logits
from tests.test_gpu_vocab_shard import _adv, run_sharded

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,shards,Vs", [("bf16", 2, 4096), ("bf16", 2, 4104), ("bf16", 2, 4099), ("bf16", 2, 12800),
                                             ("bf16", 2, 12811), ("f32", 2, 2048), ("f32", 3, 2051), ("f32", 2, 6404),
                                             ("bf16", 8, 1000), ("bf16", 63, 24), ("bf16", 64, 24), ("bf16", 65, 24),
                                             ("bf16", 131, 8)])
def test_variants(dtype, shards, Vs):
    V = shards * Vs
    cfg = Config("shards", 2, 4, V, dtype, 2.0, 0.5, (1, 3), (1, 3), 4.0, (1, 8), 0.1, 4.0, seed=V % 97)
    b = make_batch(cfg, "cuda", with_prox=True)
    b["logits"][::3, :Vs] = float("-inf")  # the first shard of every third row holds no probability
    b["actions"][::3] = b["actions"][::3] % (V - Vs) + Vs
    A64, A32 = _adv(b)
    oi = oracle_inputs(b, A64)
    ref = oracle.loss_rows(to_np_logits(b["logits"]), oi["actions"], oi["behave"], oi["prox"], oi["adv"], oi["seg"], cfg.G,
                           V=V, norm=oracle.NORM_CONST_K, k=cfg.k, dual_clip_c=3.0)
    bounds = list(range(0, V + 1, Vs))
    losses, dl, _, _ = run_sharded(b, A32, bounds, norm=gpu_norm(oracle.NORM_CONST_K), k=cfg.k, c=3.0)
    assert len(set(losses)) == 1
    assert abs(losses[0] - ref.loss) <= LOSS_RTOL * np.abs(ref.token_contrib).sum()
    check_dlogits(dl_to_f64(dl), ref.dlogits, dtype == "bf16", what=f"{shards} x {Vs}")
