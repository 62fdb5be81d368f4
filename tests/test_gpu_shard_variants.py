"""The sharded loss at the row lengths where its kernel changes (512 and 1,600 vectors of 16 bytes, whole and ragged), at
shard counts below, at and above a wave's 64 lanes, records of fully masked shards among them, against the oracle over the
whole rows with the gates of tests/gpu_parity.py."""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_05597_amd as grpo
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


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("V", [5, 1001, 6400])
def test_dlogits_at_another_distance(V, dtype):
    # element loads and stores, against the vector kernel's dlogits at the logits' own distance from a 16-byte boundary
    T, dt = 50, torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator("cuda").manual_seed(V)
    x = torch.randn((T, V), generator=g, device="cuda").to(dt)
    act = torch.randint(0, V, (T,), generator=g, device="cuda", dtype=torch.int32)
    behave = torch.log_softmax(x.float(), 1).gather(1, act.long()[:, None])[:, 0].contiguous()
    sto = torch.tensor([0, 20, 35, T], dtype=torch.int32, device="cuda")
    tso = torch.tensor([0, 1, 3], dtype=torch.int32, device="cuda")
    adv = torch.tensor([1.0, -1.0], device="cuda")
    stats = grpo.grpo_vocab_shard_stats(x, act, 0).view(1, T, -1)
    out = []
    for shift in (0, 1):
        dl = torch.full((T * V + 16,), 7.0, dtype=dt, device="cuda")
        loss, _ = grpo.grpo_loss_fwd_bwd_vocab_shard(x, stats, 0, V, act, behave, adv, sto, tso, 2, grad_scale=50.0,
                                                     dlogits=dl[shift:shift + T * V].view(T, V))
        assert (dl[:shift] == 7).all() and (dl[shift + T * V:] == 7).all()
        out.append((loss.item(), dl[shift:shift + T * V].double()))
    assert out[0][0] == out[1][0]
    rel = 2.0 ** -7 if dtype == "bf16" else 2.0 ** -22  # a value next to a rounding boundary goes either way
    assert ((out[0][1] - out[1][1]).abs() <= rel * out[0][1].abs()).all()
