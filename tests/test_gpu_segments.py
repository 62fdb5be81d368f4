"""The per-token tables and the reduction at the sizes where they change kernel: batches of up to 1,024 trajectories and
16,384 steps make their tables in one launch, larger ones in two, and clip counts and ratio statistics are formed for
the calls that ask for them.  Integers exactly, the loss and the statistics as in tests/gpu_parity.py."""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_05597_amd as grpo
from tests.gpu_parity import LOSS_RTOL, gpu_norm, to_np_logits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("norm", [oracle.NORM_CONST_K, oracle.NORM_TRAJ_STEPS])
@pytest.mark.parametrize("n_traj,max_steps", [(4, 3), (1024, 4), (1028, 4), (600, 52)])
def test_tables_and_reduction(n_traj, max_steps, norm):
    G, V = 4, 64
    rng = np.random.default_rng(n_traj + max_steps)
    steps = rng.integers(1, max_steps + 1, n_traj)
    toks = rng.integers(0, 3, int(steps.sum()))
    sto = np.concatenate([[0], np.cumsum(toks)]).astype(np.int32)
    tso = np.concatenate([[0], np.cumsum(steps)]).astype(np.int32)
    T = int(sto[-1])
    lg = torch.randn((T, V), generator=torch.Generator("cuda").manual_seed(1), device="cuda")
    act = torch.from_numpy(rng.integers(0, V, T).astype(np.int32)).cuda()
    lp = torch.log_softmax(lg, 1).gather(1, act.long()[:, None])[:, 0]
    behave = lp + 0.3 * torch.randn(T, generator=torch.Generator("cuda").manual_seed(2), device="cuda")
    adv = oracle.advantages(rng.integers(0, 2, n_traj).astype(np.float32), G).astype(np.float32)
    seg = oracle.segments(T, sto, tso)
    ref = oracle.loss_rows(to_np_logits(lg), act.cpu().numpy(), behave.cpu().numpy(), None, adv.astype(np.float64),
                           seg, G, norm=norm, k=5.0, dual_clip_c=3.0)
    want = oracle.ratio_stats(ref.token_logp, behave.cpu().numpy(), None, oracle.valid_tokens(act.cpu().numpy(), V, seg))
    for which in ((), ("clip_counts", "error_flags"), ("ratio_stats",),
                  ("tok_traj", "traj_tok_off", "gather_idx", "traj_loss", "clip_counts", "ratio_stats")):
        aux = grpo.LossAux.alloc(T, n_traj, "cuda", which=which)
        loss, _ = grpo.grpo_loss_fwd_bwd(lg, act, behave, torch.from_numpy(adv).cuda(), torch.from_numpy(sto).cuda(),
                                         torch.from_numpy(tso).cuda(), G, norm=gpu_norm(norm), k=5.0, dual_clip_c=3.0,
                                         aux=aux if which else None)
        torch.cuda.synchronize()
        assert abs(loss.item() - ref.loss) <= LOSS_RTOL * np.abs(ref.token_contrib).sum()
        near = 2  # tokens whose fp64 ratio lies next to a boundary may fall either way
        if aux.clip_counts is not None:
            got = aux.clip_counts.cpu().numpy()
            assert abs(got[0] - (ref.token_state & 1).sum()) <= near
            assert abs(got[1] - ((ref.token_state >> 1) & 1).sum()) <= near
        if aux.ratio_stats is not None:
            got = aux.ratio_stats.cpu().numpy()
            np.testing.assert_allclose(got[:6], want[:6], rtol=1e-5)
            assert abs(got[6] - want[6]) <= near and got[7] == want[7] == T
        if aux.tok_traj is not None:
            assert (aux.tok_traj.cpu().numpy() == seg.tok_traj).all()
            assert (aux.traj_tok_off.cpu().numpy() == seg.traj_tok_off).all()
            assert (aux.gather_idx.cpu().numpy() == oracle.gather_index(T, V, act.cpu().numpy())).all()
            np.testing.assert_allclose(aux.traj_loss.cpu().numpy(), ref.traj_loss, rtol=LOSS_RTOL,
                                       atol=LOSS_RTOL * np.abs(ref.traj_loss).max())


def test_long_trajectories():
    """Trajectories on both sides of the reduction's 1,024 tokens at a time, a token outside the loss in each."""
    G, V, toks = 5, 64, [1, 769, 1024, 1025, 2777]
    sto = np.concatenate([[0], np.cumsum(toks)]).astype(np.int32)
    tso = np.arange(G + 1, dtype=np.int32)
    T = int(sto[-1])
    lg = torch.randn((T, V), generator=torch.Generator("cuda").manual_seed(1), device="cuda")
    act = torch.randint(0, V, (T,), generator=torch.Generator("cuda").manual_seed(3), device="cuda", dtype=torch.int32)
    lp = torch.log_softmax(lg, 1).gather(1, act.long()[:, None])[:, 0]
    act[torch.from_numpy(sto[1:] - 1).long().cuda()] = V  # each trajectory's last token
    behave = lp + 0.3 * torch.randn(T, generator=torch.Generator("cuda").manual_seed(2), device="cuda")
    adv = oracle.advantages(np.array([1, 0, 1, 0, 0], np.float32), G).astype(np.float32)
    seg = oracle.segments(T, sto, tso)
    ref = oracle.loss_rows(to_np_logits(lg), act.cpu().numpy(), behave.cpu().numpy(), None, adv.astype(np.float64),
                           seg, G, norm=oracle.NORM_CONST_K, k=5.0, dual_clip_c=3.0)
    valid = oracle.valid_tokens(act.cpu().numpy(), V, seg)
    want = oracle.ratio_stats(ref.token_logp, behave.cpu().numpy(), None, valid)
    for which in ((), ("clip_counts",), ("ratio_stats", "clip_counts", "traj_loss")):
        aux = grpo.LossAux.alloc(T, G, "cuda", which=which)
        loss, _ = grpo.grpo_loss_fwd_bwd(lg, act, behave, torch.from_numpy(adv).cuda(), torch.from_numpy(sto).cuda(),
                                         torch.from_numpy(tso).cuda(), G, k=5.0, dual_clip_c=3.0,
                                         aux=aux if which else None)
        torch.cuda.synchronize()
        assert abs(loss.item() - ref.loss) <= LOSS_RTOL * np.abs(ref.token_contrib).sum()
        near = 2  # tokens whose fp64 ratio lies next to a boundary may fall either way
        if aux.clip_counts is not None:
            got = aux.clip_counts.cpu().numpy()
            assert abs(got[0] - (ref.token_state & 1).sum()) <= near
            assert abs(got[1] - ((ref.token_state >> 1) & 1).sum()) <= near
        if aux.ratio_stats is not None:
            got = aux.ratio_stats.cpu().numpy()
            np.testing.assert_allclose(got[:6], want[:6], rtol=1e-5)
            assert abs(got[6] - want[6]) <= near and got[7] == want[7] == T - G
