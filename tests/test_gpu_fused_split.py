"""The token-blocked fused path on few rows, where the dhidden product runs in ranges of the vocabulary whose fp32
partials are summed afterwards: a last range that is short, one that ends inside a 64-deep slab, H not a multiple of the
tile, several blocks on one and on two streams (the partials lie in the block's own terms).  The oracle and the gates
are those of tests/test_gpu_fused.py."""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_05597_amd as grpo
from oracle import fused
from tests.gpu_parity import check_fused_loss, gpu_norm
from tests.test_gpu_fused import bits, check_dh, check_dw
from tests.test_gpu_fused_edges import edge_batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,H,V,block,streams", [(1, 64, 20000, 8192, 1), (130, 64, 20000, 8192, 1),
                                                 (300, 192, 8200, 8192, 1), (600, 192, 8200, 256, 1),
                                                 (600, 192, 8200, 256, 2), (513, 320, 4104, 512, 2)])
def test_split_dhidden(T, H, V, block, streams):
    e = edge_batch(T, H, V, seed=T + H + V)
    A32 = oracle.advantages(e["rewards"], e["G"]).astype(np.float32)
    seg = oracle.segments(T, e["sto"], e["tso"])
    ref = fused.fused_loss(bits(e["hidden"]), bits(e["W"]), e["actions"], e["behave"], None, A32.astype(np.float64),
                           seg, e["G"], norm=oracle.NORM_CONST_K, k=4.0, dual_clip_c=3.0)
    dw0 = torch.randn((H, V), device="cuda", generator=torch.Generator("cuda").manual_seed(9)) * 1e-3
    loss, dh, dW = grpo.fused_lmhead_grpo_blocked(
        e["hidden"], e["W"], torch.from_numpy(e["actions"]).cuda(), torch.from_numpy(e["behave"]).cuda(),
        torch.from_numpy(A32).cuda(), torch.from_numpy(e["sto"]).cuda(), torch.from_numpy(e["tso"]).cuda(), e["G"],
        token_block=block, norm=gpu_norm(oracle.NORM_CONST_K), k=4.0, dual_clip_c=3.0, dw_lm=dw0.clone(),
        accumulate_dw=True, aux_stream=torch.cuda.Stream() if streams == 2 else None)
    torch.cuda.synchronize()
    check_fused_loss(loss.item(), ref.rows.token_contrib, "loss")
    W64, h64 = fused.as_f64(bits(e["W"])), fused.as_f64(bits(e["hidden"]))
    check_dh(dh.float().cpu().numpy().astype(np.float64), ref.dhidden, ref.rows.dlogits, W64)
    got = dW.cpu().numpy().astype(np.float64) - dw0.cpu().numpy().astype(np.float64)
    # the product's own bound, the rounding of fp16 terms below 2^-14 (2^-25 of |g|: at V = 20,000 many are) and one
    # fp32 rounding of dw0 + dW
    D = np.abs(ref.rows.dlogits) + 2.0 ** -18 * np.abs(ref.rows.token_g)[:, None]
    bound = 2.0 ** -7 * (np.abs(h64).T @ D) + 2.0 ** -23 * np.abs(dw0.cpu().numpy())
    err = np.abs(got - ref.dW)
    assert (err <= bound + 1e-30).all(), float((err / (bound + 1e-30)).max())


@pytest.mark.parametrize("T,H,V,c", [(70, 64, 4104, 4096), (300, 320, 2504, 1024), (600, 64, 520, 256), (2500, 128, 600, 256)])
def test_shard_and_chunked_launches(T, H, V, c):
    # one shard that is the whole vocabulary, its logits kept: a split dhidden (few rows), whole tiles of either product
    # first; and the chunked schedule with the columns of a pair longer or shorter than the rows
    e = edge_batch(T, H, V, seed=T + H + V)
    A32 = oracle.advantages(e["rewards"], e["G"]).astype(np.float32)
    seg = oracle.segments(T, e["sto"], e["tso"])
    ref = fused.fused_loss(bits(e["hidden"]), bits(e["W"]), e["actions"], e["behave"], None, A32.astype(np.float64),
                           seg, e["G"], norm=oracle.NORM_CONST_K, k=4.0, dual_clip_c=3.0)
    act = torch.from_numpy(e["actions"]).cuda()
    args = (act, torch.from_numpy(e["behave"]).cuda(), torch.from_numpy(A32).cuda(), torch.from_numpy(e["sto"]).cuda(),
            torch.from_numpy(e["tso"]).cuda(), e["G"])
    kw = dict(norm=gpu_norm(oracle.NORM_CONST_K), k=4.0, dual_clip_c=3.0)
    kept = grpo.vocab_shard_logits_buffer(T, V, "cuda")
    stats = grpo.fused_lmhead_vocab_shard_stats(e["hidden"], e["W"], act, 0, logits_out=kept)
    runs = {"shard": grpo.fused_lmhead_grpo_vocab_shard(e["hidden"], e["W"], stats[None], 0, V, *args, logits_in=kept,
                                                        **kw),
            "chunked": grpo.fused_lmhead_grpo(e["hidden"], e["W"], *args, vocab_chunk=c, **kw)}
    torch.cuda.synchronize()
    W64, h64 = fused.as_f64(bits(e["W"])), fused.as_f64(bits(e["hidden"]))
    for name, (loss, dh, dW) in runs.items():
        check_fused_loss(loss.item(), ref.rows.token_contrib, name)
        check_dh(dh.float().cpu().numpy().astype(np.float64), ref.dhidden, ref.rows.dlogits, W64, name)
        check_dw(dW.cpu().numpy().astype(np.float64), ref.dW, h64, ref.rows.dlogits, name)


@pytest.mark.parametrize("T,H,V", [(1, 2048, 32), (257, 2048, 1056), (40, 2112, 520)])
def test_forward_only_packed(T, H, V):
    # W^T packed (V a multiple of 32) and not, at a long K
    e = edge_batch(T, H, V, seed=T + V)
    ref = oracle.logp_entropy(e["z"], e["actions"])
    for entropy in (True, False):
        logp, ent = grpo.fused_lmhead_token_logp(e["hidden"], e["W"], torch.from_numpy(e["actions"]).cuda(), entropy=entropy)
        # z has a standard deviation of 0.25 sqrt(H) = 11 here: the fp32 product's error grows with it, as the logits do
        assert np.abs(logp.double().cpu().numpy() - ref.token_logp).max() <= 2e-4
        if entropy:
            assert (np.abs(ent.double().cpu().numpy() - ref.token_entropy) <= 4e-4 + 2e-5 * np.abs(ref.token_entropy)).all()


@pytest.mark.parametrize("T,H,V,block,streams", [(4095, 64, 600, 8192, 1), (4096, 64, 600, 8192, 1),
                                                 (4099, 320, 1032, 2048, 1), (4099, 320, 1032, 2048, 2)])
def test_packed_w_where_its_rows_are_not_whole_lines(T, H, V, block, streams):
    # whole dhidden tiles on the packed W from 4,096 rows on where V is not a multiple of 64, a short last block among them
    test_split_dhidden(T, H, V, block, streams)


@pytest.mark.parametrize("T,V", [(40, 520), (128, 520), (129, 520), (40, 528)])
def test_dw_stores_of_few_rows(T, V):
    # dW written and not added to: through the L2 where its rows are not multiples of 64 bytes and K is at most 128
    H = 320
    e = edge_batch(T, H, V, seed=T + V)
    A32 = oracle.advantages(e["rewards"], e["G"]).astype(np.float32)
    seg = oracle.segments(T, e["sto"], e["tso"])
    ref = fused.fused_loss(bits(e["hidden"]), bits(e["W"]), e["actions"], e["behave"], None, A32.astype(np.float64),
                           seg, e["G"], norm=oracle.NORM_CONST_K, k=4.0, dual_clip_c=3.0)
    store = torch.full((H * V + 256,), 7.0, device="cuda")
    grpo.fused_lmhead_grpo_blocked(
        e["hidden"], e["W"], torch.from_numpy(e["actions"]).cuda(), torch.from_numpy(e["behave"]).cuda(),
        torch.from_numpy(A32).cuda(), torch.from_numpy(e["sto"]).cuda(), torch.from_numpy(e["tso"]).cuda(), e["G"],
        norm=gpu_norm(oracle.NORM_CONST_K), k=4.0, dual_clip_c=3.0, dw_lm=store[:H * V].view(H, V))
    assert (store[H * V:] == 7.0).all()
    h64 = fused.as_f64(bits(e["hidden"]))
    check_dw(store[:H * V].view(H, V).cpu().numpy().astype(np.float64), ref.dW, h64, ref.rows.dlogits)
