"""GPU parity of the row kernels on rows that are not whole 16-byte vectors: odd vocabularies, strides and base
addresses, at the sizes where the split into edge elements and vectors changes kernel or leaves one of them empty.

The gates are those of tests/gpu_parity.py; bf16 dlogits are held to one rounding of an fp32 value,
2^-8 |ref| + 1e-5 max_row |ref|, whatever the row length (these rows form dlogits in fp32 throughout).
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_05597_amd as grpo
from synth.rollouts import Config, make_structure
from tests.gpu_parity import LOGP_ATOL, LOSS_RTOL, dl_to_f64, gpu_norm, to_np_logits

pytestmark = pytest.mark.gpu


def _batch(V, ld, dtype, offset, T=40, seed=3):
    """T rows of V logits, ld apart, the first `offset` elements past an aligned address; actions in the first and
    last columns, next to the first boundary, and anywhere."""
    cfg = Config("ragged", 1, 4, V, "f32", 2.0, 0.5, (2, 3), (2, 3), 4.0, (1, 64), 0.1, 4.0, seed=seed)
    st = make_structure(cfg, seed, T)
    g = torch.Generator("cuda").manual_seed(seed)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    store = torch.zeros(T * ld + 32, dtype=dt, device="cuda")
    lg = store[offset:offset + T * ld].view(T, ld)
    lg[:, :V] = (2.0 * torch.randn((T, V), generator=g, device="cuda")).to(dt)
    act = torch.randint(0, V, (T,), generator=g, device="cuda", dtype=torch.int32)
    for i, a in enumerate([0, V - 1, 1, V - 2, 7, 8, V - 8, V - 9]):
        act[i] = min(max(a, 0), V - 1)
    z = lg[:, :V].float()
    lp = z.gather(1, act.long()[:, None])[:, 0] - torch.logsumexp(z, 1)
    behave = lp + 0.05 * torch.randn(T, generator=g, device="cuda")
    adv = oracle.advantages(st.rewards, cfg.G).astype(np.float32)
    return cfg, st, lg, act, behave, adv


def _loss(cfg, st, lg, act, behave, adv, V, dl, gs):
    aux = grpo.LossAux.alloc(len(act), len(st.rewards), "cuda", which=("token_logp", "error_flags"))
    loss, _ = grpo.grpo_loss_fwd_bwd(lg, act, behave, torch.from_numpy(adv).cuda(),
                                     torch.from_numpy(st.step_tok_off).cuda(),
                                     torch.from_numpy(st.traj_step_off).cuda(), cfg.G, V=V,
                                     norm=gpu_norm(oracle.NORM_CONST_K), k=cfg.k, dual_clip_c=3.0, grad_scale=gs,
                                     dlogits=dl, aux=aux)
    torch.cuda.synchronize()
    return loss.item(), aux


# bf16: below a vector, the resident variants' ends (64 x 1 and 256 x 4 vectors and one more), the persistent kernel's
# first and last sizes and one between two of its vector counts, a padded head, past it (the streaming kernel); fp32
# rows, in the loss element by element, staged in LDS (up to 20,224 elements) or not; bf16 beyond 4 MiB (two passes)
SIZES = [(1, 1, "bf16"), (7, 7, "bf16"), (8, 9, "bf16"), (519, 519, "bf16"), (8199, 8201, "bf16"), (32003, 32003, "bf16"),
         (49159, 49159, "bf16"), (49161, 49162, "bf16"), (57353, 57353, "bf16"), (81927, 81927, "bf16"),
         (81929, 81929, "bf16"), (151669, 151936, "bf16"),
         (188423, 188423, "bf16"), (188431, 188431, "bf16"), (3, 3, "f32"), (259, 261, "f32"), (4093, 4093, "f32"),
         (77825, 77825, "f32"), (77831, 77832, "f32"), (20223, 20223, "f32"), (20225, 20225, "f32"),
         (151669, 151936, "f32"), (2097159, 2097159, "bf16"), (2097161, 2097161, "bf16")]


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("V,ld,dtype", SIZES)
def test_loss_rows(V, ld, dtype, offset):
    cfg, st, lg, act, behave, adv = _batch(V, ld, dtype, offset)
    T = len(act)
    seg = oracle.segments(st.T, st.step_tok_off, st.traj_step_off)
    ref = oracle.loss_rows(to_np_logits(lg[:, :V].contiguous()), act.cpu().numpy(), behave.cpu().numpy(), None,
                           adv.astype(np.float64), seg, cfg.G, norm=oracle.NORM_CONST_K, k=cfg.k, dual_clip_c=3.0)
    gs = float(np.float32(1.0 / np.abs(ref.token_g).max()))
    rel = 2.0 ** -8 if dtype == "bf16" else 0.0
    for shift in (offset, offset + 1):  # dlogits at the logits' distance from a boundary, then at another
        dl = torch.full((T * ld + 32,), 7.0, dtype=lg.dtype, device="cuda")[shift:shift + T * ld].view(T, ld)
        loss, aux = _loss(cfg, st, lg, act, behave, adv, V, dl, gs)
        assert abs(loss - ref.loss) <= LOSS_RTOL * np.abs(ref.token_contrib).sum()
        assert np.abs(aux.token_logp.cpu().numpy() - ref.token_logp).max() <= LOGP_ATOL
        assert aux.error_flags.item() == 0
        r = ref.dlogits * gs
        # the fp32 log2 in a row's log-sum-exp is good to about 2e-7 and |g| <= 1 here: all there is at V = 1
        bound = rel * np.abs(r) + 1e-5 * np.abs(r).max(axis=1, keepdims=True) + 4e-7
        err = np.abs(dl_to_f64(dl[:, :V]) - r)
        assert (err <= bound).all(), (shift, float((err - bound).max()))
        assert (dl[:, V:] == 7.0).all()  # columns past V are left alone


@pytest.mark.parametrize("V,T,dtype", [(57353, 300, "bf16"), (81929, 600, "bf16"), (90121, 1200, "bf16"), (188435, 600, "bf16"), (188440, 600, "bf16"),
                                       (77832, 600, "f32"), (77831, 300, "f32")])
def test_dlogits_over_the_logits(V, T, dtype):
    # bf16: several rows per workgroup, edges and vector counts changing from row to row; fp32: the kernel that reads a
    # row twice, and element by element; dlogits over the logits
    cfg, st, lg, act, behave, adv = _batch(V, V, dtype, 0 if V % 8 == 0 else 3, T=T, seed=8)
    before = lg.clone()
    seg = oracle.segments(st.T, st.step_tok_off, st.traj_step_off)
    ref = oracle.loss_rows(to_np_logits(before), act.cpu().numpy(), behave.cpu().numpy(), None,
                           adv.astype(np.float64), seg, cfg.G, norm=oracle.NORM_CONST_K, k=cfg.k, dual_clip_c=3.0)
    gs = float(np.float32(1.0 / np.abs(ref.token_g).max()))
    loss, aux = _loss(cfg, st, lg, act, behave, adv, V, lg, gs)
    assert abs(loss - ref.loss) <= LOSS_RTOL * np.abs(ref.token_contrib).sum()
    r = ref.dlogits * gs
    err = np.abs(dl_to_f64(lg) - r)
    assert (err <= (2.0 ** -8 if dtype == "bf16" else 0.0) * np.abs(r) + 1e-5 * np.abs(r).max(axis=1, keepdims=True)).all()


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("V,ld,dtype", SIZES)
def test_logp_and_records(V, ld, dtype, offset):
    _, _, lg, act, _, _ = _batch(V, ld, dtype, offset)
    ref = oracle.logp_entropy(to_np_logits(lg[:, :V].contiguous()), act.cpu().numpy())
    for entropy in (True, False):
        logp, ent = grpo.grpo_token_logp(lg, act, V=V, entropy=entropy)
        assert np.abs(logp.double().cpu().numpy() - ref.token_logp).max() <= LOGP_ATOL
        if entropy:
            assert (np.abs(ent.double().cpu().numpy() - ref.token_entropy)
                    <= 2e-5 + 2e-5 * np.abs(ref.token_entropy)).all()
    stats = grpo.grpo_vocab_shard_stats(lg, act, 0, V=V)
    m, za, s = (x.cpu().numpy() for x in grpo.vocab_stats_fields(stats))
    want = oracle.vocab_shard_stats(to_np_logits(lg[:, :V].contiguous()), act.cpu().numpy(), 0)
    np.testing.assert_array_equal(m, want.m)
    np.testing.assert_array_equal(za, want.za)
    np.testing.assert_allclose(s, want.s, rtol=5e-6)


@pytest.mark.parametrize("mask,left", [(None, 300), (None, 100), (None, 1), (-1e8, 100), (-1e9, 100), (-1e10, 100),
                                       (-1e30, 1), (-1e38, 100), (-2.3819763e38, 100)])
@pytest.mark.parametrize("V,ld,dtype", [(1003, 1003, "bf16"), (1003, 1003, "f32"), (32003, 32003, "bf16"),
                                        (57353, 57353, "bf16"), (77831, 77831, "f32"), (1000, 1000, "bf16"),
                                        (1000, 1000, "f32"), (1004, 1004, "f32"), (131, 131, "f32"),
                                        (20225, 20225, "f32"), (77832, 77832, "f32"), (151936, 151936, "bf16"),
                                        (188440, 188440, "bf16")])
def test_logits_masked_with_the_lowest_value(V, ld, dtype, mask, left):
    # all but the last `left` columns at the type's lowest value or another large negative one, as masks often are: they
    # carry no probability.  With fewer columns left than a row's kernel has threads, some thread's whole share of the
    # row is masked.  dlogits at the logits' distance from a 16-byte boundary and at another (the kernel that takes rows
    # element by element)
    left = min(left, V - 30)
    cfg, st, lg, act, behave, adv = _batch(V, ld, dtype, 0)
    lg[:, :V - left] = torch.finfo(lg.dtype).min if mask is None else mask
    act = act % left + (V - left)
    z = lg[:, V - left:V].double()
    lse = torch.logsumexp(z, 1)
    want = z.gather(1, (act.long() - (V - left))[:, None])[:, 0] - lse
    logp, ent = grpo.grpo_token_logp(lg, act, V=V)
    assert (logp.double() - want).abs().max().item() <= LOGP_ATOL
    p = torch.exp(z - lse[:, None])
    assert (ent.double() + (p * (z - lse[:, None])).sum(1)).abs().max().item() <= 4e-4
    T = len(act)
    for shift in (0, 1):
        dl = torch.full((T * ld + 32,), 7.0, dtype=lg.dtype, device="cuda")[shift:shift + T * ld].view(T, ld)
        _, aux = _loss(cfg, st, lg, act, want.float(), adv, V, dl, 1.0)
        assert (aux.token_logp.double() - want).abs().max().item() <= LOGP_ATOL and aux.error_flags.item() == 0
        assert (dl[:, :V - left] == 0).all() and torch.isfinite(dl).all()


@pytest.mark.parametrize("V,ld,T,dtype", [(188440, 188440, 128, "bf16"), (188440, 188440, 129, "bf16"),
                                          (188443, 188443, 129, "bf16"), (77828, 77828, 400, "f32"),
                                          (131076, 131076, 384, "f32"), (131076, 131076, 385, "f32"),
                                          (151936, 151936, 40, "bf16"), (65536, 65536, 40, "bf16"),
                                          (32003, 32003, 40, "f32")])
def test_loss_alone(V, ld, T, dtype):
    # no dlogits: every row kernel, and on both sides of the number of rows (on 256 CUs) from which long rows are read
    # once by their record pass
    cfg, st, lg, act, behave, adv = _batch(V, ld, dtype, 0, T=T)
    z = lg[:, :V].double()
    want = z.gather(1, act.long()[:, None])[:, 0] - torch.logsumexp(z, 1)
    loss, aux = _loss(cfg, st, lg, act, behave, adv, V, False, 1.0)
    assert (aux.token_logp.double() - want).abs().max().item() <= LOGP_ATOL and aux.error_flags.item() == 0
    both, aux2 = _loss(cfg, st, lg, act, behave, adv, V, torch.empty_like(lg), 1.0)
    assert abs(loss - both) <= LOSS_RTOL * abs(both)
    assert (aux.token_logp - aux2.token_logp).abs().max().item() <= LOGP_ATOL


def test_fp32_rows_of_more_than_8_mb():
    # on 256 CUs 384 such rows are read by the kernel that holds a part of them, 385 in two passes, to the same bits (the
    # constant normaliser gives every token the same weight in both)
    V, T = 2097156, 385
    cfg, st, lg, act, behave, adv = _batch(V, V, "f32", 0, T=T)
    got = []
    for t in (T, T - 1):
        st.step_tok_off[-1] = t
        dl = torch.empty_like(lg[:t])
        _, aux = _loss(cfg, st, lg[:t], act[:t], behave[:t], adv, V, dl, 1.0)
        assert aux.error_flags.item() == 0
        got.append((dl, aux.token_logp))
    assert torch.equal(got[0][0][:T - 1], got[1][0]) and torch.equal(got[0][1][:T - 1], got[1][1])
    p = torch.softmax(lg[T - 1].double(), 0)
    p[act[T - 1].item()] -= 1
    d = got[0][0][T - 1].double()
    g = d[act[T - 1].item()] / p[act[T - 1].item()]
    assert (d - g * p).abs().max().item() <= 1e-5 * d.abs().max().item()


# the element kernel's rows of 1, 4 and 8 elements a thread held in registers and the first beyond; the log-probs' rows of
# one wave (8 KB) and the first beyond
SHORT = [(255, 255, "f32"), (256, 257, "bf16"), (257, 257, "f32"), (1023, 1023, "bf16"), (1024, 1025, "f32"),
         (1025, 1025, "f32"), (2047, 2047, "f32"), (2048, 2049, "f32"), (2049, 2049, "f32"), (2049, 2049, "bf16"),
         (4096, 4097, "bf16"), (4097, 4097, "bf16")]


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("V,ld,dtype", SHORT)
def test_short_rows(V, ld, dtype, offset):
    test_loss_rows(V, ld, dtype, offset)
    test_logp_and_records(V, ld, dtype, offset)
    test_logits_masked_with_the_lowest_value(V, ld, dtype, None, 100)


@pytest.mark.parametrize("V,dtype", [(1, "f32"), (64, "bf16"), (101, "f32"), (1003, "bf16"), (32000, "bf16"), (32003, "f32"),
                                     (57353, "bf16"), (77828, "f32"), (151936, "bf16"), (188440, "bf16"), (200003, "bf16"),
                                     (2097160, "bf16")])
@pytest.mark.parametrize("mask", [None, -1e9])
def test_rows_masked_throughout(V, dtype, mask):
    # every third row holds the mask alone: log-prob -inf, no gradient, the flag; the other rows as without them
    cfg, st, lg, act, behave, adv = _batch(V, V, dtype, 0)
    T = len(act)
    clean = torch.empty_like(lg)
    _, ref = _loss(cfg, st, lg, act, behave, adv, V, clean, 1.0)
    lg[::3] = torch.finfo(lg.dtype).min if mask is None else mask
    rest = torch.arange(T, device="cuda") % 3 != 0
    for shift in (0, 1):
        dl = torch.full((T * V + 16,), 7.0, dtype=lg.dtype, device="cuda")[shift:shift + T * V].view(T, V)
        loss, aux = _loss(cfg, st, lg, act, behave, adv, V, dl, 1.0)
        assert np.isfinite(loss) and aux.error_flags.item() == grpo.GRPO_FLAG_NONFINITE
        assert (aux.token_logp[::3] == -np.inf).all() and (dl[::3] == 0).all()
        assert (aux.token_logp[rest] - ref.token_logp[rest]).abs().max().item() <= LOGP_ATOL
        if shift == 0:
            assert torch.equal(dl[rest], clean[rest])
    _, alone = _loss(cfg, st, lg, act, behave, adv, V, False, 1.0)
    assert (alone.token_logp[::3] == -np.inf).all() and torch.isfinite(alone.token_logp[rest]).all()
    logp, _ = grpo.grpo_token_logp(lg, act)
    assert (logp[::3] == -np.inf).all() and torch.isfinite(logp[rest]).all()
