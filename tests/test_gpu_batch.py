"""Decode batches of independent requests (the batch-sweep configuration): the step-wise entry
points with B > 1 against the oracle applied request by request."""
import numpy as np
import pytest
import torch

import moei_inputs as mi
from oracle import moei_oracle as O
from tests.helpers import EPS, dev, pack_bank, rel_max_err, split_expert

pytestmark = pytest.mark.gpu

FFN_TOL_FP32ACC = 2e-4


@pytest.fixture(scope="module")
def m():
    import paper_2401_14361_amd as mod
    mod.lib()
    return mod


def _batch_case(m, cfg, n_unique, batches, cell_bytes=4):
    L, E, k = cfg.L, cfg.E, cfg.k
    T, _, _ = mi.eamc_traces(cfg, threads=8)
    bank = mi.expert_bank(cfg, n_unique, threads=8)
    shared = mi.expert_bank(cfg.scaled(cid=cfg.cid + 50), max(L * cfg.n_shared, 1), threads=2)
    routers = [mi.router_weights(cfg, l) for l in range(L)]
    desc = m.ModelDesc.from_config(cfg)
    eamc = m.Eamc(desc, cfg.N, cell_bytes)
    eamc.load(T)
    S = L * E
    cache = m.Cache(desc, S)
    packed, sh_packed = pack_bank(m, cfg, bank), pack_bank(m, cfg, shared)
    d_bank = [dev(packed[u]) for u in range(n_unique)]
    for s in range(S):
        t = cache.slot_tensor(s)
        t.copy_(d_bank[s % n_unique].view(t.dtype))
    for s in range(L * cfg.n_shared):
        t = cache.slot_tensor(S + s)
        t.copy_(dev(sh_packed[s]).view(t.dtype))
    cache.reset(S)
    slot_of = np.arange(S, dtype=np.int32)
    for B in batches:
        reqs = [mi.make_request(cfg, 100 + b, decode=1) for b in range(B)]
        eam = np.stack([r.prefill_eam for r in reqs]).astype(np.int32)
        d_eam = dev(eam)
        ref_eam = eam.astype(np.int64)
        for l in range(L):
            x = np.stack([r.x[0, l] for r in reqs])
            logits = np.stack([O.router_logits(routers[l], x[b], reqs[b].bias[l]) for b in range(B)]).astype(np.float32)
            idx, w = m.moe_route_topk(dev(logits), k, bool(cfg.renorm))
            ridx, rw = O.route_topk(logits, k, bool(cfg.renorm))
            assert (idx.cpu().numpy() == ridx).all()
            m.eam_update(d_eam, l, idx)
            for b in range(B):
                O.eam_update(ref_eam[b], l, ridx[b])
            assert (d_eam.cpu().numpy() == ref_eam).all()
            best, sim, _ = m.eamc_match(eamc, d_eam)
            rbest = [O.eamc_match(T, ref_eam[b])[0] for b in range(B)]
            assert best.cpu().numpy().tolist() == rbest
            out = m.expert_priority(eamc, best, l, cache.slot_table(), EPS, idx)
            P, V, pf, n_pf, ev, n_ev = [o.cpu().numpy() for o in out]
            excl = [l * E + int(j) for j in ridx.reshape(-1)]
            rP, rV, rpf, rev = O.expert_priority(O.aggregate_matches(T, rbest), l, slot_of.reshape(L, E) >= 0, EPS, excl)
            assert ev[:int(n_ev[0])].tolist() == rev and pf[:int(n_pf[0])].tolist() == rpf
            np.testing.assert_allclose(V, rV, rtol=1e-6)
            y = m.expert_ffn_grouped(cache, l, idx, w, dev(x)).cpu().numpy()
            for b in range(B):
                ex = [split_expert(cfg, bank[(l * E + int(j)) % n_unique]) for j in ridx[b]]
                ex += [split_expert(cfg, shared[l * cfg.n_shared + s]) for s in range(cfg.n_shared)]
                ref = O.expert_ffn(x[b], ex, list(rw[b]) + [1.0] * cfg.n_shared)
                assert rel_max_err(y[b], ref) <= FFN_TOL_FP32ACC, (B, l, b)
        assert cache.error_flags() == 0
    # deterministic: the same batch twice gives identical bits
    y2 = m.expert_ffn_grouped(cache, L - 1, idx, w, dev(x)).cpu().numpy()
    assert (y2 == y).all()
    # a pick that is not resident contributes nothing and is flagged
    cache.reset(0)
    m.expert_ffn_grouped(cache, 0, idx, w, dev(x))
    assert cache.error_flags() & 2
    eamc.close()
    cache.close()


def test_batch_sweep_on_the_deepseek_v2_lite_shape(m):
    # batch sizes 1..16 on the DeepSeek-V2-Lite shape (two of its layers carry weights here)
    cfg = mi.get_config("C5").scaled(L=2, N=400, prompt=64)
    _batch_case(m, cfg, 24, [1, 2, 4, 8, 16])


@pytest.mark.parametrize("wdtype,H,I", [("fp32", 256, 96), ("bf16", 1024, 72), ("bf16", 4096, 40), ("fp32", 1024, 130),
                                          ("fp32", 2048, 37), ("bf16", 2048, 3)])
def test_batched_ffn_other_shapes(m, wdtype, H, I):
    cfg = mi.get_config("C5").scaled(L=2, E=16, k=3, n_shared=1, N=60, prompt=16, H=H, I=I, wdtype=wdtype)
    _batch_case(m, cfg, 32, [3, 16])


def _kernels_of(m, call):
    """(what `call` returns, launches of the vector kernel, launches of the matrix kernel)"""
    m.profile_enable(8)
    out = call()
    prof = m.profile_read()
    m.profile_disable()
    return out, prof["ffn_fused_kernel"][0], prof["ffn_grouped_mm_kernel"][0]


def _ffn_only_case(m, cfg, B, idx, w, seed=3, matrix=None, resident=None):
    """expert_ffn_grouped on given picks against the oracle, token by token.  All experts are resident, or the first `resident`;
    `matrix`: whether the call is expected on the matrix cores."""
    L, E = cfg.L, cfg.E
    rng = np.random.default_rng(seed)
    n_unique = min(E, 40)
    bank = mi.expert_bank(cfg, n_unique, threads=8)
    shared = mi.expert_bank(cfg.scaled(cid=cfg.cid + 50), max(L * cfg.n_shared, 1), threads=2)
    desc = m.ModelDesc.from_config(cfg)
    S = L * E
    cache = m.Cache(desc, S)
    packed, sh_packed = pack_bank(m, cfg, bank), pack_bank(m, cfg, shared)
    d_bank = [dev(packed[u]) for u in range(n_unique)]
    for s in range(S):
        t = cache.slot_tensor(s)
        t.copy_(d_bank[s % n_unique].view(t.dtype))
    for s in range(L * cfg.n_shared):
        t = cache.slot_tensor(S + s)
        t.copy_(dev(sh_packed[s]).view(t.dtype))
    cache.reset(S if resident is None else resident)
    x = (rng.standard_normal((B, cfg.H)) * 0.5).astype(np.float32)
    xr = mi.f32_to_bf16_bits(x) if cfg.wdtype == "bf16" else x  # stored form: the oracle decodes it exactly
    xq = dev(xr)
    layer = L - 1
    y, n_vector, n_matrix = _kernels_of(m, lambda: m.expert_ffn_grouped(cache, layer, dev(idx.astype(np.int32)), dev(w.astype(np.float32)), xq))
    assert n_vector + n_matrix == 1 and (matrix is None or n_matrix == matrix)
    y = y.cpu().numpy()
    for b in range(B):
        ex, ws = [], []
        for j, wj in zip(idx[b], w[b]):
            if j >= 0 and (resident is None or layer * E + j < resident):
                ex.append(split_expert(cfg, bank[(layer * E + int(j)) % n_unique]))
                ws.append(float(wj))
        ex += [split_expert(cfg, shared[layer * cfg.n_shared + s]) for s in range(cfg.n_shared)]
        ref = O.expert_ffn(xr[b], ex, ws + [1.0] * cfg.n_shared)
        assert rel_max_err(y[b], ref) <= FFN_TOL_FP32ACC, b
    assert cache.error_flags() == (0 if resident is None else 2)
    cache.close()


def test_batched_ffn_token_without_picks_and_one_expert_for_all(m):
    # token 2 has no picks (what the routing kernels hand over when no softmax exists for its logits):
    # only the shared expert contributes; all other tokens route to the same experts, so these
    # experts' items are full and a fourth item of one token remains (13 = 3 x 4 + 1 tokens)
    cfg = mi.get_config("C5").scaled(L=2, E=16, k=3, n_shared=1, N=8, prompt=4, H=1024, I=50, wdtype="bf16")
    B = 14
    idx = np.tile(np.array([5, 0, 11]), (B, 1))
    idx[2] = -1
    w = np.random.default_rng(1).random((B, 3)) + 0.1
    w[2] = 0.0
    _ffn_only_case(m, cfg, B, idx, w)


def test_batched_ffn_at_the_item_builders_limits(m):
    # 256 experts, 16 tokens x 32 picks = 512 picks: every thread of the item builder holds two picks
    cfg = mi.get_config("C5").scaled(L=1, E=256, k=32, n_shared=0, N=4, prompt=4, H=512, I=6, wdtype="fp32")
    rng = np.random.default_rng(7)
    B = 16
    idx = np.stack([rng.permutation(256)[:32] for _ in range(B)])
    w = rng.random((B, 32)) + 0.05
    _ffn_only_case(m, cfg, B, idx, w)


# shares of the units in which an item's start weighs more than its units: one item over all workgroups, and
# many items of one unit; items that divide the workgroups, and items that do not
@pytest.mark.parametrize("E,k,n_shared,B,I", [(1, 1, 0, 1, 5), (1, 1, 0, 4, 130), (200, 4, 2, 16, 1),
                                              (8, 8, 0, 1, 70), (3, 3, 0, 2, 70)])
def test_batched_ffn_items_shorter_than_their_start(m, E, k, n_shared, B, I):
    cfg = mi.get_config("C5").scaled(L=1, E=E, k=k, n_shared=n_shared, H=512, I=I, N=8, prompt=16)
    rng = np.random.default_rng(E + I)
    idx = np.stack([rng.choice(E, size=k, replace=False) for _ in range(B)]).astype(np.int32)
    _ffn_only_case(m, cfg, B, idx, rng.random((B, k)).astype(np.float32))


def test_batched_ffn_rejects_more_experts_than_the_item_builder_takes(m):
    cfg = mi.get_config("C5").scaled(L=1, E=260, k=2, n_shared=0, N=4, prompt=4, H=256, I=4, wdtype="fp32")
    desc = m.ModelDesc.from_config(cfg)
    cache = m.Cache(desc, 260)
    cache.reset(260)
    idx, w = dev(np.zeros((2, 2), np.int32)), dev(np.ones((2, 2), np.float32))
    with pytest.raises(m.MoeiError):
        m.expert_ffn_grouped(cache, 0, idx, w, dev(np.zeros((2, 256), np.float32)))
    cache.close()


# items of up to 16 picks (the matrix kernel): every row width, units that are no whole number of blocks, fewer than a block for
# a workgroup and many blocks, batches of 4 to 16, a full list of picks and experts
@pytest.mark.parametrize("H,I,E,k,n_shared,B", [(512, 923, 2, 2, 0, 16), (512, 1100, 3, 3, 1, 5), (512, 8, 256, 32, 0, 16),
                                                (1024, 307, 4, 3, 1, 16), (1024, 4099, 2, 1, 0, 9), (2048, 250, 3, 2, 2, 13),
                                                (2048, 250, 2, 1, 0, 4), (4096, 133, 6, 5, 1, 7), (4096, 600, 3, 2, 0, 16)])
def test_batched_ffn_on_the_matrix_cores(m, H, I, E, k, n_shared, B):
    cfg = mi.get_config("C5").scaled(L=1, E=E, k=k, n_shared=n_shared, H=H, I=I, N=8, prompt=16)
    rng = np.random.default_rng(H + I)
    idx = np.stack([rng.choice(E, size=k, replace=False) for _ in range(B)]).astype(np.int32)
    if B > 8:
        idx[3] = -1  # a token without picks
    _ffn_only_case(m, cfg, B, idx, rng.random((B, k)).astype(np.float32), matrix=True)


# experts beyond the item builder's first wavefront of 64, in each of its four, the last of them not resident
@pytest.mark.parametrize("H,I,E,k,n_shared,B,resident", [(1024, 64, 200, 16, 2, 16, 150), (512, 40, 256, 32, 0, 16, 100), (2048, 24, 65, 9, 1, 13, 64),
                                                         (512, 130, 129, 20, 0, 7, 128)])
def test_batched_ffn_on_the_matrix_cores_many_experts(m, H, I, E, k, n_shared, B, resident):
    cfg = mi.get_config("C5").scaled(L=1, E=E, k=k, n_shared=n_shared, H=H, I=I, N=8, prompt=16)
    rng = np.random.default_rng(E + k)
    idx = np.stack([rng.choice(E, size=k, replace=False) for _ in range(B)]).astype(np.int32)
    idx[0, 0] = E - 1
    _ffn_only_case(m, cfg, B, idx, rng.random((B, k)).astype(np.float32), matrix=True, resident=resident)


def test_batched_ffn_on_the_matrix_cores_infinite_weights_and_unaligned_inputs(m):
    # an infinite weight of the down projection reaches the tokens of its expert as an infinity, in the last unit of an expert
    # of 181 (a block of fewer than 16), and no other token; an expert that is not resident contributes nothing
    L, E, k, H, I, B = 1, 4, 2, 1024, 181, 12
    desc = m.ModelDesc(L, E, k, 0, H, I, m.WDTYPE_BF16, 0, EPS)
    cache = m.Cache(desc, E)
    cache.reset(E - 1)  # expert 3 has no slot
    g = torch.Generator(device="cuda").manual_seed(5)
    bank = (torch.randn((E, I, 3, H), generator=g, device="cuda") * 0.05).bfloat16()
    bank[1, I - 1, 2, 100] = float("inf")
    for e in range(E):
        cache.slot_tensor(e).copy_(bank[e].reshape(-1))
    room = torch.randn(B * H + 8, generator=g, device="cuda").bfloat16()
    x = room[1:1 + B * H].view(B, H)  # 2 bytes past a 16-byte boundary
    idx = torch.tensor([[0, 2] if b % 3 == 0 else ([1, 0] if b % 3 == 1 else [2, 3]) for b in range(B)], dtype=torch.int32, device="cuda")
    w = torch.rand((B, k), generator=g, device="cuda") + 0.1
    y, _, n_matrix = _kernels_of(m, lambda: m.expert_ffn_grouped(cache, 0, idx, w, x))
    assert n_matrix == 1
    y = y.double()
    ref = torch.zeros_like(y)
    for b in range(B):
        for j in range(k):
            e = int(idx[b, j])
            if e < 3:
                W = bank[e].double()
                a = torch.nn.functional.silu(W[:, 0] @ x[b].double()) * (W[:, 1] @ x[b].double()) * w[b, j].double()
                ref[b] += a @ W[:, 2]
    inf = torch.isinf(ref)
    assert inf.sum() == 4 and (y[inf] == ref[inf]).all()
    assert ((y - ref)[~inf].abs().max() / ref[~inf].abs().max()) <= FFN_TOL_FP32ACC
    assert cache.error_flags() & 2
    cache.close()


# a token that lists an expert twice (or more often) gets its output with each of the weights: in one item, in several, and beside
# tokens that list it once; on both kernels (3 requests and fp32 weights: the vector kernel)
@pytest.mark.parametrize("wdtype,H,I,B,matrix", [("bf16", 4096, 600, 8, True), ("bf16", 1024, 400, 16, True), ("bf16", 4096, 40, 3, False),
                                                 ("bf16", 512, 60, 3, False), ("fp32", 256, 50, 16, False)])
def test_batched_ffn_with_an_expert_listed_twice(m, wdtype, H, I, B, matrix):
    cfg = mi.get_config("C5").scaled(L=1, E=4, k=4, n_shared=1, H=H, I=I, N=8, prompt=16, wdtype=wdtype)
    rng = np.random.default_rng(H + B)
    idx = np.stack([rng.permutation(4) for _ in range(B)])
    idx[0] = [2, 1, 2, 0]
    idx[1] = 3
    idx[B - 1] = [1, 1, 0, 0]
    _ffn_only_case(m, cfg, B, idx, rng.random((B, 4)) + 0.1, matrix=matrix)


# scratch of the first call: rows of 16 tokens only where a batch of the model can take the matrix kernel (not where none saves
# enough, and not for rows that the call refuses)
@pytest.mark.parametrize("H,I,taken", [(4096, 16, True), (5120, 600, False)])
def test_batched_ffn_scratch_is_what_its_calls_take(m, H, I, taken):
    E, k, B = 64, 2, 16
    desc = m.ModelDesc(1, E, k, 0, H, I, m.WDTYPE_BF16, 0, EPS)
    caches = [m.Cache(desc, E) for _ in range(2)]
    idx, w = dev(np.tile(np.arange(k, dtype=np.int32), (B, 1))), dev(np.ones((B, k), np.float32))
    x = dev(np.zeros((B, H), dtype=np.uint16))
    free = []
    for cache in caches:  # the first one's call loads the code
        cache.reset(E)
        if taken:
            m.expert_ffn_grouped(cache, 0, idx, w, x)
        else:
            with pytest.raises(m.MoeiError):
                m.expert_ffn_grouped(cache, 0, idx, w, x)
        torch.cuda.synchronize()
        free.append(torch.cuda.mem_get_info()[0])
    units = torch.cuda.get_device_properties(0).multi_processor_count
    assert free[0] - free[1] <= units * 2 * 4 * H * 4 + (4 << 20), (free[0] - free[1]) / 2**20
    for cache in caches:
        cache.close()
