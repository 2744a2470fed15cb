"""The decode-step kernel at the edges of its tiles and of its dispatch: attended counts around
the 16 tokens of a wavefront step and the step of a workgroup, every group size, both
workgroup widths (8 head-problems: eight wavefronts, 512: four), and selections whose candidates just fit
or just exceed one wavefront."""
import numpy as np
import pytest
import torch

import paper_2412_03213_amd as ck
from oracle import clusterkv_oracle as O

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# bf16 output: 8 significant bits, so half an ulp is at most 2^-8 of the value's power of two;
# products are exact in fp32 and the probabilities keep 24 bits, so sums and exponentials add
# less than another 2^-12
TOL = 2.0 ** -8 + 2.0 ** -12


def np64(t):
    return t.detach().float().cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("S,G", [(1, 1), (1, 2), (1, 4), (1, 8), (64, 1), (64, 4)])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 257, 1025])
def test_attention_at_tile_edges(S, G, n):
    Hkv, N, n_sink, n_rec = 8, 1600, 3, 5
    g = torch.Generator(device=DEV).manual_seed(100 * n + G)
    K = torch.randn(S, Hkv, N, 128, generator=g, device=DEV).bfloat16()
    V = torch.randn(S, Hkv, N, 128, generator=g, device=DEV).bfloat16()
    q = (3 * torch.randn(S, Hkv * G, 128, generator=g, device=DEV)).bfloat16()
    stride = (n + 3) // 4 * 4
    idx = (torch.rand(S, Hkv, N - n_sink - n_rec, generator=g, device=DEV).topk(stride).indices
           + n_sink).int()
    cnt = torch.full((S, Hkv), n, dtype=torch.int32, device=DEV)
    cnt[0, 1] = 0                                         # sinks and recent tokens only
    sh = ck.Shape(S, Hkv * G, Hkv, N, 8)
    out = torch.full((S, Hkv * G, 128), float("nan"), device=DEV).bfloat16()
    ck.ck_sparse_decode_attn(sh, q, K, V, idx, cnt, n, out, n_sink=n_sink, recent_begin=N - n_rec,
                             recent_end=N)
    for s, h in [(0, 0), (0, 1), (S - 1, Hkv - 1)]:
        rows = np.concatenate([np.arange(n_sink), idx[s, h, :int(cnt[s, h])].cpu().numpy(),
                               np.arange(N - n_rec, N)])
        want = O.attention_over(np64(q[s, h * G:(h + 1) * G]), np64(K[s, h]), np64(V[s, h]), rows)
        got = np64(out[s, h * G:(h + 1) * G])
        assert np.abs(got - want).max() <= TOL * np.abs(want).max(), (s, h)


@pytest.mark.parametrize("S", [1, 64])
@pytest.mark.parametrize("C,equal", [(1, False), (63, True), (64, True), (65, True), (64, False),
                                     (130, False), (512, True), (512, False), (513, False),
                                     (700, True)])
@pytest.mark.parametrize("budget,flags", [(1, 0), (77, 0), (77, 1), (600, 0), (600, 1), (5000, 1)])
def test_selection_at_the_candidate_limit(S, C, equal, budget, flags):
    Hkv, G, N = 8, 2, 1400
    rng = np.random.default_rng(C * 7 + budget)
    g = torch.Generator(device=DEV).manual_seed(C + budget)
    sh = ck.Shape(S, Hkv * G, Hkv, N, C)
    st = ck.ClusterState(sh, DEV, budget=budget)
    st.n_clusters = C
    mu = torch.randn(S, Hkv, C, 128, generator=g, device=DEV).bfloat16()
    if equal:                                             # every cluster scores the same: ties by id
        mu[:] = mu[:, :, :1]
    st.centroids.copy_(mu)
    sizes = rng.multinomial(N, rng.dirichlet(np.full(C, 0.3)), size=(S, Hkv)).astype(np.int32)
    offs = np.zeros((S, Hkv, C + 1), np.int32)
    offs[:, :, 1:] = sizes.cumsum(-1)
    sidx = np.stack([rng.permutation(N) for _ in range(S * Hkv)]).reshape(S, Hkv, N).astype(np.int32)
    st.sizes.copy_(torch.from_numpy(sizes))
    st.offsets.copy_(torch.from_numpy(offs))
    st.sorted_idx.copy_(torch.from_numpy(sidx))
    K = torch.randn(S, Hkv, N, 128, generator=g, device=DEV).bfloat16()
    V = torch.randn(S, Hkv, N, 128, generator=g, device=DEV).bfloat16()
    q = torch.randn(S, Hkv * G, 128, generator=g, device=DEV).bfloat16()
    out = ck.decode_step(st, q, K, V, flags=flags).clone()
    three = ck.ClusterState(sh, DEV, budget=budget)
    for name in ("centroids", "sizes", "offsets", "sorted_idx"):
        getattr(three, name).copy_(getattr(st, name))
    three.n_clusters = C
    assert torch.equal(out, ck.decode_step(three, q, K, V, flags=flags, fused=False))
    mode = O.TRIM_LAST if flags else O.WHOLE
    for s, h in [(0, 0), (S - 1, Hkv - 1)]:
        scores = st.scores[s, h].double().cpu().numpy()
        # from the step's own scores, so that nothing is a near-tie
        order, n_sel, n_tok = O.select_clusters(scores, sizes[s, h], budget, mode)
        assert int(st.n_sel_clusters[s, h]) == n_sel
        assert int(st.n_sel_tokens[s, h]) == int(st.n_tokens[s, h]) == n_tok
        assert np.array_equal(st.sel_clusters[s, h, :n_sel].cpu().numpy(), order[:n_sel])
        rows = O.gather_indices(order, n_sel, offs[s, h], sidx[s, h], budget, mode)
        assert np.array_equal(st.token_idx[s, h, :n_tok].cpu().numpy(), rows)
        want = O.attention_over(np64(q[s, h * G:(h + 1) * G]), np64(K[s, h]), np64(V[s, h]), rows)
        got = np64(out[s, h * G:(h + 1) * G])
        assert np.abs(got - want).max() <= TOL * max(np.abs(want).max(), 1e-30)


@pytest.mark.parametrize("S", [1, 64])
@pytest.mark.parametrize("G", [1, 4, 8])
def test_infinite_values_and_unattended_rows(S, G):
    """An infinite value makes its channel infinite (not NaN: parts of a probability are zero),
    and row 0, which stands in for positions beyond the end, is not looked at."""
    Hkv, N, n = 8, 300, 37
    g = torch.Generator(device=DEV).manual_seed(G)
    K = torch.randn(S, Hkv, N, 128, generator=g, device=DEV).bfloat16()
    V = torch.randn(S, Hkv, N, 128, generator=g, device=DEV).bfloat16()
    q = torch.zeros(S, Hkv * G, 128, device=DEV).bfloat16()   # all probabilities exactly 2^0
    idx = (torch.rand(S, Hkv, N - 1, generator=g, device=DEV).topk(40).indices + 1).int()
    cnt = torch.full((S, Hkv), n, dtype=torch.int32, device=DEV)
    sh = ck.Shape(S, Hkv * G, Hkv, N, 8)
    out = torch.zeros(S, Hkv * G, 128, device=DEV).bfloat16()
    ck.ck_sparse_decode_attn(sh, q, K, V, idx, cnt, n, out)
    clean = out.clone()
    V[:, :, 0] = float("inf")
    K[:, :, 0] = float("nan")
    ck.ck_sparse_decode_attn(sh, q, K, V, idx, cnt, n, out)
    assert torch.equal(out, clean)
    b, h = torch.meshgrid(torch.arange(S, device=DEV), torch.arange(Hkv, device=DEV), indexing="ij")
    V[b, h, idx[:, :, 7].long(), 5] = float("inf")
    V[b, h, idx[:, :, 36].long(), 77] = float("-inf")
    ck.ck_sparse_decode_attn(sh, q, K, V, idx, cnt, n, out)
    clean[:, :, 5] = float("inf")
    clean[:, :, 77] = float("-inf")
    assert torch.equal(out, clean)


@pytest.mark.parametrize("S", [1, 64])
@pytest.mark.parametrize("G", [1, 4, 8])
@pytest.mark.parametrize("drop", [60.0, 100.0, 115.0, 140.0])
def test_unlikely_tokens_with_large_values(S, G, drop):
    """A token whose probability is about 2^-drop beside ordinary ones: a large finite value adds
    its product and nothing else (exactly nothing once the probability is zero), and an infinite
    one makes its channel infinite as long as there is a probability."""
    Hkv, N, n = 8, 300, 37
    g = torch.Generator(device=DEV).manual_seed(G)
    K = torch.randn(S, Hkv, N, 128, generator=g, device=DEV).bfloat16()
    V = torch.randn(S, Hkv, N, 128, generator=g, device=DEV).bfloat16()
    q = torch.zeros(S, Hkv * G, 128, device=DEV).bfloat16()
    q[..., 0] = 8.0
    K[..., 0] = 0.0
    idx = (torch.rand(S, Hkv, N, generator=g, device=DEV).topk(40).indices).int()
    cnt = torch.full((S, Hkv), n, dtype=torch.int32, device=DEV)
    b, h = torch.meshgrid(torch.arange(S, device=DEV), torch.arange(Hkv, device=DEV), indexing="ij")
    at = idx[:, :, 7].long()
    K[b, h, at, 0] = -drop / (8.0 * 128 ** -0.5 * 1.4426950408889634)
    V[b, h, at, :] = 0.0
    sh = ck.Shape(S, Hkv * G, Hkv, N, 8)
    out = torch.zeros(S, Hkv * G, 128, device=DEV).bfloat16()
    ck.ck_sparse_decode_attn(sh, q, K, V, idx, cnt, n, out)
    clean = out.clone()
    V[b, h, at, 5] = 3.3e38 if drop > 126 else 2.0 ** drop
    V[b, h, at, 6] = -3.3e38 if drop > 126 else 3.0 * 2.0 ** drop
    ck.ck_sparse_decode_attn(sh, q, K, V, idx, cnt, n, out)
    if drop > 126:
        assert torch.equal(out, clean)
        return
    for s, kv in [(0, 0), (S - 1, Hkv - 1)]:
        want = O.attention_over(np64(q[s, kv * G:(kv + 1) * G]), np64(K[s, kv]), np64(V[s, kv]),
                                idx[s, kv, :n].cpu().numpy())
        got = np64(out[s, kv * G:(kv + 1) * G])
        assert np.abs(got - want).max() <= TOL * np.abs(want).max(), (s, kv)
    V[b, h, at, 5] = float("inf")
    V[b, h, at, 6] = float("-inf")
    ck.ck_sparse_decode_attn(sh, q, K, V, idx, cnt, n, out)
    clean[:, :, 5] = float("inf")
    clean[:, :, 6] = float("-inf")
    assert torch.equal(out, clean)
