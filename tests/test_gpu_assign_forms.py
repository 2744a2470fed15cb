"""The assignment kernels at the edges of their tiles, rings and blocks: every key's label and the
label-ordered chunks behind the metadata, against the same contraction in 64 bits."""
import pytest
import torch

import paper_2412_03213_amd as ck

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
NEAR_TIE = 1e-4                      # cosine gap below which either of two labels may stand

# (head-problems, tokens, clusters) by the form that takes them (see forms.py; held to it by test_abi_cpu.py)
FORMS = {
    "wide": [(1, 65537, 513),            # one row in the last tile, one token in the last workgroup
             (2, 32800, 544),            # whole tiles, ragged last workgroup
             (1, 66000, 575),            # 18 tiles: the ring of six three times round
             (3, 21900, 609),            # 20 tiles, one row in the last
             (2, 33000, 2048)],          # most clusters
    "stream": [(1, 65537, 512),          # one token in the last block, largest table
               (2, 40960, 129), (2, 60000, 129)],
    "stream early": [(1, 65537, 128), (8, 13000, 128), (8, 12000, 128),
                     (8, 50000, 65),     # 98 blocks a head-problem: four to a workgroup
                     (40, 10000, 65),    # 20 blocks, four to a workgroup of five
                     (64, 20000, 66),    # 40 blocks, ten rounds' worth in two
                     (300, 700, 65)],    # more head-problems than compute units
    "few 128 one": [(3, 10922, 64), (8, 8193, 64), (700, 500, 5), (8, 50000, 40), (40, 10000, 33),
                    (64, 20000, 31), (300, 600, 7)],
    "few 128": [(1, 32768, 65), (8, 8193, 128), (9, 10100, 128), (2, 39000, 160)],
    "few 128 tight": [(16, 9000, 80)],
    "few 256 one": [(5, 13107, 64)],
    "few 256": [(1, 32769, 129),
                (2, 32768, 700),         # a table of eleven chunks
                (1, 65536, 2048)],
    "few 256 tight": [(33, 1900, 100)],
}
ALL = [shape for shapes in FORMS.values() for shape in shapes]
L2_FORMS = {
    "wide": [(1, 65537, 513), (2, 32801, 2047)],
    "stream": [(1, 65537, 511)],
    "stream early": [(8, 13000, 100), (8, 50000, 65)],
    "few 128 one": [(2, 385, 9)],
    "few 128": [(1, 2500, 2047), (8, 8193, 100), (9, 10100, 100)],
    "few 128 tight": [(16, 9000, 80)],
    "few 256 one": [(1, 40000, 64)],
    "few 256": [(2, 20000, 600)],
    "few 256 tight": [(33, 1900, 100)],
}


@pytest.mark.parametrize("hp,n,C", ALL)
def test_labels_against_64_bits(hp, n, C):
    g = torch.Generator(device=DEV).manual_seed(n + C)
    K = torch.randn(1, hp, n + 3, 128, generator=g, device=DEV).to(torch.bfloat16)
    hat = torch.randn(1, hp, C, 128, generator=g, device=DEV)
    hat = (hat / hat.norm(dim=-1, keepdim=True)).to(torch.bfloat16)
    labels = torch.full((1, hp, n + 3), -1, dtype=torch.int32, device=DEV)
    ck.ck_kmeans_assign(ck.Shape(1, hp, hp, n + 3, C), K, 2, n, hat, 0, C, labels)
    torch.cuda.synchronize()
    assert (labels[:, :, :2] == -1).all() and (labels[:, :, n + 2:] == -1).all()
    ties = 0
    for h in range(hp):
        keys = K[0, h, 2:n + 2].double()
        sim = keys @ hat[0, h].double().T
        two = sim.topk(min(2, C), dim=-1).values
        gap = (two[:, 0] - two[:, -1]) / keys.norm(dim=-1)
        wrong = labels[0, h, 2:n + 2] != sim.argmax(-1)
        assert not (wrong & (gap >= NEAR_TIE)).any(), h
        ties += int((gap < NEAR_TIE).sum())
    assert ties < 0.01 * hp * n


@pytest.mark.parametrize("hp,n,C", ALL)
def test_iterations_leave_consistent_metadata(hp, n, C):
    g = torch.Generator(device=DEV).manual_seed(n - C)
    K = torch.randn(1, hp, n, 128, generator=g, device=DEV).to(torch.bfloat16)
    init = torch.rand(1, hp, n, generator=g, device=DEV).topk(C, dim=-1).indices.int()
    st = ck.ClusterState(ck.Shape(1, hp, hp, n, C), DEV, budget=64)
    st.cluster(K, init, 0, n, C, 2)
    torch.cuda.synchronize()
    lab = st.labels[0].long()
    sizes = torch.zeros(hp, C, dtype=torch.int64, device=DEV).scatter_add_(1, lab, torch.ones_like(lab))
    assert torch.equal(st.sizes[0].long(), sizes)
    assert torch.equal(st.offsets[0, :, 1:].long(), sizes.cumsum(1))
    assert torch.equal(st.sorted_idx[0].long(), lab.sort(dim=1, stable=True).indices)


@pytest.mark.parametrize("hp,n,C", [shape for shapes in L2_FORMS.values() for shape in shapes])
def test_l2_labels_against_64_bits(hp, n, C):
    """One iteration by l2 assigns every key to the nearest of the given rows.  A similarity
    x mu - |mu|^2 / 2 is off by at most 128 * 2^-24 of |x| |mu| + |mu|^2 / 2 (fp32 sums of exact
    products) and 2^-19 of itself (packed maximum): 1e-5, and two are compared."""
    g = torch.Generator(device=DEV).manual_seed(n * C)
    K = torch.randn(1, hp, n + 2, 128, generator=g, device=DEV).to(torch.bfloat16)
    init = (torch.rand(1, hp, n, generator=g, device=DEV).topk(C, dim=-1).indices + 2).int()
    st = ck.ClusterState(ck.Shape(1, hp, hp, n + 2, C), DEV, budget=64)
    st.cluster(K, init, 2, n, C, 1, ck.CK_METRIC_L2)
    torch.cuda.synchronize()
    ties = 0
    for h in range(hp):
        keys, mu = K[0, h, 2:].double(), K[0, h][init[0, h].long()].double()
        two = (keys @ mu.T - mu.square().sum(-1) / 2).topk(2, dim=-1)
        longest = mu.norm(dim=-1).max()
        near = two.values[:, 0] - two.values[:, 1] < 2 ** -15 * (keys.norm(dim=-1) + longest / 2) * longest
        wrong = st.labels[0, h, 2:] != two.indices[:, 0]
        assert not (wrong & ~near).any(), h
        ties += int(near.sum())
    assert ties < 0.01 * hp * n
