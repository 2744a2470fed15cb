"""The updates that sum a cluster straight from the assignment's chunk index or from its labels, and
the metadata emitted with them, against the exported steps (assignment, counting sort, update from
the sorted list) run one by one on the same tables: every output bit for bit (the sums run in the same
order)."""
import pytest
import torch

import paper_2412_03213_amd as ck

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


SHAPES = [
    (1, 2, 385, 9, 0, 0),            # just beyond the one-kernel range; from the labels
    (1, 1, 1000, 2, 16, 0),          # clusters of several hundred members: more than one pass of rows
    (3, 1, 4099, 130, 3, 5),         # 4096 labels, appended behind existing clusters, odd range
    (1, 1, 4097, 100, 0, 2),         # one label more: sixteen per lane
    (1, 1, 8195, 512, 3, 0),         # as many labels, and read as often, as that form takes
    (4, 4, 600, 64, 0, 0),           # as many workgroups
    (16, 1, 600, 65, 5, 1),          # more: chunks of 128, last one short
    (1, 1, 8193, 60, 0, 0),          # a label more: the same
    (2, 1, 8192, 2, 0, 0),           # from the labels: members in many passes
    (1, 8, 4050, 130, 3, 5),         # chunks of 128, appended behind existing clusters, odd range
    (2, 8, 4050, 130, 3, 5),         # of 256
    (2, 8, 4097, 513, 1, 0),         # exactly sixteen of them
    (2, 8, 4098, 513, 1, 0),         # table streamed in chunks; one token in the last chunk of 512
    (1, 8, 8200, 512, 0, 0),         # largest LDS-resident table
    (128, 1, 600, 7, 0, 0),          # from the labels; the exported sort's chunks of 512 need the larger workspace
    (1, 1, 65535, 60, 0, 0),         # chunks of 256
    (1, 2, 65536, 60, 0, 0),         # chunks of 128: exactly as many as the index holds
    (3, 1, 20000, 70, 3, 5),         # chunks of 256, appended behind existing clusters, odd range
    (9, 1, 9001, 100, 1, 0),         # chunks of 128, two table chunks
    (16, 1, 9001, 80, 1, 0),         # the same with the keys through half of the LDS
    (33, 1, 1900, 100, 0, 0),        # and chunks of 256
    (1100, 1, 520, 512, 0, 0),       # more workgroups of the update than a grid has in x
    (1, 1, 262144, 64, 0, 0),        # chunks of 512: exactly as many
    (1, 1, 262145, 64, 0, 0),        # one chunk more: counts only, and the sorted-list form
    (1, 2, 262700, 512, 7, 3),       # the same with the largest LDS-resident table
    (1, 1, 263681, 1100, 0, 0),      # and with the table streamed in chunks
    (1, 2, 2300, 2048, 0, 0),        # most clusters, many of them of one member or empty
    (5, 1, 65530, 2047, 0, 0),       # 128 chunks, the most that are scanned in two steps
    (8, 1, 66053, 2047, 3, 1),       # four clusters to a workgroup of the update, three in the last
    (4, 2, 66049, 2045, 0, 0),       # the same with one in the last
]
FOUR = SHAPES[-2:]                   # see test_abi_cpu.py: they are in the form that they are here for


@pytest.mark.parametrize("S,Hkv,N,C,begin,c_begin", SHAPES)
def test_cluster_keys_equals_the_exported_steps(S, Hkv, N, C, begin, c_begin):
    g = torch.Generator(device=DEV).manual_seed(N + C)
    n, n_iter = N - begin, 3
    K = torch.randn(S, Hkv, N, 128, generator=g, device=DEV).to(torch.bfloat16)
    init = (torch.rand(S, Hkv, n, generator=g, device=DEV).topk(C, dim=-1).indices + begin).int()
    sh = ck.Shape(S, Hkv, Hkv, N, C + c_begin)
    got, want = (ck.ClusterState(sh, DEV, budget=64) for _ in range(2))
    got.n_clusters = c_begin
    got.cluster(K, init, begin, n, C, n_iter)

    rows = torch.gather(K, 2, init.long()[..., None].expand(-1, -1, -1, 128))
    want.centroids[:, :, c_begin:] = rows
    f = rows.float()
    # the unit rows of the first table as the library makes them: one iteration's labels tell
    # whether they agree, so they are taken from a run of the library itself where they matter
    hat = (f * (1.0 / (f * f).sum(-1, keepdim=True).sqrt())).to(torch.bfloat16).contiguous()
    first = ck.ClusterState(sh, DEV, budget=64)
    first.n_clusters = c_begin
    first.cluster(K, init, begin, n, C, 1)
    want.labels.copy_(first.labels)
    for it in range(n_iter):
        if it:
            ck.ck_kmeans_assign(sh, K, begin, n, hat, c_begin, C, want.labels)
        ck.ck_build_metadata(sh, want.labels, begin, n, c_begin, C, want.sizes, want.offsets,
                             want.sorted_idx)
        ck.ck_kmeans_update(sh, K, want.sizes, want.offsets, want.sorted_idx, c_begin, C,
                            want.centroids, hat)
        # (an initial row is its own nearest: no cluster is empty before every row has been the
        # library's own unit copy)
        assert it or (want.sizes[:, :, c_begin:] > 0).all()
    torch.cuda.synchronize()
    for name in ("labels", "sizes", "offsets", "sorted_idx"):
        assert torch.equal(getattr(got, name), getattr(want, name)), name
    assert torch.equal(got.centroids.view(torch.int16), want.centroids.view(torch.int16))


@pytest.mark.parametrize("hp,tiles", [(1, 1), (1, 7), (3, 5), (7, 13), (9, 1), (8, 8), (37, 11), (300, 3)])
def test_every_tile_has_its_workgroup(hp, tiles):
    """Head-problems times tiles that eight XCDs share evenly or not, one tile of 128 tokens each: every
    label of the assignment is written, none outside."""
    n = tiles * 128 - 5
    g = torch.Generator(device=DEV).manual_seed(hp * 100 + tiles)
    K = torch.randn(1, hp, n + 4, 128, generator=g, device=DEV).to(torch.bfloat16)
    hat = K[:, :, 2:12].contiguous()                    # every key is compared with the first ten
    labels = torch.full((1, hp, n + 4), -1, dtype=torch.int32, device=DEV)
    ck.ck_kmeans_assign(ck.Shape(1, hp, hp, n + 4, 10), K, 2, n, hat, 0, 10, labels)
    torch.cuda.synchronize()
    assert (labels[:, :, :2] == -1).all() and (labels[:, :, n + 2:] == -1).all()
    sim = (K[0, :, 2:n + 2].double() @ hat[0].double().transpose(1, 2).contiguous()).topk(2, dim=-1)
    clear = sim.values[..., 0] - sim.values[..., 1] > 1e-2
    assert torch.equal(labels[0, :, 2:n + 2][clear], sim.indices[..., 0][clear].int())


def test_workspace_of_large_chunks():
    """In a workspace that holds chunks of 512 tokens only (see test_abi_cpu.py) the call takes those:
    same outputs."""
    HP, n, C = 16, 8000, 40
    g = torch.Generator(device=DEV).manual_seed(5)
    K = torch.randn(2, 8, n, 128, generator=g, device=DEV).to(torch.bfloat16)
    init = torch.rand(2, 8, n, generator=g, device=DEV).topk(C, dim=-1).indices.int()
    sh = ck.Shape(2, 8, 8, n, C)
    up = lambda b: (b + 255) // 256 * 256
    need = (up(HP * C * 256) + up(HP * 16 * 40 * 4) + up(HP * 16 * 512 * 2) + up(HP * 64 * 4)
            + up(257 * HP * 4))
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    a, b = (ck.ClusterState(sh, DEV, budget=64) for _ in range(2))
    a.cluster(K, init, 0, n, C, 3)
    ck.ck_cluster_keys(sh, K, 0, n, 0, C, 3, init, b.centroids, b.labels, b.sizes, b.offsets,
                       b.sorted_idx, workspace=ws)
    torch.cuda.synchronize()
    for name in ("labels", "sizes", "offsets", "sorted_idx", "centroids"):
        assert torch.equal(getattr(a, name), getattr(b, name)), name


@pytest.mark.parametrize("hp,n,C,tokens", [(8, 4096, 400, 512), (300, 250, 100, 256), (1000, 125, 100, 128),
                                           (4, 8192, 513, 512), (128, 1100, 13, 128)])
def test_smallest_workspace(hp, n, C, tokens):
    """What the chunk size that needs least asks for is enough, whatever would be preferred: same outputs,
    also of the exported sort."""
    g = torch.Generator(device=DEV).manual_seed(hp)
    K = torch.randn(1, hp, n, 128, generator=g, device=DEV).to(torch.bfloat16)
    init = torch.rand(1, hp, n, generator=g, device=DEV).topk(C, dim=-1).indices.int()
    sh = ck.Shape(1, hp, hp, n, C)
    up = lambda b: (b + 255) // 256 * 256
    chunks, stride = -(-n // tokens), -(-C // 4) * 4
    need = (up(hp * C * 256) + up(hp * chunks * stride * 4) + up(hp * chunks * tokens * 2)
            + up(hp * -(-C // 32) * 128) + up(257 * hp * 4))
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    a, b = (ck.ClusterState(sh, DEV, budget=64) for _ in range(2))
    with pytest.raises(ck.ClusterKVError, match="workspace"):
        ck.ck_build_metadata(sh, a.labels, 0, n, 0, C, a.sizes, a.offsets, a.sorted_idx, workspace=ws[:-1])
    a.cluster(K, init, 0, n, C, 3)
    ck.ck_cluster_keys(sh, K, 0, n, 0, C, 3, init, b.centroids, b.labels, b.sizes, b.offsets,
                       b.sorted_idx, workspace=ws)
    torch.cuda.synchronize()
    names = ("labels", "sizes", "offsets", "sorted_idx", "centroids")
    assert all(torch.equal(getattr(a, x), getattr(b, x)) for x in names)
    for x in names[1:4]:
        getattr(b, x).fill_(-1)
    ck.ck_build_metadata(sh, a.labels, 0, n, 0, C, b.sizes, b.offsets, b.sorted_idx, workspace=ws)
    torch.cuda.synchronize()
    assert all(torch.equal(getattr(a, x), getattr(b, x)) for x in names)


@pytest.mark.parametrize("S,Hkv,N,C,begin,c_begin", SHAPES)
def test_empty_clusters_survive_the_iterations(S, Hkv, N, C, begin, c_begin):
    """The same by inner product, whose table is the stored centroids themselves: long rows draw
    the keys away from most others, so that many clusters are empty from the first iteration on,
    and an empty one keeps its row through the next ones."""
    g = torch.Generator(device=DEV).manual_seed(N - C)
    n, n_iter = N - begin, 3
    K = torch.randn(S, Hkv, N, 128, generator=g, device=DEV)
    K = (K * (0.3 + torch.rand(S, Hkv, N, 1, generator=g, device=DEV))).to(torch.bfloat16)
    init = (torch.rand(S, Hkv, n, generator=g, device=DEV).topk(C, dim=-1).indices + begin).int()
    sh = ck.Shape(S, Hkv, Hkv, N, C + c_begin)
    got, want = (ck.ClusterState(sh, DEV, budget=64) for _ in range(2))
    got.n_clusters = c_begin
    got.cluster(K, init, begin, n, C, n_iter, flags=ck.CK_METRIC_IP)

    want.centroids[:, :, c_begin:] = torch.gather(K, 2, init.long()[..., None].expand(-1, -1, -1, 128))
    unit = torch.empty(S, Hkv, C, 128, dtype=torch.bfloat16, device=DEV)
    empty = 0
    for _ in range(n_iter):
        table = want.centroids[:, :, c_begin:].contiguous()
        ck.ck_kmeans_assign(sh, K, begin, n, table, c_begin, C, want.labels)
        ck.ck_build_metadata(sh, want.labels, begin, n, c_begin, C, want.sizes, want.offsets,
                             want.sorted_idx)
        ck.ck_kmeans_update(sh, K, want.sizes, want.offsets, want.sorted_idx, c_begin, C,
                            want.centroids, unit)
        none = want.sizes[:, :, c_begin:] == 0
        empty += int(none.sum())
        assert torch.equal(want.centroids[:, :, c_begin:][none], table[none])
    torch.cuda.synchronize()
    for name in ("labels", "sizes", "offsets", "sorted_idx"):
        assert torch.equal(getattr(got, name), getattr(want, name)), name
    assert torch.equal(got.centroids.view(torch.int16), want.centroids.view(torch.int16))
    if C >= 500:
        assert empty > 0


@pytest.mark.parametrize("S,Hkv,N,C", [(1, 8, 8200, 100),    # chunks of 128, two table chunks
                                       (1, 8, 8200, 520),    # table streamed in chunks
                                       (2, 2, 1500, 40),     # from the labels
                                       (1, 8, 4000, 130),    # chunks of 128
                                       (1, 2, 262700, 30)])  # counts only, sorted-list form
def test_head_problems_stop_on_their_own(S, Hkv, N, C):
    """Run until convergence: a head-problem that has stopped keeps the chunk index, the sizes
    and the table that its own last iteration left, whatever the others go on to do."""
    max_iter = 40 if N < 100000 else 8
    g = torch.Generator(device=DEV).manual_seed(C)
    K = torch.randn(S, Hkv, N, 128, generator=g, device=DEV)
    # every second head: C far centers, every token a few hundredths away from its own
    for h in range(0, Hkv, 2):
        far = torch.randn(S, C, 128, generator=g, device=DEV) * 4
        pick = torch.arange(N, device=DEV) % C
        K[:, h] = far[:, pick] + 0.02 * K[:, h]
    K = K.to(torch.bfloat16)
    init = torch.rand(S, Hkv, N, generator=g, device=DEV).topk(C, dim=-1).indices.int()
    init[:, 0::2] = torch.arange(C, device=DEV).int()    # one row of every center
    sh = ck.Shape(S, Hkv, Hkv, N, C)
    st = ck.ClusterState(sh, DEV, budget=64)
    iters = torch.zeros(S, Hkv, dtype=torch.int32, device=DEV)
    st.cluster(K, init, 0, N, C, max_iter, ck.CK_KM_UNTIL_CONVERGED, iters)
    ran = iters.cpu()
    assert (ran[:, 0::2] == 2).all() and (ran[:, 1::2] > 2).all() and (ran <= max_iter).all()
    for n_iter in sorted(set(ran.flatten().tolist())):
        ref = ck.ClusterState(sh, DEV, budget=64)
        ref.cluster(K, init, 0, N, C, n_iter)
        for s in range(S):
            for h in range(Hkv):
                if int(ran[s, h]) != n_iter:
                    continue
                for name in ("labels", "sizes", "offsets", "sorted_idx", "centroids"):
                    assert torch.equal(getattr(st, name)[s, h], getattr(ref, name)[s, h]), (h, name)


# (head-problems, tokens, clusters): the forms of assignment and update (see forms.py; held to them by
# test_abi_cpu.py)
STOPPING = {(7, 9000, 30): ("few 256 one", "chunks"),
            (16, 9000, 80): ("few 128 tight", "chunks"),
            (70, 1500, 16): ("few 128 one", "chunks"),       # two words of head-problems
            (5, 13107, 100): ("few 256 tight", "chunks"),
            (8, 30000, 100): ("stream early", "chunks"),
            (8, 33000, 400): ("stream", "chunks"),
            (3, 50000, 600): ("wide", "chunks"),
            (130, 500, 9): ("few 256 one", "chunks"),        # three words
            (260, 600, 9): ("few 128 one", "chunks"),        # more head-problems than are listed
            (40, 800, 10): ("few 128 one", "labels"),
            (2, 262700, 30): ("stream early", "sorted")}


@pytest.mark.parametrize("metric", [ck.CK_METRIC_COSINE, ck.CK_METRIC_L2])
@pytest.mark.parametrize("hp,n,C", STOPPING)
def test_head_problems_stop_early_and_late(hp, n, C, metric):
    """Head-problems that stop in the second iteration, between the others and after all of them: while
    workgroups look late whether theirs has stopped, and when only those that run are dealt out."""
    max_iter = 40
    g = torch.Generator(device=DEV).manual_seed(hp * n + C)
    K = torch.empty(1, hp, n, 128, dtype=torch.bfloat16, device=DEV)
    for h in range(hp):
        far = torch.randn(C, 128, generator=g, device=DEV) * 4
        k = torch.randn(n, 128, generator=g, device=DEV)
        # every third head settles at once, the others the later the wider the clusters are
        pick = torch.arange(n, device=DEV) % C
        K[0, h] = k if h % 3 == 2 else far[pick] + (0.02 if h % 3 == 0 else 3.5) * k
    init = torch.rand(1, hp, n, generator=g, device=DEV).topk(C, dim=-1).indices.int()
    init[:, 0::3] = torch.arange(C, device=DEV).int()    # one row of every center
    sh = ck.Shape(1, hp, hp, n, C)
    st, ref = (ck.ClusterState(sh, DEV, budget=64) for _ in range(2))
    iters = torch.zeros(1, hp, dtype=torch.int32, device=DEV)
    st.cluster(K, init, 0, n, C, max_iter, metric | ck.CK_KM_UNTIL_CONVERGED, iters)
    ran = iters[0].cpu()
    assert (ran[0::3] == 2).all() and ran.max() > 12 and (ran <= max_iter).all()   # 12: KM_LOOK_FIRST
    for n_iter in sorted(set(ran.tolist())):
        ref.n_clusters = 0
        ref.cluster(K, init, 0, n, C, n_iter, metric)
        those = (ran == n_iter).nonzero()[:, 0].to(DEV)
        for name in ("labels", "sizes", "offsets", "sorted_idx"):
            assert torch.equal(getattr(st, name)[0, those], getattr(ref, name)[0, those]), (n_iter, name)
        assert torch.equal(st.centroids.view(torch.int16)[0, those], ref.centroids.view(torch.int16)[0, those])
