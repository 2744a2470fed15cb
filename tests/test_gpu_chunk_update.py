"""The update that sums a cluster straight from the assignment's chunk index, and the metadata
emitted from it, against the exported steps (assignment, counting sort, update from the sorted
list) run one by one on the same tables: every output bit for bit (the sums run in the same
order)."""
import pytest
import torch

import paper_2412_03213_amd as ck

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("S,Hkv,N,C,begin,c_begin", [
    (1, 2, 385, 9, 0, 0),            # just beyond the one-kernel range; chunks of 128, last one short
    (1, 1, 1000, 2, 16, 0),          # clusters of several hundred members: more than one pass of ids
    (3, 1, 4099, 130, 3, 5),         # appended behind existing clusters, odd range
    (2, 8, 4097, 513, 1, 0),         # table streamed in chunks; one token in the last chunk of 512
    (1, 8, 8200, 512, 0, 0),         # largest LDS-resident table
    (1, 1, 65535, 60, 0, 0),         # chunks of 128: exactly as many as the index holds
    (1, 1, 262144, 64, 0, 0),        # chunks of 512: exactly as many
    (1, 1, 262145, 64, 0, 0),        # one chunk more: counts only, and the sorted-list form
    (1, 2, 262700, 512, 7, 3),       # the same with the largest LDS-resident table
    (1, 1, 263681, 1100, 0, 0),      # and with the table streamed in chunks
    (1, 2, 2300, 2048, 0, 0),        # most clusters, many of them of one member or empty
])
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
        keep = hat.clone()
        ck.ck_kmeans_update(sh, K, want.sizes, want.offsets, want.sorted_idx, c_begin, C,
                            want.centroids, hat)
        if it == 0 and (want.sizes[:, :, c_begin:] == 0).any():
            # a row that stays empty keeps its first unit copy, whose last bit torch may round
            # differently from the library: such clusters end the comparison after one step
            assert torch.equal(keep[want.sizes[:, :, c_begin:] == 0],
                               hat[want.sizes[:, :, c_begin:] == 0])
            n_cmp = first
            break
    else:
        n_cmp = got
    torch.cuda.synchronize()
    for name in ("labels", "sizes", "offsets", "sorted_idx"):
        assert torch.equal(getattr(n_cmp, name), getattr(want, name)), name
    assert torch.equal(n_cmp.centroids.view(torch.int16), want.centroids.view(torch.int16))
