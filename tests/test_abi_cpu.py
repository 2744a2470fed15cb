"""Host-side checks of the C-ABI library that need no GPU: it loads, exports
every symbol the header declares, and rejects bad arguments before enqueuing
anything (so these calls are safe without a device)."""
import ctypes
import os
import re
import sys

import pytest
import torch

import paper_2412_03213_amd as ck
from paper_2412_03213_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "clusterkv.h")


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(ck_[a-z0-9_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = ck.load_library()
    names = declared_functions()
    assert set(names) == set(binding.EXPORTS)
    for n in names:
        assert getattr(lib, n) is not None
    assert ck.ck_version() == 100


def test_header_constants_match_binding():
    text = open(HEADER).read()
    consts = dict(re.findall(r"#define\s+(CK_[A-Z0-9_]+)\s+\(?(-?\d+)u?\)?", text))
    assert int(consts["CK_BF16"]) == ck.CK_BF16 and int(consts["CK_F32"]) == ck.CK_F32
    assert int(consts["CK_SEL_WHOLE"]) == ck.CK_SEL_WHOLE
    assert int(consts["CK_SEL_TRIM_LAST"]) == ck.CK_SEL_TRIM_LAST
    assert int(consts["CK_MAX_CLUSTERS"]) == ck.CK_MAX_CLUSTERS
    assert int(consts["CK_METRIC_COSINE"]) == ck.CK_METRIC_COSINE
    assert int(consts["CK_METRIC_L2"]) == ck.CK_METRIC_L2
    assert int(consts["CK_METRIC_IP"]) == ck.CK_METRIC_IP
    assert int(consts["CK_KM_UNTIL_CONVERGED"]) == ck.CK_KM_UNTIL_CONVERGED
    assert ctypes.sizeof(binding._CkShape) == 32


def test_strerror_and_workspace_sizes():
    lib = ck.load_library()
    assert lib.ck_strerror(0) == b"success"
    for code in (-1, -2, -3, -4, -5):
        assert lib.ck_strerror(code) not in (b"success", b"unknown error code")
    sh = ck.Shape(1, 32, 8, 32768, 400)
    assert ck.ck_workspace_bytes(sh, binding.CK_WS_CLUSTER_KEYS, 32768, 400) > 8 * 400 * 256
    assert ck.ck_workspace_bytes(sh, binding.CK_WS_SPARSE_ATTN, 1024) > 0
    assert ck.ck_workspace_bytes(sh, 99, 1024) == 0
    assert ck.ck_workspace_bytes(ck.Shape(1, 32, 8, 32768, 400, d=64), 0, 100, 4) == 0


def test_clustering_takes_a_workspace_of_large_chunks():
    """A workspace for more tokens serves fewer, whatever chunks either would take by itself: what an
    index of chunks of 512 tokens needs is enough, one byte less is not."""
    binding.load_library()
    HP, n, C = 16, 8000, 40                             # chunks of 128 by itself
    sh = ck.Shape(2, 8, 8, n, C)
    own = ck.ck_workspace_bytes(sh, binding.CK_WS_CLUSTER_KEYS, n, C)
    up = lambda b: (b + 255) // 256 * 256
    need = (up(HP * C * 256) + up(HP * 16 * 40 * 4) + up(HP * 16 * 512 * 2) + up(HP * 64 * 4)
            + up(257 * HP * 4))
    assert own > need
    A = 4096                                            # an aligned address that is never dereferenced
    lib = binding.load_library()
    call = lambda bytes_: lib.ck_build_metadata(ctypes.byref(sh.c()), A, 0, n, 0, C, A, A, A, A, bytes_, None)
    assert call(need - 1) == -3


# Head-problem tokens on both sides of 32768, 65536 and a full round of the chip, rows from one chunk of 128
# tokens to hundreds, C around 64, 128 and 160: every choice of chunk size, and ranges that fill large chunks badly.
WS_SHAPES = [(hp, n, C)
             for hp in (1, 3, 8, 16, 64, 128, 700, 1000)
             for T in (20000, 32768, 32769, 40000, 65535, 65536, 70000, 80000, 131072, 200000)
             for n in (max(1, T // hp), T // hp + 1)
             for C in (4, 7, 13, 40, 64, 65, 100, 128, 129, 160, 161, 400, 700) if C <= n]
WS_SHAPES += [(128, 600, 7), (128, 1100, 13), (64, 1025, 12), (700, 100, 4), (1, 300000, 50), (8, 131072, 1600)]


def clustering_needs(hp, n, C):
    """Bytes that ck_build_metadata and ck_cluster_keys ask for, from what they say to a workspace of one
    byte.  The addresses are aligned and never dereferenced."""
    lib, sh = binding.load_library(), ck.Shape(1, hp, hp, n, C).c()
    out = []
    for rc in (lib.ck_build_metadata(ctypes.byref(sh), A, 0, n, 0, C, A, A, A, A, 1, None),
               lib.ck_cluster_keys(ctypes.byref(sh), A, 0, n, 0, C, 1, A, A, A, A, A, A, A, 1, None)):
        assert rc == -3
        out.append(int(re.search(r"(\d+) needed", lib.ck_last_error_detail().decode()).group(1)))
    return out


def test_prescribed_workspace_is_enough():
    for hp, n, C in WS_SHAPES:
        have = ck.ck_workspace_bytes(ck.Shape(1, hp, hp, n, C), binding.CK_WS_CLUSTER_KEYS, n, C)
        assert max(clustering_needs(hp, n, C)) <= have, (hp, n, C)


@pytest.mark.parametrize("hp", [1, 8, 128, 700, 1000])
def test_workspace_for_more_serves_less(hp):
    """Fewer tokens, fewer clusters or both, across every change of the chunk size."""
    rows = sorted({max(4, T // hp + d) for T in (20000, 32768, 34000, 65536, 70000, 131072) for d in (-1, 0, 1, 13)})
    counts = [4, 40, 64, 65, 128, 160, 161, 400]
    size = {(n, C): ck.ck_workspace_bytes(ck.Shape(1, hp, hp, n, C), binding.CK_WS_CLUSTER_KEYS, n, C)
            for n in rows for C in counts}
    for n in rows:
        for C in counts:
            if C <= n:
                need = max(clustering_needs(hp, n, C))
                short = [k for k, b in size.items() if k[0] >= n and k[1] >= C and b < need]
                assert not short, (n, C, short)


@pytest.mark.parametrize("G", [1, 4, 8])
def test_attention_workspace_is_one_round_of_workgroups(G):
    """The workspace shows the number of splits: every XCD (32 compute units, one workgroup of
    eight wavefronts or two of four each) runs its share of the head-problems in one round where
    the 2048 positions of a workgroup allow it (up to 256 head-problems), and a workspace for a larger attended total
    holds every smaller one (its splits may be more)."""
    for HP in [*range(1, 140), 160, 200, 256, 257, 320, 512, 600, 2048]:
        sh = ck.Shape(1, HP * G, HP, 1 << 22, 8)
        per_xcd, last = -(-HP // 8), 0
        for total in [1, 64, 65, 127, 128, 129, 500, 1000, 1024, 1025, 2047, 2048, 2049, 2300, 4096,
                      8192, 32864, 131072, 1 << 20]:
            b = ck.ck_workspace_bytes(sh, binding.CK_WS_SPARSE_ATTN, total)
            splits = (b - (HP * 8 + 255) // 256 * 256) // (HP * G * 130 * 4)
            need = -(-total // 2048)
            room = 32 if per_xcd * need <= 32 else 64
            if 32 < per_xcd <= 40:                       # taken in turns, in smaller pieces
                room = 3 * per_xcd
            assert need <= splits <= max(need, room // per_xcd), (HP, total)
            assert splits <= max(1, -(-total // 64))
            assert b >= last, (HP, total)
            last = b
            if per_xcd * need <= 64:                     # fits the library's own scratch buffer
                assert b <= 4 << 20


A = 0x1000  # a 16-byte aligned fake device address: validation never dereferences it


def expect(code, fn, *args, **kw):
    with pytest.raises(ck.ClusterKVError) as e:
        fn(*args, **kw)
    assert e.value.code == code, str(e.value)


def test_argument_validation_without_a_device():
    sh = ck.Shape(1, 32, 8, 1000, 40)
    ws = A
    lib = ck.load_library()

    def cluster(sh=sh, K=A, tb=0, tc=1000, cb=0, cc=40, it=10, init=A, cent=A, lab=A, sz=A, off=A,
                sidx=A, ws=A, wsb=1 << 30):
        s = sh.c()
        rc = lib.ck_cluster_keys(ctypes.byref(s), K, tb, tc, cb, cc, it, init, cent, lab, sz, off,
                                 sidx, ws, wsb, None)
        if rc:
            raise ck.ClusterKVError(rc, lib.ck_strerror(rc).decode(),
                                    lib.ck_last_error_detail().decode())

    expect(-1, cluster, K=None)
    expect(-1, cluster, tb=500, tc=501)
    expect(-1, cluster, cb=30, cc=11)
    expect(-1, cluster, tc=30, cc=40)
    expect(-1, cluster, it=0)
    expect(-2, cluster, sh=ck.Shape(1, 32, 8, 1000, 40, d=64))
    expect(-2, cluster, sh=ck.Shape(1, 24, 8, 1000, 40))            # group of 3
    expect(-2, cluster, sh=ck.Shape(1, 32, 8, 1000, 40, dtype=ck.CK_F32))
    expect(-2, cluster, sh=ck.Shape(1, 32, 8, 5000, 4000), tc=5000, cc=2049)
    expect(-3, cluster, ws=None)
    expect(-3, cluster, wsb=16)
    expect(-4, cluster, lab=A + 4)
    expect(-1, cluster, sh=ck.Shape(1, 30, 8, 1000, 40))            # Hq not a multiple of Hkv

    def cluster_opt(flags=0, it=10, iters=None, lab=A):
        s = sh.c()
        rc = lib.ck_cluster_keys_opt(ctypes.byref(s), A, 0, 1000, 0, 40, it, flags, A, A, lab, A, A,
                                     A, iters, A, 1 << 30, None)
        if rc:
            raise ck.ClusterKVError(rc, lib.ck_strerror(rc).decode(),
                                    lib.ck_last_error_detail().decode())

    expect(-1, cluster_opt, flags=3)                                # no such metric
    expect(-1, cluster_opt, flags=8)                                # unknown bit
    expect(-1, cluster_opt, it=0)
    expect(-2, cluster_opt, flags=ck.CK_KM_UNTIL_CONVERGED, it=257)
    expect(-4, cluster_opt, iters=A + 4)
    expect(-4, cluster_opt, flags=ck.CK_METRIC_L2 | ck.CK_KM_UNTIL_CONVERGED, lab=A + 8)

    expect(-1, ck.ck_select_clusters, sh, A, A, A, 0, 10, 0, A, A, A, A)
    expect(-1, ck.ck_select_clusters, sh, A, A, A, 41, 10, 0, A, A, A, A)
    expect(-1, ck.ck_select_clusters, sh, A, A, A, 40, 0, 0, A, A, A, A)
    expect(-1, ck.ck_select_clusters, sh, A, A, A, 40, 10, 7, A, A, A, A)
    expect(-1, ck.ck_select_clusters, sh, None, A, A, 40, 10, 0, A, A, A, A)
    expect(-1, ck.ck_select_clusters, sh, A, A, A, 40, 10, 0, A, A, A, None)
    expect(-4, ck.ck_select_clusters, sh, A, A + 8, A, 40, 10, 0, A, A, A, A)

    def fused(**kw):
        args = dict(q=A, K=A, V=A, cent=A, sizes=A, offs=A, sidx=A, nc=40, B=16, flags=0,
                    scores=A, sel=A, nsel=A, ntok=A, idx=A, n=A, out=A, workspace=A)
        args.update(kw)
        ck.ck_decode_step(sh, args["q"], args["K"], args["V"], args["cent"], args["sizes"],
                          args["offs"], args["sidx"], args["nc"], args["B"], args["flags"],
                          args["scores"], args["sel"], args["nsel"], args["ntok"], args["idx"],
                          args["n"], args["out"], workspace=args["workspace"])

    expect(-1, fused, sidx=None)
    expect(-1, fused, nc=41)
    expect(-1, fused, B=0)
    expect(-1, fused, flags=2)
    expect(-3, fused, workspace=0)
    expect(-4, fused, scores=A + 4)

    expect(-1, ck.ck_gather_indices, sh, A, A, A, A, 0, 0, A, A)
    expect(-1, ck.ck_gather_indices, sh, A, None, A, A, 16, 0, A, A)

    expect(-1, ck.ck_kmeans_assign, sh, A, 0, 1001, A, 0, 40, A)
    expect(-1, ck.ck_kmeans_assign, sh, A, 0, 1000, None, 0, 40, A)
    expect(-3, ck.ck_build_metadata, sh, A, 0, 1000, 0, 40, A, A, A, workspace=0)
    expect(-1, ck.ck_kmeans_objective, sh, A, 0, 1001, A, 0, 40, A, A, A, workspace=A)
    expect(-1, ck.ck_kmeans_objective, sh, A, 0, 1000, A, 0, 40, A, None, A, workspace=A)
    expect(-3, ck.ck_kmeans_objective, sh, A, 0, 1000, A, 0, 40, A, A, A, workspace=0)
    assert ck.ck_workspace_bytes(sh, binding.CK_WS_OBJECTIVE, 1000) >= 8 * 2 * 8
    expect(-1, ck.ck_kmeans_update, sh, A, A, A, A, 0, 41, A, A)

    def attn(**kw):
        args = dict(sh=sh, q=A, K=A, V=A, idx=A, n=A, stride=1024, mx=1024, sink=0, rb=0, re=0,
                    scale=0.088, out=A, ws=A, wsb=1 << 30)
        args.update(kw)
        s = args["sh"].c()
        rc = lib.ck_sparse_decode_attn(ctypes.byref(s), args["q"], args["K"], args["V"],
                                       args["idx"], args["n"], args["stride"], args["mx"],
                                       args["sink"], args["rb"], args["re"], args["scale"],
                                       args["out"], args["ws"], args["wsb"], None)
        if rc:
            raise ck.ClusterKVError(rc, lib.ck_strerror(rc).decode(),
                                    lib.ck_last_error_detail().decode())

    expect(-1, attn, out=None)
    expect(-1, attn, sink=1001)
    expect(-1, attn, rb=0, re=1001)
    expect(-1, attn, stride=512)
    expect(-1, attn, scale=0.0)
    expect(-1, attn, idx=None)
    expect(-3, attn, wsb=8)
    expect(-3, attn, ws=None)
    expect(-4, attn, V=A + 2)

    # the same call on the built-in scratch buffer: same validation, and shapes whose
    # partials exceed the buffer are rejected before anything touches a device
    def attn_static(**kw):
        args = dict(sh=sh, q=A, K=A, V=A, idx=A, n=A, stride=1024, mx=1024, sink=0, rb=0, re=0,
                    scale=0.088, out=A)
        args.update(kw)
        s = args["sh"].c()
        rc = lib.ck_sparse_decode_attn_static(ctypes.byref(s), args["q"], args["K"], args["V"],
                                              args["idx"], args["n"], args["stride"], args["mx"],
                                              args["sink"], args["rb"], args["re"],
                                              args["scale"], args["out"], None)
        if rc:
            raise ck.ClusterKVError(rc, lib.ck_strerror(rc).decode(),
                                    lib.ck_last_error_detail().decode())

    expect(-1, attn_static, out=None)
    expect(-1, attn_static, sink=1001)
    expect(-1, attn_static, stride=512)
    expect(-4, attn_static, V=A + 2)
    big = ck.Shape(512, 32, 8, 4096, 40)                            # 4096 head-problems x 4 heads
    assert ck.ck_workspace_bytes(big, binding.CK_WS_SPARSE_ATTN, 1024) > (4 << 20)
    expect(-3, attn_static, sh=big)

    # evaluation entry points
    expect(-1, ck.ck_full_decode_attn, sh, A, A, A, 0, A, workspace=A)
    expect(-1, ck.ck_full_decode_attn, sh, A, A, A, 1001, A, workspace=A)
    expect(-1, ck.ck_full_decode_attn, sh, A, A, None, 1000, A, workspace=A)
    expect(-3, ck.ck_full_decode_attn, sh, A, A, A, 1000, A, workspace=0)
    expect(-1, ck.ck_token_scores, sh, A, A, 0, 1001, A)
    expect(-1, ck.ck_token_scores, sh, A, A, 0, 1000, None)
    expect(-4, ck.ck_token_scores, sh, A, A + 4, 0, 1000, A)
    expect(-1, ck.ck_topk_select, 0, A, 1000, 0, 1000, 10, A, A)
    expect(-1, ck.ck_topk_select, 8, A, 1000, 0, 0, 10, A, A)
    expect(-1, ck.ck_topk_select, 8, A, 1000, 0, 1000, -1, A, A)
    expect(-1, ck.ck_topk_select, 8, A, 1000, 1, 1000, 10, A, A)        # range leaves the row
    expect(-1, ck.ck_topk_select, 8, A, 1000, 0, 1000, 10, A, None)
    expect(-1, ck.ck_recall_hits, 8, A, A, A, None, A)
    expect(-1, ck.ck_recall_hits, 70000, A, A, A, A, A)
    expect(-1, ck.ck_page_keys, sh, A, 0, 1000, 0, A)                   # page_size 0, stride 0
    expect(-1, ck.ck_page_keys, sh, A, 0, 1001, 16, A)
    expect(-1, ck.ck_expand_pages, 8, A, A, 0, 0, 1000, A, A)
    expect(-1, ck.ck_expand_pages, 8, A, None, 16, 0, 1000, A, A)

    # cluster cache
    two = ctypes.c_void_p * 2

    def cache_struct(cap=64, K0=A):
        return binding._CkClusterCache(two(K0, A), two(A, A), two(A, A), two(A, A), two(A, A),
                                       cap, 0)

    def cached(cache=None, B=16, parity=0, miss=A, nc=40, ws=A):
        ck.ck_cached_decode_step(sh, A, A, A, A, A, A, A, nc, B,
                                 cache_struct() if cache is None else cache, parity, A, A, A, A,
                                 miss, A, workspace=ws)

    expect(-1, cached, B=65)                                        # budget above the cache rows
    expect(-1, cached, parity=2)
    expect(-1, cached, miss=None)
    expect(-1, cached, nc=41)
    expect(-1, cached, cache=cache_struct(cap=0))
    expect(-1, cached, cache=cache_struct(K0=None))
    expect(-4, cached, cache=cache_struct(K0=A + 4))
    expect(-3, cached, ws=0)
    expect(-1, ck.ck_cache_reset, sh, cache_struct(cap=0))
    expect(-1, ck.ck_host_device_ptr, 0)


def test_missing_library_is_an_error(monkeypatch, tmp_path):
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "LIB_PATH", str(tmp_path / "nope.so"))
    with pytest.raises(RuntimeError):
        binding.load_library(build_if_missing=False)


def _without_host_module(monkeypatch):
    monkeypatch.setitem(sys.modules, "paper_2412_03213_amd._ckhost", None)
    monkeypatch.delattr(ck, "_ckhost", raising=False)
    monkeypatch.setattr(binding, "_lib", None)


def test_library_is_enough_without_the_host_module(monkeypatch):
    """No module for this interpreter: the library loads, and calls go through ctypes."""
    _without_host_module(monkeypatch)
    lib = ck.load_library(build_if_missing=False)
    assert lib.host_decode_step(1, 2, 3) is None
    z = torch.zeros(16)
    with pytest.raises(ck.ClusterKVError):                        # S = 0
        ck.ck_decode_step(ck.Shape(0, 2, 2, 16, 4), z, z, z, z, z, z, z, 4, 8, 0, z, z, z, z, z, z,
                          z, workspace=z)


def test_build_goes_on_without_a_host_compiler(monkeypatch, tmp_path, capsys):
    from paper_2412_03213_amd import build as b
    monkeypatch.setattr(b, "SOURCES", [])                         # the library stands
    monkeypatch.setattr(b, "HOST_LIB", str(tmp_path / "_ckhost.so"))
    monkeypatch.setattr(b, "CXX", "no-such-compiler")
    assert b.build(verbose=False) == b.LIB
    assert "ctypes" in capsys.readouterr().out and not os.path.exists(b.HOST_LIB)


def test_stream_without_the_raw_form(monkeypatch):
    monkeypatch.setattr(binding, "_raw_stream", None)
    assert binding._stream(torch.zeros(1)) == 0


@pytest.mark.parametrize("change, error", [
    ({}, ck.ClusterKVError),                                      # S = 0: refused by the library
    ({"K": "strided"}, ValueError),                               # marshalling refuses it
    ({"budget": 2.0}, ctypes.ArgumentError),
    ({"flags": None}, ctypes.ArgumentError),
    ({"scores": None}, ck.ClusterKVError),
    ({"V": 4096}, ck.ClusterKVError),                             # raw address
    ({"n_sink": 1 << 40}, ck.ClusterKVError),
    ({"budget": (1 << 32) + 5}, ck.ClusterKVError),               # cut to 32 bits as before
])
def test_decode_step_refuses_the_same_calls_on_either_way(change, error):
    """The native marshalling hands every argument that is not plain to the ctypes call."""
    bf, i32 = dict(dtype=torch.bfloat16), dict(dtype=torch.int32)
    kv = torch.zeros(1, 2, 16, 128, **bf)
    a = dict(q=torch.zeros(1, 2, 128, **bf), K=kv, V=kv, centroids=torch.zeros(1, 2, 4, 128, **bf),
             sizes=torch.zeros(1, 2, 4, **i32), offsets=torch.zeros(1, 2, 5, **i32),
             sorted_idx=torch.zeros(1, 2, 16, **i32), n_clusters=4, budget=8, flags=0,
             scores=torch.zeros(1, 2, 4), sel_clusters=torch.zeros(1, 2, 4, **i32),
             n_sel_clusters=torch.zeros(1, 2, **i32), n_sel_tokens=torch.zeros(1, 2, **i32),
             token_idx=torch.zeros(1, 2, 8, **i32), n_tokens=torch.zeros(1, 2, **i32),
             out=torch.zeros(1, 2, 128, **bf), workspace=torch.zeros(65536, dtype=torch.uint8))
    for k, v in change.items():
        a[k] = kv.transpose(2, 3) if isinstance(v, str) else v
    sh = ck.Shape(0, 2, 2, 16, 4)
    with pytest.raises(error) as native:
        ck.ck_decode_step(sh, **a)
    lib = ck.load_library()
    real, lib.host_decode_step = lib.host_decode_step, lambda *args: None
    try:
        with pytest.raises(error) as general:
            ck.ck_decode_step(sh, **a)
    finally:
        lib.host_decode_step = real
    assert str(native.value) == str(general.value)


def test_form_of_the_chunk_update():
    """The launcher's choice between one cluster and four per workgroup, on both sides of each of
    its lines, and that the GPU tests of the second form are in it."""
    rule = ck.load_library()._ZN2ck29update_clusters_per_workgroupEiii
    rule.restype, rule.argtypes = ctypes.c_int, [ctypes.c_int] * 3
    assert rule(256, 1600, 8) == 4 and rule(129, 2048, 8) == 4
    assert rule(128, 2048, 64) == 1                     # few chunks
    assert rule(512, 767, 64) == 1 and rule(512, 768, 64) == 4
    assert rule(512, 2048, 1) == 1 and rule(512, 2048, 2) == 4
    assert rule(512, 2048, 65535) == 4                  # the product of all three is beyond 32 bits
    from tests.test_gpu_chunk_update import FOUR
    for S, Hkv, N, C, begin, _ in FOUR:
        assert (N - begin) * S * Hkv >= 65536           # chunks of 512 tokens
        assert rule((N - begin + 511) // 512, C, S * Hkv) == 4 and C % 4


def test_forms_of_the_assignment():
    """The shapes of the GPU tests run the kernels that they are listed under."""
    from tests import forms
    from tests.test_gpu_assign_forms import FORMS, L2_FORMS
    from tests.test_gpu_chunk_update import STOPPING
    for lists in (FORMS, L2_FORMS):
        for form, shapes in lists.items():
            assert [forms.assignment(*shape) for shape in shapes] == [form] * len(shapes)
    for shape, kernels in STOPPING.items():
        assert (forms.assignment(*shape), forms.update(*shape)) == kernels, shape
