"""Workspace sizes of sequences (no device needed): every snapshot's calls must fit,
also where a smaller snapshot needs more than the largest."""

import ctypes as C

import pytest


def aligned(x):
    return (x + 255) // 256 * 256


@pytest.mark.parametrize("prec,k,depth,big,small", [
    ("fp32", 128, 2, 4096, 3840),     # solve: more splits at 3840
    ("bf16", 128, 2, 2560, 2304),
    ("bf16", 16, 2, 7168, 6912),      # chain: 6912 splits its squarings' last round
    ("fp16", 40, 5, 8192, 6912),
    ("fp64", 32, 3, 4096, 3840),
    ("fp64", 32, 3, 3840, 256)])
def test_small_snapshots_fit(prec, k, depth, big, small):
    import paper_1802_05421_amd._lib as L
    lib, T = L.load(), 30
    p = L.PREC[prec]

    def needs(n):
        r = [C.c_size_t() for _ in range(4)]
        assert lib.cdl_workspace_bytes(n, T, k, depth, p, *[C.byref(x) for x in r]) == 0
        return [x.value for x in r]

    def sequence(sizes, flags):
        snaps = (L.Snapshot * len(sizes))()
        for s, n in zip(snaps, sizes):
            s.n, s.T, s.ldx = n, T, T
        q = L.SeqParams(k=k, prec=p, depth=depth, depth_max=depth, flags=flags)
        b = C.c_size_t()
        assert lib.cdl_sequence_workspace_bytes(len(sizes), snaps, C.byref(q), C.byref(b)) == 0
        return b.value

    more = sum(max(0, a - b) for a, b in zip(needs(small), needs(big)))
    maps = 2 * (aligned(4 * 2 * big) - aligned(4 * (big + small)))
    # one set of workspaces; two with the asynchronous flag
    for flags, sets in ((0, 1), (1, 2)):
        assert sequence([big, small], flags) - sequence([big, big], flags) + maps >= sets * more


def test_chain_buffers_hold_every_norm():
    # FP64 levels of up to 256 nodes are squared in 36 tiles of 32 x 32, one norm
    # each, beside the 10 exact norms of level 0 and three vectors of 256
    import paper_1802_05421_amd._lib as L
    off = L.load().cdl_chain_level_offset(256, L.PREC["fp64"])
    assert off >= 3 * aligned(8 * 256) + aligned(8 * 36) + aligned(8 * 10)
