"""bench.py reports recorded HBM traffic only for the kernel sources that it was measured on:
the hashed text holds the kernels that the timed launches run and the rules that choose them."""
import json
import os

import bench

KERNELS = {"schur_gemm": ["void zgemm_kernel(", "void zgemm_tile("],
           "panel": ["void panel_stream_kernel(", "void panel_kernel(", "bool panel_shape(", "ld_agent("]}


def text(sources):
    out = ""
    for name, start, end in sources:
        with open(os.path.join(bench.CSRC, name)) as f:
            t = f.read()
        a = t.index(start) if start else 0
        out += t[a:t.index(end, a) if end else len(t)]
    return out


def test_hash_covers_the_timed_kernels():
    assert sorted(KERNELS) == sorted(bench.TRAFFIC)
    for which, (_, sources, _) in bench.TRAFFIC.items():
        for k in KERNELS[which]:
            assert k in text(sources), (which, k)


def test_records_name_the_sources_they_hash():
    """A record that applies was taken on the text that is hashed now."""
    for fname, sources, overlap in bench.TRAFFIC.values():
        with open(os.path.join(bench.ROOT, "profiles", fname)) as f:
            rec = json.load(f)
        assert rec["lu_overlap"] == overlap
        if rec["kernel_source_sha256_16"] == bench.kernel_hash(sources):
            assert [(x["file"], x["from"], x["to"]) for x in rec["kernel_source"]] == [tuple(s) for s in sources]
