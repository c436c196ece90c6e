"""Head-tile copies (HND and ROCm pools) at the edges of their dispatch: strips of whole rows, of eight columns, of
equal parts, tiles that fill their waves badly, tiles of any size in an HND pool, slices side by side or one
after another.

Each case runs through the CPU model of the kernels (bounds, every byte written once, bytes equal to the
oracle's) and, on a GPU, through the library against the oracle.
"""
from __future__ import annotations

import pytest

import synthkv
from edgecases import custom

import kernel_model as km
from test_kernel_model import check_model


def _case(layout, heads, dim, elem=2, bs=16, old=(2, 1), new=(1, 2), **kw):
    return layout, custom(num_layers=4, num_kv_heads=heads, head_dim=dim, elem_bytes=elem, old_block_size=bs,
                          new_block_size=kw.pop("new_bs", bs), old_topo=old, new_topo=new, num_seqs=4,
                          length_law=("uniform", 1, 5 * bs), **kw)


CASES = {
    # ROCm: whole rows, eight columns, two equal strips, an unequal last strip, one column of a large block
    "rocm_whole": _case(km.ROCM, 2, 128),
    "rocm_eight": _case(km.ROCM, 4, 128),
    "rocm_equal": _case(km.ROCM, 4, 72),
    "rocm_last": _case(km.ROCM, 2, 152, new_bs=8),
    "rocm_column": _case(km.ROCM, 2, 16, bs=512, elem=1),
    "rocm_fp8": _case(km.ROCM, 2, 128, elem=1, new_bs=32),
    "rocm_f32": _case(km.ROCM, 2, 20, elem=4, bs=4, new_bs=8),
    "rocm_large": _case(km.ROCM, 2, 32, elem=4, bs=128),
    # ROCm: lanes left idle (tile groups)
    "rocm_groups": _case(km.ROCM, 2, 72, new_bs=8),
    "rocm_groups_f32": _case(km.ROCM, 2, 12, elem=4, bs=4),
    # HND: waves that meet one, two, four, eight and any number of tiles
    "hnd_1": _case(km.HND, 4, 128, new=(1, 1)),
    "hnd_2": _case(km.HND, 4, 40, bs=12, new=(1, 1)),
    "hnd_4": _case(km.HND, 4, 40, bs=5, new=(1, 1)),
    "hnd_8": _case(km.HND, 4, 72, bs=1, new=(1, 1)),
    "hnd_any": _case(km.HND, 4, 16, bs=1, new_bs=3, new=(1, 1)),
    # slices of one layer side by side: two and four of them, and too many for one launch
    "peers_2": _case(km.HND, 4, 64, elem=4, bs=8, old=(4, 1), new=(2, 2)),
    "peers_4": _case(km.ROCM, 4, 64, old=(4, 1), new=(1, 1)),
    "peers_4_back": _case(km.ROCM, 4, 64, old=(1, 1), new=(4, 1)),
    "peers_16": _case(km.HND, 16, 64, old=(16, 1), new=(1, 1)),
    "unequal": _case(km.ROCM, 12, 16, old=(4, 1), new=(6, 1)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_model(name):
    layout, w = CASES[name]
    check_model(w, lo=layout, ln=layout)


LOCAL = {   # kept slices between a ROCm pool and another layout: whole rows, eight columns, equal strips, idle lanes
    "whole": (2, 128, 2, 16), "eight": (4, 128, 2, 16), "equal": (4, 72, 2, 16), "groups": (2, 72, 2, 8),
    "fp8": (4, 128, 1, 16), "f32": (4, 64, 4, 8), "column": (2, 16, 1, 512),
}


def _local_case(name):
    heads, dim, elem, bs = LOCAL[name]
    return _case(km.ROCM, heads, dim, elem=elem, bs=bs, old=(2, 1), new=(1, 2))[1]


@pytest.mark.parametrize("lo,ln", [(km.ROCM, km.NHD), (km.NHD, km.ROCM), (km.ROCM, km.HND), (km.HND, km.ROCM)])
@pytest.mark.parametrize("name", list(LOCAL))
def test_model_local(name, lo, ln):
    m = check_model(_local_case(name), local=True, lo=lo, ln=ln)
    kernels = {x.kernel for x in m.local_launches(0, 0, m.L)}
    assert kernels == {"copy_local_tiles" if name == "groups" else "copy_local_strips"}


@pytest.mark.gpu
@pytest.mark.parametrize("lo,ln", [(km.ROCM, km.NHD), (km.NHD, km.ROCM), (km.ROCM, km.HND), (km.HND, km.ROCM)])
@pytest.mark.parametrize("name", list(LOCAL))
def test_gpu_local(name, lo, ln):
    from test_gpu_parity import _local_layouts_case
    _local_layouts_case(_local_case(name), lo, ln, reuse=False)


def test_dispatch_is_reached():
    """The cases take every kernel, every count of tiles per wave and both orders of a layer's slices."""
    seen, strips = set(), set()
    for layout, w in CASES.values():
        m = km.Migration(w, synthkv.make_inputs(w), layout, layout, data=False)
        for pack, ranks, run in ((True, m.old, m.pack_launches), (False, m.new, m.unpack_launches)):
            for r in range(ranks.tp * ranks.pp):
                for x in run(r, 0, m.L):
                    seen.add((pack, x.kernel, x.args.get("n"), x.args.get("peers", 0) > 1))
                    if x.kernel == "copy_strips":
                        strips |= {(x.args["strip"], s.row_bytes // 16) for s in x.args["items"]}
    for pack in (True, False):
        assert {s[1] for s in seen if s[0] == pack} >= {"copy_strips", "copy_tile_groups", "copy_head_rows"}
        assert {s[3] for s in seen if s[0] == pack and s[1] == "copy_strips"} == {True, False}
    assert {s[2] for s in seen if s[1] == "copy_head_rows"} == {0, 1, 2, 4, 8}
    assert any(a == b for a, b in strips) and any(a == 8 < b for a, b in strips) and any(b % a for a, b in strips)


@pytest.mark.parametrize("layout,other", [(km.HND, km.HND), (km.ROCM, km.ROCM), (km.ROCM, km.NHD), (km.NHD, km.ROCM)])
def test_blocks_that_one_launch_cannot_number(layout, other):
    """A slice of 2^31 vectors in each block: more than a dispatch counts work-items for, with K and V.  It goes by ranges
    of heads that adjoin, and every launch has blocks to copy."""
    heads, hb, bs = 1 << 26, 16, 32
    w = custom(num_layers=1, num_kv_heads=heads, head_dim=hb, elem_bytes=1, old_block_size=bs, new_block_size=bs,
               old_topo=(1, 1), new_topo=(1, 1), num_seqs=2, length_law=("fixed", 1))
    m = km.Migration(w, synthkv.make_inputs(w), layout, other, data=False)
    calls = [m.local_launches(0, 0, 1)] if layout != other else [m.pack_launches(0, 0, 1), m.unpack_launches(0, 0, 1)]
    for launches in calls:
        assert all(x.args.get("n_desc", x.args.get("n_new")) == 2 for x in launches)
        parts = [i for x in launches for i in x.args["items"]]
        n = [getattr(i, "head_count", i.row_bytes // hb) for i in parts]
        assert sum(n) == heads and max(n) * bs <= km.MAX_TILE_VECTORS
        for at, lay, row in (("src_k", layout, hb), ("dst_k", other, hb), ("paged_k", other, hb), ("stage", km.NHD, hb)):
            if hasattr(parts[0], at):
                step = row if lay == km.NHD else row * bs
                assert all(getattr(b, at) - getattr(a, at) == k * step for a, b, k in zip(parts, parts[1:], n))
    if layout != other:
        m.copy_local(0, sample=16)
    else:
        m.pack(0, sample=16)
        m.unpack(0, sample=16)


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(CASES))
def test_gpu(name):
    from test_gpu_parity import _layouts_case
    layout, w = CASES[name]
    _layouts_case(w, layout, layout, reuse=False)
    _layouts_case(w, layout, layout, reuse=True)
