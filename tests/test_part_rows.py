"""Parts of token rows that are not whole 16-byte vectors, packed, unpacked and copied locally: 8-byte words, vectors at any
address, whole rows to a wave and rows that a wave's end cuts, at the edges of each; and local copies that re-block, by
one or two old blocks a wave, by more, and by lane.

Each case runs through the CPU model of the kernels (bounds, every byte written once, bytes equal to the
oracle's) and, on a GPU, through the library against the oracle.
"""
from __future__ import annotations

import pytest

import synthkv
from edgecases import custom

import kernel_model as km
from test_kernel_model import check_model


def _parts(head_bytes, bs=16, new_bs=None, back=False, tokens=None):
    """Six one-byte-element heads: three to a rank on one side, two on the other, so that slices are one or two of them."""
    topos = [(2, 1), (3, 1)]
    return custom(num_layers=2, num_kv_heads=6, head_dim=head_bytes, elem_bytes=1, old_block_size=bs,
                  new_block_size=new_bs or bs, num_seqs=4, length_law=("uniform", 1, tokens or 5 * bs + 3),
                  old_topo=topos[back], new_topo=topos[not back])


# one head / two heads: under a word, words, both sides of the limits of 256 and 512 bytes, of half a wave of vectors,
# addresses of 4, 2 and 1 bytes
SIZES = ((8, 3), (24, 1), (72, 16), (120, 5), (128 + 8, 16), (248, 16), (256, 3), (264, 2), (504, 2), (520, 3),
         (4, 16), (12, 2), (36, 16), (100, 24), (260, 3), (516, 2), (2, 8), (34, 16), (17, 4), (33, 16), (129, 4), (1031, 4))
CASES = {f"{hb}_{bs}{'_back' if back else ''}": _parts(hb, bs, back=back) for hb, bs in SIZES for back in (False, True)}

# (head bytes, old block, new block): rows from one old block, two, many; waves that meet one new block to many
BLOCKS = ((256, 64, 20), (256, 16, 1), (256, 1, 16), (512, 3, 64), (1024, 16, 128), (64, 16, 64), (64, 64, 16), (64, 2, 2),
          (16, 8, 8), (16, 16, 1), (16, 16, 64), (16, 16, 96), (128, 1, 1), (200, 64, 20), (200, 20, 64), (72, 7, 5), (100, 3, 40), (33, 16, 4), (36, 32, 16), (256, 16, 16), (200, 20, 20), (64, 4, 4), (256, 1, 1),
          (272, 7, 1), (496, 64, 1), (512, 16, 1), (128, 16, 6), (128, 16, 8), (256, 2, 3), (384, 3, 2))
# rows of whole ranks: look-ups by row (64 to 1008 bytes a block, 4 to 63 vectors a row), and rows too short for it
WHOLE = ((64, 1, 1), (64, 5, 5), (64, 12, 15), (80, 8, 8), (144, 16, 4), (336, 3, 3), (1008, 2, 1), (48, 16, 16), (1024, 1, 1))
REBLOCK = {f"{hb}_{bo}_{bn}": custom(num_layers=2, num_kv_heads=4, head_dim=hb, elem_bytes=1, old_block_size=bo,
                                     new_block_size=bn, num_seqs=4, length_law=("uniform", 1, 150), old_topo=(2, 1),
                                     new_topo=(4, 1)) for hb, bo, bn in BLOCKS}
REBLOCK.update({f"whole_{hb}_{bo}_{bn}": custom(num_layers=2, num_kv_heads=2, head_dim=hb, elem_bytes=1, old_block_size=bo,
                                                new_block_size=bn, num_seqs=4, length_law=("uniform", 1, 150),
                                                old_topo=(2, 1), new_topo=(2, 1)) for hb, bo, bn in WHOLE})


@pytest.mark.parametrize("name", list(CASES))
def test_model(name):
    check_model(CASES[name])
    check_model(CASES[name], local=True)


@pytest.mark.parametrize("name", list(REBLOCK))
def test_model_reblock(name):
    check_model(REBLOCK[name], local=True)


def test_dispatch_is_reached():
    """The cases take every kind of word and every shape of a wave, packed, unpacked and local."""
    seen, local, rows = set(), set(), set()
    for w in list(CASES.values()) + list(REBLOCK.values()):
        m = km.Migration(w, synthkv.make_inputs(w), data=False)
        for pack, ranks, run in ((True, m.old, m.pack_launches), (False, m.new, m.unpack_launches)):
            for r in range(ranks.tp * ranks.pp):
                seen |= {(pack, x.args["shape"], x.args["vec"]) for x in run(r, 0, m.L) if x.kernel == "copy_runs"}
        for r in range(min(m.old.tp, m.new.tp)):
            local |= {(x.args["n"], x.args["m"], x.args["vec"]) for x in m.local_launches(r, 0, m.L)
                      if x.kernel == "copy_local"}
            rows |= {i.row_bytes for x in m.local_launches(r, 0, m.L) if x.kernel == "copy_local_rows" for i in x.args["items"]}
    assert seen >= {(True, "cut", 8), (True, "cut", 0), (False, "rows", 8), (False, "rows", 0), (False, "cut", 0)}
    assert {v for _, _, v in local} == {16, 8, 0} and rows == {64, 80, 128, 144, 256, 384}
    assert {(n, m) for n, m, _ in local} >= {(0, 1), (1, 1), (1, 2), (2, 1), (2, 2), (4, 1), (4, 0), (1, 0), (2, 0)}


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(CASES))
def test_gpu(name):
    from test_gpu_parity import check_against_oracle
    check_against_oracle(CASES[name], synthkv.make_inputs(CASES[name]), log_name=name)
    check_against_oracle(CASES[name], synthkv.make_inputs(CASES[name]), local=True, log_name=name + " local")


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(REBLOCK))
def test_gpu_reblock(name):
    from test_gpu_parity import check_against_oracle
    check_against_oracle(REBLOCK[name], synthkv.make_inputs(REBLOCK[name]), local=True, log_name=name)
