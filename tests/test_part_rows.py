"""Local copies that re-block, by one or two old blocks a wave, by more, and by lane, of rows that go by whole vectors, by
8-byte words and by vectors at any address.

Each case runs through the CPU model of the kernels (bounds, every byte written once, bytes equal to the
oracle's) and, on a GPU, through the library against the oracle.
"""
from __future__ import annotations

import pytest

import synthkv
from edgecases import custom

import kernel_model as km
from test_kernel_model import check_model


# (head bytes, old block, new block): rows from one old block, two, many; waves that meet one new block to many
BLOCKS = ((256, 64, 20), (256, 16, 1), (256, 1, 16), (512, 3, 64), (1024, 16, 128), (64, 16, 64), (64, 64, 16), (64, 2, 2),
          (16, 8, 8), (16, 16, 1), (16, 16, 64), (16, 16, 96), (128, 1, 1), (200, 64, 20), (200, 20, 64), (72, 7, 5), (100, 3, 40), (33, 16, 4), (36, 32, 16), (256, 16, 16), (200, 20, 20), (64, 4, 4))
REBLOCK = {f"{hb}_{bo}_{bn}": custom(num_layers=2, num_kv_heads=4, head_dim=hb, elem_bytes=1, old_block_size=bo,
                                     new_block_size=bn, num_seqs=4, length_law=("uniform", 1, 150), old_topo=(2, 1),
                                     new_topo=(4, 1)) for hb, bo, bn in BLOCKS}


@pytest.mark.parametrize("name", list(REBLOCK))
def test_model_reblock(name):
    check_model(REBLOCK[name], local=True)


def test_dispatch_is_reached():
    """The cases take every kind of word and every way in which a wave finds its rows' sources."""
    local = set()
    for w in REBLOCK.values():
        m = km.Migration(w, synthkv.make_inputs(w), data=False)
        for r in range(min(m.old.tp, m.new.tp)):
            local |= {(x.args["n"], x.args["m"], x.args["vec"]) for x in m.local_launches(r, 0, m.L)}
    assert {v for _, _, v in local} == {16, 8, 0}
    assert {(n, m) for n, m, _ in local} >= {(0, 1), (1, 1), (1, 2), (2, 1), (2, 2), (4, 1), (4, 0), (1, 0), (2, 0)}


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(REBLOCK))
def test_gpu_reblock(name):
    from test_gpu_parity import check_against_oracle
    check_against_oracle(REBLOCK[name], synthkv.make_inputs(REBLOCK[name]), local=True, log_name=name)
