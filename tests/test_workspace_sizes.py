"""The workspace a call gets when none is given (host arithmetic; the tensors are
host tensors)."""
import os

import pytest
import torch

import paper_2602_05774_amd as vsd
from paper_2602_05774_amd import _lib
from paper_2602_05774_amd.vsd import _workspace

pytestmark = pytest.mark.skipif(not os.path.exists(_lib.LIB_PATH), reason="libvsd.so not built")
BF = torch.bfloat16


@pytest.mark.parametrize("rows,Vd,Vt", ((4, 256, 256), (1280, 32000, 128256), (21760, 1000, 5000)))
def test_fused_head_takes_the_best_size(rows, Vd, Vt):
    """The tiles' states are up to 64 MiB, the KL lists of at most 256 runs x 256 rows up to 4.5 MB more."""
    prob = vsd.Problem(1, rows, 1, 1, Vd, Vt)
    head = vsd.LmHead(torch.zeros(4, 64, dtype=BF), torch.zeros(256, 64, dtype=BF))
    need, best = vsd.score_workspace_needed_bytes(prob, BF, 64), vsd.score_workspace_bytes(prob, BF, 64)
    assert need < best <= need + (69 << 20)
    assert _workspace(prob, head, None).numel() == best


def test_a_given_workspace_is_taken_from_the_needed_size_on():
    prob = vsd.Problem(1, 4, 2, 3, 100, 200)
    need, best = vsd.score_workspace_needed_bytes(prob, BF), vsd.score_workspace_bytes(prob, BF)
    X = torch.zeros(prob.R, 104, dtype=BF)
    assert need < best  # few paths: verification's result slots
    for size in (need, best):
        given = torch.empty(size, dtype=torch.uint8)
        assert _workspace(prob, X, given) is given
    assert _workspace(prob, X, torch.empty(need - 1, dtype=torch.uint8)).numel() == best
    many = vsd.Problem(1, 4, 512, 3, 100, 200)
    assert vsd.score_workspace_needed_bytes(many, BF) == vsd.score_workspace_bytes(many, BF)
