"""The workspace a call gets when none is given: the needed size, and more only
where the call uses it (host arithmetic; the tensors are host tensors)."""
import os

import pytest
import torch

import paper_2602_05774_amd as vsd
from paper_2602_05774_amd import _lib
from paper_2602_05774_amd.vsd import _workspace

pytestmark = pytest.mark.skipif(not os.path.exists(_lib.LIB_PATH), reason="libvsd.so not built")
BF = torch.bfloat16


def test_fused_head_with_the_kl_term_takes_the_needed_size():
    prob = vsd.Problem(1, 4, 1, 1, 256, 256)
    head = vsd.LmHead(torch.zeros(4, 64, dtype=BF), torch.zeros(256, 64, dtype=BF))
    need, best = vsd.score_workspace_needed_bytes(prob, BF, 64), vsd.score_workspace_bytes(prob, BF, 64)
    assert need < best
    assert _workspace(prob, head, None, vsd.Params()).numel() == best
    assert _workspace(prob, head, None, vsd.Params(kl_weight=0.1, kl_topk=4)).numel() == need


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
