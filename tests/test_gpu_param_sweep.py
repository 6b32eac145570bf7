"""The shipped network on the held-out clouds of the shipped sweep (measured
times of every grid): it gains on them, and no pick costs a cloud noticeably
more than the default rule."""
import os

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
PKG = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_06255_amd")


def test_held_out_picks():
    from paper_2606_06255_amd import param_model as pm
    d = np.load(os.path.join(PKG, "param_sweep.npz"), allow_pickle=False)
    total = d["N"].shape[0] - 1                    # the last is the dense cloud
    held = slice(total - total // 11, total)       # ten in eleven were trained on
    model = pm.ParamModel(torch.device("cuda:0"))
    r = pm.evaluate(model.net, d["X"][held], d["MS"][held], d["N"][held], model.margin)
    print("%d clouds: gain %.3f, worst %.3f" % (len(r["clouds"]), r["gain_vs_default"], r["worst_vs_default"]))
    assert r["gain_vs_default"] >= 1.05
    assert r["worst_vs_default"] <= 1.05
