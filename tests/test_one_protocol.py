"""When a list of protocols counts as one protocol for all devices."""
import numpy as np
import pytest

from paper_2511_09413_amd import _one_protocol

A = ([0.0, 1.0], [1.0, -1.0])
ARR = (np.array([0.0, 1.0]), np.array([1.0, -1.0]))


@pytest.mark.parametrize("protocols,one", [
    ([A, A], True), ([A, ([0.0, 1.0], [1.0, -1.0])], True), ([ARR, ARR], True),
    ([A, ([0.0, 1.0], [1.0, -1.5])], False), ([A, A, ([0.0], [1.0])], False),
    ([ARR, (ARR[0].copy(), ARR[1])], False), ([A, ARR], False), ([ARR, A], False),
    ([([0.0], [float("nan")]), ([0.0], [float("nan") * 1])], False),
    ([([0.0], [1.0]), ([np.array([0.0, 2.0])], [1.0])], False), ([A, ((0.0, 1.0), (1.0, -1.0))], False)])
def test_one_protocol(protocols, one):
    assert _one_protocol(protocols) is one
