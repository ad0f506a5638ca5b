"""A network without layers: an optimizer step has nothing to update."""
from paper_2501_04194_amd import mlp


def test_adam_of_no_layers():
    net = mlp.BF16MLP([4], "cpu")
    net.adam([], [])
    assert net.step_count == 1 and net.W == []
