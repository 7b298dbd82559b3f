"""Host side of PackedNet: a pass enqueues the calls that the network, as it is now, stands for.  The library is a
stand-in here: packing returns empty tensors, a chain notes the calls it is given."""
import copy
from types import SimpleNamespace

import pytest
import torch

from paper_2106_12169_amd import binding as B
from paper_2106_12169_amd import workloads as wl
from paper_2106_12169_amd.network import PackedNet

LAYERS = dict(image_hw=64, num_classes=100, widths=(32, 64, 96, 128))


class Chain:
    made = 0
    ran = None

    def __init__(self):
        Chain.made += 1
        self.calls = []

    def __getattr__(self, name):
        return lambda *args: self.calls.append((name, args))

    def __len__(self):
        return len(self.calls)

    def run(self, image):
        Chain.ran = self.calls


@pytest.fixture
def make(monkeypatch):
    monkeypatch.setattr(B, "_N", SimpleNamespace(Chain=Chain, versions=B.native().versions))
    for name in ("apnn_pack", "apnn_pack_input_weights", "apnn_pack_conv_weights"):
        monkeypatch.setattr(B, name, lambda w, bits, enc: torch.zeros(1, dtype=torch.int32))
    monkeypatch.setattr(torch.cuda, "synchronize", lambda: None)

    def net(batch=8, **kw):
        layers = wl.resnet18_layers(**{**LAYERS, **kw})
        return PackedNet(layers, wl.network_params(layers), batch, device="cpu")
    return net


def calls(net):
    net.forward(torch.zeros(1))
    return Chain.ran


def held(calls):
    """Every tensor that a pass hands to the library, by identity."""
    return {id(a) for _, args in calls for a in args if isinstance(a, torch.Tensor)}


def test_a_network_is_recorded_once_while_nothing_changes(make):
    net = make()
    Chain.made = 0
    first = calls(net)
    assert calls(net) is first and Chain.made == 0


@pytest.mark.parametrize("dup", [copy.copy, copy.deepcopy])
@pytest.mark.parametrize("name", ["w", "scale", "bias", "buf"])
def test_networks_that_share_their_tensors_all_see_an_exchange(make, dup, name):
    net = make()
    other = dup(net)
    calls(net), calls(other)
    key = net.layers[2].name
    new = torch.zeros(1)
    for n in (net, other):
        getattr(n, name)[key] = new
        assert id(new) in held(calls(n))
    if dup is copy.copy:
        for first, second in ((net, other), (other, net)):
            new = torch.zeros(1)
            getattr(net, name)[key] = new
            assert id(new) in held(calls(first)) and id(new) in held(calls(second))


@pytest.mark.parametrize("name", ["w", "scale", "bias", "buf"])
def test_an_assigned_dict_stays_the_callers(make, name):
    net = make()
    mine = dict(getattr(net, name))
    setattr(net, name, mine)
    calls(net)
    mine[net.layers[2].name] = new = torch.zeros(1)
    assert id(new) in held(calls(net))


def test_entries_from_a_dict_with_methods_of_its_own_are_asked_for_in_every_pass(make):
    class Latest(dict):
        def __getitem__(self, key):
            return latest if key == "fc" else dict.__getitem__(self, key)
    net = make()
    net.w = Latest(net.w)
    for latest in (torch.zeros(1), torch.zeros(1)):
        assert id(latest) in held(calls(net))
