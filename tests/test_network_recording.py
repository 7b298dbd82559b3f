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


def described(calls):
    """The calls with tensors left out: descriptors and scalars."""
    return [(name, [a for a in args if not isinstance(a, torch.Tensor)]) for name, args in calls]


def test_a_changed_batch_is_the_batch_of_the_next_pass(make):
    net = make(8)
    calls(net)
    net.batch = 3
    assert described(calls(net)) == described(calls(make(3)))
    net.batch = 8
    assert described(calls(net)) == described(calls(make(8)))


@pytest.mark.parametrize("how", ["field", "dict", "entry", "list", "by name", "subclass"])
def test_a_changed_layer_is_the_layer_of_the_next_pass(make, how):
    net = make()
    i = next(i for i, L in enumerate(net.layers) if L.res)
    if how == "subclass":                                # whose fields may come from anywhere
        class Scaled(wl.NetLayer):
            res_scale = property(lambda self: scale, lambda self, value: None)
        scale = 0.0
        net.layers[i] = Scaled(**vars(net.layers[i]))
    calls(net)
    scale = 7.25
    if how == "field":
        net.layers[i].res_scale = scale
    elif how == "dict":
        vars(net.layers[i])["res_scale"] = scale
    elif how in ("entry", "list"):
        new = copy.copy(net.layers[i])
        new.res_scale = scale
        if how == "entry":
            net.layers[i] = new
        else:
            net.layers = tuple(new if L is net.layers[i] else L for L in net.layers)
    elif how == "by name":                               # the source of a residual connection tells its bits
        L = net.layers[i]
        net._by_name[L.res] = src = copy.copy(net._by_name[L.res])
        src.q_out = scale
    assert any(scale in args for _, args in described(calls(net)))


def test_a_changed_tail_is_the_tail_of_the_next_pass(make):
    net = make()
    assert [name for name, _ in calls(net)][-1] == "sumpool_fc"
    net.fused_tail = None
    assert [name for name, _ in calls(net)][-2:] == ["sumpool", "layer"] and net.launches == len(Chain.ran)


def test_a_network_without_a_recording_makes_one(make):
    net = make()
    old = copy.copy(net)
    old.__dict__.pop("_recording")                       # as stored when passes were not recorded
    assert described(calls(old)) == described(calls(net))
