"""The layers that the GPU tests of the staged convolutions run are staged, and in the form that their override names.  An override that does
not apply to a layer is declined without an error and another kernel answers, so a test of a form could pass without it: here the host code
of the launcher (conv_halo.hip) is asked, with stand-ins for the kernels (tests/sanitize/conv_halo_driver.cpp)."""
import shutil
import subprocess

import pytest

from paper_2106_12169_amd import binding as B
from tests import test_gpu_conv_halo as base
from tests import test_gpu_conv_halo_forms as forms
from tests.test_sanitizers import CSRC, ROOT, _host_program

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")


@pytest.fixture(scope="module")
def layouts(tmp_path_factory):
    """(override, layer, whether int32 results) -> what the launcher asks for, or None."""
    tmp = tmp_path_factory.mktemp("staged")
    exe = _host_program(tmp, "layouts", [f"{CSRC}/conv_halo.hip", f"{ROOT}/tests/sanitize/conv_halo_driver.cpp"])

    def ask(cases):
        lines = []
        for force, layer, ints in cases:
            BS, Cin, Cout, H, W, R, S, stride, pad, encW, p, encX, q, q_out, q_res, pool = layer
            lines.append((BS, H, W, Cin, Cout, R, S, stride, pad, int(encW == B.ENC_PM1), p, int(encX == B.ENC_PM1), q, pool, int(ints), q_out, q_res, force))
        path = tmp / "layers.txt"
        path.write_text("\n".join(" ".join(map(str, line)) for line in lines) + "\n")
        r = subprocess.run([exe, str(path)], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-3000:]
        out = []
        for line in r.stdout.splitlines():
            words = line.split()
            out.append(dict(zip(words[1::2], map(int, words[2::2]))) if words[0] == "1" else None)
        assert len(out) == len(lines)
        return out
    return ask


def _as_layer(BS, Cin, Cout, H, W, R, p, encW, q):
    return (BS, Cin, Cout, H, W, R, R, 1, R // 2, encW, p, base.U, q, 2, 0, 0)


def _in_form(force, pool, got):
    """3, 4: eight waves; 5, 6: bits; 7, 8: codes; the even ones twice the pixels."""
    assert got is not None
    tile = 2 if force % 2 == 0 else 1
    assert got["fp"] == (tile + 2 if pool else tile)
    assert got["pairs"] == (2 if force in (3, 4) else 1)
    if force > 2:
        assert got["packed"] == (force in (5, 6))


def test_forced_forms_are_what_runs(layouts):
    cases = [(f, layer, False) for f in (1, 2) for layer in base.LAYERS] + [(f, layer, False) for f, layer in forms.FORMS]
    cases += [(f, forms.short_layer(*s), False) for f, s in forms.SHORT_FORMS]
    cases += [(f, _as_layer(*layer), True) for f, layer in forms.INT_FORMS]
    for (force, layer, _), got in zip(cases, layouts(cases)):
        _in_form(force, layer[-1], got)


def test_every_kind_of_eight_wave_block_runs(layouts):
    cases = [(f, layer, False) for f, layer in forms.FORMS if f in (3, 4)]
    kinds = {(got["kind"], got["stay"], layer[1] % 256 == 0) for (_, layer, _), got in zip(cases, layouts(cases))}
    assert kinds == {(kind, stay, wide) for kind in (0, 1, 3) for stay in (0, 1) for wide in (False, True)}      # features, weights, their loads
    pooled = {(layer[-1], got["stay"]) for (_, layer, _), got in zip(cases, layouts(cases)) if layer[-1]}
    assert pooled == {(1, 0), (1, 1), (2, 0), (2, 1)}


def test_walked_layers_walk(layouts):
    cases = [(f, layer, False) for f, _, layer in forms.WALKS]
    for (force, buffers, layer), got in zip(forms.WALKS, layouts(cases)):
        _in_form(force, layer[-1], got)
        assert got["stay"] and got["step"] < got["tilesM"] and got["buffers"] == buffers
    assert {(f in (3, 4), buffers, bool(layer[-1])) for f, buffers, layer in forms.WALKS} >= {(True, b, pool) for b in (1, 2) for pool in (False, True)}


def test_several_digits_are_read_in_pairs_where_three_blocks_share_a_unit(layouts):
    """Steps in pairs up to 768 tiles, or where LDS leaves room for three blocks a compute unit; else one by one with four."""
    layer = (2, 32, 64, 1130, 60, 1, 1, 1, 0, base.P, 1, base.U, 5, 2, 0, 0)          # 1060 tiles
    few = (1, *layer[1:])
    large = (2, 96, 64, 1130, 60, 3, 3, 1, 1, base.P, 1, base.U, 5, 2, 0, 0)
    got = layouts([(5, layer, False), (5, few, False), (5, large, False), (7, (2, 64, 64, 56, 56, 3, 3, 1, 1, base.P, 1, base.U, 2, 2, 0, 0), False)])
    assert [g["three"] for g in got] == [0, 1, 1, 0]
    assert got[2]["tilesM"] > 768 and 4 * -(-got[2]["lds"] // 1280) > 128


def test_short_sums_come_without_the_table(layouts):
    """Granules (two steps; one where bits stay, in larger tiles and in pooled ones) of the sums: one, two and three of each."""
    cases = [(f, forms.short_layer(*s), False) for f, s in forms.SHORT_FORMS if f > 2]
    seen = set()
    for (force, layer, _), got in zip(cases, layouts(cases)):
        one = (got["packed"] and not got["three"]) or got["fp"] > 1
        entries = got["steps"] * ((layer[12] + 1) // 2)
        seen.add((bool(one), min(entries if one else (entries + 1) // 2, 3)))
    assert seen == {(one, n) for one in (False, True) for n in (1, 2, 3)}
