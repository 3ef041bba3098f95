"""CPU check of the rules that deal a launch's work items out to workgroups (csrc/lcsa_attn_form.h), against the measured times
of the launch forms in profiles/: where the rule says so, the other forms are not faster by more than the runs differ."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PAIRS, SPLIT, ALONE = 0, 1, 2


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("form")
    src, lib = tmp / "form.cpp", tmp / "form.so"
    src.write_text('#include "lcsa_attn_form.h"\n'
                   'extern "C" int form(int items, int units, int k) { return lcsa::attn_form(items, units, k); }\n'
                   'extern "C" int few(int items, int units, long long tokens, int blocks) { return lcsa::attn_few(items, units, tokens, blocks); }\n'
                   'extern "C" int bwd_form(int items, int units, int k) { return lcsa::bwd_query_form(items, units, k); }\n'
                   'extern "C" int shares(int items, int units, long long bytes) { return lcsa::append_shares(items, units, bytes); }\n'
                   'extern "C" int workgroups(int form, int items) { return lcsa::attn_workgroups((lcsa::AttnForm)form, items); }\n')
    subprocess.run(["g++", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2510_12747_amd", "csrc"),
                    "-o", str(lib), str(src)], check=True)
    return ctypes.CDLL(str(lib))


def measured():
    """(items, k, {form: us}) of every row of the tables of single geometries"""
    forms = None
    for line in open(os.path.join(ROOT, "profiles", "attn_mfma_kernel_split_and_paired_items.txt")):
        f = line.split()
        if not f:
            forms = None
        elif f[:1] == ["items"]:
            forms = [c for c in f if c in ("alone", "pairs", "split")]
            at = {c: f.index(c) for c in forms + ["k"]}
        elif forms:
            yield int(f[0]), int(f[at["k"]]), {c: float(f[at[c]]) for c in forms}


def test_the_rule_never_picks_a_form_that_was_measured_slower(rule):
    """The rule behind attn_few(): up to 128 items it decides for blocks of few tokens only."""
    names = {PAIRS: "pairs", SPLIT: "split", ALONE: "alone"}
    rows = list(measured())
    assert len(rows) > 150
    for items, k, us in rows:
        form = names[rule.form(items, 256, k)]
        assert us[form] <= 1.03 * min(us.values()), (items, k, form, us)


def test_edges_of_the_rule(rule):
    for units in (1, 32, 256, 304):
        for k in (0, 1, 2, 64, 1 << 24):
            assert rule.form(1, units, k) == rule.form(units, units, k) == (SPLIT if k > 1 else ALONE)
            assert rule.form(units + 1, units, k) == rule.form(2 * units, units, k) == PAIRS      # one round of pairs
            assert rule.form(4 * units, units, k) == PAIRS                                        # 4 rounds against 2
            assert rule.form(1 << 30, units, k) == PAIRS
    # 2 n + 1 rounds split against n + 1 of pairs: the shortest rows that are split
    for n, k in ((1, 6), (2, 12), (3, 19), (4, 27), (5, 36)):
        for items in (2 * n * 256 + 1, (2 * n + 1) * 256):
            assert [rule.form(items, 256, k - 1), rule.form(items, 256, k), rule.form(items, 256, 1 << 30)] == [PAIRS, SPLIT, SPLIT]
        assert rule.form((2 * n + 2) * 256, 256, 1 << 30) == PAIRS        # as many half rounds either way
    assert rule.form(13 * 256, 256, 1 << 30) == PAIRS
    assert [rule.workgroups(f, 7) for f in (PAIRS, SPLIT, ALONE)] == [4, 7, 7]


def table(letter):
    """Rows of numbers of one table of the other launch forms"""
    path = os.path.join(ROOT, "profiles", "launch_forms_few_items_backward_general.txt")
    text = open(path).read().split(f"\n{letter}. ")[1].split("\n\n")[0]
    return [[float(x) for x in line.split()] for line in text.splitlines()[2:]]


def test_two_workgroups_an_item_where_that_was_measured_faster(rule):
    rows = table("A")
    assert len(rows) == 70
    for items, k, pairs, split, alone, few in rows:
        items, k = int(items), int(k)
        us = few if rule.few(items, 256, ctypes.c_longlong(9 * 128), 9) & 1 else {PAIRS: pairs, SPLIT: split, ALONE: alone}[rule.form(items, 256, k)]
        assert us <= 1.04 * min(pairs, split, alone, few), (items, k)


def test_two_workgroups_an_item_over_random_geometries(rule):
    """Means of the ratio to the better form; by the rule 1.008, by always and never taking two workgroups an item 1.017 and 1.115."""
    rows, picked, always, never = table("B"), 1.0, 1.0, 1.0
    assert len(rows) == 400
    for items, k, tokens, largest, split, few in rows:
        best = min(split, few)
        picked *= (few if rule.few(int(items), 256, ctypes.c_longlong(round(tokens * 10)), 10) & 1 else split) / best
        always, never = always * few / best, never * split / best
    assert picked ** (1 / len(rows)) < 1.01 < always ** (1 / len(rows)) < 1.05 < never ** (1 / len(rows))


def test_the_query_side_backward_rule_never_picks_a_form_that_was_measured_slower(rule):
    rows = table("C")
    assert len(rows) > 140
    for items, k, *us in rows:
        assert us[rule.bwd_form(int(items), 256, int(k))] <= 1.04 * min(us), (items, k)


def test_edges_of_the_query_side_backward_rule(rule):
    four, eight, halves = 0, 1, 2
    for units in (32, 256, 304):
        for k in (0, 1, 17, 1 << 24):
            assert [rule.bwd_form(n, units, k) for n in (1, units // 2, units // 2 + 1, units)] == [halves, halves, eight, eight]
            assert [rule.bwd_form(n, units, k) for n in (units + 1, 2 * units, 3 * units + 1, 1 << 30)] == [four] * 4
        for n in (2 * units + 1, 3 * units):
            assert [rule.bwd_form(n, units, k) for k in (0, 16, 17, 1 << 24)] == [four, four, eight, eight]


def test_edges_of_the_rule_for_few_items(rule):
    full = lambda n: rule.few(n, 256, ctypes.c_longlong(9 * 128), 9) & 1
    assert [full(n) for n in (1, 128, 129, 1 << 30)] == [1, 1, 0, 0]
    # grids whose blocks hold few tokens: 1 x 80 in (16, 8) blocks, 26 x 8 in (4, 32), 24 x 8 and 24 x 9 in (8, 16), 21 x 37 in (8, 16)
    for tokens, blocks, few in ((80, 10, 0), (208, 7, 0), (192, 3, 0), (193, 3, 1), (216, 3, 1), (777, 9, 1), (1 << 30, 1 << 24, 0), ((1 << 30) + 1, 1 << 24, 1)):
        assert rule.few(8, 256, ctypes.c_longlong(tokens), blocks) & 1 == few, (tokens, blocks)
    assert rule.workgroups(3, 7) == 14


def test_tiles_share_a_workgroup_of_the_append_where_that_was_measured_faster(rule):
    """Never slower than a tile each by more than the runs differ; means of the ratio to the better form: the rule 1.002, a tile
    each 1.21, four always 1.08."""
    path = os.path.join(ROOT, "profiles", "append_general_tiles_a_workgroup.txt")
    rows, picked, single, four_always = [[float(x) for x in line.split()] for line in open(path) if not line.startswith("#")], 1.0, 1.0, 1.0
    assert len(rows) == 545
    for size, items, _, _, _, one, four in rows:
        us = four if rule.shares(int(items), 256, ctypes.c_longlong(int(size))) & 1 else one
        assert us <= 1.02 * one and (us <= 1.08 * four or size == 49152 or items <= 192), (size, items)
        picked, single, four_always = picked * us / min(one, four), single * one / min(one, four), four_always * four / min(one, four)
    assert picked ** (1 / len(rows)) < 1.003 < 1.05 < four_always ** (1 / len(rows)) < single ** (1 / len(rows))


def test_edges_of_the_sharing_rule(rule):
    kb = lambda n, items: rule.shares(items, 256, ctypes.c_longlong(int(n * 1024))) & 1
    for size, first in ((1, 193), (16, 193), (16.5, 256), (32, 256)):
        assert [kb(size, n) for n in (1, first - 1, first, 1 << 30)] == [0, 0, 1, 1]
    for size, many in ((33, 1), (64, 1), (65, 0), (1024, 0)):
        assert [kb(size, n) for n in (193, 216, 512, 513, 1024, 1025, 1280, 1281, 1 << 30)] == [0, 0, 0, 1, 1, 0, 0, many, many]
    assert [rule.shares(n, 32, ctypes.c_longlong(4096)) & 1 for n in (24, 25)] == [0, 1]
