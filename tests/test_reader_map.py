"""How the work-groups of several queries per sequence are dealt to the eight XCDs: every one placed once, equal counts, and equal
work also where the queries see different numbers of rows.  reader_map.hpp itself, compiled for the host."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2503_01586_amd", "csrc")


@pytest.fixture(scope="module")
def places(tmp_path_factory):
    d = tmp_path_factory.mktemp("map")
    (d / "m.cpp").write_text('#include "reader_map.hpp"\n'
                             'extern "C" int run(int n, int all) { return ekv::reader_run(n, all); }\n'
                             'extern "C" int place(int b, int all, int run) { return ekv::reader_place(b, all, run, ekv::reader_turns(all, run)); }\n')
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-I", CSRC, str(d / "m.cpp"), "-o", str(d / "m.so")], check=True)
    lib = ctypes.CDLL(str(d / "m.so"))

    def of(all_, readers):
        """places[xcd]: the places of the line that the work-groups of this XCD take, in the order of their start"""
        run = lib.run(readers, all_)
        p = np.array([lib.place(b, all_, run) for b in range((all_ + 7) // 8 * 8)])
        return [[int(v) for v in p[x::8] if v >= 0] for x in range(8)]
    return of


@pytest.mark.parametrize("readers", [3, 4, 5, 8, 15, 16, 17, 40, 129, 1024])
@pytest.mark.parametrize("items", [1, 2, 7, 8, 12, 48, 51, 100])
def test_every_work_group_once_and_equal_counts(places, readers, items):
    got = places(items * readers, readers)
    assert sorted(v for x in got for v in x) == list(range(items * readers))
    counts = [len(x) for x in got]
    assert max(counts) == -(-items * readers // 8)
    # rows are fetched by as few XCDs as the runs allow: a run each, and the eighths of what is left
    fetches = sum(len({v // readers for v in x}) for x in got)
    assert fetches <= items * -(-readers // 16) + 2 * 8


def _share(got, work):
    per_xcd = [sum(work[v] for v in x) for x in got]
    return max(per_xcd) / (sum(per_xcd) / 8)


@pytest.mark.parametrize("T, before", [(257, 0), (300, 0), (504, 0), (512, 0), (700, 0), (2048, 0), (1024, 3072)])
@pytest.mark.parametrize("head_groups", [1, 2])
def test_queries_over_their_own_prompt(places, T, before, head_groups):
    """One split, query t sees before + t + 1 rows; more work-groups than compute units.  Contiguous eighths of the line would
    give the last XCD 1.87 times its share."""
    readers = T * head_groups
    work = [before + v // head_groups + 1 for v in range(readers)]
    assert _share(places(readers, readers), work) <= (1.12 if T <= 512 else 1.04)


@pytest.mark.parametrize("T, splits", [(2, 4), (5, 3), (8, 2), (5, 12)])
def test_a_batch_sorted_by_length(places, T, splits):
    B, readers = 40, T
    work = [(100 + 50 * (v // (splits * readers))) for v in range(B * splits * readers)]
    assert _share(places(len(work), readers), work) <= 1.05
    assert _share(places(len(work), readers), work[::-1]) <= 1.05
