"""Launch shapes of the tile kernel (csrc/hb_tile_shape.h), compiled for the
host: what the kernel derives from a shape stays inside its LDS and keeps the
alignment that its stores are declared with, and the search that every call
makes finds what trying everything finds."""
import ctypes
import itertools
import math
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2010_04804_amd", "csrc")
LDS, CUS = 160 * 1024, 256

SOURCE = r"""
#include "hb_tile_shape.h"
extern "C" {
void shape(int n_trees, int n_cols, int n_outputs, int levels, int tree_bytes, int rank, int n_thr, int steps,
           long long n_rows, int ids, long long ws_bytes, int lds_max, int cus, int *out) {
  const hb::TileSpec t{n_trees, n_cols, n_outputs, levels, tree_bytes, rank != 0, n_thr, steps};
  const hb::TileShape s = hb::best_shape(t, n_rows, ids != 0, ws_bytes, lds_max, cus);
  const int v[] = {s.rows, s.split, s.parts, s.nt, s.ilp, s.bufs, s.st_chunks, s.buf_off, s.stage_off, s.lds, s.tried};
  for (int i = 0; i < 11; ++i) out[i] = v[i];
}
int flush_tree(int k, int st) { return hb::tile_flush_tree(k, st); }
int slot_stride(int rows) { return (int)hb::tile_slot_stride(rows); }
int store_align() { return hb::kTileIdStoreAlign; }
int pad_trees(int tree_bytes) { return hb::tile_pad_trees(tree_bytes); }
}
"""
FIELDS = ["rows", "split", "parts", "nt", "ilp", "bufs", "st_chunks", "buf_off", "stage_off", "lds", "tried"]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("tile_shape")
    (d / "shape.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(d / "shape.so"),
                    str(d / "shape.cpp")], check=True)
    return ctypes.CDLL(str(d / "shape.so"))


# model kind: levels, bytes per tree, rank tile, thresholds per (column, tree)
TREES = {"perfect5": (5, 256, False, 0), "perfect8": (8, 2048, False, 0), "perfect9": (9, 4096, False, 0),
         "perfect11": (11, 16384, False, 0), "rank8": (8, 1024, True, 255), "rank12": (12, 16384, True, 4095),
         "leafwise31": (12, 496, False, 0), "leafwise256": (12, 4096, False, 0)}


def spec(kind, T, F, K):
    levels, tree_bytes, rank, per_tree = TREES[kind]
    n_thr = T * per_tree if rank else 0
    steps = F * max(1, (max(n_thr // F, 1)).bit_length()) if rank else 0
    return (T, F, K, levels, tree_bytes, int(rank), n_thr, steps)


def best(lib, kind, T, F, K, n, ids, ws):
    out = (ctypes.c_int * 11)()
    lib.shape(*spec(kind, T, F, K), ctypes.c_longlong(n), int(ids), ctypes.c_longlong(ws), LDS, CUS, out)
    return dict(zip(FIELDS, out))


CASES = [(k, T, F, K, n, ws) for k, T, F, K, (n, ws) in itertools.product(
    TREES, (4, 60, 100, 300, 800, 3500), (10, 28, 60, 130, 300), (1, 2, 7),
    ((1100, 1 << 30), (8000, 1 << 30), (16_000, 1 << 20), (50_021, 0), (100_003, 0), (1_000_000, 0)))]


def flush_sizes(s, T):
    """Trees per flush: full groups of chunks, and the groups that end a
    workgroup's part of the trees."""
    chunks = -(-T // s["nt"])
    per = s["split"] or chunks
    out = set()
    for begin in range(0, chunks, per):
        end, c = min(begin + per, chunks), begin
        while c < end:
            m = min(s["st_chunks"], end - c)
            out.add((c * s["nt"], min(m * s["nt"], T - c * s["nt"])))
            c += m
    return out


def test_leaf_id_flush_reads_its_staging_and_stores_aligned(lib):
    """Each lane of a flush takes four consecutive trees: the slots it reads
    are staged ones (the second staging buffer ends the kernel's LDS), and its
    16-byte stores begin at ids that the declared alignment allows. Many
    shapes have flushes that start at no multiple of four trees."""
    align, odd = lib.store_align(), 0
    for kind, T, F, K, n, ws in CASES:
        s = best(lib, kind, T, F, K, n, True, ws)
        if not s["rows"]:
            continue
        st = s["st_chunks"] * s["nt"]
        stride = lib.slot_stride(s["rows"])
        label = (kind, T, F, K, n, s)
        assert st <= 32 and s["lds"] <= LDS, label
        for t0, m in flush_sizes(s, T):
            assert 1 <= m <= st, label
            last = max(lib.flush_tree(4 * lane + j, m) for lane in range(8) for j in range(4) if 4 * lane < m)
            end = s["stage_off"] + st * stride + last * stride + 2 * (s["rows"] - 1) + 2
            assert last < m and end <= s["lds"], label
            if T % 4 == 0:  # rows of the output are 16-byte aligned
                odd += t0 % 4 != 0
                assert 4 * t0 % align == 0, label
    assert odd > 0  # such shapes are reached


def everything(kind, T, F, K, n, ids, ws):
    """The shape of the least estimated time, every chunk size and every split tried."""
    T, F, K, levels, tb, rank, n_thr, steps = spec(kind, T, F, K)
    best, least = None, 0.0
    for lg in range(7 if rank else 6, 11):
        R, G = 1 << lg, 1024 >> lg
        rw, buf = R // 64, -(-F * R * (2 if rank else 4) // 16) * 16
        tiles = -(-n // R)
        ranks = 0.22 * n_thr + 11.0 * steps * rw if rank else 0.0
        load = 2000.0 + 3.0 * F * rw + ranks if ws else ranks
        for bufs, ilp in itertools.product((2, 1), (1, 2, 3, 4, 8)):
            for nt in range(G * ilp, (32 if ids else 64) + 1, G * ilp):
                stage = buf + bufs * nt * tb
                if nt * tb > 65536 or stage + (2 * nt * (2 * R + 4) if ids else 0) > LDS:
                    break
                chunks = -(-T // nt)
                walk = nt * levels * rw * max(7.0 + 1.0 / ilp, 260.0 / (16 * ilp))
                hand = 1300.0 + nt * tb / 40.0 + (700.0 + nt * tb / 64.0 if bufs == 1 else 0.0)
                cost, split, parts = -(-tiles // CUS) * (chunks * (walk + hand) + load), 0, 1
                for per in range(1, chunks if ws and tiles < CUS else 1):
                    p = -(-chunks // per)
                    if p * n * K * 8 <= ws:
                        c = math.ceil(tiles * p / CUS) * (per * (walk + hand) + load) + 10000.0
                        if c < cost:
                            cost, split, parts = c, per, p
                if best is None or cost < least * 0.999:
                    best, least = (R, split, parts, nt, ilp, bufs), cost
    return best


def test_search_finds_the_shape_and_stays_short(lib):
    """Every call searches its shape: the search is exact, and the estimates it
    makes do not grow with the trees (trying everything takes about 30 a tree)."""
    keys = ("rows", "split", "parts", "nt", "ilp", "bufs")
    for kind, T, F, K, n, ids, ws in [
            (k, T, F, K, n, ids, ws) for k, (T, F, K), (n, ws), ids in itertools.product(
                TREES, ((1, 5, 1), (37, 60, 2), (100, 130, 1), (500, 28, 7)),
                ((1025, 1 << 30), (4000, 1 << 16), (8000, 32 << 20), (16_384, 1 << 30), (50_021, 0), (300_007, 0)),
                (False, True))]:
        s = best(lib, kind, T, F, K, n, ids, ws)
        want = everything(kind, T, F, K, n, ids, ws)
        assert want == (tuple(s[k] for k in keys) if s["rows"] else None), (kind, T, F, K, n, ids, ws)
    for kind, T, F, n, ids in itertools.product(TREES, (1, 100, 3500, 20_000), (1, 28, 130),
                                                (1025, 2000, 4000, 8000, 16_384, 1_000_000), (False, True)):
        s = best(lib, kind, T, F, 1, n, ids, (1 << 30) if n <= 16_384 else 0)
        assert s["tried"] <= 1200, (kind, T, F, n, ids, s)


def test_chunks_stay_inside_the_padded_tables(lib):
    """The tables hold tile_pad_trees trees past the last one: the last chunk of
    every shape ends inside them."""
    for kind, T, F, K, n, ws in CASES:
        for ids in (False, True):
            s = best(lib, kind, T, F, K, n, ids, ws)
            if s["rows"]:
                assert -(-T // s["nt"]) * s["nt"] <= T + lib.pad_trees(TREES[kind][1]), (kind, T, F, K, n, ids, s)
    assert [lib.pad_trees(b) for b in (16, 1024, 1040, 32768, 65520, 65536)] == [64, 64, 63, 2, 1, 1]
