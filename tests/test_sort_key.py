"""The list build's wrapping and sort key (sort_key.h, compiled here for the host) over every magnitude a
finite coordinate can have: no key and no bucket lies outside the arrays they index."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2011_01207_amd", "csrc")
SOURCE = """
#include "sort_key.h"
extern "C" void keys(int n, const double* pos, const double* box, int ny, int nz, int shift, int nbucket,
                     double* wrapped, unsigned* key, int* bucket)
{
    for (int i = 0; i < n; ++i) {
        double* w = wrapped + 3 * i;
        for (int a = 0; a < 3; ++a)
            w[a] = amoeba::wrap_box(pos[3 * i + a], box[a]);
        key[i] = amoeba::sort_key(w[0], w[1], w[2], box[0], box[1], box[2], ny, nz);
        bucket[i] = amoeba::bucket_of(key[i], shift, nbucket);
    }
}
"""


@pytest.fixture(scope="module", params=[["-ffp-contract=off"], ["-mfma", "-ffp-contract=fast"]], ids=["plain", "fma"])
def host_keys(request, tmp_path_factory):
    """The two ways a compiler may round x - L floor(x / L)."""
    d = tmp_path_factory.mktemp("sort_key")
    src, so = d / "k.cpp", d / "k.so"
    src.write_text(SOURCE)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-D__host__=", "-D__device__=",
                           "-D__forceinline__=inline", *request.param, "-I", CSRC, str(src), "-o", str(so)])
    return ctypes.CDLL(str(so)).keys


@pytest.mark.parametrize("box,ny,nz,npad", [((18.63, 18.63, 18.63), 3, 3, 704), ((98.65, 98.65, 98.65), 12, 12, 96000),
                                            ((205.2, 31.7, 900.0), 255, 1, 128), ((7e-3, 1e5, 64.0), 1, 255, 4096)])
def test_keys_of_every_finite_position_are_in_range(host_keys, box, ny, nz, npad):
    rng = np.random.default_rng(11)
    edges = np.array(box)
    # every magnitude, multiples of the edges and their neighbours, both signs
    mag = 10.0 ** rng.uniform(-320, 308, (60000, 3))
    near = edges * np.floor(10.0 ** rng.uniform(0, 15, (60000, 3)))
    near = np.where(rng.random(near.shape) < 0.5, near, np.nextafter(near, np.inf * rng.choice([-1, 1], near.shape)))
    mid = 10.0 ** rng.uniform(13, 24, (60000, 3))
    special = np.array([0.0, -0.0, 5e-324, -5e-324, -1e-20, 1.7976931348623157e308, -1.7976931348623157e308, 1.0])
    pos = np.concatenate([mag, near, mid, rng.choice(special, (2000, 3))])
    pos *= rng.choice([-1.0, 1.0], pos.shape)
    bad = np.zeros((3, 3))
    bad[0, 0], bad[1, 1], bad[2, 2] = np.nan, np.inf, -np.inf
    pos = np.ascontiguousarray(np.concatenate([pos, bad]))
    nkeys, shift = ny * nz << 12, 0
    while ((nkeys - 1) >> shift) + 2 > npad:
        shift += 1
    nbucket = ((nkeys - 1) >> shift) + 2
    n = len(pos)
    wrapped, key, bucket = np.empty_like(pos), np.empty(n, np.uint32), np.empty(n, np.int32)
    p = ctypes.c_void_p
    host_keys(n, p(pos.ctypes.data), p(edges.ctypes.data), ny, nz, shift, nbucket, p(wrapped.ctypes.data),
              p(key.ctypes.data), p(bucket.ctypes.data))
    assert np.all(key[-3:] == 0xffffffff) and np.all(bucket[-3:] == nbucket - 1)
    pos, wrapped, key, bucket = pos[:-3], wrapped[:-3], key[:-3].astype(np.int64), bucket[:-3]
    assert np.all((wrapped >= 0.0) & (wrapped < edges))
    assert np.all((key >= 0) & (key < nkeys)) and np.all((bucket >= 0) & (bucket < nbucket - 1))
    # ordinary positions stay the plain formula's, to its rounding
    r = np.fmod(pos, edges)
    r = np.where(r < 0.0, r + edges, r)
    gap = np.abs(wrapped - r)
    gap = np.minimum(gap, edges - gap)
    assert np.all(gap <= 2.0 ** -51 * np.maximum(np.abs(pos), edges))
    inside = (pos >= 0.0) & (pos < edges)
    assert np.array_equal(wrapped[inside], pos[inside])
