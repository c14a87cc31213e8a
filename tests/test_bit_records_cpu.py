"""Site records of the bit-held sweep (bits_host.cpp) decoded on the host: every
site's field from its record equals sum_j J_ij m_j + h_i, for every record form
(dense cubes in aligned and unaligned rows, sides of two with their double bonds,
fields, zero couplings, graphs with odd groups and sites of up to 15 terms), and
sites of more terms are refused."""
import shutil
import subprocess
from pathlib import Path

import numpy as np
import pytest

import synth

ROOT = Path(__file__).resolve().parent.parent
CUBE4, CUBE, GENERAL = 0, 1, 2


@pytest.fixture(scope="module")
def decoder(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("host compiler not available")
    exe = tmp_path_factory.mktemp("bits") / "bit_records"
    csrc = ROOT / "paper_2510_23419_amd" / "csrc"
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + str(csrc),
                    "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    str(ROOT / "tests" / "helpers" / "bit_records.cpp"), str(csrc / "bits_host.cpp"), "-o", str(exe)],
                   check=True)
    return exe


def _decode(exe, n, bi, bj, bJ, h, groups, lx, seed):
    rows = [[] for _ in range(n)]
    for a, b, j in zip(bi.tolist(), bj.tolist(), bJ.tolist()):
        rows[a].append((b, j))
        rows[b].append((a, j))
    start = np.cumsum([0] + [len(r) for r in rows])
    m = synth.random_spins(1, n, seed)[0]
    h = np.zeros(n, int) if h is None else h
    flat = [x for r in rows for x in r]
    text = " ".join(map(str, [n, int(groups.max()) + 1, lx, len(flat)])) + "\n"
    for v in (start, [x[0] for x in flat], [x[1] for x in flat], h, groups, m):
        text += " ".join(map(str, v)) + "\n"
    out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, (out.returncode, out.stderr)
    if out.stdout.startswith("refused"):
        return None
    head, fields = out.stdout.strip().split("\n")
    want = [sum(j * int(m[b]) for b, j in rows[i]) + int(h[i]) for i in range(n)]
    assert list(map(int, fields.split())) == want
    return tuple(map(int, head.split()))


@pytest.mark.parametrize("dims,field,zeros,form", [
    ((2, 2, 2), "zero", 0.0, CUBE), ((4, 2, 2), "zero", 0.0, CUBE4), ((8, 6, 4), "zero", 0.0, CUBE4),
    ((12, 2, 6), "zero", 0.0, CUBE4), ((6, 6, 6), "zero", 0.0, CUBE), ((10, 4, 2), "zero", 0.0, CUBE),
    ((8, 4, 4), "uniform3", 0.0, GENERAL), ((6, 4, 2), "zero", 0.3, GENERAL), ((4, 4, 4), "uniform3", 0.3, GENERAL)])
def test_cube_records(decoder, dims, field, zeros, form):
    inst = synth.ea_instance(dims, seed=sum(dims), field=field)
    inst["J"] = (inst["J"] * (np.random.default_rng(1).random(inst["J"].shape) >= zeros)).astype(np.int8)
    g = synth.ea_bond_list(inst)
    n = g["n"]
    i = np.arange(n)
    colour = (i % dims[0] + i // dims[0] % dims[1] + i // (dims[0] * dims[1])) % 2
    head = _decode(decoder, n, g["bond_i"], g["bond_j"], g["bond_J"], g["h"], colour, dims[0], seed=3)
    assert head[0] == form and head[1] == n and head[2] == 0


def _star_graph(n, hub_terms, seed):
    """Hubs of the given numbers of bonds to later vertices, hubs in group 0."""
    rng = np.random.default_rng(seed)
    bi, bj = [], []
    k = len(hub_terms)
    for a, t in enumerate(hub_terms):
        for b in rng.choice(np.arange(k, n), size=t, replace=False):
            bi.append(a)
            bj.append(int(b))
    bJ = np.where(rng.random(len(bi)) < 0.5, 1, -1).astype(np.int8)
    groups = (np.arange(n) >= k).astype(int)
    return np.array(bi), np.array(bj), bJ, groups


@pytest.mark.parametrize("terms,h,wide", [([7, 3, 1], 0, 0), ([8], 0, 1), ([7, 7, 2], 1, 1), ([15, 8, 9], 0, 2),
                                          ([15, 4, 2, 0, 9], 0, 1), ([16], 0, None), ([15], 1, None)])
def test_graph_records(decoder, terms, h, wide):
    """Wide pairs begin at eight terms (a field is a term), odd groups are padded, and a
    site of more than 15 terms is refused."""
    n = 61
    bi, bj, bJ, groups = _star_graph(n, terms, seed=sum(terms))
    hv = np.zeros(n, int)
    hv[:len(terms)] = h
    head = _decode(decoder, n, bi, bj, bJ, hv, groups, 0, seed=5)
    if wide is None:
        assert head is None
    else:
        assert head[0] == GENERAL and head[2] == wide
