"""The threaded jump chain of the register-weight kernel's walk, checked in
the compiled code object (host-side, no GPU): the leaves of every walk sit at
the stride its address arithmetic assumes, each leaf reads its own lane, adds
each of its taps once to the right accumulator, and ends in the jump to the
next set bit; the sentinel leaves lead to the next ballot's table or out.  A
wrong stride would send a nonzero into the middle of another leaf."""
import os
import re
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

from paper_1704_07724_amd import build as B  # noqa: E402

sys.path.insert(0, B.CSRC)
import gen_dispatch as G  # noqa: E402

LLVM = "/opt/rocm/llvm/bin"
FIND = ["s_ff1_i32_b64", "s_bitset0_b64", "s_mulk_i32", "s_add_u32", "s_addc_u32"]


def walks(text):
    """{site: {label: [(address, mnemonic, operands)]}} in order of address."""
    sites, cur = {}, None
    for line in text.splitlines():
        m = re.match(r"^([0-9a-f]+) <(.+)>:", line)
        if m:
            w = re.match(r"(W\d+)_(base|q\d+)$", m.group(2))
            cur = sites.setdefault(w.group(1), {}).setdefault(w.group(2), []) if w else None
            if w:
                sites[w.group(1)].setdefault("at", {})[w.group(2)] = int(m.group(1), 16)
            continue
        m = re.match(r"^\s+(\S+)\s*([^/]*)//\s*([0-9A-F]+):", line)
        if m and cur is not None:
            cur.append((int(m.group(3), 16), m.group(1), [o.strip() for o in m.group(2).split(",")]))
    return sites


def number(s):
    return int(s, 0)


@pytest.mark.parametrize("R", [1, 3, 5])
def test_walk_tables_exact(tmp_path, R):
    if not os.path.exists(B.HIPCC) or not os.path.exists(os.path.join(LLVM, "llvm-objdump")):
        pytest.skip("ROCm toolchain not available")
    B.generate()
    src = tmp_path / "walks.hip"
    tiles = [(t + (1,))[:5] + (0,) for t in G.WALK_TILES + G.RING_TILES if t[0] == R]
    tiles += [t + (1, 1) for t in G.GRAD_TILES if t[0] == R]
    tiles += [t + (2,) for t in G.STRIDED_TILES if t[0] == R]  # 2: not the gradient's, stride 2
    src.write_text('#include "sparse_tile.hpp"\n' + "\n".join(
        """__global__ __launch_bounds__(64) void k_{1}_{2}_{3}_{4}_{5}(const float *x, float *y) {{
    using W = isc::tile::{6}<{0}, {1}, {2}, {3}, {4}{7}>;
    unsigned long long m[W::kChunks];
    float v[W::kChunks], acc[{1} * {2} * {4}], w[{0} * {0} * {4}];
    for (int i = 0; i < W::kChunks; ++i) {{ v[i] = x[i * 64 + threadIdx.x]; m[i] = __ballot(v[i] != 0.0f); }}
    for (int i = 0; i < {0} * {0} * {4}; ++i) w[i] = x[4096 + i * 64 + threadIdx.x];
    for (int i = 0; i < {1} * {2} * {4}; ++i) acc[i] = x[16384 + i * 64 + threadIdx.x];
    W::run(m, v, acc, w);
    for (int i = 0; i < {1} * {2} * {4}; ++i) y[i * 64 + threadIdx.x] = acc[i];
    for (int i = 0; i < {0} * {0} * {4}; ++i) y[32768 + i * 64 + threadIdx.x] = w[i];
}}""".format(*t, "AsmGradWalk" if t[5] == 1 else "AsmWalk", ", 2" if t[5] == 2 else "") for t in tiles))
    obj = str(tmp_path / "walks.o")
    subprocess.run([B.HIPCC] + B.DEVICE_FLAGS + ["--offload-device-only", "--no-gpu-bundle-output", "-c", str(src),
                                                 "-o", obj], check=True, capture_output=True)
    text = subprocess.run([os.path.join(LLVM, "llvm-objdump"), "-d", "--mcpu=gfx950", obj], check=True,
                          capture_output=True, text=True).stdout
    parts = re.split(r"(?m)^[0-9a-f]+ <_Z\S*k_(\d+)_(\d+)_(\d)_(\d)_(\d)\S*>:", text)
    found = {}
    for i in range(1, len(parts), 6):
        s = walks(parts[i + 5])
        assert len(s) == 1
        found[(R, int(parts[i]), int(parts[i + 1]), int(parts[i + 2]), int(parts[i + 3]), int(parts[i + 4]))] = next(iter(s.values()))
    assert sorted(found) == sorted(tiles)
    for tile, site in found.items():
        check_walk(*tile, site)


def check_walk(R, TH, TW, same, kpl, kind, site):
    what = (R, TH, TW, same, kpl, kind)
    grad, T = kind == 1, max(1, kind)
    pos = G.walk_positions(R, TH, TW, same, T)
    nq = len(pos)
    chunks = -(-nq // G.WALK_CHUNK)
    counts = [min(G.WALK_CHUNK, nq - e * G.WALK_CHUNK) for e in range(chunks)]
    base = site["base"]
    at = {int(k[1:]): a for k, a in site["at"].items() if k[0] == "q"}
    q0 = at[0]
    assert [i[1] for i in base[:8]] == ["s_add_u32", "s_addc_u32"] + FIND + ["s_setpc_b64"], what
    assert base[0][0] + number(base[0][2][-1]) == q0, what
    stride = number(base[4][2][-1])
    masks = {0: base[2][2][1]}
    acc, wreg, xreg = {}, {}, {}
    tbl, nxt = base[5][2][1], base[7][2][0]
    labels = [64 * e + l for e in range(chunks) for l in range(counts[e] + 1 if e == chunks - 1 else 64)]
    assert sorted(at) == labels, what
    for i in labels:
        e, l = divmod(i, 64)
        ins = site.get("q%d" % i, [])
        assert at[i] == q0 + i * stride, (what, i)
        ends = [k for k, t in enumerate(ins) if t[1] == "s_setpc_b64"]
        body = ins[:ends[0] + 1] if ends else ins
        names = [t[1] for t in body]
        assert not ends or body[-1][0] + 4 <= q0 + (i + 1) * stride, (what, i)
        if l == counts[e]:
            if e == chunks - 1:  # out of the walk: none of its code follows
                assert i == labels[-1], (what, i)
                continue
            assert names == ["s_add_u32", "s_addc_u32"] + FIND + ["s_setpc_b64"], (what, i)
            assert body[0][2][:2] == [tbl, tbl] and number(body[0][2][2]) == 64 * stride, (what, i)
            assert number(body[4][2][-1]) == stride and body[2][2][1] == body[3][2][0], (what, i)
            masks[e + 1] = body[2][2][1]
            continue
        taps = [(a * kpl + j, k * kpl + j) for a, k in G.leaf_fmas(R, TH, TW, *pos[e * G.WALK_CHUNK + l], T)
                for j in range(kpl)]
        fmas = [t for t in body if t[1] == "v_fmac_f32_e32"]
        find = [t for t in body if t[1] in FIND]
        assert [t[1] for t in find] == FIND and len(body) == 7 + len(taps), (what, i)
        assert names[0] == "v_readlane_b32" and names[-1] == "s_setpc_b64" and names[1] in FIND and names[2] in FIND
        v, xr, lane = body[0][2]
        assert number(lane) == l and xreg.setdefault(e, xr) == xr, (what, i)
        assert find[0][2][1] == masks[e] and find[1][2][0] == masks[e], (what, i)
        assert number(find[2][2][-1]) == stride and find[3][2][1] == tbl and body[-1][2][0] == nxt, (what, i)
        for t, (a, k) in zip(fmas, taps):
            ra, rw = (t[2][2], t[2][0]) if grad else (t[2][0], t[2][2])
            assert t[2][1] == v and acc.setdefault(a, ra) == ra and wreg.setdefault(k, rw) == rw, (what, i)
    assert len(set(masks.values())) == chunks and len(set(xreg.values())) == chunks, what
    assert len(set(acc.values())) == TH * TW * kpl and len(set(wreg.values())) == R * R * kpl, what
    assert not set(acc.values()) & (set(wreg.values()) | set(xreg.values())), what
