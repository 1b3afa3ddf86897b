"""Generate dispatch_gen.hpp: the computed-jump dispatch of the register-tile
sparse kernels (one output map per lane), as inline assembly.

A nonzero input at window row wy and shifted column xp of a TH x TW output
tile adds v * w[r][s] to acc[wy - r][xp - s] for every filter tap (r, s)
whose output lands in the tile (ISC step 2, Sec. "Sparse Convolution").
The C++ form of this is a binary tree of scalar branches over the leaf key
q = wy * WCOLS + xp; here each leaf is a straight-line block of v_fmac_f32
instructions aligned to a fixed power-of-two stride, and the dispatch jumps
straight to leaf q:  s_getpc, two 64-bit adds, s_setpc -- about seven scalar
instructions per nonzero instead of two per tree level.  The key is clamped
to the table, so no input can send the jump outside it.

    python gen_dispatch.py OUT.hpp

writes a header with a specialisation of isc::tile::AsmDispatch<R, TH, TW>
for every shape the kernels instantiate.
"""
import sys

# every one-map-per-lane tile the kernels instantiate: TH x TW <= 64
SHAPES = [(R, TH, TW) for R in (1, 3, 5) for TW in (8, 16, 28) for TH in (1, 2, 4, 8) if TH * TW <= 64]


def leaf_fmas(R, TH, TW, wy, xp, T=1):
    """(output, tap) pairs a nonzero at window row wy, column xp meets."""
    out = []
    for r in range(R):
        oy, odd = divmod(wy - r, T)
        if odd or not 0 <= oy < TH:
            continue
        for s in range(R):
            ox, odd = divmod(xp - s, T)
            if not odd and 0 <= ox < TW:
                out.append((oy * TW + ox, r * R + s))
    return out


def specialisation(R, TH, TW):
    wrows, wcols = TH + R - 1, TW + R - 1
    nq = wrows * wcols
    maxf = max(len(leaf_fmas(R, TH, TW, q // wcols, q % wcols)) for q in range(nq))
    stride_log2 = 2
    while (1 << stride_log2) < 4 * (maxf + 1):   # FMAs (4 bytes each) + the branch back
        stride_log2 += 1
    lines = [
        '"s_min_u32 s92, %[key], {}\\n"'.format(nq - 1),
        '"s_lshl_b32 s92, s92, {}\\n"'.format(stride_log2),
        '"s_getpc_b64 s[90:91]\\n"',
        '"L%=_base:\\n"',
        '"s_add_u32 s90, s90, L%=_q0-L%=_base\\n"',
        '"s_addc_u32 s91, s91, 0\\n"',
        '"s_add_u32 s90, s90, s92\\n"',
        '"s_addc_u32 s91, s91, 0\\n"',
        '"s_setpc_b64 s[90:91]\\n"',
    ]
    for q in range(nq):
        body = "".join(" v_fmac_f32_e32 %[a{}], %[v], %[w{}]\\n".format(a, w)
                       for a, w in leaf_fmas(R, TH, TW, q // wcols, q % wcols))
        lines.append('".p2align {}\\n" "L%=_q{}:\\n{} s_branch L%=_end\\n"'.format(stride_log2, q, body))
    lines.append('"L%=_end:\\n"')
    na, nw = TH * TW, R * R
    outs = ", ".join('[a{0}] "+v"(acc[{1}][{2}][0])'.format(i, i // TW, i % TW) for i in range(na))
    ins = ", ".join('[w{0}] "v"(w[{1}][{2}][0])'.format(i, i // R, i % R) for i in range(nw))
    asm = "\n            ".join(lines)
    return '''template <>
struct AsmDispatch<{R}, {TH}, {TW}> {{
    static constexpr bool kAvailable = true;
    // {nq} leaves of at most {maxf} FMAs, stride {stride} bytes
    static __device__ __forceinline__ void run(int key, int vbits, float (&acc)[{TH}][{TW}][1],
                                               const float (&w)[{R}][{R}][1]) {{
        asm volatile(
            {asm}
            : {outs}
            : [key] "s"(key), [v] "s"(vbits), {ins}
            : "s90", "s91", "s92", "scc");
    }}
}};
'''.format(R=R, TH=TH, TW=TW, nq=nq, maxf=maxf, stride=1 << stride_log2, asm=asm, outs=outs, ins=ins)


# ---- the whole walk of a window as one threaded jump chain ----------------
#
# Tiles of the register-weight kernel: (R, TH, TW, SAME).  SAME 1: padding
# R/2 on a map at most TW wide, where the window's columns outside the tile
# are all padding and are left out; 2: the same for the rows too (the tile
# holds the whole map); 0: every window position.
WALK_TILES = [(R, TH, TW, 0) for R in (1, 3, 5) for TH, TW in ((4, 8), (2, 8), (3, 16), (2, 16), (1, 16))]
WALK_TILES += [(R, TH, TW, 0) for R in (1, 3) for TH, TW in ((8, 8), (6, 16))]
WALK_TILES += [(1, TH, TW, 0) for TH, TW in ((7, 7), (7, 14), (5, 14), (3, 14))]
WALK_TILES += [(R, TH, TW, 1) for R in (3, 5) for TH, TW in ((4, 8), (4, 13), (4, 14), (3, 14), (3, 16))]
WALK_TILES += [(3, TH, TW, 1) for TH, TW in ((7, 13), (5, 13), (3, 13), (7, 14), (5, 14), (6, 16))]
WALK_TILES += [(R, 7, 7, 2) for R in (3, 5)] + [(3, 8, 8, 2)]
# Tiles of the filter-ring kernel: (R, TH, TW, 0, KPL).
RING_TILES = [(5, TH, TW, 0, 1) for TH, TW in ((9, 9), (7, 14), (5, 14), (3, 14))] + [(5, 1, 28, 0, 2)]
RING_TILES += [(3, TH, 14, 0, 1) for TH in (7, 4, 2)] + [(3, 4, 14, 0, 2)]
RING_TILES += [(1, TH, 14, 0, 1) for TH in (4, 2)] + [(1, 4, 14, 0, 2)]  # 7 x 14: WALK_TILES
# The same at stride 2.
STRIDED_TILES = [(3, 4, 7, 0, 1), (3, 4, 7, 0, 2), (3, 2, 7, 0, 1), (5, 4, 7, 0, 1), (5, 4, 7, 0, 2), (5, 2, 7, 0, 1),
                 (1, 4, 14, 0, 1), (1, 4, 14, 0, 2), (1, 2, 14, 0, 1)]
# Tiles of the weight-gradient kernel: (R, TH, TW, SAME).
GRAD_TILES = [(3, 7, 13, 1), (3, 7, 14, 1), (3, 7, 7, 2), (3, 7, 14, 0), (3, 4, 16, 0), (3, 2, 16, 0), (5, 7, 7, 2),
              (5, 9, 9, 0), (5, 4, 14, 0), (5, 2, 14, 0), (1, 7, 7, 0), (1, 7, 14, 0), (1, 2, 14, 0)]
WALK_CHUNK = 63  # window positions per ballot; the next bit is the sentinel
WALK_HEAD = 32   # bytes of a leaf besides its FMAs: lane read (8), five scalar instructions (20), the jump (4)


def walk_positions(R, TH, TW, same, T=1):
    """(window row, window column) of each position, in order; at stride T > 1
    a 1x1 filter's window holds only the rows and columns it reads."""
    if T > 1:
        step = T if R < T else 1
        return [(wy, xp) for wy in range(0, (TH - 1) * T + R, step) for xp in range(0, (TW - 1) * T + R, step)]
    rows = range(R // 2, R // 2 + TH) if same == 2 else range(TH + R - 1)
    cols = range(R // 2, R // 2 + TW) if same else range(TW + R - 1)
    return [(wy, xp) for wy in rows for xp in cols]


def walk_specialisation(R, TH, TW, same, kpl=1, grad=False, T=1):
    """AsmWalk<R, TH, TW, SAME, KPL, T> (AsmGradWalk with grad): every set bit of the window's ballots, in order.

    Leaf q (chunk q / 64, lane q % 64 of that ballot) reads its nonzero's
    value from its lane, finds the next set bit, computes that bit's leaf
    address between its FMAs, and jumps there: one jump and five scalar
    instructions per nonzero.  The bit after a chunk's last position is always
    set; its leaf starts the next chunk or falls out of the walk, so every
    jump lands on a leaf.
    """
    pos = walk_positions(R, TH, TW, same, T)
    nq = len(pos)
    epl = -(-nq // WALK_CHUNK)
    maxf = kpl * max(len(leaf_fmas(R, TH, TW, wy, xp, T)) for wy, xp in pos)
    stride = max(WALK_HEAD + 4 * maxf, 36 if epl > 1 else 0)

    def find_next(e):
        return [" s_ff1_i32_b64 s46, %[m{}]".format(e), " s_bitset0_b64 %[m{}], s46".format(e),
                " s_mulk_i32 s46, {}".format(stride), " s_add_u32 s48, s44, s46", " s_addc_u32 s49, s45, 0"]

    # forward: a (the tile's outputs) += x * w; gradient: w += x * a
    fma = " v_fmac_f32_e32 %[w{1}], s47, %[a{0}]" if grad else " v_fmac_f32_e32 %[a{0}], s47, %[w{1}]"
    jump = [" s_setpc_b64 s[48:49]"]
    lines = [" s_getpc_b64 s[44:45]", "W%=_base:", " s_add_u32 s44, s44, W%=_q0-W%=_base", " s_addc_u32 s45, s45, 0"]
    lines += find_next(0) + jump
    for e in range(epl):
        last = e == epl - 1
        n = min(WALK_CHUNK, nq - e * WALK_CHUNK)
        for l in range(n):
            wy, xp = pos[e * WALK_CHUNK + l]
            fmas = [fma.format(a * kpl + j, w * kpl + j)
                    for a, w in leaf_fmas(R, TH, TW, wy, xp, T) for j in range(kpl)]
            nx = find_next(e)
            # the scalar chain between the FMAs; two instructions between the
            # lane read and the first use of its scalar
            body = [" v_readlane_b32 s47, %[x{}], {}".format(e, l)] + nx[:2]
            for i in range(2, 5):
                body += fmas[i - 2:i - 1] + [nx[i]]
            body += fmas[3:] + jump
            assert sorted(body) == sorted(body[:1] + nx + fmas + jump)
            size = WALK_HEAD + 4 * len(fmas)
            lines += ["W%=_q{}:".format(e * 64 + l)] + body
            if size < stride:
                lines.append(" .fill {}, 4, 0xbf800000".format((stride - size) // 4))
        lines.append("W%=_q{}:".format(e * 64 + n))
        if not last:  # the sentinel: the next chunk's table and first bit
            assert n == WALK_CHUNK
            lines += [" s_add_u32 s44, s44, {}".format(64 * stride), " s_addc_u32 s45, s45, 0"]
            lines += find_next(e + 1) + jump
            if stride > 36:
                lines.append(" .fill {}, 4, 0xbf800000".format((stride - 36) // 4))
    na, nw = TH * TW * kpl, R * R * kpl
    asm = "\n            ".join('"%s\\n"' % l for l in lines)
    ro, rw = ('"v"', '"+v"') if grad else ('"+v"', '"v"')
    tile = ["[a{0}] {1}(acc[{0}])".format(i, ro) for i in range(na)]
    taps = ["[w{0}] {1}(w[{0}])".format(i, rw) for i in range(nw)]
    outs = ", ".join((taps if grad else tile) + ['[m{0}] "+s"(mask[{0}])'.format(e) for e in range(epl)])
    ins = ", ".join((tile if grad else taps) + ['[x{0}] "v"(x[{0}])'.format(e) for e in range(epl)])
    return '''template <>
struct {name}<{R}, {TH}, {TW}, {same}, {kpl}{strt}> {{
    static constexpr bool kReg = {reg};  // a tile of the register-weight kernel
    // {nq} positions: window rows from {r0}, {nc} columns from {c0}, kStep apart
    static constexpr int kRow0 = {r0}, kCol0 = {c0}, kCols = {nc}, kStep = {step}, kPositions = {nq}, kChunks = {epl};
    // leaves of at most {maxf} FMAs, stride {stride} bytes
    static __device__ __forceinline__ void run(unsigned long long (&mask)[{epl}], const float (&x)[{epl}],
                                               {ca}float (&acc)[{na}], {cw}float (&w)[{nw}]) {{
        asm volatile(
            {asm}
            : {outs}
            : {ins}
            : "s44", "s45", "s46", "s47", "s48", "s49", "scc");
    }}
}};
'''.format(R=R, TH=TH, TW=TW, same=same, epl=epl, nq=nq, maxf=maxf, stride=stride, na=na, nw=nw, asm=asm, outs=outs,
           ins=ins, kpl=kpl, name="AsmGradWalk" if grad else "AsmWalk", ca="const " if grad else "",
           cw="" if grad else "const ",
           reg="true" if kpl == 1 and T == 1 and (R, TH, TW, same) in WALK_TILES else "false", r0=pos[0][0], c0=pos[0][1], step=pos[1][1] - pos[0][1],
           nc=(pos[-1][1] - pos[0][1]) // (pos[1][1] - pos[0][1]) + 1, strt="" if grad else ", %d" % T)



def main(out_path):
    parts = ['''// Generated by gen_dispatch.py -- computed-jump dispatch of the register-tile
// sparse kernels (one output map per lane).  Do not edit.
#pragma once

namespace isc {
namespace tile {

template <int R, int TH, int TW>
struct AsmDispatch {
    static constexpr bool kAvailable = false;
};

''']
    for R, TH, TW in SHAPES:
        parts.append(specialisation(R, TH, TW))
    parts.append('''template <int R, int TH, int TW, int SAME, int KPL = 1, int T = 1>
struct AsmWalk {
    static constexpr bool kReg = false;
};

''')
    parts.append("template <int R, int TH, int TW, int SAME, int KPL = 1>\nstruct AsmGradWalk;\n\n")
    for tile in GRAD_TILES:
        parts.append(walk_specialisation(*tile, grad=True))
    for tile in WALK_TILES + RING_TILES:
        parts.append(walk_specialisation(*tile))
    for tile in STRIDED_TILES:
        parts.append(walk_specialisation(*tile, T=2))
    parts.append('''}  // namespace tile
}  // namespace isc
''')
    text = "\n".join(parts)
    try:
        if open(out_path).read() == text:
            return
    except OSError:
        pass
    with open(out_path, "w") as f:
        f.write(text)


if __name__ == "__main__":
    main(sys.argv[1])
