"""Guard on the generated code of the two dominant kernels (y = x W_eff^T and dx = dy W_eff on 256x256 tiles).

Their main loop uses all 512 vector registers of a lane (256 accumulators, the double-buffered fragments, the
load offsets), and the instruction order inside it is fixed by hand.  A harmless-looking change elsewhere in the
kernel can tip the register allocator into moving the accumulators between the two register files, or into
spilling, inside that loop: every result stays correct and the kernel runs 40 % slower.  No parity test sees that,
so this one compiles the kernel source to assembly (own source, device code only) and checks the loop blocks.
Needs hipcc, not a GPU; takes about a minute."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

KERNELS = {
    # the variants for contractions of whole k-tiles and the general ones, which clear the end of a cut k-tile in LDS
    "gemm_y  <256,256,bf16,A rows x K, B rows x K, whole k-tiles>": "nt_gemm_kernelILi256ELi256ELi0ELb0ELb0ELi2ELb1E",
    "gemm_dx <256,256,bf16,A rows x K, B K x rows, whole k-tiles>": "nt_gemm_kernelILi256ELi256ELi0ELb0ELb1ELi2ELb1E",
    "gemm_y  <256,256,bf16,A rows x K, B rows x K>": "nt_gemm_kernelILi256ELi256ELi0ELb0ELb0ELi2ELb0E",
    "gemm_dx <256,256,bf16,A rows x K, B K x rows>": "nt_gemm_kernelILi256ELi256ELi0ELb0ELb1ELi2ELb0E",
}


def _assembly(tmp_path_factory, source):
    from paper_2405_16528_amd import build as B
    out = tmp_path_factory.mktemp("isa") / (source + ".s")
    flags = [f for f in B.FLAGS if f not in ("-shared", "-fPIC")]
    cmd = [B.hipcc(), *flags, "-S", "--cuda-device-only", "-I", os.path.join(ROOT, "include"),
           os.path.join(B.PKG, "csrc", source), "-o", str(out)]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    return out.read_text()


@pytest.fixture(scope="module")
def assembly_of(tmp_path_factory):
    made = {}

    def of(source):
        if source not in made:
            made[source] = _assembly(tmp_path_factory, source)
        return made[source]
    return of


@pytest.fixture(scope="module")
def assembly(assembly_of):
    return assembly_of("gemm_nt.hip")


@pytest.fixture(scope="module")
def few_assembly(assembly_of):
    return assembly_of("few.hip")


def _loop_blocks(asm, mangled_part):
    start = asm.index(mangled_part)
    start = asm.index("\n", start)
    body = asm[start:asm.index(".Lfunc_end", start)]  # (a function may hold more than one s_endpgm)
    blocks, label, lines = [], "entry", []
    for line in body.split("\n"):
        if re.match(r"^\.LBB\d+_\d+:", line):
            blocks.append((label, lines))
            label, lines = line, []
        else:
            lines.append(line)
    blocks.append((label, lines))
    # LLVM marks the blocks of a loop in the label's comment
    return [(lab, ls) for (lab, ls) in blocks if "Loop" in lab and any("v_mfma" in x for x in ls)]


@pytest.mark.parametrize("name", list(KERNELS))
def test_main_loop_has_no_register_file_traffic(assembly, name):
    loops = _loop_blocks(assembly, KERNELS[name])
    assert loops, "main loop not found"
    text = [x for (_, ls) in loops for x in ls]
    n_mfma = sum("v_mfma_f32_16x16x32_bf16" in x for x in text)
    assert n_mfma == 128, f"{name}: {n_mfma} MFMAs in the loop blocks, expected the 128 of one k-tile"
    moved = [x.strip() for x in text if "v_accvgpr" in x]
    assert not moved, f"{name}: accumulators moved between register files inside the loop: {moved[:3]} ..."
    spilled = [x.strip() for x in text if "scratch_" in x]
    assert not spilled, f"{name}: spills inside the loop: {spilled[:3]} ..."
    # the k-tile's memory instructions: 32 fragment reads (twice as many when B is read transposed) and 16 loads
    n_loads = sum("global_load_lds_dwordx4" in x for x in text)
    assert n_loads == 16, f"{name}: {n_loads} direct loads in the loop blocks, expected 16"
    # M0 is written by the hand-written load sequence only (it cannot be declared as a clobber): every write of M0 in
    # the loop is the s_add of that sequence, followed by the wait state and the load it serves.  (A mask in EXEC between the two
    # holds back the next matrix instruction; neither variant has one.)
    for i, x in enumerate(text):
        if re.search(r"\bm0\b", x) and "s_add_u32 m0" not in x:
            raise AssertionError(f"{name}: M0 used outside the direct-load sequence: {x.strip()}")
        if "s_add_u32 m0" in x:
            assert text[i + 1].strip() == "s_nop 0" and text[i + 2].strip().startswith("global_load_lds_dwordx4"), (name, text[i + 1:i + 3])


@pytest.mark.parametrize("source", ["gemm_nt.hip", "gemm_pair.hip", "gemm_weight.hip", "nf4_tile.hip"])
def test_direct_loads_wait_for_M0(assembly_of, source):
    """gfx950 wants one wait state between a write of M0 and a load that takes its LDS address from there; the compiler puts an
    s_nop into its own code and does not look inside inline assembly.  Every direct load of the library is inline assembly."""
    asm = assembly_of(source)
    since, loads = None, 0  # instructions since the last write of M0 (None: none in this kernel yet)
    for line in asm.split("\n"):
        x = line.split(";")[0].strip()
        if x.startswith("_Z") and x.endswith(":"):
            since = None
        if not re.match(r"(s|v|ds|global|buffer|flat|scratch)_", x):
            continue
        if x.startswith("global_load_lds"):
            loads += 1
            assert since is not None and since >= 1, f"{source}: {x} follows the write of M0 at once"
        if re.match(r"s_\w+ m0\b", x):
            since = 0
        elif since is not None:
            since += 1
    assert loads > 0


def _lds_writes_at_barriers(body):
    """For every s_barrier of a kernel: whether a wave can come there with one of its own LDS writes outstanding, on some path through
    the kernel, and the wait in front of it.  LDS operations of a wave complete in order, so `s_waitcnt lgkmcnt(n)` means that a
    write with n or more LDS operations behind it is in place.  Carried through the branches until nothing changes."""
    blocks, at = [[]], {}
    for line in body.split("\n"):
        x = line.split(";")[0].strip()
        if re.match(r"\.LBB\w+:", x):
            blocks.append([])
            at[x[:-1]] = len(blocks) - 1
        elif re.match(r"(s|ds)_", x):
            blocks[-1].append(x)
            if x.startswith(("s_branch", "s_cbranch", "s_endpgm")):
                blocks.append([])
    in_place = 1 << 20  # else: operations since the last write, the fewest of all paths
    entry, barriers, todo = {0: in_place}, {}, [0]
    while todo:
        i = todo.pop()
        since, follow = entry[i], [i + 1]
        for n, x in enumerate(blocks[i]):
            if x.startswith("ds_write"):
                since = 0
            elif x.startswith("ds_"):
                since = min(since + 1, in_place)
            elif x.startswith("s_waitcnt"):
                left = re.search(r"lgkmcnt\((\d+)\)", x)
                if left and since >= int(left[1]):
                    since = in_place
            elif x.startswith("s_barrier"):
                barriers[i, n] = (since < in_place, blocks[i][n - 1] if n else "")
            elif x.startswith("s_branch"):
                follow = [at[x.split()[1]]]
            elif x.startswith("s_cbranch"):
                follow.append(at[x.split()[1]])
            elif x.startswith("s_endpgm"):
                follow = []
        for j in follow:
            if j < len(blocks) and since < entry.get(j, in_place + 1):
                entry[j] = since
                todo.append(j)
    return list(barriers.values())


def test_lds_writes_are_followed_around_a_loop():
    """A write at the end of a loop, a barrier at its top: 15 reads between them are enough wherever they are, 14 are not."""
    def body(before, behind):
        reads = "\tds_read_b32 v1, v2\n"
        return (f"\ts_nop 0\n.LBB0_1:\n\ts_waitcnt lgkmcnt(15)\n\ts_barrier\n{reads * 20}\tds_write_b128 v1, v[2:5]\n"
                f"{reads * before}\ts_cbranch_scc1 .LBB0_3\n{reads * behind}.LBB0_2:\n\ts_branch .LBB0_1\n.LBB0_3:\n\ts_endpgm\n")
    for before, behind in ((15, 0), (0, 15), (7, 8)):
        assert _lds_writes_at_barriers(body(before, behind)) == [(False, "s_waitcnt lgkmcnt(15)")]
        for less in ((max(before - 1, 0), behind), (before, max(behind - 1, 0))):
            assert _lds_writes_at_barriers(body(*less))[0][0] == (sum(less) < 15)


@pytest.mark.parametrize("source,lenient", [("nf4_tile.hip", 6), ("gemm_nt.hip", 0), ("gemm_pair.hip", 0), ("gemm_weight.hip", 0)])
def test_barriers_come_behind_the_lds_writes(assembly_of, source, lenient):
    """A tile that has been written to LDS is in place at the barrier that publishes it.  nf4_tile.hip goes to the six barriers of its
    form without branches with up to 15 LDS operations outstanding: there 15 reads or more have to be behind the last write, an
    order that nothing in the source forces, also on the way around the loop and into it from the general form."""
    asm, kernels = assembly_of(source), 0
    for m in re.finditer(r"^(_Z\S+):", asm, re.M):
        end = asm.find(".Lfunc_end", m.end())
        if end < 0 or "s_barrier" not in asm[m.end():end]:
            continue
        barriers = _lds_writes_at_barriers(asm[m.end():end])
        assert not [wait for outstanding, wait in barriers if outstanding], m[1]
        assert sum(wait == "s_waitcnt lgkmcnt(15)" for _, wait in barriers) == lenient, m[1]
        kernels += 1
    assert kernels >= 6


def test_few_token_kernels_keep_to_their_registers(few_assembly):
    """16 waves leave 128 registers to a lane.  Only 64 rows of NF4 codes with two token tiles may spill (one round of those is
    still ahead of two rounds of 48 rows), and not more than they do.  Every variant that a launch selects, and no other."""
    spills = {}
    for name, count in re.findall(r"\.name: +(\S*few_(?:tokens|beside)_kernel\S*)\n(?:.*\n)*?.*\.vgpr_spill_count: +(\d+)", few_assembly):
        key = re.search(r"few_(?:tokens_kernelILb(?P<nf4>\d)ELi(?P<t>\d)ELi(?P<n>\d)ELi(?P<to>\d)E|beside_kernelILi(?P<bt>\d)ELi(?P<rt>\d)ELi(?P<ru>\d)E)", name)
        assert key, name
        key = (("beside", *(int(key[k]) for k in ("bt", "rt", "ru"))) if key["bt"]
               else ("NF4" if key["nf4"] == "1" else "bf16", int(key["t"]), int(key["n"]), {"0": "result", "2": "on sums"}[key["to"]]))
        assert key not in spills, name
        spills[key] = int(count)
    expected = {(w, t, n, "result") for w in ("NF4", "bf16") for t in (1, 2) for n in (1, 2, 3, 4)} - {("bf16", t, 4, "result") for t in (1, 2)}
    # the rank-r term on top of the weight's sums, and U beside the weight: of 64 rows of the weight with one token tile only
    expected |= {("NF4", t, n, "on sums") for t in (1, 2) for n in (1, 2, 3, 4)} - {("NF4", 2, 4, "on sums")}
    expected |= {("beside", t, *n) for t in (1, 2) for n in ((1, 1), (2, 1), (3, 1), (3, 2), (4, 1), (4, 2)) if t == 1 or n[0] < 4}
    assert set(spills) == expected, set(spills) ^ expected
    assert spills.pop(("NF4", 2, 4, "result")) <= 20
    assert not any(spills.values()), spills


@pytest.mark.parametrize("source", ["gemm_nt.hip", "gemm_pair.hip", "gemm_weight.hip", "nf4_tile.hip"])
def test_main_loops_keep_to_their_registers(assembly_of, source):
    """The blocks of every product's main loop, also of the eight-wave forms (256 registers to a lane): nothing goes to scratch memory
    and no accumulator moves.  Outside of them the 256x256 tiles alone spill, set-up and change of segment, and not more than they
    do: with eight waves up to 19 registers (fold, merge, unquantised merge, grouped merge), 2 with four."""
    asm = assembly_of(source)
    spills = {name: int(count) for name, count in re.findall(r"\.name: +(_Z\S+)\n(?:.*\n)*?.*\.vgpr_spill_count: +(\d+)", asm)}
    kernels = 0
    for name, count in spills.items():
        loops = _loop_blocks(asm, "\n" + name + ":")
        if not loops:
            continue
        kernels += 1
        moved = [x.strip() for _, lines in loops for x in lines if "scratch_" in x or "v_accvgpr" in x]
        assert not moved, (name, moved[:3])
        eight = "grouped_kernelILi256E" in name or re.search(r"nt_gemm_kernelILi256ELi256E.*ELi8EEE", name)
        assert count <= (19 if eight else 2 if "nt_gemm_kernelILi256ELi256E" in name else 0), (name, count)
    assert kernels >= 6


@pytest.mark.parametrize("source", ["gemm_nt.hip", "gemm_pair.hip", "gemm_weight.hip", "nf4_tile.hip"])
def test_main_loops_wait_for_loads_by_hand_only(assembly_of, source):
    """The direct loads of a k-tile are counted and waited for by hand.  Where a kernel also has loads into registers, on another
    branch, the compiler may take it that they are still on their way and wait for all loads in every k-tile."""
    asm, kernels = assembly_of(source), 0
    for m in re.finditer(r"^(_Z\S+):", asm, re.M):
        if ".Lfunc_end" not in asm[m.end():]:
            continue  # (a constant)
        loops = _loop_blocks(asm, "\n" + m[1] + ":")
        if not loops:
            continue
        kernels += 1
        for _, lines in loops:
            by_hand = False
            for x in lines:
                by_hand = "#ASMSTART" in x or (by_hand and "#ASMEND" not in x)
                assert by_hand or not ("s_waitcnt" in x and "vmcnt" in x), (m[1], x.strip())
    assert kernels >= 6


@pytest.mark.parametrize("source,kernel", [("codec.hip", "nf4_dequantize_kernel"), ("gemm_pair.hip", "nt_copy_kernel")])
def test_streaming_kernels_keep_out_of_scratch_memory(assembly_of, source, kernel):
    """The expansions of codes with rows that end inside a group of eight, and their neighbours: an array indexed at run time
    would live in scratch memory, and every group would go through it."""
    size = dict(re.findall(r"\.name: +(_Z\S+)\n(?:.*\n)*?.*\.private_segment_fixed_size: +(\d+)", assembly_of(source)))
    assert any(kernel in k for k in size)
    assert not {k: n for k, n in size.items() if int(n)}


def test_no_kernel_that_nothing_launches(assembly):
    """Slices of a product whose left operand is stored rows x K are planned on tiles of 256x128 and less only."""
    assert "nt_gemm_kernelILi256ELi128ELi1ELb0E" in assembly  # (the name the next line would find)
    assert "nt_gemm_kernelILi256ELi256ELi1ELb0E" not in assembly
