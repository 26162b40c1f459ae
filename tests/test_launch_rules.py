"""Host checks of what an attention launch takes for granted (csrc/bd_rules.h): the rules themselves, compiled for the CPU,
and the registers and LDS of the kernels in the built library, read from their metadata.  No GPU."""
import glob
import os
import re
import shutil
import subprocess

import pytest

from paper_2503_18773_amd import binding as B

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2503_18773_amd", "csrc")
LLVM = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin")
VGPRS, LDS = 512, 160 * 1024   # of a SIMD, per lane; of a compute unit

needs_gxx = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
needs_kernels = pytest.mark.skipif(not os.path.exists(B._LIB_PATH) or not os.path.exists(os.path.join(LLVM, "llvm-readelf")),
                                   reason="needs the built library and the LLVM tools")


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rules") / "launch_rules_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, os.path.join(HERE, "host", "launch_rules_check.cpp"),
                    "-o", exe], check=True)
    return lambda *q: subprocess.run([exe, *map(str, q)], capture_output=True, text=True, check=True).stdout.splitlines()


@pytest.fixture(scope="module")
def resident(tmp_path_factory):
    """{mangled kernel name: workgroups of 256 threads that a compute unit holds}"""
    where = tmp_path_factory.mktemp("objects")
    shutil.copy(B._LIB_PATH, where)
    subprocess.run([os.path.join(LLVM, "llvm-objdump"), "--offloading", os.path.basename(B._LIB_PATH)], cwd=where, check=True,
                   capture_output=True)
    found = {}
    for obj in glob.glob(str(where / "*gfx950")):
        notes = subprocess.run([os.path.join(LLVM, "llvm-readelf"), "--notes", obj], capture_output=True, text=True, check=True).stdout
        for kernel in notes.split("- .agpr_count:")[1:]:
            name, = re.findall(r"^    \.name: +(\S+)", kernel, re.M)
            vgprs, = re.findall(r"^    \.vgpr_count: +(\d+)", kernel, re.M)
            lds, = re.findall(r"^    \.group_segment_fixed_size: +(\d+)", kernel, re.M)
            granules = (int(vgprs) + 7) // 8 * 8
            found[name] = min(VGPRS // max(granules, 8), LDS // max(int(lds), 1))
    assert len(found) > 60, sorted(found)
    return found


@needs_gxx
@needs_kernels
def test_kernels_are_as_many_on_a_unit_as_their_launch_counts_on(rules, resident):
    """Where two of an instance's workgroups share a compute unit, the order of a ragged batch puts them in layers."""
    seen = 0
    for name, held in resident.items():
        mx = re.search(r"(?:decode|step)_mxg?_kernelI(?:Li(\d+)E)?Lb([01])E", name)
        grp = re.search(r"(?:decode|step)_grp_kernelILi(\d)ELi(\d+)ELi(\d+)ELb[01]ELb([01])E", name)
        integer = re.search(r"(?:decode|step)_int_kernelILi\d+ELi(\d+)ELi(\d)E", name)
        most = 2
        if mx:
            said, = rules("mx", mx.group(1) or 4, mx.group(2))
        elif grp:
            said, = rules("grp", *grp.groups())
        elif integer:
            said, = rules("int", *integer.groups())
            most = 3
        else:
            continue
        seen += 1
        assert int(said) == min(held, most), f"{name}: {held} on a compute unit, launched as {said}"
    # 6 of MXFP4; 2 bits x 2 groups x 2 head counts x 2 K modes x paged or not of the groups; 2 bits x 3 head counts x 2 K
    # modes x paged and the three forms; and the paged ones once more that raise the lengths
    assert seen == 6 + 32 + 48 + 3 + 16 + 12
    # workgroups of 512 threads: one, which is what their rule counts on
    wide = [held for name, held in resident.items() if "wide_int_kernel" in name]
    assert [held // 2 for held in wide] == [1, 1]


@needs_gxx
@pytest.mark.parametrize("batch", [33, 48, 49, 64])
def test_instances_that_fill_a_unit_run_longest_first(rules, batch):
    """8 KV heads, one split, tables of 24 blocks: 257 to 512 workgroups, of which 256 run at a time."""
    waves, = rules("mx", 16, 1)
    line, = rules("order", 8, batch, 512, waves, 24)
    assert line == " ".join(map(str, range(batch))) + " ; 0"


@needs_gxx
@pytest.mark.parametrize("per_seq,batch", [(8, 33), (8, 40), (8, 64), (24, 16), (80, 4), (129, 2), (172, 2), (256, 2)])
def test_two_layers_hold_every_sequence_once(rules, per_seq, batch):
    line, = rules("order", per_seq, batch, 512, 2, 8)
    order, second = line.split(" ; ")
    order, second = list(map(int, order.split())), int(second)
    assert sorted(order) == list(range(batch)) and 0 < second <= batch // 2
    assert order[batch - second:] == list(range(batch - 1, batch - 1 - second, -1))     # shortest first, on top of ...
    assert order[:second] == list(range(batch - 2 * second, batch - second))            # ... the next shortest


MANY_BLOCKS, ONE_BLOCK, ONE_BLOCK_SLICE = 0, 1, 2


@needs_gxx
@pytest.mark.parametrize("gqp", [4, 8])
def test_calls_of_three_workgroups_a_unit_take_a_form_that_fits_three_times(rules, gqp):
    """bd_choose_splits hands out up to 768 workgroups where no wave has more than one block; so many are one round whatever
    residual they carry."""
    asked = [(nb, splits, res_len, wgs) for splits in (1, 2, 3, 4, 16, 64) for nb in (0, 1, 4 * splits - 3, 4 * splits)
             for res_len in (0, 1, 30, 31, 32, 33, 60, 61, 64, 127, 128) for wgs in (513, 640, 768)]
    forms = rules(*(x for q in asked for x in ("blocks", *q)))
    fits = dict(zip("012", rules(*(x for form in range(3) for x in ("int", gqp, form)))))
    assert [q for q, form in zip(asked, forms) if fits[form] != "3"] == []


@needs_gxx
@pytest.mark.parametrize("splits", [1, 2, 5])
def test_forms_of_the_integer_kernel(rules, splits):
    """More than one block a wave: the loop; slices of more than one round beside one block: the loop up to one workgroup per
    unit."""
    ask = lambda nb, res_len, wgs: int(rules("blocks", nb, splits, res_len, wgs)[0])
    assert ask(4 * splits + 1, 0, 768) == ask(4 * splits + 1, 100, 768) == MANY_BLOCKS
    assert ask(4 * splits, 30 * splits, 768) == ask(0, 0, 1) == ask(4 * splits, 30 * splits, 8) == ONE_BLOCK
    if 30 * splits < 128:
        assert ask(4 * splits, 30 * splits + 1, 256) == MANY_BLOCKS and ask(4 * splits, 30 * splits + 1, 257) == ONE_BLOCK_SLICE


ONE_BLOCK_WIDE = 3


@needs_gxx
@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("gq", [1, 4, 5])
@pytest.mark.parametrize("kt", [0, 1])
def test_workgroups_of_eight_waves_are_one_round(rules, bits, gq, kt):
    """A call takes them where four waves would have two blocks each, none more than one with eight, and all of them, the
    packing ones included, have a compute unit of their own; else the form that it takes in four waves."""
    asked = [(nb, splits, res, bits, gq, kt, units, packs) for splits in (1, 2, 5) for nb in (4 * splits, 4 * splits + 1, 6 * splits, 6 * splits + 1, 8 * splits, 8 * splits + 1)
             for res in (0, 128) for units in (1, 128 // splits, 128 // splits + 1, 256 // splits, 256 // splits + 1) for packs in (0, 1)]
    forms = [int(x) for x in rules(*(y for a in asked for y in ("form", *a)))]
    four = [int(x) for x in rules(*(y for a in asked for y in ("blocks", *a[:3], a[1] * a[6])))]
    for a, form, other in zip(asked, forms, four):
        nb, splits, _, _, _, _, units, packs = a
        wide = gq <= 4 and not kt and 4 * splits < nb <= (6 if bits == 4 and splits > 1 else 8) * splits and units * (splits + packs) <= 256
        assert form == (ONE_BLOCK_WIDE if wide else other), a


def test_waves_that_do_not_quantize_wait_at_every_barrier_of_those_that_do():
    """quant_block_barriers is what a workgroup of eight waves counts on: one barrier too few or too many never ends."""
    text = open(os.path.join(CSRC, "bd_quant_block.h")).read()
    text = re.sub(r"//.*", "", text)
    body = text[text.index("void quant_block_at("):text.index("void quant_block(")]
    k, v = body[:body.index("if constexpr ((PART & kPartV) != 0) {")], body[body.index("if constexpr ((PART & kPartV) != 0) {"):]
    by_channel = k[k.index("uint32_t mn["):]
    barrier = re.compile(r"__syncthreads|barrier|workgroup_global_sync")
    assert len(barrier.findall(by_channel)) == len(barrier.findall(k)) == len(barrier.findall(v)) == 1
    assert re.search(r"quant_block_barriers\(bool kt\) \{ return kt \? 1 : 2; \}", text)


FLUSH_AFTER, FLUSH_LAST = 2, 3


@needs_gxx
@pytest.mark.parametrize("splits,batch", [(1, 1), (1, 24), (1, 40), (1, 64), (3, 3), (3, 24), (5, 12), (7, 65), (1, 2 ** 14 - 1)])
def test_lazy_steps_order_and_place_what_attends_as_the_eager_ones(rules, splits, batch):
    """Odd split counts: the attending workgroups' grid and order are the eager step's, every sequence has one row of packing
    workgroups behind them, and the grid is one that a launch takes."""
    eager, = rules("order", splits * 8, batch, 2 ** 30, 2, 32 // splits)
    line, = rules("lazy", splits, 8, batch, 32)
    grid, packed = line.split(" ;")
    x, y, z, order, mode = map(int, grid.split())
    assert (x, y, mode) == (splits, 8, FLUSH_LAST) and batch < z <= 65535
    assert (order & 255 == 0) == eager.startswith("as given") and order >> 10 == int(eager.split(";")[1])
    if batch < 1000:
        packed = list(map(int, packed.split()))
        assert packed[:batch] == list(range(batch)) and all(s >= batch for s in packed[batch:]) and len(packed) < batch + splits


@needs_gxx
@pytest.mark.parametrize("splits,batch", [(2, 40), (4, 24), (3, 2), (1, 2 ** 14), (1, 65535), (65533, 1)])
def test_lazy_steps_whose_packing_workgroups_stay_in_front(rules, splits, batch):
    line, = rules("lazy", splits, 1, batch, 32)
    x, y, z, order, mode = map(int, line.split(" ;")[0].split())
    assert (x, y, z, mode) == (splits + 1, 1, batch, FLUSH_AFTER)


@needs_gxx
@pytest.mark.parametrize("per_seq,batch", [(1, 1), (2, 1), (8, 15), (8, 16), (8, 17), (16, 40), (3, 64), (1, 65535), (65535, 1)])
def test_counters_of_a_step_in_one_split_count_every_workgroup_once(rules, per_seq, batch):
    """What the shards' counters of a launch that raises the lengths wait for, against the sequences b that count at shard
    b % shards; they fit the smallest workspace (one query head)."""
    counts = [int(x) for x in rules("raise", per_seq, batch, 520 * batch)[0].split()]
    assert counts == [per_seq * len(range(s, batch, len(counts))) for s in range(min(batch, 16))]
    assert rules("raise", per_seq, batch, 64 * (len(counts) + 1) - 1) == ["no"]
    assert rules("raise", 1 << 20, batch, 520 * batch) == ["no"]
