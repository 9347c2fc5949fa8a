"""Launch plans of qg_gemm_small, looked at without a GPU (tests/launches.py; 256 compute units)."""
import random

import pytest

from tests.launches import launches
from tests.test_gpu_parity import AHEAD_CASES, I8_CASES, M1_CASES, MANY_ROWS_CASES, ROW_BLOCK_CASES, ROWS_CASES, SELF_CASES, UNIT_CASES


@pytest.fixture(scope="module")
def tmp(tmp_path_factory):
    return tmp_path_factory.mktemp("hip_stub")


def _product(result):
    """The raw-code product of a call and the kernels around it."""
    assert result["status"] == 0
    k, = [k for k in result["kernels"] if k["name"] == "gemm_codes"]
    return k, [k["name"] for k in result["kernels"]]


# Few tiles and a K long enough to be cut: the product takes the compute units that parts of K can fill, whatever
# adding the parts costs (with 64 to 80 of the 256 these were slower than before they shared A operands in LDS)
@pytest.mark.parametrize("problem,workgroups", [
    ((5120, 5120, 3, 64, 16), 200), ((4096, 4096, 3, 64, 8), 256), ((4096, 4096, 3, 4096, 8), 128),
    ((8192, 8192, 2, 128, 16), 250), ((1500, 20480, 4, 16, 8), 96), ((4096, 11008, 4, 16, 24), 250)])
def test_short_products_fill_the_chip(tmp, problem, workgroups):
    k, _ = _product(launches(tmp, [{"problem": problem}])[0])
    assert k["grid"][0] >= workgroups


# 4 bits, where both kernel families take the layout: the faster one as measured, by rows, size and group
@pytest.mark.parametrize("problem,raw", [
    ((8192, 8192, 4, 32, 33), False), ((8192, 8192, 4, 32, 64), False), ((8192, 8192, 4, 64, 40), True),
    ((8192, 8192, 4, 128, 64), True), ((8192, 8192, 4, 32, 32), True), ((8192, 8192, 4, 32, 65), True),
    ((13824, 5120, 4, 32, 40), True), ((5120, 5120, 4, 32, 24), False)])
def test_kernel_family_of_4_bit_products(tmp, problem, raw):
    names = [k["name"] for k in launches(tmp, [{"problem": problem}])[0]["kernels"]]
    assert ("gemm_codes" in names) == raw, names


def test_large_lds_is_asked_for_on_every_device(tmp):
    # ... and once: further calls on a device ask no more
    call = {"problem": (4096, 4096, 2, 64, 100)}
    results = launches(tmp, [dict(call, device=d) for d in (0, 1, 0, 1, 70, 70)])
    assert [r["status"] for r in results] == [0] * 6
    assert all(_product(r)[0]["lds"] > 65536 for r in results)
    assert [r["limits"] for r in results] == [1, 2, 2, 2, 3, 4]


@pytest.mark.parametrize("problem", [(4096, 11008, 4, 128, 128), (18000, 2048, 4, 128, 100), (13824, 5120, 4, 64, 48),
                                     (8192, 8192, 4, 32, 40), (5120, 5120, 3, 64, 16)])
def test_search_times_the_built_in_plan(tmp, problem):
    def plan(result):
        return [(k["name"], k["template"], k["grid"], k.get("args", {}).get("quota")) for k in result["kernels"]]

    results = launches(tmp, [{"problem": problem}] + [{"problem": problem, "splits": s} for s in range(1, 9)] +
                       [{"problem": problem, "search": True}])
    same = [s for s in range(1, 9) if plan(results[s]) == plan(results[0])]
    assert same and results[9]["status"] == 0
    assert results[9]["us"][same[0] - 1] >= 0          # shape 0 (built-in kernel), that many ranges


# ... and prices the raw-code cuts on the scale of the others: some of them on the kernel asked for by number are timed
@pytest.mark.parametrize("problem", [(8192, 8192, 4, 32, 40), (5120, 5120, 4, 128, 64)])
def test_search_times_raw_code_cuts(tmp, problem):
    result, = launches(tmp, [{"problem": problem, "search": True}])
    assert result["status"] == 0 and any(us >= 0 for us in result["us"][14 * 8:])


# The GPU test of the cuts of K takes the cuts it names
@pytest.mark.parametrize("case", [c for c in UNIT_CASES if c[6] is not None])
def test_unit_cases_are_cut_as_stated(tmp, case):
    *problem, splits, (dealt, parts, fused, row_blocks) = case
    k, names = _product(launches(tmp, [{"problem": problem, "splits": splits, "shape": 13}])[0])
    a = k["args"]
    most = a["ranges"] or (a["units"] + a["quota"] - 2) // a["quota"] + 1
    assert (a["ranges"] == 0, most, a["fused"], a["zblocks"]) == (dealt, parts, fused, row_blocks)
    assert ("add_parts" in names) == (parts > 1 and not fused)


@pytest.mark.parametrize("problem,splits,last_workgroup", [
    ((1088, 704, 4, 32, 64), 3, False), ((4096, 4096, 4, 128, 64), 2, False), ((12300, 768, 2, 32, 100), 2, True),
    ((22016, 8192, 2, 32, 128), 0, True), ((130, 3072, 3, 64, 9), 2, True), ((130, 3072, 3, 64, 32), 3, True)])
def test_who_adds_two_or_three_parts(tmp, problem, splits, last_workgroup):
    # at 64 rows the last workgroup from some megabytes of parts on, at 32 always
    k, names = _product(launches(tmp, [{"problem": problem, "splits": splits, "shape": 13}])[0])
    assert (k["args"]["fused"] == 1, "add_parts" not in names) == (last_workgroup, last_workgroup)


# The GPU tests of the blocks of 32 rows take the cuts they name
@pytest.mark.parametrize("case", ROW_BLOCK_CASES)
def test_row_block_cases_are_cut_as_stated(tmp, case):
    *problem, blocks, parts, fused = case
    k, names = _product(launches(tmp, [{"problem": problem}])[0])
    a, (_, _, mb, tn, *_) = k["args"], k["template"]
    tiles = (problem[0] + 63) // 64
    assert (mb, a["ranges"], a["fused"], k["grid"][0]) == (1, parts, fused, -(-tiles // tn) * blocks * parts)
    assert ("add_parts" in names) == (parts > 1 and not fused)


# Blocks of 64 rows: whole ranges of K where units dealt evenly measured slower (ranges), and dealt (0) where faster
@pytest.mark.parametrize("problem,ranges", [
    ((14611, 6784, 2, 128, 70), 2), ((7614, 20608, 3, 64, 90), 4), ((7702, 10464, 2, 32, 86), 4), ((9374, 17408, 4, 128, 116), 3),
    ((6991, 8320, 2, 64, 70), 4), ((22016, 8192, 2, 32, 128), 0)])
def test_blocks_of_64_rows_are_cut_as_measured(tmp, problem, ranges):
    k, _ = _product(launches(tmp, [{"problem": problem}])[0])
    assert (k["template"][2], k["args"]["ranges"]) == (2, ranges)


@pytest.mark.parametrize("case", SELF_CASES)
def test_own_operand_cases_are_cut_as_stated(tmp, case):
    *problem, parts = case
    k, names = _product(launches(tmp, [{"problem": problem}])[0])
    assert (k["template"][2], k["template"][5], k["args"]["self"]) == (1, 2, 1) and k["args"]["ranges"] == parts
    assert names == ["gemm_codes"] + ["add_parts"] * (parts != 1)


# The GPU tests of operands made ahead take every instance of the kernel (bits, groups per step, blocks of rows, tiles, k-slices, who adds) that
# the plan takes with them over random products
def test_cases_of_operands_made_ahead_take_every_instance(tmp):
    rng = random.Random(1)
    problems = []
    while len(problems) < 3000:
        bits = rng.choice([2, 3, 4])
        group = rng.choice([32, 64, 128, 256, 512, 0] + [16] * (bits == 4))
        grain = group or 128
        K = max(1, round(512 * 43.0 ** rng.random() / grain)) * grain
        N = round(512 * (min(22016, 22016 * 8192 // K) / 512) ** rng.random())
        problems.append((N, K, bits, group or K, round(2 * 64.0 ** rng.random())))

    def instances(calls):
        kernels = [k for r in launches(tmp, [{"problem": c} for c in calls]) for k in r["kernels"] if k["name"] == "gemm_codes"]
        return [tuple(k["template"]) for k in kernels if not k["args"]["self"]]

    tested = instances(AHEAD_CASES)
    assert len(tested) == len(AHEAD_CASES)
    assert set(instances(problems)) <= set(tested) and len(set(tested)) == 50


@pytest.mark.parametrize("problem,name", [(c, "gemv_mma4i") for c in ROWS_CASES] + [
    ((11008, 4096, 4, 128, 16), "gemm_rows16"), ((11967, 2048, 4, 128, 4), "gemm_rows16"), ((6000, 1664, 4, 64, 12), "gemm_rows16"),
    ((16888, 864, 4, 32, 5), "gemm_codes"), ((11295, 1280, 3, 1280, 14), "gemm_codes")])
def test_one_launch_up_to_16_rows(tmp, problem, name):
    assert [k["name"] for k in launches(tmp, [{"problem": problem}])[0]["kernels"]] == [name]


# One row is a GEMV at every width; at 4 bits, where products of more rows leave other things in the workspace, without
# meeting slots or with slots emptied first
@pytest.mark.parametrize("case", M1_CASES)
def test_one_row_is_a_gemv(tmp, case):
    *problem, filled = case
    *before, k = launches(tmp, [{"problem": (*problem, 1)}])[0]["kernels"]
    assert k["name"].startswith("gemv_") and [b["name"] for b in before] == ["fill_u32"] * filled
    assert filled or not k["slots"] or problem[2] != 4


# ... and of as many parts as a K of that length can be cut into
@pytest.mark.parametrize("N,K,M,parts", [(22016, 1024, 128, 0), (22016, 1920, 128, 0), (22016, 1952, 128, 2), (1000, 2080, 40, 2), (300, 8224, 128, 8)])
def test_int8_workspace_holds_the_parts_of_a_long_k_alone(tmp, N, K, M, parts):
    result, = launches(tmp, [{"problem": (N, K, 3, 32, M)}])
    units, blocks = (K + 127) // 128, (M + 7) // 8
    operands = blocks * units * (4096 + 32)
    assert 0 <= result["size"] - 16 * 8448 * ((N + 63) // 64) - operands - 4 * parts * M * N < 1024
    assert all(b <= result["size"] for k in result["kernels"] for _, b in k.get("writes", []))


# 3-bit groups of 32, more rows than one launch of matrix-vector products takes: those where the int8 kernel's chain of units
# is the longer way
@pytest.mark.parametrize("problem,names", [(c, ["gemv_mma4i"] * launches_) for *c, launches_ in MANY_ROWS_CASES] + [
    ((4096, 4096, 3, 32, 17), ["prepare_rows_i8", "gemm_rows_i8", "add_splits"]), ((9934, 576, 3, 32, 17), ["prepare_rows_i8", "gemm_rows_i8"])])
def test_3_bit_groups_of_32_beyond_16_rows(tmp, problem, names):
    assert [k["name"] for k in launches(tmp, [{"problem": problem}])[0]["kernels"]] == names


# The GPU tests of the int8 kernel take it, with one, two and four blocks of eight rows, K in one range and in several
def test_int8_cases_take_that_kernel(tmp):
    kernels = [r["kernels"] for r in launches(tmp, [{"problem": (N, K, 3, 32, M)} for N, K, M in I8_CASES])]
    assert all([k["name"] for k in ks][:2] == ["prepare_rows_i8", "gemm_rows_i8"] for ks in kernels)
    assert {ks[1]["template"][0] for ks in kernels} == {1, 2, 4} and {len(ks) for ks in kernels} == {2, 3}


# 4 bits below the sizes where raw codes are taken whatever the estimates say: the dequantizing kernels cut K between
# groups only, so that long groups go to raw codes, and so do products that take one launch there
@pytest.mark.parametrize("problem,raw", [
    ((1500, 20480, 4, 20480, 33), True), ((4096, 4096, 4, 4096, 24), True), ((1024, 8192, 4, 128, 96), True),
    ((512, 768, 4, 768, 20), False), ((512, 512, 4, 64, 64), True), ((2048, 2048, 4, 128, 100), True)])
def test_kernel_family_of_small_4_bit_products(tmp, problem, raw):
    names = [k["name"] for k in launches(tmp, [{"problem": problem}])[0]["kernels"]]
    assert ("gemm_codes" in names) == raw, names


# 3-bit groups of 32: the rows of a call are products on int8 digits or matrix-vector products whose partial sums meet in the
# workspace, by M; a buffer of any accepted size serves every M it is large enough for
@pytest.mark.parametrize("N,K", [(4096, 4096), (4096, 11008), (1000, 2080), (20000, 256)])
def test_int8_operands_stay_out_of_the_meeting_slots(tmp, N, K):
    rows = list(range(1, 129))
    slots = 8448 * ((N + 63) // 64)                                       # of one row (as qg_workspace_bytes asks for M = 1)
    own = launches(tmp, [{"problem": (N, K, 3, 32, M)} for M in rows])
    sizes = [16 * slots, 9 * slots] + [own[M - 1]["size"] for M in (1, 2, 8, 15, 16, 17, 40, 128)]
    assert own[0]["size"] == slots and all(r["status"] == 0 for r in own)
    for size in sizes:
        results = [r for r in launches(tmp, [{"problem": (N, K, 3, 32, M), "size": size} for M in rows]) if r["status"] == 0]
        kernels = [k for r in results for k in r["kernels"]]
        writes = [w for k in kernels for w in k.get("writes", [])]
        reads = [s for k in kernels for s in k.get("slots", [])]
        assert results and all(a >= 0 and b <= size for a, b in writes + reads)
        assert not reads or all(a >= max(b for _, b in reads) for a, _ in writes)


# 4-bit matrix-vector products: the steps of a wavefront go by the launch's codes beyond 64 MiB and for one matrix; several matrices of
# 32 to 64 MiB take about six
@pytest.mark.parametrize("problems,steps", [
    ([(20992, 17152, 4, 64)], [17]), ([(41856, 9472, 4, 64)], [19]), ([(39424, 11008, 4, 128)], [15]), ([(16384, 8192, 4, 64)], [6]),
    ([(5120, 5120, 4, 32)] * 4 + [(12032, 5120, 4, 32)] * 2 + [(5120, 12032, 4, 32)], [14, 16]),
    ([(2560, 2560, 4, 64)] * 4 + [(6912, 2560, 4, 64)] * 2 + [(2560, 6912, 4, 64)], [7])])
def test_steps_of_a_4_bit_wavefront(tmp, problems, steps):
    result, = launches(tmp, [{"grouped": problems}])
    assert result["status"] == 0 and sorted({cut[4] for cut in result["cuts"]}) == steps
