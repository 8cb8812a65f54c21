"""What calls do on the host - argument checks, plans, sizes, the kernels they launch - without a GPU:
the library runs against stand-ins for the HIP functions (host_calls.c) and no kernel executes."""
import os
import re
import subprocess

import pytest

from paper_2009_06693_amd import binding as B

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "host_calls")
    lib = os.path.abspath(B.LIB_PATH)
    subprocess.run(["gcc", "-O1", "-Wall", "-rdynamic", os.path.join(HERE, "host_calls.c"), lib, "-o", exe,
                    f"-Wl,-rpath,{os.path.dirname(lib)}", "-Wl,--allow-shlib-undefined"], check=True)

    def run(app, num_roots, V=1000, E=4000, weighted=0, free_bytes=0, **params):
        args = [str(x) for x in (V, E, weighted, free_bytes, app, num_roots)]
        args += [f"{k}={','.join(map(str, v)) if isinstance(v, (list, tuple)) else v}" for k, v in params.items()]
        r = subprocess.run([exe, *args], capture_output=True, text=True)
        assert r.returncode == 0, (args, r.returncode, r.stdout, r.stderr)
        got = {"launches": [], "lds": []}
        for line in r.stdout.splitlines():
            what, *rest = line.split()
            if what == "launch":
                got["launches"].append(rest[0])
                got["lds"].append(int(rest[2]))
            else:
                got[what] = [int(x) for x in rest]
        return got
    return run


@pytest.mark.parametrize("fanout", [[65536, 65536], [1 << 14, 1 << 14], [1 << 20] * 3])
def test_a_call_without_roots_returns_whatever_the_fanouts(program, fanout):
    """No samples, hence no limit on the slots of one: the calls return, launch no sampling and ask for little."""
    got = program(B.ND_KHOP, 0, fanout=fanout, unique_rounds=2)
    assert got["query"][0] == 0 and got["query"][1] < 1 << 20 and got["query"][2] == len(fanout)
    assert got["static"] == [0]
    assert not any("khop" in k or "sample" in k for k in got["launches"])


@pytest.mark.parametrize("byte", [0, 0x7E, 0xFE])
def test_status_and_statistics_of_a_workspace_that_no_call_has_used(program, byte):
    """What lies there is not taken for places and numbers of words to fetch (no status bit is set in these bytes)."""
    assert program(B.ND_KHOP, 10, fanout=[3], unused=byte)["unused"] == [0, 0]


@pytest.mark.parametrize("weighted", [0, 1])
def test_links_are_taken_from_a_quarter_of_the_free_memory(program, weighted):
    """The rest is left to the caller, who may have had room for a call's outputs and nothing else."""
    V, E = 1000, 8_000_000
    graph = (V + 1) * 8 + E * 4 + (E * 12 + V * 4 if weighted else 0)
    links = E * (32 if weighted else 16)
    during = graph + 256 + (E * 4 if weighted else 0)      # flags, and the weights as given
    got = program(B.ND_DEEPWALK, 10, V=V, E=E, weighted=weighted, free_bytes=during + 4 * links, num_steps=2)
    assert got["allocated"] == [graph + links] and any("walk_free" in k for k in got["launches"])
    got = program(B.ND_DEEPWALK, 10, V=V, E=E, weighted=weighted, free_bytes=during + 4 * links - 1, num_steps=2)
    assert got["allocated"] == [graph] and any("walk_window" in k for k in got["launches"])


def _tables(V, E):
    return (E // 2 + V + 1) * 16


def test_membership_tables_that_could_not_be_made_are_made_when_there_is_room(program):
    """One refused allocation does not decide for the rest of the graph's life."""
    V, E = 1000, 80_000
    graph = (V + 1) * 8 + E * 4 + E * 16
    for queries, tables in ((1, 0), (2, _tables(V, E)), (3, _tables(V, E))):
        got = program(B.ND_NODE2VEC, 10, V=V, E=E, num_steps=2, fail_malloc=1, queries=queries)
        assert got["query"][0] == 0 and got["allocated"] == [graph + tables]


def test_membership_tables_are_taken_from_a_quarter_of_the_free_memory(program):
    V, E = 1000, 80_000
    graph = (V + 1) * 8 + E * 4 + E * 16
    for left, tables in ((4 * _tables(V, E), _tables(V, E)), (4 * _tables(V, E) - 1, 0)):
        got = program(B.ND_NODE2VEC, 10, V=V, E=E, num_steps=2, left=left)
        assert got["query"][0] == 0 and got["allocated"] == [graph + tables]


def test_membership_tables_are_made_on_the_device_of_the_graph(program):
    """Whatever device is current when sizes are asked for, and that one stays current."""
    V, E = 1000, 80_000
    graph = (V + 1) * 8 + E * 4 + E * 16
    got = program(B.ND_NODE2VEC, 10, V=V, E=E, num_steps=2, device=1)
    assert got["allocated"] == [graph + _tables(V, E)] and got["device"] == [1]


_LIMIT = (7 << 29) // 64  # entries whose cells take 3.5 GB


@pytest.mark.parametrize("app", [B.ND_DEEPWALK, B.ND_PPR])
@pytest.mark.parametrize("E,walks,query_walks,built,used", [
    (_LIMIT, 600_000, 600_000, True, True), (_LIMIT + 1, 600_000, 600_000, False, False),
    (_LIMIT + 1, 32_768, 32_768, True, True), (_LIMIT + 1, 32_769, 32_769, False, False),
    (2 * _LIMIT, 64, 64, True, True), (2 * _LIMIT, 600_000, 64, True, False)])
def test_weighted_walks_draw_from_cells_where_they_are_the_faster(program, app, E, walks, query_walks, built, used):
    """Many walks on graphs whose cells take 4 GB and more are slower by them (600 K walks of 20 steps on 117 M entries
    590 us, 445 by the links): they use none, whoever had them built, and ask for none."""
    V = 1000
    graph = (V + 1) * 8 + E * 4 + E * 12 + V * 4 + E * 32
    got = program(app, walks, V=V, E=E, weighted=1, num_steps=2, use_weights=1, query_roots=query_walks)
    assert got["static"] == [0] and got["allocated"] == [graph + (E * 64 if built else 0)]
    assert ("kernelILi3E" if used else "kernelILi1E") in got["launches"][0]


@pytest.mark.parametrize("per,fanout,samples,lanes", [
    (4, [7], 50_000, 64), (64, [64, 64], 3, 64), (65, [1], 9, 128), (1, [128, 3], 300, 128), (2, [129], 1, 256),
    (256, [256], 9000, 256), (64, [512, 512], 2000, 512), (512, [2048], 300, 512), (512, [2048], 256, 1024),
    (4096, [4096, 512], 257, 1024), (4096, [512], 257, 512), (64, [4096], 257, 512)])
def test_layer_samples_take_as_many_lanes_as_they_have_transits_and_draws(program, per, fanout, samples, lanes):
    """A workgroup that is wider than its sample keeps others from the compute unit (50,000 samples of 4 transits and
    7 draws took 210 us with 512 lanes each, 140 step by step); the widest where a unit has one sample at a time."""
    got = program(B.ND_LAYER, samples * per, fanout=fanout, roots_per_sample=per)
    assert got["static"] == [0] and len(got["launches"]) >= 1
    assert f"Li{lanes}EE" in got["launches"][0] and "layer_fused" in got["launches"][0]


@pytest.mark.parametrize("n,samples,totals,lanes", [
    (3399, 256, True, 1024), (3399, 257, False, 512), (3399, 512, False, 512), (3399, 513, True, 1024),
    (2914, 512, True, 512), (2915, 512, False, 512), (2915, 513, True, 1024), (3400, 257, True, 1024),
    (1908, 513, True, 512), (1909, 513, False, 512), (2226, 513, False, 512), (2227, 513, True, 512),
    (2100, 512, True, 512), (2100, 768, False, 512), (2100, 769, True, 512)])
def test_weighted_layer_samples_that_ran_at_once_do_not_wait_for_the_rows_totals(program, n, samples, totals, lanes):
    """Totals take 4 bytes of LDS per transit: not where fewer samples then fit a unit and a second round begins (512 of
    [2920, 2920]: 132 us, 110 without); 1,024 lanes where one fits, its static LDS counted (3,400 transits)."""
    got = program(B.ND_LAYER, samples * n, V=100_000, E=200_000, weighted=1, use_weights=1, fanout=[n, n],
                  roots_per_sample=n)
    assert got["static"] == [0] and "layer_fused" in got["launches"][0] and f"Li{lanes}EE" in got["launches"][0]
    assert got["lds"][0] == n * (28 if totals else 24)


def test_layer_samples_of_which_one_fits_a_unit_take_all_its_lanes(program):
    """Two of 3,400 transits fit 160 KB only without the kernel's static LDS."""
    for n, lanes in ((3399, 512), (3400, 1024)):
        got = program(B.ND_LAYER, 300 * n, fanout=[n, n], roots_per_sample=n)
        assert f"Li{lanes}EE" in got["launches"][0]


@pytest.mark.parametrize("fanout,samples,E,kernel", [
    (4096, 16_384, 4000, "Li2ELb1E"), (4096, 16_383, 4000, "Li2ELb0E"), (4096, 16_384, 20_000_000, "Li2ELb1E"),
    (4097, 16_384, 8 << 20, "Li1ELb1E"), (4097, 16_384, (8 << 20) + 1, "Li1ELb0E"), (4097, 16_376, 4000, "Li1ELb0E")])
@pytest.mark.parametrize("weighted", [0, 1])
def test_khop_outputs_that_leave_one_by_one_pass_the_caches_of_small_graphs_only(program, fanout, samples, E, kernel,
                                                                                weighted):
    """Past the caches from 64 M draws of the last hop on: in pairs, and one by one where L2 holds the entries (400 M draws
    of [7, 13] on R-MAT 22: 1,581 us one by one past the caches, 1,520 through them)."""
    got = program(B.ND_KHOP, samples, V=1_000_000, E=E, fanout=[fanout], weighted=weighted)
    assert got["static"] == [0] and f"khop_fused_kernelILi{1 + weighted}E{kernel}" in got["launches"][0]


def _mrw_kernels(got):
    """Of each launch of a multi-dimensional walk, whether rows stay in LDS and whether bits are looked up."""
    found = [re.search(r"mrw_free_kernelILi\dElLi\d+ELb(\d)ELb(\d)E", k) for k in got["launches"]]
    return [m.groups() for m in found if m]


@pytest.mark.parametrize("V,roots,steps,kept", [
    (1 << 19, 100, 96, [1]), ((1 << 19) - 1, 100, 96, [0]), (1 << 19, 100, 95, [0]), (1 << 19, 4, 100, [1]),
    (1 << 22, 100, 64, [0]), (1 << 22, 100, 70, [0]), (57_000, 100, 128, [0]), (1 << 22, 100, 223, [1, 0]),
    (1 << 22, 100, 224, [1, 1]), (1 << 19, 153, 100, [1]), (1 << 19, 154, 100, [0]), (1 << 19, 614, 100, [1]),
    (1 << 19, 615, 100, [0])])
@pytest.mark.parametrize("samples", [16, 8192])
def test_rows_of_moved_roots_stay_where_they_are_looked_at_again(program, V, roots, steps, kept, samples):
    """From half of a second round of 64 steps on and from 4 MB of offsets (100 roots, 70 steps 8.63 us where rows stay
    and 8.41 without, 1 MB of offsets 9.26 and 9.06), as far as they fit 48 KB."""
    got = program(B.ND_MULTIRW, samples * roots, V=V, num_steps=steps, roots_per_sample=roots)
    assert got["static"] == [0] and _mrw_kernels(got) == [(str(k), "0") for k in kept]


@pytest.mark.parametrize("V,empty,roots,samples,steps,bits", [
    (1 << 20, 0.351, 100, 8192, 100, [1]), (1 << 20, 0.349, 100, 8192, 100, [0]), ((1 << 20) - 1, 0.5, 100, 8192, 100, [0]),
    (1 << 20, 0.5, 100, 8191, 100, [0]), (1 << 20, 0.451, 30, 8192, 100, [1]), (1 << 20, 0.449, 30, 8192, 100, [0]),
    (1 << 20, 0.9, 29, 8192, 100, [0]), (1 << 20, 0.41, 60, 8192, 70, [1]), (1 << 20, 0.9, 60, 8192, 64, [0]),
    (1 << 20, 0.5, 100, 8192, 192, [1, 0]), (1 << 20, 0.28, 614, 8192, 100, [1]), (1 << 20, 0.27, 614, 8192, 100, [0]),
    (1 << 20, 0.9, 154, 8192, 100, [0])])
def test_bits_tell_empty_rows_where_enough_of_them_are(program, V, empty, roots, samples, steps, bits):
    """The fewer roots a sample has the more rows have to be empty, from 8,192 samples and 8 MB of offsets on (30 roots,
    41,943 samples, a quarter empty: 3 % slower with bits).  They are made when sizes are asked for and are a bit per vertex."""
    got = program(B.ND_MULTIRW, samples * roots, V=V, empty=int(empty * V), num_steps=steps, roots_per_sample=roots)
    assert [int(b) for _, b in _mrw_kernels(got)] == bits
    assert all(k == "1" for k, b in _mrw_kernels(got) if b == "1")
    assert got["allocated"] == [(V + 1) * 8 + 4000 * 4 + 4000 * 16 + ((V + 63) // 64 * 8 if any(bits) else 0)]


@pytest.mark.parametrize("fanout,rounds", [([25, 10], 0), ([15, 10, 4], 0), ([25, 10], 3), ([30], 3)])
@pytest.mark.parametrize("draws,E,past", [(24_000_000, 44_000_000, True), (24_000_000, 43_000_000, False),
                                          (23_990_000, 120_000_000, False), (32_000_000, 36_000_000, True),
                                          (32_000_000, 35_000_000, False), (67_500_000, 4000, True), (66_000_000, 4000, False)])
def test_outputs_that_the_last_level_cache_holds_stay_in_it(program, fanout, rounds, draws, E, past):
    """A copy of 48 MB of outputs behind the call that wrote them took 6 % longer, call included, and their records 14 %, when
    they had gone to memory (57 K vertices, [25,10]).  They pass the caches from 24 M draws on, if 256 MB do not hold
    them and the entries."""
    per = 1
    for f in fanout:
        per *= f
    got = program(B.ND_KHOP, -(-draws // per), V=4_000_000, E=E, fanout=fanout, unique_rounds=rounds,
                  workspace=1)
    assert got["call"] == [0]
    name = [k for k in got["launches"] if "khop" in k][0]
    flag = re.search(r"khop_unique_kernelILi\dElLi\d+ELi\dELb(\d)E" if rounds else r"khop_fused_kernelILi\dELi2ELb(\d)E", name).group(1)
    assert flag == str(int(past)), got["launches"]


def _packed(V, E):
    """Bytes of the packed columns."""
    return -(-E // 32) * max(1, (V - 1).bit_length()) * 4 + 4


def _graph_bytes(V, E):
    return (V + 1) * 8 + E * 4 + E * 16


@pytest.mark.parametrize("fanout,samples,V,E,packed", [
    ([6, 10], 100_000, 1000, 12_000, True), ([6, 10], 99_999, 1000, 12_000, False),      # 6 M draws
    ([6, 10], 100_000, 1000, 11_999, False), ([6, 9], 111_112, 1000, 10_800, True),      # 6/5 of the last fanout
    ([6, 9], 111_112, 1000, 10_799, False), ([2, 10], 10_000, 1000, 128_000, True),
    ([2, 10], 9_999, 1000, 128_000, False), ([2, 10], 10_000, 1000, 127_999, False),     # 200 K draws, degree 128
    ([200], 1000, 1000, 128_000, True), ([1, 1], 6_000_000, 1 << 25, 3 << 24, True),     # 25 bits
    ([1, 1], 6_000_000, (1 << 25) + 1, (3 << 24) + 2, False)])
def test_khop_reads_packed_columns_where_draws_are_many_and_rows_long(program, fanout, samples, V, E, packed):
    """Both sides of each line of the rule, by the kernels that are launched and by the memory that the query takes."""
    got = program(B.ND_KHOP, samples, V=V, E=E, fanout=fanout, workspace=1)
    assert got["call"] == [0] and got["allocated"] == [_graph_bytes(V, E) + (_packed(V, E) if packed else 0)]
    reads = [re.search(r"khop_fused_kernelILi1ELi\dELb\dELb(\d)E", k) for k in got["launches"]]
    assert [m.group(1) for m in reads if m] == [str(int(packed))], got["launches"]


def test_grouped_khop_reads_packed_columns_too(program):
    """The first hop, which is not grouped, and the sub-wavefront class of the second."""
    V, E = 1_000_000, 120_000_000
    got = program(B.ND_KHOP, V, V=V, E=E, fanout=[10, 10], workspace=1)
    assert got["call"] == [0] and got["allocated"] == [_graph_bytes(V, E) + _packed(V, E)]
    first = [k for k in got["launches"] if "khop_first" in k]
    second = [k for k in got["launches"] if "sample_tp_kernel" in k]
    assert len(first) == 1 and "ILb1E" in first[0] and len(second) == 1 and "ILi0ELb1E" in second[0]


def test_packed_columns_are_taken_from_a_quarter_of_the_free_memory(program):
    V, E = 1000, 128_000
    for left, packed in ((4 * _packed(V, E), _packed(V, E)), (4 * _packed(V, E) - 1, 0)):
        got = program(B.ND_KHOP, 10_000, V=V, E=E, fanout=[2, 10], left=left, workspace=1)
        assert got["call"] == [0] and got["allocated"] == [_graph_bytes(V, E) + packed]


@pytest.mark.parametrize("fanout,samples,V,E", [([25, 10], 30_000, 100_000, 2_000_000), ([1 << 20], 6, 1 << 20, 160 << 20),
                                                ([15, 10, 5], 9000, 57_000, 1_600_000), ([2, 10], 10_000, 1000, 128_000),
                                                ([4000], 50, 1000, 128_000), ([10, 10], 1_000_000, 1_000_000, 120_000_000)])
def test_sizes_of_khop_asked_for_with_the_groups_of_all_samples_build_nothing(program, fanout, samples, V, E):
    """A way to decline the packed columns: the sizes are the same, and the call reads the columns as they are."""
    same = program(B.ND_KHOP, samples, V=V, E=E, fanout=fanout, workspace=1)
    got = program(B.ND_KHOP, samples, V=V, E=E, fanout=fanout, workspace=1, query_window=-1)
    assert got["query"] == same["query"] and got["call"] == same["call"] == [0]
    assert got["allocated"] == [_graph_bytes(V, E)] and same["allocated"] == [_graph_bytes(V, E) + _packed(V, E)]
    assert len(got["launches"]) == len(same["launches"])
