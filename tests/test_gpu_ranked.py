"""GPU parity of the ranked multicast kernel at the edges of what it takes:
rank counts that do not fill their last route word, routes longer than four
links, (chunk, vertex) slot counts around each slots-per-lane step up to
1024, rows that are not word aligned, and path codes that rest on the number
of node crossings. Bit for bit against the oracle. Needs an MI355X."""
from dataclasses import replace

import numpy as np
import pytest

from oracle import OraclePlan
from workloads import configs as cf
from workloads import generate

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_04867_amd import binding
    binding.lib()
    torch.cuda.set_device(0)
    yield


def ring(P, k=2, cpr=1, chunk_bytes=65536):
    row_ptr, col, a, b = cf.csr_from_edges(P, cf.ring_edges(list(range(P)), 700, 46))
    return cf.Workload(f"ring{P}x{cpr}", P, P, row_ptr, col, a, b, None, cf.ALLGATHER, cpr,
                       chunk_bytes, cf.KSHORTEST, k=k)


def broadcast(base, C):
    """C chunks from ranks 0, 1, ... to every rank."""
    return cf.explicit_multicast(base, [c % base.P for c in range(C)],
                                 [list(range(base.P))] * C)


def check(w, n=65, seed=3, shift=0):
    from paper_2111_04867_amd.binding import Plan
    plan, ref = Plan.from_workload(w), OraclePlan.from_workload(w)
    opts = plan.route_options()
    assert (opts == ref.route_options()).all()
    routes, prio = generate(seed, 0, n, opts, plan.prio_stride)
    rng = np.random.default_rng(seed)
    routes[rng.random(routes.shape) < 0.01] = 0xFF  # some pairs unrouted
    prio[rng.random(prio.shape) < 0.3] &= 3         # and equal priorities
    print(f"[gpu] ranked {w.name} kind={w.kind} contig={w.contiguity} P={plan.P} "
          f"slots={plan.num_chunks * plan.V} hops={plan.max_hops} shift={shift}", flush=True)
    buf = torch.full((routes.size + shift,), 7, dtype=torch.uint8, device="cuda")
    buf[shift:] = torch.from_numpy(routes.reshape(-1))
    pr = torch.from_numpy(prio.view(np.int32)).cuda()
    mk = torch.empty(n, dtype=torch.int32, device="cuda")
    ok = torch.empty(n, dtype=torch.uint8, device="cuda")
    plan.eval_tensors(buf[shift:].view(n, -1), pr, mk, ok)
    torch.cuda.synchronize()
    rmk, rok = ref.eval(routes, prio)
    assert np.array_equal(mk.cpu().numpy().view(np.uint32), rmk), w.name
    assert np.array_equal(ok.cpu().numpy(), rok), w.name


def kinds(w):
    yield w
    yield cf.as_reduction(w, cf.REDUCESCATTER)
    yield cf.as_reduction(w, cf.ALLREDUCE)


@pytest.mark.parametrize("P", [3, 4, 5, 6, 7, 9, 11, 13, 17, 18, 21, 25, 29, 31, 32])
def test_rank_counts_and_long_routes(P):
    for w in kinds(ring(P)):  # routes of up to P - 1 links
        check(w, n=33 if P > 16 else 65)


@pytest.mark.parametrize("P", [5, 7, 10, 14, 17])
@pytest.mark.parametrize("shift", [0, 1, 2, 3])
def test_unaligned_rows(P, shift):
    check(cf.full_ag(P, k=3), n=17, shift=shift)


def test_word_aligned_ranks_behind_an_odd_pointer():
    for shift in (1, 2):
        check(cf.cubemesh8_ag(), n=70, shift=shift)


# slots per lane 1, 2, 4, 6, 8, 10 and 16, first and last slot count of each
@pytest.mark.parametrize("P,C", [(8, 8), (9, 8), (16, 8), (13, 10), (16, 16), (17, 16), (24, 16),
                                 (11, 35), (16, 32), (27, 19), (20, 32), (23, 28), (32, 32),
                                 (9, 85), (12, 85)])
def test_slot_counts(P, C):
    w = broadcast(cf.full_ag(P, k=2), C)
    check(w, n=40)


@pytest.mark.parametrize("per,cpr,kib", [(3, 1, 17), (4, 2, 1000), (5, 1, 333), (6, 2, 64),
                                         (6, 1, 4)])
@pytest.mark.parametrize("contiguity", [0, 1])
def test_two_nodes(per, cpr, kib, contiguity):
    """Two link costs whose sums are only told apart when each path crosses
    between the nodes at most once."""
    w = replace(cf.two_node_full(per, cf.ALLGATHER, cpr, k=3, chunk_bytes=1024 * kib,
                                 contiguity=contiguity), max_cross=1,
                relay=np.ones(2 * per, dtype=np.uint8))
    check(w, n=40)
    if not contiguity:
        for x in kinds(w):
            check(x, n=40)


def test_three_mesh_nodes():
    """24 ranks on three cube-meshes joined between relays: 576 slots."""
    P = V = 24
    edges = []
    for n in range(3):
        edges += cf.cube_mesh_edges(8 * n, cf.NVLINK_ALPHA, cf.NDV2_NVLINK_BETA)
    relays = [8 * n + r for n in range(3) for r in (0, 4)]
    edges += [(s, d, cf.IB_ALPHA, cf.IB_BETA) for s in relays for d in relays if s // 8 != d // 8]
    row_ptr, col, a, b = cf.csr_from_edges(V, edges)
    relay = np.zeros(V, dtype=np.uint8)
    relay[relays] = 1
    w = cf.Workload("threenode24_ag", V, P, row_ptr, col, a, b,
                    np.array([r // 8 for r in range(V)], dtype=np.int32), cf.ALLGATHER, 1, 1 << 20,
                    cf.KSHORTEST, k=3, max_cross=1, relay=relay)
    for x in kinds(w):
        check(x, n=150)
    check(cf.with_contiguity(w), n=150)


# Crossings that cost just under 13 links inside a node: the gap `short`
# between sums sets the codes' bits. 29000 per link and 13 x 29000 - short per
# crossing take 10 + 6 bits, 11 + 7, 13 + 8 and 13 + 9 (the most a key holds),
# then more than it holds (the layered or general kernel, as before)
@pytest.mark.parametrize("short", [900, 345, 120, 88, 80, 7, 1])
@pytest.mark.parametrize("per,cpr", [(6, 1), (8, 1), (6, 2)])
def test_code_bits(short, per, cpr):
    P = 2 * per
    edges = [(n * per + i, n * per + j, 29000, 0) for n in (0, 1) for i in range(per)
             for j in range(per) if i != j]
    edges += [(s, (s + per) % P, 13 * 29000 - short - 109, 106) for s in (0, 1, per, per + 1)]
    row_ptr, col, a, b = cf.csr_from_edges(P, edges)
    relay = np.zeros(P, dtype=np.uint8)
    relay[[0, 1, per, per + 1]] = 1
    w = cf.Workload(f"codes{short}", P, P, row_ptr, col, a, b,
                    np.array([r // per for r in range(P)], dtype=np.int32), cf.ALLGATHER, cpr,
                    1024, cf.KSHORTEST, k=3, max_cross=1, relay=relay)
    for x in kinds(w):
        check(x, n=70)
    check(cf.with_contiguity(w), n=70)


# the same plans under time-aware greedy orders, in path and reverse path order
@pytest.mark.parametrize("order", [cf.with_greedy, cf.with_reverse_greedy],
                         ids=["greedy", "reverse"])
@pytest.mark.parametrize("P", [3, 5, 6, 9, 14, 17, 22])
def test_greedy_rank_counts_and_long_routes(P, order):
    for w in kinds(ring(P)):
        check(order(w), n=33)
    check(order(cf.full_ag(min(P, 14), k=3)), n=33, shift=P % 4)


@pytest.mark.parametrize("order", [cf.with_greedy, cf.with_reverse_greedy],
                         ids=["greedy", "reverse"])
@pytest.mark.parametrize("P,C", [(8, 8), (13, 5), (9, 14), (16, 16), (10, 26), (7, 73), (16, 32),
                                 (27, 19), (15, 35)])
def test_greedy_slot_counts(P, C, order):
    """Slots per lane 1, 2, 4 and 8, up to 512 slots, and the first plans past
    them."""
    check(order(broadcast(cf.full_ag(P, k=2) if P != 27 else ring(P), C)), n=33)


@pytest.mark.parametrize("P,C,k", [(9, 5, 3), (12, 10, 2), (9, 28, 2), (16, 14, 3), (18, 18, 3),
                                   (22, 15, 3), (24, 16, 8), (24, 21, 2), (31, 16, 2), (32, 16, 4),
                                   (16, 32, 8), (14, 28, 4)])
def test_entering_links(P, C, k):
    """Entering links in global memory and in LDS, at every slots-per-lane
    step up to 8 and every row width past 8 ranks."""
    if P % 8 == 0 and P > 16:
        w = broadcast(cf.cubemesh_nodes_ag(P // 8, k=k), C)
    elif P == 16 and k == 8:
        w = torus_broadcast(4, P, C, k)
    else:
        w = broadcast(cf.full_ag(P, k=k) if P * P <= 256 else ring(P, k=k), C)
    from paper_2111_04867_amd.binding import Plan
    assert Plan.from_workload(w).kernels == "tree_rank"
    check(w, n=50)
    if w.node_of is None:
        w = replace(w, node_of=np.array([r * 2 // w.V for r in range(w.V)], dtype=np.int32))
    check(cf.with_contiguity(w), n=50)


# 12, 14 and 16 slots per lane at every row width, contiguous transfers too
@pytest.mark.parametrize("P,C", [(12, 64), (12, 70), (16, 52), (24, 34), (16, 45), (22, 40),
                                 (12, 85), (28, 30), (30, 32)])
def test_slots_past_640(P, C):
    from paper_2111_04867_amd.binding import Plan
    w = broadcast(cf.full_ag(P, k=2) if P <= 16 else ring(P), C)
    assert Plan.from_workload(w).kernels == "tree_rank"
    check(w, n=33)
    nodes = np.array([r * 2 // P for r in range(P)], dtype=np.int32)
    check(cf.with_contiguity(replace(w, node_of=nodes)), n=33)


def torus_broadcast(side, P, C, k):
    """C chunks to the first P of side x side torus vertices, the others
    switches: tables of P * P * side^2 * k bytes."""
    V = side * side
    edges = []
    for v in range(V):
        r, c = divmod(v, side)
        for u in (r * side + (c + 1) % side, (r + 1) % side * side + c):
            edges += [(v, u, 700, 46), (u, v, 700, 46)]
    row_ptr, col, a, b = cf.csr_from_edges(V, edges)
    return broadcast(cf.Workload(f"torus{side}_{P}", V, P, row_ptr, col, a, b, None, cf.ALLGATHER,
                                 1, 65536, cf.KSHORTEST, k=k), C)


@pytest.mark.parametrize("order", [cf.with_greedy, cf.with_reverse_greedy],
                         ids=["greedy", "reverse"])
@pytest.mark.parametrize("make", [lambda: broadcast(cf.cubemesh_nodes_ag(4, k=4), 16),
                                  lambda: broadcast(cf.cubemesh_nodes_ag(3, k=8), 20),
                                  lambda: broadcast(cf.cubemesh_nodes_ag(3, k=3), 5),
                                  lambda: torus_broadcast(6, 16, 14, 8),
                                  lambda: torus_broadcast(4, 16, 32, 8)],
                         ids=["4x8", "3x8", "3x8_small", "torus6", "torus4"])
def test_greedy_entering_links(make, order):
    """Entering links in global memory, past 256 slots (24 and 32 ranks; 16
    whose table would leave few wavefronts) and below, and in LDS."""
    w = order(make())
    from paper_2111_04867_amd.binding import Plan
    assert Plan.from_workload(w).kernels == "tree_greedy"
    check(w, n=33)


@pytest.mark.parametrize("order", [cf.with_greedy, cf.with_reverse_greedy],
                         ids=["greedy", "reverse"])
@pytest.mark.parametrize("per,cpr,kib", [(3, 1, 17), (5, 1, 333), (6, 2, 4)])
def test_greedy_two_nodes(per, cpr, kib, order):
    base = cf.two_node_full(per, cf.ALLGATHER, cpr, k=3, chunk_bytes=1024 * kib, contiguity=0)
    w = replace(base, max_cross=1, relay=np.ones(2 * per, dtype=np.uint8))
    for x in kinds(w):
        check(order(x), n=33)
