"""GPU parity of the switch-hyperedge connection count (the is_util count of
App. B.3 that the uc-max / uc-min policies of Sec. 5.1 weigh), bit for bit
against the oracle, through the C ABI. Needs an MI355X."""
import numpy as np
import pytest

from oracle import OraclePlan
from workloads import configs as cf
from workloads import generate

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def say(msg):
    print(msg, flush=True)


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_04867_amd import binding
    binding.lib()
    torch.cuda.set_device(0)
    yield


def star(P, kind, relays=True, cpr=1):
    row_ptr, col, a, b = cf.csr_from_edges(P + 1, cf.switch_edges(range(P), P, 700, 8))
    mode = cf.RELAY1 if relays else cf.KSHORTEST
    return cf.Workload(f"star{P}", P + 1, P, row_ptr, col, a, b, None, kind, cpr, 65536, mode,
                       k=1)


def two_switches(per, kind):
    P = 2 * per
    edges = cf.switch_edges(range(per), P, 700, 8) + cf.switch_edges(range(per, P), P + 1, 700, 8)
    for i in range(per):
        edges += [(i, per + i, 1700, 106), (per + i, i, 1700, 106)]
    row_ptr, col, a, b = cf.csr_from_edges(P + 2, edges)
    node_of = np.array([0] * per + [1] * per + [0, 1], dtype=np.int32)
    relay = np.array([1] * P + [0, 0], dtype=np.uint8)
    return cf.Workload(f"twoswitch{per}", P + 2, P, row_ptr, col, a, b, node_of, kind, 1, 65536,
                       cf.HIER_RELAY, k=2, max_cross=1, relay=relay)


def hybrid(P, kind):
    """P ranks on one switch plus a bidirectional ring of direct links: some
    routes use the switch and some do not, so the count varies."""
    edges = cf.switch_edges(range(P), P, 700, 8) + cf.ring_edges(range(P), 1500, 8)
    row_ptr, col, a, b = cf.csr_from_edges(P + 1, edges)
    return cf.Workload(f"hybrid{P}", P + 1, P, row_ptr, col, a, b, None, kind, 1, 65536,
                       cf.KSHORTEST, k=4)


def check(w, n, seed, unrouted=0.0):
    from paper_2111_04867_amd.binding import Plan
    plan, ref = Plan.from_workload(w), OraclePlan.from_workload(w)
    opts = plan.route_options()
    assert (opts == ref.route_options()).all()
    routes, _ = generate(seed, 0, n, opts, plan.prio_stride)
    if unrouted:
        rng = np.random.default_rng(seed)
        routes[rng.random(routes.shape) < unrouted] = 0xFF
    say(f"[gpu] connections {w.name} kind={w.kind}: {n} candidates, seed {seed}")
    got = plan.connections(routes)
    want = ref.connections(routes)
    bad = np.nonzero(got != want)[0]
    assert bad.size == 0, (f"{w.name}: {bad.size} mismatches, first at {bad[:5].tolist()}: "
                           f"gpu {got[bad[:5]].tolist()} oracle {want[bad[:5]].tolist()}")
    return got


@pytest.mark.parametrize("name", ["switch16_a2a", "fournode64_a2a", "twonode16_ag",
                                  "cubemesh8_ag"])
def test_named_workloads(name):
    w = cf.named(name)
    n = min(w.n_candidates, 512)
    got = check(w, n, w.seed)
    if name == "fournode64_a2a":
        assert (got == 4 * 16 * 15).all()  # every on-node pair goes direct via the switch
    if name in ("twonode16_ag", "cubemesh8_ag"):
        assert (got == 0).all()  # no switch vertex


@pytest.mark.parametrize("kind", [cf.ALLTOALL, cf.ALLGATHER, cf.REDUCESCATTER, cf.ALLREDUCE])
@pytest.mark.parametrize("P,cpr", [(3, 1), (5, 2), (16, 1), (33, 1)])
def test_star(kind, P, cpr):
    check(star(P, kind, cpr=cpr), 300, 100 + P, unrouted=0.05)


@pytest.mark.parametrize("kind", [cf.ALLTOALL, cf.ALLGATHER, cf.REDUCESCATTER, cf.ALLREDUCE])
@pytest.mark.parametrize("P", [5, 8, 24])
def test_switch_plus_ring(kind, P):
    got = check(hybrid(P, kind), 400, 11 + P, unrouted=0.02)
    assert len(set(got.tolist())) > 1


@pytest.mark.parametrize("kind", [cf.ALLTOALL, cf.ALLGATHER, cf.ALLREDUCE])
def test_two_switch_nodes(kind):
    check(two_switches(4, kind), 400, 7)


def test_batch_split_and_empty():
    from paper_2111_04867_amd.binding import Plan
    w = cf.switch16_a2a(n_candidates=1000)
    plan = Plan.from_workload(w)
    routes, _ = generate(w.seed, 0, 1000, plan.route_options(), plan.prio_stride)
    whole = plan.connections(routes)
    parts = np.concatenate([plan.connections(routes[:333]), plan.connections(routes[333:])])
    assert np.array_equal(whole, parts)
    d_r = torch.empty((0, plan.route_stride), dtype=torch.uint8, device="cuda")
    d_c = torch.empty(1, dtype=torch.int32, device="cuda")
    plan.connections_tensors(d_r, d_c)  # n == 0 is a no-op
    torch.cuda.synchronize()


def switch_chain(P):
    """Ranks in a row with a switch between neighbours: the route from one
    end to the other forms P - 1 switched pairs."""
    edges = []
    for i in range(P - 1):
        edges += cf.switch_edges((i, i + 1), P + i, 700, 8)
    row_ptr, col, a, b = cf.csr_from_edges(2 * P - 1, edges)
    return cf.Workload(f"switchchain{P}", 2 * P - 1, P, row_ptr, col, a, b, None, cf.ALLTOALL, 1,
                       65536, cf.KSHORTEST, k=1)


def many_options(P, k):
    """A switch, a ring and chords: up to k routes per pair."""
    w = hybrid(P, cf.ALLTOALL)
    edges = cf.switch_edges(range(P), P, 700, 8) + cf.ring_edges(range(P), 1500, 8)
    edges += [(i, (i + 2) % P, 1900, 8) for i in range(P)]
    w.row_ptr, w.col, w.alpha_ns, w.beta_ps_per_byte = cf.csr_from_edges(P + 1, edges)
    w.k = k
    return w


@pytest.mark.parametrize("w,n", [
    (switch_chain(3), 65),         # two pairs per route: one wavefront per candidate
    (switch_chain(5), 65),         # up to four: one block per candidate
    (star(2, cf.ALLTOALL), 7),     # one route word, 4 lanes per candidate
    (star(8, cf.ALLTOALL), 1),     # 16 lanes per candidate, one candidate
    (star(16, cf.ALLTOALL), 4099),  # 64 lanes, one word each, several rounds
    (star(17, cf.ALLTOALL), 130),  # 289 chunks: two words per lane, odd rows
    (star(20, cf.ALLTOALL, cpr=2), 70),
    (many_options(16, 120), 33),   # record table beyond LDS, one word per lane
    (star(64, cf.ALLTOALL, relays=False), 40),  # largest byte matrix
    (star(65, cf.ALLTOALL, relays=False), 9),   # past it
    # record tables of 2000 to 16000 records: batches on either side of the
    # one from which they are copied to LDS, words of rows and odd rows
    (star(14, cf.ALLTOALL), 1500), (star(14, cf.ALLTOALL), 2700),
    (star(16, cf.ALLTOALL), 1799), (star(16, cf.ALLTOALL), 1801),
    (star(17, cf.ALLTOALL), 2900), (star(20, cf.ALLTOALL, cpr=2), 1800),
    (star(24, cf.ALLTOALL), 3), (star(64, cf.ALLTOALL, relays=False), 200),
], ids=lambda x: x.name if hasattr(x, "name") else str(x))
def test_alltoall_variants(w, n):
    check(w, n, 3 + n, unrouted=0.05)


def test_unaligned_routes():
    """Route rows of whole words behind a pointer that is not word aligned."""
    from paper_2111_04867_amd.binding import Plan
    w = cf.switch16_a2a()
    plan = Plan.from_workload(w)
    routes, _ = generate(w.seed, 0, 257, plan.route_options(), plan.prio_stride)
    buf = torch.zeros(routes.size + 1, dtype=torch.uint8, device="cuda")
    buf[1:] = torch.from_numpy(routes.reshape(-1))
    out = torch.empty(257, dtype=torch.int32, device="cuda")
    plan.connections_tensors(buf[1:].view(257, plan.route_stride), out)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy().view(np.uint32), plan.connections(routes))
