"""Which kernel a plan runs on and what the plan reports of it (no GPU): the
launch and the report share one rule, so a plan's kernels are checked here
and their results in the GPU tests."""
from dataclasses import replace

import pytest

from paper_2111_04867_amd.binding import Plan
from workloads import configs as cf

LDS_PER_BLOCK = 160 * 1024  # gfx950


def mesh_broadcast(nodes, chunks, k):
    return cf.broadcast(cf.cubemesh_nodes_ag(nodes, k=k), chunks)


def uni_ring(chunks):
    """64 ranks on a one-way ring: the general kernel's largest plans."""
    return replace(cf.uni_ring_ag(64, chunk_bytes=65536), chunks_per_rank=chunks)


KERNELS = [
    (cf.ring4_ag(), "tree_rank"),
    (cf.cubemesh8_ag(), "tree_rank"),
    (cf.twonode16_ag(), "tree_rank"),
    (cf.named("twonode16_ag_contig"), "tree_rank"),
    (cf.named("twonode16_ar"), "tree_rank+tree_rank"),
    (cf.as_reduction(cf.named("twonode16_ag_contig"), cf.ALLREDUCE), "tree_layers+tree_rank"),
    (cf.named("twonode16_ag_greedy"), "tree_greedy"),
    (cf.named("twonode16_ag_rgreedy"), "tree_greedy"),
    (cf.cubemesh_nodes_ag(3), "tree_rank"),
    (cf.with_greedy(cf.cubemesh_nodes_ag(3)), "tree_eval"),  # 576 slots
    (uni_ring(1), "tree_eval"),
    (cf.switch16_a2a(), "path_eval_fast"),
    (cf.named("fournode64_a2a_contig"), "path_eval_fast"),
    (cf.named("switch16_a2a_ports"), "path_eval_ports"),
    (cf.named("switch16_a2a_greedy"), "path_greedy"),
    (cf.named("fournode64_a2a_greedy"), "path_greedy_block"),
]


@pytest.mark.parametrize("w,kernels", KERNELS, ids=[w.name for w, _ in KERNELS])
def test_kernel_of_a_plan(w, kernels):
    assert Plan.from_workload(w).kernels == kernels


# plans whose entering-link table (P * V * P * K bytes) takes more LDS than a
# block has, or would leave a CU few of the 8 wavefronts its registers admit:
# at most 48 KB for a block of one of them, shared tables of 34 KB with it
@pytest.mark.parametrize("nodes,chunks,k", [(4, 16, 2), (4, 16, 3), (4, 16, 4), (4, 16, 8),
                                            (3, 20, 8), (3, 8, 4), (3, 21, 3)])
@pytest.mark.parametrize("order", [cf.with_greedy, cf.with_reverse_greedy],
                         ids=["greedy", "reverse"])
def test_greedy_keeps_large_tables_out_of_lds(nodes, chunks, k, order):
    p = Plan.from_workload(order(mesh_broadcast(nodes, chunks, k)))
    assert p.kernels == "tree_greedy"
    assert p.info["lds_bytes"] <= 48 * 1024


# the same for the ranked kernel, its shared tables (43 KB at 32 ranks) and one
# wavefront's state without the entering links
@pytest.mark.parametrize("nodes,chunks,k", [(4, 16, 2), (4, 16, 3), (4, 16, 4), (4, 16, 8),
                                            (4, 4, 3), (3, 20, 8), (3, 8, 4), (3, 21, 3)])
@pytest.mark.parametrize("contiguity", [0, 1])
def test_ranked_keeps_large_tables_out_of_lds(nodes, chunks, k, contiguity):
    w = mesh_broadcast(nodes, chunks, k)
    p = Plan.from_workload(cf.with_contiguity(w) if contiguity else w)
    assert p.kernels == "tree_rank"
    assert p.info["lds_bytes"] <= 58 * 1024


@pytest.mark.parametrize("order", [lambda w: w, cf.with_greedy, cf.with_reverse_greedy,
                                   lambda w: cf.as_reduction(w, cf.ALLREDUCE)],
                         ids=["static", "greedy", "reverse", "allreduce"])
def test_lds_bytes_above_the_limit_exactly_where_refused(order):
    """Broadcasts on four meshes have tables that outgrow a block's LDS in one
    kernel or another, which then must not be the one that is reported; the
    ring's plans grow until no kernel takes them."""
    if order(uni_ring(1)).kind == cf.ALLREDUCE:
        plans = [cf.cubemesh_nodes_ag(n, k=k) for n in (2, 3, 4) for k in (2, 4, 8)]
    else:
        plans = [mesh_broadcast(4, 16, k) for k in (2, 3, 4, 8)] + [uni_ring(c)
                                                                  for c in (1, 2, 3, 4)]
    refused = 0
    for w in plans:
        p = Plan.from_workload(order(w))
        assert p.info["lds_bytes"] > 0
        assert (p.info["lds_bytes"] > LDS_PER_BLOCK) == (p.kernels == "none"), (w.name, p.kernels)
        refused += p.kernels == "none"
    assert len(plans) == 9 or 0 < refused < 4
