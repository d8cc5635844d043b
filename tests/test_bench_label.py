"""The benchmark's label of the score kernel where it depends on what a work item costs (no GPU needed): batches whose best number of
pieces changes with that cost."""
import bench
import tri_rules as R


def test_label_follows_the_item_cost():
    batches = [(6, 55, 146504), (5, 135, 106147), (8, 53, 228562), (6, 46, 40790), (6, 661, 8165), (8, 34, 57011), (7, 112, 89969)]
    for group, instances, n in batches:
        sixteen = R.sixteen_lane_kernel(group, instances, n, 256)
        assert (bench.score_kernel_name(group, instances, n, 256, True, False, True, False) == "score_mfma_kernel") == sixteen, (group, instances, n)
