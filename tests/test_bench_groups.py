"""Profiles group a kernel as the library's own timers do."""

import bench


def test_kernel_groups():
    ns = "void lbvh::(anonymous namespace)::"
    for name, group in [("k_onesweep<unsigned int, 1024, 8, 8, true>(unsigned int const*", "query_order"),
                        ("k_onesweep<unsigned int, 512, 4, 8, true>", "query_order"),
                        ("k_onesweep<unsigned int, 1024, 8, 8, false>", "sort_pass"),
                        ("k_onesweep<unsigned long, 1024, 16, 8, false>", "sort_pass"),
                        ("k_bottomup_l0<1, unsigned int, true>", "bottomup"),
                        ("k_qorder_keys<lbvh::(anonymous namespace)::QBox>", "query_order"),
                        ("k_query_reset", "query_split"), ("k_cut<lbvh::(anonymous namespace)::QBox>", "query_split"),
                        ("k_walk<lbvh::(anonymous namespace)::QBox>", "query_count"),
                        ("k_task_count<lbvh::(anonymous namespace)::Ray>", "query_count"),
                        ("k_task_places", "scan"), ("k_scan", "scan"),
                        ("k_fill_light<lbvh::(anonymous namespace)::Sphere>", "query_fill"),
                        ("k_fill_tasks<lbvh::(anonymous namespace)::Sphere>", "query_fill"),
                        ("k_scene_sort<0, unsigned long, 9, 512, 8>", "scene_sort"),
                        ("k_ray_first", "ray_first")]:
        assert bench._group(ns + name) == group, name
