"""GPU parity of replays of four wavefronts with the CPU oracle.  Launches of up to 512 replays (768 with up to 12 replicas) have
six per replay and launches of up to 1,024 on up to 32 replicas eight per two, so the other tests' few replays nearly all run
those; here the same tests run with their replays repeated in launches of more than 1,024, which have four, and what one of
the repetitions gives is compared."""
import pytest

from tests import test_gpu_engine, test_gpu_fuzz, test_gpu_launch_edges, test_gpu_online, test_gpu_parity, test_gpu_policies, test_gpu_proxy
from tests.gpu_helpers import four_wavefronts

pytestmark = pytest.mark.gpu

ANY = ("least-request", "session-affinity", "random")
CASES = (
    [(test_gpu_fuzz.test_random_cases, (seed,)) for seed in range(36) if seed % 3 != 2] +
    [(test_gpu_engine.test_random_cases, (seed,)) for seed in range(0, 24, 2)] +
    [(test_gpu_proxy.test_random_cases, (seed,)) for seed in range(0, 24, 2)] +
    [(test_gpu_engine.test_slot_counts, (B,)) for B in (1, 8, 9, 64)] +
    [(test_gpu_engine.test_saturated_and_idle_replicas, x) for x in ((None, 0.25), (1.0, 1.0))] +
    [(test_gpu_engine.test_baseline_policies_under_the_engine_model, (policy,)) for policy in ANY] +
    [(test_gpu_engine.test_zero_rates_zero_outputs_and_simultaneous_arrivals, ()),
     (test_gpu_engine.test_online_tuner_under_the_engine_model, ()),
     (test_gpu_online.test_all_weights_tuned_and_wide_range, ()),
     (test_gpu_parity.test_hand_traces, ("hand_trace_D.json",)),
     (test_gpu_parity.test_time_scales_in_one_launch, ()),
     (test_gpu_parity.test_many_segments_per_request, ()),
     (test_gpu_parity.test_requests_with_more_segments_than_a_staged_batch_holds, ()),
     (test_gpu_policies.test_policies_at_the_replica_and_slot_limits, ()),
     (test_gpu_proxy.test_epoch_boundaries_and_time_scales, ()),
     (test_gpu_proxy.test_long_paths_and_an_index_of_its_own, ())] +
    [(test_gpu_online.test_window_and_hop_shapes, x) for x in ((1, 1, 300), (4, 2, 301), (100, 7, 777))] +
    [(test_gpu_policies.test_policies_with_bounded_caches, (policy,)) for policy in ANY] +
    [(test_gpu_proxy.test_workloads, (2, 3000, index)) for index in ("none", "unbounded", "double", "tight")] +
    [(test_gpu_proxy.test_completion_events_that_overtake_each_other, (B,)) for B in (1, 3)] +
    [(test_gpu_launch_edges.test_look_ahead_either_way, x) for x in ((15, 300), (24, 300), (64, 1500))] +
    [(test_gpu_launch_edges.test_sets_of_service_slots, x) for x in ((1, 1), (13, 5), (39, 10), (64, 16))] +
    [(test_gpu_launch_edges.test_requests_that_are_waited_for, x) for x in ((0, 0.0), (40, 0.3), (4000, 4.0))])


@pytest.mark.parametrize("case", CASES, ids=lambda case: "-".join([case[0].__module__[15:], case[0].__name__[5:], *map(str, case[1])]))
def test_four_wavefronts(case):
    test, args = case
    with four_wavefronts():
        test(*args)
