"""Batches at head dimension 64 that reach the launch geometries of the scoring passes one by one.  The CPU
test checks that each batch does get its geometry, the GPU tests run the same batches against the oracle."""

# name: (batch, (keys per work-group, head split) of pass 1, the same of pass 2)
HEAD_64 = {
    # more than one round of 512-key work-groups: pass 2 takes 256 keys; parts added by k_finish
    "split_many_rounds": (dict(lengths=[7001, 1, 10241, 300], num_q_heads=8, num_kv_heads=8, n_obs=96), (512, 8), (256, 8)),
    # the same with every head in one work-group: the sweep itself selects
    "whole_many_rounds": (dict(lengths=[513, 512, 511, 257, 256, 255, 1, 0] + [300, 700] * 125, num_q_heads=8,
                               num_kv_heads=2, n_obs=96), (512, 1), (256, 1)),
    # one full round of split work-groups: pass 2 keeps 512 keys
    "split_one_round": (dict(lengths=[14721], num_q_heads=8, num_kv_heads=8, n_obs=96), (512, 8), (512, 8)),
    # one round, heads not split: 512 keys with eight staging units a head, 256 with fewer
    "whole_one_round_long_window": (dict(lengths=[60001, 56001], num_q_heads=2, num_kv_heads=1, n_obs=512), (512, 1), (512, 1)),
    "whole_one_round": (dict(lengths=[60001, 56001], num_q_heads=2, num_kv_heads=1, n_obs=96), (512, 1), (256, 1)),
    # one round of slots, many of them blocks of short sequences that are kept whole
    "one_round_short_sequences": (dict(lengths=[1] * 20 + [5000], num_q_heads=8, num_kv_heads=8, n_obs=96), (512, 8), (256, 8)),
    # too few key blocks for 512 keys in either pass
    "few_blocks": (dict(lengths=[512 * 12 + 1], num_q_heads=8, num_kv_heads=2, n_obs=96), (256, 2), (256, 2)),
    # after earlier context pass 2 has a geometry of its own
    "context": (dict(lengths=[8192, 7000], earlier=[700, 5000], num_q_heads=8, num_kv_heads=8, n_obs=96), (512, 8), (512, 8)),
}
