"""The host runtime's behaviour around failures and limits, against a HIP
runtime made of host memory (fake_hip.cpp): no GPU needed."""
import fake_hip


def test_failed_source_staging_leaves_the_handle_usable():
    """A combined solve whose staging of source parameters cannot be
    allocated reports that, and the handle's other solves go on as before;
    so does the combined one once there is memory again."""
    fake_hip.run('''
h = problem((9, 10, 11), 4, G=3)
assert solve(h)[0] == dsn.DSN_OK
fake.fake_host_limit(10000)
assert solve(h, n_src=200, combine=True)[0] == dsn.DSN_ERR_OUT_OF_MEMORY
assert solve(h)[0] == dsn.DSN_OK, dsn.last_error()
assert solve(h, n_src=3, combine=True)[0] == dsn.DSN_OK, dsn.last_error()
fake.fake_host_limit(1 << 40)
assert solve(h, n_src=200, combine=True)[0] == dsn.DSN_OK, dsn.last_error()
h.close()
''')
