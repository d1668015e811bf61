/* Stands in for the runtime's function that begins every kernel launch, so that a test can tell on a machine without a GPU whether a
 * call launched anything.  A result other than zero skips the launch. */
int launches = 0;
int __hipPushCallConfiguration(void)
{
    ++launches;
    return 1;
}
