/* Device queries that answer what the test sets (loaded before the HIP
 * runtime): stub_device is the current device, -1 none, and stub_units its
 * compute units, each holding one block. */
int stub_device = -1, stub_units = 0;
int hipGetDevice(int* dev) {
    *dev = stub_device;
    return stub_device < 0 ? 100 : 0; /* hipErrorNoDevice */
}
int hipDeviceGetAttribute(int* value, int what, int dev) {
    (void)what;
    *value = dev == stub_device ? stub_units : 0;
    return 0;
}
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* blocks, const void* f, int threads, unsigned long lds) {
    (void)f, (void)threads, (void)lds;
    *blocks = 1;
    return 0;
}
